// The exchange of a reduction that ends after n - 64 steps (csrc/fd_tri_plan.h, steps_until and waits_until), for every number of rows:
// what a work-group stores at the end it has all entries for, and a slot is emptied when everyone who waits for what it held has
// read it, and before anyone can publish or wait for its next entries.
// Argument "planted": the same with nobody waiting for the last step, which must fail.
#include <cstdio>
#include <cstring>
#include <vector>

#include "fd_tri_plan.h"

using sage::TriPlan;

static bool planted = false;
static int failures = 0;
#define REQUIRE(cond, what)                                                     \
    do {                                                                        \
        if (!(cond) && ++failures <= 5) printf("J = %d, n = %d, step %d: %s\n", J, n, k, what); \
    } while (0)

template <int J>
void check(int n) {
    using P = TriPlan<J>;
    constexpr int G = P::NWG;
    const int last = n - 64;
    int closing = -1, k = -1;
    std::vector<int> steps(G), waits(G);
    for (int g = 0; g < G; ++g) {
        if (P::closes(g, n)) closing = g;
        steps[g] = P::last_column(g, n) < 0 ? 0 : P::steps_until(g, n, last);
        waits[g] = P::last_column(g, n) < 0 ? 0 : P::waits_until(g, n, last);
        if (planted && waits[g] == last) waits[g] = last - 1;
        REQUIRE(waits[g] >= steps[g] - 1 && steps[g] <= last && waits[g] <= last, "more steps than there are");
        // the update of step last - 1 is in every column that is left
        REQUIRE(P::last_column(g, n) < last || (steps[g] == last && waits[g] == last), "a column left without its last update");
    }
    REQUIRE(closing >= 0 && steps[closing] == last && waits[closing] == last, "the closing work-group does not see every step");
    auto publishes = [&](int g, int s) { return s < steps[g] && P::last_column(g, n) > s; };
    std::vector<int> read(G * G, 0), next;  // read[a][b]: steps that b is certain to have read when a has read all of the steps so far
    for (k = 0; k < last; ++k) {
        for (int b = 0; b < G && k >= 2; ++b)
            REQUIRE(b == closing || waits[b] <= k - 2 || read[closing * G + b] > k - 2, "emptied before everyone has read it");
        for (int g = 0; g < G; ++g)
            if (k + 2 < last && (publishes(g, k + 2) || waits[g] > k + 2))
                REQUIRE(waits[g] > k + 1 && publishes(closing, k + 1), "used before it is empty");
        next = read;
        for (int a = 0; a < G; ++a)
            if (k < waits[a])
                for (int p = 0; p < G; ++p)
                    if (publishes(p, k))
                        for (int b = 0; b < G; ++b) {
                            const int v = b == p ? (k < waits[p] ? k : waits[p]) : read[p * G + b];
                            if (v > next[a * G + b]) next[a * G + b] = v;
                        }
        read.swap(next);
    }
}

int main(int argc, char** argv) {
    planted = argc > 1 && !strcmp(argv[1], "planted");
    for (int n = 65; n <= 128; ++n) check<2>(n);
    for (int n = 65; n <= 256; n += n < 140 ? 1 : 3) check<4>(n);
    for (int n = 65; n <= 512; n += n < 140 ? 1 : 9) check<8>(n);
    check<4>(256);
    check<8>(512);
    if (failures) printf("%d failures\n", failures);
    else printf("tri_tail_check ok\n");
    return failures ? 1 : 0;
}
