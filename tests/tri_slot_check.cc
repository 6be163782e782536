// The slots of the exchange of the reduction by several work-groups (csrc/fd_tri_plan.h), for every number of rows: a slot is
// emptied when everyone who waits for what it held has read it, and before anyone can publish or wait for its next entries.
// Argument "planted": the same checks with the slot of the step before emptied, which must fail.
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
    int closing = -1;
    for (int g = 0; g < G; ++g)
        if (P::closes(g, n)) closing = g;
    int k = -1;
    REQUIRE(closing >= 0, "no work-group closes");
    auto publishes = [&](int g, int s) { return s < P::steps(g, n) && P::last_column(g, n) > s; };
    // read[a][b]: steps that b is certain to have read when a has read all of the steps so far
    std::vector<int> read(G * G, 0), next;
    const int back = planted ? 1 : 2;  // step k empties the slot of step k + 2, that is of step k - back
    for (k = 0; k < n - 1; ++k) {
        if (!planted) REQUIRE(k < 2 || P::slot(k + 2) == P::slot(k - 2), "the slot is another step's");
        REQUIRE(P::slot(k + 2) != P::slot(k) && P::slot(k + 2) != P::slot(k + 1) && P::slot(k + 2) != P::slot(k + 3),
                "the slot is in use");
        for (int b = 0; b < G && k >= back; ++b)
            REQUIRE(b == closing || P::waits(b, n) <= k - back || read[closing * G + b] > k - back,
                    "emptied before everyone has read it");
        // who publishes or waits in step k + 2 has read the closing work-group's entry of step k + 1
        for (int g = 0; g < G; ++g)
            if (k + 2 < n - 1 && (publishes(g, k + 2) || P::waits(g, n) > k + 2))
                REQUIRE(P::waits(g, n) > k + 1 && publishes(closing, k + 1), "used before it is empty");
        next = read;
        for (int a = 0; a < G; ++a)
            if (k < P::waits(a, n))
                for (int p = 0; p < G; ++p)
                    if (publishes(p, k))
                        for (int b = 0; b < G; ++b) {
                            const int v = b == p ? (k < P::waits(p, n) ? k : P::waits(p, n)) : read[p * G + b];
                            if (v > next[a * G + b]) next[a * G + b] = v;
                        }
        read.swap(next);
    }
}

int main(int argc, char** argv) {
    planted = argc > 1 && !strcmp(argv[1], "planted");
    for (int n = 1; n <= 128; ++n) check<2>(n);
    for (int n = 1; n <= 256; n += n < 70 ? 1 : 3) check<4>(n);
    for (int n = 1; n <= 512; n += n < 70 ? 1 : 9) check<8>(n);
    check<4>(256);
    check<8>(512);
    if (failures) printf("%d failures\n", failures);
    else printf("tri_slot_check ok\n");
    return failures ? 1 : 0;
}
