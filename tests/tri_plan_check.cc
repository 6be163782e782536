// The exchange protocol of the reduction by several work-groups (csrc/fd_tri_plan.h), for every number of rows: whatever the
// delays, no entry is overwritten before everyone who waits for it has read it, everyone's entries are published, and one
// work-group gets to the end and stores the results. Argument "planted": the same checks on a protocol in which every work-group stays
// to the end, which must fail.
#include <cstdio>
#include <cstring>
#include <vector>

#include "fd_tri_plan.h"

using sage::TriPlan;

static bool planted = false;
static int failures = 0;
#define REQUIRE(cond, ...)                            \
    do {                                              \
        if (!(cond) && ++failures <= 5) {             \
            printf("J = %d, n = %d: ", J, n);         \
            printf(__VA_ARGS__);                      \
            printf("\n");                             \
        }                                             \
    } while (0)

template <int J>
void check(int n) {
    using P = TriPlan<J>;
    constexpr int G = P::NWG;
    int steps[G], waits[G];
    for (int g = 0; g < G; ++g) {
        steps[g] = planted ? n - 1 : P::steps(g, n);
        waits[g] = planted ? n - 1 : P::waits(g, n);
        REQUIRE(waits[g] <= steps[g] && steps[g] <= n - 1, "work-group %d: %d waits, %d steps", g, waits[g], steps[g]);
    }
    // columns: owned by the waves as the kernel counts them
    std::vector<int> group(n, -1);
    for (int w = 0; w < P::NW; ++w)
        for (int s = 0; s < P::CW; ++s) {
            const int c = P::column(w, s);
            if (c >= n) continue;
            REQUIRE(group[c] < 0 && P::wave_of(c) == w, "column %d", c);
            group[c] = w / 4;
        }
    for (int c = 0; c < n; ++c) REQUIRE(group[c] >= 0, "column %d has no owner", c);
    auto publishes = [&](int g, int k) {  // q at a row above k, or column k + 1
        if (k >= steps[g]) return false;
        return P::last_column(g, n) > k;
    };
    // known[a][b]: steps that b is certain to have read when a has read all it waits for so far
    std::vector<int> known(G * G, 0), next(G * G);
    for (int k = 0; k < n - 1; ++k) {
        for (int c = k + 1; c < n; ++c)
            REQUIRE(k < steps[group[c]], "step %d: nobody publishes q[%d]", k, c);
        // entries of step k go over those of step k - 2
        for (int a = 0; a < G && k >= 2; ++a)
            for (int b = 0; b < G && publishes(a, k); ++b)
                REQUIRE(b == a || waits[b] < k - 1 || known[a * G + b] >= k - 1,
                        "work-group %d overwrites step %d, which work-group %d may not have read", a, k - 2, b);
        // whoever waits for step k has what all its publishers knew, and their own reading of the steps before it
        std::vector<int> all(G, 0);
        for (int a = 0; a < G; ++a)
            if (publishes(a, k))
                for (int b = 0; b < G; ++b) {
                    const int v = b == a ? (k < waits[a] ? k : waits[a]) : known[a * G + b];
                    all[b] = v > all[b] ? v : all[b];
                }
        next = known;
        for (int a = 0; a < G; ++a)
            if (k < waits[a])
                for (int b = 0; b < G; ++b) next[a * G + b] = all[b] > known[a * G + b] ? all[b] : known[a * G + b];
        known.swap(next);
    }
    int closing = 0;  // stores every reflector and the last diagonal element: one work-group, which has all of every step
    for (int g = 0; g < G; ++g)
        if (P::closes(g, n) && ++closing) REQUIRE(steps[g] == n - 1 && waits[g] == n - 1, "work-group %d stores the results", g);
    REQUIRE(closing == 1, "%d work-groups store the results", closing);
}

// the work-groups of the closing role in every order of being on the XCD or not: one of them has the results to store
static void check_claims() {
    constexpr int J = 0;
    for (int period = 1, n = 0; period <= 8; period *= 2)
        for (unsigned on = 0; on < 1u << period; ++on) {
            unsigned word = 0;
            int closing = 0, alone = 0, last = 0;
            for (int i = 0; i < period; ++i) {
                const bool here = on >> i & 1u;
                word += sage::claim_add(here);
                const sage::TriClaim r = sage::claim_role(word, here, period);
                closing += r == sage::CLAIM_CLOSE;
                alone += r == sage::CLAIM_ALONE;
                last += sage::claim_last(word, period);
                REQUIRE(r != sage::CLAIM_CLOSE || here, "a work-group elsewhere closes");
                REQUIRE(!sage::claim_last(word, period) || i == period - 1, "the word is cleared early");
            }
            REQUIRE(closing == (on != 0) && alone == (on == 0) && last == 1, "period %d, pattern %x", period, on);
        }
}

int main(int argc, char** argv) {
    planted = argc > 1 && !strcmp(argv[1], "planted");
    for (int n = 1; n <= 128; ++n) check<2>(n);
    for (int n = 1; n <= 256; ++n) check<4>(n);
    for (int n = 1; n <= 512; ++n) check<8>(n);
    check_claims();
    if (failures) printf("%d failures\n", failures);
    else printf("tri_plan_check ok\n");
    return failures ? 1 : 0;
}
