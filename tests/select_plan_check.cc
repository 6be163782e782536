// The work space of the top-m selection (csrc/select_plan.h): large enough for every call up to the size it was made for, and not
// larger than its longest call needs. Argument "planted": as many blocks as a call of the largest size uses, which must fail.
#include <cstdio>
#include <cstring>
#include <initializer_list>

#include "select_plan.h"

using namespace sage;

static bool planted = false;
static int failures = 0;

static void check(int64_t cap, int64_t N) {
    const int64_t blocks = planted ? topm_blocks(cap) : topm_work_blocks(cap);
    const int64_t keys = topm_long(N) ? SELECT_LONG : SELECT_BLOCK;
    if (topm_blocks(N) * keys < N || topm_blocks(N) > blocks) {
        if (++failures <= 5) printf("%lld keys, work space for %lld: %lld blocks of %lld\n", (long long)N, (long long)cap,
                                    (long long)topm_blocks(N), (long long)blocks);
    }
}

int main(int argc, char** argv) {
    planted = argc > 1 && !strcmp(argv[1], "planted");
    const int64_t edge = SELECT_SHORT_MAX * SELECT_BLOCK, top = 16777216;  // the largest call of sage_topm_static
    for (int64_t cap : {(int64_t)1, (int64_t)32769, edge - 1, edge, edge + 1, (int64_t)5000003, top - 1, top, top + 1, 10 * top}) {
        for (int64_t N : {(int64_t)1, (int64_t)4096, (int64_t)4097, (int64_t)32769, edge - 4096, edge - 1, edge, edge + 1,
                          edge + 16384, top - 16384, top - 1, top, top + 1, 10 * top})
            if (N <= cap) check(cap, N);
        for (int64_t N = cap; N > 0; N -= 1 + cap / 1000) check(cap, N);
        // no table that no call uses
        const int64_t most = cap > edge ? (cap / SELECT_LONG + 1 > SELECT_SHORT_MAX ? cap / SELECT_LONG + 1 : SELECT_SHORT_MAX)
                                        : (cap + SELECT_BLOCK - 1) / SELECT_BLOCK;
        if (topm_work_blocks(cap) > most) ++failures;
    }
    if (topm_work_words(topm_work_blocks(top)) * 4 > 2200000) ++failures;
    if (failures) printf("%d failures\n", failures);
    else printf("select_plan_check ok\n");
    return failures ? 1 : 0;
}
