// The placement of work-groups on XCDs (csrc/xcd_map.h).
#include <cstdio>
#include <vector>

#include "xcd_map.h"

using namespace sage;

static int failures = 0;
#define REQUIRE(cond)                                                   \
    do {                                                                \
        if (!(cond) && ++failures) printf("line %d: %s\n", __LINE__, #cond); \
    } while (0)

static void check_map() {
    std::vector<int> on(512);
    for (int p = 1; p <= 8; p *= 2)
        for (int first = 0; first < 8; ++first) {  // any rotation, and ids that are not the first ones
            for (int i = 0; i < 512; ++i) on[i] = ((i + first) % p + (p < 8 ? first : 0)) & 7;
            const XcdMap m = xcd_map_of(on.data(), 512);
            REQUIRE(m.period == p);
            for (int i = 0; i < p; ++i) REQUIRE(m.id[i] == on[i]);
            on[300] = (on[300] + 1) & 7;  // one work-group elsewhere
            REQUIRE(xcd_map_of(on.data(), 512).period == 0);
        }
    for (int i = 0; i < 512; ++i) on[i] = i % 3;
    REQUIRE(xcd_map_of(on.data(), 512).period == 0);
    for (int i = 0; i < 512; ++i) on[i] = (i / 2) % 8;  // two neighbours on one
    REQUIRE(xcd_map_of(on.data(), 512).period == 0);
}

int main() {
    check_map();
    if (!failures) printf("xcd_check ok\n");
    return failures ? 1 : 0;
}
