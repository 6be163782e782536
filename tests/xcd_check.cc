// The placement of work-groups on XCDs, and the work of launches that leave one alone (csrc/xcd_map.h).
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

// every unit once, whatever the number of units and the place left out
static void check_spare() {
    for (int hole = -1; hole < 8; ++hole)
        for (long long units = 0; units <= 300; ++units) {
            std::vector<int> done(units, 0);
            const long long grid = spare_grid(units, hole);
            REQUIRE(hole < 0 || grid % 8 == 0);
            for (long long b = 0; b < grid; ++b) {
                const long long u = spare_unit((unsigned)b, hole);
                REQUIRE(u >= -1 && (u >= 0 || (int)(b & 7) == hole));
                if (u >= 0 && u < units) ++done[u];
            }
            for (int d : done) REQUIRE(d == 1);
        }
}

// every part of every range once, the parts of a range on one XCD
static void check_ranges() {
    for (int hole = -1; hole < 8; ++hole)
        for (int count = 1; count <= 5; ++count)
            for (int ranges = 1; ranges <= 230; ranges += ranges < 20 ? 1 : 7) {
                std::vector<int> done(ranges * count, 0), place(ranges, -1);
                const long long grid = spare_grid(range_units(ranges, count, hole), hole);
                for (long long b = 0; b < grid; ++b) {
                    const long long u = spare_unit((unsigned)b, hole);
                    if (u < 0) continue;
                    const RangeUnit r = range_unit((int)u, count, hole);
                    REQUIRE(r.range >= 0 && r.part >= 0 && r.part < count);
                    if (r.range >= ranges) continue;
                    ++done[r.range * count + r.part];
                    REQUIRE(place[r.range] < 0 || place[r.range] == (int)(b & 7));
                    place[r.range] = (int)(b & 7);
                }
                for (int d : done) REQUIRE(d == 1);
            }
}

int main() {
    check_map();
    check_spare();
    check_ranges();
    if (!failures) printf("xcd_check ok\n");
    return failures ? 1 : 0;
}
