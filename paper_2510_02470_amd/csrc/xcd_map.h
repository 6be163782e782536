// Which XCD the work-groups of a launch run on. Plain integer functions, so that they can be checked without a GPU
// (tests/xcd_check.cc).
#pragma once

namespace sage {

// Work-groups i and i + period of a launch run on the same XCD and `period` consecutive ones on different XCDs, those of
// `id`. 8 on the whole chip, the number of XCDs of a partition otherwise; 0: neither can be said. Which of them the first gets
// differs from stream to stream, and for one stream when queues come and go (tried: another stream's first launch moved it
// by one). Nothing that decides a result may rest on any of this.
struct XcdMap {
    int period = 0;
    int id[8] = {};
};

// from the XCDs (0 .. 7) that the work-groups 0 .. count - 1 of one launch ran on
inline XcdMap xcd_map_of(const int* on, int count) {
    for (int p = 1; p <= 8; p *= 2) {
        unsigned seen = 0;
        XcdMap m;
        bool ok = count >= 2 * p;
        for (int i = 0; ok && i < count; ++i) {
            if (i < p) {
                ok = on[i] >= 0 && on[i] < 8 && !(seen >> on[i] & 1);
                if (ok) seen |= 1u << on[i];
                m.id[i] = on[i];
            } else {
                ok = on[i] == on[i - p];
            }
        }
        m.period = p;
        if (ok) return m;
    }
    return XcdMap{};
}

// A launch that leaves one XCD alone: of eight work-groups the one at place `hole` has nothing to do and the others share
// the units of work between them, in order. -1: all eight work. (Which work-groups these are is a matter of their numbers
// only, so all units are done wherever they run.)
constexpr long long spare_unit(unsigned block, int hole) {
    if (hole < 0) return block;
    const int place = (int)(block & 7u);
    return place == hole ? -1 : (long long)(block >> 3) * 7 + place - (place > hole);
}
constexpr long long spare_grid(long long units, int hole) { return hole < 0 ? units : (units + 6) / 7 * 8; }  // work-groups


// Units that read a range in common, `count` to a range: of such a launch they are neighbours on one XCD, whose L2 they share.
struct RangeUnit {
    int range, part;
};
constexpr int range_stride(int hole) { return hole < 0 ? 8 : 7; }  // units that are this far apart
constexpr RangeUnit range_unit(int unit, int count, int hole) {
    const int w = range_stride(hole);
    return RangeUnit{unit / (w * count) * w + unit % w, unit / w % count};
}
constexpr int range_units(int ranges, int count, int hole) {  // (those of ranges beyond the last have nothing to do)
    const int w = range_stride(hole);
    return (ranges + w - 1) / w * w * count;
}

}  // namespace sage
