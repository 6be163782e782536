// Which halves of the ring of new rows hold what, which shrinks leave their rows unwritten, and which buffers their coefficients go
// through (fd_defer.hip). Plain integer functions, so that they can be checked without a GPU (tests/defer_check.cc).
#pragma once
#include <stdint.h>

namespace sage {

struct DeferPlan {
    // of the context
    int max = 0;          // blocks whose shrink is deferred, at most (0: every shrink writes its rows at once)
    bool beside = false;  // their rows are written, and the next block's products formed, beside the next eigensolve
    // The halves: cur holds the current rows, `next` those that are stored ahead, `spare` takes turns with cur while nothing is
    // deferred (so that two cycles in a captured graph end where they began); `count` blocks, block b in half slots >> 4 b & 15.
    int cur = 0, next = 1, spare = 1, count = 0;
    unsigned slots = 0;
    int group = 0;  // not beside: shrinks that are put together this time
    // A call was captured: a graph holds the halves cur and spare by their addresses, and replays of it may stand between other
    // calls. So those two alone take turns from then on (no shrink is deferred): calls of an even number of cycles end where they began.
    bool captured = false;
    // The coefficients: a shrink whose rows are not written by itself leaves M in buffer m; after it the rows of the `count` deferred
    // ones are W [top; blocks], W in buffer w (MS, MS + 1: its own two) once M is folded into it. With one block W is M, without a copy, so
    // the next fold, on the side stream, reads the last two M's while the eigensolve beside it writes the one after: three in turn.
    int MS = 3;
    int m = 0, w = 0;
    bool folded = true;

    static int halves_of(int max) { return max > 1 ? max + 1 : 2; }
    int halves() const { return halves_of(max); }
    // The next smaller plan, where memory is short: of four blocks put together two remain, otherwise every shrink writes its rows at once.
    int fewer() const { return !beside && max > 2 ? 2 : 0; }
    // Between calls: the current rows are in the first of the halves that remain (which is all that 64 buffer rows need).
    void give_up() {
        max = fewer();
        cur = 0;
        next = spare = 1;
    }
    int free_half() const {
        if (count == 0 && spare != cur) return spare;
        unsigned used = 1u << cur;
        for (int b = 0; b < count; ++b) used |= 1u << (slots >> (4 * b) & 15u);
        return __builtin_ctz(~used);
    }

    struct Step {
        bool defer;        // this shrink's rows are not written at once
        bool write_first;  // there is room for no more blocks: the rows of those that are there come first
        bool last;         // the rows are written right after it: the call ends on the next block, or the group is whole
    };
    // The shrink of the full half cur. next_rows: rows of the running call after it; ahead: the next ell of them are stored ahead;
    // allowed: the block and the next one can be deferred. An update call never ends with blocks.
    Step step(bool ahead, bool allowed, int64_t next_rows, int ell) {
        Step s{ahead && allowed && !captured && max > 0, count > 0 && count == max, false};
        if (s.defer && !beside && count == 0) {
            // the shrinks left in this call, this one included, in equal groups
            const int64_t left = next_rows / ell + (next_rows % ell ? 1 : 0), groups = (left + max - 1) / max;
            group = (int)((left + groups - 1) / groups);
            s.defer = group > 1;
        }
        s.last = s.defer && (next_rows == ell || (!beside && count + 1 == group));
        return s;
    }
    unsigned slots_with_cur() const { return slots | (unsigned)cur << (4 * count); }
    void push() {
        slots = slots_with_cur();
        count += 1;
    }
    void written() {
        slots = 0;
        count = 0;
    }
    int next_m() const { return m + 1 < MS ? m + 1 : 0; }  // where the running shrink's M goes
    void made_m() {
        m = next_m();
        folded = false;
    }
    struct Fold {
        int from, out;  // out <- [M_top from, M_new]; out < 0: W is M itself, nothing to do
    };
    Fold fold() {
        folded = true;
        const int from = w;
        w = count == 1 ? m : from == MS ? MS + 1 : MS;
        return Fold{from, count == 1 ? -1 : w};
    }
    void advance(bool ahead) {
        const int old = cur;
        cur = ahead ? next : free_half();
        if (count == 0) spare = old;
    }
};

}  // namespace sage
