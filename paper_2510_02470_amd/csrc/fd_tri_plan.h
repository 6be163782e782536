// Who does what in a reduction by several work-groups (tri_many_kernel). Plain integer functions, so that the protocol can be
// checked without a GPU (tests/tri_plan_check.cc).
//
// Step k of the reduction of n rows exchanges q and c at the rows above k: entry q[i] comes from the wave that owns column i,
// all of c from the one that owns column k + 1. So a work-group has something to publish in the steps below its last column,
// and it needs the entries of a step only to make those of the next. It leaves after its last entry; one without a column
// below n has no part in the solve.
//
// An entry is the value itself, 8 bytes; a slot that holds no entry yet holds a pattern no result has (EMPTY, all ones). Step k uses
// slot k & 3. The work-group of the last column, which takes part in every step, empties slot (k + 2) & 3 in step k, before
// its barrier of that step: it has all of step k - 1 then, to which every reader of step k - 2 that is not done contributed
// after it had read step k - 2. Who publishes or waits for entries of step k + 2 has that work-group's entry of step k + 1, which
// it published after the slot was empty.
#pragma once

namespace sage {

template <int J>
struct TriPlan {
    static constexpr int N = 64 * J;
    static constexpr int CW = J >= 8 ? 4 : 2;   // columns of a wave
    static constexpr int NW = N / CW;           // waves that hold columns
    static constexpr int NWG = NW / 4;          // work-groups
    static constexpr int ST = J / CW;           // columns of a wave are 64 ST apart
    static constexpr int THREADS = 256 + N;     // of a work-group: four waves compute, a thread waits for two of 2 N entries
    static constexpr int SLOTS = 4;
    static constexpr int slot(int k) { return k & (SLOTS - 1); }

    static constexpr int column(int wave, int s) { return (wave & 63) + 64 * ((wave >> 6) + ST * s); }
    static constexpr int wave_of(int col) { return (col & 63) + 64 * ((col >> 6) & (ST - 1)); }

    // of work-group wg, among the first n columns; -1: none
    static constexpr int last_column(int wg, int n) {
        int last = -1;
        for (int s = 0; s < CW; ++s) {
            const int first = column(4 * wg, s);  // its four waves own four neighbours
            if (first < n) last = first + 3 < n ? first + 3 : n - 1;
        }
        return last;
    }
    // It takes part in steps 0 .. steps - 1 and waits for the entries of steps 0 .. waits - 1. The work-group of the last
    // column goes on to the end: it alone is left in step n - 2, reads its own entries of it, and knows the last diagonal element.
    static constexpr int steps(int wg, int n) { return last_column(wg, n) > 0 ? last_column(wg, n) : 0; }
    static constexpr int waits(int wg, int n) {
        return last_column(wg, n) == n - 1 ? n - 1 : (steps(wg, n) > 0 ? steps(wg, n) - 1 : 0);
    }
    // The same where the reduction ends after `until` steps, 0 < until < n, and leaves the columns from `until` on: whoever owns one of them
    // waits for every step.
    static constexpr int steps_until(int wg, int n, int until) { return steps(wg, n) < until ? steps(wg, n) : until; }
    static constexpr int waits_until(int wg, int n, int until) { return last_column(wg, n) >= until ? until : waits(wg, n); }
    // It also sees every step, and stores the results: nothing that a delayed work-group does can reach them.
    static constexpr bool closes(int wg, int n) { return last_column(wg, n) == n - 1; }
};

// Every role is given to `period` work-groups, of which one is expected on the XCD of the solve and the others leave. So that a
// solve has its results whatever the placement, those of the closing role add to a word that is zero before: with `here`, on the
// XCD. The first one there closes the solve; if none is, the last to come does all of it alone. The last one clears the word.
enum TriClaim { CLAIM_LEAVE, CLAIM_CLOSE, CLAIM_ALONE };
constexpr unsigned claim_add(bool here) { return here ? 0x101u : 1u; }
constexpr bool claim_last(unsigned word, int period) { return (int)(word & 0xFFu) == period; }
constexpr TriClaim claim_role(unsigned word, bool here, int period) {  // word: with one's own addition
    if (here) return (word >> 8) == 1u ? CLAIM_CLOSE : CLAIM_LEAVE;
    return claim_last(word, period) && (word >> 8) == 0u ? CLAIM_ALONE : CLAIM_LEAVE;
}

}  // namespace sage
