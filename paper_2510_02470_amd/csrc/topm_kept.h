// Whether the first two histograms of kept work space (topm_static.hip) are zero when a run of several launches begins. Every such run
// leaves them so, unless one of its launches was refused. Host state, so it knows of eager runs only: what a graph holds runs later,
// any number of times or never. So a captured run brings its own clearing launch and says nothing about the work space (2 us of 20 for a
// million scores, which only eager runs save). Checked without a GPU (tests/topm_kept_check.cc).
#pragma once
#include <atomic>

namespace sage {

struct KeptHistograms {
    std::atomic<bool> cut_short{false};  // a launch was refused, and no eager run has cleared since
    // An eager run, or one that is captured or may be, is about to be enqueued: does it begin with the clearing launch?
    bool clear_first(bool eager) { return !eager || cut_short.exchange(false); }
    // One of its launches was refused.
    void refused() { cut_short.store(true); }
};

}  // namespace sage
