// Kept work space of the top-m selection (csrc/topm_kept.h): runs of several launches, eager, captured and replayed, with launches that are
// refused, in any order. No kernel may add to a histogram that is not zero. What each kernel clears is that of csrc/select.hip.
// Arguments: "enqueued", with an eager run's clearing taken for done when it is only captured; "bare", with captured runs that rely on the
// eager ones. Both must fail.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "topm_kept.h"

using sage::KeptHistograms;

static int failures = 0;

struct Device {
    bool dirty[3] = {false, false, false};
    void add(int h, const char* who) {
        if (dirty[h] && ++failures <= 5) printf("%s: histogram %d is not zero\n", who, h);
        dirty[h] = true;
    }
    // launches of a run from the clearing one (0) or the first histogram (1) up to, not including, `end`
    void run(bool clears, int end, const char* who) {
        for (int launch = clears ? 0 : 1; launch < end; ++launch) switch (launch) {
            case 0: dirty[0] = dirty[1] = dirty[2] = false; break;
            case 1: dirty[2] = false; add(0, who); break;
            case 2: add(1, who); break;
            case 3: dirty[0] = false; add(2, who); break;
            case 4: dirty[1] = false; break;
        }
    }
};

int main(int argc, char** argv) {
    const bool enqueued = argc > 1 && !strcmp(argv[1], "enqueued"), bare = argc > 1 && !strcmp(argv[1], "bare");
    srand(1);
    int cleared = 0, eager_runs = 0;
    for (int trial = 0; trial < 20000; ++trial) {
        Device d;
        KeptHistograms kept;
        std::vector<bool> graphs;  // does it clear
        for (int calls = 12; calls > 0; --calls) {
            const int what = rand() % 10;
            if (what < 4) {  // an eager call
                const bool clears = kept.clear_first(true);
                d.run(clears, 5, "eager");
                ++eager_runs;
                cleared += clears;
            } else if (what < 6) {  // one that is refused from some launch on
                const bool clears = kept.clear_first(true);
                const int first = clears ? 0 : 1;
                d.run(clears, first + rand() % (5 - first), "refused");
                kept.refused();
            } else if (what < 8) {  // one that is captured
                graphs.push_back(bare ? kept.cut_short.load() : kept.clear_first(enqueued ? kept.cut_short.load() : false));
                if (rand() % 4 == 0) {  // ... or not
                    graphs.pop_back();
                    kept.refused();
                }
            } else if (!graphs.empty()) {
                d.run(graphs[rand() % graphs.size()], 5, "replay");
            }
        }
    }
    if (cleared == eager_runs || cleared == 0) ++failures, printf("eager runs always or never clear\n");
    if (failures) printf("%d failures\n", failures);
    else printf("topm_kept_check ok\n");
    return failures ? 1 : 0;
}
