// A simulated stream for StageGraphs: launches run one per tick of the fake clock, in order.
// Input: the number of stages and, per stage, its launches and the ticks that pass before the
// next one.  Output: graphs destroyed while a launch of theirs had yet to run (must be 0), the most
// graphs alive at once, those alive at the end, and ticks the host waited.
#include <algorithm>
#include <cstdio>

#include "mfwf.h"
#include "stage_graphs.h"

static long issued = 0, ran = 0, alive = 0, most = 0, early = 0, waited = 0;
static bool ended = false;  // the solve is over: the graphs that are left wait for themselves

struct SimGraph {
    long last = 0, at = -1;  // launches issued up to its last one; at its mark
    SimGraph() { most = std::max(most, ++alive); }
    ~SimGraph() {
        if (ended) wait_for(at < 0 ? issued : at);  // as the device graph
        early += ran < last;
        alive--;
    }
    void launch(long n) { last = issued += n; }
    static void wait_for(long n) {
        waited += std::max(0L, n - ran);
        ran = std::max(ran, n);
    }
    int mark() { return at = issued, MFWF_OK; }
    int passed(bool &yes) { return yes = ran >= at, MFWF_OK; }
    int wait() { return wait_for(at), MFWF_OK; }
};

int main() {
    int stages;
    if (std::scanf("%d", &stages) != 1) return 1;
    {
        mfwf::StageGraphs<SimGraph> graphs;
        for (int s = 0; s < stages; s++) {
            long launches, ticks;
            if (std::scanf("%ld %ld", &launches, &ticks) != 2) return 1;
            SimGraph *g = nullptr;
            if (graphs.next(g) != MFWF_OK) return 2;
            g->launch(launches);
            ran = std::min(issued, ran + ticks);
        }
        ended = true;
    }
    std::printf("%ld %ld %ld %ld\n", early, most, alive, waited);
    return 0;
}
