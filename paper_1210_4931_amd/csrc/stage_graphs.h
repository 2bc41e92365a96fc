// The captured iterations of a solve's stages, free of any device call.  A stage's launches read
// its executable graph while they run, which is after the host has gone on to the next stage, so
// a graph is kept until its last launch has run; and a schedule of many stages holds kKeep
// graphs at a time, not one per stage.
//
// G, one captured iteration, provides the status codes of mfwf.h from
//   int mark();               a point on the stream after the launches made so far
//   int passed(bool &yes);    whether the stream has passed the mark
//   int wait();               until it has
// and its destructor waits for its stream (a solve that ends early leaves through it).
#pragma once

#include <cstddef>
#include <deque>
#include <memory>

namespace mfwf {

template <typename G, size_t kKeep = 4>
class StageGraphs {
public:
    // a graph for the next stage; the stage before it makes no further launches
    int next(G *&out) {
        if (!kept.empty()) {
            if (int st = kept.back()->mark()) return st;
        }
        while (!kept.empty()) {  // the oldest first: the stream runs them in order
            bool yes = false;
            if (kept.size() >= kKeep) {
                if (int st = kept.front()->wait()) return st;
                yes = true;
            } else if (int st = kept.front()->passed(yes)) {
                return st;
            }
            if (!yes) break;
            kept.pop_front();
        }
        kept.push_back(std::make_unique<G>());
        out = kept.back().get();
        return 0;
    }

private:
    std::deque<std::unique_ptr<G>> kept;
};

}  // namespace mfwf
