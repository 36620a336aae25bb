// Which captured graphs a GNEB handle makes, and when.  Host C++ only.
#pragma once

#include <cstdint>

namespace spx {

// Iterations in the longer of the two captured graphs.  Between two graph
// launches the device waits 8 us, between two kernels of one graph not at all
// (films of 100 us an iteration).
// Capturing the long one costs about 0.6 ms, so it waits until the handle has
// been asked for kLongAfter iterations.
constexpr int kGraphIters = 8;
constexpr int kLongAfter = 128;

struct GnebGraphs {
    bool on = true;      // graphs at all; else direct launches
    bool run_on = true;  // the long graph too
    int64_t asked = 0;   // iterations asked for
};

// A call of n_iter iterations: make(q) captures graph q (0: one iteration, 1:
// kGraphIters of them) that the call could use and the handle has not got, and
// says whether it could.  Without graph 0 the handle launches directly from
// then on; without graph 1 it goes on with graph 0.
template <typename Make>
void make_gneb_graphs(GnebGraphs &u, bool have0, bool have1, int n_iter, Make &&make) {
    u.asked += n_iter;
    if (!u.on) return;
    if (n_iter > 1 && !have0 && !make(0)) {
        u.on = false;
        return;
    }
    if (n_iter >= kGraphIters && !have1 && u.run_on && u.asked >= kLongAfter && !make(1)) u.run_on = false;
}

}  // namespace spx
