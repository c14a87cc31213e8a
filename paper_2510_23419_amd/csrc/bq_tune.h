// bq_tune.h — what the biclique kernel tuner makes of its timings (host only, apart from the
// device work so that the host can exercise it).
#pragma once

#include <vector>

#include "bq.h"

namespace pbit {

// Timed cost of one kernel (with its replica tile or slice width rt) at a shape: of a launch
// and of each sweep in it.
struct BqCost {
    BqVariant variant;
    int rt;
    double load_ms, sweep_ms;
};

// The timed kernel that costs least over `sweeps` sweeps, up to `chunk(variant)` of them per
// launch and no more than `run`, the sweeps from one energy check to the next; the cluster
// kernel only where this anneal can take it.  Null if none was timed.
template <class Chunk>
const BqCost *cheapest(const std::vector<BqCost> &costs, bool cluster_ok, int sweeps, int run, Chunk chunk)
{
    const BqCost *best = nullptr;
    double best_ms = 0.0;
    for (const BqCost &c : costs) {
        if (c.variant == BqVariant::Cluster && !cluster_ok) continue;
        const int most = chunk(c.variant), per = run < most ? run : most;
        const double ms = (double)((sweeps + per - 1) / per) * c.load_ms + sweeps * c.sweep_ms;
        if (!best || ms < best_ms) {
            best = &c;
            best_ms = ms;
        }
    }
    return best;
}

// Times a kernel that runs any number of sweeps per launch over 1 and, if m > 0, 1 + m sweeps:
// time(sweeps) gives milliseconds, ran() whether the launches just timed ran their sweeps.
// False if some did not: their time is no sweep's.
template <class Time, class Ran>
bool time_runs(Time time, Ran ran, int m, double *one, double *more)
{
    *one = time(1);
    if (!ran()) return false;
    if (m > 0) {
        *more = time(1 + m);
        if (!ran()) return false;
    }
    return true;
}

}  // namespace pbit
