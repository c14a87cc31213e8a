// bq_tune.h — what the biclique kernel tuner makes of its timings (host only, apart from the
// device work so that the host can exercise it).
#pragma once

namespace pbit {

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
