// Choice of a tile configuration by measurement: plain C++ over a timing
// function, so that the host tests can drive it with a device whose clock
// moves.
#pragma once
#include <cmath>

// Of the configurations 0 .. n - 1, `own` being the plan's: the one to take.
// time(i) runs configuration i and returns its mean time, < 0 on failure (then
// the result is -1).
//
// The chip holds a fast clock until its power limit bites, some milliseconds
// into a run, so what is timed first looks faster than it is: the frame's
// 64x128x4 was taken over 32x128x8 that way, 0.290 ms against 0.253.  Hence the
// plan's own configuration runs until two successive means agree (1 %), and
// every other one is timed between two runs of the own one and judged by the
// ratio.  The one with the smallest ratio then meets the own one five times
// more, and is taken if it is faster each time.
template <typename F>
int rs_tune_pick(int n, int own, F &&time)
{
    double before = time(own);
    for (int k = 0; k < 20; ++k) {
        const double t = time(own);
        if (before < 0.0 || t < 0.0) return -1;
        const bool settled = std::fabs(t - before) <= 0.01 * t;
        before = t;
        if (settled) break;
    }
    // time of configuration i relative to the own one's right before and after
    auto ratio = [&](int i) -> double {
        const double t = time(i), after = time(own);
        if (t < 0.0 || after < 0.0) return -1.0;
        const double mean = 0.5 * (before + after);
        before = after;
        return t / mean;
    };
    int best = own;
    double least = 1.0;
    for (int i = 0; i < n; ++i) {
        if (i == own) continue;
        const double r = ratio(i);
        if (r < 0.0) return -1;
        if (r < least) {
            least = r;
            best = i;
        }
    }
    for (int k = 0; k < 5 && best != own; ++k) {
        const double r = ratio(best);
        if (r < 0.0) return -1;
        if (r >= 0.998) best = own;
    }
    return best;
}
