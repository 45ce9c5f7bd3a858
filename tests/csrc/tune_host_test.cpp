// Host test of the tile choice (paper_2307_09226_amd/csrc/rs_tune.h) on a
// simulated device whose clock falls as it warms up.  Prints "ALL OK" and exits
// 0 on success.
#include "rs_tune.h"

#include <cstdio>
#include <cstdlib>
#include <functional>
#include <initializer_list>
#include <vector>

#define CHECK(cond)                                                                       \
    do {                                                                                  \
        if (!(cond)) {                                                                    \
            std::fprintf(stderr, "%s:%d: CHECK failed: %s\n", __FILE__, __LINE__, #cond); \
            std::exit(1);                                                                 \
        }                                                                                 \
    } while (0)

// Configurations take ms[i] on the warm device.  The cold one is `boost` times
// as fast and falls back with the time constant tau (ms of work); noise is a
// fixed sequence of +-`noise`.
struct device {
    std::vector<double> ms;
    double boost, tau, noise;
    double work = 0.0;
    int calls = 0, fail_at = -1;

    double operator()(int i)
    {
        if (calls++ == fail_at) return -1.0;
        const double speed = 1.0 + (boost - 1.0) * std::exp(-work / tau);
        const double t = ms[i] / speed * (1.0 + noise * ((calls * 7) % 5 - 2) / 2.0);
        work += t;
        return t;
    }
};

int main()
{
    // the frame: 64x128x4 is the first of the list and 15 % slower than the
    // rule's 32x128x8 on a warm device
    for (double boost : {1.0, 1.1, 1.25, 1.5})
        for (double tau : {0.1, 2.0, 10.0, 40.0})
            for (double noise : {0.0, 0.002, 0.01}) {
                std::vector<double> ms = {0.290, 0.33, 0.253, 0.255, 0.40, 0.36, 0.35, 0.31, 0.30, 0.31, 0.33};
                device d{ms, boost, tau, noise};
                CHECK(rs_tune_pick(11, 2, std::ref(d)) == 2);
                // one that is 10 % faster is found wherever it stands
                for (int fast : {0, 3, 5, 10}) {
                    device e{ms, boost, tau, noise};
                    e.ms[fast] = 0.253 * 0.9;
                    CHECK(rs_tune_pick(11, 2, std::ref(e)) == fast);
                }
                // another start, the same choice
                device f{ms, boost, tau, noise};
                const int got = rs_tune_pick(11, 8, std::ref(f));
                CHECK(got == 2 || got == 3);   // 1 % apart
            }
    // a failure at any measurement; 2 to settle, 2 for each of the others, 10 at last
    for (int at = 0; at < 24; ++at) {
        device d{{1.0, 2.0, 3.0, 4.0}, 1.0, 1.0, 0.0};
        d.fail_at = at;
        CHECK(rs_tune_pick(4, 1, std::ref(d)) == (at < 2 + 2 * 3 + 10 ? -1 : 0));
    }
    // 1.5 % faster on a quiet device
    device g{{1.0, 0.985, 1.2}, 1.2, 5.0, 0.002};
    CHECK(rs_tune_pick(3, 0, std::ref(g)) == 1);
    std::puts("ALL OK");
    return 0;
}
