// Host test of the range-Doppler paths and workspace layout
// (paper_2307_09226_amd/csrc/rs_rd_layout.h), built with g++ under the
// sanitizers.  Prints "ALL OK" and exits 0 on success.
#include "rs_rd_layout.h"

#include <cstdio>
#include <cstdlib>
#include <initializer_list>

#define CHECK(cond)                                                                                          \
    do {                                                                                                     \
        if (!(cond)) {                                                                                       \
            std::fprintf(stderr, "%s:%d: CHECK failed: %s (C %d Ns %d L %d F %lld)\n", __FILE__, __LINE__, #cond, \
                         q.C, q.Ns, q.L, (long long)F);                                                      \
            std::exit(1);                                                                                    \
        }                                                                                                    \
    } while (0)

template <typename F>
static void for_shapes(F &&f)
{
    for (int Ns = 2; Ns <= 4096; Ns *= 2)
        for (int L = 2; L <= 1024; L *= 2)
            for (int C : {1, 2, 3, 4, 5, 8, 12, 31, 64, 97, 192, 1000}) {
                rs_rd_shape q;
                q.Ns = Ns;
                q.L = L;
                q.C = C;
                q.ncu = 256;
                f(q);
            }
}

// The runs of a frame's channels: every run has channels, all of them are in
// one, and their maps take no more than half of the spectra's bytes.
static void runs(const rs_rd_shape &q)
{
    for (int64_t F : {1, 2, 3, 7, 16, 40, 100, 333, 1000, 5000, 20000, 300000, 20000000}) {
        const rs_rd_layout y = rs_rd_plan_layout(q, F, true);
        if (y.fused) {
            CHECK(q.Ns == 256 && y.W <= q.ncu && y.W * y.J >= F);
            continue;
        }
        CHECK(y.groups >= 1 && y.kb * q.L <= kGroupElems);
        // rounds of frames: workspace and grids do not grow with the call (a
        // frame's own size, and the maxima, aside)
        const int64_t cells = (int64_t)q.Ns * q.L, frame = 8 * cells * q.C;
        CHECK(y.group >= 1 && y.group <= F);
        CHECK(y.group == 1 || y.group * frame <= ((int64_t)2 << 30));
        CHECK(y.parts <= (size_t)std::max<int64_t>((int64_t)2 << 30, frame) * 3 / 2 + 512);
        CHECK(q.Ns != 256 || q.L > 32 || y.group == 1 || y.total <= ((size_t)256 << 20) + (size_t)F * y.groups * 8);
        CHECK(y.group == 1 || y.group * std::max<int64_t>(y.groups, cells / 256) * 256 < ((int64_t)1 << 32));
        if (!y.S) continue;
        CHECK((int64_t)y.S * y.per >= q.C && (int64_t)(y.S - 1) * y.per < q.C);
        CHECK(y.S == 1 || y.pw - y.slots <= (y.slots - y.mid) / 2 + 256);
        CHECK(q.Ns * (int64_t)q.L % kMapCells == 0);
    }
}

// A workspace for `F` frames serves every smaller call, and is not much larger
// than the largest of their needs.
static void bound(const rs_rd_shape &q)
{
    for (int pg = 0; pg < 2; ++pg) {
        size_t most = 0;
        const int64_t dense = q.C <= 12 || q.C == 192 ? 900 : 120;
        for (int64_t F = 1; F <= dense; ++F) {
            most = std::max(most, rs_rd_plan_layout(q, F, pg).total);
            if (F > 40 && F % 37 > 1) continue;
            const size_t b = rs_rd_workspace_bytes(q, F, pg);
            CHECK(b >= most && b <= 2 * most);
        }
        for (int64_t F : {4095, 4096, 4097, 5000, 100000, 3000001}) {
            const size_t b = rs_rd_workspace_bytes(q, F, pg);
            for (int64_t n = F; n > 0; n -= 1 + (F - n) * (F - n)) CHECK(rs_rd_plan_layout(q, n, pg).total <= b);
            for (int64_t n = 1; n < F; n = n * 5 / 4 + 1) CHECK(rs_rd_plan_layout(q, n, pg).total <= b);
            const int64_t r = rs_rd_round(q);
            for (int64_t n : {r - 1, r, r + 1, 2 * r, 2 * r + 1, 3 * r})
                if (n >= 1 && n <= F) CHECK(rs_rd_plan_layout(q, n, pg).total <= b);
        }
    }
}

int main()
{
    for_shapes([](const rs_rd_shape &q) {
        if (q.Ns == 256 || q.L == 16 || q.L == 64 || q.Ns * q.L <= 16) bound(q);
    });
    for_shapes(runs);
    std::puts("ALL OK");
    return 0;
}
