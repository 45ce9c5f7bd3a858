// Paths and workspace layout of a range-Doppler call: plain C++, so that the
// host tests can sweep it.
#pragma once
#include <stddef.h>
#include <stdint.h>

#include <algorithm>

constexpr int kRdThreads = 256;
constexpr int kGroupElems = 4096;     // KB * L of k_doppler_power, at most (dynamic LDS <= 64 KiB)
constexpr int kMergeCells = 4096;     // cells per k_rd_merge workgroup (256 threads, 4 float4 each)
constexpr int kMapCells = 256;        // cells per k_map_merge workgroup
constexpr int kFNs = 256;             // fast-time length of the fused path
constexpr size_t kRdPeakPartBytes = 8;
// k_doppler_reg workgroups per compute unit aimed at (192 channels of 512 x
// 256: 131 us with 1, 126 with 2, 133 with 4)
constexpr int kDopplerPerCu = 2;

// Bytes of fast-time spectra that the two-pass path holds at once (a frame's at
// least); more frames go through it in rounds, so that neither the workspace nor
// a launch's grid grows with the call.  A round costs its launches' tails (63
// frames of 192 x 512 x 64: 1.79 ms in one, 2.00 in seven), hence 2 GiB.  At
// 256 x 16 and 256 x 32 one workgroup could hold a channel without any spectra:
// there no more than a plan keeps for its allocating calls, at the same speed
// (8,138 frames of 12 x 256 x 16: 2.03 ms with 3 GiB, 2.04 with 256 MiB).
inline int64_t rs_rd_spectra_bytes(int Ns, int L) { return Ns == kFNs && L <= 32 ? (int64_t)240 << 20 : (int64_t)2 << 30; }

struct rs_rd_shape {
    int Ns = 0, L = 0, C = 0, ncu = 1;
};

// Whether the fused path is the faster one: it reads the cubes once (the
// two-pass path moves three times the bytes) but runs one workgroup per
// compute unit, one channel at a time, and merges a partial map per workgroup
// and frame, so it needs enough (frame, channel, block) rows, and frames of
// which few workgroups share one -- or channels so few that a frame's map
// weighs as much as its cube.  Measured, fused / two-pass in us (C, L, frames):
// 12, 128: 1: 33.2 / 20.4, 10: 36.6 / 32.7, 16: 40.5 / 40.7, 32: 57 / 65,
// 100: 136 / 216; 8, 64: 32: 31 / 33; 192, 128: 1: 122 / 41, 2: 97 / 62, 4: 106 / 113;
// 64, 128: 6: 57 / 56, 8: 70 / 76, 10: 83 / 97; 64, 64: 13: 62 / 59;
// 1, 64: 64: 22 / 18, 100: 23 / 23, 150: 23 / 28; 2, 64: 48: 22 / 22, 100: 28 / 35;
// 4, 64: 16: 25 / 24, 32: 29 / 29; 1, 128: 100: 31 / 33;
// 12, 32: 30: 34 / 29; 3, 32: 48: 24 / 27; 1, 32: 100: 22 / 20, 150: 24 / 26, 4000: 228 / 316;
// 2, 32: 1000: 103 / 118; 4, 32: 1000: 184 / 191; 12, 16: 100: 58 / 34; 1, 16: 4000: 184 / 154.
inline bool rs_rd_fused_pays(int64_t nframes, int C, int Ns, int L)
{
    if (Ns != kFNs) return false;
    const int64_t items = nframes * C, rows = items * L;
    if (L == 32) return C <= 4 && items >= 144;
    if (L != 64 && L != 128) return false;
    return (nframes >= 16 && rows >= 16384) || (nframes >= 8 && rows >= 53248) || rows >= 98304 ||
           (C <= 4 && items >= 96);
}

// The two-pass path's range FFTs: in registers (k_range_reg) for Ns 64..1024.
// Rows of 16 and 32 points leave a register row to one or two threads, whose
// loads do not coalesce: 1 channel of 16 x 64, 16,000 frames, 145 us through LDS
// and 171 us in registers.
inline bool rs_rd_range_in_registers(int Ns) { return Ns >= 64 && Ns <= 1024; }

// The two-pass path's Doppler FFTs: in registers with the channels in runs
// (k_doppler_reg, then k_map_merge over the runs' maps), or in LDS with a
// workgroup looping over a group's channels, which needs no second launch and
// no second pass over the map.  While that leaves compute units without a
// workgroup, the loop is what takes the time; else the bytes, of which the map
// is half a cube's with one channel.  Measured, LDS / registers in us (C,
// Ns x L, frames): 192, 512 x 64, 1: 576 / 45; 4, 16 x 256, 1: 45 / 17; 8, 64 x 16, 10:
// 22 / 16; 1, 16 x 64, 1: 13 / 16; 2, 32 x 32, 3: 15 / 17; 1, 16 x 64, 16,000: 145 / 293;
// 1, 256 x 256, 100: 90 / 114; 2, 256 x 256, 100: 178 / 164; 3, 16 x 32, 16,000: 204 / 260;
// 4, 32 x 16, 16,000: 310 / 240; 2, 4096 x 64, 3: 37 / 41; 1, 256 x 16, 4,000: 216 / 154.
inline bool rs_rd_doppler_in_registers(int64_t nframes, const rs_rd_shape &q)
{
    if (q.L < 16 || q.L > 256 || q.Ns < 16) return false;
    const int64_t groups = nframes * (q.Ns / 16), work = (int64_t)q.C * q.L;
    if (groups < q.ncu) return work >= 160 || (work >= 96 && (q.C >= 4 || q.Ns >= 128));
    const int least = q.Ns > 1024 ? 3 : (int64_t)q.Ns * q.L >= 4096 ? 2 : q.Ns <= 16 ? 5 : q.Ns <= 32 ? 4 : 3;
    return q.C >= least || (q.L == 16 && q.Ns >= 64 && groups >= 8 * (int64_t)q.ncu);
}

// Workgroups of the fused path: at most one per compute unit (a
// workgroup's LDS fills one), as few as keep the longest run at
// ceil(F C / compute units) items, the items split evenly over them; a
// frame's items can fall into several runs, whose partial maps k_rd_merge
// adds (fewer workgroups, fewer partial maps).
inline int64_t rs_rd_fused_workgroups(int64_t nframes, int C, int ncu)
{
    const int64_t n = nframes * C;
    const int64_t per = (n + ncu - 1) / std::max(1, ncu);
    return std::max<int64_t>(1, (n + per - 1) / per);
}

// Workspace of one call, in 256-byte aligned pieces.  Fused path: the
// partial maps [W][J][cells], the map when the caller wants none, the block
// maxima.  Two-pass path: the float2 fast-time spectra and the runs' partial
// maps [group][S][cells] (S > 1) of a group of frames, the map when the caller
// wants none, the group maxima.
struct rs_rd_layout {
    bool fused = false;
    int64_t W = 0, J = 0, nitems = 0;
    int groups = 0, kb = 0;          // maxima per frame; range bins per k_doppler_power workgroup
    int64_t group = 0;               // frames of one round of the two passes
    int S = 0, per = 0, logkb = 0;   // channel runs of k_doppler_reg (S = 0: k_doppler_power)
    size_t mid = 0, slots = 0, pw = 0, parts = 0, total = 0;   // byte offsets / sizes
};

// Range bins of a k_doppler_power workgroup.
inline int rs_rd_bins(const rs_rd_shape &q) { return std::max(1, std::min(std::min(16, kGroupElems / q.L), q.Ns)); }

// Frames of a full round (a grid stays below 2^32 threads).
inline int64_t rs_rd_round(const rs_rd_shape &q)
{
    const int64_t spectra = (int64_t)q.C * q.Ns * q.L * 8, groups = q.Ns / rs_rd_bins(q);
    return std::max<int64_t>(1, std::min(rs_rd_spectra_bytes(q.Ns, q.L) / spectra, ((int64_t)1 << 23) / groups));
}

inline size_t rs_rd_up(size_t b) { return (b + 255) & ~(size_t)255; }

inline rs_rd_layout rs_rd_plan_layout(const rs_rd_shape &q, int64_t nframes, bool power_given)
{
    rs_rd_layout y;
    const int Ns = q.Ns, L = q.L, C = q.C;
    const int64_t cells = (int64_t)Ns * L;
    y.fused = rs_rd_fused_pays(nframes, C, Ns, L);
    size_t mid_bytes, slot_bytes = 0;
    if (y.fused) {
        y.nitems = nframes * C;
        y.W = rs_rd_fused_workgroups(nframes, C, q.ncu);
        const int64_t per = (y.nitems + y.W - 1) / y.W;
        y.J = (per - 1 + C - 1) / C + 1;   // frames a run of `per` items can touch
        y.groups = (int)(cells / kMergeCells);
        mid_bytes = (size_t)(y.W * y.J * cells) * sizeof(float);
    } else {
        y.kb = rs_rd_bins(q);
        y.groups = Ns / y.kb;
        const int64_t most = rs_rd_round(q), rounds = (nframes + most - 1) / most;
        y.group = (nframes + rounds - 1) / rounds;
        mid_bytes = (size_t)(y.group * C * cells) * 8;
        if (rs_rd_doppler_in_registers(y.group, q)) {
            // KB range bins x L / 16 threads per channel, CP channels side by
            // side; enough runs of channels for kDopplerPerCu workgroups per
            // compute unit
            const int kb = std::min(Ns, kRdThreads * 16 / L), cp = kRdThreads / (kb * (L / 16));
            while ((1 << y.logkb) < kb) ++y.logkb;
            const int64_t base = y.group * (Ns / kb);
            int64_t blocks = ((int64_t)q.ncu * kDopplerPerCu + base - 1) / base;
            blocks = std::max<int64_t>(1, std::min<int64_t>(blocks, (C + cp - 1) / cp));
            y.per = (int)((C + blocks * cp - 1) / (blocks * cp));
            y.S = (C + y.per - 1) / y.per;
            y.groups = (int)(cells / kMapCells);
            // one run: its map is the frame's
            slot_bytes = y.S == 1 ? 0 : (size_t)(y.group * y.S * cells) * sizeof(float);
        }
    }
    const size_t pw_bytes = power_given ? 0 : (size_t)(nframes * cells) * sizeof(float);
    const size_t part_bytes = (size_t)nframes * y.groups * kRdPeakPartBytes;
    y.mid = 0;
    y.slots = rs_rd_up(mid_bytes);
    y.pw = y.slots + rs_rd_up(slot_bytes);
    y.parts = y.pw + rs_rd_up(pw_bytes);
    y.total = y.parts + rs_rd_up(part_bytes);
    return y;
}

// Workspace that serves any call of up to `nframes` frames: a program sizes it
// for its largest call.  A call's own need falls here and there as frames are
// added (fewer runs of channels; the fused path takes over with a partial map
// per workgroup instead of the spectra).
inline size_t rs_rd_workspace_bytes(const rs_rd_shape &q, int64_t nframes, bool power_given)
{
    const int64_t cells = (int64_t)q.Ns * q.L;
    // the paths and the runs change below this many frames of a round only
    const int64_t few = std::min(nframes, std::max<int64_t>(4096, 16 * (int64_t)q.ncu));
    size_t mid = 0, parts = 0;
    int groups = 0;
    auto two_pass = [&](int64_t n) {
        const rs_rd_layout y = rs_rd_plan_layout(q, n, true);
        if (y.fused) return;
        mid = std::max(mid, y.pw);
        parts = std::max(parts, (size_t)n * y.groups);
        groups = std::max(groups, y.groups);
    };
    for (int64_t n = 1; n <= few; ++n) two_pass(n);
    const bool fused = rs_rd_fused_pays(nframes, q.C, q.Ns, q.L);
    if (nframes > few && !fused) {
        two_pass(std::min(nframes, rs_rd_round(q)));   // a longer call's rounds hold no more
        parts = (size_t)nframes * groups;
    }
    if (fused) {
        const int64_t items = nframes * q.C, per = (items + q.ncu - 1) / q.ncu;
        const int64_t maps = std::min<int64_t>(q.ncu, items) * ((per + q.C - 2) / q.C + 1);
        mid = std::max(mid, rs_rd_up((size_t)(maps * cells) * sizeof(float)));
        parts = std::max(parts, (size_t)(nframes * (cells / kMergeCells)));
    }
    return mid + (power_given ? 0 : rs_rd_up((size_t)(nframes * cells) * sizeof(float))) +
           rs_rd_up(parts * kRdPeakPartBytes);
}
