// Split-FP16 matrix-core form on mirrored sample pairs (gfx950,
// v_mfma_f32_32x32x16_f16): the kernel of complex64 plans.
//
// For one virtual channel c the cube is the complex sum over pixels
//   Y_c[l][n] = sum_p exp(j2pi (psi_{p,c} + b_{p,c} n)) a_p exp(-j2pi beta_p l)
// (Sec. II, eq. (1) per channel, pixel sum of eq. (2)).  Fast time is taken
// from its middle nc = (Ns - 1) / 2: the samples n = nc +- k have conjugate
// fast-time phasors, so with
//   D_c[p][l] = a_p exp(j2pi (psi_{p,c} + b_{p,c} nc - beta_p l))
// the two sums
//   C = sum_p cos(2pi b k) D,   S = sum_p sin(2pi b k) D
// give both samples, Y[nc + k] = C + j S and Y[nc - k] = C - j S: two real
// MACs per term and part instead of four, half the matrix work of the
// complex contraction sample by sample.  As a real product: rows the real and
// imaginary parts of D over l, columns the cosines and sines over the pairs
// k, depth the pixels.  Phase arguments are evaluated and reduced mod 1 in
// binary64, phasors in binary32 with the hardware sin / cos (input in
// revolutions); each binary32 value x is split into hi = rne16(x) and
// lo = rne16(x - hi), and hi*hi + hi*lo + lo*hi are accumulated in fp32 by the
// matrix cores: 6 real MACs = 12 flop per term.
//
// Tiling (workgroup = NW waves):
//   item  = (channel, n tile of NW*WN samples = NW*WN/2 pairs, l tile of TL
//           blocks, pixel chunk)
//   step  = KP pixels (32; 16 where two buffers of 32 would not fit the LDS);
//           both operands of a step are evaluated once per workgroup into one
//           of two LDS buffers while the other one is multiplied
//   wave  = LW blocks x HW pairs: its accumulators hold re / im x cos / sin of
//           the same cells, so C +- j S is formed in registers
// Phasors: a thread takes two neighbouring pixels (packed side by side along
// the depth) and every LQ-th index; of four phasors one is evaluated from its
// binary64-reduced phase, two follow by one binary32 rotation with
// exp(+-j2pi frac(LQ b)), the last by two.
// Schedule: the products of a row block and 16 pixels come in two halves, and
// behind each half stands a slice of the next step's phasor work, its
// instructions placed between the matrix instructions (a wave issues in
// order: vector work that stands behind a block of products waits for the
// matrix core, which it could have run beside).  Phase-shifted waves (NW = 8)
// do the same with the vector part of each slice first in the second wave of
// a SIMD.  The step's barrier stands before its last products, whose operands
// are in registers by then, and the next step's first operands are loaded
// under those.
//
// What bounds it (65,536-pixel frame, 3 x 4, Ns 256, L 128): the matrix cores
// under the chip's power limit.  With 12 instead of 24 flop per term the
// kernel takes 0.247 ms against 0.378 ms on one GPU: matrix cores busy 0.60 of
// the cycles at 1.98 GHz (0.75 at 2.07 GHz before); with the phasor work left
// out the same products take 0.176 ms (0.75 at 2.23 GHz), and schedules that
// keep the matrix cores busier (0.62) run at a lower clock (1.92 GHz) and gain
// 1 %.  Its 1.24 PFLOP/s compare with 1.11 PFLOP/s of a large library fp16
// product on such a GPU.
//
// Pixel strengths are scaled per chunk by an exact power of two (found by
// each work item from its chunk's strengths, or by k_chunk_scale for
// strengths per block) so that the largest maps into [2^14, 2^15) and fp16 keeps
// its relative precision for the small ones; the partial sum is scaled back
// exactly when it is written.
//
// Strengths per block (BS = true, jobs with amp_lstride != 0): only the
// evaluation of D changes: the rotated phasor carries the chunk scale alone
// and each D entry is multiplied by its strength, read from global memory at
// the start of the step before it.  Jobs without per-block strengths in the
// same launch multiply by 1 (exact), so their cubes keep the bits of the
// launch without BS.
//
// Segments: a launch may cover only steps [seg_begin, seg_end) (of 16 pixels)
// of every chunk.  The raw fp32 accumulators are then parked in the partial
// buffer (C at a pair's upper sample, S at its lower one) and reloaded by the
// next segment, which makes the result independent of how a chunk is split
// into segments.  The middle sample of an odd Ns (k = 0) is its own mirror and has
// room for C alone: its sine operand has to be exactly 0.  It is: where the
// phasor comes by a rotation back from index LQ, both factors are the sine and
// cosine s, c of the same reduced phase, the residue s c - rn(s c) is at most
// 2^-26, and both fp16 halves of that are 0 (2^-25 rounds to 0); where it is
// evaluated, its phase is 0.
#include "rs_device.h"
#include "rs_split16.h"

#include <type_traits>
#include <utility>

namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kPB = 256;       // pixels per parameter block
constexpr int kVPM = 2;        // vector instructions scheduled behind each matrix instruction
constexpr int kAmpExp = 14;    // largest scaled strength in [2^14, 2^15)

typedef rs_half2v half2v;
__device__ __forceinline__ float frac32(double v) { return rs_frac32(v); }
__device__ __forceinline__ half2v hi2(float x, float y) { return rs_hi2(x, y); }
__device__ __forceinline__ half2v lo2(float x, float y, half2v h) { return rs_lo2(x, y, h); }
__device__ __forceinline__ unsigned bits(half2v v) { return rs_bits(v); }
__device__ __forceinline__ void pin(float &u, float &w) { rs_pin(u, w); }

// f(integral_constant<int, 0>), ..., f(integral_constant<int, N - 1>)
template <int N, typename F, int... I>
__device__ __forceinline__ void static_for_impl(F &&f, std::integer_sequence<int, I...>)
{
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F &&f)
{
    static_for_impl<N>(f, std::make_integer_sequence<int, N>{});
}

typedef std::integral_constant<int, 0> buf0_t;
typedef std::integral_constant<int, 1> buf1_t;

// Rows of the operand planes are 64 bytes, four 16-byte slots; slot s of row
// i sits at s ^ swz(i).  A matrix operand read (16 lanes: 16 rows, one slot)
// and a phasor store (64 lanes: whole or half rows) then touch every LDS bank
// once.
__device__ __forceinline__ int swz(int i) { return ((i >> 1) & 2) | ((i >> 3) & 1); }

// Phasor parameters of a block of kPB pixels, by pixel (neighbouring pixels
// are read together).
struct __align__(16) par_block {
    double fb[kPB];        // F: beat frequency b, cycles per sample
    double dbase[kPB];     // D: frac(psi) + frac(b nc), cycles
    double dslope[kPB];    // D: -beta, cycles per block
    float2 fr[kPB];        // exp(j2pi frac(LQ b))
    float2 dr[kPB];        // exp(-j2pi frac(LQ beta))
    float da[kPB];         // scaled strength
};

template <int WN, int TL, int NW, bool PHASE, bool BS>
__global__ __launch_bounds__(64 * NW, 1) void k_mfma_mirror(rs_launch Lc)
{
    constexpr int NT = 64 * NW;                   // threads per workgroup
    constexpr int TN = NW * WN;                   // fast-time samples of the tile
    constexpr int NH = TN / 2;                    // mirrored sample pairs of the tile
    constexpr int KP = NH + TL <= 256 ? 32 : 16;  // pixels per step (two D and F buffers fit the LDS)
    constexpr int KT = KP / 16;                   // 16-deep matrix steps per step
    constexpr int SPB = kPB / KP;                 // steps per parameter block
    // wave tile: LW blocks (l) x HW sample pairs, RB x CB accumulators: rows
    // re, im of the l blocks; columns cos, sin of the pairs
    constexpr int LW = TL * NH / NW >= 2048 ? 64 : 32;
    constexpr int HW = TL * NH / NW / LW;
    constexpr int RB = 2 * LW / 32, CB = 2 * HW / 32;
    constexpr int WH = NH / HW;                   // waves along the pairs
    static_assert(HW % 32 == 0 && (TL / LW) * WH == NW, "wave grid");
    // phasor evaluation: thread = a pair of pixels and every LQ-th index
    constexpr int PP = KP / 2;
    constexpr int LQ = NT / PP;
    constexpr int FI = NH / LQ, DI = TL / LQ;     // F and D phasors per pixel and thread
    static_assert(FI * LQ == NH && DI * LQ == TL && LQ % 16 == 0, "phasor mapping");
    constexpr int FBYTES = NH * 2 * KP * 4, DBYTES = TL * 2 * KP * 4;
    // Separate LDS objects for the two buffers: the compiler then knows that
    // the next step's stores never alias the operands being read.
    __shared__ __align__(256) char sB0[FBYTES + DBYTES];
    __shared__ __align__(256) char sB1[FBYTES + DBYTES];
    __shared__ par_block sPar[2];
    __shared__ rs_item_consts sK;
    __shared__ int64_t sItem;
    __shared__ float sRed[NW];

    const int tid = threadIdx.x;
    const int wave = tid >> 6, lane = tid & 63;
    const int g = lane >> 5, li = lane & 31;
    const int wl = wave / WH, wh = wave % WH;

    bool first_item = true;
    for (;;) {
        const int64_t item = rs_next_item(Lc, &sItem, first_item);
        first_item = false;
        if (item < 0) break;
        const int jidx = rs_find_job<RS_BY_ITEM>(Lc, item);
        const rs_job &J = rs_job_of(Lc, jidx);
        const rs_item it = rs_decode_item(J, J.item_first + (item - J.item_begin));
        const int h0 = it.nt * NH, l0 = it.lt * TL;
        const int64_t pb = (int64_t)it.s * J.chunk;
        const int64_t pe = min(J.P, pb + (int64_t)J.chunk);
        const int nsteps = (int)((pe - pb + KP - 1) / KP);
        const int k0 = J.seg_begin / KT;            // segments start at whole parameter blocks
        const int k1 = (int)min(((int64_t)J.seg_end + KT - 1) / KT, (int64_t)nsteps);
        if (k0 >= k1) continue;                      // chunk finished in an earlier segment
        const bool seg_first = k0 == 0, seg_last = k1 == nsteps;
        const int m = it.c / J.N, r = it.c % J.N;
        // sample pairs: h -> fast-time samples ns - nh + h and nh - 1 - h, at
        // +-(h + hofs) from the middle nc
        const int nh = (J.Ns + 1) >> 1;
        const double nc = 0.5 * (double)(J.Ns - 1);
        const double hofs = (J.Ns & 1) ? 0.0 : 0.5;
        // strength exponent shift of the chunk: from k_chunk_scale where the
        // job has a scale array (strengths per block), else found below
        int sh = J.scale ? J.scale[it.s] : 0;
        float a_scale = 1.0f;
        const bool per_block = BS && J.amp_lstride != 0;
        // every reader of the previous item's sK has passed a barrier since
        if (tid == 0) rs_item_consts_of(J, m, r, sK);

        // ---- pixel parameter blocks (256 pixels), raw data prefetched one
        // block ahead so that the global-memory latency stays hidden.  The
        // loads are unconditional (index clamped into the chunk) and their
        // validity is decided when the block is used: a conditional zero
        // would make the compiler wait for the loads right away.  With 512
        // threads the first half evaluates the F parameters of a block and
        // the second half the D parameters. ----------
        const int pt = tid & (kPB - 1);
        float rxp, ryp, rzp, rap, rvp;
        auto fetch_block = [&](int blk) {
            const int64_t p = min(pb + (int64_t)blk * kPB + pt, pe - 1);
            rxp = rs_gload(sK.x, p);
            ryp = rs_gload(sK.y, p);
            rzp = rs_gload(sK.z, p);
            rap = rs_gload(sK.amp, p);
            rvp = rs_gload(sK.vr, p);
        };
        auto load_block = [&](int blk) {
            const bool in = pb + (int64_t)blk * kPB + pt < pe;
            par_block &q = sPar[blk & 1];
            double psi, b, beta;
            rs_chan_args(sK, rxp, ryp, rzp, rvp, m, sK.tx, sK.rx, &psi, &b, &beta);
            if (!in) psi = b = beta = 0.0;
            if (NT == kPB || tid < kPB) {
                const float f = frac32(b * (double)LQ);
                q.fb[pt] = b;
                q.fr[pt] = make_float2(__builtin_amdgcn_cosf(f), __builtin_amdgcn_sinf(f));
            }
            if (NT == kPB || tid >= kPB) {
                const float f = frac32(-beta * (double)LQ);
                q.dbase[pt] = rs_frac(psi) + rs_frac(b * nc);
                q.dslope[pt] = -beta;
                q.dr[pt] = make_float2(__builtin_amdgcn_cosf(f), __builtin_amdgcn_sinf(f));
                q.da[pt] = !in ? 0.f : (per_block ? a_scale : rap * a_scale);
            }
        };

        // ---- phasors of a step: the pixels 2 pp, 2 pp + 1 of the step and
        // the indices it + LQ k of the tile --------------------------------
        const int pp = tid & (PP - 1), ix = tid / PP;
        const int wbase = ix * 64 + (((pp >> 2) ^ swz(ix)) << 4) + ((pp & 3) << 2);
        const double fidx0 = (double)(h0 + ix) + hofs;  // F: index of k = 0, from the middle
        const double didx0 = (double)(l0 + ix);         // D
        // Entry (component 0 / 1, index ix + LQ k) of both pixels: hi and lo.
        // KP = 32: planes of 64-byte rows (32 pixels) for hi and for lo; KP =
        // 16: hi and lo share a row.
        auto put = [&](char *hi, char *lo, int ofs, int n, int comp, int k, float a, float b) {
            const half2v h = hi2(a, b), l = lo2(a, b, h);
            if constexpr (KP == 32) {
                *reinterpret_cast<unsigned *>(hi + ofs + (comp * 2 * n + LQ * k) * 64) = bits(h);
                *reinterpret_cast<unsigned *>(hi + ofs + ((comp * 2 + 1) * n + LQ * k) * 64) = bits(l);
            } else {
                *reinterpret_cast<unsigned *>(hi + ofs + (comp * n + LQ * k) * 64) = bits(h);
                *reinterpret_cast<unsigned *>(lo + ofs + (comp * n + LQ * k) * 64) = bits(l);
            }
        };
        // State of the evaluation of a step: parameters of the two pixels, the
        // sub-group's reduced phases, then its phasors.
        struct phs {
            double fb[2], dbase[2], dslope[2];
            float2 r[2];
            float da[2], f[2];
            float u[2][4], w[2][4];
            float al[2][DI];
        };
        constexpr int SF = (FI + 3) / 4, SD = (DI + 3) / 4;  // sub-groups of up to 4 phasors
        constexpr int IF = FI < 4 ? FI : 4, ID = DI < 4 ? DI : 4;
        static_assert(FI % IF == 0 && DI % ID == 0 && (IF & (IF - 1)) == 0 && (ID & (ID - 1)) == 0, "sub-groups");
        constexpr int NOPS = 1 + SF * (3 + IF) + SD * (3 + ID);
        // strengths of this thread's D entries of step st (1 where the job
        // has none per block, or the pixel or block lies past the end)
        auto load_al = [&](int st, phs &s) {
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int64_t p = pb + (int64_t)st * KP + 2 * pp + j;
#pragma unroll
                for (int k = 0; k < DI; ++k) {
                    const int l = l0 + ix + LQ * k;
                    s.al[j][k] = per_block && p < pe && l < sK.L ? rs_gload(sK.amp, p + (int64_t)l * sK.amp_lstride) : 1.0f;
                }
            }
        };
        // One op of the evaluation of step st into buffer `nxt`.  Op 0 reads
        // the pixels' F parameters.  Then per sub-group of I phasors (F first):
        // the binary64-reduced phases of the two pixels at the sub-group's
        // second index (the first if I < 4), their sin / cos, the other
        // phasors by rotation with r = the step of LQ indices, and I ops that
        // split and store one index each.  The op before the first D
        // sub-group reads the D parameters.  Small ops: a wave that waits for
        // its own results does so next to a few matrix instructions.
        auto phasor_op = [&](auto op, int st, auto nxt, phs &s) {
            constexpr int O = decltype(op)::value;
            const par_block &q = sPar[(st / SPB) & 1];
            const int p0 = (st % SPB) * KP + 2 * pp;
            if constexpr (O == 0) {
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    s.fb[j] = q.fb[p0 + j];
                    s.r[j] = q.fr[p0 + j];
                }
            } else {
                constexpr bool isF = O - 1 < SF * (3 + IF);
                constexpr int I = isF ? IF : ID;
                constexpr int o = isF ? O - 1 : O - 1 - SF * (3 + IF);
                constexpr int sg = o / (3 + I), stage = o % (3 + I);
                constexpr int pv = I == 4 ? 1 : 0;
                if constexpr (stage == 0) {
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        if constexpr (isF)
                            s.f[j] = frac32(s.fb[j] * (fidx0 + (double)((sg * 4 + pv) * LQ)));
                        else
                            s.f[j] = frac32(__builtin_fma(s.dslope[j], didx0 + (double)((sg * 4 + pv) * LQ), s.dbase[j]));
                    }
                } else if constexpr (stage == 1) {
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        s.u[j][pv] = __builtin_amdgcn_cosf(s.f[j]);
                        s.w[j][pv] = __builtin_amdgcn_sinf(s.f[j]);
                        if constexpr (!isF) {
                            s.u[j][pv] *= s.da[j];
                            s.w[j][pv] *= s.da[j];
                        }
                        pin(s.u[j][pv], s.w[j][pv]);
                    }
                } else if constexpr (stage == 2) {
                    if constexpr (I > 1) {
#pragma unroll
                        for (int j = 0; j < 2; ++j) {
                            // times r, and (I = 4) times its conjugate
                            const float cu = s.u[j][pv], cw = s.w[j][pv], rx = s.r[j].x, ry = s.r[j].y;
                            const float wy = cw * ry, uy = cu * ry;
                            s.u[j][pv + 1] = __builtin_fmaf(cu, rx, -wy);
                            s.w[j][pv + 1] = __builtin_fmaf(cw, rx, uy);
                            pin(s.u[j][pv + 1], s.w[j][pv + 1]);
                            if constexpr (I == 4) {
                                s.u[j][0] = __builtin_fmaf(cu, rx, wy);
                                s.w[j][0] = __builtin_fmaf(cw, rx, -uy);
                                pin(s.u[j][0], s.w[j][0]);
                                s.u[j][3] = s.u[j][2];
                                s.w[j][3] = s.w[j][2];
                                rs_rot(s.u[j][3], s.w[j][3], rx, ry);
                            }
                        }
                    }
                } else {
                    constexpr int k = stage - 3, kk = sg * 4 + k;
                    float u0 = s.u[0][k], u1 = s.u[1][k], w0 = s.w[0][k], w1 = s.w[1][k];
                    if constexpr (BS && !isF) {
                        u0 *= s.al[0][kk];
                        w0 *= s.al[0][kk];
                        u1 *= s.al[1][kk];
                        w1 *= s.al[1][kk];
                        pin(u0, w0);
                        pin(u1, w1);
                    }
                    int wb = wbase;
                    asm volatile("" : "+v"(wb));
                    char *dst = (decltype(nxt)::value ? sB1 : sB0) + wb;
                    put(dst, dst + ((wb ^ 32) - wb), isF ? 0 : FBYTES, isF ? NH : TL, 0, kk, u0, u1);
                    put(dst, dst + ((wb ^ 32) - wb), isF ? 0 : FBYTES, isF ? NH : TL, 1, kk, w0, w1);
                    if constexpr (O == SF * (3 + IF) - (IF > 1 ? 1 : 0)) {
#pragma unroll
                        for (int j = 0; j < 2; ++j) {
                            s.dbase[j] = q.dbase[p0 + j];
                            s.dslope[j] = q.dslope[p0 + j];
                            s.r[j] = q.dr[p0 + j];
                            s.da[j] = q.da[p0 + j];
                        }
                    }
                }
            }
        };

        float2 *part = reinterpret_cast<float2 *>(J.partial) +
                       ((int64_t)it.s * (J.M * J.N) + it.c) * (int64_t)J.L * J.Ns;

        // accumulator (rb, cb) element e: l and pair of this lane
        auto l_of = [&](int rb, int e, int gg) { return l0 + wl * LW + rb * 32 + 8 * (e >> 2) + 4 * gg + (e & 3); };
        auto h_of = [&](int cb, int ll) { return h0 + wh * HW + cb * 32 + ll; };

        f32x16 acc[RB][CB];
        if (seg_first) {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                    for (int e = 0; e < 16; ++e) acc[rb][cb][e] = 0.f;
        } else {
            // resume: raw accumulators parked by the previous segment, the
            // cosine sum at the pair's upper sample and the sine sum at its
            // lower one (a pair that is one sample has no sine sum)
            int rli = li, rg = g;
            asm volatile("" : "+v"(rli), "+v"(rg));
#pragma unroll
            for (int rb = 0; rb < RB / 2; ++rb)
#pragma unroll
                for (int cb = 0; cb < CB / 2; ++cb) {
                    const int h = h_of(cb, rli);
#pragma unroll
                    for (int e = 0; e < 16; ++e) {
                        const int l = l_of(rb, e, rg);
                        float2 c = make_float2(0.f, 0.f), s = make_float2(0.f, 0.f);
                        if (h < nh && l < J.L) {
                            const float2 *row = part + (int64_t)l * J.Ns;
                            c = row[J.Ns - nh + h];
                            if (J.Ns - nh + h != nh - 1 - h) s = row[nh - 1 - h];
                        }
                        acc[rb][cb][e] = c.x;
                        acc[rb + RB / 2][cb][e] = c.y;
                        acc[rb][cb + CB / 2][e] = s.x;
                        acc[rb + RB / 2][cb + CB / 2][e] = s.y;
                    }
                }
        }

        // ---- one step ------------------------------------------------------
        // Matrix part: NG = KT RB groups, each the 3 CB products of one row
        // block and one 16-deep matrix step; its D operands (hi, lo) are
        // loaded one group ahead, the F operands of a matrix step two groups
        // ahead.  Vector part: NOPS ops that evaluate the phasors of step
        // st + 1 into the other buffer, spread over the first NG - 1 groups.
        // The step's barrier stands before its last group, whose operands
        // are in registers by then: the next step's first operands are
        // loaded right after it, under the last group's products.
        constexpr int NG = KT * RB;
        static_assert(NG % 2 == 0, "operand sets alternate over the steps");
        // lane offsets of the operand reads
        const int rbase_f = wh * HW * 64 + li * 64 + ((g ^ swz(li)) << 4);
        const int rbase_d = wl * LW * 64 + li * 64 + ((g ^ swz(li)) << 4);
        half8 fh[2][CB], fl[2][CB], dh[2], dl[2];
        // operand of component comp, half `prt` (hi, lo), block blk of 32
        // indices, matrix step t
        auto load_f = [&](const char *buf, int t, int set) {
            int r0 = rbase_f;
            asm volatile("" : "+v"(r0));
            const char *p[2] = {buf + r0, buf + (r0 ^ 32)};
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) {
                const int comp = cb / (CB / 2), blk = cb % (CB / 2);
                fh[set][cb] = KP == 32 ? *reinterpret_cast<const half8 *>(p[t] + (comp * 2 * NH + blk * 32) * 64)
                                       : *reinterpret_cast<const half8 *>(p[0] + (comp * NH + blk * 32) * 64);
                fl[set][cb] = KP == 32 ? *reinterpret_cast<const half8 *>(p[t] + ((comp * 2 + 1) * NH + blk * 32) * 64)
                                       : *reinterpret_cast<const half8 *>(p[1] + (comp * NH + blk * 32) * 64);
            }
        };
        auto load_d = [&](const char *buf, int gi) {
            const int r0 = rbase_d;
            const char *p[2] = {buf + FBYTES + r0, buf + FBYTES + (r0 ^ 32)};
            const int t = gi / RB, rb = gi % RB;
            const int comp = rb / (RB / 2), blk = rb % (RB / 2);
            dh[gi & 1] = KP == 32 ? *reinterpret_cast<const half8 *>(p[t] + (comp * 2 * TL + blk * 32) * 64)
                                  : *reinterpret_cast<const half8 *>(p[0] + (comp * TL + blk * 32) * 64);
            dl[gi & 1] = KP == 32 ? *reinterpret_cast<const half8 *>(p[t] + ((comp * 2 + 1) * TL + blk * 32) * 64)
                                  : *reinterpret_cast<const half8 *>(p[1] + (comp * TL + blk * 32) * 64);
        };
        auto step = [&](int st, auto cur, auto nxt) {
            constexpr int C = decltype(cur)::value, N = decltype(nxt)::value;
            const char *cbuf = C ? sB1 : sB0;
            const char *nbuf = N ? sB1 : sB0;
            // the next block's raw pixels, then its parameters, the two
            // halves of the workgroup in different steps
            if ((st / SPB + 1) * SPB < nsteps) {
                if (st % SPB == 0) fetch_block(st / SPB + 1);
                if (st % SPB == ((NT == kPB || wave < NW / 2) ? 2 : 4)) load_block(st / SPB + 1);
            }
            phs s;
            if constexpr (BS) load_al(st + 1, s);
            // half hf of group gi: its first or last 3 CB / 2 products
            auto mfma_half = [&](int gi, int hf) {
                const int t = gi / RB, rb = gi % RB;
                const int fs = KT == 2 ? t : C;
                if (hf == 0) {
                    if (gi + 1 < NG) {
                        load_d(cbuf, gi + 1);
                        if (KT == 2 && gi == RB - 2) load_f(cbuf, 1, 1);
                    } else {
                        load_f(nbuf, 0, KT == 2 ? 0 : N);
                        load_d(nbuf, 0);
                    }
                }
#pragma unroll
                for (int i = 0; i < 3 * CB; ++i) {
                    if (i / (3 * CB / 2) != hf) continue;
                    const int cb = i % CB;  // hi * hi of every column block, then hi * lo, then lo * hi
                    const half8 d_ = i < 2 * CB ? dh[gi & 1] : dl[gi & 1];
                    const half8 f_ = i / CB == 1 ? fl[fs][cb] : fh[fs][cb];
                    acc[rb][cb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(d_, f_, acc[rb][cb], 0, 0, 0);
                }
            };
            // vector slices: the parameter reads in the first, the other ops
            // from the second to the last but two (their stores have left the
            // wave by the barrier)
            constexpr int NSL = 2 * (NG - 1);
            auto slice_of = [](int o) { return o == 0 ? 0 : 1 + (o - 1) * (NSL > 6 ? NSL - 3 : NSL - 1) / (NOPS - 1); };
            auto slice = [&](auto sl) {
                static_for<NOPS>([&](auto op) {
                    constexpr int O = decltype(op)::value;
                    if constexpr (slice_of(O) == decltype(sl)::value) phasor_op(op, st + 1, nxt, s);
                });
            };
            // A slice's instructions between its matrix instructions: a wave
            // issues one, then vector and LDS work for as long as the matrix
            // core is busy with it (and with the other wave's)
            auto interleave = [](auto first) {
#pragma unroll
                for (int i = 0; i < 3 * CB / 2; ++i) {
                    if (decltype(first)::value) __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // matrix
                    __builtin_amdgcn_sched_group_barrier(0x002, kVPM, 0);                          // vector
                    __builtin_amdgcn_sched_group_barrier(0x200, 2, 0);                             // LDS store
                    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);                             // LDS load
                    if (!decltype(first)::value) __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
            };
            if (PHASE && wave >= NW / 2) {
                // second wave of each SIMD: vector work first
                static_for<2 * NG>([&](auto sl) {
                    constexpr int S = decltype(sl)::value;
                    if constexpr (S == NSL) __syncthreads();
                    if constexpr (S < NSL) slice(sl);
                    mfma_half(S / 2, S % 2);
                    interleave(std::false_type{});
                });
            } else {
                static_for<2 * NG>([&](auto sl) {
                    constexpr int S = decltype(sl)::value;
                    if constexpr (S == NSL) __syncthreads();
                    mfma_half(S / 2, S % 2);
                    if constexpr (S < NSL) slice(sl);
                    interleave(std::true_type{});
                });
            }
        };

        // The chunk's exponent shift sh = 14 - floor(log2(max |a|)), as
        // k_chunk_scale computes it, found by the item itself while the first
        // parameter block is in flight (every item of the chunk finds the
        // same value).
        auto chunk_shift = [&]() {
            float am = 0.f;
            for (int64_t p = pb + tid; p < pe; p += NT) am = fmaxf(am, fabsf(rs_gload(sK.amp, p)));
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) am = fmaxf(am, __shfl_xor(am, o));
            if (lane == 0) sRed[wave] = am;
            __syncthreads();
            am = sRed[0];
#pragma unroll
            for (int w = 1; w < NW; ++w) am = fmaxf(am, sRed[w]);
            const int ex = (am > 0.f && am <= 3.4e38f) ? ilogbf(am) : kAmpExp;
            const int v = kAmpExp - ex;
            return v > 126 ? 126 : (v < -126 ? -126 : v);
        };

        __syncthreads();  // previous item's readers of the LDS buffers are done
        fetch_block(k0 / SPB);
        if (!J.scale) sh = chunk_shift();
        a_scale = ldexpf(1.0f, sh);
        load_block(k0 / SPB);
        __syncthreads();
        {
            phs s;
            if constexpr (BS) load_al(k0, s);
            static_for<NOPS>([&](auto op) { phasor_op(op, k0, buf0_t{}, s); });  // k0 is even: buffer 0
        }
        __syncthreads();
        load_f(sB0, 0, 0);
        load_d(sB0, 0);
        // Steps in pairs (an odd count ends with a step of pixels past the
        // end, whose strengths are 0): a loop left in its middle would make
        // the compiler copy the accumulators.
        int st = k0;
        do {
            step(st, buf0_t{}, buf1_t{});
            step(st + 1, buf1_t{}, buf0_t{});
            st += 2;
        } while (st < k1);

        // ---- park or write the partial tile ---------------------------------
        // Lane coordinates pass through an empty asm statement so that the
        // store addresses are computed here, not hoisted above the step loop.
        int wli = li, wg = g;
        asm volatile("" : "+v"(wli), "+v"(wg));
        const float osc = ldexpf(1.0f, -sh);
#pragma unroll
        for (int rb = 0; rb < RB / 2; ++rb)
#pragma unroll
            for (int cb = 0; cb < CB / 2; ++cb) {
                const int h = h_of(cb, wli);
                const int np = J.Ns - nh + h, nm = nh - 1 - h;
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int l = l_of(rb, e, wg);
                    const float cr = acc[rb][cb][e], ci = acc[rb + RB / 2][cb][e];
                    const float sr = acc[rb][cb + CB / 2][e], si = acc[rb + RB / 2][cb + CB / 2][e];
                    if (h < nh && l < J.L) {
                        float2 *row = part + (int64_t)l * J.Ns;
                        if (seg_last) {
                            row[np] = make_float2((cr - si) * osc, (ci + sr) * osc);
                            row[nm] = make_float2((cr + si) * osc, (ci - sr) * osc);
                        } else {
                            row[np] = make_float2(cr, ci);
                            if (nm != np) row[nm] = make_float2(sr, si);
                        }
                    }
                }
            }
    }
}

// interleave: the software-pipelined schedule for NW = 8 too (shapes with
// NW = 4 always use it)
template <int WN, int TL, int NW, bool BS>
void launch_one(const rs_launch &L, bool interleave, int grid, hipStream_t st)
{
    if constexpr (NW == 8) {
        if (!interleave) {
            hipLaunchKernelGGL((k_mfma_mirror<WN, TL, NW, true, BS>), dim3(grid), dim3(64 * NW), 0, st, L);
            return;
        }
    }
    hipLaunchKernelGGL((k_mfma_mirror<WN, TL, NW, false, BS>), dim3(grid), dim3(64 * NW), 0, st, L);
}

template <bool BS>
void launch_shape(const rs_launch &L, int wn, int tl, int nw, bool interleave, int grid, hipStream_t st)
{
    if (tl == 128) {
        if (wn == 64) launch_one<64, 128, 4, BS>(L, interleave, grid, st);
        else if (nw == 8) launch_one<32, 128, 8, BS>(L, interleave, grid, st);
        else launch_one<32, 128, 4, BS>(L, interleave, grid, st);
    } else {
        if (wn == 32 && nw == 8) launch_one<32, 64, 8, BS>(L, interleave, grid, st);
        else if (wn == 32) launch_one<32, 64, 4, BS>(L, interleave, grid, st);
        else if (wn == 64 && nw == 8) launch_one<64, 64, 8, BS>(L, interleave, grid, st);
        else if (wn == 64) launch_one<64, 64, 4, BS>(L, interleave, grid, st);
        else launch_one<128, 64, 4, BS>(L, interleave, grid, st);
    }
}

}  // namespace

void rs_launch_mirror(const rs_launch &L, int wn, int tl, int nw, bool interleave, bool block_strength, int grid,
                      hipStream_t st)
{
    if (block_strength)
        launch_shape<true>(L, wn, tl, nw, interleave, grid, st);
    else
        launch_shape<false>(L, wn, tl, nw, interleave, grid, st);
}
