// Plain form: binary64 direct sum (gfx950, v_mfma_f64_16x16x4_f64).
//
// Y[c][l][n] = sum_p a_p exp(j2pi(psi_{p,c} + b_{p,c} n - beta_p l))  (Sec. II,
// eq. (1) per virtual channel, pixel sum of eq. (2)).  Fast time is taken
// from its middle nc = (Ns - 1) / 2: with
//   D[p][l] = a_p exp(j2pi(frac(psi) + frac(b nc) - beta l))
//   C = sum_p cos(2pi b k) D,   S = sum_p sin(2pi b k) D
// the mirrored samples are Y[nc + k] = C + j S and Y[nc - k] = C - j S: two
// binary64 multiply-adds per term instead of four (4 flop per term).  The sums
// are a real product: rows the real and imaginary parts of D over l, columns
// the cosines and sines over the pairs k, depth the pixels.
//
// The binary64 matrix instruction has the vector units' rate (64 cycles for
// 2,048 flop) and holds them while it runs (a vector instruction beside it
// waits 38 cycles), so nothing is gained by overlap; it is taken for its
// operands: one 8-byte LDS read per lane and operand feeds 16 x 16 x 4 products,
// where vector multiply-adds read 12 operand pairs for 64.
//
// Measured on the 65,536-pixel frame (3 x 4, Ns 256, L 128): 1.71 ms for 103
// GFLOP = 60 TFLOP/s, against 4.28 ms for vector multiply-adds sample by
// sample (206 GFLOP, 48 TFLOP/s); a large binary64 library product reaches 73
// on the same GPU.  Without the phasor work the same products take 1.50 ms
// (LDS operands and one barrier per step), the phasors alone 0.43 ms.
//
// Work item = (channel, tile of 2 NH samples x TL blocks, pixel chunk).  A
// wave owns LW blocks x HW pairs: re / im x cos / sin of the same cells, so
// C +- j S is formed in registers.  Per step of 16 pixels the phasors of the
// next step go to the other of two LDS buffers, one barrier per step.  A
// thread evaluates eight phasors of a pixel, every R-th index: the first
// from its reduced phase (binary64 sincospi), the others by binary64
// rotation with exp(j2pi frac(R b)) or exp(-j2pi frac(R beta)), at most 7
// rotations (~1e-15 relative).  The rotations and the pixels' phase arguments
// come in blocks of 256 pixels from waves that evaluate no phasors.  With
// strengths per block (amp_lstride != 0) the slow-time run rotates the unit
// phasor and multiplies each entry by a_{p,l}.  Chunks write binary64 partial
// tiles that the reduce kernel sums in a fixed order.
#include "rs_device.h"

namespace {

typedef double d4 __attribute__((ext_vector_type(4)));

constexpr int kKP = 16;       // pixels per step
constexpr int kPB = 256;      // pixels per parameter block
constexpr int kSPB = kPB / kKP;

struct __align__(16) pix_par {
    double fb, frx, fry;      // beat frequency b; exp(j2pi frac(RF b))
    double da;                // strength
    double dbase, dslope;     // frac(psi) + frac(b nc); -beta
    double drx, dry;          // exp(-j2pi frac(RD beta))
};

template <int NH, int TL, int NW>
__global__ __launch_bounds__(64 * NW, 2) void k_plain_fp64(rs_launch Lc)
{
    // Vector work of a step: the first WD waves evaluate D, WF waves F, the last
    // WP a part of the next parameter block.
    constexpr int RUN = 8;                                 // phasors per thread and pixel
    constexpr int RF = NH / RUN, RD = TL / RUN;            // runs per pixel
    constexpr int WD = RD * kKP / 64, WF = RF * kKP / 64, WP = 2;
    constexpr int WF0 = NW == 8 ? 4 : WD;                  // first wave evaluating F
    constexpr int PR = kPB / (64 * WP);                    // pixels of a block per parameter thread
    static_assert(WD >= 1 && WF >= 1 && WD <= WF0 && WF0 + WF + WP <= NW && PR <= 4, "roles");
    constexpr int LW = NW == 8 ? TL / 4 : TL / 2, HW = NH / 2;  // wave tile
    constexpr int RB = 2 * LW / 16, CB = 2 * HW / 16;
    // record of a pixel: D re, D im, F cos, F sin; the pad puts the records
    // of neighbouring pixels, which one operand read spans, in the other half
    // of the LDS banks
    constexpr int REC = 2 * TL + 2 * NH + 16;
    __shared__ __align__(256) double sX[2][kKP * REC];
    __shared__ pix_par sPar[2][kPB];
    __shared__ rs_item_consts sK;
    __shared__ int64_t s_item;

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int wl = wave >> 1, wh = wave & 1;
    bool first = true;
    for (;;) {
        const int64_t item = rs_next_item(Lc, &s_item, first);
        first = false;
        if (item < 0) break;
        const int jidx = rs_find_job<RS_BY_ITEM>(Lc, item);
        const rs_job &J = rs_job_of(Lc, jidx);
        const rs_item it = rs_decode_item(J, J.item_first + (item - J.item_begin));
        const int h0 = it.nt * NH, l0 = it.lt * TL;
        const int64_t pb = (int64_t)it.s * J.chunk;
        const int64_t pe = min(J.P, pb + (int64_t)J.chunk);
        const int nsteps = (int)((pe - pb + kKP - 1) / kKP);
        const int m = it.c / J.N, r = it.c % J.N;
        // sample pairs: h -> fast-time samples ns - nh + h and nh - 1 - h, at
        // +-(h + hofs) from the middle nc
        const int nh = (J.Ns + 1) >> 1;
        const double nc = 0.5 * (double)(J.Ns - 1);
        const double hofs = (J.Ns & 1) ? 0.0 : 0.5;
        // every reader of the previous item's sK has passed a barrier since
        if (tid == 0) rs_item_consts_of(J, m, r, sK);
        __syncthreads();

        // raw values of a pixel, loaded ahead of their use; the index is
        // clamped into the chunk and the pixel's validity decided when it is
        // used
        float rx, ry, rz, ra, rv;
        auto fetch = [&](int64_t p) {
            p = min(p, pe - 1);
            rx = rs_gload(sK.x, p);
            ry = rs_gload(sK.y, p);
            rz = rs_gload(sK.z, p);
            ra = rs_gload(sK.amp, p);
            rv = rs_gload(sK.vr, p);
        };
        auto params = [&](int blk, int i) {
            pix_par q;
            double psi, b, beta;
            rs_chan_args(sK, rx, ry, rz, rv, m, sK.tx, sK.rx, &psi, &b, &beta);
            const bool in = pb + (int64_t)blk * kPB + i < pe;
            if (!in) psi = b = beta = 0.0;
            q.fb = b;
            sincospi(2.0 * rs_frac(b * (double)RF), &q.fry, &q.frx);
            q.da = in ? (double)ra : 0.0;
            q.dbase = rs_frac(psi) + rs_frac(b * nc);
            q.dslope = -beta;
            sincospi(2.0 * rs_frac(-beta * (double)RD), &q.dry, &q.drx);
            sPar[blk & 1][i] = q;
        };
        // phasors of step st into buffer st & 1
        auto phasors_d = [&](int st) {
            const pix_par *par = &sPar[(st / kSPB) & 1][(st % kSPB) * kKP];
            double *buf = sX[st & 1];
            const int q = tid / RD, k0 = tid % RD;
            const pix_par &pp = par[q];
            double *dst = buf + q * REC + k0;
            double ph = __builtin_fma(pp.dslope, (double)(l0 + k0), pp.dbase);
            ph = ph - __builtin_floor(ph + 0.5);
            const double tx = pp.drx, ty = pp.dry;
            double s, c;
            sincospi(2.0 * ph, &s, &c);
            const bool per_block = sK.amp_lstride != 0;
            if (!per_block) {
                c *= pp.da;
                s *= pp.da;
            }
            const int64_t p = pb + (int64_t)st * kKP + q;
#pragma unroll
            for (int k = 0; k < RUN; ++k) {
                double ce = c, se = s;
                if (per_block) {
                    const int l = l0 + k0 + RD * k;
                    const double al =
                        p < pe && l < sK.L ? (double)rs_gload(sK.amp, p + (int64_t)l * sK.amp_lstride) : 0.0;
                    ce *= al;
                    se *= al;
                }
                dst[RD * k] = ce;
                dst[TL + RD * k] = se;
                const double cn = __builtin_fma(c, tx, -(s * ty));
                s = __builtin_fma(c, ty, s * tx);
                c = cn;
            }
        };
        auto phasors_f = [&](int st) {
            const pix_par *par = &sPar[(st / kSPB) & 1][(st % kSPB) * kKP];
            double *buf = sX[st & 1];
            const int t = tid - 64 * WF0;
            const int q = t / RF, k0 = t % RF;
            const pix_par &pp = par[q];
            double *dst = buf + q * REC + 2 * TL + k0;
            const double tx = pp.frx, ty = pp.fry;
            double s, c;
            sincospi(2.0 * rs_frac(pp.fb * ((double)(h0 + k0) + hofs)), &s, &c);
#pragma unroll
            for (int k = 0; k < RUN; ++k) {
                dst[RF * k] = c;
                dst[NH + RF * k] = s;
                const double cn = __builtin_fma(c, tx, -(s * ty));
                s = __builtin_fma(c, ty, s * tx);
                c = cn;
            }
        };

        d4 acc[RB][CB];
#pragma unroll
        for (int i = 0; i < RB; ++i)
#pragma unroll
            for (int j = 0; j < CB; ++j) acc[i][j] = d4{0.0, 0.0, 0.0, 0.0};

        // operand of this lane: pixel lane / 16 of a group of four, index
        // lane % 16 of a block of 16
        const int obase = (lane >> 4) * REC + (lane & 15);
        const int pidx = tid - 64 * (NW - WP);  // parameter threads
        // Iteration st multiplies step st and evaluates step st + 1; -2 is the
        // first parameter block (by the first 256 threads), -1 the first
        // step's phasors.  D comes before the products (waves 0..), F and the
        // parameters after them (with 8 waves in the second wave of a SIMD): a
        // vector instruction issues every ~38 cycles beside the other wave's
        // matrix instructions and costs them nothing, so each wave's vector
        // part runs under the other's products.  One call site each: the
        // binary64 sincospi code is long.
        for (int st = -2; st < nsteps; ++st) {
            if (wave < WD && st >= -1 && st + 1 < nsteps) phasors_d(st + 1);
            if (st >= 0) {
                const double *op = sX[st & 1] + obase;
#pragma unroll
                for (int t = 0; t < kKP / 4; ++t) {
                    double d[RB], f[CB];
#pragma unroll
                    for (int i = 0; i < RB; ++i)
                        d[i] = op[4 * t * REC + (i / (RB / 2)) * TL + wl * LW + (i % (RB / 2)) * 16];
#pragma unroll
                    for (int j = 0; j < CB; ++j)
                        f[j] = op[4 * t * REC + 2 * TL + (j / (CB / 2)) * NH + wh * HW + (j % (CB / 2)) * 16];
#pragma unroll
                    for (int i = 0; i < RB; ++i)
#pragma unroll
                        for (int j = 0; j < CB; ++j)
                            acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(d[i], f[j], acc[i][j], 0, 0, 0);
                }
            }
            if (wave >= WF0 && wave < WF0 + WF && st >= -1 && st + 1 < nsteps) phasors_f(st + 1);
            int blk = 0, i = tid;
            bool par = st == -2 && tid < kPB;
            if (par) fetch(pb + i);
            if (st >= 0 && wave >= NW - WP) {
                // the next block: round j of PR loads at step 4 j and is
                // evaluated two steps later
                const int ph = st % kSPB;
                blk = st / kSPB + 1;
                i = pidx + (ph >> 2) * 64 * WP;
                const bool now = ph < 4 * PR && blk * kSPB < nsteps;
                if (now && (ph & 3) == 0) fetch(pb + (int64_t)blk * kPB + i);
                par = now && (ph & 3) == 2;
            }
            if (par) params(blk, i);
            __syncthreads();
        }

        double2 *out = reinterpret_cast<double2 *>(J.partial) +
                       ((int64_t)it.s * (J.M * J.N) + it.c) * (int64_t)J.L * J.Ns;
#pragma unroll
        for (int i = 0; i < RB / 2; ++i)
#pragma unroll
            for (int j = 0; j < CB / 2; ++j) {
                const int h = h0 + wh * HW + j * 16 + (lane & 15);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int l = l0 + wl * LW + i * 16 + 4 * e + (lane >> 4);
                    if (h < nh && l < J.L) {
                        const double cr = acc[i][j][e], ci = acc[i + RB / 2][j][e];
                        const double sr = acc[i][j + CB / 2][e], si = acc[i + RB / 2][j + CB / 2][e];
                        double2 *row = out + (int64_t)l * J.Ns;
                        row[J.Ns - nh + h] = make_double2(cr - si, ci + sr);
                        row[nh - 1 - h] = make_double2(cr + si, ci - sr);
                    }
                }
            }
    }
}

}  // namespace

void rs_launch_plain(const rs_launch &L, int tn, int tl, int grid, hipStream_t st)
{
    if (tl == 128)
        hipLaunchKernelGGL((k_plain_fp64<64, 128, 8>), dim3(grid), dim3(512), 0, st, L);
    else if (tn == 128)
        hipLaunchKernelGGL((k_plain_fp64<64, 64, 8>), dim3(grid), dim3(512), 0, st, L);
    else
        hipLaunchKernelGGL((k_plain_fp64<32, 32, 4>), dim3(grid), dim3(256), 0, st, L);
}
