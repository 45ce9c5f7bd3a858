// Synthetic scenes on the device: each pixel of a g_az x g_el grid casts a
// ray from the origin into an axis-aligned room and an optional ellipsoid
// pedestrian (the stand-in for the rendered image whose pixels the paper
// turns into scatterers, Sec. II).  A thread takes one pixel of a few
// frames: its ray direction (two binary64 sincospi) and the reciprocals of its
// components are shared by them; what depends on the frame alone (half sides,
// reciprocal semi-axes, the centre in units of them) comes from the host.
// binary64 geometry, float32 structure-of-arrays output (20 bytes written
// and 4 read per pixel and frame).
//
// The frames travel in the kernel arguments, kFramesPerLaunch a launch: no
// allocation, no copy and no wait for one (a pageable copy held the caller
// until the previous call's kernel had finished).  Measured on 100 frames of
// 256 x 256 (157 MB, 33 us at a copy's rate): 53 us a call back to back, against
// 74 us for one launch behind the copy with three to nine binary64 divisions a
// frame (25.3e6 vector instructions, 13.5e6 now).
#include "rs_api_internal.h"

#include <algorithm>
#include <cmath>
#include <cstring>

namespace {

constexpr int kFramesPerThread = 4;   // frames one thread casts along its pixel's ray
constexpr int kFramesPerLaunch = 28;  // frames in the arguments of one launch (4 KiB in all)

// One frame: half room sides, reciprocal semi-axes, o = -centre / semi-axes,
// cc = |o|^2 - 1, centre and velocity of the pedestrian.
struct frame {
    double hw, d, hh;
    double is[3], o[3], cc, c[3], v[3];
    int64_t ped;
};
struct frames {
    frame f[kFramesPerLaunch];
};
static_assert(sizeof(frames) + 128 <= 4096, "kernel arguments");

// The ray of one pixel (direction u, ru[k] = 1 / u[k]) against one frame's room
// and pedestrian; writes the pixel's scatterer at index g of the output arrays.
__device__ __forceinline__ void cast(const frame &S, const double (&u)[3], const double (&ru)[3], int64_t g,
                                     const float *noise, float *ox, float *oy, float *oz, float *oamp, float *ovr)
{
    // nearest wall: planes x = +-W/2, y = D, z = +-H/2 (1 / 0 = inf: no hit)
    const double tx = S.hw * fabs(ru[0]);
    const double ty = u[1] > 0 ? S.d * ru[1] : __builtin_huge_val();
    const double tz = S.hh * fabs(ru[2]);
    double t = tx, cosi = fabs(u[0]);
    if (ty < t) {
        t = ty;
        cosi = fabs(u[1]);
    }
    if (tz < t) {
        t = tz;
        cosi = fabs(u[2]);
    }
    double v = 0.0;
    if (S.ped) {
        // |(t u - c) / s| = 1:  a t^2 + b t + cc = 0 with d = u / s, o = -c / s
        double d[3];
        for (int k = 0; k < 3; ++k) d[k] = u[k] * S.is[k];
        const double a = d[0] * d[0] + d[1] * d[1] + d[2] * d[2];
        const double b = 2.0 * (d[0] * S.o[0] + d[1] * S.o[1] + d[2] * S.o[2]);
        const double disc = b * b - 4.0 * a * S.cc;
        if (disc > 0) {
            const double sq = sqrt(disc);
            const double t1 = (-b - sq) / (2.0 * a), t2 = (-b + sq) / (2.0 * a);
            const double te = t1 > 0 ? t1 : t2;
            if (te > 0 && te < t) {
                // outward normal (x - c) / s^2 at the hit, normalised
                double nrm[3], nn = 0.0;
                for (int k = 0; k < 3; ++k) {
                    nrm[k] = (u[k] * te - S.c[k]) * (S.is[k] * S.is[k]);
                    nn += nrm[k] * nrm[k];
                }
                nn = sqrt(nn);
                t = te;
                cosi = fabs((u[0] * nrm[0] + u[1] * nrm[1] + u[2] * nrm[2]) / nn);
                v = -(u[0] * S.v[0] + u[1] * S.v[1] + u[2] * S.v[2]);
            }
        }
    }
    const double nz = noise ? (double)noise[g] : 1.0;
    ox[g] = (float)(u[0] * t);
    oy[g] = (float)(u[1] * t);
    oz[g] = (float)(u[2] * t);
    oamp[g] = (float)(cosi / (t * t) * nz);
    ovr[g] = (float)v;
}

// Thread = (pixel p, group blockIdx.y of kFramesPerThread frames): the pixel's
// ray direction is evaluated once and cast into each frame of the group.
// Frame f of the launch is frame first + f of the call.
__global__ __launch_bounds__(256) void k_render(const frames fr, int64_t P, int first, int nframes, int g_az, int g_el,
                                                const float *noise, float *ox, float *oy, float *oz, float *oamp,
                                                float *ovr)
{
    const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (p >= P) return;
    const int f0 = blockIdx.y * kFramesPerThread;
    const int i = (int)(p % g_az), j = (int)(p / g_az);
    // ray direction of the pixel centre (angles in degrees / 180 = half turns)
    const double az = (-60.0 + 120.0 * ((double)i + 0.5) / (double)g_az) / 180.0;
    const double el = (-30.0 + 60.0 * ((double)j + 0.5) / (double)g_el) / 180.0;
    double saz, caz, sel, cel;
    sincospi(az, &saz, &caz);
    sincospi(el, &sel, &cel);
    const double u[3] = {cel * saz, cel * caz, sel};
    const double ru[3] = {1.0 / u[0], 1.0 / u[1], 1.0 / u[2]};
    const int f1 = min(nframes, f0 + kFramesPerThread);
    for (int f = f0; f < f1; ++f) cast(fr.f[f], u, ru, (int64_t)(first + f) * P + p, noise, ox, oy, oz, oamp, ovr);
}

bool pos_finite(double v) { return std::isfinite(v) && v > 0.0; }

}  // namespace

extern "C" rs_status rs_render_scenes(const rs_scene *scenes, int32_t nframes, int32_t g_az, int32_t g_el,
                                      const float *noise, float *x, float *y, float *z, float *amp, float *vr,
                                      void *stream)
{
    if (nframes < 0) return rs_fail(RS_E_INVALID, "nframes < 0");
    if (nframes == 0) return RS_OK;
    if (!scenes || !x || !y || !z || !amp || !vr) return rs_fail(RS_E_INVALID, "NULL scene or output array");
    if (g_az < 1 || g_el < 1) return rs_fail(RS_E_INVALID, "grid sides must be >= 1");
    const int64_t P = (int64_t)g_az * g_el;
    if (P * nframes > ((int64_t)1 << 31)) return rs_fail(RS_E_INVALID, "more than 2^31 pixels");
    for (int f = 0; f < nframes; ++f) {
        const rs_scene &S = scenes[f];
        if (!pos_finite(S.room_w) || !pos_finite(S.room_d) || !pos_finite(S.room_h))
            return rs_fail(RS_E_INVALID, "frame %d: room sides must be finite and > 0", f);
        if (S.pedestrian)
            for (int k = 0; k < 3; ++k)
                if (!pos_finite(S.semi_axes[k]) || !std::isfinite(S.centre[k]) || !std::isfinite(S.velocity[k]))
                    return rs_fail(RS_E_INVALID, "frame %d: bad pedestrian", f);
    }
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    const bool timed = rs_timer_begin(st);
    for (int first = 0; first < nframes; first += kFramesPerLaunch) {
        const int n = std::min(kFramesPerLaunch, nframes - first);
        frames fr;
        std::memset(&fr, 0, sizeof fr);
        for (int f = 0; f < n; ++f) {
            const rs_scene &S = scenes[first + f];
            frame &q = fr.f[f];
            q.hw = S.room_w / 2;
            q.d = S.room_d;
            q.hh = S.room_h / 2;
            q.ped = S.pedestrian != 0;
            if (!q.ped) continue;
            for (int k = 0; k < 3; ++k) {
                q.is[k] = 1.0 / S.semi_axes[k];
                q.o[k] = -S.centre[k] / S.semi_axes[k];
                q.cc += q.o[k] * q.o[k];
                q.c[k] = S.centre[k];
                q.v[k] = S.velocity[k];
            }
            q.cc -= 1.0;
        }
        hipLaunchKernelGGL(k_render, dim3((unsigned)((P + 255) / 256), (unsigned)((n + kFramesPerThread - 1) / kFramesPerThread)),
                           dim3(256), 0, st, fr, P, first, n, g_az, g_el, noise, x, y, z, amp, vr);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return rs_fail(RS_E_DEVICE, "render launch: %s", hipGetErrorString(e));
    }
    if (timed) rs_timer_end(st);
    return RS_OK;
}
