// The compositing walk of one wave over a tile's depth-ordered list (Eq. (3),
// the per-pixel loop of Algorithm 1): shared by the compositing kernels.
#pragma once
#include "common.h"

namespace gs {

constexpr double WALK_LOG2E = 1.4426950408889634;
constexpr int WALK_BATCH = 64;  // list entries tested at a time, one per lane
constexpr int WALK_STEP = 4;    // entries evaluated together

// Pixel centres of a wave's 64 pixels of a tile (pixels row-major inside the
// tile, wave w takes 64 w .. 64 w + 63; tile sides are powers of two): first
// and last column and row inside the image.
struct WaveBox {
    double x0, x1, y0, y1;
};

// false: the wave has no pixel inside the image
__device__ __forceinline__ bool wave_box(int wave, int txi, int tyi, int tw, int th, int H, int W, WaveBox& b)
{
    const int k0 = 64 * wave;
    if (k0 >= tw * th) return false;
    const int xs = tw >= 64 ? k0 % tw : 0, nx = tw >= 64 ? 64 : tw;
    const int ys = k0 / tw, ny = tw >= 64 ? 1 : 64 / tw;
    const int c0 = txi * tw + xs, r0 = tyi * th + ys;
    if (c0 >= W || r0 >= H) return false;
    b.x0 = c0 + 0.5;
    b.x1 = min(c0 + nx, W) - 0.5;
    b.y0 = r0 + 0.5;
    b.y1 = min(r0 + ny, H) - 0.5;
    return true;
}

// Whether entry r can reach alpha_min at some pixel of the box: the least
// value of its conic form over the box against 2 ln(sigma / alpha_min).  The
// 0.01 of slack (half a percent of alpha) is far above the roundings here
// and in the walk's own alpha, so an entry left out is one that every pixel
// of the box skips.  plain: no pixel of the box wraps its azimuth offset.
__device__ __forceinline__ bool box_reached(const GRec& r, const WaveBox& b, double W, float amin, bool& plain)
{
    double xl = b.x0 - r.px, xh = b.x1 - r.px;
    const double half = 0.5 * W;
    const double shift = xl >= half ? -W : (xh < -half ? W : 0.0);
    plain = xl >= -half && xh < half;
    if (!plain && shift == 0.0) return true;  // the pixels disagree about the wrap
    xl += shift;
    xh += shift;
    const double yl = b.y0 - r.py, yh = b.y1 - r.py;
    // the face of the box nearest the centre, on each axis the centre is
    // outside of: the minimum lies on one of those faces
    const double xe = xl > 0.0 ? xl : (xh < 0.0 ? xh : 0.0);
    const double ye = yl > 0.0 ? yl : (yh < 0.0 ? yh : 0.0);
    const double ys = fmin(fmax(-r.cb * xe * __builtin_amdgcn_rcp(r.cc), yl), yh);
    const double xs = fmin(fmax(-r.cb * ye * __builtin_amdgcn_rcp(r.ca), xl), xh);
    const double qx = r.ca * xe * xe + 2.0 * r.cb * xe * ys + r.cc * ys * ys;
    const double qy = r.ca * xs * xs + 2.0 * r.cb * xs * ye + r.cc * ye * ye;
    const bool ux = xe != 0.0, uy = ye != 0.0;
    const double qmin = ux ? (uy ? fmin(qx, qy) : qx) : (uy ? qy : 0.0);
    const float qmax = 1.3862943611f * __builtin_amdgcn_logf(r.sigma / amin);  // 2 ln 2 log2()
    return !(qmin > (double)qmax + 0.01);
}

// A queued entry: the record with 2 cb in place of cb (an exact doubling).
struct alignas(16) WalkRec {
    double px, py, ca, cb2, cc;
    float sigma, att;
};

// alpha of an entry at the pixel centre (pcx, pcy); PLAIN: no wrap here
template <bool PLAIN>
__device__ __forceinline__ float walk_alpha(const WalkRec& r, double pcx, double pcy, double half, double W, float amax)
{
    double dx = pcx - r.px;
    if constexpr (!PLAIN) dx += dx >= half ? -W : (dx < -half ? W : 0.0);
    const double dy = pcy - r.py;
    const double qv = r.ca * dx * dx + r.cb2 * dx * dy + r.cc * dy * dy;
    const float G = __builtin_amdgcn_exp2f((float)(-0.5 * WALK_LOG2E * qv));
    return fminf(amax, r.sigma * G);
}

// A pixel's state along the walk.
struct WalkState {
    float T;
    float thr;           // alpha_min while the pixel walks, infinity once it has stopped
    uint32_t last, cnt;  // list position behind the last entry taken; entries taken
};

__device__ __forceinline__ bool walk_done(const WalkState& p) { return __ballot(p.thr < INFINITY) == 0ull; }

// Applies one entry: its weight at the pixel (0 where it is skipped), T, the
// stop before an entry that would take T below tmin.
__device__ __forceinline__ float walk_apply(WalkState& p, float alpha, float att, uint32_t pos, float tmin)
{
    const float Tn = p.T * (1.0f - alpha);
    const bool hit = alpha >= p.thr;
    const bool low = Tn < tmin;
    const bool take = hit && !low;
    const float w = take ? p.T * alpha * att : 0.0f;
    p.thr = hit && low ? INFINITY : p.thr;
    p.T = take ? Tn : p.T;
    p.last = take ? pos : p.last;
    p.cnt += take ? 1u : 0u;
    return w;
}

// A wave's entries of the current batch that reach its box, in list order.
struct alignas(16) WalkQueue {
    WalkRec rec[WALK_BATCH];
    uint32_t pos[WALK_BATCH];  // list position + 1
    uint32_t g[WALK_BATCH];
};

__device__ __forceinline__ void walk_wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Queues the lanes' entries (valid ones) that reach the box, pads the queue
// to a multiple of WALK_STEP with entries no pixel takes (sigma 0), and
// returns the number queued; slot: the lane's place, or -1; plain: no queued
// entry's offset wraps at any pixel of the box.
__device__ __forceinline__ int walk_queue(WalkQueue& Q, const GRec& r, uint32_t g, uint32_t pos, bool valid,
                                          const WaveBox& b, double W, float amin, int lane, int& slot, bool& plain)
{
    bool pl;
    const bool keep = box_reached(r, b, W, amin, pl) && valid;
    const unsigned long long m = __ballot(keep);
    plain = __ballot(keep && !pl) == 0ull;
    const int n = __popcll(m);
    slot = keep ? __popcll(m & ((1ull << lane) - 1ull)) : -1;
    if (keep) {
        Q.rec[slot] = WalkRec{r.px, r.py, r.ca, 2.0 * r.cb, r.cc, r.sigma, r.att};
        Q.pos[slot] = pos;
        Q.g[slot] = g;
    }
    const int pad = (n + WALK_STEP - 1) / WALK_STEP * WALK_STEP;
    const uint32_t g0 = __builtin_amdgcn_readlane(g, m ? __ffsll(m) - 1 : 0);
    if (lane >= n && lane < pad) {
        // (the Gaussian of a queued entry: its attributes may be read, times 0)
        Q.rec[lane] = WalkRec{};
        Q.pos[lane] = 0u;
        Q.g[lane] = g0;
    }
    return n;
}

// The alphas of WALK_STEP queued entries from j on at the lane's pixel: the
// records first, then the evaluations (independent of each other).
template <bool PLAIN>
__device__ __forceinline__ void walk_alphas(const WalkQueue& Q, int j, double pcx, double pcy, double half, double W,
                                            float amax, float* al)
{
    WalkRec r[WALK_STEP];
#pragma unroll
    for (int i = 0; i < WALK_STEP; ++i) r[i] = Q.rec[j + i];
#pragma unroll
    for (int i = 0; i < WALK_STEP; ++i) al[i] = walk_alpha<PLAIN>(r[i], pcx, pcy, half, W, amax);
}

// Their weights: the alphas, then the chain.
template <bool PLAIN>
__device__ __forceinline__ void walk_step(const WalkQueue& Q, int j, WalkState& p, double pcx, double pcy, double half,
                                          double W, float amax, float tmin, float* w)
{
    walk_alphas<PLAIN>(Q, j, pcx, pcy, half, W, amax, w);
#pragma unroll
    for (int i = 0; i < WALK_STEP; ++i) w[i] = walk_apply(p, w[i], Q.rec[j + i].att, Q.pos[j + i], tmin);
}

}  // namespace gs
