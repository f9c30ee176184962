// Backward of the front-to-back compositing (Eq. (3)), one workgroup per
// (64 pixels of a tile, channel group, attribute set).
//
// With c_k = a_k sum_f g_f v_{k,f} (g = dL/dout of the pixel, summed over
// the group's channels) and T_k the transmittance in front of entry k:
//   dL/dv_{k,f}   = T_k alpha_k a_k g_f
//   dL/dalpha_k   = T_k c_k - R_k / (1 - alpha_k),  R_k = sum_{m>k} T_m alpha_m c_m
//   dL/da_k       = T_k alpha_k sum_f g_f v_{k,f}
// R_k = D - P_k with D = sum_f g_f out_f (the forward output) and P_k the
// running prefix, so the list is re-walked front to back, recomputing alpha
// and T instead of storing them; the walk ends at the pixel's recorded stop
// position.  alpha = min(alpha_max, sigma G): a clamped pair passes no
// gradient to sigma or G.  Through G = exp(-q/2) and the conic quadratic
// form q the gradient reaches the pixel-space centre and the conic.
//
// Per list entry the per-pixel terms are summed over the wave by a
// butterfly reduce-scatter (every lane ends with one summed value) and leave
// by atomics into a per-pair accumulator (only the workgroups of one tile
// share an address) that a second pass folds into the per-Gaussian sums and
// the attribute gradients.  The nearest Gaussians cover every tile, so
// per-Gaussian atomics of every 64 pixels would serialise on a few addresses
// and add thousands of terms to one running FP32 sum.
#include <type_traits>

#include "common.h"
#include "walk.h"

namespace gs {

constexpr double LOG2E_B = 1.4426950408889634;

// The same reduce-scatter for 8 values without the LDS crossbar: lane
// halves and quarter rows are exchanged with v_permlane32_swap /
// v_permlane16_swap (each swap also moves the partner's half, so one add
// completes a stage), the xor-8 stage and the final sum over 8 lanes use
// DPP row rotations and quad permutations.  Lane l ends with the wave
// total of value l >> 3 in x[0].
// (every lane has a source lane in these patterns; old = 0 with bound_ctrl
// lets the compiler fold the move into the add as a DPP operand)
__device__ __forceinline__ float dpp_f(float v, int ctrl_sel)
{
    const int iv = __float_as_int(v);
    int r;
    switch (ctrl_sel) {
        case 0: r = __builtin_amdgcn_update_dpp(0, iv, 0x128, 0xF, 0xF, true); break;  // row_ror:8
        case 1: r = __builtin_amdgcn_update_dpp(0, iv, 0xB1, 0xF, 0xF, true); break;   // quad_perm [1,0,3,2]
        case 2: r = __builtin_amdgcn_update_dpp(0, iv, 0x4E, 0xF, 0xF, true); break;   // quad_perm [2,3,0,1]
        default: r = __builtin_amdgcn_update_dpp(0, iv, 0x141, 0xF, 0xF, true); break; // row_half_mirror
    }
    return __int_as_float(r);
}

__device__ __forceinline__ void wave_reduce_scatter8(float* x, int lane)
{
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x[i]), __float_as_uint(x[i + 4]), false, false);
        x[i] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x[i]), __float_as_uint(x[i + 2]), false, false);
        x[i] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
    const float t0 = x[0] + dpp_f(x[0], 0), t1 = x[1] + dpp_f(x[1], 0);
    float v = (lane & 8) ? t1 : t0;
    v += dpp_f(v, 1);
    v += dpp_f(v, 2);
    v += dpp_f(v, 3);
    x[0] = v;
}

typedef float f32x4 __attribute__((ext_vector_type(4)));

// Where the attribute gradients of a tile's entries are summed over the tile
// before they go to the Gaussians' rows (pair: the tile's part of the
// per-pair accumulator, 8 floats per list entry, of which the first m entries
// are walked and hold their geometric terms).
//   one value per entry: slot 7 of its 8 floats (the geometric terms are seven)
//   `row` values: behind the walked entries' terms, as many entries from the
//   front as the unwalked ones leave room for; the entries behind those add
//   straight to the Gaussians' rows.  Lists are mostly far longer than their
//   walks (thousands against tens), so that is rare; the front entries, the
//   nearest Gaussians, are those that most tiles add to.
// 12,000 Gaussians, 16 receivers of one channel at 45 x 180: rms error of the
// attribute gradients 2.2e-7 against 64 bits with every 64 pixels added
// straight, 1.05e-7 so; 50,000 Gaussians at 90 x 360: 484 us a fit either way.
struct PairAttr {
    int row;    // values per entry over all sets that share the accumulator; 0: none
    int slot7;  // the one value is in slot 7
    __device__ uint32_t entries(uint32_t m, uint32_t len) const
    {
        if (slot7) return m;
        const unsigned long long room = (unsigned long long)(len - m) * 8u;
        return row ? (uint32_t)min((unsigned long long)m, room / (uint32_t)row) : 0u;
    }
    __device__ size_t at(uint32_t m, uint32_t e) const
    {
        return slot7 ? (size_t)e * 8 + 7 : (size_t)m * 8 + (size_t)e * (uint32_t)row;
    }
};

constexpr int BWD_WAVES = 4;                      // waves that share 64 pixels
constexpr int BWD_SUB = WALK_BATCH / BWD_WAVES;   // entries of a batch per wave, at most

// A queued entry: the walk's record and the FP32 conic for the gradient factors.
struct alignas(16) BwdRec {
    double px, py, ca, cb2, cc;
    float sigma, att;
    float caf, cbf, ccf;
    uint32_t pos, g;  // place in the tile's list; Gaussian
};

// One workgroup per (64 pixels of a tile, channel group, set).  Walks are
// short (40 - 70 entries where the opacity saturates) but a few are ten times
// longer, and one wave spends ~900 cycles per entry on the gradient terms and
// their sums over the wave, so a workgroup per tile with a wave per 64 pixels
// lasted as long as its longest walk.  Here four waves share the pixels: per batch of 64
// list entries each tests all against the pixels' box, takes a contiguous
// quarter of those that reach it, forms the transmittance product and the
// prefix sum P of its quarter, and after one exchange knows T and P in front
// of it (P = P_0 + T_0 P_local).  The sums go to memory by atomics straight
// from the wave, into the pair's row (PairAttr: attribute gradients too).
// CG >= 16: gv = v . g per (entry, pixel) and the attribute gradient
// dA[e][f] = sum_p w[p][e] g[p][f] are products on the FP32 matrix cores
// (v_mfma_f32_16x16x4_f32), with g and w in LDS; smaller groups reduce over
// the wave with the butterfly.
// 16 receivers of 50,000 Gaussians at 90 x 360, one channel: 258 us with a
// wave per 64 pixels and every entry of the tile walked, 163 us so; 4
// receivers of 20,000, 32 channel floats: 557 us, 116 us so.
template <int CG>
__global__ __launch_bounds__(64 * BWD_WAVES) __attribute__((amdgpu_waves_per_eu(CG == 64 ? 3 : 4))) void k_blend_bwd(
    const GRec* __restrict__ rec, size_t s_rec, const uint32_t* __restrict__ plist, size_t s_plist,
    const uint2* __restrict__ ranges, size_t s_ranges, const float* __restrict__ attr, int64_t a_stride,
    int Fc, int C, int H, int W, int tw, int th, int TX, float amin, float amax,
    const float* __restrict__ out, const float* __restrict__ dout, const float* __restrict__ tgt,
    const float* __restrict__ mgrad, float gscale, const uint32_t* __restrict__ n_last, size_t s_pix,
    float* __restrict__ gacc, size_t s_gacc, float* __restrict__ d_attr, int64_t da_stride, int shared_geo,
    PairAttr pa)
{
    constexpr bool MFMA = CG >= 16;
    constexpr int NB = MFMA ? CG / 16 : 1;
    // entries evaluated together: 4 where the registers hold them
    constexpr int BWD_STEP = CG == 1 ? 4 : 2;
    const int npb = tw * th >> 6;  // 64-pixel boxes per tile
    const int tile = blockIdx.x / npb, box_i = blockIdx.x % npb, cg = blockIdx.y, set = blockIdx.z;
    const int q = shared_geo ? 0 : set;
    const int txi = tile % TX, tyi = tile / TX;
    WaveBox box;
    if (!wave_box(box_i, txi, tyi, tw, th, H, W, box)) return;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int t = 64 * box_i + lane;
    const int col = txi * tw + t % tw, row = tyi * th + t / tw;
    const bool inside = col < W && row < H;
    const uint2 rg = ranges[q * s_ranges + tile];
    const double pcx = col + 0.5, pcy = row + 0.5, halfW = 0.5 * W;
    rec += q * s_rec;
    plist += q * s_plist + rg.x;
    gacc += q * s_gacc + (size_t)rg.x * 8;
    const int ch0 = cg * CG, nch = min(CG, Fc - ch0);  // the last group may be partly filled
    const float* A = attr + set * a_stride + ch0;
    float* dA = d_attr + set * da_stride + ch0;
    const size_t HW = (size_t)H * W, pix = inside ? (size_t)row * W + col : 0;
    const int F = Fc / C;

    __shared__ BwdRec s_ent[BWD_WAVES][BWD_SUB];
    __shared__ float s_tp[2][BWD_WAVES][2][64];  // T product and P of a wave's quarter (two batches)
    __shared__ float s_g[MFMA ? CG : 1][MFMA ? 65 : 1];  // g, rows padded
    __shared__ float s_v[MFMA ? 1 : BWD_WAVES][MFMA ? 1 : BWD_SUB][MFMA ? 1 : CG];  // attribute rows of the queue
    // gv of the queue from the matrix cores, replaced by the pixel weights w
    __shared__ float s_w[MFMA ? BWD_WAVES : 1][MFMA ? BWD_SUB : 1][65];

    const uint32_t stop = inside ? n_last[q * s_pix + pix] : 0u;
    // the walk ends at the largest stop position of the pixels; m: of the tile's
    uint32_t nent, m = 0u;
    {
        __shared__ uint32_t s_m[BWD_WAVES];
        const int tt = threadIdx.x, tc = txi * tw + tt % tw, tr = tyi * th + tt / tw;
        uint32_t x = tt < tw * th && tc < W && tr < H ? n_last[q * s_pix + (size_t)tr * W + tc] : 0u;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) x = max(x, (uint32_t)__shfl_xor((int)x, o, 64));
        if (lane == 0) s_m[wave] = x;
        __syncthreads();
        nent = __builtin_amdgcn_readfirstlane(s_m[box_i]);
#pragma unroll
        for (int w = 0; w < BWD_WAVES; ++w) m = max(m, s_m[w]);
        m = __builtin_amdgcn_readfirstlane(min(m, rg.y - rg.x));
    }
    if (nent == 0) return;
    const uint32_t na = pa.entries(m, rg.y - rg.x);
    // the first channel of the group in entry 0's row, and the floats from
    // one entry's to the next
    float* const pv = gacc + pa.at(m, 0) + (shared_geo && da_stride ? (size_t)set * Fc : 0) + ch0;
    const uint32_t pstep = pa.slot7 ? 8u : (uint32_t)pa.row;

    // dL/dout of the pixel's channel ch0 + k: the elementwise part (read, or
    // formed from the output and the target) + the set's channel-mean term;
    // and D = g . out
    auto upstream = [&](int k, float& o) -> float {
        const int ch = ch0 + min(k, nch - 1);
        const int f = ch / C, comp = ch - f * C;
        const size_t idx = (((size_t)set * F + f) * HW + pix) * C + comp;
        o = out[idx];
        const float g = (tgt ? gscale * (o - tgt[idx]) : dout[idx]) + (mgrad ? mgrad[(size_t)set * Fc + ch] : 0.0f);
        return inside && k < nch ? g : 0.0f;
    };
    float gch[MFMA ? 1 : CG];
    float D = 0.0f;
    if constexpr (MFMA) {
        // each wave a quarter of the channels, shared through LDS
        constexpr int CW = CG / BWD_WAVES;
        float gk[CW], ok[CW];
#pragma unroll
        for (int k = 0; k < CW; ++k) gk[k] = upstream(wave * CW + k, ok[k]);
#pragma unroll
        for (int k = 0; k < CW; ++k) {
            s_g[wave * CW + k][lane] = gk[k];
            D += inside && wave * CW + k < nch ? gk[k] * ok[k] : 0.0f;
        }
        s_tp[0][wave][0][lane] = D;
        __syncthreads();
        D = 0.0f;
#pragma unroll
        for (int w = 0; w < BWD_WAVES; ++w) D += s_tp[0][w][0][lane];
    } else {
        float ok[CG];
#pragma unroll
        for (int k = 0; k < CG; ++k) gch[k] = upstream(k, ok[k]);
#pragma unroll
        for (int k = 0; k < CG; ++k) D += inside && k < nch ? gch[k] * ok[k] : 0.0f;
    }

    float T = 1.0f, P = 0.0f;  // in front of the batch
    uint32_t gn = 0;
    GRec rn{};
    auto fetch = [&](uint32_t b0) {
        const uint32_t i = b0 + lane;
        gn = i < nent ? plist[i] : gn;
        rn = rec[gn];
    };
    gn = plist[0];
    fetch(0);
    int buf = 1;
    for (uint32_t b0 = 0; b0 < nent; b0 += WALK_BATCH, buf ^= 1) {
        // the wave's quarter of the entries that reach the pixels
        const GRec r = rn;
        const uint32_t g = gn;
        bool pl;
        const bool keep = box_reached(r, box, W, amin, pl) && b0 + lane < nent;
        const unsigned long long km = __ballot(keep);
        const bool plain = __ballot(keep && !pl) == 0ull;
        const int n = __popcll(km);
        const int per = ((n + BWD_WAVES - 1) / BWD_WAVES + BWD_STEP - 1) / BWD_STEP * BWD_STEP;
        const int n0 = min(n, wave * per), cnt = min(n, n0 + per) - n0;  // uniform
        const int slot = __popcll(km & ((1ull << lane) - 1ull)) - n0;
        if (keep && slot >= 0 && slot < cnt) {
            s_ent[wave][slot] = BwdRec{r.px, r.py, r.ca, 2.0 * r.cb, r.cc, r.sigma, r.att, (float)r.ca, (float)r.cb,
                                       (float)r.cc, b0 + lane, g};
            if constexpr (!MFMA) {
#pragma unroll
                for (int k = 0; k < CG; ++k) s_v[wave][slot][k] = k < nch ? A[(size_t)g * Fc + k] : 0.0f;
            }
        }
        walk_wave_sync();
        if (b0 + WALK_BATCH < nent) fetch(b0 + WALK_BATCH);
        if constexpr (MFMA) {
            if (cnt > 0) {
                // gv[e][p] = sum_f v[e][f] g[p][f]: A = v rows (lane: entry
                // lane % 16, channel 4k + lane / 16), B = g^T (channel
                // 4k + lane / 16, pixel 16 pb + lane % 16)
                const int e = lane & 15;
                const bool ev = e < cnt;
                const float* vr = A + (size_t)s_ent[wave][ev ? e : 0].g * Fc + (lane >> 4);
                float va[CG / 4];
#pragma unroll
                for (int k = 0; k < CG / 4; ++k) va[k] = ev && 4 * k + (lane >> 4) < nch ? vr[4 * k] : 0.0f;
                f32x4 gv4[4];
#pragma unroll
                for (int pb = 0; pb < 4; ++pb) gv4[pb] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int k = 0; k < CG / 4; ++k)
#pragma unroll
                    for (int pb = 0; pb < 4; ++pb)
                        gv4[pb] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                            va[k], s_g[4 * k + (lane >> 4)][16 * pb + (lane & 15)], gv4[pb], 0, 0, 0);
                // lane holds entries 4 (lane / 16) + r of pixel 16 pb + lane % 16
#pragma unroll
                for (int pb = 0; pb < 4; ++pb)
#pragma unroll
                    for (int rr = 0; rr < 4; ++rr) s_w[wave][4 * (lane >> 4) + rr][16 * pb + (lane & 15)] = gv4[pb][rr];
                walk_wave_sync();
            }
        }
        auto value = [&](int e) -> float {  // v . g of queue entry e
            if constexpr (MFMA) return s_w[wave][e][lane];
            float gv = 0.0f;
#pragma unroll
            for (int k = 0; k < (MFMA ? 1 : CG); ++k) gv = fmaf(gch[k], s_v[wave][e][k], gv);
            return gv;
        };
        auto offset = [&](const BwdRec& br, double& dx, double& dy) {
            dx = pcx - br.px;
            if (!plain) dx += dx >= halfW ? -(double)W : (dx < -halfW ? (double)W : 0.0);
            dy = pcy - br.py;
        };
        // G where the pixel takes the entry, else -1, and the quarter's T and P
        float G[BWD_SUB], Tl = 1.0f, Pl = 0.0f;
#pragma unroll
        for (int j = 0; j < BWD_SUB; j += BWD_STEP) {
            if (j >= cnt) break;
            float al[BWD_STEP], cA[BWD_STEP];
#pragma unroll
            for (int i = 0; i < BWD_STEP; ++i) {
                const int e = min(j + i, cnt - 1);
                const BwdRec& br = s_ent[wave][e];
                double dx, dy;
                offset(br, dx, dy);
                const double qv = br.ca * dx * dx + br.cb2 * dx * dy + br.cc * dy * dy;
                const float Gv = __builtin_amdgcn_exp2f((float)(-0.5 * WALK_LOG2E * qv));
                al[i] = fminf(amax, br.sigma * Gv);
                const bool take = j + i < cnt && br.pos < stop && al[i] >= amin;
                G[j + i] = take ? Gv : -1.0f;
                al[i] = take ? al[i] : 0.0f;
                cA[i] = br.att * value(e);
            }
#pragma unroll
            for (int i = 0; i < BWD_STEP; ++i) {
                Pl += Tl * al[i] * cA[i];
                Tl *= 1.0f - al[i];
            }
        }
        s_tp[buf][wave][0][lane] = Tl;
        s_tp[buf][wave][1][lane] = Pl;
        __syncthreads();
        float Te = T, Pe = P;  // in front of the quarter
#pragma unroll
        for (int w = 0; w < BWD_WAVES; ++w) {
            if (w == wave) {
                Te = T;
                Pe = P;
            }
            P += T * s_tp[buf][w][1][lane];
            T *= s_tp[buf][w][0][lane];
        }
        // the terms, entry by entry; a pixel that does not take an entry gets
        // Ta = 0, so every term is zero and T, P stay
#pragma unroll
        for (int j = 0; j < BWD_SUB; j += BWD_STEP) {
            if (j >= cnt) break;
            float geo[BWD_STEP][8], wt[BWD_STEP];
#pragma unroll
            for (int i = 0; i < BWD_STEP; ++i) {
                const int e = min(j + i, cnt - 1);
                const BwdRec& br = s_ent[wave][e];
                double dx, dy;
                offset(br, dx, dy);
                const float dxf = (float)dx, dyf = (float)dy, gv = value(e);
                const bool take = !(G[j + i] < 0.0f);
                const float Gv = take ? G[j + i] : 0.0f;
                const float sg = br.sigma * Gv;
                const float al = take ? fminf(amax, sg) : 0.0f;
                const float cA = br.att * gv;
                const float Ta = Te * al;
                Pe += Ta * cA;
                // alpha <= alpha_max < 1; a one-ulp reciprocal is ample here
                const float dalpha = Te * cA - (D - Pe) * __builtin_amdgcn_rcpf(1.0f - al);
                const float dsg = (take && sg < amax) ? dalpha : 0.0f;  // clamp passes nothing
                const float dq = -0.5f * dsg * br.sigma * Gv;
                const float w = Ta * br.att;
                // gradient factors in FP32 from the exact offsets
                const float dq2 = -2.0f * dq;
                geo[i][0] = dq2 * fmaf(br.caf, dxf, br.cbf * dyf);  // d/dpx
                geo[i][1] = dq2 * fmaf(br.cbf, dxf, br.ccf * dyf);  // d/dpy
                geo[i][2] = dq * (dxf * dxf);                       // d/dA
                geo[i][3] = dq * (2.0f * dxf * dyf);                // d/dB
                geo[i][4] = dq * (dyf * dyf);                       // d/dC
                geo[i][5] = dsg * Gv;                               // d/dsigma
                geo[i][6] = Ta * gv;                                // d/da
                geo[i][7] = CG == 1 ? w * gch[0] : 0.0f;            // d/dv of the only channel
                wt[i] = w;
                Te *= 1.0f - al;
            }
            // the sums over the wave: 8 lanes end with each of an entry's 8
            // terms, and the entries leave from different ones of them
            bool any = false;
#pragma unroll
            for (int i = 0; i < BWD_STEP; ++i) {
                if constexpr (MFMA)
                    if (j + i < cnt) s_w[wave][j + i][lane] = wt[i];
                any |= !(G[j + i] < 0.0f);
            }
            if (__ballot(any) == 0ull) continue;
            const BwdRec& be = s_ent[wave][min(j + (lane & (BWD_STEP - 1)), cnt - 1)];
            const uint32_t pos = be.pos;
            auto attr_row = [&]() { return pos < na ? pv + (size_t)pos * pstep : dA + (size_t)be.g * Fc; };
            float v = 0.0f;
#pragma unroll
            for (int i = 0; i < BWD_STEP; ++i) {
                wave_reduce_scatter8(geo[i], lane);
                v = (lane & 7) == i ? geo[i][0] : v;
            }
            if (v != 0.0f) {
                float* p = gacc + (size_t)pos * 8 + (lane >> 3);
                if (CG == 1 && !pa.slot7 && lane >= 56) p = attr_row();
                unsafeAtomicAdd(p, v);
            }
            if constexpr (!MFMA && CG > 1) {
                constexpr int shA = CG == 8 ? 3 : (CG == 4 ? 4 : 5);
                v = 0.0f;
#pragma unroll
                for (int i = 0; i < BWD_STEP; ++i) {
                    float red[CG];
#pragma unroll
                    for (int k = 0; k < CG; ++k) red[k] = wt[i] * gch[k];
                    wave_reduce_scatter<CG>(red, lane);
                    v = (lane & ((1 << shA) - 1)) == i ? red[0] : v;
                }
                if (v != 0.0f && (lane >> shA) < nch) unsafeAtomicAdd(attr_row() + (lane >> shA), v);
            }
        }
        if constexpr (MFMA) {
            if (cnt > 0) {
                // (rows behind cnt hold what the first product left; their
                // sums are not used)
                walk_wave_sync();
                // (in CH chains of 16 / CH steps that are then added, as many
                // as the registers hold: one chain rounds as often as the
                // sum over the pixels is long)
                constexpr int CH = NB == 1 ? 8 : (NB == 2 ? 4 : 2);
                f32x4 part[CH][NB], acc[NB];
#pragma unroll
                for (int st = 0; st < 16; ++st) {
                    const float a = s_w[wave][lane & 15][4 * st + (lane >> 4)];
                    const int h = st % CH;
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb)
                        part[h][nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                            a, s_g[16 * nb + (lane & 15)][4 * st + (lane >> 4)],
                            st < CH ? f32x4{0.0f, 0.0f, 0.0f, 0.0f} : part[h][nb], 0, 0, 0);
                }
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
#pragma unroll
                    for (int d = 1; d < CH; d *= 2)
#pragma unroll
                        for (int h = 0; h < CH; h += 2 * d) part[h][nb] += part[h + d][nb];
                    acc[nb] = part[0][nb];
                }
                // lane holds entries 4 (lane / 16) + r, channel 16 nb + lane % 16
#pragma unroll
                for (int rr = 0; rr < 4; ++rr) {
                    const int e = 4 * (lane >> 4) + rr;
                    if (e < cnt) {
                        const BwdRec& be = s_ent[wave][e];
                        float* p = (be.pos < na ? pv + (size_t)be.pos * pstep : dA + (size_t)be.g * Fc) + (lane & 15);
#pragma unroll
                        for (int nb = 0; nb < NB; ++nb)
                            if (acc[nb][rr] != 0.0f && 16 * nb + (lane & 15) < nch) unsafeAtomicAdd(p + 16 * nb, acc[nb][rr]);
                    }
                }
            }
        }
        walk_wave_sync();
    }
}

// ---------------------------------------------------------------------------
// Backward over attribute sets that share one geometry (one prepared query,
// S attribute sets: the transmitter batch of the training step).
//
// T_k, alpha_k, G_k and a_k do not depend on the set, so the per-set terms
// above combine linearly:
//   sum over sets and channels of dL/dalpha_k
//     = T_k a_k GV_k - (D - P_k) / (1 - alpha_k),
//   GV_k = sum_{s,f} g_{s,f} v_{s,k,f},  D = sum_{s,f} g_{s,f} out_{s,f},
//   P_k = sum_{m<=k} T_m alpha_m a_m GV_m,
// and dL/dv_{s,k,f} = w_k g_{s,f} with the set-independent weight
// w_k = T_k alpha_k a_k.  One workgroup takes 64 pixels of a tile and every
// column (set, channel) at once: per batch of entries the matrix cores form
// GV (entries x pixels, contracted over all S*F*c columns), one wave walks
// the pixels' lists once for the geometric terms and the weights, and the
// matrix cores form dL/dv = W^T g (entries x columns, contracted over the
// pixels).  Eight waves split the columns; the geometry is evaluated once
// per (pixel, entry) instead of once per set and channel group.
// ---------------------------------------------------------------------------
constexpr int SG_WAVES = 8;   // column split
constexpr int SG_E = 64;      // entries per batch
constexpr int SG_PIX = 64;    // pixels per workgroup

struct SgUp {  // upstream gradient g = upstream + mean term
    const float* out;
    const float* dout;
    const float* tgt;
    const float* mgrad;
    float scale;
    const float* gscale;  // with tgt: device factor on scale (the mean term carries it already), or null
};

// Raw upstream words of one element: dout, or (out, target) with TGT.
template <bool TGT>
struct SgRaw {
    float a, b;
};
template <bool TGT>
__device__ __forceinline__ SgRaw<TGT> sg_fetch(const SgUp& u, size_t idx)
{
    if constexpr (TGT) return SgRaw<TGT>{u.out[idx], u.tgt[idx]};
    else return SgRaw<TGT>{u.dout[idx], 0.0f};
}
template <bool TGT>
__device__ __forceinline__ float sg_value(const SgUp& u, SgRaw<TGT> r)
{
    if constexpr (TGT) return u.scale * (r.a - r.b);
    else return r.a;
}
// (re, im) or two consecutive real channels at element index idx (even)
template <bool TGT>
__device__ __forceinline__ float2 sg_load2(const SgUp& u, size_t idx)
{
    if constexpr (TGT) {
        const float2 o = *(const float2*)(u.out + idx), t = *(const float2*)(u.tgt + idx);
        return float2{u.scale * (o.x - t.x), u.scale * (o.y - t.y)};
    } else {
        return *(const float2*)(u.dout + idx);
    }
}

// stands in for an absent mean-term vector (read with stride 0)
__device__ const float4 sg_zero4 = {0.0f, 0.0f, 0.0f, 0.0f};

template <int CS, bool TGT>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4))) void k_blend_bwd_sg(
    const GRec* __restrict__ rec, const uint32_t* __restrict__ plist, const uint2* __restrict__ ranges,
    const float* __restrict__ attr, int64_t a_stride, int S, int Fc, int H, int W, int tw_log, int th, int TX,
    float amin, float amax, SgUp up_in, const uint32_t* __restrict__ n_last, float* __restrict__ gacc,
    float* __restrict__ d_attr, int64_t da_stride, int min_walk, float* __restrict__ lacc)
{
    SgUp up = up_in;
    if (TGT && up.gscale) up.scale *= *up.gscale;
    const int tw = 1 << tw_log;
    const int tile = blockIdx.x, pg = blockIdx.y;
    // (wave-uniform values go through readfirstlane so that they live in
    // scalar registers)
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int j4 = lane >> 4, l16 = lane & 15;
    const int txi = tile % TX, tyi = tile / TX;
    const uint2 rg = ranges[tile];
    const size_t HW = (size_t)H * W;
    const int F = Fc >> CS;
    const int ncb = S * Fc / 16;  // 16-column blocks (Fc % 16 == 0)
    const int cb_lo = wave * ncb / SG_WAVES, cb_hi = (wave + 1) * ncb / SG_WAVES;
    // mean term m[s * Fc + c], or zeros
    const float* mg = up.mgrad ? up.mgrad : (const float*)&sg_zero4;
    const size_t mstr = up.mgrad ? 1 : 0;

    // The tile's pixels inside the image (vw x vh, row-major) are packed
    // into groups of 64: edge tiles need fewer groups, and the spare
    // workgroups leave at once.
    const int vw = min(tw, W - txi * tw), vh = min(th, H - tyi * th);
    if (pg * SG_PIX >= vw * vh) return;
    auto pixel_of = [&](int k) -> int {
        return k < vw * vh ? (tyi * th + k / vw) * W + txi * tw + k % vw : -1;
    };

    __shared__ float s_gv[SG_E][SG_PIX + 1];  // GV of the batch
    __shared__ float s_w[SG_E][SG_PIX + 1];   // weights w of the batch
    __shared__ int s_pix[SG_PIX];             // image offset of each pixel of the group (-1 outside)
    __shared__ double s_px[SG_E], s_py[SG_E], s_ca[SG_E], s_cb[SG_E], s_cc[SG_E];
    __shared__ float s_caf[SG_E], s_cbf[SG_E], s_ccf[SG_E], s_sig[SG_E], s_att[SG_E];
    __shared__ uint32_t s_g[SG_E];
    __shared__ float s_D[SG_PIX];
    __shared__ uint32_t s_maxstop;

    // the walking wave's pixel (lane) and its stop position
    const int wpix = pixel_of(pg * SG_PIX + lane);
    const uint32_t stop = (wave == 0 && wpix >= 0) ? n_last[wpix] : 0u;
    if (threadIdx.x == 0) s_maxstop = 0;
    if (threadIdx.x < SG_PIX) {
        s_D[threadIdx.x] = 0.0f;
        s_pix[threadIdx.x] = pixel_of(pg * SG_PIX + threadIdx.x);
    }
    for (int e = threadIdx.x; e < SG_E * (SG_PIX + 1); e += blockDim.x) (&s_gv[0][0])[e] = 0.0f;
    __syncthreads();
    if (stop) atomicMax(&s_maxstop, stop);
    __syncthreads();
    // (min_walk > 0: only groups whose walk is longer than min_walk entries)
    if (min_walk > 0 && s_maxstop <= (uint32_t)min_walk) return;
    const uint32_t end = __builtin_amdgcn_readfirstlane(rg.x + s_maxstop);
    // one batch holds the whole walk of the group (the common case): D is
    // then the walk's own final prefix sum_k w_k GV_k (out = sum_k w_k v_k),
    // else it is formed from the forward output first
    const bool one_batch = end - rg.x <= (uint32_t)SG_E;

    if (end > rg.x && !one_batch) {
        int pixB[4];
#pragma unroll
        for (int pb = 0; pb < 4; ++pb) pixB[pb] = s_pix[16 * pb + l16];
        float dp[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        for (int cb = cb_lo; cb < cb_hi; ++cb) {
            const int s = cb * 16 / Fc;
            const int ch = cb * 16 - s * Fc + 4 * j4;
            float mk[4];
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) mk[kk] = mg[((size_t)s * Fc + ch + kk) * mstr];
            float ls = 0.0f;  // squared error of the block (with lacc)
#pragma unroll
            for (int pb = 0; pb < 4; ++pb) {
                const int px = pixB[pb];
                if (px < 0) continue;
#pragma unroll
                for (int kk = 0; kk < 4; ++kk) {
                    const size_t i = (((size_t)(s * F + ((ch + kk) >> CS)) * HW + px) << CS) + ((ch + kk) & CS);
                    const SgRaw<TGT> raw = sg_fetch<TGT>(up, i);
                    dp[pb] += (sg_value<TGT>(up, raw) + mk[kk]) * up.out[i];
                    if constexpr (TGT) {
                        const float d = raw.a - raw.b;
                        ls = fmaf(d, d, ls);
                    }
                }
            }
            if (TGT && lacc) {
                for (int o = 32; o > 0; o >>= 1) ls += __shfl_xor(ls, o, 64);
                if (lane == 0 && ls != 0.0f) atomicAdd(lacc + s, ls);
            }
        }
#pragma unroll
        for (int pb = 0; pb < 4; ++pb) {
            float v = dp[pb];
            v += __shfl_xor(v, 16, 64);
            v += __shfl_xor(v, 32, 64);
            if (j4 == 0 && cb_hi > cb_lo) atomicAdd(&s_D[16 * pb + l16], v);
        }
    }

    float T = 1.0f, P = 0.0f, D = 0.0f;

    for (uint32_t b0 = rg.x; b0 < end; b0 += SG_E) {
        const int m = (int)min((uint32_t)SG_E, end - b0);
        const int neb = (m + 15) >> 4;
        const bool first = b0 == rg.x;
        if ((int)threadIdx.x < m) {
            const uint32_t g = plist[b0 + threadIdx.x];
            const GRec r = rec[g];
            s_px[threadIdx.x] = r.px;
            s_py[threadIdx.x] = r.py;
            s_ca[threadIdx.x] = r.ca;
            s_cb[threadIdx.x] = r.cb;
            s_cc[threadIdx.x] = r.cc;
            s_caf[threadIdx.x] = (float)r.ca;
            s_cbf[threadIdx.x] = (float)r.cb;
            s_ccf[threadIdx.x] = (float)r.cc;
            s_sig[threadIdx.x] = r.sigma;
            s_att[threadIdx.x] = r.att;
            s_g[threadIdx.x] = g;
        }
        __syncthreads();

        // ---- GV[e][p] = sum over this wave's columns of v[e][c] g[p][c]
        // K-step kk of a 16-column block pairs lane group j4 with channel
        // ch0 + 4 j4 + kk, so each lane reads 4 consecutive channels.
        // NEB = entry blocks of 16 in the batch (a compile-time count keeps
        // the matrix-core sequence free of branches).
        // Wave w takes pixel blocks 2 (w & 1) and 2 (w & 1) + 1 and one of
        // SG_WAVES / 2 column ranges (32 accumulator registers).
        auto gv_phase = [&](auto nebc) {
            constexpr int NEB = decltype(nebc)::value;
            const int ph = wave & 1, cq = wave >> 1;
            const int q_lo = cq * ncb / (SG_WAVES / 2), q_hi = (cq + 1) * ncb / (SG_WAVES / 2);
            int pixB[2];
#pragma unroll
            for (int pb = 0; pb < 2; ++pb) pixB[pb] = s_pix[16 * (2 * ph + pb) + l16];
            f32x4 acc[NEB][2];
#pragma unroll
            for (int eb = 0; eb < NEB; ++eb)
#pragma unroll
                for (int pb = 0; pb < 2; ++pb) acc[eb][pb] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            uint32_t ge[NEB];
#pragma unroll
            for (int eb = 0; eb < NEB; ++eb) {
                const int e = 16 * eb + l16;
                ge[eb] = e < m ? s_g[e] : 0xFFFFFFFFu;
            }
            // Operands of one 16-column block: v of 4 consecutive channels per
            // entry block, the raw upstream words of those channels per pixel
            // block, and the mean terms; the next block's are fetched while
            // this block multiplies (software pipelining).
            constexpr int NR = TGT ? 2 : 1;
            struct Ops {
                float4 a[NEB];
                float b[2][4][NR];
                float4 mm;
            };
            auto load = [&](int cb, Ops& o) {
                const int s = cb * 16 / Fc;
                const int ch = cb * 16 - s * Fc + 4 * j4;
                const float* As = attr + s * a_stride + ch;
#pragma unroll
                for (int eb = 0; eb < NEB; ++eb)
                    o.a[eb] = ge[eb] != 0xFFFFFFFFu ? *(const float4*)(As + (size_t)ge[eb] * Fc)
                                                    : float4{0.0f, 0.0f, 0.0f, 0.0f};
                o.mm = *(const float4*)(mg + ((size_t)s * Fc + ch) * mstr);
#pragma unroll
                for (int pb = 0; pb < 2; ++pb) {
                    const size_t px = pixB[pb] >= 0 ? (size_t)pixB[pb] : 0;
                    if constexpr (CS == 1) {
#pragma unroll
                        for (int h = 0; h < 2; ++h) {
                            const size_t i = ((size_t)(s * F + (ch >> 1) + h) * HW + px) * 2;
                            const float2 u = *(const float2*)(TGT ? up.out + i : up.dout + i);
                            o.b[pb][2 * h][0] = u.x;
                            o.b[pb][2 * h + 1][0] = u.y;
                            if constexpr (TGT) {
                                const float2 t = *(const float2*)(up.tgt + i);
                                o.b[pb][2 * h][NR - 1] = t.x;
                                o.b[pb][2 * h + 1][NR - 1] = t.y;
                            }
                        }
                    } else {
#pragma unroll
                        for (int kk = 0; kk < 4; ++kk) {
                            const size_t i = (size_t)(s * F + ch + kk) * HW + px;
                            o.b[pb][kk][0] = TGT ? up.out[i] : up.dout[i];
                            if constexpr (TGT) o.b[pb][kk][NR - 1] = up.tgt[i];
                        }
                    }
                }
            };
            Ops ops[2];
            if (q_hi > q_lo) load(q_lo, ops[0]);
            for (int cb = q_lo; cb < q_hi; cb += 2) {
#pragma unroll
                for (int half = 0; half < 2; ++half) {
                    const int cc = cb + half;
                    if (cc < q_hi) {
                        if (cc + 1 < q_hi) load(cc + 1, ops[half ^ 1]);
                        __builtin_amdgcn_sched_barrier(0);
                        const Ops& o = ops[half];
                        const float mk[4] = {o.mm.x, o.mm.y, o.mm.z, o.mm.w};
#pragma unroll
                        for (int kk = 0; kk < 4; ++kk) {
                            float bv[2];
#pragma unroll
                            for (int pb = 0; pb < 2; ++pb) {
                                const float u = TGT ? up.scale * (o.b[pb][kk][0] - o.b[pb][kk][NR - 1]) : o.b[pb][kk][0];
                                bv[pb] = pixB[pb] >= 0 ? u + mk[kk] : 0.0f;
                            }
#pragma unroll
                            for (int eb = 0; eb < NEB; ++eb) {
                                const float av = kk == 0 ? o.a[eb].x : (kk == 1 ? o.a[eb].y : (kk == 2 ? o.a[eb].z : o.a[eb].w));
#pragma unroll
                                for (int pb = 0; pb < 2; ++pb)
                                    acc[eb][pb] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, bv[pb], acc[eb][pb], 0, 0, 0);
                            }
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            }
            // lane holds GV of entry 16 eb + 4 j4 + r, pixel 16 (2 ph + pb) + l16
            if (q_hi > q_lo) {
#pragma unroll
                for (int eb = 0; eb < NEB; ++eb)
#pragma unroll
                    for (int pb = 0; pb < 2; ++pb)
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            atomicAdd(&s_gv[16 * eb + 4 * j4 + r][16 * (2 * ph + pb) + l16], acc[eb][pb][r]);
            }
        };
        switch (neb) {
            case 1: gv_phase(std::integral_constant<int, 1>{}); break;
            case 2: gv_phase(std::integral_constant<int, 2>{}); break;
            case 3: gv_phase(std::integral_constant<int, 3>{}); break;
            default: gv_phase(std::integral_constant<int, 4>{}); break;
        }
        __syncthreads();

        // ---- the walk: one lane per pixel, front to back
        if (wave == 0) {
            const double pcx = (wpix >= 0 ? wpix % W : 0) + 0.5, pcy = (wpix >= 0 ? wpix / W : 0) + 0.5;
            const double halfW = 0.5 * W;
            // offsets, G and alpha of entry e at this lane's pixel
            auto geom = [&](int e, double& dx, double& dy, float& G) -> float {
                dx = pcx - s_px[e];
                dx += dx >= halfW ? -(double)W : (dx < -halfW ? (double)W : 0.0);
                dy = pcy - s_py[e];
                const double qv = s_ca[e] * dx * dx + 2.0 * s_cb[e] * dx * dy + s_cc[e] * dy * dy;
                G = __builtin_amdgcn_exp2f((float)(-0.5 * LOG2E_B * qv));
                return s_sig[e] * G;
            };
            if (first) {
                if (one_batch) {
                    // D = the final prefix of the walk below, same operations
                    float Tq = 1.0f, Pq = 0.0f;
                    for (int e = 0; e < m; ++e) {
                        double dx, dy;
                        float G;
                        const float sg = geom(e, dx, dy, G);
                        const float alpha = fminf(amax, sg);
                        const bool take = (b0 + e - rg.x) < stop && alpha >= amin;
                        const float cA = s_att[e] * s_gv[e][lane];
                        const float Ta = take ? Tq * alpha : 0.0f;
                        Pq = Pq + Ta * cA;
                        Tq = take ? Tq * (1.0f - alpha) : Tq;
                    }
                    D = Pq;
                } else {
                    D = s_D[lane];
                }
            }
            for (int e = 0; e < m; ++e) {
                float w = 0.0f;
                double dx, dy;
                float G;
                const float sg = geom(e, dx, dy, G);
                const float sig = s_sig[e], att = s_att[e];
                const float alpha = fminf(amax, sg);
                const bool take = (b0 + e - rg.x) < stop && alpha >= amin;
                if (__ballot(take) != 0ull) {
                    const float gv = s_gv[e][lane];
                    const float cA = att * gv;
                    const float Ta = take ? T * alpha : 0.0f;
                    const float Pn = P + Ta * cA;
                    const float dalpha = T * cA - (D - Pn) * __builtin_amdgcn_rcpf(1.0f - alpha);
                    const float dsg = (take && sg < amax) ? dalpha : 0.0f;
                    const float dq = -0.5f * dsg * sig * G;
                    w = Ta * att;
                    const float dxf = (float)dx, dyf = (float)dy;
                    const float dq2 = -2.0f * dq;
                    float geo[8];
                    geo[0] = dq2 * fmaf(s_caf[e], dxf, s_cbf[e] * dyf);
                    geo[1] = dq2 * fmaf(s_cbf[e], dxf, s_ccf[e] * dyf);
                    geo[2] = dq * (dxf * dxf);
                    geo[3] = dq * (2.0f * dxf * dyf);
                    geo[4] = dq * (dyf * dyf);
                    geo[5] = dsg * G;
                    geo[6] = Ta * gv;
                    geo[7] = 0.0f;
                    T = take ? T * (1.0f - alpha) : T;
                    P = Pn;
                    wave_reduce_scatter8(geo, lane);
                    if ((lane & 7) == 0 && lane < 56 && geo[0] != 0.0f)
                        unsafeAtomicAdd(gacc + (size_t)(b0 + e) * 8 + (lane >> 3), geo[0]);
                }
                s_w[e][lane] = w;
                s_gv[e][lane] = 0.0f;  // cleared for the next batch
            }
        }
        __syncthreads();

        // ---- dL/dv[e][c] = sum_p w[e][p] g[p][c]: K-step kk pairs lane
        // group j4 with pixel 4 kk + j4.  The next block's upstream words
        // are fetched before this block's products (software pipelining).
        auto da_phase = [&](auto nebc) {
            constexpr int NEB = decltype(nebc)::value;
            uint32_t pvalid = 0;
#pragma unroll
            for (int kk = 0; kk < 16; ++kk) pvalid |= (s_pix[4 * kk + j4] >= 0 ? 1u : 0u) << kk;
            SgRaw<TGT> rb[2][16];
            // a uniform base per set and 32-bit lane offsets (one register
            // per address)
            auto fetch = [&](int cb, SgRaw<TGT>* r) {
                const int s = cb * 16 / Fc;
                const int c = cb * 16 - s * Fc + l16;
                const size_t sbase = ((size_t)s * F * HW) << CS;
                const uint32_t coff = ((uint32_t)((c >> CS) * HW) << CS) + (uint32_t)(c & CS);
#pragma unroll
                for (int kk = 0; kk < 16; ++kk) {
                    const int px = s_pix[4 * kk + j4];
                    r[kk] = sg_fetch<TGT>(up, sbase + (coff + (px >= 0 ? ((uint32_t)px << CS) : 0u)));
                }
            };
            for (int cb = cb_lo; cb < cb_hi; cb += 2) {
#pragma unroll
                for (int half = 0; half < 2; ++half) {
                    const int cc = cb + half;
                    if (cc < cb_hi) {
                        fetch(cc, rb[half]);
                        const int s = cc * 16 / Fc;
                        const int c = cc * 16 - s * Fc + l16;
                        const float mk = mg[((size_t)s * Fc + c) * mstr];
                        f32x4 acc[NEB];
#pragma unroll
                        for (int eb = 0; eb < NEB; ++eb) acc[eb] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
                        // the weights in four groups of four K-steps, the
                        // next group read from LDS while this one multiplies
                        float wv[2][4][NEB];
                        auto ldw = [&](int grp, float (*w)[NEB]) {
#pragma unroll
                            for (int k4 = 0; k4 < 4; ++k4)
#pragma unroll
                                for (int eb = 0; eb < NEB; ++eb) w[k4][eb] = s_w[16 * eb + l16][4 * (4 * grp + k4) + j4];
                        };
                        ldw(0, wv[0]);
#pragma unroll
                        for (int grp = 0; grp < 4; ++grp) {
                            if (grp < 3) ldw(grp + 1, wv[(grp + 1) & 1]);
                            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                            for (int k4 = 0; k4 < 4; ++k4) {
                                const int kk = 4 * grp + k4;
                                const float bvl =
                                    ((pvalid >> kk) & 1u) ? sg_value<TGT>(up, rb[half][kk]) + mk : 0.0f;
#pragma unroll
                                for (int eb = 0; eb < NEB; ++eb)
                                    acc[eb] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[grp & 1][k4][eb], bvl, acc[eb],
                                                                                   0, 0, 0);
                            }
                            __builtin_amdgcn_sched_barrier(0);
                        }
                        // lane holds entry 16 eb + 4 j4 + r, column c
                        float* dA = d_attr + s * da_stride + c;
#pragma unroll
                        for (int eb = 0; eb < NEB; ++eb)
#pragma unroll
                            for (int r = 0; r < 4; ++r) {
                                const int e = 16 * eb + 4 * j4 + r;
                                if (e < m && acc[eb][r] != 0.0f) unsafeAtomicAdd(dA + (size_t)s_g[e] * Fc, acc[eb][r]);
                            }
                    }
                }
            }
        };
        if (cb_hi > cb_lo) {
            switch (neb) {
                case 1: da_phase(std::integral_constant<int, 1>{}); break;
                case 2: da_phase(std::integral_constant<int, 2>{}); break;
                case 3: da_phase(std::integral_constant<int, 3>{}); break;
                default: da_phase(std::integral_constant<int, 4>{}); break;
            }
        }
        __syncthreads();
    }
}

// The per-pair accumulator is used over the walked part of each tile's list
// only, up to the largest stop position of the tile's pixels: tens of
// entries of lists that run to thousands.  Workgroups of a (tile, query)
// zero it (FOLD false, before a backward) or fold it into the per-Gaussian
// accumulators and the attribute gradients and clear it again (FOLD true;
// blockIdx.z: the geometric terms, then PAIR_COLS columns of the attribute
// rows each).  Over all pairs
// these two passes took 30 and 87 us at 6.7 million pairs (300,000 Gaussians,
// 180 x 720), 16 and 28 us at 2.7 million of 16 receivers; 6 and 13, 5 and
// 24 us so (the last bound by the atomics of Gaussians that many tiles walk).
constexpr int PAIR_COLS = 32;
constexpr int PAIR_ROW_MAX = 1024;  // longer rows hardly fit anywhere, and every PAIR_COLS of them cost a workgroup per tile

template <bool FOLD>
__global__ __launch_bounds__(256) void k_geo_pairs(float* __restrict__ gacc, size_t s_gacc,
                                                   const uint32_t* __restrict__ plist, size_t s_plist,
                                                   const uint2* __restrict__ ranges, size_t s_ranges,
                                                   const uint32_t* __restrict__ n_last, size_t s_pix, int H, int W,
                                                   int tw, int th, int TX, float* __restrict__ g2d, size_t s_g2d,
                                                   PairAttr pa, float* __restrict__ d_attr, int64_t da_stride, int Fc)
{
    const int q = blockIdx.y, tile = blockIdx.x, t = threadIdx.x;
    const int col = tile % TX * tw + t % tw, row = tile / TX * th + t / tw;
    uint32_t m = t < tw * th && col < W && row < H ? n_last[q * s_pix + (size_t)row * W + col] : 0u;
    __shared__ uint32_t s_m[4];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, o, 64));
    if ((t & 63) == 0) s_m[t >> 6] = m;
    __syncthreads();
    const uint2 rg = ranges[q * s_ranges + tile];
    const uint32_t len = rg.y - rg.x;
    m = min(max(max(s_m[0], s_m[1]), max(s_m[2], s_m[3])), len);
    const uint32_t na = pa.entries(m, len);
    float* acc = gacc + q * s_gacc + (size_t)rg.x * 8;
    if constexpr (!FOLD) {
        // (the attribute rows end inside the tile's len 8-float rows, also
        // when rounded up to four floats)
        const size_t n4 = (size_t)m * 2 + (pa.slot7 ? 0 : ((size_t)na * pa.row + 3) / 4);
        for (size_t e = t; e < n4; e += 256) ((float4*)acc)[e] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    } else {
        plist += q * s_plist + rg.x;
        if (blockIdx.z == 0) {
            g2d += q * s_g2d;
            for (uint32_t e = t; e < m * 8u; e += 256) {
                const float v = acc[e];
                if (v != 0.0f) {
                    acc[e] = 0.0f;
                    const size_t g = plist[e / 8];
                    float* p = g2d + g * 8 + (e & 7);
                    if (pa.slot7 && (e & 7) == 7) p = d_attr + q * da_stride + g;
                    unsafeAtomicAdd(p, v);
                }
            }
            return;
        }
        // columns [c0, c0 + nc) of the rows: set c / Fc, channel c % Fc (one
        // set, or all sets over the one geometry)
        const int c0 = ((int)blockIdx.z - 1) * PAIR_COLS, nc = min(PAIR_COLS, pa.row - c0);
        const int k = t % PAIR_COLS, c = c0 + k, s = c / Fc;
        if (k >= nc) return;
        float* arow = acc + pa.at(m, 0) + c;
        float* d = d_attr + (q + s) * da_stride + (c - s * Fc);
        constexpr int EP = 256 / PAIR_COLS, UN = 4;  // entries per step; steps whose loads go together
        for (uint32_t e0 = t / PAIR_COLS; e0 < na; e0 += EP * UN) {
            float v[UN];
            uint32_t g[UN];
#pragma unroll
            for (int u = 0; u < UN; ++u) {
                const uint32_t e = e0 + u * EP;
                v[u] = e < na ? arow[(size_t)e * pa.row] : 0.0f;
                g[u] = e < na ? plist[e] : 0u;
            }
#pragma unroll
            for (int u = 0; u < UN; ++u) {
                if (v[u] != 0.0f) {
                    arow[(size_t)(e0 + u * EP) * pa.row] = 0.0f;
                    unsafeAtomicAdd(d + (size_t)g[u] * Fc, v[u]);
                }
            }
        }
    }
}

template <bool FOLD>
static void launch_geo_pairs(const Layout& L, char* ws, PairAttr pa, float* d_attr, int64_t da_stride, int Fc,
                             hipStream_t s)
{
    const int z = FOLD && !pa.slot7 ? 1 + (pa.row + PAIR_COLS - 1) / PAIR_COLS : 1;
    hipLaunchKernelGGL(k_geo_pairs<FOLD>, dim3(L.T, L.nq, z), dim3(256), 0, s, (float*)(ws + L.gacc), L.s_gacc / 4,
                       (const uint32_t*)(ws + L.plist), L.s_plist / 4, (const uint2*)(ws + L.ranges),
                       L.s_ranges / sizeof(uint2), (const uint32_t*)(ws + L.n_last), L.s_pix / 4, L.H, L.W, L.tw,
                       L.th, L.TX, (float*)(ws + L.g2d), L.s_g2d / 4, pa, d_attr, da_stride, Fc);
}

void launch_geo_clear(const Layout& L, char* ws, hipStream_t s)
{
    launch_geo_pairs<false>(L, ws, PairAttr{0, 0}, nullptr, 0, 1, s);
}
void launch_geo_fold(const Layout& L, char* ws, hipStream_t s)
{
    launch_geo_pairs<true>(L, ws, PairAttr{0, 0}, nullptr, 0, 1, s);
}

template <int CG>
static void bwd_cg(dim3 grid, dim3 block, hipStream_t s, const gs_attrs& a, const gs_params& p, const Layout& L,
                   char* ws, const float* out, const BwdUpstream& up, float* d_attr, int64_t da_stride, int C, int shared,
                   PairAttr pa)
{
    hipLaunchKernelGGL(k_blend_bwd<CG>, grid, block, 0, s, (const GRec*)(ws + L.rec), L.s_rec / sizeof(GRec),
                       (const uint32_t*)(ws + L.plist), L.s_plist / 4, (const uint2*)(ws + L.ranges),
                       L.s_ranges / sizeof(uint2), a.data, a.query_stride, a.n_chan * C, C, L.H, L.W, L.tw, L.th,
                       L.TX, p.alpha_min, p.alpha_max, out, up.dout, up.target, up.mean_grad, up.scale,
                       (const uint32_t*)(ws + L.n_last), L.s_pix / 4,
                       (float*)(ws + L.gacc), L.s_gacc / 4, d_attr, da_stride, shared, pa);
}

// k_blend_bwd_sg with g = scale (out - target) + mean_grad over the groups
// whose walk is longer than min_walk entries only; the squared error of
// their pixels is added to lacc[set]
void launch_blend_bwd_sg_long(const gs_attrs& a, const gs_params& p, const Layout& L, int n_sets, char* ws,
                              const float* out, const float* target, const float* mean_grad, float scale,
                              const float* gscale, float* d_attr, int min_walk, float* lacc, hipStream_t s)
{
    int tw_log = 0;
    while ((1 << tw_log) < L.tw) ++tw_log;
    const SgUp sup{out, nullptr, target, mean_grad, scale, gscale};
    const int Fc = a.n_chan * (a.is_complex ? 2 : 1);
    auto kern = a.is_complex ? k_blend_bwd_sg<1, true> : k_blend_bwd_sg<0, true>;
    hipLaunchKernelGGL(kern, dim3(L.T, (L.tw * L.th) / SG_PIX), dim3(SG_WAVES * 64), 0, s, (const GRec*)(ws + L.rec),
                       (const uint32_t*)(ws + L.plist), (const uint2*)(ws + L.ranges), a.data, a.query_stride, n_sets,
                       Fc, L.H, L.W, tw_log, L.th, L.TX, p.alpha_min, p.alpha_max, sup,
                       (const uint32_t*)(ws + L.n_last), (float*)(ws + L.gacc), d_attr, a.query_stride, min_walk,
                       lacc);
}

gs_status launch_blend_bwd(const gs_attrs& a, const gs_params& p, const Layout& L, int n_sets, char* ws,
                           const float* out, const BwdUpstream& up, float* d_attr, hipStream_t s)
{
    const int C = a.is_complex ? 2 : 1;
    const int Fc = a.n_chan * C;
    // (32-bit element offsets inside one set's spectrum)
    const bool offs32 = (uint64_t)Fc * L.H * L.W < (1ull << 30);
    const int64_t das = a.query_stride;  // d_attr mirrors the attribute layout
    PairAttr pa{0, 0};
    if (L.nq == 1 && Fc % 16 == 0 && offs32 && !(p.options & GS_OPT_BWD_PER_GROUP)) {
        // one geometry for every set: the factorised backward
        int tw_log = 0;
        while ((1 << tw_log) < L.tw) ++tw_log;
        const SgUp sup{out, up.dout, up.target, up.mean_grad, up.scale, nullptr};
        const dim3 grid(L.T, (L.tw * L.th) / SG_PIX), block(SG_WAVES * 64);
        void* tok;
        launch_geo_pairs<false>(L, ws, pa, d_attr, das, Fc, s);
        timing_begin(TK_BLEND_BWD, s, &tok);
        auto kern = C == 2 ? (up.target ? k_blend_bwd_sg<1, true> : k_blend_bwd_sg<1, false>)
                           : (up.target ? k_blend_bwd_sg<0, true> : k_blend_bwd_sg<0, false>);
        hipLaunchKernelGGL(kern, grid, block, 0, s, (const GRec*)(ws + L.rec), (const uint32_t*)(ws + L.plist),
                           (const uint2*)(ws + L.ranges), a.data, a.query_stride, n_sets, Fc, L.H, L.W, tw_log,
                           L.th, L.TX, p.alpha_min, p.alpha_max, sup, (const uint32_t*)(ws + L.n_last),
                           (float*)(ws + L.gacc), d_attr, a.query_stride, 0, (float*)nullptr);
        timing_end(tok, s);
    } else {
    // the caller's group where it is valid; else the smallest
    // power of two that holds every channel float, 64 at most and the last
    // group partly filled: a walk per group costs more than empty channels
    int cg = p.chan_group;
    if (!chan_group_valid(Fc, cg))
        for (cg = 1; cg < 64 && cg < Fc;) cg *= 2;
    const int ngr = (Fc + cg - 1) / cg;
    if (ngr > 65535) return GS_ERR_CAPACITY;
    const int shared = (L.nq == 1 && n_sets > 1) ? 1 : 0;
    dim3 grid(L.T * ((L.tw * L.th) >> 6), ngr, n_sets), block(64 * BWD_WAVES);
    const int64_t row = shared && das ? (int64_t)Fc * n_sets : Fc;
    pa.slot7 = row == 1;
    pa.row = row <= PAIR_ROW_MAX ? (int)row : 0;
    launch_geo_pairs<false>(L, ws, pa, d_attr, das, Fc, s);
    void* tok;
    timing_begin(TK_BLEND_BWD, s, &tok);
    switch (cg) {
        case 1: bwd_cg<1>(grid, block, s, a, p, L, ws, out, up, d_attr, das, C, shared, pa); break;
        case 2: bwd_cg<2>(grid, block, s, a, p, L, ws, out, up, d_attr, das, C, shared, pa); break;
        case 4: bwd_cg<4>(grid, block, s, a, p, L, ws, out, up, d_attr, das, C, shared, pa); break;
        case 8: bwd_cg<8>(grid, block, s, a, p, L, ws, out, up, d_attr, das, C, shared, pa); break;
        case 16: bwd_cg<16>(grid, block, s, a, p, L, ws, out, up, d_attr, das, C, shared, pa); break;
        case 32: bwd_cg<32>(grid, block, s, a, p, L, ws, out, up, d_attr, das, C, shared, pa); break;
        default: bwd_cg<64>(grid, block, s, a, p, L, ws, out, up, d_attr, das, C, shared, pa); break;
    }
    timing_end(tok, s);
    }
    launch_geo_pairs<true>(L, ws, pa, d_attr, das, Fc, s);
    return GS_OK;
}

}  // namespace gs
