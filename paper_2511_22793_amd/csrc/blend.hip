// Front-to-back compositing of the per-tile depth-ordered lists (Eq. (3),
// Sec. 4.2; the per-pixel loop of Algorithm 1).  One workgroup per
// (tile, channel group, query), one thread per pixel; its waves run on their
// own (no workgroup barrier).  A wave takes the list 64 entries at a time:
//   each lane tests one entry against the box of the wave's 64 pixels, the
//   entries that reach it are queued in LDS in list order (the next 64
//   records are already on their way), and the queue is walked four entries
//   at a time: their
//     dx, dy      pixel-centre offset, azimuth wrapped into [-W/2, W/2)  (FP64)
//     q           conic quadratic form                                  (FP64)
//     G           exp(-q/2) via v_exp_f32                               (FP32)
//     alpha       min(alpha_max, opacity G)
//   are independent of each other, only the short chain
//     skip when alpha < alpha_min, stop below T_min, T, weight
//   runs entry by entry, and
//     out_f      += T alpha a_i v_{i,f} for the group's channels        (FP32)
// What bounds it is that chain and the entries evaluated per wave.  A tile's
// list holds every Gaussian whose rectangle touches the tile (thousands where
// the view runs along a wall), most of which miss a given 64 pixels; one
// entry at a time cost ~300 cycles of latency each.
// One channel: 2048 Gaussians, one receiver 61 -> 26 us, 50k Gaussians, 16
// receivers 245 -> 81 us, 300k Gaussians, one receiver 27 -> 11 us.
#include <type_traits>

#include "common.h"
#include "walk.h"

namespace gs {

constexpr double LOG2E = WALK_LOG2E;

// Attribute rows are read-only for the whole launch: reading them through a
// constant-address-space pointer lets a wave-uniform row go through the
// scalar cache (s_load) whatever the kernel stores elsewhere.
typedef __attribute__((address_space(4))) const float CFloat;
// The other buffers are global memory; naming the address space keeps the
// persistent kernel (which reads its pointers from a table) off flat
// instructions.
#define GLOBAL_AS __attribute__((address_space(1)))

// LDS of one wave (a launch has a slot for each of its waves: tiles of 64 and
// 128 pixels keep as many waves on a CU as those of 256): the queue, and pixel weights of a
// run of 16 entries (matrix-core path), the output transpose (64 pixels x
// 17), or the queued entries' attribute values (up to 8 channels).

struct alignas(16) BlendWave {
    WalkQueue Q;
    union {
        float w[16][68];
        float tr[64 * 17];
        float v[WALK_BATCH][BLEND_ROW_CG];
    } u;
};

typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ void wave_sync_lds() { walk_wave_sync(); }

// One wave's part of one (tile, channel group, set) of a blend job.  A group
// may reach past the last channel: those channels are zero and not stored.
// The buffers are passed as restrict parameters so that, once inlined, the
// attribute rows are known not to alias the stores.
template <int CG, bool FUSE = false>
__device__ __forceinline__ void blend_tile_impl(const BlendJob& J, BlendWave* SW, int tile, int cg, int set,
                                                const GRec* __restrict__ rec, const uint32_t* __restrict__ plist,
                                                const uint2* __restrict__ ranges, const float* __restrict__ attr,
                                                float* __restrict__ out, float* __restrict__ T_final,
                                                uint32_t* __restrict__ n_last, uint32_t* __restrict__ n_contrib)
{
    const int q = J.shared_geo ? 0 : set;  // geometry query
    const int nthr = J.tw * J.th;
    const int txi = tile % J.TX, tyi = tile / J.TX;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lx = threadIdx.x % J.tw, ly = threadIdx.x / J.tw;
    const int col = txi * J.tw + lx, row = tyi * J.th + ly;
    const bool inside = (int)threadIdx.x < nthr && col < J.W && row < J.H;
    WaveBox box;
    const bool any = wave_box(wave, txi, tyi, J.tw, J.th, J.H, J.W, box);
    if (!any && (!FUSE || wave >= (nthr >> 6))) return;
    BlendWave& S = SW[wave];
    uint2 rg;
    {
        const unsigned long long r = ((const GLOBAL_AS unsigned long long*)ranges)[q * J.s_ranges + tile];
        rg.x = (uint32_t)r;
        rg.y = (uint32_t)(r >> 32);
    }
    const uint32_t len = any ? rg.y - rg.x : 0u;
    const double pcx = col + 0.5, pcy = row + 0.5, halfW = 0.5 * J.W;
    const double Wd = (double)J.W;
    rec += q * J.s_rec;
    plist += q * J.s_plist + rg.x;
    const int Fc = J.Fc;
    const int chn = min(CG, Fc - cg * CG);  // channels of this group
    const float* A = attr + set * J.a_stride + cg * CG;
    const float amin = J.amin, amax = J.amax, tmin = J.tmin;

    WalkState px{1.0f, inside ? amin : INFINITY, 0u, 0u};
    const size_t HW = (size_t)J.H * J.W, pix = inside ? (size_t)row * J.W + col : 0;
    const int cs = J.C - 1;  // C is 1 or 2
    const size_t obase = (size_t)set * Fc * HW;
    // CG = 16, 32 (the fused loss stage): the channel sums
    // out[p][f] = sum_e w[p][e] v[e][f] of a run of 16 entries go to the FP32
    // matrix cores (v_mfma_f32_16x16x4_f32, A = the wave's pixel weights from
    // LDS, B = the entries' attribute rows); the walk only produces the
    // weights.  Smaller groups accumulate on the VALU, the values queued with
    // the entries.
    constexpr bool MF = CG >= 16;
    static_assert(!MF || FUSE, "more channel floats go to blend_mx_unit");
    constexpr int NB = MF ? CG / 16 : 1;
    constexpr int VG = MF ? 1 : CG;
    float acc[VG];
    f32x4 macc[MF ? 4 : 1][NB];
    if constexpr (MF) {
#pragma unroll
        for (int pb = 0; pb < 4; ++pb)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) macc[pb][nb] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    } else {
#pragma unroll
        for (int k = 0; k < CG; ++k) acc[k] = 0.0f;
    }

    // the lane's entry of the batch ahead: its Gaussian, record and values,
    // and the Gaussian of the batch after that
    uint32_t g_next = 0u, g_after = 0u;
    GRec r_next;
    float v_next[VG];
    auto fetch_g = [&](uint32_t b) -> uint32_t {
        return b + lane < len ? ((const GLOBAL_AS uint32_t*)plist)[b + lane] : 0u;
    };
    auto fetch = [&]() {
        const GLOBAL_AS GRec& r = ((const GLOBAL_AS GRec*)rec)[g_next];
        r_next = GRec{r.px, r.py, r.ca, r.cb, r.cc, r.sigma, r.att};
        if constexpr (!MF) {
            const CFloat* vp = (const CFloat*)(A + (size_t)g_next * Fc);
#pragma unroll
            for (int k = 0; k < CG; ++k) v_next[k] = k < chn ? vp[k] : 0.0f;
        }
    };
    if (len > 0) {
        g_next = fetch_g(0);
        g_after = fetch_g(WALK_BATCH);
        fetch();
    }
    for (uint32_t b0 = 0; b0 < len; b0 += WALK_BATCH) {
        int slot;
        bool plain, odd = false;  // odd: a queued entry has a value that is not finite
        const int m = walk_queue(S.Q, r_next, g_next, b0 + lane + 1, b0 + lane < len, box, Wd, amin, lane, slot, plain);
        if constexpr (!MF) {
            const bool pad = lane >= m && lane < (m + WALK_STEP - 1) / WALK_STEP * WALK_STEP;
            float z = 0.0f;
#pragma unroll
            for (int k = 0; k < CG; ++k) {
                if (slot >= 0) S.u.v[slot][k] = v_next[k];
                if (pad) S.u.v[lane][k] = 0.0f;
                z = fmaf(v_next[k], 0.0f, z);
            }
            odd = __ballot(slot >= 0 && z != 0.0f) != 0ull;
        }
        if (b0 + WALK_BATCH < len) {
            g_next = g_after;
            g_after = fetch_g(b0 + 2 * WALK_BATCH);
            fetch();
        }
        wave_sync_lds();
        auto walk = [&](auto pl, auto od) {
            constexpr bool PLAIN = decltype(pl)::value, ODD = decltype(od)::value;
            if constexpr (MF) {
                for (int j0 = 0; j0 < m; j0 += 16) {
                    if (walk_done(px)) break;  // all the wave's pixels stopped
                    // B operands of the run, loaded ahead of the walk: lane holds
                    // v[entry 4 ks + lane/16][channel 16 nb + lane%16]
                    float bv[4][NB];
#pragma unroll
                    for (int ks = 0; ks < 4; ++ks) {
                        const int e = j0 + 4 * ks + (lane >> 4);
                        const bool ev = e < m;
                        const CFloat* vr = (const CFloat*)(A + (size_t)(ev ? S.Q.g[e] : 0u) * Fc + (lane & 15));
#pragma unroll
                        for (int nb = 0; nb < NB; ++nb)
                            bv[ks][nb] = ev && 16 * nb + (lane & 15) < chn ? vr[16 * nb] : 0.0f;
                    }
                    int steps = 0;  // K-steps whose weights are in LDS
#pragma unroll 1
                    for (int ks = 0; ks < 4; ++ks) {
                        const int j = j0 + WALK_STEP * ks;
                        if (j >= m || walk_done(px)) break;
                        float w[WALK_STEP];
                        walk_step<PLAIN>(S.Q, j, px, pcx, pcy, halfW, Wd, amax, tmin, w);
#pragma unroll
                        for (int i = 0; i < WALK_STEP; ++i) S.u.w[WALK_STEP * ks + i][lane] = w[i];
                        steps = ks + 1;
                    }
                    wave_sync_lds();
                    float z = 0.0f;
#pragma unroll
                    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
                        for (int nb = 0; nb < NB; ++nb) z = fmaf(bv[ks][nb], 0.0f, z);
                    if (__ballot(z != 0.0f) != 0ull) {
                        // entry by entry, where it weighs
                        for (int r = 0; r < WALK_STEP * steps && j0 + r < m; ++r) {
                            const CFloat* vr = (const CFloat*)(A + (size_t)S.Q.g[j0 + r] * Fc + (lane & 15));
#pragma unroll
                            for (int nb = 0; nb < NB; ++nb) {
                                const float v = 16 * nb + (lane & 15) < chn ? vr[16 * nb] : 0.0f;
#pragma unroll
                                for (int pb = 0; pb < 4; ++pb)
#pragma unroll
                                    for (int i = 0; i < 4; ++i) {
                                        const float w = S.u.w[r][16 * pb + 4 * (lane >> 4) + i];
                                        macc[pb][nb][i] = w != 0.0f ? fmaf(w, v, macc[pb][nb][i]) : macc[pb][nb][i];
                                    }
                            }
                        }
                        wave_sync_lds();
                        continue;
                    }
#pragma unroll
                    for (int ks = 0; ks < 4; ++ks) {
                        if (ks < steps) {
#pragma unroll
                            for (int pb = 0; pb < 4; ++pb) {
                                const float a = S.u.w[4 * ks + (lane >> 4)][16 * pb + (lane & 15)];
#pragma unroll
                                for (int nb = 0; nb < NB; ++nb)
                                    macc[pb][nb] =
                                        __builtin_amdgcn_mfma_f32_16x16x4f32(a, bv[ks][nb], macc[pb][nb], 0, 0, 0);
                            }
                        }
                    }
                    wave_sync_lds();
                }
            } else {
#pragma unroll 1
                for (int j = 0; j < m; j += WALK_STEP) {
                    if (walk_done(px)) break;
                    float w[WALK_STEP];
                    walk_step<PLAIN>(S.Q, j, px, pcx, pcy, halfW, Wd, amax, tmin, w);
#pragma unroll
                    for (int i = 0; i < WALK_STEP; ++i)
#pragma unroll
                        for (int k = 0; k < CG; ++k) {
                            const float x = fmaf(w[i], S.u.v[j + i][k], acc[k]);
                            acc[k] = !ODD || w[i] != 0.0f ? x : acc[k];
                        }
                }
            }
        };
        if (!MF && odd) walk(std::false_type{}, std::true_type{});
        else if (plain) walk(std::true_type{}, std::false_type{});
        else walk(std::false_type{}, std::false_type{});
        if (walk_done(px)) break;
        wave_sync_lds();  // the next batch reuses the queue
    }
    wave_sync_lds();  // the transpose, and the caller's next item, reuse the LDS
    // the fused loss (FUSE: k_blend with a target): per written element the
    // target, the elementwise gradient part and the three sums,
    // reduce-scattered over the wave (lane 4 k + 0 ends with channel k's
    // totals) and stored per wave
    constexpr bool fuse = FUSE;
    // one of the sums (slot 0: out, 1: tgt, 2: squared error) of V channels
    // from ch0 on
    auto loss_sum = [&](auto vc, float* x, int ch0, int slot) {
        constexpr int V = decltype(vc)::value;
        wave_reduce_scatter<V>(x, lane);
        constexpr int sh = V == 16 ? 2 : (V == 8 ? 3 : (V == 4 ? 4 : (V == 2 ? 5 : 6)));
        const int ch = ch0 + (lane >> sh);
        if ((lane & ((1 << sh) - 1)) == 0 && ch < Fc) {
            J.lpart[(((size_t)set * Fc + ch) * 3 + slot) * J.lnp + (size_t)tile * (nthr >> 6) + wave] = x[0];
        }
    };
    if constexpr (MF) {
        // lane holds out[pixel 16 pb + 4 (lane/16) + r][channel 16 nb + lane%16]:
        // transpose through LDS so that each lane writes its own pixel
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            float* tr = S.u.tr;  // [64 pixels][17]
#pragma unroll
            for (int pb = 0; pb < 4; ++pb)
#pragma unroll
                for (int r = 0; r < 4; ++r) tr[(16 * pb + 4 * (lane >> 4) + r) * 17 + (lane & 15)] = macc[pb][nb][r];
            wave_sync_lds();
            // two 16-value arrays at a time next to the accumulators; the 16
            // target loads are issued before any store (the buffers are not
            // known not to alias, so a store would order the loads after it)
            const int ch0 = cg * CG + 16 * nb;
            float x[16], y[16];
#pragma unroll
            for (int k = 0; k < 16; ++k)
                y[k] = inside && ch0 + k < Fc ? J.tgt[obase + spec_offset(ch0 + k, pix, cs, HW)] : 0.0f;
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                const size_t idx = obase + spec_offset(ch0 + k, pix, cs, HW);
                const float o = tr[lane * 17 + k];
                if (inside && ch0 + k < Fc) {
                    ((GLOBAL_AS float*)out)[idx] = o;
                    if (J.dpart) J.dpart[idx] = J.lscale * (o - y[k]);
                }
                x[k] = inside ? o : 0.0f;
            }
            loss_sum(std::integral_constant<int, 16>{}, x, ch0, 0);
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                const float d = tr[lane * 17 + k] - y[k];
                x[k] = inside ? d * d : 0.0f;
            }
            loss_sum(std::integral_constant<int, 16>{}, x, ch0, 2);
            loss_sum(std::integral_constant<int, 16>{}, y, ch0, 1);
            wave_sync_lds();
        }
    } else {
        if constexpr (fuse) {
            float x[CG], y[CG];
#pragma unroll
            for (int k = 0; k < CG; ++k)
                y[k] = inside && k < chn ? J.tgt[obase + spec_offset(cg * CG + k, pix, cs, HW)] : 0.0f;
#pragma unroll
            for (int k = 0; k < CG; ++k) {
                const size_t idx = obase + spec_offset(cg * CG + k, pix, cs, HW);
                if (inside && k < chn) {
                    ((GLOBAL_AS float*)out)[idx] = acc[k];
                    if (J.dpart) J.dpart[idx] = J.lscale * (acc[k] - y[k]);
                }
                x[k] = inside ? (acc[k] - y[k]) * (acc[k] - y[k]) : 0.0f;
            }
            loss_sum(std::integral_constant<int, CG>{}, x, cg * CG, 2);
            loss_sum(std::integral_constant<int, CG>{}, y, cg * CG, 1);
#pragma unroll
            for (int k = 0; k < CG; ++k) x[k] = inside ? acc[k] : 0.0f;
            loss_sum(std::integral_constant<int, CG>{}, x, cg * CG, 0);
        }
    }
    if (!inside) return;
    if constexpr (!MF) {
        if constexpr (!fuse) {
#pragma unroll
            for (int k = 0; k < CG; ++k) {
                const int ch = cg * CG + k;
                if (k < chn) ((GLOBAL_AS float*)out)[obase + spec_offset(ch, pix, cs, HW)] = acc[k];
            }
        }
    }
    if (cg == 0 && set == q && T_final) {
        ((GLOBAL_AS float*)T_final)[q * J.s_pix + pix] = px.T;
        ((GLOBAL_AS uint32_t*)n_last)[q * J.s_pix + pix] = px.last;
        ((GLOBAL_AS uint32_t*)n_contrib)[q * J.s_pix + pix] = px.cnt;
    }
}

template <int CG>
__device__ __forceinline__ void blend_tile(const BlendJob& J, BlendWave* S, int tile, int cg, int set)
{
    blend_tile_impl<CG>(J, S, tile, cg, set, J.rec, J.plist, J.ranges, J.attr, J.out, J.T_final, J.n_last,
                        J.n_contrib);
}

// waves per SIMD the registers are sized for: the four records in flight and
// the accumulators of the matrix-core groups
__host__ __device__ constexpr int blend_waves(int cg) { return cg >= 32 ? 2 : (cg >= 16 ? 3 : 4); }

template <int CG, bool FUSE>
__global__ __launch_bounds__(256)
    __attribute__((amdgpu_waves_per_eu(blend_waves(CG), blend_waves(CG)))) void k_blend(BlendJob J, const GRec* __restrict__ rec,
                                               const uint32_t* __restrict__ plist, const uint2* __restrict__ ranges,
                                               const float* __restrict__ attr, float* __restrict__ out,
                                               float* __restrict__ T_final, uint32_t* __restrict__ n_last,
                                               uint32_t* __restrict__ n_contrib)
{
    extern __shared__ __align__(16) char s_waves[];  // a BlendWave per wave
    blend_tile_impl<CG, FUSE>(J, (BlendWave*)s_waves, blockIdx.x, blockIdx.y, blockIdx.z, rec, plist, ranges, attr, out, T_final,
                              n_last, n_contrib);
}

// ---------------------------------------------------------------------------
// Compositing of many channels: the weights w_k(p) = T_k alpha_k a_k do not
// depend on the channel (nor, over one shared geometry, on the attribute
// set), so for every column c = (set, channel component) of the spectrum
//   out(p, c) = sum_k w_k(p) v(k, c)
// is one product of the weights (entries x pixels) with the attribute rows
// (entries x columns).  A wave owns 64 pixels of a tile (the tile's in-image
// pixels packed into groups of 64) and a range of column blocks.  It walks
// the list until MX_STEPS steps of 4 entries that weigh anywhere are buffered
// in LDS or the walk ends, takes the weights into registers as matrix-core
// operands (v_mfma_f32_16x16x4_f32, B = entries x pixels), and then its column
// blocks (A = columns x entries); a lane ends with neighbouring columns of
// one pixel and stores them.  A walk longer than the buffer starts the next
// products from the stored sums, so every sum is one chain of fused
// multiply-adds in list order however it is cut (and is what k_blend forms
// one entry at a time).
// Bound: matrix cores (32 cycles per 4 entries x 16 pixels x 16 columns) and
// the spectrum's stores (non-temporal: cached ones left the L2 as half
// lines).
// 64 sets of 128 columns at 100k Gaussians, 90 x 360 (1.06 GB stored): 614 us
// with one wave of eight walking while the others wait, 349 now (391 with
// cached stores); 4 receivers of 32 columns at 20k Gaussians: 555 us with the
// list walked one entry at a time, 75 now.
// ---------------------------------------------------------------------------
constexpr int MX_WIDE = 2;
constexpr int MX_STEPS = 16;
constexpr int MX_ROWS = WALK_STEP * MX_STEPS;
constexpr uint32_t MX_OOB = 0x80000000u;  // past mx_rsrc's range
constexpr int MX_NT = 2;                  // non-temporal: the spectrum is not read again here
__device__ __forceinline__ __amdgpu_buffer_rsrc_t mx_rsrc(const void* base)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, 0x7FFFFFFF, 0x00020000);
}
// LDS of one wave: the queue, the buffered weights (pixel p at column
// 4 (p % 16) + p / 16, so that a lane's operands of one step are one 16-byte
// read) and the Gaussians of the buffered entries.
struct alignas(16) MxWave {
    WalkQueue Q;
    float w[MX_ROWS][64];
    uint32_t g[MX_ROWS];
};

// What the products of one group need besides the buffered weights.
struct MxOut {
    const float* attr;
    float* out;
    int64_t a_stride;
    size_t HW;
    int Fc, cs, nbs;  // channel floats, log2 of the components, blocks per set
    bool across;
    int set, k0, kn, vw, x0, y0, W;
    __device__ __forceinline__ int pixel(int k) const
    {
        return k < kn ? (y0 + k / vw) * W + x0 + k % vw : -1;
    }
    // block cb: its set and first column
    __device__ __forceinline__ int block(int cb, int width, int& c0) const
    {
        const int s = across ? cb / nbs : set;
        c0 = (across ? cb - s * nbs : cb) * width;
        return s;
    }
};

// out (+)= W^T V over NS steps for the column blocks [cb_lo, cb_hi), a set's
// attributes and spectrum addressed by 32-bit byte offsets (the launcher has
// checked that they fit and are aligned): accesses past the last column or
// outside the image, and the rows past the buffered steps, go past the
// buffers' range (reads give 0).  NV = 2: complex columns, 32 a block.
// Loads wait in issue order behind the stores before them, so a block's are
// issued ahead of the previous block's stores.  NV = 1: returns the first
// block with a value that is not finite, which is left to mx_products_big with
// those behind it (a zero weight takes such a value to every pixel of the
// wave, also to those that stopped in front of it); else cb_hi.
template <int NV, int NS>
__device__ __forceinline__ int mx_products(const MxOut& O, const MxWave& S, int steps, bool stored, int cb_lo, int cb_hi)
{
    const int lane = threadIdx.x & 63, j4 = lane >> 4, l16 = lane & 15;
    const uint32_t HW4 = (uint32_t)O.HW * 4u;  // bytes of a column's plane (of a pair's: 2 HW4)
    float wB[NS][4];                           // weight of entry 4 ks + j4 at pixel 16 pb + l16
    uint32_t row[NS];                          // byte offset of entry 4 ks + j4's columns
#pragma unroll
    for (int ks = 0; ks < NS; ++ks) {
        const float4 v = *(const float4*)&S.w[WALK_STEP * ks + j4][4 * l16];
        wB[ks][0] = v.x;
        wB[ks][1] = v.y;
        wB[ks][2] = v.z;
        wB[ks][3] = v.w;
        const uint32_t g = S.g[WALK_STEP * ks + j4];
        row[ks] = ks < steps ? (g * (uint32_t)O.Fc + NV * l16) * 4u : MX_OOB;
    }
    uint32_t so[4];  // byte offset of the lane's first column at pixel 16 pb + l16
#pragma unroll
    for (int pb = 0; pb < 4; ++pb) {
        const int px = O.pixel(O.k0 + 16 * pb + l16);
        so[pb] = px >= 0 ? 4u * NV * j4 * HW4 + ((uint32_t)px << O.cs) * 4u : MX_OOB;
    }
    float av[NS][NV];  // column NV l16 + v of entry 4 ks + j4
    auto load = [&](int cb) {
        int c0;
        const int s = O.block(cb, 16 * NV, c0);
        const __amdgpu_buffer_rsrc_t r = mx_rsrc(O.attr + s * O.a_stride + c0);
        const uint32_t past = NV > 1 || c0 + l16 < O.Fc ? 0u : MX_OOB;
#pragma unroll
        for (int ks = 0; ks < NS; ++ks) {
            if constexpr (NV == 1) {
                av[ks][0] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, row[ks] | past, 0, 0));
            } else {
                const auto x = __builtin_amdgcn_raw_buffer_load_b64(r, row[ks], 0, 0);
                __builtin_memcpy(av[ks], &x, 8);
            }
        }
    };
    load(cb_lo);
#pragma unroll 1
    for (int cb = cb_lo; cb < cb_hi; ++cb) {
        int c0;
        const int s = O.block(cb, 16 * NV, c0);
        float* ob = O.out + ((size_t)s * O.Fc + c0) * O.HW;
        const __amdgpu_buffer_rsrc_t r = mx_rsrc(ob);
        // acc[v][pb][i]: column c0 + NV (4 j4 + i) + v of pixel 16 pb + l16
        f32x4 acc[NV][4];
#pragma unroll
        for (int v = 0; v < NV; ++v)
#pragma unroll
            for (int pb = 0; pb < 4; ++pb) acc[v][pb] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        // byte offset of the lane's column offset e (of 4 NV) at pixel block pb
        auto at = [&](int e, int pb) -> uint32_t {
            const uint32_t past = NV > 1 || c0 + 4 * j4 + e < O.Fc ? 0u : MX_OOB;
            const uint32_t plane = O.cs ? (uint32_t)(e & ~1) * HW4 + (e & 1) * 4u : e * HW4;
            return (so[pb] + plane) | past | (so[pb] & MX_OOB);
        };
        if (stored) {
#pragma unroll
            for (int e = 0; e < 4 * NV; ++e)
#pragma unroll
                for (int pb = 0; pb < 4; ++pb)
                    acc[e % NV][pb][e / NV] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, at(e, pb), 0, 0));
        }
#pragma unroll
        for (int ks = 0; ks < NS; ++ks)
#pragma unroll
            for (int v = 0; v < NV; ++v)
#pragma unroll
                for (int pb = 0; pb < 4; ++pb)
                    acc[v][pb] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[ks][v], wB[ks][pb], acc[v][pb], 0, 0, 0);
        bool odd = false;  // a value that is not finite
        if constexpr (NV == 1) {
            float z = 0.0f;
#pragma unroll
            for (int ks = 0; ks < NS; ++ks) z = fmaf(av[ks][0], 0.0f, z);
            odd = __ballot(z != 0.0f) != 0ull;
        }
        if (cb + 1 < cb_hi) load(cb + 1);
        __builtin_amdgcn_sched_barrier(0);
        if (odd) return cb;
        // the value of column offset e, in column order
        auto val = [&](int pb, int e) { return __float_as_uint(acc[e % NV][pb][e / NV]); };
        if (NV > 1 || O.cs) {
#pragma unroll
            for (int e = 0; e < 4 * NV; e += 2)
#pragma unroll
                for (int pb = 0; pb < 4; ++pb) {
                    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
                    __builtin_amdgcn_raw_buffer_store_b64(u32x2{val(pb, e), val(pb, e + 1)}, r, at(e, pb), 0, MX_NT);
                }
        } else {
#pragma unroll
            for (int e = 0; e < 4 * NV; ++e)
#pragma unroll
                for (int pb = 0; pb < 4; ++pb) __builtin_amdgcn_raw_buffer_store_b32(val(pb, e), r, at(e, pb), 0, MX_NT);
        }
    }
    return cb_hi;
}

// The same in 64-bit addressing, for attributes or spectra past 2 GiB a set,
// for complex spectra that are not 8-byte aligned and for blocks with values
// that are not finite: those entries are added where they weigh only.
__device__ __forceinline__ void mx_products_big(const MxOut& O, const MxWave& S, int steps, bool stored, int cb_lo,
                                                int cb_hi)
{
    const int lane = threadIdx.x & 63, j4 = lane >> 4, l16 = lane & 15;
#pragma unroll 1
    for (int cb = cb_lo; cb < cb_hi; ++cb) {
        int c0;
        const int s = O.block(cb, 16, c0);
        const CFloat* vb = (const CFloat*)(O.attr + s * O.a_stride + c0 + l16);
        float* ob = O.out + (size_t)s * O.Fc * O.HW;
        const int c = c0 + 4 * j4;
        f32x4 acc[4];
#pragma unroll
        for (int pb = 0; pb < 4; ++pb) {
            const int px = O.pixel(O.k0 + 16 * pb + l16);
#pragma unroll
            for (int i = 0; i < 4; ++i)
                acc[pb][i] = stored && px >= 0 && c + i < O.Fc
                                 ? ((const GLOBAL_AS float*)ob)[spec_offset(c + i, px, O.cs, O.HW)]
                                 : 0.0f;
        }
#pragma unroll 1
        for (int ks = 0; ks < steps; ++ks) {
            const float a = c0 + l16 < O.Fc ? vb[(size_t)S.g[WALK_STEP * ks + j4] * O.Fc] : 0.0f;
            if (__ballot(a * 0.0f != 0.0f) != 0ull) {
                for (int k = WALK_STEP * ks; k < WALK_STEP * (ks + 1); ++k) {
                    const CFloat* vr = (const CFloat*)(O.attr + s * O.a_stride + (size_t)S.g[k] * O.Fc + c);
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const float v = c + i < O.Fc ? vr[i] : 0.0f;
#pragma unroll
                        for (int pb = 0; pb < 4; ++pb) {
                            const float wk = S.w[k][4 * l16 + pb];
                            acc[pb][i] = wk != 0.0f ? fmaf(wk, v, acc[pb][i]) : acc[pb][i];
                        }
                    }
                }
                continue;
            }
            const float4 w = *(const float4*)&S.w[WALK_STEP * ks + j4][4 * l16];
            acc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, w.x, acc[0], 0, 0, 0);
            acc[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, w.y, acc[1], 0, 0, 0);
            acc[2] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, w.z, acc[2], 0, 0, 0);
            acc[3] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, w.w, acc[3], 0, 0, 0);
        }
#pragma unroll
        for (int pb = 0; pb < 4; ++pb) {
            const int px = O.pixel(O.k0 + 16 * pb + l16);
            if (px < 0) continue;
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (c + i < O.Fc) ((GLOBAL_AS float*)ob)[spec_offset(c + i, px, O.cs, O.HW)] = acc[pb][i];
        }
    }
}

// Column blocks [cb_lo, cb_hi) of group pg of `tile`, 16 NV columns each (a
// lane loads NV neighbouring columns of an entry); with J.across the blocks
// run over the sets too (block = set * blocks per set + block), otherwise
// they are those of `set`.  state: this unit stores the per-pixel walk state.
// BIG: attributes and spectrum addressed in 64 bits (NV = 1).
template <int NV, bool BIG>
__device__ __forceinline__ void blend_mx_unit(const BlendJob& J, MxWave& S, int tile, int pg, int set, int cb_lo,
                                              int cb_hi, bool state, const GRec* __restrict__ rec,
                                              const uint32_t* __restrict__ plist, const uint2* __restrict__ ranges,
                                              const float* __restrict__ attr, float* __restrict__ out,
                                              float* __restrict__ T_final, uint32_t* __restrict__ n_last,
                                              uint32_t* __restrict__ n_contrib, int min_walk)
{
    const int q = J.shared_geo ? 0 : set;  // geometry query
    const int lane = threadIdx.x & 63, j4 = lane >> 4, l16 = lane & 15;
    const int txi = tile % J.TX, tyi = tile / J.TX;
    const int vw = min(J.tw, J.W - txi * J.tw), vh = min(J.th, J.H - tyi * J.th);
    const int k0 = 64 * pg, kn = min(vw * vh, k0 + 64);  // the group's pixels of the tile
    if (k0 >= kn) return;
    auto pixel = [&](int k) { return k < kn ? (tyi * J.th + k / vw) * J.W + txi * J.tw + k % vw : -1; };
    const int mypix = pixel(k0 + lane);
    if (min_walk > 0) {
        int m = mypix >= 0 ? (int)((const GLOBAL_AS uint32_t*)n_last)[mypix] : 0;
        for (int o = 32; o > 0; o >>= 1) m = max(m, __shfl_xor(m, o, 64));
        if (m <= min_walk) return;
    }
    uint2 rg;
    {
        const unsigned long long r = ((const GLOBAL_AS unsigned long long*)ranges)[q * J.s_ranges + tile];
        rg.x = (uint32_t)r;
        rg.y = (uint32_t)(r >> 32);
    }
    const uint32_t len = rg.y - rg.x;
    rec += q * J.s_rec;
    plist += q * J.s_plist + rg.x;
    const double pcx = (mypix >= 0 ? mypix % J.W : 0) + 0.5, pcy = (mypix >= 0 ? mypix / J.W : 0) + 0.5;
    const double halfW = 0.5 * J.W, Wd = (double)J.W;
    const int y0 = k0 / vw, y1 = (kn - 1) / vw;  // a group of several rows spans the tile's columns
    const WaveBox box{txi * J.tw + (y0 == y1 ? k0 % vw : 0) + 0.5, txi * J.tw + (y0 == y1 ? (kn - 1) % vw : vw - 1) + 0.5,
                      tyi * J.th + y0 + 0.5, tyi * J.th + y1 + 0.5};
    const float amin = J.amin, amax = J.amax, tmin = J.tmin;
    const int Fc = J.Fc, cs = J.C - 1;
    const size_t HW = (size_t)J.H * J.W;
    const int nbs = (Fc + 16 * NV - 1) / (16 * NV);  // blocks per set

    WalkState px{1.0f, mypix >= 0 ? amin : INFINITY, 0u, 0u};
    int steps = 0;  // buffered steps
    // the lane's Gaussian of the batch ahead
    auto fetch_g = [&](uint32_t b) -> uint32_t {
        return b + lane < len ? ((const GLOBAL_AS uint32_t*)plist)[b + lane] : 0u;
    };
    uint32_t g_next = fetch_g(0);
    uint32_t b0 = 0;  // first list position not queued yet
    int j = 0, m = 0;
    bool plain = true, end = len == 0, stored = false;
    for (;;) {
        // fill the buffer
        while (!end && steps < MX_STEPS) {
            if (j >= m) {
                if (b0 >= len) {
                    end = true;
                    break;
                }
                int slot;
                const uint32_t g = g_next;
                const GLOBAL_AS GRec& r = ((const GLOBAL_AS GRec*)rec)[g];
                const GRec rr{r.px, r.py, r.ca, r.cb, r.cc, r.sigma, r.att};
                g_next = fetch_g(b0 + WALK_BATCH);
                wave_sync_lds();
                m = walk_queue(S.Q, rr, g, b0 + lane + 1, b0 + lane < len, box, Wd, amin, lane, slot, plain);
                b0 += WALK_BATCH;
                wave_sync_lds();
                j = 0;
                continue;
            }
            float w[WALK_STEP];
            if (plain) walk_step<true>(S.Q, j, px, pcx, pcy, halfW, Wd, amax, tmin, w);
            else walk_step<false>(S.Q, j, px, pcx, pcy, halfW, Wd, amax, tmin, w);
            if (__ballot(w[0] != 0.0f || w[1] != 0.0f || w[2] != 0.0f || w[3] != 0.0f) != 0ull) {
#pragma unroll
                for (int i = 0; i < WALK_STEP; ++i) S.w[WALK_STEP * steps + i][4 * l16 + j4] = w[i];
                if (lane < WALK_STEP) S.g[WALK_STEP * steps + lane] = S.Q.g[j + lane];
                ++steps;
            }
            j += WALK_STEP;
            if (walk_done(px)) end = true;
        }
        if (end && steps > 0) {
            // the last step's entries that weigh nowhere (those behind the last
            // stop) go with the values of one that weighs
            wave_sync_lds();
            const int last = WALK_STEP * (steps - 1);
            uint32_t any = 0u;
#pragma unroll
            for (int i = 0; i < WALK_STEP; ++i) any |= __ballot(S.w[last + i][lane] != 0.0f) != 0ull ? 1u << i : 0u;
            if (lane < WALK_STEP && !(any >> lane & 1u)) S.g[last + lane] = S.g[last + __ffs(any) - 1];
        }
        // the products over the buffered entries, rounded up to a multiple of
        // 4 steps with zero weights (the step count is a constant of each
        // form: a branch per step would wait for every load one by one)
        const int ns = steps <= 4 ? 4 : (steps + 3) & ~3;
        for (int r = WALK_STEP * steps; r < WALK_STEP * ns; ++r) S.w[r][lane] = 0.0f;
        wave_sync_lds();
        const MxOut O{attr, out, J.a_stride, HW, Fc, cs, nbs, J.across != 0, set, k0, kn, vw, txi * J.tw, tyi * J.th, J.W};
        if constexpr (BIG) {
            mx_products_big(O, S, steps, stored, cb_lo, cb_hi);
        } else {
            int cb;
            if (ns == 4) cb = mx_products<NV, 4>(O, S, steps, stored, cb_lo, cb_hi);
            else if (ns == 8) cb = mx_products<NV, 8>(O, S, steps, stored, cb_lo, cb_hi);
            else if (ns == 12) cb = mx_products<NV, 12>(O, S, steps, stored, cb_lo, cb_hi);
            else cb = mx_products<NV, 16>(O, S, steps, stored, cb_lo, cb_hi);
            if (NV == 1 && cb < cb_hi) mx_products_big(O, S, steps, stored, cb, cb_hi);
        }
        stored = true;
        steps = 0;
        wave_sync_lds();
        if (end) break;
    }
    if (state && mypix >= 0 && T_final) {
        ((GLOBAL_AS float*)T_final)[q * J.s_pix + mypix] = px.T;
        ((GLOBAL_AS uint32_t*)n_last)[q * J.s_pix + mypix] = px.last;
        ((GLOBAL_AS uint32_t*)n_contrib)[q * J.s_pix + mypix] = px.cnt;
    }
}

// blockIdx.x = tile * J.ncg + column range (the ranges of a tile on
// neighbouring workgroups, so on different XCDs, each of which
// then reads its own columns of the attribute rows), blockIdx.z = set where
// the sets have their own geometry.
template <int NV, bool BIG>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_blend_mx(
    BlendJob J, const GRec* __restrict__ rec, const uint32_t* __restrict__ plist, const uint2* __restrict__ ranges,
    const float* __restrict__ attr, float* __restrict__ out, float* __restrict__ T_final,
    uint32_t* __restrict__ n_last, uint32_t* __restrict__ n_contrib)
{
    extern __shared__ __align__(16) char s_waves[];  // an MxWave per wave
    MxWave* const S = (MxWave*)s_waves;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tile = blockIdx.x / J.ncg, cg = blockIdx.x % J.ncg, set = blockIdx.z;
    const int nb = (J.Fc + 16 * NV - 1) / (16 * NV) * (J.across ? J.nsets : 1);
    const int cb_lo = (int)((int64_t)cg * nb / J.ncg), cb_hi = (int)((int64_t)(cg + 1) * nb / J.ncg);
    blend_mx_unit<NV, BIG>(J, S[wave], tile, wave, set, cb_lo, cb_hi, cg == 0 && set == (J.shared_geo ? 0 : set), rec,
                           plist, ranges, attr, out, T_final, n_last, n_contrib, 0);
}

// The same over the groups whose walk is longer than min_walk entries, all
// sets of one geometry: mostly none or a few, so a launch of MX_LONG_GRID
// workgroups looks for them.  (One workgroup per unit, 3312 of 80 KB of LDS
// each at 138 tiles and 64 column blocks, waited for LDS beside the training
// kernels and cost 25 us of a 740 us step to find nothing.)
constexpr int MX_LONG_GRID = 512;

template <int NV, bool BIG>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_blend_mx_long(
    BlendJob J, const GRec* __restrict__ rec, const uint32_t* __restrict__ plist, const uint2* __restrict__ ranges,
    const float* __restrict__ attr, float* __restrict__ out, float* __restrict__ T_final,
    uint32_t* __restrict__ n_last, uint32_t* __restrict__ n_contrib, int items, int min_walk)
{
    extern __shared__ __align__(16) char s_waves[];  // an MxWave per wave
    MxWave* const S = (MxWave*)s_waves;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nb = (J.Fc + 16 * NV - 1) / (16 * NV) * J.nsets;
    for (int it = blockIdx.x; it < items; it += gridDim.x) {
        const int tile = it / J.ncg, cg = it % J.ncg;
        const int cb_lo = (int)((int64_t)cg * nb / J.ncg), cb_hi = (int)((int64_t)(cg + 1) * nb / J.ncg);
        blend_mx_unit<NV, BIG>(J, S[wave], tile, wave, 0, cb_lo, cb_hi, cg == 0, rec, plist, ranges, attr, out,
                               T_final, n_last, n_contrib, min_walk);
    }
}

// Persistent blend over a table of jobs (scenes of any size, grid, tile
// shape and channel count): each workgroup takes (job, tile, channel group,
// set) items and stamps the completion time of the item's query.  Items are
// numbered job by job, then set by set, then channel group, then tile, so a
// query's items are contiguous and the job order is the service order.  The
// first part of the items is dealt out in turn (item k to workgroup k mod
// the grid); only the last quarter comes from a device counter, one item
// ahead of its use: an atomic per item on one counter, ~13 ns each and one
// after the other, bounded the launch (96 receivers over 8 scenes, 72k items: 2.11 ms; with the items dealt
// out and the matrix-core form's single walk per tile 1.40 ms).
// Every workgroup exits once its dealt items are done and the counter passes
// the total.
// MX: some job takes the matrix-core form.  Its 256 registers allow two waves
// per SIMD and its LDS as many (20 KB a wave); a batch without such a job runs
// without either (8 KB a wave, four waves per SIMD).  The LDS is sized by the
// waves launched (persist_lds): with four waves' worth whatever the workgroup,
// workgroups of 64 and 128 threads ran 2 and 4 waves per CU (4 jobs of 50,000
// Gaussians, 8 receivers, 16 complex channels: 1036 -> 708 us in 8 x 8 tiles,
// 756 -> 642 in 8 x 16; one channel: 820 -> 685, 613 -> 516 and 443 -> 416 us
// in 8 x 8, 8 x 16 and 16 x 16).
union PersistLds {
    BlendWave v;
    MxWave m;
};

__host__ __device__ constexpr size_t persist_lds(bool mx) { return mx ? sizeof(PersistLds) : sizeof(BlendWave); }

template <bool MX>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(MX ? 2 : 4))) void k_blend_persist(
    const BlendJob* __restrict__ jobs, int njobs, uint32_t total, uint32_t* counter, unsigned long long* done_ts)
{
    extern __shared__ __align__(16) char s_waves[];
    BlendWave* const SV = (BlendWave*)s_waves;
    __shared__ uint32_t s_item[2];
    const int lane = threadIdx.x & 63;
    const uint32_t rounds = (total - total / 4) / gridDim.x, dealt = rounds * gridDim.x;
    const uint32_t first = lane < njobs ? jobs[lane].item_begin : 0xFFFFFFFFu;
    for (uint32_t k = 0;; ++k) {
        // the item after the dealt ones, one ahead
        uint32_t ahead = 0u;
        if (threadIdx.x == 0 && k + 1 >= rounds) ahead = dealt + atomicAdd(counter, 1u);
        uint32_t item = k * gridDim.x + blockIdx.x;
        if (k >= rounds) {
            if (k == 0) {  // nothing was dealt: the first item is not known yet
                if (threadIdx.x == 0) {
                    s_item[1] = ahead;
                    ahead = dealt + atomicAdd(counter, 1u);
                }
                __syncthreads();
            }
            item = s_item[(k + 1) & 1];
        }
        item = __builtin_amdgcn_readfirstlane(item);
        if (item >= total) break;
        int j = __popcll(__ballot(first <= item)) - 1;  // last job with item_begin <= item
        if (njobs > 64) {
            int lo = 0, hi = njobs - 1;
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (jobs[mid].item_begin <= item) lo = mid;
                else hi = mid - 1;
            }
            j = lo;
        }
        const BlendJob& J = jobs[j];
        const uint32_t local = item - J.item_begin;
        const int tile = (int)(local % (uint32_t)J.T);
        const uint32_t rest = local / (uint32_t)J.T;
        const int cg = (int)(rest % (uint32_t)J.ncg);
        const int set = (int)(rest / (uint32_t)J.ncg);
        bool row = true;
        if constexpr (MX) {
            row = J.cg <= BLEND_ROW_CG;
            if (!row) {
                const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
                const int nb = (J.Fc + 16 * J.nv - 1) / (16 * J.nv);
                const int cb_lo = cg * nb / J.ncg, cb_hi = (cg + 1) * nb / J.ncg;
#define MX_ARGS J, ((MxWave*)s_waves)[wave], tile, wave, set, cb_lo, cb_hi, cg == 0, J.rec, J.plist, J.ranges, J.attr, J.out, \
                J.T_final, J.n_last, J.n_contrib, 0
                if (J.big) blend_mx_unit<1, true>(MX_ARGS);
                else if (J.nv > 1) blend_mx_unit<MX_WIDE, false>(MX_ARGS);
                else blend_mx_unit<1, false>(MX_ARGS);
#undef MX_ARGS
            }
        }
        if (row) {
            switch (J.cg) {
                case 1: blend_tile<1>(J, SV, tile, cg, set); break;
                case 2: blend_tile<2>(J, SV, tile, cg, set); break;
                case 4: blend_tile<4>(J, SV, tile, cg, set); break;
                default: blend_tile<8>(J, SV, tile, cg, set); break;
            }
        }
        // the next item's index (two slots: a wave may still read the other),
        // and every wave's part of this item is done
        if (threadIdx.x == 0) s_item[k & 1] = ahead;
        __syncthreads();
        if (threadIdx.x == 0 && done_ts) atomicMax(&done_ts[J.query0 + set], (unsigned long long)wall_clock64());
    }
}

__global__ void k_stamp(unsigned long long* ts)
{
    if (threadIdx.x == 0) *ts = (unsigned long long)wall_clock64();
}

// Geometry-only walk: marks every Gaussian that reaches at least one pixel
// (alpha >= alpha_min before the pixel stops) and records the per-pixel
// state.  Its output decides which (set, Gaussian) rows the attribute
// network must evaluate: no other Gaussian can change a pixel.
// One wave per 64 pixels of a tile (the tile's pixels row-major, in groups of
// 64): the groups of a tile walk the same list independently, so every CU
// has work (a tile per workgroup left half the chip idle at 138 tiles).
constexpr int LIVE_PIX = 64;
__global__ __launch_bounds__(LIVE_PIX) void k_live(
    const GRec* __restrict__ rec, size_t s_rec, const uint32_t* __restrict__ plist, size_t s_plist,
    const uint2* __restrict__ ranges, size_t s_ranges, int H, int W, int tw, int th, int TX, float amin, float amax,
    float tmin, uint32_t* __restrict__ flags_live, size_t s_live, float* __restrict__ T_final,
    uint32_t* __restrict__ n_last, uint32_t* __restrict__ n_contrib, size_t s_pix, float* __restrict__ wtot,
    size_t s_wtot)
{
    const int tile = blockIdx.x, q = blockIdx.z;
    constexpr int nthr = LIVE_PIX;
    const int txi = tile % TX, tyi = tile / TX;
    const int k = blockIdx.y * LIVE_PIX + threadIdx.x;  // pixel of the tile
    const int lx = k % tw, ly = k / tw;
    const int col = txi * tw + lx, row = tyi * th + ly;
    const bool inside = ly < th && col < W && row < H;
    if (__syncthreads_count(inside) == 0) return;  // a group past the image
    const uint2 rg = ranges[q * s_ranges + tile];
    const double pcx = col + 0.5, pcy = row + 0.5, halfW = 0.5 * W;
    rec += q * s_rec;
    plist += q * s_plist;
    flags_live += q * s_live;
    __shared__ double s_px[LIVE_PIX], s_py[LIVE_PIX], s_ca[LIVE_PIX], s_cb[LIVE_PIX], s_cc[LIVE_PIX];
    __shared__ float s_sig[LIVE_PIX], s_att[LIVE_PIX];
    __shared__ uint32_t s_g[LIVE_PIX];
    // per-pixel weights of the batch's entries, [entry][pixel] (a row of 65
    // keeps both the per-pixel writes and the per-entry sums conflict-free)
    __shared__ float s_w[LIVE_PIX][LIVE_PIX + 1];
    if (wtot) wtot += q * s_wtot;
    float T = 1.0f;
    uint32_t last = 0, cnt = 0;
    bool done = !inside;
    for (uint32_t b0 = rg.x; b0 < rg.y; b0 += nthr) {
        if (__syncthreads_count(done) == nthr) break;
        const uint32_t i = b0 + threadIdx.x;
        if (i < rg.y) {
            const uint32_t g = plist[i];
            const GRec r = rec[g];
            s_px[threadIdx.x] = r.px;
            s_py[threadIdx.x] = r.py;
            s_ca[threadIdx.x] = r.ca;
            s_cb[threadIdx.x] = r.cb;
            s_cc[threadIdx.x] = r.cc;
            s_sig[threadIdx.x] = r.sigma;
            s_att[threadIdx.x] = r.att;
            s_g[threadIdx.x] = g;
        }
        __syncthreads();
        const int m = (int)min((uint32_t)nthr, rg.y - b0);
        int jend = 0;  // entries walked by some pixel of the wave
        for (int j = 0; j < m; ++j) {
            if (__ballot(!done) == 0ull) break;
            jend = j + 1;
            float wgt = 0.0f;
            if (!done) {
                double dx = pcx - s_px[j];
                dx += dx >= halfW ? -(double)W : (dx < -halfW ? (double)W : 0.0);
                const double dy = pcy - s_py[j];
                const double qv = s_ca[j] * dx * dx + 2.0 * s_cb[j] * dx * dy + s_cc[j] * dy * dy;
                const float G = __builtin_amdgcn_exp2f((float)(-0.5 * LOG2E * qv));
                const float alpha = fminf(amax, s_sig[j] * G);
                const float Tn = T * (1.0f - alpha);
                const bool stop = alpha >= amin && Tn < tmin;
                const bool take = alpha >= amin && !stop;
                done = stop;
                if (take) flags_live[s_g[j]] = 1u;
                wgt = take ? T * alpha * s_att[j] : 0.0f;
                T = take ? Tn : T;
                last = take ? b0 + j + 1 - rg.x : last;
                cnt += take ? 1u : 0u;
            }
            if (wtot) s_w[j][threadIdx.x] = wgt;
        }
        if (wtot) {
            // thread t sums entry t's weight over the 64 pixels
            __syncthreads();
            if ((int)threadIdx.x < jend) {
                float ws = 0.0f;
#pragma unroll 8
                for (int i = 0; i < LIVE_PIX; ++i) ws += s_w[threadIdx.x][i];
                if (ws != 0.0f) unsafeAtomicAdd(&wtot[s_g[threadIdx.x]], ws);
            }
        }
    }
    if (!inside) return;
    const size_t pix = (size_t)row * W + col;
    T_final[q * s_pix + pix] = T;
    n_last[q * s_pix + pix] = last;
    n_contrib[q * s_pix + pix] = cnt;
}

// Compacts the live flags of each query into a list (order unspecified).
__global__ __launch_bounds__(256) void k_compact_live(const uint32_t* __restrict__ flags_live, size_t s_live, int n,
                                                      uint32_t* __restrict__ list, size_t s_list,
                                                      uint32_t* __restrict__ count)
{
    const int q = blockIdx.y;
    const int i = blockIdx.x * 256 + threadIdx.x;
    const bool on = i < n && flags_live[q * s_live + i] != 0u;
    const unsigned long long b = __ballot(on);
    const int lane = threadIdx.x & 63;
    uint32_t base = 0;
    if (lane == 0 && b) base = atomicAdd(&count[q], (uint32_t)__popcll(b));
    base = __shfl(base, 0, 64);
    if (on) list[q * s_list + base + __popcll(b & ((1ull << lane) - 1ull))] = (uint32_t)i;
}

void launch_live(const gs_params& p, const Layout& L, char* ws, uint32_t* list, size_t s_list, uint32_t* count,
                 hipStream_t s)
{
    uint32_t* fl = (uint32_t*)(ws + L.live);
    {
        // the live flags and weight sums of every query (their query
        // strides included: one contiguous range each) and the counts
        FillSegs f{};
        f.p[0] = fl; f.count[0] = (size_t)L.nq * (L.s_live / 4);
        f.p[1] = count; f.count[1] = (size_t)L.nq;
        f.p[2] = (uint32_t*)(ws + L.wtot); f.count[2] = (size_t)L.nq * (L.s_wtot / 4);
        f.n = 3;
        launch_fill_segs(f, s);
    }
    hipLaunchKernelGGL(k_live, dim3(L.T, (L.tw * L.th + LIVE_PIX - 1) / LIVE_PIX, L.nq), dim3(LIVE_PIX), 0, s,
                       (const GRec*)(ws + L.rec),
                       L.s_rec / sizeof(GRec), (const uint32_t*)(ws + L.plist), L.s_plist / 4,
                       (const uint2*)(ws + L.ranges), L.s_ranges / sizeof(uint2), L.H, L.W, L.tw, L.th, L.TX,
                       p.alpha_min, p.alpha_max, p.T_min, fl, L.s_live / 4, (float*)(ws + L.T_final),
                       (uint32_t*)(ws + L.n_last), (uint32_t*)(ws + L.n_contrib), L.s_pix / 4,
                       (float*)(ws + L.wtot), L.s_wtot / 4);
    hipLaunchKernelGGL(k_compact_live, dim3((L.n + 255) / 256, L.nq), dim3(256), 0, s, fl, L.s_live / 4, L.n, list,
                       s_list, count);
}

BlendJob make_blend_job(const gs_attrs& a, const gs_params& p, const Layout& L, int n_sets, char* ws, float* out)
{
    const int C = a.is_complex ? 2 : 1;
    BlendJob J{};
    J.rec = (const GRec*)(ws + L.rec);
    J.s_rec = L.s_rec / sizeof(GRec);
    J.plist = (const uint32_t*)(ws + L.plist);
    J.s_plist = L.s_plist / 4;
    J.ranges = (const uint2*)(ws + L.ranges);
    J.s_ranges = L.s_ranges / sizeof(uint2);
    J.attr = a.data;
    J.a_stride = a.query_stride;
    J.Fc = a.n_chan * C;
    J.C = C;
    J.H = L.H;
    J.W = L.W;
    J.tw = L.tw;
    J.th = L.th;
    J.TX = L.TX;
    J.T = L.T;
    J.nsets = n_sets;
    J.shared_geo = (L.nq == 1 && n_sets > 1) ? 1 : 0;
    J.across = 0;
    J.amin = p.alpha_min;
    J.amax = p.alpha_max;
    J.tmin = p.T_min;
    J.out = out;
    J.T_final = (float*)(ws + L.T_final);
    J.n_last = (uint32_t*)(ws + L.n_last);
    J.n_contrib = (uint32_t*)(ws + L.n_contrib);
    J.s_pix = L.s_pix / 4;
    J.tgt = nullptr;
    J.dpart = nullptr;
    J.lpart = nullptr;
    J.lnp = 0;
    J.lscale = 0.0f;
    return J;
}

// Whether the caller's channel group is valid: a power of two up to 64 that
// divides F*c.
bool chan_group_valid(int Fc, int g) { return g > 0 && g <= 64 && (g & (g - 1)) == 0 && Fc % g == 0; }

// Channel floats per workgroup of the compositing kernels: the caller's
// choice where it is valid; else up to 8 channel floats go to k_blend in one
// group (the smallest power of two that holds them), more to the matrix-core
// kernel in blocks of 16, all columns of a set after one walk.  The walk over
// the list is repeated for every group, so one partly empty group costs less
// than several full ones: 10 channel
// floats at 61,803 Gaussians, three receivers: 159 us in five groups of two,
// 62 in one block of 16.
int choose_blend_group(int Fc, int requested)
{
    if (chan_group_valid(Fc, requested)) return requested;
    if (Fc > BLEND_ROW_CG) return (Fc + 15) / 16 * 16;
    int cg = 1;
    while (cg < Fc) cg *= 2;
    return cg;
}

// Column ranges of the matrix-core kernel over `nb` column blocks: enough
// waves to fill the chip several times over (8 are resident per CU, by 240
// registers and by 20 KB of LDS a wave: 2048 on the chip; 8192 waves took 369
// us at 64 sets of 128 columns, 16384 349, 24576 406), at least MX_MIN_BLOCKS
// 16-column blocks after each walk, and a multiple of the 8 XCDs where there
// are that many.
constexpr int MX_WAVES = 16384, MX_MIN_BLOCKS = 4;
static int mx_split(int64_t groups, int nb, int nv)
{
    int64_t r = std::min<int64_t>((MX_WAVES + groups - 1) / groups, (int64_t)nb * nv / MX_MIN_BLOCKS);
    if (r >= 8) r = r / 8 * 8;
    return (int)std::max<int64_t>(std::min<int64_t>(r, nb), 1);
}

// The addressing of the matrix-core form: 32-bit byte offsets where a set's
// attributes and spectrum (n Gaussians) allow it and pairs are aligned, else
// 64-bit; and MX_WIDE columns a lane where a set's complex columns divide and
// are aligned for it.
void blend_mx_form(BlendJob* J, int64_t n)
{
    const int64_t bytes = (std::max<int64_t>(n, (int64_t)J->H * J->W) + 1) * ((J->Fc + 31) / 16 * 16) * 4;
    J->big = bytes >= 0x7FFFFFFFll || ((uintptr_t)J->out & 7) != 0;
    J->nv = !J->big && J->C == 2 && J->Fc % (16 * MX_WIDE) == 0 && ((uintptr_t)J->attr & (4 * MX_WIDE - 1)) == 0 &&
                    J->a_stride % MX_WIDE == 0
                ? MX_WIDE
                : 1;
}

static gs_status launch_mx(BlendJob J, const Layout& L, hipStream_t s, int min_walk = 0)
{
    blend_mx_form(&J, L.n);
    const int nb = (J.Fc + 16 * J.nv - 1) / (16 * J.nv) * (J.across ? J.nsets : 1), z = J.across ? 1 : J.nsets;
    const int gpt = (L.tw * L.th) >> 6;
    const unsigned lds = (unsigned)(gpt * sizeof(MxWave));
    if (J.ncg == 0) J.ncg = mx_split((int64_t)L.T * gpt * z, nb, J.nv);
    J.ncg = std::min(J.ncg, nb);
    if ((int64_t)L.T * J.ncg > 0x7FFFFFFF) return GS_ERR_CAPACITY;
    if (min_walk > 0) {
        auto kern = J.big ? k_blend_mx_long<1, true>
                          : (J.nv > 1 ? k_blend_mx_long<MX_WIDE, false> : k_blend_mx_long<1, false>);
        const int items = L.T * J.ncg;
        hipLaunchKernelGGL(kern, dim3(std::min(items, MX_LONG_GRID)), dim3(64 * gpt), lds, s, J, J.rec, J.plist,
                           J.ranges, J.attr, J.out, J.T_final, J.n_last, J.n_contrib, items, min_walk);
        return GS_OK;
    }
    auto kern = J.big ? k_blend_mx<1, true> : (J.nv > 1 ? k_blend_mx<MX_WIDE, false> : k_blend_mx<1, false>);
    hipLaunchKernelGGL(kern, dim3((unsigned)(L.T * J.ncg), 1, z), dim3(64 * gpt), lds, s, J, J.rec, J.plist, J.ranges,
                       J.attr, J.out, J.T_final, J.n_last, J.n_contrib);
    return GS_OK;
}

gs_status launch_blend(const gs_attrs& a, const gs_params& p, const Layout& L, int n_sets, char* ws, float* out,
                       hipStream_t s, const float* tgt, float* dpart, float* lpart, float lscale)
{
    const int C = a.is_complex ? 2 : 1;
    const int Fc = a.n_chan * C;
    int cg = choose_blend_group(Fc, p.chan_group);
    BlendJob J = make_blend_job(a, p, L, n_sets, ws, out);
    const bool per_set = (p.options & GS_OPT_BLEND_PER_GROUP) != 0;
    if (!tgt && (cg > BLEND_ROW_CG || (L.nq == 1 && Fc % 16 == 0 && !per_set))) {
        // every column after a pixel's walk; over the one prepared geometry
        // the columns of all sets
        J.across = L.nq == 1 && !per_set;
        J.ncg = !J.across && p.chan_group == cg ? Fc / cg : 0;
        void* tok;
        timing_begin(TK_BLEND, s, &tok);
        const gs_status st = launch_mx(J, L, s);
        timing_end(tok, s);
        return st;
    }
    // (the fused loss stage runs in k_blend, whose groups end at 32)
    if (tgt && cg > 32) cg = 32;
    if (tgt && (cg & (cg - 1))) cg = cg > 16 ? 32 : 16;
    const int ncg = (Fc + cg - 1) / cg;
    if (ncg > 65535) return GS_ERR_CAPACITY;
    J.cg = cg;
    J.ncg = ncg;
    J.tgt = tgt;
    J.dpart = dpart;
    J.lpart = lpart;
    J.lnp = L.T * ((L.tw * L.th) >> 6);
    J.lscale = lscale;
    dim3 grid(L.T, ncg, n_sets), block(L.tw * L.th);
    const unsigned lds = (unsigned)(((L.tw * L.th) >> 6) * sizeof(BlendWave));
#define ARGS J.rec, J.plist, J.ranges, J.attr, J.out, J.T_final, J.n_last, J.n_contrib
    void* tok;
    timing_begin(TK_BLEND, s, &tok);
    if (tgt) {
        switch (cg) {
            case 1: hipLaunchKernelGGL((k_blend<1, true>), grid, block, lds, s, J, ARGS); break;
            case 2: hipLaunchKernelGGL((k_blend<2, true>), grid, block, lds, s, J, ARGS); break;
            case 4: hipLaunchKernelGGL((k_blend<4, true>), grid, block, lds, s, J, ARGS); break;
            case 8: hipLaunchKernelGGL((k_blend<8, true>), grid, block, lds, s, J, ARGS); break;
            case 16: hipLaunchKernelGGL((k_blend<16, true>), grid, block, lds, s, J, ARGS); break;
            default: hipLaunchKernelGGL((k_blend<32, true>), grid, block, lds, s, J, ARGS); break;
        }
    } else {
        switch (cg) {
            case 1: hipLaunchKernelGGL((k_blend<1, false>), grid, block, lds, s, J, ARGS); break;
            case 2: hipLaunchKernelGGL((k_blend<2, false>), grid, block, lds, s, J, ARGS); break;
            case 4: hipLaunchKernelGGL((k_blend<4, false>), grid, block, lds, s, J, ARGS); break;
            default: hipLaunchKernelGGL((k_blend<8, false>), grid, block, lds, s, J, ARGS); break;
        }
    }
    timing_end(tok, s);
#undef ARGS
    return GS_OK;
}

// the shared-geometry compositing over the groups whose walk (live-pass stop
// positions) is longer than min_walk entries only
gs_status launch_blend_sg_long(const gs_attrs& a, const gs_params& p, const Layout& L, int n_sets, char* ws,
                               float* out, int min_walk, hipStream_t s)
{
    BlendJob J = make_blend_job(a, p, L, n_sets, ws, out);
    J.across = 1;
    return launch_mx(J, L, s, min_walk);
}

void launch_blend_persist(const BlendJob* jobs, int njobs, bool mx, uint32_t total, uint32_t* counter,
                          unsigned long long* done_ts, int workgroups, int block, hipStream_t s)
{
    hipLaunchKernelGGL(mx ? k_blend_persist<true> : k_blend_persist<false>, dim3(workgroups), dim3(block),
                       (unsigned)(persist_lds(mx) * (block / 64)), s, jobs, njobs, total, counter, done_ts);
}

hipError_t persist_occupancy(int block, bool mx, int* per_cu)
{
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(per_cu, mx ? k_blend_persist<true> : k_blend_persist<false>,
                                                        block, persist_lds(mx) * (block / 64));
}

void launch_stamp(unsigned long long* ts, hipStream_t s) { hipLaunchKernelGGL(k_stamp, dim3(1), dim3(64), 0, s, ts); }

}  // namespace gs
