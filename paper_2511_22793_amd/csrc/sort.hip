// Depth ordering and tile binning (the "directional sorting" of the method:
// Gaussians are binned to tiles and each tile's list is ordered by distance
// to the receiver, Sec. 4.2 and the per-pixel loop of Algorithm 1).
//
// 1. depth sort of the FP32 distance keys, index order breaking ties: by
//    ranking, or by sampled splitters into bins that each fit a workgroup;
//    beyond half a million keys a stable LSD radix sort (8-bit digits, one pass =
//    count + scan + scatter);
// 2. tiles-touched scan: exclusive prefix sum of the tile counts in depth
//    order, giving each Gaussian's first pair slot and the pair total;
// 3. pair emission: key = tile << rank_bits | depth_rank, unique per pair;
// 4. pair sort: the same radix sort over the tile digits only (pairs are
//    emitted in depth order, so a stable sort by tile completes the order);
// 5. tile ranges: [start, end) of each tile in the sorted pair array, and
//    the Gaussian id of every sorted pair.
// Every query of a batch is an independent segment (blockIdx.y).
#include "common.h"

namespace gs {

__global__ void k_fill_u32(uint32_t* p, size_t count, size_t q_stride, uint32_t v)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) p[blockIdx.y * q_stride + i] = v;
}

// Zero-fills up to FILL_SEGS buffers in one launch (blockIdx.y = segment).
__global__ void k_fill_segs(FillSegs f)
{
    const int k = blockIdx.y;
    if (k >= f.n) return;
    uint32_t* p = f.p[k];
    const size_t c = f.count[k];
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < c; i += (size_t)gridDim.x * blockDim.x)
        p[i] = 0u;
}

void launch_fill_segs(const FillSegs& f, hipStream_t s)
{
    size_t mx = 1;
    for (int k = 0; k < f.n; ++k) mx = f.count[k] > mx ? f.count[k] : mx;
    const size_t blocks = (mx + 255) / 256;
    hipLaunchKernelGGL(k_fill_segs, dim3((unsigned)(blocks < 1024 ? blocks : 1024), f.n), dim3(256), 0, s, f);
}

void launch_fill_u32(uint32_t* p, size_t count, size_t q_stride, int nq, uint32_t v, hipStream_t s)
{
    if (count == 0) return;
    dim3 grid((unsigned)((count + 255) / 256), nq);
    hipLaunchKernelGGL(k_fill_u32, grid, dim3(256), 0, s, p, count, q_stride, v);
}

__device__ __forceinline__ uint32_t seg_count(const uint32_t* n_dev, size_t n_stride, uint32_t n_fixed, int q)
{
    return n_dev ? n_dev[q * n_stride] : n_fixed;
}

// Per-workgroup digit histogram (RB-bit digits) of a block of 64*WV*IT
// keys; counts laid out [digit][block] per query.
template <int RB, int IT = SORT_ITEMS, int WV = SORT_THREADS / 64>
__global__ __launch_bounds__(64 * WV) void k_sort_count(
    const uint32_t* __restrict__ keys, size_t s_keys, const uint32_t* __restrict__ n_dev, size_t n_stride,
    uint32_t n_fixed, int shift, uint32_t* __restrict__ counts, size_t s_counts, int max_blocks)
{
    constexpr int R = 1 << RB;
    constexpr int NT = 64 * WV;
    constexpr uint32_t TILE = NT * IT;
    const int q = blockIdx.y;
    const uint32_t n = seg_count(n_dev, n_stride, n_fixed, q);
    const uint32_t base = blockIdx.x * TILE;
    if (base >= n) return;
    __shared__ uint32_t hist[R];
    for (int d = threadIdx.x; d < R; d += NT) hist[d] = 0;
    __syncthreads();
    keys += q * s_keys;
    uint32_t kv[IT];
#pragma unroll
    for (int i = 0; i < IT; ++i) {
        const uint32_t e = base + i * NT + threadIdx.x;
        kv[i] = e < n ? keys[e] : 0u;
    }
#pragma unroll
    for (int i = 0; i < IT; ++i) {
        const uint32_t e = base + i * NT + threadIdx.x;
        if (e < n) atomicAdd(&hist[(kv[i] >> shift) & (R - 1)], 1u);
    }
    __syncthreads();
    for (int d = threadIdx.x; d < R; d += NT)
        counts[q * s_counts + (size_t)d * max_blocks + blockIdx.x] = hist[d];
}

// Exclusive scan over blocks for one digit (one workgroup per digit and
// query); writes the digit total to totals[digit].
__global__ __launch_bounds__(256) void k_sort_scan(uint32_t* __restrict__ counts, size_t s_counts,
                                                   uint32_t* __restrict__ totals, size_t s_totals,
                                                   const uint32_t* __restrict__ n_dev, size_t n_stride,
                                                   uint32_t n_fixed, int max_blocks, uint32_t tile)
{
    const int d = blockIdx.x, q = blockIdx.y;
    const uint32_t n = seg_count(n_dev, n_stride, n_fixed, q);
    const int nb = (int)((n + tile - 1) / tile);
    uint32_t* row = counts + q * s_counts + (size_t)d * max_blocks;
    __shared__ uint32_t wsum[4];
    __shared__ uint32_t carry;
    if (threadIdx.x == 0) carry = 0;
    __syncthreads();
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    for (int b0 = 0; b0 < nb; b0 += 256) {
        const int b = b0 + threadIdx.x;
        const uint32_t v = b < nb ? row[b] : 0u;
        // inclusive wave scan
        uint32_t x = v;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t y = __shfl_up(x, o, 64);
            if (lane >= o) x += y;
        }
        if (lane == 63) wsum[w] = x;
        __syncthreads();
        uint32_t wbase = carry;
        for (int k = 0; k < w; ++k) wbase += wsum[k];
        if (b < nb) row[b] = wbase + x - v;
        __syncthreads();
        if (threadIdx.x == 255) carry = wbase + x;
        __syncthreads();
    }
    if (threadIdx.x == 0) totals[q * s_totals + d] = carry;
}

// Stable scatter of RB-bit digits.  Wave w of the WV-wave workgroup owns
// keys [w*64*IT, (w+1)*64*IT) of the block, consumed as IT rounds of 64
// consecutive keys.  A key's rank is (digit base) + (same digit in earlier
// blocks) + (in earlier waves) + (in earlier rounds of this wave) + (lanes
// below it with the same digit in this round, from an RB-ballot match mask).
// With `order` set (the single tile pass over pair keys) the output is the
// pair's Gaussian, order[key & rank_mask], instead of the key.
template <int RB, int IT = SORT_ITEMS, bool KV = true, int WV = SORT_THREADS / 64>
__global__ __launch_bounds__(64 * WV) void k_sort_scatter(
    const uint32_t* __restrict__ kin, const uint32_t* __restrict__ vin, uint32_t* __restrict__ kout,
    uint32_t* __restrict__ vout, size_t s_keys, const uint32_t* __restrict__ n_dev, size_t n_stride,
    uint32_t n_fixed, int shift, const uint32_t* __restrict__ counts, size_t s_counts,
    const uint32_t* __restrict__ totals, size_t s_totals, int max_blocks, const uint32_t* __restrict__ order,
    size_t s_order, uint32_t* __restrict__ plist, size_t s_plist, uint32_t rank_mask, uint2* __restrict__ ranges,
    size_t s_ranges, int T)
{
    constexpr int R = 1 << RB;
    constexpr int NT = 64 * WV;
    constexpr int DPT = R >= NT ? R / NT : 1;  // digits per thread in the digit scans
    constexpr int NDT = R / DPT;               // threads owning digits
    constexpr uint32_t TILE = NT * IT;
    const int q = blockIdx.y;
    const uint32_t n = seg_count(n_dev, n_stride, n_fixed, q);
    const uint32_t base = blockIdx.x * TILE;
    // (with `ranges`, block 0 always runs: it writes the tile ranges, also
    // when there are no keys)
    if (base >= n && !(ranges && blockIdx.x == 0)) return;
    __shared__ uint32_t s_goff[R];
    __shared__ uint32_t s_wcnt[WV][R];
    __shared__ uint32_t s_wsum[WV];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    kin += q * s_keys;
    if (!order) kout += q * s_keys;
    if (vin) {
        vin += q * s_keys;
        vout += q * s_keys;
    }
    // digit bases: exclusive scan of the totals over digits (thread tid <
    // NDT owns digits [tid*DPT, tid*DPT + DPT)).
    {
        const bool own = tid < NDT;
        uint32_t t[DPT], tsum = 0;
#pragma unroll
        for (int k = 0; k < DPT; ++k) t[k] = own ? totals[q * s_totals + tid * DPT + k] : 0u;
#pragma unroll
        for (int k = 0; k < DPT; ++k) tsum += t[k];
        uint32_t x = tsum;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t y = __shfl_up(x, o, 64);
            if (lane >= o) x += y;
        }
        if (lane == 63) s_wsum[w] = x;
        for (int d = tid; d < WV * R; d += NT) s_wcnt[d / R][d % R] = 0;
        __syncthreads();
        uint32_t run = x - tsum;
        for (int k = 0; k < w; ++k) run += s_wsum[k];
        if (own) {
#pragma unroll
            for (int k = 0; k < DPT; ++k) {
                const int d = tid * DPT + k;
                s_goff[d] = run + counts[q * s_counts + (size_t)d * max_blocks + blockIdx.x];
                // the tile pass: [start, end) of tile d is its digit range
                if (ranges && blockIdx.x == 0 && d < T) ranges[q * s_ranges + d] = make_uint2(run, run + t[k]);
                run += t[k];
            }
        }
    }
    __syncthreads();
    const unsigned long long lt = (1ull << lane) - 1ull;
    uint32_t key[IT], val[KV ? IT : 1], pos[IT];
    // issue every load before the rank chain so that they overlap
#pragma unroll
    for (int j = 0; j < IT; ++j) {
        const uint32_t e = base + w * (TILE / WV) + j * 64 + lane;
        key[j] = e < n ? kin[e] : 0u;
        if constexpr (KV) val[j] = (e < n && vin) ? vin[e] : 0u;
    }
#pragma unroll
    for (int j = 0; j < IT; ++j) {
        const uint32_t e = base + w * (TILE / WV) + j * 64 + lane;
        const bool valid = e < n;
        const uint32_t dig = (key[j] >> shift) & (R - 1);
        // lanes whose digit differs from this lane's in some bit: per bit,
        // the ballot of the bit, inverted where this lane's bit is set
        // (bm: the bit as an all-ones or all-zeros word)
        uint32_t dlo = 0u, dhi = 0u;
#pragma unroll
        for (int b = 0; b < RB; ++b) {
            const int32_t bm = (int32_t)(dig << (31 - b)) >> 31;
            const unsigned long long bb = __ballot(bm != 0);
            dlo |= (uint32_t)bb ^ (uint32_t)bm;
            dhi |= (uint32_t)(bb >> 32) ^ (uint32_t)bm;
        }
        const unsigned long long m = __ballot(valid) & ~(((unsigned long long)dhi << 32) | dlo);
        const uint32_t r = (uint32_t)__popcll(m & lt);
        const uint32_t c = s_wcnt[w][dig];
        pos[j] = c + r;
        // the highest lane of each digit group advances the wave's counter
        const bool leader = valid && ((m >> lane) == 1ull);
        __builtin_amdgcn_wave_barrier();
        if (leader) s_wcnt[w][dig] = c + r + 1;
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    for (int d = tid; d < R; d += NT) {
        uint32_t run = 0;
#pragma unroll
        for (int k = 0; k < WV; ++k) {
            const uint32_t c = s_wcnt[k][d];
            s_wcnt[k][d] = run;
            run += c;
        }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < IT; ++j) {
        const uint32_t e = base + w * (TILE / WV) + j * 64 + lane;
        if (e < n) {
            const uint32_t dig = (key[j] >> shift) & (R - 1);
            const uint32_t dst = s_goff[dig] + s_wcnt[w][dig] + pos[j];
            if (dst < n) {  // always true when the counts are consistent
                if (order) {
                    plist[q * s_plist + dst] = order[q * s_order + (key[j] & rank_mask)];
                } else {
                    kout[dst] = key[j];
                    if constexpr (KV) {
                        if (vout) vout[dst] = val[j];
                    }
                }
            }
        }
    }
}

// One counting pass over the RB-bit digits at `shift`: per-block counts,
// their scan over blocks, the stable scatter.  `blocks` is the count-row
// stride (the layout sizes the rows for it).
template <int RB, int IT, bool KV, int WV>
static void sort_pass(const uint32_t* kin, const uint32_t* vin, uint32_t* kout, uint32_t* vout, size_t s_keys,
                      const uint32_t* n_dev, size_t n_stride, uint32_t n_fixed, int shift, int blocks,
                      const Layout& L, char* ws, const uint32_t* order, size_t s_order, uint32_t* plist,
                      size_t s_plist, uint32_t rank_mask, hipStream_t s, uint2* ranges = nullptr)
{
    uint32_t* counts = (uint32_t*)(ws + L.counts);
    uint32_t* totals = (uint32_t*)(ws + L.totals);
    const size_t sc = L.s_counts / 4, st = L.s_totals / 4;
    hipLaunchKernelGGL((k_sort_count<RB, IT, WV>), dim3(blocks, L.nq), dim3(64 * WV), 0, s, kin, s_keys, n_dev,
                       n_stride, n_fixed, shift, counts, sc, blocks);
    hipLaunchKernelGGL(k_sort_scan, dim3(1 << RB, L.nq), dim3(256), 0, s, counts, sc, totals, st, n_dev, n_stride,
                       n_fixed, blocks, (uint32_t)(64 * WV * IT));
    hipLaunchKernelGGL((k_sort_scatter<RB, IT, KV, WV>), dim3(blocks, L.nq), dim3(64 * WV), 0, s, kin, vin, kout,
                       vout, s_keys, n_dev, n_stride, n_fixed, shift, counts, sc, totals, st, blocks, order, s_order,
                       plist, s_plist, rank_mask, ranges, L.s_ranges / sizeof(uint2), L.T);
}

// Sorts `passes` digits starting at bit 0; returns the buffer index (0 = a,
// 1 = b) that holds the result.
static int radix_sort(uint32_t* ka, uint32_t* kb, uint32_t* va, uint32_t* vb, size_t s_keys,
                      const uint32_t* n_dev, size_t n_stride, uint32_t n_fixed, int first_bit, int passes,
                      int blocks, bool wide, const Layout& L, char* ws, hipStream_t s)
{
    uint32_t *kin = ka, *kout = kb, *vin = va, *vout = vb;
    for (int p = 0; p < passes; ++p) {
        const int shift = first_bit + p * RADIX_BITS;
        if (wide)
            sort_pass<RADIX_BITS, SORT_ITEMS, true, SORT_WIDE_WAVES>(kin, vin, kout, vout, s_keys, n_dev, n_stride,
                                                                     n_fixed, shift, blocks, L, ws, nullptr, 0,
                                                                     nullptr, 0, 0u, s);
        else
            sort_pass<RADIX_BITS, SORT_ITEMS, true, SORT_THREADS / 64>(kin, vin, kout, vout, s_keys, n_dev, n_stride,
                                                                       n_fixed, shift, blocks, L, ws, nullptr, 0,
                                                                       nullptr, 0, 0u, s);
        uint32_t* t = kin; kin = kout; kout = t;
        t = vin; vin = vout; vout = t;
    }
    return passes & 1;
}

// Exclusive scan within a 256-thread workgroup; returns the prefix of v.
__device__ __forceinline__ uint32_t block_exclusive_scan_256(uint32_t v, uint32_t* wsum)
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint32_t x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    if (lane == 63) wsum[w] = x;
    __syncthreads();
    uint32_t base = 0;
    for (int k = 0; k < w; ++k) base += wsum[k];
    return base + x - v;
}

// ---- depth sort ----------------------------------------------------------
// Elements are (key, index) pairs compared as one 64-bit number, so equal
// keys stay in index order and no stage has to be stable.
//
// Up to DS_ONE keys: every key is ranked against all others.
// Up to DS_MAX keys: 4 keys per bin, at jittered places, are ranked against
// each other and every fourth becomes a splitter; each key finds its bin by
// binary search and takes a place in it (one atomic per workgroup and bin);
// the keys move to their bins; a workgroup per bin sorts it.  Four launches
// and two passes over the keys where the radix sort has 8 to 12 and four; at
// these sizes the launches and their latency are the time (2,000 keys: 35 us
// in 8 launches by the radix sort, 6 us so; 100,000: 48 and 28 us; 300,000:
// 64 us in 12 launches and 40 us).
// With 4 samples per bin a bin's size is close to a gamma variable of shape 4:
// 1024 bins of 512 keys on average, at DS_MAX, have one of more than 2048 in
// 8 sorts of 100, one of more than 4096 in 1e-7.  A workgroup takes up to 4096
// (DS_CAP) in its registers; beyond DS_MAX the bins outgrow that.  With 2048 as
// the limit 16 receivers of 524,288 Gaussians prepared in 1.11 ms, or in 2.00
// where a bin was larger (1.28 now; 1.58 by the radix sort).  A larger bin (the
// samples' places are known, so one can be built) is sorted in place in
// global memory by its workgroup: slow, but right.
constexpr int DS_ONE = 4096;
constexpr int DS_MAX = 1 << 19;
constexpr int DS_MAX_BINS = 1024; // words of a query's totals
constexpr int DS_BIN = 320;       // keys per bin aimed at
constexpr int DS_OVER = 4;        // samples per bin
constexpr int DS_RANK = 32;       // elements ranked per workgroup
constexpr int DS_WAVES = 4;       // waves that sort a bin, 2, 4, 8 or 16 keys per thread
constexpr int DS_CAP = 64 * 16 * DS_WAVES;
constexpr int DS_XCHG = 8;        // keys per thread that the exchange between waves holds at once

static int depth_bins(int n)
{
    int b = 16;
    while (b < DS_MAX_BINS && n / b > DS_BIN) b *= 2;
    return b;
}

typedef unsigned long long DsKey;

// x of lane ^ m, by DPP and permlane swaps (the LDS crossbar of __shfl_xor
// made the sorts below 1.4 times slower); m a constant after unrolling.
template <int CTRL>
__device__ __forceinline__ uint32_t lane_dpp(uint32_t x)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xF, 0xF, true);
}

__device__ __forceinline__ uint32_t lane_swap16(uint32_t x)
{
    const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    return threadIdx.x & 16 ? r[0] : r[1];
}

__device__ __forceinline__ uint32_t lane_swap32(uint32_t x)
{
    const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    return threadIdx.x & 32 ? r[0] : r[1];
}

template <int M>
__device__ __forceinline__ uint32_t lane_xor(uint32_t x)
{
    constexpr int Q1 = 0xB1, Q2 = 0x4E, Q3 = 0x1B;      // quad_perm: lane ^ 1, 2, 3
    constexpr int M7 = 0x141, R8 = 0x128, M15 = 0x140;  // row_half_mirror, row_ror:8, row_mirror
    if constexpr (M == 1) return lane_dpp<Q1>(x);
    if constexpr (M == 2) return lane_dpp<Q2>(x);
    if constexpr (M == 3) return lane_dpp<Q3>(x);
    if constexpr (M == 4) return lane_dpp<Q3>(lane_dpp<M7>(x));
    if constexpr (M == 7) return lane_dpp<M7>(x);
    if constexpr (M == 8) return lane_dpp<R8>(x);
    if constexpr (M == 15) return lane_dpp<M15>(x);
    if constexpr (M == 16) return lane_swap16(x);
    if constexpr (M == 31) return lane_swap16(lane_dpp<M15>(x));
    if constexpr (M == 32) return lane_swap32(x);
    if constexpr (M == 63) return lane_swap32(lane_swap16(lane_dpp<M15>(x)));
    return x;
}

// Sorts 64 NW E elements held E per thread by 64 NW threads, ascending:
// element E tid + i ends in v[i] of thread tid.  A bitonic network whose
// comparators all point upwards (the first stage of each merge mirrors):
// inside a thread by registers, between lanes by lane permutations, between
// waves through LDS (x: 64 NW min(E, DS_XCHG) elements, in as many turns as E
// takes).
template <int NW, int E, int K, int J>
__device__ __forceinline__ void sort_stage(DsKey* v, int tid, DsKey* x)
{
    constexpr int NT = 64 * NW;
    constexpr bool mirror = J == K / 2;
    if constexpr (J < E) {
#pragma unroll
        for (int i = 0; i < E; ++i) {
            const int o = i ^ (mirror ? K - 1 : J);
            if (o > i) {
                const DsKey a = v[i], b = v[o];
                const bool sw = a > b;
                v[i] = sw ? b : a;
                v[o] = sw ? a : b;
            }
        }
    } else {
        constexpr int tm = mirror ? K / E - 1 : J / E, rm = mirror ? E - 1 : 0;
        const bool low = (tid & (J / E)) == 0;
        DsKey p[E];
        if constexpr (tm < 64) {
#pragma unroll
            for (int i = 0; i < E; ++i)
                p[i] = ((DsKey)lane_xor<tm>((uint32_t)(v[i ^ rm] >> 32)) << 32) | lane_xor<tm>((uint32_t)v[i ^ rm]);
        } else {
            constexpr int X = E < DS_XCHG ? E : DS_XCHG;
#pragma unroll
            for (int i0 = 0; i0 < E; i0 += X) {
                __syncthreads();
#pragma unroll
                for (int i = 0; i < X; ++i) x[i * NT + tid] = v[i0 + i];
                __syncthreads();
#pragma unroll
                for (int i = 0; i < X; ++i) p[(i0 + i) ^ rm] = x[i * NT + (tid ^ tm)];
            }
        }
#pragma unroll
        for (int i = 0; i < E; ++i) v[i] = (p[i] < v[i]) == low ? p[i] : v[i];
    }
    if constexpr (J > 1)
        sort_stage<NW, E, K, J / 2>(v, tid, x);
    else if constexpr (K < E * NT)
        sort_stage<NW, E, 2 * K, K>(v, tid, x);
}

template <int NW, int E>
__device__ __forceinline__ void sort_regs(DsKey* v, int tid, DsKey* x)
{
    sort_stage<NW, E, 2, 1>(v, tid, x);
}

// m elements from (keys, vals) to (kout, vout), which may be the same arrays:
// everything is read before anything is written.
template <int NW, int E>
__device__ __forceinline__ void sort_run(const uint32_t* keys, const uint32_t* vals, uint32_t* kout, uint32_t* vout,
                                         uint32_t m, int tid, DsKey* x)
{
    DsKey v[E];
#pragma unroll
    for (int i = 0; i < E; ++i) {
        const uint32_t e = i * 64 * NW + tid;
        v[i] = e < m ? ((DsKey)keys[e] << 32) | vals[e] : ~0ull;
    }
    sort_regs<NW, E>(v, tid, x);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < E; ++i) {
        const uint32_t e = tid * E + i;
        if (e < m) {
            kout[e] = (uint32_t)(v[i] >> 32);
            vout[e] = (uint32_t)v[i];
        }
    }
}

// Ranks DS_RANK elements per workgroup against M of them (8 threads per
// element, an eighth of the M each).  ALL: the M = n elements are the keys
// themselves, which go straight to their ranks: the whole sort.  Else they
// are M = DS_OVER B samples, the one of rank DS_OVER k becomes split[k], and
// workgroup 0 clears the bins' counts.
template <bool ALL>
__global__ __launch_bounds__(256) void k_depth_rank(const uint32_t* __restrict__ keys, size_t s_keys, uint32_t n,
                                                    int M, DsKey* __restrict__ split, size_t s_split,
                                                    uint32_t* __restrict__ tot, size_t s_tot,
                                                    uint32_t* __restrict__ kout, uint32_t* __restrict__ vout)
{
    const int q = blockIdx.y;
    __shared__ alignas(16) DsKey v[DS_ONE];
    __shared__ uint32_t s_rank[DS_RANK];
    static_assert(DS_OVER * DS_MAX_BINS <= DS_ONE, "depth sort");
    keys += q * s_keys;
    const int log_m = 31 - __clz(M);
    const uint32_t step = n >> log_m;
    const int Mp = (M + 15) & ~15;  // padded: whole pairs per eighth
    constexpr int UN = DS_ONE / 256;
    uint32_t e[UN], kv[UN];
#pragma unroll
    for (int u = 0; u < UN; ++u) {
        const int i = u * 256 + threadIdx.x;
        e[u] = i;
        // (M, a power of two, divides by a shift)
        if constexpr (!ALL)
            e[u] = (uint32_t)(((uint64_t)i * n) >> log_m) + __umulhi((uint32_t)i * 0x9E3779B1u, step);
        kv[u] = i < M ? keys[e[u]] : 0u;
    }
#pragma unroll
    for (int u = 0; u < UN; ++u) {
        const int i = u * 256 + threadIdx.x;
        if (i < Mp) v[i] = i < M ? ((DsKey)kv[u] << 32) | e[u] : ~0ull;
    }
    if (threadIdx.x < DS_RANK) s_rank[threadIdx.x] = 0u;
    if (!ALL && blockIdx.x == 0)
        for (int b = threadIdx.x; b < M / DS_OVER; b += 256) tot[q * s_tot + b] = 0u;
    __syncthreads();
    constexpr int SEG = 256 / DS_RANK;
    const int sm = threadIdx.x % DS_RANK, seg = threadIdx.x / DS_RANK;
    const int me = blockIdx.x * DS_RANK + sm;
    const DsKey mine = me < M ? v[me] : ~0ull;
    const int len = Mp / SEG / 2;
    const ulonglong2* p = (const ulonglong2*)v + seg * len;
    uint32_t r = 0u;
#pragma unroll 8
    for (int i = 0; i < len; ++i) {
        const ulonglong2 c = p[i];
        r += c.x < mine ? 1u : 0u;
        r += c.y < mine ? 1u : 0u;
    }
    atomicAdd(&s_rank[sm], r);
    __syncthreads();
    if (threadIdx.x < DS_RANK && me < M) {
        const uint32_t rank = s_rank[sm];
        if constexpr (ALL) {
            kout[q * s_keys + rank] = (uint32_t)(mine >> 32);
            vout[q * s_keys + rank] = (uint32_t)mine;
        } else if (rank % DS_OVER == 0) {
            split[q * s_split + rank / DS_OVER] = mine;
        }
    }
}

// Each key's bin and its place there, packed: bin << 20 | place (places
// are below n <= 2^19).  A bin's place counter is advanced once per workgroup.
__global__ __launch_bounds__(SORT_THREADS) void k_depth_bin(const uint32_t* __restrict__ keys, size_t s_keys,
                                                            uint32_t n, const DsKey* __restrict__ split,
                                                            size_t s_split, int B, uint32_t* __restrict__ tot,
                                                            size_t s_tot, uint32_t* __restrict__ packed)
{
    const int q = blockIdx.y;
    __shared__ DsKey s_split_[DS_MAX_BINS];
    __shared__ uint32_t s_cnt[DS_MAX_BINS];
    keys += q * s_keys;
    const uint32_t base = blockIdx.x * SORT_TILE + threadIdx.x;
    uint32_t kv[SORT_ITEMS];
#pragma unroll
    for (int i = 0; i < SORT_ITEMS; ++i) {
        const uint32_t e = base + i * SORT_THREADS;
        kv[i] = e < n ? keys[e] : 0u;
    }
    for (int b = threadIdx.x; b < B; b += SORT_THREADS) {
        s_split_[b] = split[q * s_split + b];
        s_cnt[b] = 0u;
    }
    __syncthreads();
    int bin[SORT_ITEMS];
#pragma unroll
    for (int i = 0; i < SORT_ITEMS; ++i) bin[i] = 0;
    for (int st = B / 2; st > 0; st /= 2) {
#pragma unroll
        for (int i = 0; i < SORT_ITEMS; ++i) {
            const DsKey c = ((DsKey)kv[i] << 32) | (base + i * SORT_THREADS);
            bin[i] += c >= s_split_[bin[i] + st] ? st : 0;
        }
    }
    uint32_t pl[SORT_ITEMS];
#pragma unroll
    for (int i = 0; i < SORT_ITEMS; ++i)
        pl[i] = base + i * SORT_THREADS < n ? atomicAdd(&s_cnt[bin[i]], 1u) : 0u;
    __syncthreads();
    for (int b = threadIdx.x; b < B; b += SORT_THREADS) {
        const uint32_t c = s_cnt[b];
        s_cnt[b] = c ? atomicAdd(&tot[q * s_tot + b], c) : 0u;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < SORT_ITEMS; ++i) {
        const uint32_t e = base + i * SORT_THREADS;
        if (e < n) packed[q * s_keys + e] = (uint32_t)bin[i] << 20 | (s_cnt[bin[i]] + pl[i]);
    }
}

// Moves every key (and its index) to its place: bin start + place.
__global__ __launch_bounds__(SORT_THREADS) void k_depth_move(const uint32_t* __restrict__ keys, size_t s_keys,
                                                             uint32_t n, int B, const uint32_t* __restrict__ tot,
                                                             size_t s_tot, const uint32_t* __restrict__ packed,
                                                             uint32_t* __restrict__ kout, uint32_t* __restrict__ vout)
{
    const int q = blockIdx.y;
    __shared__ uint32_t s_start[DS_MAX_BINS];
    __shared__ uint32_t wsum[4];
    const uint32_t base = blockIdx.x * SORT_TILE + threadIdx.x;
    uint32_t kv[SORT_ITEMS], pv[SORT_ITEMS];
#pragma unroll
    for (int i = 0; i < SORT_ITEMS; ++i) {
        const uint32_t e = base + i * SORT_THREADS;
        kv[i] = e < n ? keys[q * s_keys + e] : 0u;
        pv[i] = e < n ? packed[q * s_keys + e] : 0u;
    }
    constexpr int BPT = DS_MAX_BINS / SORT_THREADS;
    uint32_t c[BPT], sum = 0u;
#pragma unroll
    for (int k = 0; k < BPT; ++k) {
        const int b = threadIdx.x * BPT + k;
        c[k] = b < B ? tot[q * s_tot + b] : 0u;
        sum += c[k];
    }
    uint32_t run = block_exclusive_scan_256(sum, wsum);
#pragma unroll
    for (int k = 0; k < BPT; ++k) {
        s_start[threadIdx.x * BPT + k] = run;
        run += c[k];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < SORT_ITEMS; ++i) {
        const uint32_t e = base + i * SORT_THREADS;
        if (e < n) {
            const uint32_t dst = s_start[pv[i] >> 20] + (pv[i] & 0xFFFFFu);
            kout[q * s_keys + dst] = kv[i];
            vout[q * s_keys + dst] = e;
        }
    }
}

// Sorts one bin (blockIdx.x): kin (keys) and val (indices, in place).
__global__ __launch_bounds__(64 * DS_WAVES) void k_depth_local(uint32_t* kin, uint32_t* __restrict__ kout,
                                                               uint32_t* val, size_t s_keys,
                                                               const uint32_t* __restrict__ tot, size_t s_tot)
{
    constexpr int NT = 64 * DS_WAVES;
    const int q = blockIdx.y, bin = blockIdx.x;
    __shared__ DsKey x[NT * DS_XCHG];
    const uint32_t m = tot[q * s_tot + bin];
    if (m == 0) return;
    uint32_t pre = 0u;
#pragma unroll
    for (int k = 0; k < DS_MAX_BINS / 64; ++k) {
        const int b = k * 64 + (threadIdx.x & 63);
        pre += b < bin ? tot[q * s_tot + b] : 0u;
    }
    for (int o = 32; o > 0; o >>= 1) pre += __shfl_xor(pre, o, 64);
    const size_t base = q * s_keys + (size_t)pre;
    kin += base;
    kout += base;
    val += base;
    if (m <= NT * 2u) {
        sort_run<DS_WAVES, 2>(kin, val, kout, val, m, threadIdx.x, x);
        return;
    }
    if (m <= NT * 4u) {
        sort_run<DS_WAVES, 4>(kin, val, kout, val, m, threadIdx.x, x);
        return;
    }
    if (m <= NT * 8u) {
        sort_run<DS_WAVES, 8>(kin, val, kout, val, m, threadIdx.x, x);
        return;
    }
    if (m <= (uint32_t)DS_CAP) {
        sort_run<DS_WAVES, 16>(kin, val, kout, val, m, threadIdx.x, x);
        return;
    }
    // the same network on the two arrays in global memory (the missing
    // elements of the next power of two, infinite, stay where they are)
    volatile uint32_t* kg = kin;
    volatile uint32_t* vg = val;
    uint32_t half = 1u;
    while (half * 2u < m) half *= 2u;
    for (uint32_t k = 2; k <= 2u * half; k *= 2u) {
        for (uint32_t j = k / 2; j > 0; j /= 2u) {
            for (uint32_t t = threadIdx.x; t < half; t += NT) {
                const uint32_t r = t & (j - 1u), i = 2u * (t - r) + r, o = i ^ (j == k / 2 ? k - 1u : j);
                if (o < m) {
                    const uint32_t ka = kg[i], kb = kg[o], va = vg[i], vb = vg[o];
                    if (ka > kb || (ka == kb && va > vb)) {
                        kg[i] = kb;
                        kg[o] = ka;
                        vg[i] = vb;
                        vg[o] = va;
                    }
                }
            }
            __syncthreads();
        }
    }
    for (uint32_t i = threadIdx.x; i < m; i += NT) kout[i] = kg[i];
}

size_t depth_keys_in(const Layout& L) { return L.n <= DS_ONE ? L.keys_b : L.keys_a; }

void launch_depth_sort(const Layout& L, char* ws, hipStream_t s)
{
    uint32_t *ka = (uint32_t*)(ws + L.keys_a), *kb = (uint32_t*)(ws + L.keys_b);
    uint32_t *va = (uint32_t*)(ws + L.vals_a), *vb = (uint32_t*)(ws + L.vals_b);
    const size_t sk = L.s_keys / 4;
    if (L.n > DS_MAX) {
        // keys a -> ... -> a after 4 passes (even), values follow
        radix_sort(ka, kb, va, vb, sk, nullptr, 0, (uint32_t)L.n, 0, 4, L.sort_blocks, L.sort_wide != 0, L, ws, s);
        return;
    }
    const uint32_t n = (uint32_t)L.n;
    if (L.n <= DS_ONE) {
        // (the projection left the keys in b)
        hipLaunchKernelGGL(k_depth_rank<true>, dim3((n + DS_RANK - 1) / DS_RANK, L.nq), dim3(256), 0, s, kb, sk, n,
                           L.n, (DsKey*)nullptr, (size_t)0, (uint32_t*)nullptr, (size_t)0, ka, va);
        return;
    }
    // (the splitters take 8 bytes per DS_BIN / 2 keys or more: they fit the
    // count rows, of at least n / 8 bytes)
    const int B = depth_bins(L.n);
    DsKey* split = (DsKey*)(ws + L.counts);
    uint32_t* tot = (uint32_t*)(ws + L.totals);
    const size_t ss = L.s_counts / sizeof(DsKey), st = L.s_totals / 4;
    hipLaunchKernelGGL(k_depth_rank<false>, dim3(DS_OVER * B / DS_RANK, L.nq), dim3(256), 0, s, ka, sk, n,
                       DS_OVER * B, split, ss, tot, st, (uint32_t*)nullptr, (uint32_t*)nullptr);
    const dim3 grid((n + SORT_TILE - 1) / SORT_TILE, L.nq);
    hipLaunchKernelGGL(k_depth_bin, grid, dim3(SORT_THREADS), 0, s, ka, sk, n, split, ss, B, tot, st, vb);
    hipLaunchKernelGGL(k_depth_move, grid, dim3(SORT_THREADS), 0, s, ka, sk, n, B, tot, st, vb, kb, va);
    hipLaunchKernelGGL(k_depth_local, dim3(B, L.nq), dim3(64 * DS_WAVES), 0, s, kb, ka, va, sk, tot, st);
}

// ---- tiles-touched scan and pair emission -------------------------------
// Scan granularity: EMIT_RANKS consecutive depth ranks per workgroup.
constexpr int EMIT_RANKS = 64;
// up to this many blocks the emission adds up the block sums itself (each
// workgroup reads the sums before its own: quadratic, so only for a few
// thousand blocks)
constexpr int EMIT_SCAN_BLOCKS = 2048;

// Sum of the tile counts of each EMIT_RANKS block of the depth order (one
// wave per block).  Culled Gaussians sort to the end (key ~0), so the last
// valid key's rank gives the visible count: its thread stores it.  The same
// threads count the invalid inputs (rare: the atomic runs only for a wave
// that has one).
__global__ __launch_bounds__(64) void k_scan_reduce(const uint32_t* __restrict__ keys,
                                                    const uint32_t* __restrict__ order, size_t s_order, uint32_t n,
                                                    const uint4* __restrict__ tinfo, size_t s_tinfo,
                                                    const uint32_t* __restrict__ status, size_t s_status,
                                                    uint32_t* __restrict__ flags, size_t s_flags,
                                                    uint32_t* __restrict__ partial, size_t s_partial)
{
    const int q = blockIdx.y;
    const uint32_t k = blockIdx.x * EMIT_RANKS + threadIdx.x;
    keys += q * s_order;
    flags += q * s_flags;
    uint32_t v = 0u;
    bool bad = false;
    if (k < n) {
        bad = status[q * s_status + k] == ST_INVALID;
        if (keys[k] != 0xFFFFFFFFu) {
            v = tinfo[q * s_tinfo + order[q * s_order + k]].w;
            if (k + 1 == n || keys[k + 1] == 0xFFFFFFFFu) flags[FL_NVIS] = k + 1;
        }
    }
    const unsigned long long nb = __ballot(bad);
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    if (threadIdx.x == 0) {
        partial[q * s_partial + blockIdx.x] = v;
        if (nb) atomicAdd(&flags[FL_INVALID], (uint32_t)__popcll(nb));
    }
}

// Exclusive scan of the block sums; records the pair count and overflow.
// One workgroup, latency-bound: 8 sums per thread in one pass up to 524,288
// Gaussians (4688 sums: 15 us by 256 threads, one sum each at a time, 6 so).
__global__ __launch_bounds__(1024) void k_scan_top(uint32_t* __restrict__ partial, size_t s_partial, int nblocks,
                                                   uint32_t* __restrict__ flags, size_t s_flags, int64_t cap)
{
    constexpr int IT = 8;
    const int q = blockIdx.x, t = threadIdx.x, lane = t & 63, w = t >> 6;
    partial += q * s_partial;
    flags += q * s_flags;
    __shared__ unsigned long long wsum[16];
    unsigned long long carry = 0;
    for (int b0 = 0; b0 < nblocks; b0 += 1024 * IT) {
        uint32_t v[IT];
#pragma unroll
        for (int i = 0; i < IT; ++i) {
            const int b = b0 + t * IT + i;
            v[i] = b < nblocks ? partial[b] : 0u;
        }
        unsigned long long sum = 0;
#pragma unroll
        for (int i = 0; i < IT; ++i) sum += v[i];
        unsigned long long x = sum;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const unsigned long long y = __shfl_up(x, o, 64);
            if (lane >= o) x += y;
        }
        if (lane == 63) wsum[w] = x;
        __syncthreads();
        unsigned long long run = carry + x - sum;
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const unsigned long long ws = wsum[k];
            run += k < w ? ws : 0ull;
            carry += ws;
        }
#pragma unroll
        for (int i = 0; i < IT; ++i) {
            const int b = b0 + t * IT + i;
            if (b < nblocks) partial[b] = (uint32_t)run;
            run += v[i];
        }
        __syncthreads();  // the next chunk's sums
    }
    if (t == 0) {
        const unsigned long long P = carry;
        flags[FL_PAIRS] = (uint32_t)(P > 0xFFFFFFFFull ? 0xFFFFFFFFull : P);
        flags[FL_OVERFLOW] = P > (unsigned long long)cap ? 1u : 0u;
        flags[FL_PUSED] = (uint32_t)(P > (unsigned long long)cap ? (unsigned long long)cap : P);
    }
}

// Emits the pair keys in depth order.  A workgroup owns 64 consecutive
// ranks; their pairs are spread over its 256 lanes (pair p belongs to the
// last rank whose first pair slot is <= p; each lane walks forward through
// the 64 prefix offsets as its p grows by 256), so the stores stay coalesced
// and the work balanced however unequal the tile counts are.
// SCAN: `partial` holds the block sums (no k_scan_top): each workgroup adds
// up the sums before its own (for a few thousand blocks at most), and the
// last active one records the pair count and overflow.
template <bool SCAN>
__global__ __launch_bounds__(256) void k_emit(const uint32_t* __restrict__ order, size_t s_order,
                                             const uint4* __restrict__ tinfo, size_t s_tinfo,
                                             uint32_t* __restrict__ flags, size_t s_flags,
                                             const uint32_t* __restrict__ partial, size_t s_partial,
                                             uint32_t* __restrict__ pkeys, size_t s_pkeys, int64_t cap,
                                             int TX, int rank_bits)
{
    const int q = blockIdx.y;
    const uint32_t nvis = flags[q * s_flags + FL_NVIS];
    const uint32_t base = blockIdx.x * EMIT_RANKS;
    if (base >= nvis) return;
    uint32_t o0 = 0;
    if constexpr (SCAN) {
        __shared__ unsigned long long s_pre;
        if (threadIdx.x == 0) s_pre = 0ull;
        __syncthreads();
        unsigned long long v = 0ull;
        for (uint32_t b = threadIdx.x; b < blockIdx.x; b += 256) v += partial[q * s_partial + b];
        if (v) atomicAdd(&s_pre, v);
        __syncthreads();
        const unsigned long long pre = s_pre;
        o0 = (uint32_t)pre;
        if (threadIdx.x == 0 && blockIdx.x == (nvis - 1) / EMIT_RANKS) {
            const unsigned long long P = pre + partial[q * s_partial + blockIdx.x];
            flags[q * s_flags + FL_PAIRS] = (uint32_t)(P > 0xFFFFFFFFull ? 0xFFFFFFFFull : P);
            flags[q * s_flags + FL_OVERFLOW] = P > (unsigned long long)cap ? 1u : 0u;
            flags[q * s_flags + FL_PUSED] = (uint32_t)(P > (unsigned long long)cap ? (unsigned long long)cap : P);
        }
    } else {
        o0 = partial[q * s_partial + blockIdx.x];
    }
    order += q * s_order;
    tinfo += q * s_tinfo;
    pkeys += q * s_pkeys;
    __shared__ uint4 s_ti[EMIT_RANKS];
    __shared__ uint32_t s_start[EMIT_RANKS + 1];
    __shared__ uint32_t s_total;
    const int lane = threadIdx.x & 63;
    if (threadIdx.x < 64) {
        const uint32_t k = base + lane;
        const uint4 ti = k < nvis ? tinfo[order[k]] : make_uint4(0, 0, 0, 0);
        uint32_t x = ti.w;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t y = __shfl_up(x, o, 64);
            if (lane >= o) x += y;
        }
        s_ti[lane] = ti;
        s_start[lane] = x - ti.w;
        if (lane == 63) {
            s_start[EMIT_RANKS] = 0xFFFFFFFFu;  // sentinel
            s_total = x;
        }
    }
    __syncthreads();
    const uint32_t total = s_total;
    int j = 0;  // largest j with s_start[j] <= p; only moves forward as p grows
    for (uint32_t p = threadIdx.x; p < total; p += 256) {
        while (s_start[j + 1] <= p) ++j;
        const uint4 t = s_ti[j];
        const uint32_t e = p - s_start[j];
        const int xa0 = t.x & 0xFFFF, xa1 = t.x >> 16, xb0 = t.y & 0xFFFF, xb1 = t.y >> 16;
        const int ty0 = t.z & 0xFFFF;
        const int na = xa1 - xa0 + 1, nb = xb1 >= xb0 ? xb1 - xb0 + 1 : 0, ncols = na + nb;
        // row = e / ncols: (e + 0.5) / ncols is at least 0.5/ncols from an
        // integer and the float product's error is below that while
        // e < 2^22 (the layout caps the tile count there)
        const int r = (int)(((float)e + 0.5f) * (1.0f / (float)ncols));
        const int c = (int)e - r * ncols;
        const int tx = c < na ? xa0 + c : xb0 + (c - na);
        const uint32_t dst = o0 + p;
        if ((int64_t)dst < cap) pkeys[dst] = ((uint32_t)((ty0 + r) * TX + tx) << rank_bits) | (base + j);
    }
}

// Tile ranges from the sorted pair keys; also resolves each pair's Gaussian.
__global__ __launch_bounds__(256) void k_ranges(const uint32_t* __restrict__ pkeys, size_t s_pkeys,
                                                const uint32_t* __restrict__ order, size_t s_order,
                                                const uint32_t* __restrict__ flags, size_t s_flags,
                                                uint32_t* __restrict__ plist, size_t s_plist,
                                                uint2* __restrict__ ranges, size_t s_ranges, int rank_bits,
                                                uint32_t T)
{
    const int q = blockIdx.y;
    const uint32_t P = flags[q * s_flags + FL_PUSED];
    pkeys += q * s_pkeys;
    ranges += q * s_ranges;
    for (uint32_t p = blockIdx.x * blockDim.x + threadIdx.x; p < P; p += gridDim.x * blockDim.x) {
        const uint32_t key = pkeys[p];
        const uint32_t t = key >> rank_bits;
        plist[q * s_plist + p] = order[q * s_order + (key & ((1u << rank_bits) - 1u))];
        const uint32_t prev = p > 0 ? (pkeys[p - 1] >> rank_bits) : 0xFFFFFFFFu;
        if (t >= T || (p > 0 && prev >= T)) continue;  // never taken for keys written by k_emit
        if (t != prev) {
            ranges[t].x = p;
            if (p > 0) ranges[prev].y = p;
        }
        if (p == P - 1) ranges[t].y = P;
    }
}

void launch_binning(const Layout& L, char* ws, hipStream_t s)
{
    const uint32_t* order = (const uint32_t*)(ws + L.vals_a);
    const uint4* tinfo = (const uint4*)(ws + L.tinfo);
    uint32_t* flags = (uint32_t*)(ws + L.flags);
    uint32_t* partial = (uint32_t*)(ws + L.partial);
    const size_t so = L.s_keys / 4, sti = L.s_tinfo / sizeof(uint4), sf = L.s_flags / 4, sp = L.s_partial / 4;
    const int nblk = (L.n + EMIT_RANKS - 1) / EMIT_RANKS;
    hipLaunchKernelGGL(k_scan_reduce, dim3(nblk, L.nq), dim3(64), 0, s, (const uint32_t*)(ws + L.keys_a), order, so,
                       (uint32_t)L.n, tinfo, sti, (const uint32_t*)(ws + L.status), L.s_status / 4, flags, sf, partial,
                       sp);
    uint32_t* pa = (uint32_t*)(ws + L.pkeys_a);
    uint32_t* pb = (uint32_t*)(ws + L.pkeys_b);
    const size_t spk = L.s_pkeys / 4;
    if (nblk <= EMIT_SCAN_BLOCKS) {
        hipLaunchKernelGGL(k_emit<true>, dim3(nblk, L.nq), dim3(256), 0, s, order, so, tinfo, sti, flags, sf,
                           partial, sp, pa, spk, L.cap, L.TX, L.rank_bits);
    } else {
        hipLaunchKernelGGL(k_scan_top, dim3(L.nq), dim3(1024), 0, s, partial, sp, nblk, flags, sf, L.cap);
        hipLaunchKernelGGL(k_emit<false>, dim3(nblk, L.nq), dim3(256), 0, s, order, so, tinfo, sti, flags, sf,
                           partial, sp, pa, spk, L.cap, L.TX, L.rank_bits);
    }
    // pairs are emitted in depth-rank order, so a stable sort on the tile
    // digits alone yields (tile, depth) order
    uint2* ranges = (uint2*)(ws + L.ranges);
    if (L.tile_bits <= TILE_PASS_MAX_BITS) {
        // one counting pass over all tile digits: the scatter writes each
        // pair's Gaussian straight into the list, and the tile ranges are
        // the scan of the per-tile totals
        const uint32_t* nd = flags + FL_PUSED;
        const uint32_t rmask = (1u << L.rank_bits) - 1u;
        uint32_t* plist = (uint32_t*)(ws + L.plist);
        const size_t spl = L.s_plist / 4;
        constexpr int WN = SORT_THREADS / 64, WW = SORT_WIDE_WAVES;
        if (L.tile_bits <= RADIX_BITS) {
            // 256 digits: the usual blocks of SORT_ITEMS keys per thread
            if (L.pair_wide)
                sort_pass<RADIX_BITS, SORT_ITEMS, false, WW>(pa, nullptr, nullptr, nullptr, spk, nd, sf, 0u,
                                                             L.rank_bits, L.pair_blocks, L, ws, order, so, plist,
                                                             spl, rmask, s, ranges);
            else
                sort_pass<RADIX_BITS, SORT_ITEMS, false, WN>(pa, nullptr, nullptr, nullptr, spk, nd, sf, 0u,
                                                             L.rank_bits, L.pair_blocks, L, ws, order, so, plist,
                                                             spl, rmask, s, ranges);
        } else {
            // 1024 digits: blocks of TILE_PASS_ITEMS (TILE_PASS_WIDE_ITEMS)
            // keys per thread keep the digit-by-block count matrix small
            if (L.pair_wide)
                sort_pass<TILE_PASS_MAX_BITS, TILE_PASS_WIDE_ITEMS, false, WW>(pa, nullptr, nullptr, nullptr, spk, nd,
                                                                          sf, 0u, L.rank_bits, L.tile_blocks, L, ws,
                                                                          order, so, plist, spl, rmask, s, ranges);
            else
                sort_pass<TILE_PASS_MAX_BITS, TILE_PASS_ITEMS, false, WN>(pa, nullptr, nullptr, nullptr, spk, nd,
                                                                          sf, 0u, L.rank_bits, L.tile_blocks, L, ws,
                                                                          order, so, plist, spl, rmask, s, ranges);
        }
        // (the scatter's block 0 wrote the tile ranges: the digit ranges)
        return;
    }
    const int which = radix_sort(pa, pb, nullptr, nullptr, spk, flags + FL_PUSED, sf, 0, L.rank_bits,
                                 L.pair_passes, L.pair_blocks, L.pair_wide != 0, L, ws, s);
    uint32_t* sorted = which ? pb : pa;
    launch_fill_u32((uint32_t*)ranges, (size_t)L.T * 2, L.s_ranges / 4, L.nq, 0u, s);
    const int64_t rblocks = (L.cap + 255) / 256;
    dim3 grid((unsigned)(rblocks < 1024 ? rblocks : 1024), L.nq);
    hipLaunchKernelGGL(k_ranges, grid, dim3(256), 0, s, sorted, spk, order, so, flags, sf,
                       (uint32_t*)(ws + L.plist), L.s_plist / 4, ranges, L.s_ranges / sizeof(uint2), L.rank_bits,
                       (uint32_t)L.T);
}

}  // namespace gs
