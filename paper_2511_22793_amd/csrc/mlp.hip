// Attribute network on the BF16 matrix cores of gfx950
// (v_mfma_f32_16x16x32_bf16, FP32 accumulation).
//
// Per (set s, Gaussian g) row, a shared form of the emission predictor of
// Eq. (1):
//   h1 = relu(Z1[g] + c[s])          Z1 = E W1e^T (query-independent),
//                                    c[s] = b1 + W1t gamma(tx_s)
//   h2 = relu(W2 h1 + b2)
//   o  = W3 h2 + b3                  (64 amplitudes, 64 phases)
//   A_f = sigmoid(o_f - ln d_sg), phi_f = o_{64+f},  attr = A e^{j phi}
// with d_sg = max(|tx_s - mu_g|, r_near).  Rows come from a list of
// Gaussians (e.g. those that reach some pixel) shared by all sets or one
// list per set.
//
// MFMA 16x16x32 operand layout (lane l of a wave):
//   A (16 x 32): row l%16, k = 8*(l/16) .. +7   (8 bf16)
//   B (32 x 16): col l%16, k = 8*(l/16) .. +7   (8 bf16)
//   C (16 x 16): col l%16, rows 4*(l/16) .. +3  (4 floats)
#include "common.h"
#include "mlp.h"

namespace gs {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f32x4 mfma(bf16x8 a, bf16x8 b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ uint16_t f2bf(float x)  // round to nearest even
{
    uint32_t u = __float_as_uint(x);
    if ((u & 0x7F800000u) == 0x7F800000u && (u & 0x7FFFFFu)) return (uint16_t)((u >> 16) | 0x40);  // NaN
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

__device__ __forceinline__ float bf2f(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

__device__ __forceinline__ bf16x8 load8(const uint16_t* p)  // 16-byte aligned
{
    const uint4 v = *(const uint4*)p;
    bf16x8 r;
    __builtin_memcpy(&r, &v, 16);
    return r;
}

// ---- Z1 = E W1e^T, one wave per 16 Gaussians -----------------------------
__global__ __launch_bounds__(256) void k_mlp_embed(const uint16_t* __restrict__ E, int n,
                                                   const uint16_t* __restrict__ W1, float* __restrict__ Z1)
{
    const int lane = threadIdx.x & 63;
    const int tile = blockIdx.x * 4 + (threadIdx.x >> 6);
    const int r0 = tile * 16;
    if (r0 >= n) return;
    const int row = r0 + (lane & 15);
    bf16x8 a = {};
    if (row < n) a = load8(E + (size_t)row * MLP_EMB + 8 * (lane >> 4));
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
        const bf16x8 b = load8(W1 + (size_t)(nt * 16 + (lane & 15)) * MLP_IN + 8 * (lane >> 4));
        f32x4 c = {0, 0, 0, 0};
        c = mfma(a, b, c);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int rr = r0 + 4 * (lane >> 4) + i;
            if (rr < n) Z1[(size_t)rr * MLP_HID + nt * 16 + (lane & 15)] = c[i];
        }
    }
}

// ---- c[s] = b1 + W1t bf16(gamma(tx_s)) -----------------------------------
__global__ __launch_bounds__(64) void k_mlp_bias(const uint16_t* __restrict__ W1, const float* __restrict__ b1,
                                                 const float* __restrict__ tx, float lo0, float lo1, float lo2,
                                                 float hi0, float hi1, float hi2, float* __restrict__ cb,
                                                 uint16_t* __restrict__ genc)
{
    const int s = blockIdx.x, j = threadIdx.x;
    __shared__ float g[MLP_ENC];
    __shared__ double su[3];
    if (j < 3) {
        const float lo = j == 0 ? lo0 : (j == 1 ? lo1 : lo2), hi = j == 0 ? hi0 : (j == 1 ? hi1 : hi2);
        const double u = 2.0 * ((double)tx[3 * s + j] - lo) / ((double)hi - lo) - 1.0;
        su[j] = u;
        g[j] = bf2f(f2bf((float)u));
    }
    __syncthreads();
    if (j < 3 * MLP_BANDS) {  // one (band, coordinate) angle per thread
        const int k = j / 3, d = j % 3;
        const double a = ldexp(M_PI, k) * su[d];
        g[3 + 6 * k + d] = bf2f(f2bf((float)sin(a)));
        g[6 + 6 * k + d] = bf2f(f2bf((float)cos(a)));
    }
    __syncthreads();
    float acc = b1[j];
    for (int k = 0; k < MLP_ENC; ++k) acc = fmaf(bf2f(W1[(size_t)j * MLP_IN + MLP_EMB + k]), g[k], acc);
    cb[s * MLP_HID + j] = acc;
    if (genc)
        for (int k = j; k < MLP_ENC; k += 64) genc[s * MLP_ENC_PAD + k] = f2bf(g[k]);
}

// ---------------------------------------------------------------------------
// The row kernels: one wave per 16 rows, every layer as (weights) x (rows):
// the weights are the A operand (from LDS), the rows the columns of B.  A
// result tile then has a row's 4 consecutive features in one lane (row
// lane%16, features 16 nt + 4 (lane/16) + i), so it goes to the wave's LDS
// rows as one 8-byte store, comes back as the next layer's B operand (8
// consecutive features of a row) as one 16-byte load, and the attribute row
// is read and written in 32-byte pieces.  Waves share the staged weights
// only; nothing in the row loop waits for another wave.
// ---------------------------------------------------------------------------
constexpr int WROW = MLP_HID + 8;   // LDS row of 64 bf16 (16-byte aligned, fewer bank conflicts)
constexpr int EROW = MLP_EMB + 8;   // LDS row of 32 bf16

__device__ __forceinline__ void wave_sync_lds()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// dst[r][0 .. ncols) = W[r * ld .. ] for r < rows, in 16-byte chunks
template <int NCOLS, int DROW>
__device__ __forceinline__ void stage_rows(uint16_t* dst, const uint16_t* __restrict__ W, int ld, int rows)
{
#pragma unroll 4
    for (int c = threadIdx.x; c < rows * (NCOLS / 8); c += blockDim.x) {
        const int r = c / (NCOLS / 8), k = (c % (NCOLS / 8)) * 8;
        *(uint4*)(dst + r * DROW + k) = *(const uint4*)(W + (size_t)r * ld + k);
    }
}

// A or B operand of the transpose of a row-major LDS matrix: element k of
// the lane's 8 is base[8 (lane/16) + k][lane % 16] (two transposing loads of
// 4 rows x 16 columns per 16 lanes)
typedef short s16x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ bf16x8 load8_tr(const uint16_t* base, int ld, int lane)
{
    typedef __attribute__((address_space(3))) s16x4 Lds4;
    const uint16_t* p = base + (8 * (lane >> 4) + ((lane & 15) >> 2)) * ld + 4 * (lane & 3);
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((Lds4*)p);
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((Lds4*)(p + 4 * ld));
    bf16x8 r;
    __builtin_memcpy(&r, &lo, 8);
    __builtin_memcpy((char*)&r + 8, &hi, 8);
    return r;
}

__device__ __forceinline__ uint2 pack4(const float* x)  // 4 bf16 (round to nearest even)
{
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    const bf16x2 a = {(__bf16)x[0], (__bf16)x[1]}, b = {(__bf16)x[2], (__bf16)x[3]};
    uint2 v;
    __builtin_memcpy(&v.x, &a, 4);
    __builtin_memcpy(&v.y, &b, 4);
    return v;
}

__device__ __forceinline__ void load_vec4(float* d, const float* p, bool wide)
{
    if (wide) {
        const float4 v = *(const float4*)p;
        d[0] = v.x; d[1] = v.y; d[2] = v.z; d[3] = v.w;
    } else {
        const float2 v = ((const float2*)p)[0], u = ((const float2*)p)[1];
        d[0] = v.x; d[1] = v.y; d[2] = u.x; d[3] = u.y;
    }
}

__device__ __forceinline__ void store_vec4(float* p, float x, float y, float z, float w, bool wide)
{
    if (wide) {
        *(float4*)p = make_float4(x, y, z, w);
    } else {
        ((float2*)p)[0] = make_float2(x, y);
        ((float2*)p)[1] = make_float2(z, w);
    }
}

// ln max(|tx - mean_g|, r_near)
__device__ __forceinline__ float log_dist(const MlpArgs& A, int g, float tx0, float tx1, float tx2)
{
    const float e0 = A.mean[g] - tx0, e1 = A.mean[A.n + g] - tx1, e2 = A.mean[2 * A.n + g] - tx2;
    return logf(fmaxf(sqrtf(e0 * e0 + e1 * e1 + e2 * e2), A.r_near));
}

// Bound: the attribute rows written and the saved activations (768 bytes a
// row at 64 channels) against one sincos and one exp per channel.  At 320,176
// rows of 64 channels 86 us
// (109 with the rows as the A operand: 2-byte LDS stores, workgroup barriers
// between the layers).
template <int NF>
__global__ __launch_bounds__(256) void k_mlp_fwd(MlpArgs A)
{
    const int s = blockIdx.y;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int r = lane & 15, q = lane >> 4;
    const uint32_t* list = A.list + (size_t)s * A.list_stride;
    const int count = (int)A.count[A.count_stride ? s : 0];
    if ((int)blockIdx.x * 64 >= count) return;  // no rows for this workgroup
    __shared__ __attribute__((aligned(16))) uint16_t s_W2[MLP_HID * WROW];
    __shared__ __attribute__((aligned(16))) uint16_t s_W3[2 * NF * WROW];
    __shared__ __attribute__((aligned(16))) uint16_t s_h[4][16 * WROW];
    __shared__ __attribute__((aligned(16))) float s_b[MLP_HID + 2 * NF];  // b2, b3
    for (int k = threadIdx.x; k < MLP_HID + 2 * NF; k += 256) s_b[k] = k < MLP_HID ? A.b2[k] : A.b3[k - MLP_HID];
    stage_rows<MLP_HID, WROW>(s_W2, A.W2, MLP_HID, MLP_HID);
    stage_rows<MLP_HID, WROW>(s_W3, A.W3, MLP_HID, 2 * NF);
    const float* cs = A.cb + s * MLP_HID;
    const float tx0 = A.tx[3 * s], tx1 = A.tx[3 * s + 1], tx2 = A.tx[3 * s + 2];
    uint16_t* h2s = s_h[w];
    __syncthreads();
    for (int base = blockIdx.x * 64 + w * 16; base < count; base += gridDim.x * 64) {
        const int i = base + r;
        const bool on = i < count;
        const int g = on ? (int)list[i] : 0;
        const size_t save = ((size_t)s * A.row_cap + i) * MLP_HID;
        // h1 = relu(Z1[g] + c[s]): features 32 kc + 8 q .. + 7 of row r
        bf16x8 hb[2];
#pragma unroll
        for (int kc = 0; kc < 2; ++kc) {
            const int f = 32 * kc + 8 * q;
            float z[8], c[8], h[8];
            load_vec4(z, A.Z1 + (size_t)g * MLP_HID + f, true);
            load_vec4(z + 4, A.Z1 + (size_t)g * MLP_HID + f + 4, true);
            load_vec4(c, cs + f, true);
            load_vec4(c + 4, cs + f + 4, true);
#pragma unroll
            for (int j = 0; j < 8; ++j) h[j] = on ? fmaxf(z[j] + c[j], 0.0f) : 0.0f;
            const uint2 v[2] = {pack4(h), pack4(h + 4)};
            __builtin_memcpy(&hb[kc], v, 16);
            if (A.save_h1 && on) *(uint4*)(A.save_h1 + save + f) = make_uint4(v[0].x, v[0].y, v[1].x, v[1].y);
        }
        // h2 = relu(W2 h1 + b2)
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) {
            f32x4 c = {0, 0, 0, 0};
#pragma unroll
            for (int kc = 0; kc < 2; ++kc) c = mfma(load8(s_W2 + (nt * 16 + r) * WROW + kc * 32 + 8 * q), hb[kc], c);
            float h[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) h[j] = fmaxf(c[j] + s_b[nt * 16 + 4 * q + j], 0.0f);
            *(uint2*)(h2s + r * WROW + nt * 16 + 4 * q) = pack4(h);
        }
        wave_sync_lds();
#pragma unroll
        for (int kc = 0; kc < 2; ++kc) {
            hb[kc] = load8(h2s + r * WROW + kc * 32 + 8 * q);
            if (A.save_h2 && on) {
                uint4 v;
                __builtin_memcpy(&v, &hb[kc], 16);
                *(uint4*)(A.save_h2 + save + kc * 32 + 8 * q) = v;
            }
        }
        wave_sync_lds();
        // o = W3 h2 + b3, amplitude and phase tiles of the same channels together
        const float lnd = log_dist(A, g, tx0, tx1, tx2);
        float* out = A.attr + (size_t)s * A.attr_stride + (size_t)g * (2 * NF);
#pragma unroll
        for (int nt = 0; nt < NF / 16; ++nt) {
            const int f = nt * 16 + 4 * q;
            f32x4 ca = {0, 0, 0, 0}, cp = {0, 0, 0, 0};
#pragma unroll
            for (int kc = 0; kc < 2; ++kc) {
                ca = mfma(load8(s_W3 + (nt * 16 + r) * WROW + kc * 32 + 8 * q), hb[kc], ca);
                cp = mfma(load8(s_W3 + (NF + nt * 16 + r) * WROW + kc * 32 + 8 * q), hb[kc], cp);
            }
            float re[4], im[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float oa = ca[j] + s_b[MLP_HID + f + j] - lnd;
                const float op = cp[j] + s_b[MLP_HID + NF + f + j];
                const float amp = 1.0f / (1.0f + expf(-oa));
                float sn, cs_;
                sincosf(op, &sn, &cs_);
                re[j] = amp * cs_;
                im[j] = amp * sn;
            }
            if (on) {
                store_vec4(out + 2 * f, re[0], im[0], re[1], im[1], A.wide);
                store_vec4(out + 2 * f + 4, re[2], im[2], re[3], im[3], A.wide);
            }
        }
    }
}

// Backward through the epilogue and the three layers for each row.  Writes
// the rounded products' operands (d_o, dZ2, dZ1 as bf16) for the weight
// gradients, bias sums, per-set dZ1 sums and dE (atomics).  The transposed
// weights of the products come from the staged rows by transposing LDS
// loads.  A row's attribute gradients are loaded ahead of its first layer
// (one wait for all of them); the bias sums stay in registers over the
// wave's rows and are reduced over lanes and waves once.
// Bound: 512 bytes of d_attr, 256 of saved activations read and 512 of saved
// gradients written per row against sincos, exp and the chain rule per
// channel.  At 320,176 rows of 64 channels 202 us
// (364 with loads waited for one by one, barriers between the layers and
// transposed weight copies in memory).
template <int NF>
__global__ __launch_bounds__(256, 2) void k_mlp_bwd_data(MlpArgs A)
{
    constexpr int OROW = 2 * NF + 8;
    const int s = blockIdx.y;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int r = lane & 15, q = lane >> 4;
    const uint32_t* list = A.list + (size_t)s * A.list_stride;
    const int count = (int)A.count[A.count_stride ? s : 0];
    // only workgroups with rows run (the grid is sized for the largest count)
    if ((int)blockIdx.x * 64 >= count) return;
    __shared__ __attribute__((aligned(16))) uint16_t s_W3[2 * NF * WROW];
    __shared__ __attribute__((aligned(16))) uint16_t s_W2[MLP_HID * WROW];
    __shared__ __attribute__((aligned(16))) uint16_t s_W1[MLP_HID * EROW];
    __shared__ __attribute__((aligned(16))) uint16_t s_do[4][16 * OROW];
    __shared__ __attribute__((aligned(16))) uint16_t s_dz[4][16 * WROW];
    __shared__ __attribute__((aligned(16))) float s_b[2 * NF];  // b3
    __shared__ float s_sum[2 * NF + 2 * MLP_HID];
    for (int k = threadIdx.x; k < 2 * NF; k += 256) s_b[k] = A.b3[k];
    stage_rows<MLP_HID, WROW>(s_W3, A.W3, MLP_HID, 2 * NF);
    stage_rows<MLP_HID, WROW>(s_W2, A.W2, MLP_HID, MLP_HID);
    stage_rows<MLP_EMB, EROW>(s_W1, A.W1, MLP_IN, MLP_HID);
    for (int k = threadIdx.x; k < 2 * NF + 2 * MLP_HID; k += 256) s_sum[k] = 0.0f;
    const float tx0 = A.tx[3 * s], tx1 = A.tx[3 * s + 1], tx2 = A.tx[3 * s + 2];
    uint16_t *dos = s_do[w], *dzs = s_dz[w];
    float db3[2 * NF / 16][4], db2[4][4], dc[4][4];
#pragma unroll
    for (int nt = 0; nt < 2 * NF / 16; ++nt)
#pragma unroll
        for (int j = 0; j < 4; ++j) db3[nt][j] = 0.0f;
#pragma unroll
    for (int nt = 0; nt < 4; ++nt)
#pragma unroll
        for (int j = 0; j < 4; ++j) db2[nt][j] = dc[nt][j] = 0.0f;
    __syncthreads();
    for (int base = blockIdx.x * 64 + w * 16; base < count; base += gridDim.x * 64) {
        const int i = base + r;
        const bool on = i < count;
        const int g = on ? (int)list[i] : 0;
        const size_t row = (size_t)s * A.row_cap + i;
        // the row's attribute gradients: channels 16 nt + 4 q .. + 3
        float da[NF / 16][8];
        const float* dat = A.d_attr + (size_t)s * A.attr_stride + (size_t)g * (2 * NF) + 8 * q;
        bf16x8 hb[2] = {};
        uint2 h1v[4] = {}, h2v[4] = {};
#pragma unroll
        for (int nt = 0; nt < NF / 16; ++nt)
#pragma unroll
            for (int j = 0; j < 8; ++j) da[nt][j] = 0.0f;
        if (on) {
#pragma unroll
            for (int kc = 0; kc < 2; ++kc) hb[kc] = load8(A.save_h2 + row * MLP_HID + kc * 32 + 8 * q);
#pragma unroll
            for (int nt = 0; nt < NF / 16; ++nt) {
                load_vec4(da[nt], dat + 32 * nt, A.wide);
                load_vec4(da[nt] + 4, dat + 32 * nt + 4, A.wide);
            }
#pragma unroll
            for (int nt = 0; nt < 4; ++nt) {
                h2v[nt] = *(const uint2*)(A.save_h2 + row * MLP_HID + nt * 16 + 4 * q);
                h1v[nt] = *(const uint2*)(A.save_h1 + row * MLP_HID + nt * 16 + 4 * q);
            }
        }
        const float lnd = log_dist(A, g, tx0, tx1, tx2);
        if (A.clear && on) {
            float* cl = A.clear + (size_t)s * A.attr_stride + (size_t)g * (2 * NF) + 8 * q;
#pragma unroll
            for (int nt = 0; nt < NF / 16; ++nt) {
                store_vec4(cl + 32 * nt, 0.0f, 0.0f, 0.0f, 0.0f, A.wide);
                store_vec4(cl + 32 * nt + 4, 0.0f, 0.0f, 0.0f, 0.0f, A.wide);
            }
        }
        // o again, d_o from d_attr
#pragma unroll
        for (int nt = 0; nt < NF / 16; ++nt) {
            const int f = nt * 16 + 4 * q;
            f32x4 ca = {0, 0, 0, 0}, cp = {0, 0, 0, 0};
#pragma unroll
            for (int kc = 0; kc < 2; ++kc) {
                ca = mfma(load8(s_W3 + (nt * 16 + r) * WROW + kc * 32 + 8 * q), hb[kc], ca);
                cp = mfma(load8(s_W3 + (NF + nt * 16 + r) * WROW + kc * 32 + 8 * q), hb[kc], cp);
            }
            float va[4], vp[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float oa = ca[j] + s_b[f + j] - lnd;
                const float op = cp[j] + s_b[NF + f + j];
                const float amp = 1.0f / (1.0f + expf(-oa));
                float sn, cs_;
                sincosf(op, &sn, &cs_);
                const float gx = da[nt][2 * j], gy = da[nt][2 * j + 1];
                va[j] = on ? (gx * cs_ + gy * sn) * amp * (1.0f - amp) : 0.0f;
                vp[j] = on ? amp * (-gx * sn + gy * cs_) : 0.0f;
                db3[nt][j] += va[j];
                db3[nt + NF / 16][j] += vp[j];
            }
            *(uint2*)(dos + r * OROW + f) = pack4(va);
            *(uint2*)(dos + r * OROW + NF + f) = pack4(vp);
        }
        wave_sync_lds();
        // dh2 = d_o W3 (K = 2 NF in 32-wide chunks), dZ2 = dh2 [h2 > 0]
        f32x4 dh[4];
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) dh[nt] = f32x4{0, 0, 0, 0};
#pragma unroll
        for (int kc = 0; kc < 2 * NF / 32; ++kc) {
            const bf16x8 b = load8(dos + r * OROW + kc * 32 + 8 * q);
            if (on) {
                uint4 v;
                __builtin_memcpy(&v, &b, 16);
                *(uint4*)(A.save_do + row * 2 * NF + kc * 32 + 8 * q) = v;
            }
#pragma unroll
            for (int nt = 0; nt < 4; ++nt) dh[nt] = mfma(load8_tr(s_W3 + kc * 32 * WROW + nt * 16, WROW, lane), b, dh[nt]);
        }
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) {
            uint16_t h[4];
            __builtin_memcpy(h, &h2v[nt], 8);
            float v[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                v[j] = dh[nt][j] * (bf2f(h[j]) > 0.0f ? 1.0f : 0.0f);
                db2[nt][j] += v[j];
            }
            *(uint2*)(dzs + r * WROW + nt * 16 + 4 * q) = pack4(v);
        }
        wave_sync_lds();
        // dh1 = dZ2 W2, dZ1 = dh1 [h1 > 0]
        f32x4 d1[4];
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) d1[nt] = f32x4{0, 0, 0, 0};
#pragma unroll
        for (int kc = 0; kc < 2; ++kc) {
            const bf16x8 b = load8(dzs + r * WROW + kc * 32 + 8 * q);
            if (on) {
                uint4 v;
                __builtin_memcpy(&v, &b, 16);
                *(uint4*)(A.save_dz2 + row * MLP_HID + kc * 32 + 8 * q) = v;
            }
#pragma unroll
            for (int nt = 0; nt < 4; ++nt) d1[nt] = mfma(load8_tr(s_W2 + kc * 32 * WROW + nt * 16, WROW, lane), b, d1[nt]);
        }
        wave_sync_lds();
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) {
            uint16_t h[4];
            __builtin_memcpy(h, &h1v[nt], 8);
            float v[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                v[j] = d1[nt][j] * (bf2f(h[j]) > 0.0f ? 1.0f : 0.0f);
                dc[nt][j] += v[j];
            }
            *(uint2*)(dzs + r * WROW + nt * 16 + 4 * q) = pack4(v);
        }
        wave_sync_lds();
        // dE[g] += dZ1 W1e
        f32x4 de[2];
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) de[nt] = f32x4{0, 0, 0, 0};
#pragma unroll
        for (int kc = 0; kc < 2; ++kc) {
            const bf16x8 b = load8(dzs + r * WROW + kc * 32 + 8 * q);
            if (on) {
                uint4 v;
                __builtin_memcpy(&v, &b, 16);
                *(uint4*)(A.save_dz1 + row * MLP_HID + kc * 32 + 8 * q) = v;
            }
#pragma unroll
            for (int nt = 0; nt < 2; ++nt) de[nt] = mfma(load8_tr(s_W1 + kc * 32 * EROW + nt * 16, EROW, lane), b, de[nt]);
        }
        if (on) {
#pragma unroll
            for (int nt = 0; nt < 2; ++nt)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    unsafeAtomicAdd(A.dE + (size_t)g * MLP_EMB + nt * 16 + 4 * q + j, de[nt][j]);
        }
        wave_sync_lds();  // the next rows reuse the LDS rows
    }
    // bias sums over the wave's rows (lanes of one q), then over the waves
    auto flush = [&](float (*v)[4], int tiles, int off) {
#pragma unroll
        for (int nt = 0; nt < 8; ++nt) {
            if (nt >= tiles) break;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                float x = v[nt][j];
                x += __shfl_xor(x, 1, 64);
                x += __shfl_xor(x, 2, 64);
                x += __shfl_xor(x, 4, 64);
                x += __shfl_xor(x, 8, 64);
                if (r == 0) atomicAdd(&s_sum[off + nt * 16 + 4 * q + j], x);
            }
        }
    };
    flush(db3, 2 * NF / 16, 0);
    flush(db2, 4, 2 * NF);
    flush(dc, 4, 2 * NF + MLP_HID);
    __syncthreads();
    for (int k = threadIdx.x; k < 2 * NF; k += 256) unsafeAtomicAdd(A.db3 + k, s_sum[k]);
    if (threadIdx.x < MLP_HID) {
        unsafeAtomicAdd(A.db2 + threadIdx.x, s_sum[2 * NF + threadIdx.x]);
        unsafeAtomicAdd(A.dc + s * MLP_HID + threadIdx.x, s_sum[2 * NF + MLP_HID + threadIdx.x]);
    }
}

// ---------------------------------------------------------------------------
// Split-K weight gradients C[M][N] = sum over rows of a[r][m] b[r][n] (bf16
// operands, FP32 accumulation), all three in one launch (blockIdx.y):
//   0: dW3 = d_o^T h2    1: dW2 = dZ2^T h1    2: dW1e = dZ1^T E[g]
// Each workgroup (8 waves) takes K blocks of WG_ROWS rows of a set
// round-robin: the rows go row-major through LDS (16-byte loads and stores,
// the next block's in flight in registers behind the products) and both
// operands leave it through transposing loads, so no element is moved on its
// own.  Bound: reading the saved rows once (246 MB at 320,176 rows of 64
// channels): 73 us (1452 with 2-byte transposing LDS stores of 32-row blocks).
// ---------------------------------------------------------------------------
constexpr int WG_WAVES = 8;
constexpr int WG_ROWS = 128;  // rows per K block

struct WgradArgs {
    const uint16_t *do_, *h2, *dz2, *h1, *dz1, *E;
    const uint32_t* list;
    size_t list_stride;
    const uint32_t* count;
    int count_stride, S;
    size_t cap;
    float* partial;
};

constexpr int WG3_LEN1 = MLP_HID * MLP_HID, WG3_LEN2 = MLP_HID * MLP_EMB;
__host__ __device__ constexpr int wg3_len0(int nf) { return 2 * nf * MLP_HID; }

template <int M, int N, bool GATHER>
__device__ __forceinline__ void wgrad_body(uint16_t* lds, const WgradArgs& A, const uint16_t* __restrict__ a,
                                           const uint16_t* __restrict__ b, float* __restrict__ P)
{
    constexpr int AR = M + 8, BR = N + 8;
    constexpr int NT = N / 16, PER = (M / 16) * NT / WG_WAVES;
    constexpr int T = 64 * WG_WAVES;
    constexpr int CA = M / 8, CB = N / 8;  // 16-byte chunks of a row
    constexpr int NA = WG_ROWS * CA / T, NB = WG_ROWS * CB / T;
    static_assert(PER >= 1 && NA >= 1 && NB >= 1, "wgrad shapes");
    uint16_t *sA = lds, *sB = lds + WG_ROWS * AR;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int mt = w * PER / NT, nt0 = (w * PER) % NT;
    f32x4 acc[PER];
#pragma unroll
    for (int t = 0; t < PER; ++t) acc[t] = f32x4{0, 0, 0, 0};
    uint4 va[NA], vb[NB];
    auto load = [&](int s, int cnt, int kb) {
#pragma unroll
        for (int u = 0; u < NA; ++u) {
            const int e = u * T + threadIdx.x, i = kb * WG_ROWS + e / CA;
            va[u] = i < cnt ? *(const uint4*)(a + ((size_t)s * A.cap + i) * M + (e % CA) * 8) : make_uint4(0, 0, 0, 0);
        }
#pragma unroll
        for (int u = 0; u < NB; ++u) {
            const int e = u * T + threadIdx.x, i = kb * WG_ROWS + e / CB;
            vb[u] = make_uint4(0, 0, 0, 0);
            if (i < cnt) {
                const size_t row = GATHER ? (size_t)A.list[(size_t)s * A.list_stride + i] : (size_t)s * A.cap + i;
                vb[u] = *(const uint4*)(b + row * N + (e % CB) * 8);
            }
        }
    };
    // K blocks enumerate (set, block): s and kb name the one in registers
    int s = 0, kb = blockIdx.x, cnt = 0;
    auto settle = [&]() {  // moves (s, kb) to an existing block, or s to S
        for (; s < A.S; ++s) {
            cnt = (int)A.count[A.count_stride ? s : 0];
            const int nblk = (cnt + WG_ROWS - 1) / WG_ROWS;
            if (kb < nblk) return;
            kb -= nblk;
        }
    };
    settle();
    if (s < A.S) load(s, cnt, kb);
    while (s < A.S) {
        __syncthreads();  // the previous block's products are done
#pragma unroll
        for (int u = 0; u < NA; ++u) {
            const int e = u * T + threadIdx.x;
            *(uint4*)(sA + (e / CA) * AR + (e % CA) * 8) = va[u];
        }
#pragma unroll
        for (int u = 0; u < NB; ++u) {
            const int e = u * T + threadIdx.x;
            *(uint4*)(sB + (e / CB) * BR + (e % CB) * 8) = vb[u];
        }
        __syncthreads();
        kb += gridDim.x;
        settle();
        if (s < A.S) load(s, cnt, kb);
#pragma unroll
        for (int kc = 0; kc < WG_ROWS / 32; ++kc) {
            const bf16x8 av = load8_tr(sA + kc * 32 * AR + mt * 16, AR, lane);
#pragma unroll
            for (int t = 0; t < PER; ++t)
                acc[t] = mfma(av, load8_tr(sB + kc * 32 * BR + (nt0 + t) * 16, BR, lane), acc[t]);
        }
    }
#pragma unroll
    for (int t = 0; t < PER; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i)
            P[(mt * 16 + 4 * (lane >> 4) + i) * N + (nt0 + t) * 16 + (lane & 15)] = acc[t][i];
}

template <int NF>
__global__ __launch_bounds__(64 * WG_WAVES) void k_wgrad3(WgradArgs A)
{
    __shared__ __attribute__((aligned(16))) uint16_t lds[WG_ROWS * (2 * NF + 8 + MLP_HID + 8)];
    const size_t P = gridDim.x, x = blockIdx.x;
    constexpr int LEN0 = wg3_len0(NF);
    if (blockIdx.y == 0)
        wgrad_body<2 * NF, MLP_HID, false>(lds, A, A.do_, A.h2, A.partial + x * LEN0);
    else if (blockIdx.y == 1)
        wgrad_body<MLP_HID, MLP_HID, false>(lds, A, A.dz2, A.h1, A.partial + P * LEN0 + x * WG3_LEN1);
    else
        wgrad_body<MLP_HID, MLP_EMB, true>(lds, A, A.dz1, A.E, A.partial + P * (LEN0 + WG3_LEN1) + x * WG3_LEN2);
}

// Sums the partials of the three weight gradients into dW3, dW2 and the
// embedding columns of dW1 (the first `rb` workgroups); the others form the
// encoding columns and the bias: dW1t = sum_s dc_s gamma_s^T (bf16 gamma),
// db1 = sum_s dc_s, four columns each.
template <int NF>
__global__ __launch_bounds__(256) void k_mlp_reduce(const float* __restrict__ partial, int nparts, int rb,
                                                    const float* __restrict__ dc, const uint16_t* __restrict__ genc,
                                                    int S, float* __restrict__ dW3, float* __restrict__ dW2,
                                                    float* __restrict__ dW1, float* __restrict__ db1)
{
    if ((int)blockIdx.x >= rb) {
        const int j = threadIdx.x & 63;  // hidden unit
        const int k = ((int)blockIdx.x - rb) * 4 + (threadIdx.x >> 6);
        if (k > MLP_ENC) return;
        // the sets added in order, 16 sets' loads in flight ahead of the products
        float acc = 0.0f;
        int s = 0;
        for (; s + 16 <= S; s += 16) {
            float d[16], g[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                d[u] = dc[(s + u) * MLP_HID + j];
                g[u] = k < MLP_ENC ? bf2f(genc[(s + u) * MLP_ENC_PAD + k]) : 1.0f;
            }
#pragma unroll
            for (int u = 0; u < 16; ++u) acc += d[u] * g[u];
        }
        for (; s < S; ++s) acc += dc[s * MLP_HID + j] * (k < MLP_ENC ? bf2f(genc[s * MLP_ENC_PAD + k]) : 1.0f);
        if (k < MLP_ENC) dW1[(size_t)j * MLP_IN + MLP_EMB + k] = acc;
        else db1[j] = acc;
        return;
    }
    constexpr int WG3_LEN0 = wg3_len0(NF);
    int e = blockIdx.x * blockDim.x + threadIdx.x;
    const float* base = partial;
    int len = WG3_LEN0, ncols = MLP_HID, ld = MLP_HID;
    float* out = dW3;
    if (e >= WG3_LEN0) {
        e -= WG3_LEN0;
        base += (size_t)nparts * WG3_LEN0;
        len = WG3_LEN1;
        out = dW2;
        if (e >= WG3_LEN1) {
            e -= WG3_LEN1;
            base += (size_t)nparts * WG3_LEN1;
            len = WG3_LEN2;
            ncols = MLP_EMB;
            ld = MLP_IN;
            out = dW1;
            if (e >= WG3_LEN2) return;
        }
    }
    // the partials added in order, 16 loads in flight ahead of the additions
    float acc = 0.0f;
    int p = 0;
    for (; p + 16 <= nparts; p += 16) {
        float b[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) b[u] = base[(size_t)(p + u) * len + e];
#pragma unroll
        for (int u = 0; u < 16; ++u) acc += b[u];
    }
    for (; p < nparts; ++p) acc += base[(size_t)p * len + e];
    out[(size_t)(e / ncols) * ld + e % ncols] = acc;
}

// Workgroups per set of the row kernels: about two rounds of the chip's
// resident ones over all sets, no more than a set's rows need.
static int rows_grid(const gs_mlp_rows* rows)
{
    if (rows->grid_x > 0) return rows->grid_x;
    const int64_t want = std::max<int64_t>(32, 512 / rows->n_sets);
    return (int)std::min<int64_t>(want, (rows->row_cap + 63) / 64);
}

}  // namespace gs

using namespace gs;

extern "C" {

gs_status gs_mlp_embed(const gs_mlp* net, const uint16_t* E, int32_t n, float* Z1, void* stream)
{
    if (!net || !net->W1 || !E || !Z1 || n < 1) return GS_ERR_INVALID_ARG;
    (void)hipGetLastError();
    const int tiles = (n + 15) / 16;
    hipLaunchKernelGGL(k_mlp_embed, dim3((tiles + 3) / 4), dim3(256), 0, (hipStream_t)stream, E, n, net->W1, Z1);
    return hipGetLastError() == hipSuccess ? GS_OK : GS_ERR_HIP;
}

static gs_status check_rows(const gs_mlp* net, const gs_mlp_rows* rows, const float* mean, int32_t n)
{
    if (!net || !rows || !mean || n < 1) return GS_ERR_INVALID_ARG;
    if (net->n_chan != 32 && net->n_chan != 64) return GS_ERR_INVALID_ARG;
    if (!net->W1 || !net->b1 || !net->W2 || !net->b2 || !net->W3 || !net->b3) return GS_ERR_INVALID_ARG;
    if (!rows->tx || !rows->list || !rows->count || rows->n_sets < 1 || rows->n_sets > 65535) return GS_ERR_INVALID_ARG;
    if (rows->row_cap < 1 || !(net->r_near > 0.0f)) return GS_ERR_INVALID_ARG;
    for (int k = 0; k < 3; ++k)
        if (!(net->box_hi[k] > net->box_lo[k])) return GS_ERR_INVALID_ARG;
    return GS_OK;
}

gs_status gs_mlp_forward(const gs_mlp* net, const float* Z1, const float* mean, int32_t n, const gs_mlp_rows* rows,
                         float* attr, int64_t attr_stride, gs_mlp_state* st, void* stream)
{
    gs_status e = check_rows(net, rows, mean, n);
    if (e != GS_OK) return e;
    const int NF = net->n_chan;
    if (!Z1 || !attr || !st || !st->cb || attr_stride < (int64_t)n * 2 * NF) return GS_ERR_INVALID_ARG;
    if ((st->save_h1 == nullptr) != (st->save_h2 == nullptr)) return GS_ERR_INVALID_ARG;
    hipStream_t s = (hipStream_t)stream;
    (void)hipGetLastError();
    hipLaunchKernelGGL(k_mlp_bias, dim3(rows->n_sets), dim3(64), 0, s, net->W1, net->b1, rows->tx, net->box_lo[0],
                       net->box_lo[1], net->box_lo[2], net->box_hi[0], net->box_hi[1], net->box_hi[2], st->cb,
                       st->genc);
    MlpArgs A{};
    A.W2 = net->W2; A.b2 = net->b2; A.W3 = net->W3; A.b3 = net->b3;
    A.Z1 = Z1; A.cb = st->cb; A.mean = mean; A.n = n; A.tx = rows->tx; A.r_near = net->r_near;
    A.list = rows->list; A.list_stride = rows->list_stride; A.count = rows->count; A.count_stride = rows->count_stride;
    A.row_cap = rows->row_cap; A.attr = attr; A.attr_stride = attr_stride;
    A.save_h1 = st->save_h1; A.save_h2 = st->save_h2;
    A.wide = ((uintptr_t)attr & 15) == 0 && attr_stride % 4 == 0;
    const int gx = rows_grid(rows);
    if (NF == 64) hipLaunchKernelGGL(k_mlp_fwd<64>, dim3(gx, rows->n_sets), dim3(256), 0, s, A);
    else hipLaunchKernelGGL(k_mlp_fwd<32>, dim3(gx, rows->n_sets), dim3(256), 0, s, A);
    return hipGetLastError() == hipSuccess ? GS_OK : GS_ERR_HIP;
}

gs_status gs_mlp_backward(const gs_mlp* net, const uint16_t* E, const float* mean, int32_t n, const gs_mlp_rows* rows,
                          float* d_attr, int64_t attr_stride, int32_t clear_d_attr, gs_mlp_state* st,
                          gs_mlp_grads* gr, void* stream)
{
    gs_status e = check_rows(net, rows, mean, n);
    if (e != GS_OK) return e;
    if (!E || !d_attr || !st || !gr || !st->save_h1 || !st->save_h2 || !st->save_do || !st->save_dz2 ||
        !st->save_dz1 || !st->genc || !st->dc || !st->partial || st->n_partial < 1)
        return GS_ERR_INVALID_ARG;
    if (!gr->dW1 || !gr->db1 || !gr->dW2 || !gr->db2 || !gr->dW3 || !gr->db3 || !gr->dE) return GS_ERR_INVALID_ARG;
    const int NF = net->n_chan;
    if (attr_stride < (int64_t)n * 2 * NF) return GS_ERR_INVALID_ARG;
    hipStream_t s = (hipStream_t)stream;
    (void)hipGetLastError();
    {
        FillSegs f{};
        f.p[0] = (uint32_t*)gr->db3; f.count[0] = 2 * NF;
        f.p[1] = (uint32_t*)gr->db2; f.count[1] = MLP_HID;
        f.p[2] = (uint32_t*)gr->dW1; f.count[2] = (size_t)MLP_HID * MLP_IN;
        f.p[3] = (uint32_t*)st->dc; f.count[3] = (size_t)rows->n_sets * MLP_HID;
        f.p[4] = (uint32_t*)gr->dE; f.count[4] = (size_t)n * MLP_EMB;
        f.n = 5;
        launch_fill_segs(f, s);
    }
    MlpArgs A{};
    A.W2 = net->W2; A.b2 = net->b2; A.W3 = net->W3; A.b3 = net->b3;
    A.W1 = net->W1;
    A.mean = mean; A.n = n; A.tx = rows->tx; A.r_near = net->r_near;
    A.list = rows->list; A.list_stride = rows->list_stride; A.count = rows->count; A.count_stride = rows->count_stride;
    A.row_cap = rows->row_cap; A.d_attr = d_attr; A.attr_stride = attr_stride;
    A.clear = clear_d_attr ? d_attr : nullptr;
    A.save_h1 = st->save_h1; A.save_h2 = st->save_h2; A.save_do = st->save_do; A.save_dz2 = st->save_dz2;
    A.save_dz1 = st->save_dz1; A.db3 = gr->db3; A.db2 = gr->db2; A.dc = st->dc; A.dE = gr->dE;
    A.wide = ((uintptr_t)d_attr & 15) == 0 && attr_stride % 4 == 0;
    const int gx = rows_grid(rows);
    if (NF == 64) hipLaunchKernelGGL(k_mlp_bwd_data<64>, dim3(gx, rows->n_sets), dim3(256), 0, s, A);
    else hipLaunchKernelGGL(k_mlp_bwd_data<32>, dim3(gx, rows->n_sets), dim3(256), 0, s, A);
    const int P = st->n_partial;
    // dW3 = d_o^T h2, dW2 = dZ2^T h1, dW1e = dZ1^T E: one split-K launch, one reduction
    WgradArgs W{st->save_do, st->save_h2, st->save_dz2, st->save_h1, st->save_dz1, E, rows->list, (size_t)rows->list_stride,
                rows->count, rows->count_stride, rows->n_sets, (size_t)rows->row_cap, st->partial};
    const int rb = (wg3_len0(NF) + WG3_LEN1 + WG3_LEN2 + 255) / 256;
    const dim3 rgrid(rb + (MLP_ENC + 1 + 3) / 4);
    if (NF == 64) {
        hipLaunchKernelGGL(k_wgrad3<64>, dim3(P, 3), dim3(64 * WG_WAVES), 0, s, W);
        hipLaunchKernelGGL(k_mlp_reduce<64>, rgrid, dim3(256), 0, s, st->partial, P, rb, st->dc, st->genc,
                           rows->n_sets, gr->dW3, gr->dW2, gr->dW1, gr->db1);
    } else {
        hipLaunchKernelGGL(k_wgrad3<32>, dim3(P, 3), dim3(64 * WG_WAVES), 0, s, W);
        hipLaunchKernelGGL(k_mlp_reduce<32>, rgrid, dim3(256), 0, s, st->partial, P, rb, st->dc, st->genc,
                           rows->n_sets, gr->dW3, gr->dW2, gr->dW1, gr->db1);
    }
    return hipGetLastError() == hipSuccess ? GS_OK : GS_ERR_HIP;
}

}  // extern "C"
