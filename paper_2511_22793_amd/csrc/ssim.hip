// Magnitude-spectrum loss, Eq. (5): per set b of real spectra
// zhat, z [F][H][W],
//   L_b = (1 - lambda_1) L1_b + lambda_1 (1 - SSIM_b),
// L1_b the mean absolute error over channels and pixels, SSIM_b the mean of
// the structural-similarity map: an 11 x 11 Gaussian window (sigma 1.5,
// normalised, separable) applied as a same-size filter with zero padding,
//   s = (2 mx my + C1)(2 sxy + C2) / ((mx^2 + my^2 + C1)(sxx + syy + C2)),
// mx = G*x, sxx = G*x^2 - mx^2, sxy = G*(x y) - mx my, C1 = 0.01^2,
// C2 = 0.03^2; and the gradient of L = (1/S) sum_b L_b.
//
// The gradient of the mean SSIM with respect to x at pixel q is, by the chain
// rule through the filtered maps (G symmetric, zero outside the image),
//   (G*a)(q) + 2 x(q) (G*b)(q) + y(q) (G*c)(q),
// a = ds/dmx, b = ds/dsxx (through G*x^2), c = ds/dsxy (through G*(x y)),
// each map zero outside the image, divided by the pixel count.
//
// One workgroup per (32 x 16 tile, channel, set), everything in LDS: the
// inputs with a 10-pixel halo, the four row-filtered maps on the tile with a
// 5-pixel halo in columns, the three derivative maps on the tile with a
// 5-pixel halo, and their filtered values on the tile.  Every thread filters
// a run of neighbouring outputs along the filter's direction, so a value
// leaves LDS about 3 times instead of once per tap, and the column filter
// goes on to the derivative maps in registers.  The
// inputs, the row maps and the derivative maps take each other's place (24 KB
// of LDS, five workgroups per CU).  Of the two variances only the sum is
// needed, and it is formed from e = x - y as
//   sxx + syy = (G*e^2 - (mx - my)^2) + 2 sxy,
// which takes off less than x^2 and y^2 would, and whose sxy rounds as that of
// the numerator beside it: rms error of the gradient against 64 bits
// 0.85e-6, 1.3e-6 with the two variances apart (five maps), 1.4e-6 with
// x^2 + y^2 filtered as one; the same time as the last.
// Bound: FP32 multiply-adds at one per lane and issue (about 310 per pixel
// with the halos).  32 spectra of 90 x 360: 76 us with one LDS read per tap,
// 29 us so.  Per-workgroup sums of |x - y| and of s go to a
// partial buffer summed in a fixed order by a second kernel.
#include "common.h"

namespace gs {

constexpr int SS_TW = 32, SS_TH = 16, SS_R = 5;
constexpr int SS_K = 2 * SS_R + 1;               // window taps
constexpr int SS_IW = SS_TW + 4 * SS_R;          // input columns (52)
constexpr int SS_IH = SS_TH + 4 * SS_R;          // input rows (36)
constexpr int SS_MW = SS_TW + 2 * SS_R;          // map columns (42)
constexpr int SS_MH = SS_TH + 2 * SS_R;          // map rows (26)
// outputs per thread of the four filter passes, and the threads they take
constexpr int SS_P1 = 7, SS_S1 = SS_MW / SS_P1;                  // rows of inputs: 6 runs x 36 rows
constexpr int SS_P2 = 5, SS_S2 = (SS_MH + SS_P2 - 1) / SS_P2;    // columns of maps: 6 runs x 42 columns
constexpr int SS_P3 = 4, SS_S3 = SS_TW / SS_P3;                  // rows of derivatives: 8 runs x 26 rows
constexpr int SS_P4 = 2, SS_S4 = SS_TH / SS_P4;                  // columns of derivatives: 8 runs x 32 columns
static_assert(SS_MW % SS_P1 == 0 && SS_S1 * SS_IH <= 256 && SS_S2 * SS_MW <= 256 && SS_S3 * SS_MH <= 256 &&
                  SS_S4 * SS_TW == 256,
              "ssim thread layout");

struct SsimWin {
    float w[SS_K];
};

// o[i] = sum_k w[k] v[i + k], the taps in order
template <int N>
__device__ __forceinline__ void ss_filter(const float* v, const SsimWin& win, float* o)
{
#pragma unroll
    for (int i = 0; i < N; ++i) o[i] = 0.0f;
#pragma unroll
    for (int k = 0; k < SS_K; ++k)
#pragma unroll
        for (int i = 0; i < N; ++i) o[i] = fmaf(win.w[k], v[i + k], o[i]);
}

__global__ __launch_bounds__(256) void k_l1_ssim(const float* __restrict__ x, const float* __restrict__ y, int H,
                                                 int W, int tiles_x, int ntiles, SsimWin win, float C1, float C2,
                                                 float gx_l1, float gx_ssim, float* __restrict__ grad,
                                                 float* __restrict__ part)
{
    const int tx0 = blockIdx.x * SS_TW, ty0 = blockIdx.y * SS_TH;
    const size_t img = blockIdx.z;  // set * F + channel
    const size_t HW = (size_t)H * W;
    x += img * HW;
    y += img * HW;
    // in turn: the inputs; the row-filtered maps; the derivative maps and,
    // behind them, their row-filtered form
    __shared__ float s_h[4 * SS_IH * SS_MW];
    float (*s_x)[SS_IW] = (float (*)[SS_IW])s_h, (*s_y)[SS_IW] = s_x + SS_IH;
    float (*s_r)[SS_IH][SS_MW] = (float (*)[SS_IH][SS_MW])s_h;
    float (*s_d)[SS_MH][SS_MW] = (float (*)[SS_MH][SS_MW])s_h;
    float (*s_f)[SS_MH][SS_TW] = (float (*)[SS_MH][SS_TW])(s_h + 3 * SS_MH * SS_MW);
    static_assert(3 * SS_MH * (SS_MW + SS_TW) <= 4 * SS_IH * SS_MW && 2 * SS_IH * SS_IW <= 4 * SS_IH * SS_MW,
                  "ssim LDS");
    __shared__ float s_red[2][4];
    const int t = threadIdx.x;

    constexpr int NL = (SS_IH * SS_IW + 255) / 256;
    float lx[NL], ly[NL];
#pragma unroll
    for (int u = 0; u < NL; ++u) {
        const int i = u * 256 + t, r = i / SS_IW, c = i % SS_IW;
        const int gr = ty0 - 2 * SS_R + r, gc = tx0 - 2 * SS_R + c;
        const bool in = i < SS_IH * SS_IW && gr >= 0 && gr < H && gc >= 0 && gc < W;
        lx[u] = in ? x[(size_t)gr * W + gc] : 0.0f;
        ly[u] = in ? y[(size_t)gr * W + gc] : 0.0f;
    }
#pragma unroll
    for (int u = 0; u < NL; ++u) {
        const int i = u * 256 + t;
        if (i < SS_IH * SS_IW) {
            (&s_x[0][0])[i] = lx[u];
            (&s_y[0][0])[i] = ly[u];
        }
    }
    __syncthreads();
    // rows: x, y, (x - y)^2, x y filtered along the columns; the thread's own
    // two pixels stay in registers for the end
    const int r4 = t / SS_TW * SS_P4, c4 = t % SS_TW;
    float px[SS_P4], py[SS_P4];
#pragma unroll
    for (int i = 0; i < SS_P4; ++i) {
        px[i] = s_x[r4 + i + 2 * SS_R][c4 + 2 * SS_R];
        py[i] = s_y[r4 + i + 2 * SS_R][c4 + 2 * SS_R];
    }
    const bool act1 = t < SS_S1 * SS_IH;
    const int r1 = act1 ? t / SS_S1 : 0, c1 = t % SS_S1 * SS_P1;
    float xv[SS_P1 + SS_K - 1], yv[SS_P1 + SS_K - 1];
#pragma unroll
    for (int k = 0; k < SS_P1 + SS_K - 1; ++k) {
        xv[k] = s_x[r1][c1 + k];
        yv[k] = s_y[r1][c1 + k];
    }
    __syncthreads();  // the inputs are read
    if (act1) {
        float p[SS_P1 + SS_K - 1], o[SS_P1];
        auto put = [&](int q, const float* v) {
            ss_filter<SS_P1>(v, win, o);
#pragma unroll
            for (int i = 0; i < SS_P1; ++i) s_r[q][r1][c1 + i] = o[i];
        };
        put(0, xv);
        put(1, yv);
#pragma unroll
        for (int k = 0; k < SS_P1 + SS_K - 1; ++k) p[k] = (xv[k] - yv[k]) * (xv[k] - yv[k]);
        put(2, p);
#pragma unroll
        for (int k = 0; k < SS_P1 + SS_K - 1; ++k) p[k] = xv[k] * yv[k];
        put(3, p);
    }
    __syncthreads();
    // columns, then SSIM and its derivative maps on the tile plus the 5-pixel
    // halo (zero outside the image); the SSIM sum over the tile's own pixels
    float ssum = 0.0f, l1sum = 0.0f;
    const int r2 = t / SS_MW * SS_P2, c2 = t % SS_MW;
    float d[3][SS_P2];
    if (t < SS_S2 * SS_MW) {
        float m[4][SS_P2];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            float v[SS_P2 + SS_K - 1];
#pragma unroll
            for (int k = 0; k < SS_P2 + SS_K - 1; ++k) v[k] = r2 + k < SS_IH ? s_r[q][r2 + k][c2] : 0.0f;
            ss_filter<SS_P2>(v, win, m[q]);
        }
#pragma unroll
        for (int i = 0; i < SS_P2; ++i) {
            const int r = r2 + i, gr = ty0 - SS_R + r, gc = tx0 - SS_R + c2;
            d[0][i] = d[1][i] = d[2][i] = 0.0f;
            if (r < SS_MH && gr >= 0 && gr < H && gc >= 0 && gc < W) {
                const float mx = m[0][i], my = m[1][i];
                const float me = mx - my, sxy = m[3][i] - mx * my;
                const float A1 = 2.0f * mx * my + C1, A2 = 2.0f * sxy + C2;
                const float B1 = mx * mx + my * my + C1, B2 = (m[2][i] - me * me) + A2;
                const float s = (A1 * A2) / (B1 * B2);
                const float iA2 = 2.0f / A2, iB2 = 1.0f / B2;
                d[0][i] = s * (my * (2.0f / A1 - iA2) - 2.0f * mx * (1.0f / B1 - iB2));
                d[1][i] = -s * iB2;
                d[2][i] = s * iA2;
                if (r >= SS_R && r < SS_R + SS_TH && c2 >= SS_R && c2 < SS_R + SS_TW) ssum += s;
            }
        }
    }
    __syncthreads();  // the row maps are read
    if (t < SS_S2 * SS_MW) {
#pragma unroll
        for (int q = 0; q < 3; ++q)
#pragma unroll
            for (int i = 0; i < SS_P2; ++i)
                if (r2 + i < SS_MH) s_d[q][r2 + i][c2] = d[q][i];
    }
    __syncthreads();
    // the derivative maps filtered along the columns (tile columns only)
    if (t < SS_S3 * SS_MH) {
        const int r = t / SS_S3, c0 = t % SS_S3 * SS_P3;
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            float v[SS_P3 + SS_K - 1], o[SS_P3];
#pragma unroll
            for (int k = 0; k < SS_P3 + SS_K - 1; ++k) v[k] = s_d[q][r][c0 + k];
            ss_filter<SS_P3>(v, win, o);
#pragma unroll
            for (int i = 0; i < SS_P3; ++i) s_f[q][r][c0 + i] = o[i];
        }
    }
    __syncthreads();
    {
        const int gc = tx0 + c4;
        float g[3][SS_P4];
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            float v[SS_P4 + SS_K - 1];
#pragma unroll
            for (int k = 0; k < SS_P4 + SS_K - 1; ++k) v[k] = s_f[q][r4 + k][c4];
            ss_filter<SS_P4>(v, win, g[q]);
        }
#pragma unroll
        for (int i = 0; i < SS_P4; ++i) {
            const int gr = ty0 + r4 + i;
            if (gr >= H || gc >= W) continue;
            const float e = px[i] - py[i];
            l1sum += fabsf(e);
            if (grad) {
                const float sg = e > 0.0f ? 1.0f : (e < 0.0f ? -1.0f : 0.0f);
                const float dss = g[0][i] + 2.0f * px[i] * g[1][i] + py[i] * g[2][i];
                grad[img * HW + (size_t)gr * W + gc] = gx_l1 * sg - gx_ssim * dss;
            }
        }
    }
    // workgroup sums (fixed order)
    for (int o = 32; o > 0; o >>= 1) {
        ssum += __shfl_xor(ssum, o, 64);
        l1sum += __shfl_xor(l1sum, o, 64);
    }
    if ((t & 63) == 0) {
        s_red[0][t >> 6] = l1sum;
        s_red[1][t >> 6] = ssum;
    }
    __syncthreads();
    if (t < 2) {
        const size_t slot = (blockIdx.z * (size_t)ntiles + blockIdx.y * tiles_x + blockIdx.x) * 2 + t;
        part[slot] = s_red[t][0] + s_red[t][1] + s_red[t][2] + s_red[t][3];
    }
}

// per set: L1 = sum |x - y| / N, SSIM = sum s / N, loss = (1 - l) L1 + l (1 - SSIM)
__global__ __launch_bounds__(256) void k_l1_ssim_finish(const float* __restrict__ part, int per_set, float inv_n,
                                                        float lambda_1, float* __restrict__ loss,
                                                        float* __restrict__ ssim, float* __restrict__ l1)
{
    const int s = blockIdx.x;
    float a = 0.0f, b = 0.0f;
    for (int i = threadIdx.x; i < per_set; i += 256) {
        a += part[((size_t)s * per_set + i) * 2];
        b += part[((size_t)s * per_set + i) * 2 + 1];
    }
    for (int o = 32; o > 0; o >>= 1) {
        a += __shfl_xor(a, o, 64);
        b += __shfl_xor(b, o, 64);
    }
    __shared__ float red[2][4];
    if ((threadIdx.x & 63) == 0) {
        red[0][threadIdx.x >> 6] = a;
        red[1][threadIdx.x >> 6] = b;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        const float L1 = (red[0][0] + red[0][1] + red[0][2] + red[0][3]) * inv_n;
        const float SS = (red[1][0] + red[1][1] + red[1][2] + red[1][3]) * inv_n;
        if (l1) l1[s] = L1;
        if (ssim) ssim[s] = SS;
        loss[s] = (1.0f - lambda_1) * L1 + lambda_1 * (1.0f - SS);
    }
}

}  // namespace gs

using namespace gs;

extern "C" {

size_t gs_loss_l1_ssim_scratch_bytes(int32_t n_sets, int32_t n_chan, int32_t H, int32_t W)
{
    if (n_sets < 1 || n_chan < 1 || H < 1 || W < 1) return 0;
    const size_t tiles = (size_t)((W + SS_TW - 1) / SS_TW) * ((H + SS_TH - 1) / SS_TH);
    return align256((size_t)n_sets * n_chan * tiles * 2 * sizeof(float));
}

gs_status gs_loss_l1_ssim(const float* spectrum, const float* target, int32_t n_sets, int32_t n_chan, int32_t H,
                          int32_t W, float lambda_1, float* loss, float* ssim, float* l1, float* d_spectrum,
                          void* scratch, size_t scratch_bytes, void* stream)
{
    if (!spectrum || !target || !loss || n_sets < 1 || n_chan < 1 || H < 1 || W < 1 ||
        !(lambda_1 >= 0.0f && lambda_1 <= 1.0f))
        return GS_ERR_INVALID_ARG;
    if ((int64_t)n_sets * n_chan > 65535) return GS_ERR_CAPACITY;
    const size_t need = gs_loss_l1_ssim_scratch_bytes(n_sets, n_chan, H, W);
    if (!scratch || ((uintptr_t)scratch & 255) || scratch_bytes < need) return GS_ERR_WORKSPACE;
    SsimWin win{};
    {
        double g[SS_K], sum = 0.0;
        for (int k = 0; k < SS_K; ++k) {
            const double d = k - SS_R;
            g[k] = exp(-d * d / (2.0 * 1.5 * 1.5));
            sum += g[k];
        }
        for (int k = 0; k < SS_K; ++k) win.w[k] = (float)(g[k] / sum);
    }
    const int tiles_x = (W + SS_TW - 1) / SS_TW, tiles_y = (H + SS_TH - 1) / SS_TH;
    const double N = (double)n_chan * H * W;
    const float gx_l1 = (float)((1.0 - lambda_1) / (N * n_sets));
    const float gx_ssim = (float)(lambda_1 / (N * n_sets));
    hipStream_t s = (hipStream_t)stream;
    (void)hipGetLastError();
    hipLaunchKernelGGL(k_l1_ssim, dim3(tiles_x, tiles_y, n_sets * n_chan), dim3(256), 0, s, spectrum, target, H, W,
                       tiles_x, tiles_x * tiles_y, win, 0.01f * 0.01f, 0.03f * 0.03f, gx_l1, gx_ssim, d_spectrum,
                       (float*)scratch);
    hipLaunchKernelGGL(k_l1_ssim_finish, dim3(n_sets), dim3(256), 0, s, (const float*)scratch,
                       n_chan * tiles_x * tiles_y, (float)(1.0 / N), lambda_1, loss, ssim, l1);
    GS_CHECK_LAUNCH();
    return GS_OK;
}

}  // extern "C"
