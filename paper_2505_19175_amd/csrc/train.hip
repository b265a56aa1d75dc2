// train.hip -- the pieces of a training step around the renderer (Sec. 3.3):
// the photometric loss (1 - lambda) L1 + lambda (1 - SSIM) and its image
// gradient, the opacity and size losses, and Adam on the raw parameters.
//
// SSIM uses local statistics under an 11x11 Gaussian window; each of the two
// SSIM kernels stages a tile of 32 x TH pixels and its 5-pixel halo (zeros
// outside the image) in LDS and applies the separable window as a row pass
// and a column pass, both register-blocked.  They are bound by the passes'
// FP32 FMAs; the optimizer kernels stream every parameter array once (HBM).
#include <math.h>

#include "adam.h"
#include "ts_device.h"
#include "ts_kernels.h"

namespace ts {

constexpr int kR = 5;             // window radius
constexpr int kTW = 32;           // output tile width
constexpr int kPW = kTW + 2 * kR; // staged patch width
constexpr int kPS = 44;           // row stride of a staged patch: whole 16-byte vectors
constexpr int kSeg = kTW / 4;     // row-pass jobs per patch row (four outputs each)
constexpr float kC1 = 0.01f * 0.01f;
constexpr float kC2 = 0.03f * 0.03f;

constexpr int64_t kFillTiles = 512;   // workgroups that fill the chip twice over

struct Win11 {
    float w[11];
};

// Stages NI images' patches (rows y0 .., columns x0 ..) of the tile, zeros
// outside the image: a wave takes every fourth row, a lane one column, so the
// row test is the wave's and an address is one add; every load of a thread is
// issued before any value is stored.
template <int NI, int TH>
__device__ __forceinline__ void stage_patch(const float* const (&img)[NI], int W, int H, int x0,
                                            int y0, float (*in)[TH + 2 * kR][kPS])
{
    constexpr int PH = TH + 2 * kR, R = (PH + 3) / 4;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, gx = x0 + lane;
    const bool col = lane < kPW && gx >= 0 && gx < W;
    float v[NI][R];
#pragma unroll
    for (int j = 0; j < R; ++j) {
        const int r = 4 * j + w, gy = y0 + r;
        const bool ok = col && r < PH && gy >= 0 && gy < H;
        const int64_t p = (int64_t)gy * W + gx;
#pragma unroll
        for (int q = 0; q < NI; ++q) v[q][j] = ok ? img[q][p] : 0.f;
    }
    if (lane < kPW) {
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const int r = 4 * j + w;
            if (r < PH) {
#pragma unroll
                for (int q = 0; q < NI; ++q) in[q][r][lane] = v[q][j];
            }
        }
    }
}

// The 14 patch values a row-pass job reads (columns 4 s .. 4 s + 13).
__device__ __forceinline__ void load_seg(const float* row, int s, float (&v)[16])
{
    const float4* src = reinterpret_cast<const float4*>(row) + s;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const float4 x = src[k];
        v[4 * k] = x.x; v[4 * k + 1] = x.y; v[4 * k + 2] = x.z; v[4 * k + 3] = x.w;
    }
}

// Four outputs of the row pass.
__device__ __forceinline__ float4 row_blur(const float (&v)[16], const Win11& W)
{
    float o[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        float acc = 0.f;
#pragma unroll
        for (int k = 0; k < 11; ++k) acc = fmaf(W.w[k], v[j + k], acc);
        o[j] = acc;
    }
    return make_float4(o[0], o[1], o[2], o[3]);
}

// Column pass: the N outputs of column c from patch row r0 down.
template <int N>
__device__ __forceinline__ void col_blur(const float (*row)[kTW], int r0, int c, const Win11& W,
                                         float (&out)[N])
{
    float v[N + 10];
#pragma unroll
    for (int r = 0; r < N + 10; ++r) v[r] = row[r0 + r][c];
#pragma unroll
    for (int y = 0; y < N; ++y) {
        float acc = 0.f;
#pragma unroll
        for (int k = 0; k < 11; ++k) acc = fmaf(W.w[k], v[y + k], acc);
        out[y] = acc;
    }
}

// Per pixel and channel: SSIM and the coefficients of its gradient,
//   d_mx = dS/dmu_x - 2 mu_x dS/dvar_x - mu_y dS/dcov,  d_exx = dS/dvar_x,
//   d_exy = dS/dcov,
// scaled by the upstream -lambda / n; and the per-workgroup sums of |x - y|
// and S (the loss value).
//
// Row pass: a job reads 14 values of x and y once and produces four outputs
// of the five quantities (x, y, x^2, y^2, xy), whose products are formed in
// registers.  Column pass: a thread owns TH / 8 pixels of one column and
// holds all five quantities, so nothing goes back to LDS.  In both passes
// every thread has work (16x16 tiles with a row of 26 or a column of 16 per
// thread left half the lanes idle): at 1280x720 forward 48.6 -> 32.3 us,
// backward 38.5 -> 25.4 us, for 55 and 77 MB of traffic.
template <int TH>
__global__ __launch_bounds__(256) void k_ssim_fwd(const float* __restrict__ x_img,
                                                  const float* __restrict__ y_img, int W, int H,
                                                  Win11 win, float up, float* __restrict__ coef,
                                                  float* __restrict__ part)
{
    constexpr int PH = TH + 2 * kR, N = TH / 8;
    __shared__ __align__(16) float in[2][PH][kPS];
    __shared__ __align__(16) float row[5][PH][kTW];
    __shared__ float red[2][4];
    const int ch = blockIdx.z, t = threadIdx.x;
    const int64_t hw = (int64_t)W * H;
    const float* const img[2] = {x_img + ch * hw, y_img + ch * hw};
    stage_patch<2, TH>(img, W, H, blockIdx.x * kTW - kR, blockIdx.y * TH - kR, in);
    __syncthreads();
    for (int j = t; j < PH * kSeg; j += 256) {
        const int r = j / kSeg, s = j % kSeg;
        float x[16], y[16], p[16];
        load_seg(in[0][r], s, x);
        load_seg(in[1][r], s, y);
        float4* dst = reinterpret_cast<float4*>(&row[0][r][4 * s]);
        constexpr int Q4 = PH * kTW / 4;
        dst[0] = row_blur(x, win);
        dst[Q4] = row_blur(y, win);
#pragma unroll
        for (int k = 0; k < 14; ++k) p[k] = x[k] * x[k];
        dst[2 * Q4] = row_blur(p, win);
#pragma unroll
        for (int k = 0; k < 14; ++k) p[k] = y[k] * y[k];
        dst[3 * Q4] = row_blur(p, win);
#pragma unroll
        for (int k = 0; k < 14; ++k) p[k] = x[k] * y[k];
        dst[4 * Q4] = row_blur(p, win);
    }
    __syncthreads();
    const int c = t % kTW, r0 = (t / kTW) * N;
    float m[5][N];
#pragma unroll
    for (int q = 0; q < 5; ++q) col_blur<N>(row[q], r0, c, win, m[q]);
    const int px = blockIdx.x * kTW + c;
    float l1 = 0.f, ssum = 0.f;
#pragma unroll
    for (int j = 0; j < N; ++j) {
        const int py = blockIdx.y * TH + r0 + j;
        if (px < W && py < H) {
            const float mx = m[0][j], my = m[1][j];
            const float vx = m[2][j] - mx * mx, vy = m[3][j] - my * my, cxy = m[4][j] - mx * my;
            const float A = 2.f * mx * my + kC1, Bn = 2.f * cxy + kC2;
            const float D1 = mx * mx + my * my + kC1, D2 = vx + vy + kC2;
            const float inv = 1.f / (D1 * D2);
            const float s = A * Bn * inv;
            const float dmx = 2.f * my * Bn * inv - s * 2.f * mx / D1;
            const float dvx = -s / D2;
            const float dcv = 2.f * A * inv;
            const int64_t p = (int64_t)py * W + px;
            float* cc = coef + ch * 3 * hw;
            cc[p] = up * (dmx - 2.f * mx * dvx - my * dcv);
            cc[hw + p] = up * dvx;
            cc[2 * hw + p] = up * dcv;
            l1 += fabsf(in[0][r0 + j + kR][c + kR] - in[1][r0 + j + kR][c + kR]);
            ssum += s;
        }
    }
    // workgroup sums (wave reduction, then one value per wave)
    for (int o = 32; o > 0; o >>= 1) {
        l1 += __shfl_xor(l1, o);
        ssum += __shfl_xor(ssum, o);
    }
    const int w = t >> 6;
    if ((t & 63) == 0) {
        red[0][w] = l1;
        red[1][w] = ssum;
    }
    __syncthreads();
    if (t == 0) {
        const int64_t b = ((int64_t)blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x;
        part[2 * b] = red[0][0] + red[0][1] + red[0][2] + red[0][3];
        part[2 * b + 1] = red[1][0] + red[1][1] + red[1][2] + red[1][3];
    }
}

// loss[0] = mean |x - y|, loss[1] = mean SSIM, from the per-workgroup sums
// (one workgroup, fixed order: reproducible).  s holds 2 x 256 doubles.
__device__ void loss_total(const float* __restrict__ part, int64_t nb, double n,
                           float* __restrict__ loss, double (*s)[256])
{
    double a = 0.0, b = 0.0;
    for (int64_t j = threadIdx.x; j < nb; j += 256) {
        a += part[2 * j];
        b += part[2 * j + 1];
    }
    s[0][threadIdx.x] = a;
    s[1][threadIdx.x] = b;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if (threadIdx.x < h) {
            s[0][threadIdx.x] += s[0][threadIdx.x + h];
            s[1][threadIdx.x] += s[1][threadIdx.x + h];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        loss[0] = (float)(s[0][0] / n);
        loss[1] = (float)(s[1][0] / n);
    }
}

// dL/dC = (1 - lambda) sign(x - y) / n + blur(d_mx) + 2 x blur(d_exx) + y blur(d_exy).
// With loss set, the grid has a fourth z-plane whose first workgroup sums
// the forward's partial sums into the loss value (the other workgroups of
// that plane exit): the reduction runs beside the gradient tiles instead of
// in a launch of its own.
template <int TH>
__global__ __launch_bounds__(256) void k_ssim_bwd(const float* __restrict__ x_img,
                                                  const float* __restrict__ y_img, int W, int H,
                                                  Win11 win, float l1w,
                                                  const float* __restrict__ coef,
                                                  float* __restrict__ grad,
                                                  const float* __restrict__ part, double n,
                                                  float* __restrict__ loss)
{
    constexpr int PH = TH + 2 * kR, N = TH / 8;
    __shared__ __align__(16) float in[3][PH][kPS];
    __shared__ __align__(16) float row[3][PH][kTW];
    static_assert(sizeof(in) >= 2 * 256 * sizeof(double), "reduction scratch");
    const int t = threadIdx.x;
    if (blockIdx.z == 3) {
        if (blockIdx.x == 0 && blockIdx.y == 0)
            loss_total(part, (int64_t)gridDim.x * gridDim.y * 3, n, loss,
                       reinterpret_cast<double (*)[256]>(&in[0][0][0]));
        return;
    }
    const int ch = blockIdx.z;
    const int64_t hw = (int64_t)W * H;
    const float* cc = coef + ch * 3 * hw;
    const float* const img[3] = {cc, cc + hw, cc + 2 * hw};
    stage_patch<3, TH>(img, W, H, blockIdx.x * kTW - kR, blockIdx.y * TH - kR, in);
    // the thread's own pixels, loaded early
    const int c = t % kTW, r0 = (t / kTW) * N;
    const int px = blockIdx.x * kTW + c, py0 = blockIdx.y * TH + r0;
    const int64_t p0 = ch * hw + (int64_t)py0 * W + px;
    float x[N], y[N];
#pragma unroll
    for (int j = 0; j < N; ++j) {
        const bool ok = px < W && py0 + j < H;
        x[j] = ok ? x_img[p0 + (int64_t)j * W] : 0.f;
        y[j] = ok ? y_img[p0 + (int64_t)j * W] : 0.f;
    }
    __syncthreads();
    for (int j = t; j < PH * kSeg; j += 256) {
        const int r = j / kSeg, s = j % kSeg;
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            float v[16];
            load_seg(in[q][r], s, v);
            *reinterpret_cast<float4*>(&row[q][r][4 * s]) = row_blur(v, win);
        }
    }
    __syncthreads();
    float b[3][N];
#pragma unroll
    for (int q = 0; q < 3; ++q) col_blur<N>(row[q], r0, c, win, b[q]);
#pragma unroll
    for (int j = 0; j < N; ++j) {
        if (px < W && py0 + j < H) {
            const float sg = x[j] > y[j] ? 1.f : (x[j] < y[j] ? -1.f : 0.f);
            grad[p0 + (int64_t)j * W] =
                fmaf(l1w, sg, b[0][j] + 2.f * x[j] * b[1][j] + y[j] * b[2][j]);
        }
    }
}

// One partial sum per 16x16 pixels of each channel covers every tile shape
// below.
static int64_t loss_parts(int W, int H)
{
    return (int64_t)((W + 15) / 16) * ((H + 15) / 16) * 3;
}

size_t image_loss_workspace_bytes(int W, int H)
{
    return (size_t)(9 * (int64_t)W * H * 4 + loss_parts(W, H) * 8 + 256);
}

void launch_image_loss(const float* rgb, const float* target, int W, int H, float lambda,
                       float* grad, float* loss, void* ws, hipStream_t stream)
{
    Win11 win;
    double g[11], sum = 0.0;
    for (int k = 0; k < 11; ++k) {
        const double d = k - 5;
        g[k] = exp(-d * d / (2.0 * 1.5 * 1.5));
        sum += g[k];
    }
    for (int k = 0; k < 11; ++k) win.w[k] = (float)(g[k] / sum);
    const double n = 3.0 * W * H;
    float* coef = reinterpret_cast<float*>(ws);
    float* part = coef + 9 * (int64_t)W * H;
    auto go = [&](auto th) {
        constexpr int TH = decltype(th)::value;
        const dim3 grid((W + kTW - 1) / kTW, (H + TH - 1) / TH, 3);
        hipLaunchKernelGGL(k_ssim_fwd<TH>, grid, dim3(256), 0, stream, rgb, target, W, H, win,
                           (float)(-lambda / n), coef, part);
        const dim3 grid_b(grid.x, grid.y, loss ? 4 : 3);
        hipLaunchKernelGGL(k_ssim_bwd<TH>, grid_b, dim3(256), 0, stream, rgb, target, W, H, win,
                           (float)((1.0 - lambda) / n), coef, grad, part, n, loss);
    };
    // Taller tiles waste less on their halo rows, but hold more LDS: 16 rows
    // (six workgroups per CU) beat 32 (three) on the forward, 32.3 against
    // 33.9 us at 1280x720.  An image too small to give each of the 256 CUs two
    // such tiles takes 8 rows, while its partial sums fit the workspace.
    auto tiles = [&](int th) { return (int64_t)((W + kTW - 1) / kTW) * ((H + th - 1) / th) * 3; };
    if (tiles(16) >= kFillTiles || tiles(8) > loss_parts(W, H))
        go(std::integral_constant<int, 16>{});
    else go(std::integral_constant<int, 8>{});
}

// ---------------------------------------------------------------------------
// Adam with the regularizers and the activation chain folded in (the
// arithmetic is in adam.h, shared with the backward projection's fused step).
// ---------------------------------------------------------------------------

// Vertices: the block's 256 vertex and gradient rows are staged through LDS
// so every global access is coalesced; each thread adds its triangle's
// size-loss gradient in LDS, then the update runs element-wise.
__global__ __launch_bounds__(256) void k_adam_vertices(float* __restrict__ v,
                                                       const float* __restrict__ gv,
                                                       float* __restrict__ m, float* __restrict__ s,
                                                       int64_t N, float beta_s, float lr, AdamK k)
{
    __shared__ float sv[256 * 9], sg[256 * 9];
    const int64_t base = (int64_t)blockIdx.x * 256;
    const int nt = (int)min((int64_t)256, N - base);
    const int n = 9 * nt;
    const int64_t off = 9 * base;
    for (int f = threadIdx.x; f < n; f += 256) {
        sv[f] = v[off + f];
        sg[f] = gv[off + f];
    }
    __syncthreads();
    const int t = threadIdx.x;
    if (t < nt && beta_s != 0.f) size_loss_grad(sv + 9 * t, sg + 9 * t, beta_s, N);
    __syncthreads();
    for (int f = threadIdx.x; f < n; f += 256) {
        float mi = m[off + f], si = s[off + f];
        v[off + f] = adam_update(sv[f], sg[f], mi, si, lr, k);
        m[off + f] = mi;
        s[off + f] = si;
    }
}

// Flat Adam; element e uses lr_a when e % row < first, else lr_b; act as in
// act_grad (0: g as given); with act 1 or 2, out[e] holds the activated old
// value and becomes the activated new one.
__global__ __launch_bounds__(256) void k_adam(float* __restrict__ p, const float* __restrict__ g,
                                              float* __restrict__ m, float* __restrict__ s,
                                              int64_t n, int row, int first, float lr_a, float lr_b,
                                              AdamK k, int act, float add,
                                              float* __restrict__ out)
{
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= n) return;
    const float gi = act != 0 ? act_grad(g[e], act, add, out[e]) : g[e];
    float mi = m[e], si = s[e];
    const float lr = (int)(e % row) < first ? lr_a : lr_b;
    const float pi = adam_update(p[e], gi, mi, si, lr, k);
    m[e] = mi;
    s[e] = si;
    p[e] = pi;
    if (act != 0) out[e] = act_value(pi, act);
}

void launch_optimizer(float* v, float* a, float* b, float* sh, float* o, float* sigma, int nsh,
                      int64_t N, const float* gv, const float* go, const float* gs,
                      const float* gsh, float* const* st, const float* lr, float beta_o,
                      float beta_s, float b1, float b2, float bc1, float bc2, float eps,
                      hipStream_t stream)
{
    if (N <= 0) return;
    const AdamK k{b1, b2, bc1, bc2, eps};
    const unsigned nb = (unsigned)((N + 255) / 256);
    hipLaunchKernelGGL(k_adam_vertices, dim3(nb), dim3(256), 0, stream, v, gv, st[0], st[1], N,
                       beta_s, lr[0], k);
    hipLaunchKernelGGL(k_adam, dim3(nb), dim3(256), 0, stream, a, go, st[2], st[3], N, 1, 1,
                       lr[1], lr[1], k, 1, beta_o / (float)N, o);
    hipLaunchKernelGGL(k_adam, dim3(nb), dim3(256), 0, stream, b, gs, st[4], st[5], N, 1, 1,
                       lr[2], lr[2], k, 2, 0.f, sigma);
    const int64_t n = (int64_t)nsh * N;
    hipLaunchKernelGGL(k_adam, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, sh, gsh,
                       st[6], st[7], n, nsh, 3, lr[3], lr[4], k, 0, 0.f, nullptr);
}

}  // namespace ts
