// densify.hip -- the densification step around the renderer (Sec. 3.2,
// "Densification"): Bernoulli sampling of triangles with probabilities from
// their opacity or inverse sigma, and midpoint subdivision of the selected
// ones in place.  Per-triangle streaming kernels, bound by HBM.
#include <type_traits>

#include "ts_device.h"
#include "ts_kernels.h"

namespace ts {

constexpr int kDensBlock = 256;
constexpr int kSumChunk = 4096;   // weights per workgroup of the sums
constexpr int kPickChunk = 4 * kDensBlock;   // triangles per workgroup of the selection
// Triangles per thread of the subdivision: eight, so that the workgroups'
// sums of the chunk counts stay short, two for soups of up to kFewTriangles
// (at 20k triangles 5 workgroups of the former kind would work one phase
// after another on an idle chip).
constexpr int kMany = 8, kFew = 2;
constexpr int64_t kFewTriangles = 1 << 18;
// From this size on, the sums that every workgroup would repeat get a launch of
// their own, since both the workgroups and the sums grow with the soup.  Selection,
// repeated / own launch: 3M 15.2 / 16.5 us, 4M 20.3 / 20.2, 8M 37.8 / 31.9, 100M
// 1260 / 292.  Subdivision (sums over spans of the chunk counts): 1M 34.6 / 37.0,
// 3M 77.3 / 73.1 (84.2 / 85.7 in the training benchmark), 4M 112 / 104, 30M 934 /
// 879, 200M 10037 / 5722.
constexpr int64_t kManyTriangles = 4 << 20;

__device__ __forceinline__ double dens_weight(float o_or_sigma, int mode)
{
    return mode == TS_DENSIFY_OPACITY ? (double)o_or_sigma : 1.0 / (double)o_or_sigma;
}

__device__ __forceinline__ bool aligned(const void* p, unsigned n)
{
    return (reinterpret_cast<uintptr_t>(p) & (n - 1u)) == 0;
}

// Values x[i .. i + 3] (zeros at or past N): one 16-byte load where whole.
__device__ __forceinline__ float4 load4(const float* __restrict__ x, int64_t i, int64_t N, bool vec)
{
    if (vec && i + 4 <= N) return *reinterpret_cast<const float4*>(x + i);
    return make_float4(i < N ? x[i] : 0.f, i + 1 < N ? x[i + 1] : 0.f, i + 2 < N ? x[i + 2] : 0.f,
                       i + 3 < N ? x[i + 3] : 0.f);
}

// Sum of 256 doubles by a fixed tree (x[t] + x[t + 128], + x[t + 64], .. + x[t
// + 1]; the last six levels inside the first wave): the result does not depend
// on timing, so the sum (and every decision taken from it) is reproducible.
__device__ __forceinline__ double block_sum(double x, double* s)
{
    const int t = threadIdx.x;
    s[t] = x;
    __syncthreads();
    if (t < kWave) {
        double y = (s[t] + s[t + 128]) + (s[t + 64] + s[t + 192]);
#pragma unroll
        for (int h = kWave / 2; h > 0; h >>= 1) y += __shfl_down(y, h);
        if (t == 0) s[0] = y;
    }
    __syncthreads();
    return s[0];
}

// Streaming stores: the children are written once and not read here.
__device__ __forceinline__ void store_stream(float* p, float a)
{
    __builtin_nontemporal_store(a, p);
}

__device__ __forceinline__ void store_stream(float4* p, const float4& a)
{
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    const f32x4 t = {a.x, a.y, a.z, a.w};
    __builtin_nontemporal_store(t, reinterpret_cast<f32x4*>(p));
}

// Per-workgroup sums of the weights (o, or 1 / sigma).  Bound by HBM: all four
// 16-byte loads of a thread are issued at once.
constexpr int kQuads = kSumChunk / (4 * kDensBlock);   // 16-byte loads per thread

__global__ __launch_bounds__(kDensBlock) void k_weight_partial(const float* __restrict__ x,
                                                               int64_t N, int mode,
                                                               double* __restrict__ partial)
{
    __shared__ double s[kDensBlock];
    const int64_t base = (int64_t)blockIdx.x * kSumChunk;
    const bool vec = aligned(x, 16);
    float4 v[kQuads];
#pragma unroll
    for (int r = 0; r < kQuads; ++r)
        v[r] = load4(x, base + 4 * (r * kDensBlock + (int)threadIdx.x), N, vec);
    double acc = 0.0;
#pragma unroll
    for (int r = 0; r < kQuads; ++r) {
        const int64_t i = base + 4 * (r * kDensBlock + (int)threadIdx.x);
        const float q[4] = {v[r].x, v[r].y, v[r].z, v[r].w};
#pragma unroll
        for (int c = 0; c < 4; ++c)
            if (i + c < N) acc += dens_weight(q[c], mode);
    }
    const double tot = block_sum(acc, s);
    if (threadIdx.x == 0) partial[blockIdx.x] = tot;
}

// The sum of the partial sums, in the order in which k_select would add them.
__global__ __launch_bounds__(kDensBlock) void k_weight_total(const double* __restrict__ partial,
                                                             int64_t np, double* __restrict__ total)
{
    __shared__ double s[kDensBlock];
    double acc = 0.0;
#pragma unroll 8
    for (int64_t j = threadIdx.x; j < np; j += kDensBlock) acc += partial[j];
    const double tot = block_sum(acc, s);
    if (threadIdx.x == 0) total[0] = tot;
}

// p_i = min(1, k w_i / sum w); selected iff u_i < p_i (all in FP64).  Every
// workgroup adds the np partial sums itself, in the same fixed order (a launch
// less; 733 sums at 3M triangles); of a larger soup, whose workgroups and sums
// both grow, it gets their total as the only one.
__global__ __launch_bounds__(kDensBlock) void k_select(const float* __restrict__ x, int64_t N,
                                                       int mode, double k,
                                                       const double* __restrict__ partial,
                                                       int64_t np, const float* __restrict__ u,
                                                       uint8_t* __restrict__ sel)
{
    __shared__ double s[kDensBlock];
    const int64_t i = (int64_t)blockIdx.x * kPickChunk + 4 * threadIdx.x;
    const float4 w4 = load4(x, i, N, aligned(x, 16)), u4 = load4(u, i, N, aligned(u, 16));
    double acc = 0.0;
    for (int64_t j = threadIdx.x; j < np; j += kDensBlock) acc += partial[j];
    const double tot = block_sum(acc, s);
    const float q[4] = {w4.x, w4.y, w4.z, w4.w}, t[4] = {u4.x, u4.y, u4.z, u4.w};
    uint32_t bits = 0;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const double p = tot > 0.0 ? fmin(1.0, k * dens_weight(q[c], mode) / tot) : 0.0;
        bits |= ((double)t[c] < p ? 1u : 0u) << (8 * c);
    }
    if (i + 4 <= N && aligned(sel, 4)) {
        *reinterpret_cast<uint32_t*>(sel + i) = bits;
    } else {
#pragma unroll
        for (int c = 0; c < 4; ++c)
            if (i + c < N) sel[i + c] = (uint8_t)(bits >> (8 * c));
    }
}

// The flags of triangles i .. i + F - 1 as bits.
template <int F>
__device__ __forceinline__ uint32_t load_flags(const uint8_t* __restrict__ sel, int64_t i,
                                               int64_t N)
{
    uint32_t f = 0;
    if (F == 8 && i + 8 <= N && aligned(sel + i, 8)) {
        const uint2 b = *reinterpret_cast<const uint2*>(sel + i);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            f |= ((b.x >> (8 * c)) & 0xffu) != 0u ? 1u << c : 0u;
            f |= ((b.y >> (8 * c)) & 0xffu) != 0u ? 16u << c : 0u;
        }
    } else {
#pragma unroll
        for (int c = 0; c < F; ++c) f |= (i + c < N && sel[i + c] != 0) ? 1u << c : 0u;
    }
    return f;
}

__device__ __forceinline__ uint32_t block_sum_u32(uint32_t x, uint32_t* s_w)
{
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) x += __shfl_xor(x, d, 64);
    if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = x;
    __syncthreads();
    x = s_w[0] + s_w[1] + s_w[2] + s_w[3];
    __syncthreads();
    return x;
}

// Selected triangles of each chunk.
template <int F>
__global__ __launch_bounds__(kDensBlock) void k_count_sel(const uint8_t* __restrict__ sel,
                                                          int64_t N, uint32_t* __restrict__ cnt)
{
    __shared__ uint32_t s_w[kDensBlock / kWave];
    const uint32_t f = load_flags<F>(sel, F * ((int64_t)blockIdx.x * kDensBlock + threadIdx.x), N);
    const uint32_t c = block_sum_u32(__popc(f), s_w);
    if (threadIdx.x == 0) cnt[blockIdx.x] = c;
}

// Sums of kSpan counts each.
constexpr int kSpan = kDensBlock;

__global__ __launch_bounds__(kDensBlock) void k_sum_counts(const uint32_t* __restrict__ cnt,
                                                           int64_t nb, uint32_t* __restrict__ span)
{
    __shared__ uint32_t s_w[kDensBlock / kWave];
    const int64_t j = (int64_t)blockIdx.x * kSpan + threadIdx.x;
    const uint32_t c = block_sum_u32(j < nb ? cnt[j] : 0u, s_w);
    if (threadIdx.x == 0) span[blockIdx.x] = c;
}

// Midpoint subdivision in place: the centre child replaces the parent, the
// three corner children go to N + 3 r + {0, 1, 2}, r the rank of the
// parent among the selected triangles; they copy its opacity, sigma and SH
// row.  Midpoints are (a + b) * 0.5 in FP32: one rounding.
//
// A workgroup takes a chunk of triangles: it adds the counts of the chunks
// before it (and of all, for the capacity test: nothing is written when the
// soup does not fit; SPANS: by their sums over spans of chunks), lists its
// selected triangles in LDS, and writes the children of consecutive ranks, which
// are contiguous, element by element.
// Bound by HBM (the SH rows: 192 bytes read and 576 written per selected
// triangle): with a wave copying one selected row at a time, each row's load
// exposed its latency.  The SH rows and the rest go to different workgroups
// (blockIdx.y), so neither waits for the other, and the children are streamed
// past the caches: 300k of 3M triangles 110 -> 80 us (about 370 MB in whole
// lines; 123 us in one workgroup with ordinary stores).
constexpr int kBatchSel = 256;   // selected triangles whose vertices are staged at once

template <int F, bool SPANS>
__global__ __launch_bounds__(kDensBlock) void k_subdivide(
    float* __restrict__ v, float* __restrict__ o, float* __restrict__ sigma, float* __restrict__ sh,
    int nsh, int64_t N, int64_t capacity, const uint8_t* __restrict__ sel,
    const uint32_t* __restrict__ cnt, const uint32_t* __restrict__ span, int64_t nb,
    uint32_t* __restrict__ out)
{
    __shared__ uint16_t s_id[F * kDensBlock];   // selected triangles of the chunk, in order
    __shared__ float s_p[kBatchSel][9];
    __shared__ uint32_t s_w[kDensBlock / kWave];
    __shared__ unsigned long long s_sum[2];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), w = tid / kWave;
    const int64_t base = (int64_t)blockIdx.x * (F * kDensBlock);
    const uint32_t f = load_flags<F>(sel, base + F * tid, N);
    if (tid < 2) s_sum[tid] = 0ull;
    __syncthreads();
    unsigned long long before = 0, all = 0;
    const int64_t mine = blockIdx.x;
    if constexpr (SPANS) {
        const int64_t own = mine / kSpan, j = own * kSpan + tid;
        for (int64_t k = tid; k < (nb + kSpan - 1) / kSpan; k += kDensBlock) {
            const uint32_t c = span[k];
            all += c;
            before += k < own ? c : 0u;
        }
        before += j < mine ? cnt[j] : 0u;
    } else {
        for (int64_t j = tid; j < nb; j += kDensBlock) {
            const uint32_t c = cnt[j];
            all += c;
            before += j < mine ? c : 0u;
        }
    }
    // integer sums: the order does not matter
    atomicAdd(&s_sum[0], before);
    atomicAdd(&s_sum[1], all);
    // this thread's selected triangles go to the list after those before it
    uint32_t inc = __popc(f);
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const uint32_t y = __shfl_up(inc, d);
        inc += lane >= d ? y : 0u;
    }
    if (lane == kWave - 1) s_w[w] = inc;
    __syncthreads();
    const uint64_t total = (uint64_t)N + 3 * s_sum[1];
    if (blockIdx.x == 0 && blockIdx.y == 0 && tid == 0) {
        out[0] = (uint32_t)min(total, (uint64_t)0xffffffffu);
        out[1] = total > (uint64_t)capacity ? 1u : 0u;
    }
    if (total > (uint64_t)capacity) return;   // does not fit: leave the soup unchanged
    uint32_t at = inc - __popc(f), n = 0;
    for (int j = 0; j < kDensBlock / kWave; ++j) {
        at += j < w ? s_w[j] : 0u;
        n += s_w[j];
    }
    for (uint32_t m = f; m != 0u; m &= m - 1u)
        s_id[at++] = (uint16_t)(F * tid + __builtin_ctz(m));
    __syncthreads();
    const int64_t j0 = N + 3 * (int64_t)s_sum[0];   // the chunk's first corner child

    // SH rows: one element (a 16-byte vector where rows are whole ones) read
    // once and written to three rows, four reads in flight per thread
    const bool vec = (nsh & 3) == 0 && aligned(sh, 16);
    const uint32_t len = vec ? (uint32_t)nsh / 4u : (uint32_t)nsh, jobs = n * len;
    auto copy_rows = [&](auto* rows) {
        constexpr int U = 4;
        for (uint32_t q0 = tid; q0 < jobs; q0 += U * kDensBlock) {
            std::remove_reference_t<decltype(*rows)> x[U];
#pragma unroll
            for (int k = 0; k < U; ++k) {
                const uint32_t q = q0 + k * kDensBlock;
                if (q < jobs) {
                    const uint32_t r = q / len;
                    x[k] = rows[(base + s_id[r]) * len + (q - r * len)];
                }
            }
#pragma unroll
            for (int k = 0; k < U; ++k) {
                const uint32_t q = q0 + k * kDensBlock;
                if (q < jobs) {
                    const uint32_t r = q / len, e = q - r * len;
                    auto* d = rows + (j0 + 3 * (int64_t)r) * len + e;
                    store_stream(d, x[k]);
                    store_stream(d + len, x[k]);
                    store_stream(d + 2 * len, x[k]);
                }
            }
        }
    };
    if (blockIdx.y == 0) {
        if (vec) copy_rows(reinterpret_cast<float4*>(sh));
        else copy_rows(sh);
        return;
    }

    // opacity and sigma: three copies
    for (uint32_t q = tid; q < 3 * n; q += kDensBlock) {
        const int64_t i = base + s_id[q / 3u];
        store_stream(o + j0 + q, o[i]);
        store_stream(sigma + j0 + q, sigma[i]);
    }

    // vertices: the parents' rows through LDS, since the centre child
    // overwrites its parent's
    for (uint32_t b = 0; b < n; b += kBatchSel) {
        const uint32_t m = min((uint32_t)kBatchSel, n - b);
        __syncthreads();
        for (uint32_t q = tid; q < 9 * m; q += kDensBlock) {
            const uint32_t r = q / 9u;
            s_p[r][q - 9 * r] = v[9 * (base + s_id[b + r]) + (q - 9 * r)];
        }
        __syncthreads();
        // vertex j of child c: the centre's (c = 3) are m01, m12, m20; corner
        // c keeps vertex c of the parent: (v0, m01, m20), (m01, v1, m12),
        // (m20, m12, v2)
        auto mid = [&](const float* p, int e, int a) {   // midpoint of edge e, axis a
            return (p[3 * e + a] + p[3 * (e == 2 ? 0 : e + 1) + a]) * 0.5f;
        };
        for (uint32_t q = tid; q < 27 * m; q += kDensBlock) {
            const uint32_t r = q / 27u, e = q - 27 * r;
            const int c = (int)(e / 9u), j = (int)(e / 3u) % 3, a = (int)(e % 3u);
            // the edge between vertices c and j
            const int k = c + j == 1 ? 0 : c + j == 3 ? 1 : 2;
            const float* p = s_p[r];
            store_stream(v + 9 * (j0 + 3 * (int64_t)b) + q,
                         c == j ? p[3 * j + a] : mid(p, k, a));
        }
        for (uint32_t q = tid; q < 9 * m; q += kDensBlock) {
            const uint32_t r = q / 9u, e = q - 9 * r;
            v[9 * (base + s_id[b + r]) + e] = mid(s_p[r], (int)(e / 3u), (int)(e % 3u));
        }
    }
}

size_t densify_workspace_bytes(int64_t N)
{
    const int64_t nw = (N + kSumChunk - 1) / kSumChunk, nb = (N + kDensBlock - 1) / kDensBlock;
    return (size_t)(8 * (nw + 1) + 4 * (nb + 2) + 256);
}

void launch_densify_select(const float* o, const float* sigma, int64_t N, int mode, double k,
                           const float* u, uint8_t* sel, void* ws, hipStream_t stream)
{
    const int64_t nw = (N + kSumChunk - 1) / kSumChunk;
    double* partial = reinterpret_cast<double*>(ws);
    const float* x = mode == TS_DENSIFY_OPACITY ? o : sigma;
    hipLaunchKernelGGL(k_weight_partial, dim3((unsigned)nw), dim3(kDensBlock), 0, stream, x, N,
                       mode, partial);
    const bool total = N > kManyTriangles;
    if (total)
        hipLaunchKernelGGL(k_weight_total, dim3(1), dim3(kDensBlock), 0, stream,
                           (const double*)partial, nw, partial + nw);
    hipLaunchKernelGGL(k_select, dim3((unsigned)((N + kPickChunk - 1) / kPickChunk)),
                       dim3(kDensBlock), 0, stream, x, N, mode, k,
                       (const double*)(total ? partial + nw : partial), total ? (int64_t)1 : nw, u,
                       sel);
}

void launch_densify_subdivide(float* v, float* o, float* sigma, float* sh, int nsh, int64_t N,
                              int64_t capacity, const uint8_t* sel, void* ws, uint32_t* d_out,
                              hipStream_t stream)
{
    uint32_t* cnt = reinterpret_cast<uint32_t*>(ws);
    auto go = [&](auto per_thread, auto spans) {
        constexpr int F = decltype(per_thread)::value;
        constexpr bool SPANS = decltype(spans)::value;
        const int64_t nb = (N + F * kDensBlock - 1) / (F * kDensBlock);
        uint32_t* span = cnt + nb;
        hipLaunchKernelGGL(k_count_sel<F>, dim3((unsigned)nb), dim3(kDensBlock), 0, stream, sel, N,
                           cnt);
        if (SPANS)
            hipLaunchKernelGGL(k_sum_counts, dim3((unsigned)((nb + kSpan - 1) / kSpan)),
                               dim3(kDensBlock), 0, stream, (const uint32_t*)cnt, nb, span);
        hipLaunchKernelGGL((k_subdivide<F, SPANS>), dim3((unsigned)nb, 2), dim3(kDensBlock), 0,
                           stream, v, o, sigma, sh, nsh, N, capacity, sel, (const uint32_t*)cnt,
                           (const uint32_t*)span, nb, d_out);
    };
    const std::integral_constant<int, kFew> few;
    const std::integral_constant<int, kMany> many;
    if (N <= kFewTriangles) go(few, std::false_type{});
    else if (N <= kManyTriangles) go(many, std::false_type{});
    else go(many, std::true_type{});
}

}  // namespace ts
