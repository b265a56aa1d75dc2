// raster.hip -- per-tile compositing on gfx950: forward (front to back) and
// backward (back to front, transmittance recovered from the final value).
//
// One 256-thread workgroup per 16x16 tile.  The tile's list is walked in
// batches of 256 entries staged through LDS: each thread copies one record as
// six 16-byte chunks and its depth into chunk-major arrays (consecutive lanes
// write consecutive slots: no bank conflicts) and marks the cells of the tile
// that can hold a pixel it composites.  Every cell walks its own list of byte
// indices of the batch's entries, so a pixel never evaluates a triangle that
// misses its cell; the lists live in LDS and are read one byte per lane per
// step: no scalar list bookkeeping.  The walk is bound by vector instructions,
// so what counts is the number of wave steps: the longest of a wave's lists.
//
// Forward: the cells are the 64 pixel quads (2x2 pixels), in rows of eight,
// 16 to a wave; lane 4 q + i shades pixel i of quad q.  Each lane has the
// quads of its entry as 64 bits, which the wave transposes, so lane q of the
// wave that walks quad q has the entries (wave w stages entries 64 w on).
// Against 4x4 blocks, four to a wave: a triangle of the 3M view covers 3-4
// pixels, which 16 lanes evaluate; 720p forward 113.7 -> 76.6 us (vector
// instructions 46.4M -> 29.9M), 1040p 160 -> 109, 300k 23.3 -> 20.8, 20k at
// 256x256 28.3 -> 22.1, sigmoid window 250 -> 210, LogSumExp 37.1 -> 32.2.
//
// Backward: the cells are 4x4 blocks.  Wave w owns the 8x8 quadrant (w & 1,
// w >> 1) and each of its four 16-lane rows (a DPP row) a 4x4 block of it:
// lane l shades pixel (l & 3, (l >> 2) & 3) of block g = l >> 4 = (g & 1,
// g >> 1), and a row sums an entry's gradients over its 16 pixels.
//
// Both walks keep their lane masks (active, contributing, composited) as
// scalars, load a step's record ahead of its arithmetic, and have no branch a
// wave usually takes.  3M triangles: forward 76.6 -> 73.0 us, backward 153 ->
// 138 us; 20k at 256x256 22.1 -> 19.5 and 39.1 -> 33.6; sigmoid window 210 -> 198
// and 480 -> 449.  The backward's sums behind a fragment stay one per channel: a
// single sum of the scalar products with the upstream gradient is two per cent
// faster there, and its cancellation cost up to five times the error on vertex
// gradients (20k triangles, 1e-5 -> 5e-5 of their norm).
//
// The window is evaluated as three FP64 affine functions per pixel (gfx950
// issues v_fma_f64 at the rate of unpacked v_fma_f32); the rest is FP32,
// written without branches so a wave issues one path per step.  Every
// kernel is instantiated per window function (TS_WINDOW_*).
#include "ts_device.h"
#include "ts_kernels.h"

#include <algorithm>

namespace ts {

constexpr int kBatch = kBlock;   // entries staged per batch
constexpr int kChunks = 6;       // 16-byte chunks of a record the raster reads (and its depth)

// phi_lse(s) of each staged entry, for the LogSumExp window only: the other
// windows get an empty base, so their LDS footprint (32000 bytes, 25 blocks
// of the 1280-byte allocation unit: five workgroups per CU) is unchanged.
template <int WIN, int NB>
struct StageExtra {
    static constexpr bool kLse = false;
};
template <int NB>
struct StageExtra<TS_WINDOW_LSE, NB> {
    static constexpr bool kLse = true;
    float ps[NB];
};

template <int WIN, int NB>
struct StageBase : StageExtra<WIN, NB> {
    static constexpr int kN = NB;
    float4 q[kChunks][NB];
    uint2 zt[NB];            // depth (bits), triangle
    uint16_t hit[NB];        // bit 4 w + g: may composite in block g of quadrant w
    uint8_t list[16][NB];    // per block 4 w + g: its entries of the batch, in order
};

// The forward's LDS.  mask[.][c][q]: which of the batch's entries 64 c ..
// 64 c + 63 quad q may composite (low and high word); words: the lists of the
// four waves, those of a wave's quads one after another, then a word per entry.
//
// The forward that keeps pruning statistics gathers them per batch entry in
// words that are free during its walk: the largest T*o (float bits;
// non-negative floats order as integers) in the entries' words, the blocks
// where they composited and their composited pixels as 16-bit halves of the
// masks (dead once every wave has read them).  One global max and one add per
// entry and tile flush them at the end of the batch.
constexpr int kWaveList = 1024;   // entries of a wave's lists: one word of masks always fits

template <int WIN>
struct FwdStage : StageExtra<WIN, kBatch> {
    static constexpr int kN = kBatch;
    float4 q[kChunks][kBatch];
    uint32_t mask[2][kBatch / 64][64];
    uint32_t words[kWaveList + kBatch];
    uint32_t done[4];   // per wave: all its pixels are done

    // the lists of wave w; an idle lane may read up to kBatch bytes past their
    // end, in the next wave's lists or the entries' words, and uses nothing of it
    __device__ uint8_t* list(int w) { return reinterpret_cast<uint8_t*>(words) + w * kWaveList; }
    // a word per staged entry
    __device__ uint32_t* tri() { return words + kWaveList; }
};

// fewest tiles of an image that has wide entries summed
constexpr int kWideImage = 1024, kWideImageSigmoid = 800;
constexpr int kWideSlots = 10;           // what 25 LDS allocation units leave room for
constexpr int kWideBlocks = 8;           // blocks that make an entry wide (4, 6: +1 us at 3M)
constexpr uint32_t kWideTri = 0xffffff00u;   // above any triangle: a slot, not a triangle

// The backward's LDS.  The gradients of an entry take one line of global atomics
// for each 4x4 block of the tile that composited it: 1-2 blocks for most
// triangles of a scene, which LDS sums would not pay for (3M triangles 0.156 ->
// 0.193 ms, 20k 0.040 -> 0.055 ms).  Pixel quads as the backward's cells, as in
// the forward: fewer vector instructions (77.0M -> 70.1M at 3M) but 1.5 times
// the lines of atomics, and slower (0.153 -> 0.195 ms, 300k 0.0245 -> 0.0477 ms).
//
// Wide entries (W): where a few triangles cover many tiles, their lines take an
// atomic per block from all over the chip, one after another.  In a batch the
// first kSlots entries that composited in half a tile's blocks are summed here
// and cost one row per tile; their zt holds the slot instead of the triangle.
// Raster backward of a 300k-triangle cluster view with such triangles 63.9 -> 22
// us; the LogSumExp step of four 300k soups 119-136 -> 107-115 us.  A step pays
// one comparison more (3M triangles 137.1 -> 139.1 us, 20k at 256x256 34.6 ->
// 35.5, a LogSumExp soup with few wide triangles 29.7 -> 31.2).  Images of fewer
// than kWideImage tiles go without: soups of small triangles would lose 2-4%
// there (300k at 640x360 16.0 -> 16.4 us), those with wide ones gain (2k triangles
// of edge 1 at 256x256 64.6 -> 36.7, at 640x360 265 -> 85).
//
// Sigmoid window: its triangles cover most blocks of many tiles, so there is a
// slot for every entry of a batch (of 128: the slots take 64 bytes each).  Raster
// backward of 300k triangles (1788 entries per tile) 580 -> 381 us, and 423 with
// every entry summed here; 1M of a fifth of the sigma (3.3 blocks an entry) 265
// -> 251, and 287 with every entry.  In small images the halved batches cost more
// than the lines saved: without slots / with, dense and narrow soups, 256 tiles
// 119 / 141 and 10.5 / 11.5 us, 768 tiles 184 / 192 and 20.7 / 22.0, 920 tiles 86
// / 70 and 20.9 / 22.2, 1850 tiles 151 / 105 and 18.8 / 17.4.  The stored-fragment
// form (WIDE and SF) sums every entry, in images of any size: 300k triangles 1.89
// ms, 1.99 with the wide ones only, 2.51 with none.
template <int WIN, bool W>
struct BwdStage : StageBase<WIN, kBatch> {};
template <int WIN>
struct BwdStage<WIN, true> : StageBase<WIN, kBatch> {
    static constexpr int kSlots = kWideSlots;
    uint32_t wide[2];              // wide entries of this batch and of the one before
    uint32_t tri[2][kSlots];       // their triangles
    float acc[kSlots * TS_G2D_STRIDE];
};
template <>
struct BwdStage<TS_WINDOW_SIGMOID, true> : StageBase<TS_WINDOW_SIGMOID, 128> {
    static constexpr int kSlots = 128;
    uint32_t wide[2];
    uint32_t tri[2][kSlots];
    float acc[kSlots * TS_G2D_STRIDE];
};

union RecView {
    float4 q[8];
    TriRecord r;
};

// The staged copy holds C_k relative to the tile's corner pixel (tx0, ty0)
// instead of the record's anchor, so a lane evaluates u_k = A_k dx + B_k dy +
// C_k with its own fixed offset in the tile (no per-step conversion).  The
// forward (ZA) needs no anchor after that: it stages the depth in the
// anchor's four bytes, so a step reads C[2], z and o with one 16-byte load.
template <bool ZA, class Stage>
__device__ __forceinline__ void write_stage(Stage& S, RecView& u, int tx0, int ty0)
{
    const double ox = (double)(tx0 - u.r.ax), oy = (double)(ty0 - u.r.ay);
#pragma unroll
    for (int k = 0; k < 3; ++k) u.r.C[k] = fma(u.r.A[k], ox, fma(u.r.B[k], oy, u.r.C[k]));
    if constexpr (ZA) u.q[4].z = u.r.z;   // bytes 72-75: the anchor
#pragma unroll
    for (int c = 0; c < kChunks; ++c) S.q[c][threadIdx.x] = u.q[c];
    if constexpr (Stage::kLse) S.ps[threadIdx.x] = u.r.phis;
}

template <class Stage>
__device__ __forceinline__ void stage_copy(Stage& S, const TriRecord* __restrict__ rec,
                                           uint32_t tri, int tx0, int ty0)
{
    const float4* src = reinterpret_cast<const float4*>(rec + tri);
    RecView u;
    constexpr int nc = Stage::kLse ? 8 : 7;   // phis sits in chunk 7
#pragma unroll
    for (int c = 0; c < nc; ++c) u.q[c] = src[c];
    write_stage<false>(S, u, tx0, ty0);
    S.zt[threadIdx.x] = make_uint2(__float_as_uint(u.r.z), tri);
}

// Copy record `tri` into LDS slot threadIdx.x and return the mask of the
// tile's sixteen 4x4 blocks that may hold a composited pixel of it: the
// tight box touches the block, and for every edge k the largest u_k over the
// block's pixel centres (at one corner, u_k being affine) reaches ut, the
// lower bound of u over pixels that composite.  The box and the three edge
// tests are the separating axes of the tight region (a triangle) and the
// block's square of pixel centres.  The slack covers the rounding of this
// evaluation and of the per-pixel one, so no pixel that composites is lost.
template <class Stage>
__device__ __forceinline__ uint32_t stage_rec(Stage& S, const TriRecord* __restrict__ rec,
                                              uint32_t tri, int tx0, int ty0)
{
    const float4* src = reinterpret_cast<const float4*>(rec + tri);
    RecView u;
#pragma unroll
    for (int c = 0; c < 8; ++c) u.q[c] = src[c];
    write_stage<false>(S, u, tx0, ty0);
    S.zt[threadIdx.x] = make_uint2(__float_as_uint(u.r.z), tri);
    uint32_t cx = 0, cy = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int x0 = tx0 + 4 * i, y0 = ty0 + 4 * i;
        cx |= (u.r.px0 <= x0 + 3 && u.r.px1 >= x0) ? (1u << i) : 0u;
        cy |= (u.r.py0 <= y0 + 3 && u.r.py1 >= y0) ? (1u << i) : 0u;
    }
    uint32_t box = 0;   // bit 4 by + bx
#pragma unroll
    for (int by = 0; by < 4; ++by) box |= ((cy >> by) & 1u) ? (cx << (4 * by)) : 0u;

    const double ut = (double)u.r.ut;
    // tile-relative coefficients read back from this thread's own LDS slot,
    // one edge at a time, to keep the register peak of the staging step low
    const double* cf = reinterpret_cast<const double*>(&S.q[0][0]);
#pragma unroll 1
    for (int k = 0; k < 3; ++k) {
        auto coef = [&](int idx) {   // double idx of the record: chunk idx / 2, half idx % 2
            return cf[2 * (size_t)((idx >> 1) * Stage::kN + threadIdx.x) + (idx & 1)];
        };
        const double A = coef(k), B = coef(3 + k), C = coef(6 + k);
        const double cxk = A > 0.0 ? 3.0 : 0.0, cyk = B > 0.0 ? 3.0 : 0.0;
        const double base = fma(A, cxk, fma(B, cyk, C));   // largest u_k over block (0, 0)
        const double slack = 0x1p-46 * (fabs(C) + 16.0 * (fabs(A) + fabs(B)));
        const double lim = ut - slack;
        const double A4 = 4.0 * A, B4 = 4.0 * B;
#pragma unroll 1
        for (int by = 0; by < 4; ++by) {
            const double rb = fma(B4, (double)by, base);
#pragma unroll
            for (int bx = 0; bx < 4; ++bx) {
                const double val = fma(A4, (double)bx, rb);
                box &= val >= lim ? ~0u : ~(1u << (4 * by + bx));
            }
        }
    }
    uint32_t m = 0;
#pragma unroll
    for (int by = 0; by < 4; ++by)
#pragma unroll
        for (int bx = 0; bx < 4; ++bx) {
            const int w = (bx >> 1) + 2 * (by >> 1), g = (bx & 1) + 2 * (by & 1);
            m |= ((box >> (4 * by + bx)) & 1u) << (4 * w + g);
        }
    return m;
}

template <int CTRL>
__device__ __forceinline__ float dpp(float x)
{
    return __builtin_bit_cast(
        float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xf, 0xf, true));
}

template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u(uint32_t x)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xf, 0xf, true);
}

// Bits [lo, hi] of eight, none if the interval misses them.
__device__ __forceinline__ uint32_t span8(int lo, int hi)
{
    lo = max(lo, 0);
    hi = min(hi, 7);
    return lo <= hi ? (2u << hi) - (1u << lo) : 0u;
}

// Copy record `tri` into LDS slot threadIdx.x and return the tile's quads
// (bit 8 y + x) that may hold a composited pixel of it: the tight box touches
// the quad, and for every edge k the largest u_k over the quad's four pixel
// centres reaches ut (the separating axes of stage_rec's test).
//
// Along a row of quads A X + (B Y + K) >= 0 is a half line, so an edge costs
// one FMA, a clamp, a conversion and a shift for eight quads.  In FP32: the
// slack of 2^-16 S, S = |C| + 16 (|A| + |B|), covers the coefficients' and
// this evaluation's rounding (2^-21 S) and the floor under |A| that keeps the
// slope finite (28 2^-22 S over the tile), and loses no selectivity to speak
// of (a thousandth of u).  A sum that FP32 cannot hold keeps every quad; a
// NaN keeps none.
struct Quads {
    uint32_t lo, hi;
};

template <class Stage>
__device__ __forceinline__ Quads stage_quads(Stage& S, const TriRecord* __restrict__ rec,
                                             uint32_t tri, int tx0, int ty0)
{
    const float4* src = reinterpret_cast<const float4*>(rec + tri);
    RecView u;
#pragma unroll
    for (int c = 0; c < 8; ++c) u.q[c] = src[c];
    const uint32_t cx = span8((u.r.px0 - tx0) >> 1, (u.r.px1 - tx0) >> 1);
    const uint32_t cy = span8((u.r.py0 - ty0) >> 1, (u.r.py1 - ty0) >> 1);
    const float ut = u.r.ut;
    write_stage<true>(S, u, tx0, ty0);   // makes C tile-relative
    uint32_t row[8];
#pragma unroll
    for (int y = 0; y < 8; ++y) row[y] = cx & (uint32_t)__builtin_amdgcn_sbfe((int)cy, y, 1);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const float A = (float)u.r.A[k], B = (float)u.r.B[k], C = (float)u.r.C[k];
        const float sum = fabsf(C) + 16.f * (fabsf(A) + fabsf(B));
        // A X + B Y + K at quad (X, Y)'s largest pixel centre, pixels 2 X, 2 Y on
        const float K = C - ut + 0x1p-16f * sum + fmaxf(A, 0.f) + fmaxf(B, 0.f);
        const float inv = __builtin_amdgcn_rcpf(2.f * fmaxf(fabsf(A), fmaf(0x1p-22f, sum, 1e-30f)));
        const bool neg = A < 0.f;          // X < t, else X > t
        const float si = neg ? inv : -inv;
        const bool big = !(sum < 1e30f);
        const float slope = big ? 0.f : 2.f * B * si;
        const float t0 = big ? (neg ? 9.f : 0.f) : fmaf(K, si, 1.f);
        const uint32_t flip = neg ? 0xffu : 0u;
        const uint32_t nan = sum == sum ? 0xffu : 0u;
#pragma unroll
        for (int y = 0; y < 8; ++y) {
            const float t = __builtin_amdgcn_fmed3f(fmaf(slope, (float)y, t0), 0.f, 8.f);
            row[y] &= ((0xffu << (uint32_t)t) ^ flip) & nan;
        }
    }
    return Quads{row[0] | (row[1] << 8) | (row[2] << 16) | (row[3] << 24),
                 row[4] | (row[5] << 8) | (row[6] << 16) | (row[7] << 24)};
}

// Transpose the wave's 64x64 bits: lane l gives the quads of entry l, lane q
// receives the entries of quad q.  Six exchanges with lane l ^ s, s = 32 .. 1,
// each of which swaps bit s of the row index and of the column index; 40 VALU,
// where 64 ballots would take several each.
__device__ __forceinline__ void transpose64(uint32_t& lo, uint32_t& hi, int lane)
{
    {
        const auto t = __builtin_amdgcn_permlane32_swap(lo, hi, false, false);
        lo = t[0];
        hi = t[1];
    }
    const uint32_t s16 = lane & 16 ? 0x07060302u : 0x05040100u;
    const uint32_t s8 = lane & 8 ? 0x03070105u : 0x06020400u;
    auto step16 = [&](uint32_t x) {
        const auto t = __builtin_amdgcn_permlane16_swap(x, x, false, false);
        return __builtin_amdgcn_perm(t[1], t[0], s16);
    };
    auto bits = [&](uint32_t x, uint32_t t, int s, uint32_t M) {
        const bool up = lane & s;
        const uint32_t rot = __builtin_amdgcn_alignbit(t, t, up ? s : 32 - s);
        const uint32_t take = up ? M : ~M;
        return (rot & take) | (x & ~take);
    };
    auto rest = [&](uint32_t x) {
        x = __builtin_amdgcn_perm(dpp_u<0x128>(x), x, s8);             // lane ^ 8
        x = bits(x, dpp_u<0x1B>(dpp_u<0x141>(x)), 4, 0x0f0f0f0fu);     // lane ^ 7 ^ 3
        x = bits(x, dpp_u<0x4E>(x), 2, 0x33333333u);
        return bits(x, dpp_u<0xB1>(x), 1, 0x55555555u);
    };
    lo = rest(step16(lo));
    hi = rest(step16(hi));
}

// Inclusive sum over the wave's lanes.
__device__ __forceinline__ int wave_scan(int x)
{
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);   // row_shr:1
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);   // row_bcast:15
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);   // row_bcast:31
    return x;
}

template <bool ZA = false, class Stage>
__device__ __forceinline__ TriRecord read_rec(const Stage& S, int j)
{
    RecView u;
#pragma unroll
    for (int c = 0; c < kChunks; ++c) u.q[c] = S.q[c][j];
    if constexpr (ZA) u.r.z = u.q[4].z;
    else u.r.z = __uint_as_float(S.zt[j].x);
    if constexpr (Stage::kLse) u.r.phis = S.ps[j];
    return u.r;
}

// Write the entry lists of the wave's four blocks for a batch of n entries:
// S.list[4 w + g] receives, in increasing order, the entries e < lim_g whose
// mark for block g is set.  Returns the four lengths (wave-uniform).
struct Lens {
    int n0, n1, n2, n3;
};

template <class Stage>
__device__ __forceinline__ Lens build_lists(Stage& S, int n, int w, int lane, int lim0,
                                            int lim1, int lim2, int lim3)
{
    Lens L{0, 0, 0, 0};
    uint8_t* l0 = S.list[4 * w];
    uint8_t* l1 = S.list[4 * w + 1];
    uint8_t* l2 = S.list[4 * w + 2];
    uint8_t* l3 = S.list[4 * w + 3];
#pragma unroll
    for (int c = 0; c < Stage::kN / 64; ++c) {
        // short lists (25 entries a tile at 300k triangles) need one round of the
        // four: forward 25.9 -> 23.4 us, backward 26.1 -> 24.8 us
        if (c * 64 >= n) break;   // the same for the wave
        const int e = c * 64 + lane;
        const uint32_t h = e < n ? ((uint32_t)S.hit[e] >> (4 * w)) & 0xfu : 0u;
        auto put = [&](uint32_t bit, int lim, uint8_t* lst, int& len) {
            const uint64_t m = ballot64(bit != 0u) & ballot64(e < lim);
            const uint32_t below = __builtin_amdgcn_mbcnt_hi(
                (uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
            if (lanes(m)) lst[len + (int)below] = (uint8_t)e;
            len += __popcll(m);
        };
        put(h & 1u, lim0, l0, L.n0);
        put(h & 2u, lim1, l1, L.n1);
        put(h & 4u, lim2, l2, L.n2);
        put(h & 8u, lim3, l3, L.n3);
    }
    // the lists are read by other lanes of this wave only: order the byte
    // writes before those reads without a workgroup barrier
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    return L;
}

__device__ __forceinline__ int per_row(int g, int j0, int j1, int j2, int j3)
{
    return g == 0 ? j0 : g == 1 ? j1 : g == 2 ? j2 : j3;
}

// min_k u_k without the arg-min, for the forward: one v_min_f64 per edge
// instead of a compare and two selects.  The three u_k are the same FMAs as
// in edge_min, so the minimum is the same double.
__device__ __forceinline__ double edge_min_value(const double* A, const double* B,
                                                 const double* C, double dx, double dy)
{
    const double u0 = fma(A[0], dx, fma(B[0], dy, C[0]));
    const double u1 = fma(A[1], dx, fma(B[1], dy, C[1]));
    const double u2 = fma(A[2], dx, fma(B[2], dy, C[2]));
    return fmin(fmin(u0, u1), u2);
}

// Window and opacity of a staged record at the pixel (dx, dy) from the
// tile's corner.  Returns whether the pixel is in the window's support (the
// forms of Eq. 1: u > 0; the sigmoid: everywhere).  Forward (K = false: no
// arg-min edge) and backward take the same alpha and the same decisions.
template <int WIN, bool K = true>
__device__ __forceinline__ bool frag_alpha(const TriRecord& r, double dx, double dy,
                                           float alpha_max, Frag& f)
{
    int k = 0;
    if constexpr (WIN == TS_WINDOW_SIGMOID) {
        const double d = K ? edge_min(r.A, r.B, r.C, dx, dy, k)
                           : edge_min_value(r.A, r.B, r.C, dx, dy);
        sigmoid_alpha(d, r.o, r.sigma, alpha_max, f);
        f.k = k;
        return true;
    } else if constexpr (WIN == TS_WINDOW_LSE) {
        const double u = lse_u(r.A, r.B, r.C, dx, dy, (double)r.phis, f);
        window_alpha((float)(u > 0.0 ? u : 0.0), r.o, r.sigma, alpha_max, f);
        return u > 0.0;
    } else {
        const double u = K ? edge_min(r.A, r.B, r.C, dx, dy, k)
                           : edge_min_value(r.A, r.B, r.C, dx, dy);
        // clamped after the conversion: one FP32 max instead of two FP64 ones
        window_alpha(fmaxf((float)u, 0.f), r.o, r.sigma, alpha_max, f);
        f.k = k;
        return u > 0.0;
    }
}

struct Pix {
    int w, g, i;    // wave, row, lane within the row
    int px, py;
};

__device__ __forceinline__ Pix pixel_of(int tx, int ty)
{
    Pix P;
    const int tid = threadIdx.x, lane = tid & 63;
    P.w = tid >> 6;
    P.g = lane >> 4;
    P.i = lane & 15;
    P.px = tx * kTile + (P.w & 1) * 8 + (P.g & 1) * 4 + (P.i & 3);
    P.py = ty * kTile + (P.w >> 1) * 8 + (P.g >> 1) * 4 + (P.i >> 2);
    return P;
}

// Largest value over the four lanes of each pixel quad.
__device__ __forceinline__ float quad_max_f(float x)
{
    x = fmaxf(x, dpp<0xB1>(x));      // quad_perm [1,0,3,2]
    return fmaxf(x, dpp<0x4E>(x));   // quad_perm [2,3,0,1]
}

// ---------------------------------------------------------------------------
// Forward
// ---------------------------------------------------------------------------

// One tile of one view.  T_final / last may be null (forward-only serving).
struct TileJob {
    int tx, ty, W, H;
    uint32_t start, end;
    float* rgb;
    float* alpha;
    float* depth;
    float* T;
    uint32_t* last;
    uint16_t* blocks;   // per list entry: blocks where it composited (null: not kept)
    float* max_weight;  // pruning statistics (null: not kept): largest T*o per triangle,
    uint32_t* pixels;   // and pixels where it is composited
    // stored-fragment variant: per pixel the number of composited fragments,
    // their first slot, and per slot the tile-list entry, alpha and the
    // transmittance in front of the fragment
    uint32_t* fcount;
    const uint32_t* foffs;
    uint32_t* fentry;
    float* falpha;
    float* fT;
};

// FS: 0 plain forward; 1 also counts each pixel's composited fragments
// (J.fcount); 2 also stores them at J.foffs[pixel] (the stored-fragment
// variant the recompute backward is measured against).
template <int WIN, bool ST, int FS = 0>
__device__ __forceinline__ void fwd_tile(const TriRecord* __restrict__ rec,
                                         const uint32_t* __restrict__ vals, const Cfg& cfg,
                                         const TileJob& J, FwdStage<WIN>& S)
{
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int qi = lane >> 2, i = lane & 3;   // quad of the wave, pixel of the quad
    const int lx = 2 * (qi & 7) + (i & 1), ly = 4 * w + 2 * (qi >> 3) + (i >> 1);
    const int px = J.tx * kTile + lx, py = J.ty * kTile + ly;
    const bool inside = px < J.W && py < J.H;
    const uint32_t start = J.start, end = J.end;

    float T = 1.f, C0 = 0.f, C1 = 0.f, C2 = 0.f, D = 0.f;
    uint32_t last = 0;
    uint64_t done = ballot64(!inside);   // lanes whose pixel takes nothing more
    uint32_t fcnt = 0, foff = 0;
    if constexpr (FS == 2) {
        if (inside) foff = J.foffs[(int64_t)py * J.W + px];
    }

    // the quad's 4x4 block: bit 4 (quadrant) + block of the quadrant
    const uint32_t my_bit = 1u << (8 * (w >> 1) + 4 * (lx >> 3) + 2 * (w & 1) + ((lx >> 2) & 1));
    const double dxt = (double)lx, dyt = (double)ly;
    uint8_t* const list = S.list(w);
    uint32_t* const tri_w = S.tri();
    uint32_t* const comp_bits = &S.mask[0][0][0];      // with statistics, once the
    uint32_t* const comp_px = comp_bits + kBatch / 2;  // masks are read: 16 bits per entry
    if (lane == 0) S.done[w] = 0u;
    uint32_t next = start + tid < end ? vals[start + tid] : 0u;   // entry to stage, loaded a batch ahead
    for (uint32_t b = start; b < end; b += kBatch) {
        const int n = (int)min((uint32_t)kBatch, end - b);
        __syncthreads();
        if ((tid & ~63) < n) {   // the wave stages entries
            Quads Q{0u, 0u};
            if (tid < n) {
                const uint32_t tri = next;
                // the statistics' max-weight word; without statistics, the blocks
                // where the entry composited (one word per entry: no shifts per step)
                tri_w[tid] = 0u;
                Q = stage_quads(S, rec, tri, J.tx * kTile, J.ty * kTile);
            }
            transpose64(Q.lo, Q.hi, lane);
            S.mask[0][w][lane] = Q.lo;
            S.mask[1][w][lane] = Q.hi;
        }
        next = b + kBatch + tid < end ? vals[b + kBatch + tid] : 0u;
        __syncthreads();
        // lane 4 q + c lists the entries of word c of the wave's quad q
        const bool word = (lane & 3) * 64 < n;
        const uint32_t mlo = word ? S.mask[0][lane & 3][16 * w + qi] : 0u;
        const uint32_t mhi = word ? S.mask[1][lane & 3][16 * w + qi] : 0u;
        if constexpr (ST) {
            __syncthreads();
            comp_bits[tid] = 0u;
            __syncthreads();
        }
        // all lists at once if they fit, else word by word
        const int cnt = __popc(mlo) + __popc(mhi);
        int incl = wave_scan(cnt);
        const bool fits = __builtin_amdgcn_readlane(incl, 63) <= kWaveList;
        for (int c = 0; c < (fits ? 1 : kBatch / 64); ++c) {
            const bool mine = fits || (lane & 3) == c;
            if (!fits) incl = wave_scan(mine ? cnt : 0);
            const int excl = incl - (mine ? cnt : 0);
            {
                uint32_t ml = mine ? mlo : 0u, mh = mine ? mhi : 0u;
                int pl = excl, ph = excl + __popc(ml);
                while (ml | mh) {
                    if (ml) {
                        list[pl++] = (uint8_t)((lane & 3) * 64 + __builtin_ctz(ml));
                        ml &= ml - 1u;
                    }
                    if (mh) {
                        list[ph++] = (uint8_t)((lane & 3) * 64 + 32 + __builtin_ctz(mh));
                        mh &= mh - 1u;
                    }
                }
            }
            // the lists are read by other lanes of this wave only: order the byte
            // writes before those reads without a workgroup barrier
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            const int from = __builtin_amdgcn_update_dpp(0, excl, 0x00, 0xf, 0xf, true);   // lane 0 of the quad
            const int len = __builtin_amdgcn_update_dpp(0, incl, 0xFF, 0xf, 0xf, true) - from;   // lane 3
            // each lane walks its quad's list; a quad stops once all its pixels are
            // done, the wave once no quad has work left
            const uint8_t* lst = list + (len > 0 ? from : 0);
            int jn = lst[0];   // next entry (read one step ahead)
            asm volatile("" : "+v"(jn));   // else kept as a byte and widened every step
            // Lane masks are scalars (a ballot of a comparison is the comparison),
            // so a step's conditions and the marks below cost no vector
            // instruction.  The test at the bottom keeps the loop a single block
            // (no copies of the blend state per step).
            uint64_t act = ballot64(0 < len) & ~done;
            if (act != 0ull) for (int k = 0;;) {
                // an idle lane reads slot 0 (always staged): a stale slot could hold
                // non-finite values, and 0 * inf in the branch-free blend is NaN
                const int jl = jn;              // this step's entry of the quad's list
                const int j = lanes(act) ? jl : 0;
                jn = lst[k + 1];
                const TriRecord r = read_rec<true>(S, j);
                Frag f;
                const bool in = frag_alpha<WIN, false>(r, dxt, dyt, cfg.alpha_max, f);
                const uint64_t contrib = act & ballot64(in) & ballot64(f.a >= cfg.alpha_min);
                const float Tn = T * (1.f - f.a);
                const uint64_t stop = contrib & ballot64(Tn < cfg.T_min);
                const uint64_t composited = contrib & ~stop;
                const bool comp = lanes(composited);
                const float wgt = comp ? f.a * T : 0.f;
                const float tw = comp ? T * r.o : 0.f;   // blending weight T*o (pruning)
                if constexpr (FS != 0) {
                    if (comp) {
                        if constexpr (FS == 2) {
                            const uint32_t q = foff + fcnt;
                            J.fentry[q] = b - start + (uint32_t)j;
                            J.falpha[q] = f.a;
                            J.fT[q] = T;
                        }
                        ++fcnt;
                    }
                }
                C0 = fmaf(wgt, r.rgb[0], C0);
                C1 = fmaf(wgt, r.rgb[1], C1);
                C2 = fmaf(wgt, r.rgb[2], C2);
                D = fmaf(wgt, r.z, D);
                T = comp ? Tn : T;
                last = comp ? b - start + (uint32_t)j + 1u : last;
                done |= stop;
                if (ST || J.blocks) {
                    uint64_t any = composited | (composited >> 1);   // lane 0 of each quad
                    any = (any | (any >> 2)) & 0x1111111111111111ull;
                    if (J.blocks && lanes(any)) {   // the entry composited in this block
                        if constexpr (ST) atomicOr(&comp_bits[jl >> 1], my_bit << (16 * (jl & 1)));
                        else atomicOr(&tri_w[jl], my_bit);
                    }
                    if constexpr (ST) {   // pruning statistics of the quad's entry, in LDS
                        const float mw = quad_max_f(tw);
                        if (lanes(any)) {
                            const uint32_t qbits = (uint32_t)(composited >> (lane & ~3)) & 0xfu;
                            atomicMax(&tri_w[jl], __float_as_uint(mw));
                            atomicAdd(&comp_px[jl >> 1], (uint32_t)__popc(qbits) << (16 * (jl & 1)));
                        }
                    }
                }
                ++k;
                act = ballot64(k < len) & ~done;
                if (act == 0ull) break;
            }
        }
        if (done == ~0ull && lane == 0) S.done[w] = 1u;
        __syncthreads();
        if (J.blocks && tid < n)
            J.blocks[b + tid] = ST ? (uint16_t)(comp_bits[tid >> 1] >> (16 * (tid & 1)))
                                   : (uint16_t)tri_w[tid];
        if constexpr (ST) {
            if (tid < n && tri_w[tid] != 0u) {
                const uint32_t tri = vals[b + tid];
                atomicMax(reinterpret_cast<uint32_t*>(J.max_weight) + tri, tri_w[tid]);
                atomicAdd(J.pixels + tri, (comp_px[tid >> 1] >> (16 * (tid & 1))) & 0xffffu);
            }
        }
        if ((S.done[0] & S.done[1] & S.done[2] & S.done[3]) != 0u) break;
    }
    if (inside) {
        const int64_t p = (int64_t)py * J.W + px;
        const int64_t hw = (int64_t)J.W * J.H;
        J.rgb[p] = fmaf(cfg.bg[0], T, C0);
        J.rgb[hw + p] = fmaf(cfg.bg[1], T, C1);
        J.rgb[2 * hw + p] = fmaf(cfg.bg[2], T, C2);
        J.alpha[p] = 1.f - T;
        J.depth[p] = D;
        if (J.T) J.T[p] = T;
        if (J.last) J.last[p] = last;
        if constexpr (FS == 1) J.fcount[p] = fcnt;
    }
}

template <int WIN, bool ST>
__global__ __launch_bounds__(256) void k_raster_fwd(
    const TriRecord* __restrict__ rec, const uint32_t* __restrict__ vals,
    const uint32_t* __restrict__ ranges, const uint32_t* __restrict__ order, Cam cam, Cfg cfg,
    int tiles_x, int num_tiles, float* __restrict__ out_rgb, float* __restrict__ out_alpha,
    float* __restrict__ out_depth, float* __restrict__ out_T, uint32_t* __restrict__ out_last,
    uint16_t* __restrict__ out_blocks, float* __restrict__ max_weight,
    uint32_t* __restrict__ pixels)
{
    __shared__ FwdStage<WIN> S;
    const int tile = order ? (int)order[blockIdx.x] : (int)blockIdx.x;
    if ((unsigned)tile >= (unsigned)num_tiles) return;   // a corrupt order never reads past ranges
    TileJob J{tile % tiles_x, tile / tiles_x, cam.W, cam.H, ranges[2 * tile],
              ranges[2 * tile + 1], out_rgb, out_alpha, out_depth, out_T, out_last, out_blocks,
              max_weight, pixels};
    fwd_tile<WIN, ST>(rec, vals, cfg, J, S);
}

// The forward of the stored-fragment variant: FS = 1 counts the composited
// fragments of every pixel, FS = 2 stores them (see fwd_tile).
template <int WIN, int FS>
__global__ __launch_bounds__(256) void k_raster_fwd_frag(
    const TriRecord* __restrict__ rec, const uint32_t* __restrict__ vals,
    const uint32_t* __restrict__ ranges, const uint32_t* __restrict__ order, Cam cam, Cfg cfg,
    int tiles_x, int num_tiles, float* __restrict__ out_rgb, float* __restrict__ out_alpha,
    float* __restrict__ out_depth, float* __restrict__ out_T, uint32_t* __restrict__ out_last,
    uint16_t* __restrict__ out_blocks, FragStore fs)
{
    __shared__ FwdStage<WIN> S;
    const int tile = order ? (int)order[blockIdx.x] : (int)blockIdx.x;
    if ((unsigned)tile >= (unsigned)num_tiles) return;
    TileJob J{tile % tiles_x, tile / tiles_x, cam.W, cam.H, ranges[2 * tile],
              ranges[2 * tile + 1], out_rgb, out_alpha, out_depth, out_T, out_last, out_blocks,
              nullptr, nullptr, fs.count, fs.offset, fs.entry, fs.alpha, fs.T};
    fwd_tile<WIN, false, FS>(rec, vals, cfg, J, S);
}

// The tiles of several views in one launch, longest first: workgroup b takes
// the positions b, b + gridDim.x, ... of the batch's tile order.  views[] is
// sorted by tile_offset; ctl[0] = views in the batch, ctl[1] = their tiles
// (both already clamped to the buffers).
//
// The grid is fixed (the launch is replayed by a graph), and up to kViewGroups
// tiles the hardware's dispatch balances them as it does those of one view; a
// workgroup with several takes ever shorter ones.  A queue head that four
// workgroups per CU advanced by atomics cost more than the tiles: two batches
// of four mixed views 193 us against 101 a launch, one 360p view 37.2 against
// 24.7 (grids of 4096 to 65280 workgroups within noise of each other).
constexpr int kViewGroups = 8192;

template <int WIN>
__global__ __launch_bounds__(256) void k_raster_fwd_views(
    const TriRecord* __restrict__ rec, const uint32_t* __restrict__ vals,
    const uint32_t* __restrict__ ranges, const uint32_t* __restrict__ order,
    const ts_view* __restrict__ views, const uint32_t* __restrict__ ctl, Cfg cfg,
    float* __restrict__ out_rgb, float* __restrict__ out_alpha, float* __restrict__ out_depth)
{
    __shared__ FwdStage<WIN> S;
    const uint32_t nviews = ctl[0], total = ctl[1];
    for (uint32_t q = blockIdx.x; q < total; q += gridDim.x) {
        __syncthreads();   // the last tile's reads of the stage are done
        const uint32_t t = order ? order[q] : q;
        if (t >= total) continue;
        uint32_t v = 0;
        while (v + 1 < nviews && views[v + 1].tile_offset <= t) ++v;
        const ts_view& V = views[v];
        const uint32_t local = t - V.tile_offset;
        const int64_t po = (int64_t)V.pixel_offset;
        TileJob J{(int)(local % V.tiles_x), (int)(local / V.tiles_x), V.cam.width, V.cam.height,
                  ranges[2 * t], ranges[2 * t + 1], out_rgb + 3 * po, out_alpha + po,
                  out_depth + po, nullptr, nullptr, nullptr, nullptr, nullptr};
        fwd_tile<WIN, false>(rec, vals, cfg, J, S);
    }
}

// ---------------------------------------------------------------------------
// Backward
// ---------------------------------------------------------------------------

// Sum 16 per-lane values over the 16 lanes of each DPP row by
// transpose-and-add: each step pairs lanes across one bit of the lane index
// within the row (row_ror:8, row_half_mirror, quad_perm) and each lane keeps
// the half of its values its partner sends it, so the values per lane halve.
// 33 VALU, no LDS.  On return lane i of a row holds the row total of slot i.
//
// The first two steps split the row by whole banks of four lanes, so the bank
// mask of a DPP add writes one half of the lanes from one value and a second
// add the other half from the other: two adds where a select of what to keep,
// one of what to send and an add stood (45 VALU; the same sums).  Inline
// assembly, since the compiler forms DPP adds of full masks only; a DPP
// operand has to be written two instructions before it is read, hence the
// s_nop ahead of each group (inside the groups the distances are larger).
// Raster backward of 3M triangles 158 -> 153 us, sigmoid window 501 -> 482 us.
#define TS_ADD8(d, x, y)                                                    \
    "v_add_f32_dpp %" #d ", %" #x ", %" #x " row_ror:8 row_mask:0xf bank_mask:0x3\n\t" \
    "v_add_f32_dpp %" #d ", %" #y ", %" #y " row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
#define TS_ADD4(d, x, y)                                                    \
    "v_add_f32_dpp %" #d ", %" #x ", %" #x " row_half_mirror row_mask:0xf bank_mask:0x5\n\t" \
    "v_add_f32_dpp %" #d ", %" #y ", %" #y " row_half_mirror row_mask:0xf bank_mask:0xa\n\t"

__device__ __forceinline__ float row_reduce16(const float (&v)[16], int i)
{
    float a8[8], a4[4], a2[2];
    // partner i ^ 8: lanes 0-7 of the row sum slots 0-7, lanes 8-15 slots 8-15
    asm("s_nop 1\n\t"
        TS_ADD8(0, 8, 16) TS_ADD8(1, 9, 17) TS_ADD8(2, 10, 18) TS_ADD8(3, 11, 19)
        TS_ADD8(4, 12, 20) TS_ADD8(5, 13, 21) TS_ADD8(6, 14, 22) TS_ADD8(7, 15, 23)
        : "=&v"(a8[0]), "=&v"(a8[1]), "=&v"(a8[2]), "=&v"(a8[3]), "=&v"(a8[4]), "=&v"(a8[5]),
          "=&v"(a8[6]), "=&v"(a8[7])
        : "v"(v[0]), "v"(v[1]), "v"(v[2]), "v"(v[3]), "v"(v[4]), "v"(v[5]), "v"(v[6]), "v"(v[7]),
          "v"(v[8]), "v"(v[9]), "v"(v[10]), "v"(v[11]), "v"(v[12]), "v"(v[13]), "v"(v[14]),
          "v"(v[15]));
    // partner i ^ 7, within each half by bit 2
    asm("s_nop 1\n\t" TS_ADD4(0, 4, 8) TS_ADD4(1, 5, 9) TS_ADD4(2, 6, 10) TS_ADD4(3, 7, 11)
        : "=&v"(a4[0]), "=&v"(a4[1]), "=&v"(a4[2]), "=&v"(a4[3])
        : "v"(a8[0]), "v"(a8[1]), "v"(a8[2]), "v"(a8[3]), "v"(a8[4]), "v"(a8[5]), "v"(a8[6]),
          "v"(a8[7]));
    const bool b1 = i & 2;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const float send = b1 ? a4[k] : a4[k + 2];
        const float keep = b1 ? a4[k + 2] : a4[k];
        a2[k] = keep + dpp<0x4E>(send);            // quad_perm [2,3,0,1] (partner i ^ 2)
    }
    const bool b0 = i & 1;
    return (b0 ? a2[1] : a2[0]) + dpp<0xB1>(b0 ? a2[0] : a2[1]);   // quad_perm [1,0,3,2]
}

// Maximum over the 16 lanes of each row.
__device__ __forceinline__ uint32_t row_max(uint32_t x)
{
    x = max(x, dpp_u<0x128>(x));
    x = max(x, dpp_u<0x141>(x));
    x = max(x, dpp_u<0x4E>(x));
    x = max(x, dpp_u<0xB1>(x));
    return x;
}

// SF: the stored-fragment variant: the composited fragments of each pixel,
// their alphas and transmittances come from the forward's store (fs) instead
// of the recomputed cut-off decisions and T_before = T_after / (1 - alpha).
template <int WIN, bool SF = false, bool WIDE = false>
__global__ __launch_bounds__(256) void k_raster_bwd(
    const TriRecord* __restrict__ rec, const uint32_t* __restrict__ vals,
    const uint32_t* __restrict__ ranges, const uint32_t* __restrict__ order, Cam cam, Cfg cfg,
    int tiles_x, int num_tiles, const float* __restrict__ dL_drgb,
    const float* __restrict__ dL_dalpha, const float* __restrict__ dL_ddepth,
    const float* __restrict__ T_final, const uint32_t* __restrict__ last_in,
    const uint16_t* __restrict__ blocks, float* __restrict__ g2d, FragStore fs)
{
    __shared__ BwdStage<WIN, WIDE> S;
    __shared__ uint32_t s_max;
    const int tile = order ? (int)order[blockIdx.x] : (int)blockIdx.x;
    if ((unsigned)tile >= (unsigned)num_tiles) return;   // a corrupt order never reads past ranges
    const int tx = tile % tiles_x, ty = tile / tiles_x;
    const int tid = threadIdx.x, lane = tid & 63;
    const Pix P = pixel_of(tx, ty);
    const bool inside = P.px < cam.W && P.py < cam.H;
    const uint32_t start = ranges[2 * tile], end = ranges[2 * tile + 1];

    const int64_t p = (int64_t)P.py * cam.W + P.px;
    const int64_t hw = (int64_t)cam.W * cam.H;
    const double dxt = (double)(P.px - tx * kTile), dyt = (double)(P.py - ty * kTile);
    float T = 1.f, Tf = 1.f, g0 = 0.f, g1 = 0.f, g2 = 0.f, gA = 0.f, gD = 0.f;
    uint32_t my_last = 0;
    if (inside) {
        Tf = T_final[p];
        T = Tf;
        my_last = min(last_in[p], end - start);   // never beyond this tile's list
        g0 = dL_drgb[p];
        g1 = dL_drgb[hw + p];
        g2 = dL_drgb[2 * hw + p];
        gA = dL_dalpha ? dL_dalpha[p] : 0.f;
        gD = dL_ddepth ? dL_ddepth[p] : 0.f;
    }
    // stored fragments of the pixel, walked from its last one back: the next
    // one to meet (entry, alpha, T) is held in registers, its successor loaded
    // as soon as it is consumed
    int fcur = -1, flo = 0;
    uint32_t fe = 0xffffffffu;
    float fa = 0.f, fTb = 1.f;
    if constexpr (SF) {
        if (inside) {
            flo = (int)fs.offset[p];
            fcur = flo + (int)fs.count[p] - 1;
            if (fcur >= flo) {
                fe = fs.entry[fcur];
                fa = fs.alpha[fcur];
                fTb = fs.T[fcur];
            }
        }
    }
    // alpha-gradient part that multiplies T_final / (1 - a): dL/dalpha minus
    // the background seen through the remaining transmittance
    const float gT = gA - (g0 * cfg.bg[0] + g1 * cfg.bg[1] + g2 * cfg.bg[2]);
    float S0 = 0.f, S1 = 0.f, S2 = 0.f, SD = 0.f;   // sum of w c and w z behind

    // entries each row needs: up to the last one any of its pixels composited
    const uint32_t rmax = row_max(my_last);
    const int rl0 = (int)__builtin_amdgcn_readlane(rmax, 0);
    const int rl1 = (int)__builtin_amdgcn_readlane(rmax, 16);
    const int rl2 = (int)__builtin_amdgcn_readlane(rmax, 32);
    const int rl3 = (int)__builtin_amdgcn_readlane(rmax, 48);
    if (tid == 0) s_max = 0u;
    __syncthreads();
    if (lane == 0) atomicMax(&s_max, (uint32_t)max(max(rl0, rl1), max(rl2, rl3)));
    __syncthreads();
    const uint32_t jmax = s_max;   // entries any pixel of the tile needs

    constexpr int NB = BwdStage<WIN, WIDE>::kN;
    constexpr bool ALL = WIDE && SF;   // every entry is summed, in the slot of its thread
    // a batch's sums -> the triangles' accumulators, and zeros again
    auto flush = [&](int n, int b) {
        if constexpr (WIDE) {
            for (int f = tid; f < n * TS_G2D_STRIDE; f += kBlock) {
                const float x = S.acc[f];
                if (x != 0.f) {
                    S.acc[f] = 0.f;
                    unsafeAtomicAdd(g2d + (int64_t)S.tri[b][f / TS_G2D_STRIDE] * TS_G2D_STRIDE +
                                        f % TS_G2D_STRIDE, x);
                }
            }
        }
    };
    if constexpr (WIDE) {
        for (int f = tid; f < S.kSlots * TS_G2D_STRIDE; f += kBlock) S.acc[f] = 0.f;
        if (tid < 2) S.wide[tid] = 0u;
    }
    int par = 0;
    // entry to stage, loaded a batch ahead
    const uint32_t lo0 = jmax > (uint32_t)NB ? jmax - NB : 0u;
    uint32_t next = tid < (int)(jmax - lo0) ? vals[start + lo0 + tid] : 0u;
    for (uint32_t hi_ = jmax; hi_ > 0;) {
        const uint32_t lo_ = hi_ > (uint32_t)NB ? hi_ - NB : 0u;
        const int n = (int)(hi_ - lo_);
        __syncthreads();
        if constexpr (WIDE) flush((int)min(S.wide[par], (uint32_t)S.kSlots), par);
        par ^= 1;
        if (tid < n) {
            const uint32_t tri = next;
            if (blocks) {   // the forward's record of where the entry composited
                stage_copy(S, rec, tri, tx * kTile, ty * kTile);
                S.hit[tid] = blocks[start + lo_ + tid];
            } else {
                S.hit[tid] = (uint16_t)stage_rec(S, rec, tri, tx * kTile, ty * kTile);
            }
            if constexpr (WIDE) {
                if constexpr (ALL) {
                    S.tri[par][tid] = tri;
                    if (tid == 0) S.wide[par] = (uint32_t)n;
                } else if (__popc(S.hit[tid]) >= kWideBlocks) {
                    const uint32_t slot = atomicAdd(&S.wide[par], 1u);
                    if (slot < (uint32_t)S.kSlots) {
                        S.tri[par][slot] = tri;
                        S.zt[tid].y = kWideTri + slot;
                    }
                }
            }
        }
        {
            const uint32_t lo1 = lo_ > (uint32_t)NB ? lo_ - NB : 0u;
            next = tid < (int)(lo_ - lo1) ? vals[start + lo1 + tid] : 0u;
        }
        __syncthreads();
        if constexpr (WIDE) {
            if (tid == 0) S.wide[par ^ 1] = 0u;   // its batch was written before the barrier
        }
        // entries of this batch each row needs (before its last composited one)
        const Lens L = build_lists(S, n, P.w, lane, rl0 - (int)lo_, rl1 - (int)lo_,
                                   rl2 - (int)lo_, rl3 - (int)lo_);
        // back to front along each row's list; positions are bytes from the start
        // of the stage, and a row past its list's front reads bytes before it
        // that it does not use
        const uint8_t* const bytes = reinterpret_cast<const uint8_t*>(&S);
        const int front = (int)(&S.list[4 * P.w + P.g][0] - bytes);
        int at = front + per_row(P.g, L.n0, L.n1, L.n2, L.n3) - 1;
        int jn = bytes[at];   // next entry (read one step ahead)
        asm volatile("" : "+v"(jn));   // else kept as a byte and widened every step
        const int lim = (int)my_last - (int)lo_;   // entries of the batch the pixel needs
        for (;;) {
            // lane masks are scalars, as in the forward
            const uint64_t act = ballot64(at >= front);
            if (act == 0ull) break;
            const int jc = lanes(act) ? jn : 0;   // idle lanes read slot 0 (always staged)
            jn = bytes[--at];
            const TriRecord r = read_rec(S, jc);
            const uint32_t tri = S.zt[jc].y;
            // the loads stay ahead of the arithmetic and of the branch below, so a
            // step waits for LDS once
            asm volatile("" ::: "memory");
            const int dx = P.px - r.ax, dy = P.py - r.ay;   // anchor form of the coefficients
            Frag f;
            const bool in = frag_alpha<WIN>(r, dxt, dyt, cfg.alpha_max, f);
            uint64_t contribs;
            float Ti;
            if constexpr (SF) {
                contribs = act & ballot64(fcur >= flo) & ballot64(fe == lo_ + (uint32_t)jc);
                if (lanes(contribs)) {
                    f.a = fa;
                    Ti = fTb;
                    --fcur;
                    if (fcur >= flo) {
                        fe = fs.entry[fcur];
                        fa = fs.alpha[fcur];
                        fTb = fs.T[fcur];
                    } else {
                        fe = 0xffffffffu;
                    }
                }
            } else {
                // my_last is 0 outside the image
                contribs = act & ballot64(jc < lim) & ballot64(in) &
                           ballot64(f.a >= cfg.alpha_min);
            }
            if (contribs == 0ull) continue;

            const bool contrib = lanes(contribs);
            const float rom = __builtin_amdgcn_rcpf(1.f - f.a);
            if constexpr (!SF) Ti = T * rom;   // transmittance before this fragment
            // selected, not a product with a zero alpha: behind an alpha of one
            // (T_min = 0) T is NaN, and lanes that composite nothing add zero
            const float wgt = contrib ? f.a * Ti : 0.f;
            if constexpr (!SF) T = contrib ? Ti : T;
            float v[16];
            v[11] = g0 * wgt;
            v[12] = g1 * wgt;
            v[13] = g2 * wgt;
            v[14] = gD * wgt;
            v[15] = 0.f;
            const float ga = g0 * (r.rgb[0] * Ti - S0 * rom) + g1 * (r.rgb[1] * Ti - S1 * rom) +
                             g2 * (r.rgb[2] * Ti - S2 * rom) + gD * (r.z * Ti - SD * rom) +
                             gT * Tf * rom;
            S0 = fmaf(wgt, r.rgb[0], S0);
            S1 = fmaf(wgt, r.rgb[1], S1);
            S2 = fmaf(wgt, r.rgb[2], S2);
            SD = fmaf(wgt, r.z, SD);
            const bool open = lanes(contribs & ballot64(f.oI <= cfg.alpha_max));   // not clamped
            const float gI = ga * r.o;
            v[9] = open ? ga * f.I : 0.f;                                  // dL/do
            if constexpr (WIN == TS_WINDOW_LSE) {
                // u = phi_lse / phi_lse(s): dphi_lse/dd_k = -w_k (softmax weight),
                // du/dr = u / phi_lse(s) (phi_lse(s) = ln 3 - r) into slot 15
                v[10] = open ? gI * f.I * (f.lg * 0.69314718055994531f) : 0.f;  // I ln u
                const float gu = open ? gI * r.sigma * f.I * __builtin_amdgcn_rcpf(f.u) : 0.f;
                const float rp = __builtin_amdgcn_rcpf(r.phis);
                const float gphi = gu * rp;
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    const float gd = -f.w[q] * gphi;
                    v[q] = gd * (float)dx;
                    v[3 + q] = gd * (float)dy;
                    v[6 + q] = gd;
                }
                v[15] = gu * f.u * rp;
            } else {
                float gu;
                if constexpr (WIN == TS_WINDOW_SIGMOID) {
                    // I = sigmoid(d / sigma): dI/dd = I (1 - I) / sigma,
                    // dI/dsigma = -I (1 - I) d / sigma^2
                    const float rs = __builtin_amdgcn_rcpf(r.sigma);
                    const float dI = f.I * f.Ic * rs;
                    v[10] = open ? -gI * dI * f.u * rs : 0.f;
                    gu = open ? gI * dI : 0.f;
                } else {
                    // computed for all lanes and selected: no branch in the step
                    const float vs = gI * f.I * (f.lg * 0.69314718055994531f);  // I ln u
                    const float vu = gI * r.sigma * f.I * __builtin_amdgcn_rcpf(f.u);
                    v[10] = open ? vs : 0.f;
                    gu = open ? vu : 0.f;
                }
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    const float gk = f.k == q ? gu : 0.f;
                    v[q] = gk * (float)dx;
                    v[3 + q] = gk * (float)dy;
                    v[6 + q] = gk;
                }
            }
            const float tot = row_reduce16(v, P.i);
            // slot 15 carries dL/dr for the LogSumExp window only
            constexpr uint64_t slots =
                WIN == TS_WINDOW_LSE ? ~0ull : 0x7fff7fff7fff7fffull;
            if (lanes(act & slots & ballot64(tot != 0.f))) {
                if (ALL || (WIDE && tri >= kWideTri)) {
                    if constexpr (WIDE) {
                        const uint32_t slot = ALL ? (uint32_t)jc : tri - kWideTri;
                        unsafeAtomicAdd(&S.acc[slot * TS_G2D_STRIDE + P.i], tot);
                    }
                } else {
                    unsafeAtomicAdd(g2d + (int64_t)tri * TS_G2D_STRIDE + P.i, tot);
                }
            }
        }
        hi_ = lo_;
    }
    if constexpr (WIDE) {
        __syncthreads();
        flush((int)min(S.wide[par], (uint32_t)S.kSlots), par);
    }
}

void launch_raster_forward(const void* rec, const uint32_t* vals, const uint32_t* ranges,
                           const uint32_t* order, const Cam& cam, const Cfg& cfg, int tiles_x,
                           int num_tiles, float* rgb, float* alpha, float* depth, float* T_final,
                           uint32_t* last, uint16_t* blocks, float* max_weight, uint32_t* pixels,
                           hipStream_t stream)
{
    const TriRecord* r = reinterpret_cast<const TriRecord*>(rec);
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(num_tiles), dim3(kBlock), 0, stream, r, vals, ranges, order,
                           cam, cfg, tiles_x, num_tiles, rgb, alpha, depth, T_final, last, blocks,
                           max_weight, pixels);
    };
    const bool st = max_weight != nullptr;
    switch (cfg.window) {
    case TS_WINDOW_SIGMOID:
        st ? go(k_raster_fwd<TS_WINDOW_SIGMOID, true>) : go(k_raster_fwd<TS_WINDOW_SIGMOID, false>);
        break;
    case TS_WINDOW_LSE:
        st ? go(k_raster_fwd<TS_WINDOW_LSE, true>) : go(k_raster_fwd<TS_WINDOW_LSE, false>);
        break;
    default:
        st ? go(k_raster_fwd<TS_WINDOW_PAPER, true>) : go(k_raster_fwd<TS_WINDOW_PAPER, false>);
        break;
    }
}

__global__ __launch_bounds__(256) void k_prune_views(uint32_t* __restrict__ pixels,
                                                     uint32_t* __restrict__ views, int64_t N)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N) return;
    views[i] += pixels[i] > 1u ? 1u : 0u;
    pixels[i] = 0u;
}

void launch_prune_views(uint32_t* pixels, uint32_t* views, int64_t N, hipStream_t stream)
{
    if (N > 0)
        hipLaunchKernelGGL(k_prune_views, dim3((unsigned)((N + 255) / 256)), dim3(256), 0, stream,
                           pixels, views, N);
}

void launch_raster_forward_views(const void* rec, const uint32_t* vals, const uint32_t* ranges,
                                 const uint32_t* order, const ts_view* views,
                                 const uint32_t* ctl, const Cfg& cfg, uint32_t max_tiles,
                                 float* rgb, float* alpha, float* depth, hipStream_t stream)
{
    const TriRecord* r = reinterpret_cast<const TriRecord*>(rec);
    const unsigned groups = std::min<uint32_t>(max_tiles, kViewGroups);
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(groups), dim3(kBlock), 0, stream, r, vals, ranges,
                           order, views, ctl, cfg, rgb, alpha, depth);
    };
    switch (cfg.window) {
    case TS_WINDOW_SIGMOID: go(k_raster_fwd_views<TS_WINDOW_SIGMOID>); break;
    case TS_WINDOW_LSE: go(k_raster_fwd_views<TS_WINDOW_LSE>); break;
    default: go(k_raster_fwd_views<TS_WINDOW_PAPER>); break;
    }
}

void launch_raster_backward(const void* rec, const uint32_t* vals, const uint32_t* ranges,
                            const uint32_t* order, const Cam& cam, const Cfg& cfg, int tiles_x,
                            int num_tiles, const float* dL_drgb, const float* dL_dalpha,
                            const float* dL_ddepth, const float* T_final,
                            const uint32_t* last, const uint16_t* blocks, float* g2d,
                            hipStream_t stream, const FragStore* fs)
{
    const TriRecord* r = reinterpret_cast<const TriRecord*>(rec);
    const FragStore none{};
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(num_tiles), dim3(kBlock), 0, stream, r, vals, ranges, order,
                           cam, cfg, tiles_x, num_tiles, dL_drgb, dL_dalpha, dL_ddepth, T_final,
                           last, blocks, g2d, fs ? *fs : none);
    };
    if (fs) {
        switch (cfg.window) {
        case TS_WINDOW_SIGMOID: go(k_raster_bwd<TS_WINDOW_SIGMOID, true, true>); break;
        case TS_WINDOW_LSE: go(k_raster_bwd<TS_WINDOW_LSE, true>); break;
        default: go(k_raster_bwd<TS_WINDOW_PAPER, true>); break;
        }
        return;
    }
    const bool wide =
        num_tiles >= (cfg.window == TS_WINDOW_SIGMOID ? kWideImageSigmoid : kWideImage);
    switch (cfg.window) {
    case TS_WINDOW_SIGMOID:
        wide ? go(k_raster_bwd<TS_WINDOW_SIGMOID, false, true>)
             : go(k_raster_bwd<TS_WINDOW_SIGMOID>);
        break;
    case TS_WINDOW_LSE:
        wide ? go(k_raster_bwd<TS_WINDOW_LSE, false, true>) : go(k_raster_bwd<TS_WINDOW_LSE>);
        break;
    default:
        wide ? go(k_raster_bwd<TS_WINDOW_PAPER, false, true>) : go(k_raster_bwd<TS_WINDOW_PAPER>);
        break;
    }
}

void launch_raster_forward_fragments(const void* rec, const uint32_t* vals,
                                     const uint32_t* ranges, const uint32_t* order,
                                     const Cam& cam, const Cfg& cfg, int tiles_x, int num_tiles,
                                     float* rgb, float* alpha, float* depth, float* T_final,
                                     uint32_t* last, uint16_t* blocks, int mode,
                                     const FragStore& fs, hipStream_t stream)
{
    const TriRecord* r = reinterpret_cast<const TriRecord*>(rec);
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(num_tiles), dim3(kBlock), 0, stream, r, vals, ranges, order,
                           cam, cfg, tiles_x, num_tiles, rgb, alpha, depth, T_final, last, blocks,
                           fs);
    };
    const bool store = mode == 2;
    switch (cfg.window) {
    case TS_WINDOW_SIGMOID:
        store ? go(k_raster_fwd_frag<TS_WINDOW_SIGMOID, 2>) : go(k_raster_fwd_frag<TS_WINDOW_SIGMOID, 1>);
        break;
    case TS_WINDOW_LSE:
        store ? go(k_raster_fwd_frag<TS_WINDOW_LSE, 2>) : go(k_raster_fwd_frag<TS_WINDOW_LSE, 1>);
        break;
    default:
        store ? go(k_raster_fwd_frag<TS_WINDOW_PAPER, 2>) : go(k_raster_fwd_frag<TS_WINDOW_PAPER, 1>);
        break;
    }
}

}  // namespace ts
