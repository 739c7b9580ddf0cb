// Section 5's image cost (arXiv:2203.03732): every vector divided by its sum,
// half the L1 distance of the normalised vectors, rounded by eq. (1).
//
// The definition takes |x - y| and its running sum in binary32 in pixel order:
// two vector instructions per pixel and pair. Here the normalised vectors are
// also rounded to 16-bit integers (the largest pixel of all becomes 65,535)
// and the distance of a pair is first taken on those, two pixels to an
// instruction and exactly in 32 bits. With the residuals of the rounding
// summed per vector, and the definition's own rounding errors bounded by the
// number of its nonzero terms, the integer distance brackets the definition's;
// a pair whose bracket holds no rounding boundary of eq. (1) has its k, and
// the others (a few in ten thousand, and the pairs without a common pixel when
// 1 / eps is a whole number, whose cost is 1 up to rounding) are listed and
// settled with the definition itself. Pixels that are zero in every vector add
// exactly nothing and are left out of both. The result equals the definition
// bit for bit.
#include "cost_common.h"
#include "internal.h"

#include <algorithm>
#include <float.h>

namespace prot {
namespace {

constexpr int kNormFloats = 12288;   // coordinates staged by a block
constexpr int kQuantVecs = 64;       // vectors per block of the rounding pass
constexpr int kQuantWords = 32;      // words (two pixels each) per step of it
constexpr int kSadWords = 16;        // words staged per step
constexpr int kSadList = 2048;       // unplaced pairs a block can list
constexpr int kSettleThreads = 512;
constexpr int kSettlePixels = 16;    // pixels staged per step
constexpr int kSettleStride = kSettlePixels + 4;
constexpr int kSettleEach = 4;       // pairs per thread and pass

// Each vector divided by its sum (binary32, the sum taken in coordinate order
// by one lane). kNormFloats coordinates of a block's vectors are staged in
// LDS. Entries must be finite and nonnegative with a positive finite sum (err
// bit 1 otherwise). Block 0 of X also records the cost scale 2 (the L1
// distance of two such vectors is at most 2) and K. With a rounding pass to
// follow, the pixels that are nonzero somewhere and the largest value are
// collected. Blocks [0, blocks_x) take X, the rest Y.
__global__ void __launch_bounds__(256) l1_normalize_kernel(PointsJob j, int blocks_x, int64_t nx,
                                                           int64_t ny)
{
    __shared__ float v[kNormFloats];
    __shared__ float sums[64];
    __shared__ uint32_t seen[kNormFloats / 32];  // pixels nonzero in this block's vectors
    __shared__ float red[4];
    __shared__ int bad;
    const bool is_y = (int)blockIdx.x >= blocks_x;
    const float *src = is_y ? j.Y : j.X;
    float *dst = is_y ? j.l1_y : j.l1_x;
    const int64_t n = is_y ? ny : nx;
    const int d = j.d;
    const int per = min(64, kNormFloats / d);
    const int64_t first = (int64_t)(is_y ? blockIdx.x - blocks_x : blockIdx.x) * per;
    if (first >= n) return;
    const int cnt = (int)min<int64_t>(per, n - first);
    if (threadIdx.x == 0) bad = 0;
    for (int i = threadIdx.x; i < (d + 31) / 32; i += blockDim.x) seen[i] = 0u;
    __syncthreads();
#pragma unroll 8
    for (int i = threadIdx.x; i < cnt * d; i += blockDim.x) {
        const float x = src[first * d + i];
        if (!(x >= 0.0f && x <= FLT_MAX)) bad = 1;
        v[i] = x;
    }
    __syncthreads();
    if ((int)threadIdx.x < cnt) {
        float t = 0.0f;
#pragma unroll 16
        for (int q = 0; q < d; ++q) t = __fadd_rn(t, v[threadIdx.x * d + q]);
        if (!(t > 0.0f && t <= FLT_MAX)) bad = 1;
        sums[threadIdx.x] = t;
    }
    __syncthreads();
    float mx = 0.0f;
    for (int i = threadIdx.x; i < cnt * d; i += blockDim.x) {
        const int b = i / d;
        const float x = __fdiv_rn(v[i], sums[b]);
        dst[first * d + i] = x;
        mx = fmaxf(mx, x);
        if (j.l1.used && x != 0.0f) {
            const int q = i - b * d;
            if (!((seen[q >> 5] >> (q & 31)) & 1u)) atomicOr(&seen[q >> 5], 1u << (q & 31));
        }
    }
    if (j.l1.used) {
        __syncthreads();
        for (int q = threadIdx.x; q < d; q += blockDim.x)
            if ((seen[q >> 5] >> (q & 31)) & 1u) j.l1.used[q] = 1u;
        for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = mx;
        __syncthreads();
        if (threadIdx.x == 0)
            __hip_atomic_fetch_max(&j.l1.meta[0],
                                   __float_as_uint(fmaxf(fmaxf(red[0], red[1]),
                                                         fmaxf(red[2], red[3]))),
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (threadIdx.x == 0) {
        if (bad) __hip_atomic_fetch_or(j.err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (blockIdx.x == 0) {
            j.m[0] = 2.0f;
            if (j.kmax_out) *j.kmax_out = (int32_t)floor(1.0 / j.eps);
        }
    }
}

__global__ void l1_reset_kernel(L1Aux a, int d, int64_t tiles, int64_t nx, int64_t ny)
{
    const int64_t i0 = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    for (int64_t i = i0; i < d; i += (int64_t)gridDim.x * blockDim.x) a.used[i] = 0u;
    for (int64_t i = i0; i < nx; i += (int64_t)gridDim.x * blockDim.x) a.ex[i] = 0.0f;
    for (int64_t i = i0; i < ny; i += (int64_t)gridDim.x * blockDim.x) a.ey[i] = 0.0f;
    for (int64_t i = i0; i < tiles; i += (int64_t)gridDim.x * blockDim.x) a.count[i] = 0u;
    if (i0 == 0) a.meta[0] = a.meta[1] = 0u;
}

// 65,535 / (largest normalised value), and its use on a value.
__device__ inline float l1_scale(const L1Aux &a)
{
    return 65535.0f / __uint_as_float(a.meta[0]);
}
__device__ inline uint32_t l1_round(float x, float scale)
{
    return (uint32_t)fminf(rintf(__fmul_rn(x, scale)), 65535.0f);
}

// The indices of the used pixels in ascending order into idx (LDS); returns
// their number. Whole block of 256.
__device__ int used_pixels(const L1Aux &a, int d, uint16_t *idx, int *cnt)
{
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, waves = (int)blockDim.x >> 6;
    int base = 0;
    for (int q0 = 0; q0 < d; q0 += (int)blockDim.x) {
        const bool u = q0 + tid < d && a.used[q0 + tid] != 0u;
        const unsigned long long bal = __ballot(u);
        if (lane == 0) cnt[wv] = __popcll(bal);
        __syncthreads();
        int before = base, total = base;
        for (int w = 0; w < waves; ++w) {
            if (w < wv) before += cnt[w];
            total += cnt[w];
        }
        if (u) idx[before + __popcll(bal & ((1ull << lane) - 1ull))] = (uint16_t)(q0 + tid);
        base = total;
        __syncthreads();
    }
    return base;
}

// The rounded vectors, word-major (word w of vector v at q[w * ldq + v], two
// used pixels a word, zero words up to a whole step of the pair kernel), and
// per vector a bound on how far it can move a pair's distance: the residuals of
// its rounding, and 2.01 x 2^-24 per nonzero pixel for the definition's own
// rounding (each term and each addition is rounded once, the sum is at most 2
// up to rounding, and adding zero is exact). Blocks [0, blocks_x) take X; a
// block does kQuantVecs vectors and, by grid.y, kQuantWords words of them.
__global__ void __launch_bounds__(256) l1_quantize_kernel(PointsJob j, int blocks_x, int64_t nx,
                                                          int64_t ny)
{
    __shared__ uint16_t idx[kNormFloats];
    __shared__ uint32_t tile[kQuantWords][kQuantVecs + 1];
    __shared__ int cnt[4];
    const L1Aux &A = j.l1;
    const bool is_y = (int)blockIdx.x >= blocks_x;
    const float *src = is_y ? j.l1_y : j.l1_x;
    uint32_t *q = is_y ? A.qy : A.qx;
    float *bound = is_y ? A.ey : A.ex;
    const int64_t ldq = is_y ? A.ldy : A.ldx, n = is_y ? ny : nx;
    const int64_t v0 = (int64_t)(is_y ? blockIdx.x - blocks_x : blockIdx.x) * kQuantVecs;
    if (v0 >= n) return;
    const int d = j.d, tid = threadIdx.x;
    const int used = used_pixels(A, d, idx, cnt);
    const int words = ((used + 1) / 2 + kSadWords - 1) / kSadWords * kSadWords;
    const int w0 = (int)blockIdx.y * kQuantWords;
    if (w0 >= words) return;
    if (blockIdx.x == 0 && blockIdx.y == 0 && tid == 0) A.meta[1] = (uint32_t)used;
    const float scale = l1_scale(A);
    const float inv = __fdiv_rn(1.0f, scale);
#pragma unroll
    for (int m = 0; m < kQuantVecs * kQuantWords / 256; ++m) {
        const int vec = (m * 256 + tid) / kQuantWords, w = tid % kQuantWords;
        const bool in = v0 + vec < n;
        float e = 0.0f;
        uint32_t word = 0u;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int p = 2 * (w0 + w) + h;
            const float x = in && p < used ? src[(v0 + vec) * d + idx[p]] : 0.0f;
            const uint32_t r = l1_round(x, scale);
            word |= r << (16 * h);
            // (2^-22 x covers the rounding of scale, inv and this product)
            e += fabsf(x - (float)r * inv) + x * 2.4e-7f + (x != 0.0f ? 1.2e-7f : 0.0f);
        }
        tile[w][vec] = word;
        for (int off = kQuantWords / 2; off > 0; off >>= 1) e += __shfl_xor(e, off);
        // (1 + 2^-10 covers the rounding of these sums)
        if (w == 0 && in) unsafeAtomicAdd(&bound[v0 + vec], e * 1.001f);
    }
    __syncthreads();
#pragma unroll
    for (int m = 0; m < kQuantVecs * kQuantWords / 256; ++m) {
        const int w = (m * 256 + tid) / kQuantVecs, vec = tid % kQuantVecs;
        if (w0 + w < words && v0 + vec < n) q[(int64_t)(w0 + w) * ldq + v0 + vec] = tile[w][vec];
    }
}

template <class T>
__device__ inline void put_k(T *k, int64_t at, int g)
{
    k[at] = (T)((sizeof(T) == 1 && g > 255) ? 255 : g);
}

// 64 G x 64 G pairs per block, 4 G x 4 G per thread (rows and columns in G
// groups of 4, so that 16 lanes read 256 consecutive bytes of a staged word),
// kSadWords words staged per step in two buffers. v_sad_u16 adds two |x - y| to a
// 32-bit sum. G = 2, and G = 1 where that leaves too few blocks for the chip
// (launch_l1_pairs). With G = 1 the next step's words wait in registers while this
// one's are added; with G = 2 the compiler keeps those 16 words in scratch (80
// bytes a lane): a step's loads are waited for, and stored there, before its sums.
// Bound: with G = 2 64 vector instructions per word and thread against 4 LDS reads,
// and those loads. 10,000 x 10,000 pairs of 784 pixels, 529 of them used: 0.95 ms,
// of which the issue of the instructions takes 0.71; 3.09 ms by the definition for
// all pairs.
template <class T, int G>
__global__ void __launch_bounds__(256) l1_sad_kernel(PointsJob j)
{
    constexpr int kSadTile = 64 * G;
    __shared__ __align__(16) uint32_t xs[2][kSadWords][kSadTile];
    __shared__ __align__(16) uint32_t ys[2][kSadWords][kSadTile];
    __shared__ uint16_t list[kSadList];
    __shared__ uint32_t n_list, s_base;
    const L1Aux &A = j.l1;
    const int64_t n = j.n_single, na = j.na_single ? j.na_single : j.n_single;
    const int64_t b0 = (int64_t)blockIdx.y * kSadTile, a0 = (int64_t)blockIdx.x * kSadTile;
    const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
    T *const k = reinterpret_cast<T *>(j.k);
    const int64_t ldk = j.ldk_single;
    if (tid == 0) n_list = 0u;
    uint32_t acc[4 * G][4 * G];
#pragma unroll
    for (int i = 0; i < 4 * G; ++i)
#pragma unroll
        for (int c = 0; c < 4 * G; ++c) acc[i][c] = 0u;
    if (a0 < na) {
        const int steps = (((int)A.meta[1] + 1) / 2 + kSadWords - 1) / kSadWords;
        // each thread stages G 16-byte pieces of either side per step
        constexpr int kRow = kSadTile / 4, kPer = 256 / kRow;  // pieces a word, words a sweep
        const int w = tid / kRow, v = (tid % kRow) * 4;
        const uint32_t *gx = A.qx + (int64_t)w * A.ldx + b0 + v;
        const uint32_t *gy = A.qy + (int64_t)w * A.ldy + a0 + v;
        uint4 px[G], py[G];
        auto fetch = [&](int s) {
#pragma unroll
            for (int h = 0; h < G; ++h) {
                px[h] = *reinterpret_cast<const uint4 *>(gx + ((int64_t)s * kSadWords + kPer * h) * A.ldx);
                py[h] = *reinterpret_cast<const uint4 *>(gy + ((int64_t)s * kSadWords + kPer * h) * A.ldy);
            }
        };
        if (steps > 0) fetch(0);
        for (int s = 0; s < steps; ++s) {
            const int buf = s & 1;
#pragma unroll
            for (int h = 0; h < G; ++h) {
                *reinterpret_cast<uint4 *>(&xs[buf][w + kPer * h][v]) = px[h];
                *reinterpret_cast<uint4 *>(&ys[buf][w + kPer * h][v]) = py[h];
            }
            __syncthreads();
            if (s + 1 < steps) fetch(s + 1);
#pragma unroll
            for (int u = 0; u < kSadWords; ++u) {
                uint32_t xr[4 * G], yc[4 * G];
#pragma unroll
                for (int h = 0; h < G; ++h) {
                    const uint4 x = *reinterpret_cast<const uint4 *>(&xs[buf][u][64 * h + ty * 4]);
                    const uint4 y = *reinterpret_cast<const uint4 *>(&ys[buf][u][64 * h + tx * 4]);
                    xr[4 * h] = x.x, xr[4 * h + 1] = x.y, xr[4 * h + 2] = x.z, xr[4 * h + 3] = x.w;
                    yc[4 * h] = y.x, yc[4 * h + 1] = y.y, yc[4 * h + 2] = y.z, yc[4 * h + 3] = y.w;
                }
#pragma unroll
                for (int i = 0; i < 4 * G; ++i)
#pragma unroll
                    for (int c = 0; c < 4 * G; ++c)
                        acc[i][c] = __builtin_amdgcn_sad_u16(xr[i], yc[c], acc[i][c]);
            }
        }
    }
    __syncthreads();
    // v = distance / (2 eps) within the margin of the definition's; placed
    // when no whole number and not the clamp at cost 1 lies within it
    const float scale = l1_scale(A);
    const int32_t K = (int32_t)floor(1.0 / j.eps);
    const float to_v = (float)(0.5 / ((double)scale * j.eps));
    const float half_eps = (float)(0.505 / j.eps);  // margin per unit of the bounds, 1% up
    const float top = (float)(1.0 / j.eps), base_margin = classify_margin(K);
    float ey[4 * G];
#pragma unroll
    for (int c = 0; c < 4 * G; ++c) {
        const int64_t a = a0 + (c & 3) + tx * 4 + (c >> 2) * 64;
        ey[c] = a < na ? A.ey[a] : 0.0f;
    }
#pragma unroll
    for (int i = 0; i < 4 * G; ++i) {
        const int r = (i & 3) + ty * 4 + (i >> 2) * 64;
        if (b0 + r >= n) continue;
        const float ex = A.ex[b0 + r];
#pragma unroll
        for (int h = 0; h < G; ++h) {
            const int c0 = tx * 4 + h * 64;
            if (a0 + c0 >= ldk) continue;
            int g[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const float vv = __fmul_rn((float)acc[i][4 * h + c], to_v);
                const float margin = (ex + ey[4 * h + c]) * half_eps + base_margin;
                const float f = __builtin_amdgcn_fractf(vv);
                g[c] = (int)vv;
                // (below the first boundary there is none to cross downwards)
                const bool placed = f + margin < 1.0f && (f > margin || g[c] == 0) &&
                                    vv + margin < top;
                if (a0 + c0 + c >= na) {
                    g[c] = 0x7FFF;
                } else if (!placed) {
                    const uint32_t at = atomicAdd(&n_list, 1u);
                    if (at < (uint32_t)kSadList) list[at] = (uint16_t)(r * kSadTile + c0 + c);
                }
            }
            if constexpr (sizeof(T) == 1) {
                uint32_t q[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) q[c] = (uint32_t)g[c] > 255u ? 255u : (uint32_t)g[c];
                *reinterpret_cast<uint32_t *>(k + (b0 + r) * ldk + a0 + c0) =
                    q[0] | (q[1] << 8) | (q[2] << 16) | (q[3] << 24);
            } else {
                uint2 q;
                q.x = (uint32_t)(uint16_t)g[0] | ((uint32_t)(uint16_t)g[1] << 16);
                q.y = (uint32_t)(uint16_t)g[2] | ((uint32_t)(uint16_t)g[3] << 16);
                *reinterpret_cast<uint2 *>(k + (b0 + r) * ldk + a0 + c0) = q;
            }
        }
    }
    __syncthreads();
    // the unplaced pairs to the list of the settling tile this block is part
    // of; a full list is left with a count above its capacity
    const uint32_t cnt = n_list;
    if (cnt == 0u) return;
    const int64_t tile = (b0 / kL1SettleTile) * A.tiles_x + a0 / kL1SettleTile;
    if (tid == 0)
        s_base = __hip_atomic_fetch_add(&A.count[tile],
                                        cnt > (uint32_t)kSadList ? (uint32_t)kL1ListCap + 1u : cnt,
                                        __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    const uint32_t base = s_base;
    if (cnt > (uint32_t)kSadList || base > (uint32_t)kL1ListCap || base + cnt > (uint32_t)kL1ListCap)
        return;
    const uint32_t r0 = (uint32_t)(b0 % kL1SettleTile), c0 = (uint32_t)(a0 % kL1SettleTile);
    for (uint32_t i = tid; i < cnt; i += 256) {
        const uint32_t e = list[i];
        A.list[tile * kL1ListCap + base + i] =
            (r0 + e / kSadTile) * kL1SettleTile + c0 + e % kSadTile;
    }
}

// The listed pairs of a kL1SettleTile x kL1SettleTile tile by the definition
// (a tile whose list overflowed is left to the next pass): the rows' and columns'
// used pixels staged kSettlePixels at a time, kSettleEach pairs per thread and
// pass, each accumulated in pixel order. Large tiles, because a listed pair
// needs its whole row and column: n^2 / tile rows are read in all.
// Bound: LDS reads of 8 bytes per pair and pixel.
template <class T>
__global__ void __launch_bounds__(kSettleThreads) l1_settle_kernel(PointsJob j)
{
    extern __shared__ __align__(16) float lds[];
    float *xs = lds, *ys = lds + kL1SettleTile * kSettleStride;
    uint16_t *idx = reinterpret_cast<uint16_t *>(lds + 2 * kL1SettleTile * kSettleStride);
    __shared__ int wcnt[kSettleThreads / 64];
    const L1Aux &A = j.l1;
    const int64_t tile = (int64_t)blockIdx.y * A.tiles_x + blockIdx.x;
    const uint32_t listed = A.count[tile];
    if (listed == 0u || listed > (uint32_t)kL1ListCap) return;
    const int tid = threadIdx.x;
    const int64_t n = j.n_single, na = j.na_single ? j.na_single : j.n_single;
    const int64_t b0 = (int64_t)blockIdx.y * kL1SettleTile, a0 = (int64_t)blockIdx.x * kL1SettleTile;
    const int rows = (int)min<int64_t>(kL1SettleTile, n - b0);
    const int cols = (int)min<int64_t>(kL1SettleTile, na - a0);
    if (cols <= 0) return;
    const int total = (int)listed;
    const int d = j.d;
    const int used = used_pixels(A, d, idx, wcnt);
    T *const k = reinterpret_cast<T *>(j.k);
    for (int e0 = 0; e0 < total; e0 += kSettleThreads * kSettleEach) {
        int at[kSettleEach];
        float acc[kSettleEach];
#pragma unroll
        for (int u = 0; u < kSettleEach; ++u) {
            const int e = e0 + u * kSettleThreads + tid;
            at[u] = -1;
            acc[u] = 0.0f;
            if (e < total) at[u] = (int)A.list[tile * kL1ListCap + e];
        }
        // a thread stages pixel p of rows r0, r0 + kStep, ...; the next step's
        // values are on their way while this one's are added
        constexpr int kStep = kSettleThreads / kSettlePixels, kLoads = kL1SettleTile / kStep;
        const int p = tid % kSettlePixels, r0 = tid / kSettlePixels;
        float fx[kLoads], fy[kLoads];
        auto fetch = [&](int p0) {
            const int px = p0 + p < used ? (int)idx[p0 + p] : -1;
#pragma unroll
            for (int u = 0; u < kLoads; ++u) {
                const int r = r0 + u * kStep;
                fx[u] = px >= 0 && r < rows ? j.l1_x[(b0 + r) * d + px] : 0.0f;
                fy[u] = px >= 0 && r < cols ? j.l1_y[(a0 + r) * d + px] : 0.0f;
            }
        };
        fetch(0);
        for (int p0 = 0; p0 < used; p0 += kSettlePixels) {
            __syncthreads();
#pragma unroll
            for (int u = 0; u < kLoads; ++u) {
                xs[(r0 + u * kStep) * kSettleStride + p] = fx[u];
                ys[(r0 + u * kStep) * kSettleStride + p] = fy[u];
            }
            __syncthreads();
            if (p0 + kSettlePixels < used) fetch(p0 + kSettlePixels);
#pragma unroll
            for (int u = 0; u < kSettleEach; ++u) {
                if (at[u] < 0) continue;
                const float *x = xs + (at[u] / kL1SettleTile) * kSettleStride;
                const float *y = ys + (at[u] % kL1SettleTile) * kSettleStride;
                float s = acc[u];
#pragma unroll
                for (int q = 0; q < kSettlePixels; q += 4) {
                    const float4 xv = *reinterpret_cast<const float4 *>(x + q);
                    const float4 yv = *reinterpret_cast<const float4 *>(y + q);
                    s = __fadd_rn(s, fabsf(__fsub_rn(xv.x, yv.x)));
                    s = __fadd_rn(s, fabsf(__fsub_rn(xv.y, yv.y)));
                    s = __fadd_rn(s, fabsf(__fsub_rn(xv.z, yv.z)));
                    s = __fadd_rn(s, fabsf(__fsub_rn(xv.w, yv.w)));
                }
                acc[u] = s;
            }
        }
#pragma unroll
        for (int u = 0; u < kSettleEach; ++u) {
            if (at[u] < 0) continue;
            // half the L1 distance, clamped to 1, eq. (1) in binary64
            const int g = (int)floor(fmin((double)acc[u] * 0.5, 1.0) / j.eps);
            put_k(k, (b0 + at[u] / kL1SettleTile) * j.ldk_single + a0 + at[u] % kL1SettleTile, g);
        }
    }
}

template <class T, int G>
void launch_l1_sad(const PointsJob &j, int64_t n, int64_t ldk, hipStream_t s)
{
    hipLaunchKernelGGL((l1_sad_kernel<T, G>),
                       dim3((unsigned)((ldk + 64 * G - 1) / (64 * G)),
                            (unsigned)((n + 64 * G - 1) / (64 * G))),
                       dim3(256), 0, s, j);
}

template <class T>
hipError_t launch_l1_pairs(const PointsJob &j, int64_t n, int64_t ldk, hipStream_t s)
{
    const size_t lds = 2 * kL1SettleTile * kSettleStride * sizeof(float) +
                       kNormFloats * sizeof(uint16_t);
    const hipError_t e = hipFuncSetAttribute(
        (const void *)l1_settle_kernel<T>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    // 128 x 128 blocks reuse a staged word twice as often; below two of them a
    // CU the chip is filled better by four times as many of 64 x 64
    if (((ldk + 127) / 128) * ((n + 127) / 128) >= 512) launch_l1_sad<T, 2>(j, n, ldk, s);
    else launch_l1_sad<T, 1>(j, n, ldk, s);
    hipLaunchKernelGGL(l1_settle_kernel<T>,
                       dim3((unsigned)j.l1.tiles_x,
                            (unsigned)((n + kL1SettleTile - 1) / kL1SettleTile)),
                       dim3(kSettleThreads), lds, s, j);
    PointsJob jn = j;  // the definition reads the normalised vectors
    jn.X = j.l1_x;
    jn.Y = j.l1_y;
    return launch_points_tile_l1_overflow(
        jn, j.l1.tiles_x * ((n + kL1SettleTile - 1) / kL1SettleTile), s);
}

}  // namespace

int64_t l1_words(int32_t d) { return ((d + 1) / 2 + kSadWords - 1) / kSadWords * kSadWords; }

hipError_t launch_points_l1(const PointsJob &j, int64_t n_max, int64_t ldk_max, hipStream_t s)
{
    // one instance (the batched solver keeps the squared cost)
    const int64_t nb = j.n_single, na = j.na_single ? j.na_single : j.n_single;
    const bool screened = j.l1.used != nullptr;
    if (screened)
        hipLaunchKernelGGL(l1_reset_kernel, dim3(64), dim3(256), 0, s, j.l1, j.d,
                           j.l1.tiles_x * ((nb + kL1SettleTile - 1) / kL1SettleTile), nb, na);
    const int per = std::min(64, kNormFloats / j.d);
    const int64_t bx = (nb + per - 1) / per, by = (na + per - 1) / per;
    if (bx + by > 0)
        hipLaunchKernelGGL(l1_normalize_kernel, dim3((unsigned)(bx + by)), dim3(256), 0, s, j,
                           (int)bx, nb, na);
    if (!screened) {
        PointsJob jn = j;
        jn.X = j.l1_x;
        jn.Y = j.l1_y;
        return launch_points_tile_l1(jn, n_max, ldk_max, s);
    }
    const int64_t qx = (nb + kQuantVecs - 1) / kQuantVecs, qy = (na + kQuantVecs - 1) / kQuantVecs;
    hipLaunchKernelGGL(l1_quantize_kernel,
                       dim3((unsigned)(qx + qy),
                            (unsigned)((l1_words(j.d) + kQuantWords - 1) / kQuantWords)),
                       dim3(256), 0, s, j, (int)qx,
                       nb, na);
    return j.k8 ? launch_l1_pairs<uint8_t>(j, nb, ldk_max, s)
                : launch_l1_pairs<int16_t>(j, nb, ldk_max, s);
}

}  // namespace prot
