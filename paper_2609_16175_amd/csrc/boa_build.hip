// Index construction on the GPU: the entry point s (the medoid) and, when
// the caller passes no adjacency, the proximity graph itself.
//
// The paper builds a Vamana graph with JAG threshold pruning (Sec. II
// "Graph construction") and enters every search at the medoid s (Alg. 2).
// This library's builder follows the same pruning rule on a different
// candidate source: exact nearest neighbours instead of Vamana's
// incremental beam-search insertion.
//   1. medoid: the point nearest (float64) to the float64 centroid, ties to
//      the lowest id; the centroid is reduced in one fixed order;
//   2. candidates: the K = min(2R, 128, n - 1) nearest points of every
//      point by brute force, ordered by (distance, id), and for each
//      attribute level the nearest min(R / 2, 32, n - 1) among the points
//      within the point's attribute threshold, all from one pass over the
//      distances;
//   3. alpha-pruning (DiskANN's dominance rule, alpha = 1.2 on Euclidean
//      distances): a candidate v of u is dropped when a kept w has
//      alpha^2 d(w, v) <= d(u, v) on squared distances;
//   4. reverse edges: every kept edge u -> v proposes v -> u; each point's
//      forward and reverse neighbours are pruned again by the same rule to
//      R - 1 edges, leaving one free slot per row;
//   5. connectivity repair from s (host): a point that a breadth-first
//      search from s does not reach gets an in-edge from its nearest
//      reached candidate that still has a free slot.
// Distances here are this builder's own: float32 sums of squared float32
// differences in dimension order, exact int32 for uint8 vectors.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "boa_internal.h"

namespace boa {

static constexpr uint64_t BKEY_NONE = ~0ull;
static constexpr int KNN_LIST = 128;      // most candidates per point
static constexpr int KNN_LEVELS = 4;      // attribute levels
static constexpr int KNN_LEVEL_LIST = 32; // most candidates per point and level
static_assert(KNN_LIST <= 128 && KNN_LEVEL_LIST <= KNN_LIST, "prune_fwd_kernel sorts 128 keys");

__device__ __forceinline__ uint64_t bkey(float d, uint32_t id)
{
    return ((uint64_t)__float_as_uint(d) << 32) | id;
}

// ---------------------------------------------------------------------------
// pair distances (builder's own arithmetic)

// squared distance of two float32 rows, dimensions in order
__device__ __forceinline__ float pair_dist_f32(const float *x, const float *y, int d)
{
    const float4 *a = reinterpret_cast<const float4 *>(x);
    const float4 *b = reinterpret_cast<const float4 *>(y);
    float acc = 0.f;
    for (int c = 0; c < (d >> 2); ++c) {
        const float4 p = a[c], q = b[c];
        float t = p.x - q.x;
        acc = __builtin_fmaf(t, t, acc);
        t = p.y - q.y;
        acc = __builtin_fmaf(t, t, acc);
        t = p.z - q.z;
        acc = __builtin_fmaf(t, t, acc);
        t = p.w - q.w;
        acc = __builtin_fmaf(t, t, acc);
    }
    return acc;
}

// Whether scale * (that distance) <= bound. The partial sums never decrease
// (nor does their product with the scale, both rounded), so the wave stops
// once no lane's is within its bound; NaN compares false as in the full sum.
__device__ __forceinline__ bool pair_within_f32(const float *x, const float *y, int d, float scale, float bound)
{
    const float4 *a = reinterpret_cast<const float4 *>(x);
    const float4 *b = reinterpret_cast<const float4 *>(y);
    const int nch = d >> 2;
    float acc = 0.f;
    for (int c0 = 0; c0 < nch; c0 += 8) {
        float4 p[8], q[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {   // (past the row: its last chunk, not added)
            p[i] = a[min(c0 + i, nch - 1)];
            q[i] = b[min(c0 + i, nch - 1)];
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if (c0 + i >= nch) break;
            float t = p[i].x - q[i].x;
            acc = __builtin_fmaf(t, t, acc);
            t = p[i].y - q[i].y;
            acc = __builtin_fmaf(t, t, acc);
            t = p[i].z - q[i].z;
            acc = __builtin_fmaf(t, t, acc);
            t = p[i].w - q[i].w;
            acc = __builtin_fmaf(t, t, acc);
        }
        if (__ballot(scale * acc <= bound) == 0ull) return false;
    }
    return scale * acc <= bound;
}

// exact squared distance of two uint8 rows: |x|^2 + |y|^2 - 2 x.y in int32
__device__ __forceinline__ float pair_dist_u8(const uint8_t *x, const uint8_t *y, int d, uint32_t nx, uint32_t ny)
{
    const uint32_t *a = reinterpret_cast<const uint32_t *>(x);
    const uint32_t *b = reinterpret_cast<const uint32_t *>(y);
    uint32_t dot = 0;
    for (int c = 0; c < (d >> 2); ++c) dot = __builtin_amdgcn_udot4(a[c], b[c], dot, false);
    return (float)(int32_t)(nx + ny - 2u * dot);
}

struct BuildView {
    const void *vectors;
    const uint32_t *norms;   // uint8 vectors: |x|^2 per point (else null)
    int64_t n;
    int32_t d;
    int32_t u8;
    const float *D;          // all n x ld distances, or null
    int64_t ld;
};

__device__ __forceinline__ float dist_ids(const BuildView &v, uint32_t a, uint32_t b)
{
    if (v.D) return v.D[(size_t)a * v.ld + b];
    if (v.u8) {
        const uint8_t *X = reinterpret_cast<const uint8_t *>(v.vectors);
        return pair_dist_u8(X + (size_t)a * v.d, X + (size_t)b * v.d, v.d, v.norms[a], v.norms[b]);
    }
    const float *X = reinterpret_cast<const float *>(v.vectors);
    return pair_dist_f32(X + (size_t)a * v.d, X + (size_t)b * v.d, v.d);
}

// ---------------------------------------------------------------------------
// in-wave bitonic sort of N u64 keys held in LDS (ascending; N = 128 or 256)

__device__ __forceinline__ void wave_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int N>
__device__ void bitonic(uint64_t *a, int lane)
{
    for (int k = 2; k <= N; k <<= 1) {
        for (int j = k >> 1; j > 0; j >>= 1) {
            // N / 2 compare-exchanges per step, N / 128 per lane
#pragma unroll
            for (int h = 0; h < N / 128; ++h) {
                const int t = lane + 64 * h;                       // pair index
                const int i = ((t & ~(j - 1)) << 1) | (t & (j - 1)); // lower element
                const int p = i + j;
                const bool up = (i & k) == 0;
                const uint64_t x = a[i], y = a[p];
                if ((x > y) == up) {
                    a[i] = y;
                    a[p] = x;
                }
            }
            wave_fence();
        }
    }
}

// ---------------------------------------------------------------------------
// 1. medoid

struct CentroidArgs {
    BuildView v;
    double *partial;     // nblocks x d
    int64_t per_block;
};

// each block sums its contiguous range of points, dimension by dimension,
// in point order (float64)
__global__ void __launch_bounds__(256) centroid_partial_kernel(CentroidArgs a)
{
    const int64_t p0 = (int64_t)blockIdx.x * a.per_block;
    const int64_t p1 = p0 + a.per_block < a.v.n ? p0 + a.per_block : a.v.n;
    for (int j = threadIdx.x; j < a.v.d; j += blockDim.x) {
        double s = 0.0;
        if (a.v.u8) {
            const uint8_t *X = reinterpret_cast<const uint8_t *>(a.v.vectors);
            for (int64_t i = p0; i < p1; ++i) s += (double)X[(size_t)i * a.v.d + j];
        } else {
            const float *X = reinterpret_cast<const float *>(a.v.vectors);
            for (int64_t i = p0; i < p1; ++i) s += (double)X[(size_t)i * a.v.d + j];
        }
        a.partial[(size_t)blockIdx.x * a.v.d + j] = s;
    }
}

struct MedoidArgs {
    BuildView v;
    const double *centroid;  // d
    double *best_d;          // per block
    uint32_t *best_id;       // per block
};

// float64 distance of every point to the centroid; each block reports its
// nearest point (ties: lowest id)
__global__ void __launch_bounds__(256) medoid_partial_kernel(MedoidArgs a)
{
    __shared__ double sd[256];
    __shared__ uint32_t si[256];
    double bd = INFINITY;
    uint32_t bi = 0xFFFFFFFFu;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < a.v.n;
         i += (int64_t)gridDim.x * blockDim.x) {
        double s = 0.0;
        for (int j = 0; j < a.v.d; ++j) {
            const double x = a.v.u8 ? (double)reinterpret_cast<const uint8_t *>(a.v.vectors)[(size_t)i * a.v.d + j]
                                    : (double)reinterpret_cast<const float *>(a.v.vectors)[(size_t)i * a.v.d + j];
            const double t = x - a.centroid[j];
            s = fma(t, t, s);
        }
        if (s < bd || (s == bd && (uint32_t)i < bi)) {
            bd = s;
            bi = (uint32_t)i;
        }
    }
    sd[threadIdx.x] = bd;
    si[threadIdx.x] = bi;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) {
            const double od = sd[threadIdx.x + w];
            const uint32_t oi = si[threadIdx.x + w];
            if (od < sd[threadIdx.x] || (od == sd[threadIdx.x] && oi < si[threadIdx.x])) {
                sd[threadIdx.x] = od;
                si[threadIdx.x] = oi;
            }
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        a.best_d[blockIdx.x] = sd[0];
        a.best_id[blockIdx.x] = si[0];
    }
}

// |x|^2 of every uint8 point, and of the point shifted by -128 (for signed
// matrix instructions)
__global__ void norms_kernel(BuildView v, uint32_t *norms, int32_t *norms_shifted)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= v.n) return;
    const uint32_t *x = reinterpret_cast<const uint32_t *>(reinterpret_cast<const uint8_t *>(v.vectors) + (size_t)i * v.d);
    uint32_t s = 0;
    int32_t t = 0;
    for (int c = 0; c < (v.d >> 2); ++c) {
        s = __builtin_amdgcn_udot4(x[c], x[c], s, false);
        const int32_t y = (int32_t)(x[c] ^ 0x80808080u);
        t = __builtin_amdgcn_sdot4(y, y, t, false);
    }
    norms[i] = s;
    norms_shifted[i] = t;
}

// ---------------------------------------------------------------------------
// 2. exact nearest candidates of every point
//
// A tile of rows and columns at a time: its distances go to memory, and a wave
// per row then picks the nearest for every list in one sweep. One sweep per list, with the distances computed
// again for each and the rows' lists holding the compute units' LDS, took 5
// times 11.7 ms at n = 30,000, d = 96, five lists; see the kernels for theirs.

static constexpr int DT = 128;   // rows and columns of a distance tile
static constexpr int DK = 16;    // dimensions staged at once (float32)

// Distances of rows [r0, r0 + rows) to the points from cb on (as many as the
// grid's columns), float32, dimensions in order (the sums of pair_dist_f32). 128 x 128 tiles, 8 x 8 pairs per thread:
// 128 vector instructions for four LDS reads per dimension, so that it runs at
// the vector units' rate (a difference and a fused multiply-add per pair and
// dimension; matrix instructions would sum in another order).
//
// SYM: all pairs at once (r0 = cb = 0, rows = n); only the tiles on and above the
// diagonal are computed, and written at their mirrored place too (the two
// differences have the same square).
template <bool SYM>
__global__ void __launch_bounds__(256) dist_f32_kernel(const float *X, int64_t n, int d, int64_t r0, int64_t rows,
                                                       int64_t cb, int64_t ld, float *D)
{
    if (SYM && blockIdx.x < blockIdx.y) return;
    __shared__ __align__(16) float A[DK][DT + 4], B[DK][DT + 4];
    const int t = threadIdx.x, tr = t >> 4, tc = t & 15;
    const int64_t row0 = r0 + (int64_t)blockIdx.y * DT, col0 = cb + (int64_t)blockIdx.x * DT;
    float acc[8][8];
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[i][j] = 0.f;
    for (int k0 = 0; k0 < d; k0 += DK) {
        // 128 points x 16 dimensions of each side, two float4 per thread; zeros
        // past the row's dimensions (they add zero) and past the last point
        float4 x[2], y[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int e = t + 256 * h, p = e >> 2, k = k0 + 4 * (e & 3);
            const float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
            x[h] = k < d && row0 + p < n ? *reinterpret_cast<const float4 *>(X + (size_t)(row0 + p) * d + k) : z;
            y[h] = k < d && col0 + p < n ? *reinterpret_cast<const float4 *>(X + (size_t)(col0 + p) * d + k) : z;
        }
        __syncthreads();
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int e = t + 256 * h, p = e >> 2, k = 4 * (e & 3);
            A[k][p] = x[h].x;
            A[k + 1][p] = x[h].y;
            A[k + 2][p] = x[h].z;
            A[k + 3][p] = x[h].w;
            B[k][p] = y[h].x;
            B[k + 1][p] = y[h].y;
            B[k + 2][p] = y[h].z;
            B[k + 3][p] = y[h].w;
        }
        __syncthreads();
#pragma unroll 4
        for (int k = 0; k < DK; ++k) {
            const float4 a0 = *reinterpret_cast<const float4 *>(&A[k][4 * tr]);
            const float4 a1 = *reinterpret_cast<const float4 *>(&A[k][64 + 4 * tr]);
            const float4 b0 = *reinterpret_cast<const float4 *>(&B[k][4 * tc]);
            const float4 b1 = *reinterpret_cast<const float4 *>(&B[k][64 + 4 * tc]);
            const float a[8] = {a0.x, a0.y, a0.z, a0.w, a1.x, a1.y, a1.z, a1.w};
            const float b[8] = {b0.x, b0.y, b0.z, b0.w, b1.x, b1.y, b1.z, b1.w};
#pragma unroll
            for (int i = 0; i < 8; ++i)
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const float e = a[i] - b[j];
                    acc[i][j] = __builtin_fmaf(e, e, acc[i][j]);
                }
        }
    }
    // (ld is a multiple of the tile: columns past n are written and not read)
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int64_t r = (int64_t)blockIdx.y * DT + (i < 4 ? 4 * tr + i : 64 + 4 * tr + i - 4);
        if (r >= rows) continue;
        float *o = D + (size_t)r * ld + (col0 - cb);
        *reinterpret_cast<float4 *>(o + 4 * tc) = make_float4(acc[i][0], acc[i][1], acc[i][2], acc[i][3]);
        *reinterpret_cast<float4 *>(o + 64 + 4 * tc) = make_float4(acc[i][4], acc[i][5], acc[i][6], acc[i][7]);
    }
    if (SYM && blockIdx.x > blockIdx.y) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int64_t c = col0 + (j < 4 ? 4 * tc + j : 64 + 4 * tc + j - 4);
            if (c >= n) continue;
            float *o = D + (size_t)c * ld + row0;
            *reinterpret_cast<float4 *>(o + 4 * tr) = make_float4(acc[0][j], acc[1][j], acc[2][j], acc[3][j]);
            *reinterpret_cast<float4 *>(o + 64 + 4 * tr) = make_float4(acc[4][j], acc[5][j], acc[6][j], acc[7][j]);
        }
    }
}

typedef int32_t int4v __attribute__((ext_vector_type(4)));
typedef int32_t int16v __attribute__((ext_vector_type(16)));

// The same for uint8 points, exact: |x - y|^2 = |x'|^2 + |y'|^2 - 2 x'.y' of
// the points shifted by -128, whose products are matrix instructions on signed
// bytes (32 x 32 pairs, 32 dimensions each: 16 consecutive bytes of a row per
// lane, as they lie in memory). A wave computes 64 x 64 pairs, a block of four
// 128 x 128; the products are a twentieth of the time, the writes the rest.
__global__ void __launch_bounds__(256) dist_u8_kernel(const uint8_t *X, const int32_t *norms, int64_t n, int d,
                                                      int64_t r0, int64_t rows, int64_t cb, int64_t ld, float *D)
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int half = lane >> 5, l32 = lane & 31;
    const int64_t row0 = r0 + (int64_t)blockIdx.y * DT + 64 * (w >> 1);
    const int64_t col0 = cb + (int64_t)blockIdx.x * DT + 64 * (w & 1);
    int16v acc[2][2] = {};
    for (int k0 = 0; k0 < d; k0 += 32) {
        const int k = k0 + 16 * half;
        int4v a[2], b[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            // (a row past the last point: point 0, its pairs are not read; bytes
            // past the row's dimensions: zero)
            const int64_t r = row0 + 32 * h + l32, c = col0 + 32 * h + l32;
            a[h] = 0;
            b[h] = 0;
            if (k < d) {
                a[h] = *reinterpret_cast<const int4v *>(X + (size_t)(r < n ? r : 0) * d + k) ^ (int32_t)0x80808080;
                b[h] = *reinterpret_cast<const int4v *>(X + (size_t)(c < n ? c : 0) * d + k) ^ (int32_t)0x80808080;
            }
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[i], b[j], acc[i][j], 0, 0, 0);
    }
    // accumulator register g of lane l: row 8 (g / 4) + 4 (l / 32) + g % 4,
    // column l % 32
#pragma unroll
    for (int i = 0; i < 2; ++i) {
#pragma unroll
        for (int g = 0; g < 16; ++g) {
            const int64_t r = row0 + 32 * i + 8 * (g >> 2) + 4 * half + (g & 3);
            if (r >= r0 + rows) continue;
            const int32_t nr = norms[r];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int64_t c = col0 + 32 * j + l32;
                const int32_t nc = norms[c < n ? c : 0];
                D[(size_t)(r - r0) * ld + (c - cb)] = (float)(nr + nc - 2 * acc[i][j][g]);
            }
        }
    }
}

struct SelectArgs {
    const float *D;          // rows [r0, r0 + rows) x ld: distances to points [c0, c1)
    int64_t n, r0, rows, ld, c0, c1;
    uint64_t *state;         // per row of the panel: its lists between two column chunks
    int32_t K, Kl, levels, m;
    const int32_t *ranks;    // m x n quantile ranks
    const int32_t *thr;      // levels x n thresholds in rank units, not decreasing over the levels
    uint32_t *cand;          // n x K ids (0xFFFFFFFF padded)
    uint32_t *lcand;         // levels x n x Kl ids
};

__device__ __forceinline__ uint64_t uniform64(uint64_t x)
{
    return ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(x >> 32)) << 32) |
           (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)x);
}

// The K (at most N / 2) smallest keys seen, in the first half of N slots of
// LDS (BKEY_NONE past their number), and behind them the newer ones: sorted and
// cut when the next ones do not fit.
template <int N>
struct TopList {
    uint64_t *a;
    int cnt, K;
    uint64_t limit;   // a key must be below it to enter
    __device__ __forceinline__ void init(uint64_t *lds, int K_, int lane)
    {
        a = lds;
        cnt = 0;
        K = K_;
        limit = BKEY_NONE;
        for (int i = lane; i < N; i += 64) a[i] = BKEY_NONE;
    }
    // the list's slots, and behind them its limit and count
    __device__ __forceinline__ void save(uint64_t *to, int lane) const
    {
        wave_fence();
        for (int i = lane; i < N; i += 64) to[i] = a[i];
        if (lane == 0) {
            to[N] = limit;
            to[N + 1] = (uint64_t)cnt;
        }
    }
    __device__ __forceinline__ void load(const uint64_t *from, int lane)
    {
        for (int i = lane; i < N; i += 64) a[i] = from[i];
        limit = uniform64(from[N]);
        cnt = (int)uniform64(from[N + 1]);
        wave_fence();
    }
    __device__ __forceinline__ void cut(int lane)
    {
        wave_fence();
        bitonic<N>(a, lane);
        for (int i = lane; i < N; i += 64)
            if (i >= K) a[i] = BKEY_NONE;
        wave_fence();
        if (cnt >= K) {
            cnt = K;
            limit = uniform64(a[K - 1]);
        }
    }
    // whether a distance (its bits) may be below the limit: nothing to push
    // where no lane's is
    __device__ __forceinline__ bool may(uint32_t bits) const { return bits <= (uint32_t)(limit >> 32); }
    __device__ __forceinline__ void push(uint64_t key, int lane)
    {
        uint64_t m = __ballot(key < limit);
        if (m == 0ull) return;
        if (cnt + (int)__popcll(m) > N) {
            cut(lane);
            m = __ballot(key < limit);
            if (m == 0ull) return;
        }
        const int below = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
        if (key < limit) a[cnt + below] = key;
        cnt += (int)__popcll(m);
    }
};

// A wave per row: one sweep over the row's distances fills the list by vector
// distance and one list per attribute level. At n = 30,000 and m = 3 a sweep
// is about 120 thousand cycles, a third of them the lists' sorts; 24 waves per
// CU (6 KB of lists each) run side by side.
__global__ void __launch_bounds__(256) select_kernel(SelectArgs a)
{
    __shared__ uint64_t lists[4][256 + 128 * KNN_LEVELS];
    const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t i = (int64_t)blockIdx.x * 4 + wid;
    if (i >= a.rows) return;
    const int64_t row = a.r0 + i;
    TopList<256> near;
    TopList<128> lvl[KNN_LEVELS];
    near.init(lists[wid], a.K, lane);
    int32_t t[KNN_LEVELS];
#pragma unroll
    for (int l = 0; l < KNN_LEVELS; ++l) {
        lvl[l].init(lists[wid] + 256 + 128 * l, a.Kl, lane);
        t[l] = l < a.levels ? a.thr[(size_t)l * a.n + row] : -1;
    }
    constexpr int STATE = 256 + 2 + KNN_LEVELS * (128 + 2);
    uint64_t *st = a.state + (size_t)i * STATE;
    if (a.c0 > 0) {
        near.load(st, lane);
#pragma unroll
        for (int l = 0; l < KNN_LEVELS; ++l)
            if (l < a.levels) lvl[l].load(st + 258 + 130 * l, lane);
    }
    int32_t mine[BOA_MAX_M];
#pragma unroll
    for (int j = 0; j < BOA_MAX_M; ++j) mine[j] = a.levels > 0 && j < a.m ? a.ranks[(size_t)j * a.n + row] : 0;
    const float *D = a.D + (size_t)i * a.ld;
    constexpr int U = 4;   // columns per lane in flight
    for (int64_t c0 = a.c0; c0 < a.c1; c0 += 64 * U) {
        float dd[U];
        int32_t gap[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t c = c0 + 64 * u + lane;
            dd[u] = D[(c < a.c1 ? c : a.c1 - 1) - a.c0];
            gap[u] = 0;
        }
        if (a.levels > 0) {
            // attribute distance: the largest gap of ranks over the columns
#pragma unroll
            for (int j = 0; j < BOA_MAX_M; ++j) {
                if (j < a.m) {   // uniform
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const int64_t c = c0 + 64 * u + lane;
                        const int32_t g = mine[j] - a.ranks[(size_t)j * a.n + (c < a.c1 ? c : a.c1 - 1)];
                        gap[u] = max(gap[u], g < 0 ? -g : g);
                    }
                }
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t c = c0 + 64 * u + lane;
            const uint32_t bits = __float_as_uint(dd[u]);
            const uint64_t key = c < a.c1 && c != row ? bkey(dd[u], (uint32_t)c) : BKEY_NONE;
            if (__ballot(near.may(bits)) != 0ull) near.push(key, lane);
#pragma unroll
            for (int l = 0; l < KNN_LEVELS; ++l) {
                if (l >= a.levels) break;   // uniform
                const bool in = gap[u] <= t[l];
                if (__ballot(in && lvl[l].may(bits)) != 0ull) lvl[l].push(in ? key : BKEY_NONE, lane);
            }
        }
    }
    if (a.c1 < a.n) {   // more columns to come
        near.save(st, lane);
#pragma unroll
        for (int l = 0; l < KNN_LEVELS; ++l)
            if (l < a.levels) lvl[l].save(st + 258 + 130 * l, lane);
        return;
    }
    near.cut(lane);
    for (int q = lane; q < a.K; q += 64) {
        const uint64_t x = near.a[q];
        a.cand[(size_t)row * a.K + q] = x == BKEY_NONE ? BOA_PAD : (uint32_t)x;
    }
#pragma unroll
    for (int l = 0; l < KNN_LEVELS; ++l) {
        if (l >= a.levels) break;
        lvl[l].cut(lane);
        for (int q = lane; q < a.Kl; q += 64) {
            const uint64_t x = lvl[l].a[q];
            a.lcand[((size_t)l * a.n + row) * a.Kl + q] = x == BKEY_NONE ? BOA_PAD : (uint32_t)x;
        }
    }
}

// Quantile rank of every cell within its column: the number of strictly
// smaller values (equal values share a rank; float32 columns compare as
// floats). A thread per cell, the column through LDS: n^2 comparisons, 0.4 ms
// a column at n = 60,000, without a sort.
__global__ void __launch_bounds__(256) ranks_kernel(const int32_t *attrs, int64_t n, int m, uint32_t f32_mask,
                                                    int32_t *ranks)
{
    __shared__ int32_t tile[1024];
    const int j = blockIdx.y;
    const bool f = (f32_mask >> j) & 1u;
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int32_t x = i < n ? attrs[(size_t)i * m + j] : 0;
    int32_t below = 0;
    for (int64_t c0 = 0; c0 < n; c0 += 1024) {
        const int cn = (int)(n - c0 < 1024 ? n - c0 : 1024);
        __syncthreads();
        for (int c = threadIdx.x; c < cn; c += 256) tile[c] = attrs[(size_t)(c0 + c) * m + j];
        __syncthreads();
        if (f) {
            const float xf = __int_as_float(x);
            for (int c = 0; c < cn; ++c) below += __int_as_float(tile[c]) < xf ? 1 : 0;
        } else {
            for (int c = 0; c < cn; ++c) below += tile[c] < x ? 1 : 0;
        }
    }
    if (i < n) ranks[(size_t)j * n + i] = below;
}

static constexpr int SAMPLE = 4096;

// ranks of the sample points floor(s n / S), S = min(SAMPLE, n): m x SAMPLE
__global__ void sample_kernel(const int32_t *ranks, int64_t n, int32_t *sample)
{
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= SAMPLE || s >= n) return;
    const int64_t id = n >= SAMPLE ? ((int64_t)s * n) / SAMPLE : s;
    sample[(size_t)blockIdx.y * SAMPLE + s] = ranks[(size_t)blockIdx.y * n + id];
}

struct ThresholdArgs {
    const int32_t *ranks;    // m x n
    const int32_t *sample;   // m x SAMPLE
    int64_t n;
    int32_t m, levels;
    int32_t order[KNN_LEVELS];   // per level: the threshold's place in the sorted distances
    int32_t *thr;            // levels x n
};

// Per point and level: the order[l]-th smallest of its attribute distances to
// the sample. A wave per point holds the S distances in registers and finds
// the smallest value with enough distances at or below it by bisection (up to
// 21 counts of S comparisons per level, in place of a selection per level on
// the host: 150 ms of 16 threads at n = 60,000).
__global__ void __launch_bounds__(256) thresholds_kernel(ThresholdArgs a)
{
    const int lane = threadIdx.x & 63;
    const int64_t u = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (u >= a.n) return;
    const int S = a.n < SAMPLE ? (int)a.n : SAMPLE;
    int32_t g[SAMPLE / 64];
#pragma unroll
    for (int i = 0; i < SAMPLE / 64; ++i) g[i] = lane + 64 * i < S ? 0 : INT32_MAX;   // (past it: never counted)
    for (int j = 0; j < a.m; ++j) {
        const int32_t *rk = a.sample + (size_t)j * SAMPLE;
        const int32_t x = a.ranks[(size_t)j * a.n + u];
#pragma unroll
        for (int i = 0; i < SAMPLE / 64; ++i) {
            const int s = lane + 64 * i;
            if (s < S) {
                const int32_t t = x - rk[s];
                g[i] = max(g[i], t < 0 ? -t : t);
            }
        }
    }
    for (int l = 0; l < a.levels; ++l) {
        int32_t lo = 0, hi = (int32_t)(a.n - 1);   // the answer is in [lo, hi]
        while (lo < hi) {
            const int32_t mid = lo + ((hi - lo) >> 1);
            int32_t c = 0;
#pragma unroll
            for (int i = 0; i < SAMPLE / 64; ++i) c += g[i] <= mid ? 1 : 0;
#pragma unroll
            for (int s = 32; s >= 1; s >>= 1) c += __shfl_xor(c, s);
            c = __builtin_amdgcn_readfirstlane(c);
            if (c > a.order[l]) hi = mid;
            else lo = mid + 1;
        }
        if (lane == 0) a.thr[(size_t)l * a.n + u] = lo;
    }
}

// ---------------------------------------------------------------------------
// 3./4. alpha-pruning of a sorted candidate list, one wave per point

struct PruneArgs {
    BuildView v;
    // source lists: forward prune reads the kNN lists (n x K); the re-prune
    // reads, per point, its forward row (n x R) and its reverse neighbours
    // (CSR rev_off / rev)
    const uint32_t *cand;
    int32_t K;
    const uint32_t *fwd;
    const uint32_t *rev_off;
    const uint32_t *rev;
    int32_t R;
    int32_t budget;
    float alpha2;      // the pruning slack alpha, squared (squared distances)
    uint32_t *out;     // n x R (0xFFFFFFFF padded)
};

// Prune the keys sorted in `keys[0, cnt)` (cnt <= 256) into out_row (at most
// `budget` ids), by the alpha-dominance rule. Every kept point is tested at
// once against all the candidates still alive, four per lane: as many steps
// as points are kept (8 to 63), instead of one per candidate (up to 256) with
// a lane per kept point: 14.5 and 5.6 ms of pruning at n = 30,000, d = 96, R = 64.
__device__ void alpha_prune(const BuildView &v, const uint64_t *keys, int cnt, int budget, float alpha2,
                            uint32_t *out_row, int R, int lane)
{
    uint64_t key[4];
    bool alive[4];
#pragma unroll
    for (int h = 0; h < 4; ++h) {
        const int i = lane + 64 * h;
        key[h] = i < cnt ? keys[i] : BKEY_NONE;
        alive[h] = key[h] != BKEY_NONE;
    }
    int nk = 0;
    uint32_t mine = BOA_PAD;   // lane i: the i-th kept id (budget < R <= 64)
    while (nk < budget) {
        // the nearest candidate alive
        uint32_t w = BOA_PAD;
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            const uint64_t m = __ballot(alive[h]);
            if (w == BOA_PAD && m) {
                const int l = __ffsll((unsigned long long)m) - 1;
                w = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)key[h], l);
                if (lane == l) alive[h] = false;
            }
        }
        if (w == BOA_PAD) break;
        if (lane == nk) mine = w;
        ++nk;
        if (nk == budget) break;
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            if (alive[h]) {
                const uint32_t c = (uint32_t)key[h];
                const float duv = __uint_as_float((uint32_t)(key[h] >> 32));
                bool dom;
                if (v.u8 || v.D) {
                    dom = alpha2 * dist_ids(v, w, c) <= duv;
                } else {
                    const float *X = reinterpret_cast<const float *>(v.vectors);
                    dom = pair_within_f32(X + (size_t)w * v.d, X + (size_t)c * v.d, v.d, alpha2, duv);
                }
                if (dom) alive[h] = false;
            }
        }
    }
    if (lane < R) out_row[lane] = mine;
}

__global__ void __launch_bounds__(256) prune_fwd_kernel(PruneArgs a)
{
    __shared__ uint64_t keys_s[4][128];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int64_t u = (int64_t)blockIdx.x * 4 + wid;
    if (u >= a.v.n) return;
    uint64_t *keys = keys_s[wid];
    // the candidates in (distance, id) order, with this pass's own distance
    const uint32_t *cand = a.cand + ((size_t)blockIdx.y * a.v.n + u) * a.K;
    for (int i = lane; i < 128; i += 64) {
        uint64_t k = BKEY_NONE;
        if (i < a.K) {
            const uint32_t c = cand[i];
            if (c != BOA_PAD) k = bkey(dist_ids(a.v, (uint32_t)u, c), c);
        }
        keys[i] = k;
    }
    wave_fence();
    bitonic<128>(keys, lane);
    alpha_prune(a.v, keys, a.K, a.budget, a.alpha2, a.out + ((size_t)blockIdx.y * a.v.n + u) * a.R, a.R, lane);
}

// Re-prune each point's forward row together with its reverse neighbours
// (the nearest 256 - R of them when there are more) to `budget` edges.
__global__ void __launch_bounds__(256) prune_union_kernel(PruneArgs a)
{
    __shared__ uint64_t keys_s[4][256];
    __shared__ uint64_t buf_s[4][256];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int64_t u = (int64_t)blockIdx.x * 4 + wid;
    if (u >= a.v.n) return;
    uint64_t *keys = keys_s[wid];
    uint64_t *buf = buf_s[wid];
    const uint32_t *frow = a.fwd + (size_t)u * a.R;
    for (int i = lane; i < 256; i += 64) {
        uint64_t k = BKEY_NONE;
        if (i < a.R) {
            const uint32_t c = frow[i];
            if (c != BOA_PAD) k = bkey(dist_ids(a.v, (uint32_t)u, c), c);
        }
        keys[i] = k;
    }
    wave_fence();
    bitonic<256>(keys, lane);
    // reverse neighbours not already forward ones, merged 128 at a time
    // into the 256 best (a row holds at most R <= 64 forward ids)
    const uint32_t r0 = a.rev_off[u], r1 = a.rev_off[u + 1];
    for (uint32_t b0 = r0; b0 < r1; b0 += 128) {
        for (int h = 0; h < 4; ++h) {
            const int i = lane + 64 * h;
            uint64_t k = BKEY_NONE;
            if (i < 128) {
                const uint32_t t = b0 + (uint32_t)i;
                if (t < r1) {
                    const uint32_t c = a.rev[t];
                    bool dup = false;
                    for (int q = 0; q < a.R; ++q) dup |= frow[q] == c;
                    if (!dup) k = bkey(dist_ids(a.v, (uint32_t)u, c), c);
                }
            } else {
                k = keys[i];   // the current upper half
            }
            buf[i] = k;
        }
        wave_fence();
        // the 256 best of keys[0,256) and the new 128: the first 128 of the
        // sorted keys stay; sort (keys[128..256) + new 128) and keep the best
        // 128 of those as the upper half
        bitonic<256>(buf, lane);
        for (int i = lane; i < 128; i += 64) keys[128 + i] = buf[i];
        wave_fence();
        bitonic<256>(keys, lane);
    }
    alpha_prune(a.v, keys, 256, a.budget, a.alpha2, a.out + (size_t)u * a.R, a.R, lane);
}

__global__ void count_in_kernel(const uint32_t *adj, int64_t n, int R, uint32_t *indeg)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n * R) return;
    const uint32_t v = adj[i];
    if (v != BOA_PAD) atomicAdd(&indeg[v], 1u);
}

__global__ void scatter_rev_kernel(const uint32_t *adj, int64_t n, int R, const uint32_t *off, uint32_t *cursor,
                                   uint32_t *rev)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n * R) return;
    const uint32_t v = adj[i];
    if (v == BOA_PAD) return;
    const uint32_t pos = atomicAdd(&cursor[v], 1u);
    rev[off[v] + pos] = (uint32_t)(i / R);
}

// 5. rows: the levels' edges appended to a point's row (one wave per point),
// narrowest level first, without ids the row has, up to one free slot
__global__ void __launch_bounds__(256) append_levels_kernel(uint32_t *adj, const uint32_t *level_rows, int64_t n, int R,
                                                            int levels, int b_lvl, unsigned long long *added)
{
    __shared__ int sum[2][4];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int64_t u = (int64_t)blockIdx.x * 4 + wid;
    const bool in = u < n;
    uint32_t v = in && lane < R ? adj[(size_t)u * R + lane] : BOA_PAD;
    int cnt = __popcll(__ballot(v != BOA_PAD));   // (the ids fill a row's front)
    const int cnt0 = cnt;
    for (int l = 0; in && l < levels; ++l) {
        const uint32_t e = lane < b_lvl ? level_rows[((size_t)l * n + u) * b_lvl + lane] : BOA_PAD;
        for (int i = 0; i < b_lvl && cnt < R - 1; ++i) {
            const uint32_t x = (uint32_t)__builtin_amdgcn_readlane((int)e, i);
            if (x == BOA_PAD) break;
            if (__ballot(v == x) != 0ull) continue;
            if (lane == cnt) v = x;
            ++cnt;
        }
    }
    if (in && lane < R) adj[(size_t)u * R + lane] = v;
    if (lane == 0) {
        sum[0][wid] = cnt - cnt0;
        sum[1][wid] = cnt;
    }
    __syncthreads();
    if (threadIdx.x < 2)
        atomicAdd(&added[threadIdx.x], (unsigned long long)(sum[threadIdx.x][0] + sum[threadIdx.x][1] +
                                                            sum[threadIdx.x][2] + sum[threadIdx.x][3]));
}

// one step of a breadth-first search, one wave per frontier node
__global__ void __launch_bounds__(256) bfs_kernel(const uint32_t *adj, int R, uint32_t *seen, const uint32_t *in,
                                                  uint32_t n_in, uint32_t *out, uint32_t *n_out)
{
    const int lane = threadIdx.x & 63;
    const uint32_t f = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (f >= n_in) return;
    const uint32_t y = lane < R ? adj[(size_t)in[f] * R + lane] : BOA_PAD;
    if (y != BOA_PAD && seen[y] == 0u && atomicExch(&seen[y], 1u) == 0u) out[atomicAdd(n_out, 1u)] = y;
}

// ---------------------------------------------------------------------------
// host side

namespace {

struct DevBuf {
    void *p = nullptr;
    ~DevBuf()
    {
        if (p) (void)hipFree(p);
    }
    hipError_t alloc(size_t bytes)
    {
        const hipError_t e = hipMalloc(&p, bytes ? bytes : 1);
        if (e != hipSuccess) p = nullptr;
        return e;
    }
    template <class T>
    T *as() const { return reinterpret_cast<T *>(p); }
};

#define BTRY(expr)                                  \
    do {                                            \
        hipError_t e_ = (expr);                     \
        if (e_ != hipSuccess) {                     \
            (void)hipGetLastError();                \
            return e_;                              \
        }                                           \
    } while (0)

}  // namespace

hipError_t compute_medoid(const void *d_vectors, int64_t n, int32_t d, int vec_dtype, uint32_t *entry)
{
    BuildView v{d_vectors, nullptr, n, d, vec_dtype == BOA_VEC_U8 ? 1 : 0, nullptr, 0};
    const int nb = (int)std::min<int64_t>(512, n);
    const int64_t per = (n + nb - 1) / nb;
    DevBuf part, cen, bd, bi;
    BTRY(part.alloc((size_t)nb * d * 8));
    BTRY(cen.alloc((size_t)d * 8));
    CentroidArgs ca{v, part.as<double>(), per};
    hipLaunchKernelGGL(centroid_partial_kernel, dim3(nb), dim3(256), 0, 0, ca);
    BTRY(hipGetLastError());
    // the partial sums added in block order on the host (float64)
    std::vector<double> hp((size_t)nb * d), c((size_t)d, 0.0);
    BTRY(hipMemcpy(hp.data(), part.p, hp.size() * 8, hipMemcpyDeviceToHost));
    for (int b = 0; b < nb; ++b)
        for (int j = 0; j < d; ++j) c[j] += hp[(size_t)b * d + j];
    for (int j = 0; j < d; ++j) c[j] /= (double)n;
    BTRY(hipMemcpy(cen.p, c.data(), (size_t)d * 8, hipMemcpyHostToDevice));
    const int mb = 1024;
    BTRY(bd.alloc((size_t)mb * 8));
    BTRY(bi.alloc((size_t)mb * 4));
    MedoidArgs ma{v, cen.as<double>(), bd.as<double>(), bi.as<uint32_t>()};
    hipLaunchKernelGGL(medoid_partial_kernel, dim3(mb), dim3(256), 0, 0, ma);
    BTRY(hipGetLastError());
    std::vector<double> hd(mb);
    std::vector<uint32_t> hi(mb);
    BTRY(hipMemcpy(hd.data(), bd.p, (size_t)mb * 8, hipMemcpyDeviceToHost));
    BTRY(hipMemcpy(hi.data(), bi.p, (size_t)mb * 4, hipMemcpyDeviceToHost));
    double best = INFINITY;
    uint32_t id = 0xFFFFFFFFu;
    for (int b = 0; b < mb; ++b)
        if (hd[b] < best || (hd[b] == best && hi[b] < id)) {
            best = hd[b];
            id = hi[b];
        }
    // (no point compares where the vectors hold a NaN: the lowest id)
    *entry = id == 0xFFFFFFFFu ? 0u : id;
    return hipSuccess;
}

namespace {

hipError_t ranks_and_thresholds(const int32_t *h_attrs, int64_t n, int m, uint32_t f32_mask, const double *q, int levels,
                                int32_t *ranks, int32_t *thr)
{
    DevBuf attrs;
    BTRY(attrs.alloc((size_t)n * m * 4));
    BTRY(hipMemcpy(attrs.p, h_attrs, (size_t)n * m * 4, hipMemcpyHostToDevice));
    hipLaunchKernelGGL(ranks_kernel, dim3((unsigned)((n + 255) / 256), (unsigned)m), dim3(256), 0, 0,
                       attrs.as<int32_t>(), n, m, f32_mask, ranks);
    BTRY(hipGetLastError());
    DevBuf sample;
    BTRY(sample.alloc((size_t)m * SAMPLE * 4));
    hipLaunchKernelGGL(sample_kernel, dim3(SAMPLE / 256, (unsigned)m), dim3(256), 0, 0, ranks, n, sample.as<int32_t>());
    BTRY(hipGetLastError());
    ThresholdArgs ta{};
    ta.ranks = ranks;
    ta.sample = sample.as<int32_t>();
    ta.n = n;
    ta.m = m;
    ta.levels = levels;
    ta.thr = thr;
    const int64_t S = std::min<int64_t>(SAMPLE, n);
    for (int l = 0; l < levels; ++l)
        ta.order[l] = (int32_t)std::max<int64_t>(0, (int64_t)std::ceil(q[l] * (double)S) - 1);
    hipLaunchKernelGGL(thresholds_kernel, dim3((unsigned)((n + 3) / 4)), dim3(256), 0, 0, ta);
    BTRY(hipGetLastError());
    return hipSuccess;   // (freeing the copy of the attributes waits for the kernels)
}

// Where all distances fit 512 MB (11,500 points), they are computed in one
// piece (half of a float32 index's mirrored) and stay for the pruning (v.D),
// whose tests are then one read each: 12.1 -> 0.3 ms at n = 10,000, d = 768.
// Otherwise in tiles of 6,144 rows (24 of the selection's waves per CU) by 6,144
// columns, 151 MB, which stay in the last cache, the rows' lists kept between
// them (38 MB): 23.6 ms at n = 60,000 uint8 (4,096 rows 27.0, with twice the
// columns 24.8; 2,048 rows 34.2). Just above the line a build takes up to seven
// times as long (float32, tiles against all kept: n = 12,500 7.6 and 3.5 ms for
// d = 96, 49 and 8.6 for d = 768; n = 20,000 15 and 8.6, 86 and 16), so a higher
// one is faster where the memory is at hand, as in a process that only builds
// (19 against 24 ms at n = 60,000). It stays here because memory that others
// have used is cleared by the driver before it is handed out again, 25 to 28 ms
// a gigabyte: that exceeds the gain of narrow rows, not that of wide ones.
constexpr int64_t WHOLE_BYTES = (int64_t)512 << 20;
constexpr int64_t PANEL_ROWS = 6144, PANEL_COLS = 48 * DT;

hipError_t find_candidates(BuildView &v, const int32_t *norms_shifted, int K, int Kl, int levels, int m,
                           const int32_t *ranks, const int32_t *thr, uint32_t *cand, uint32_t *lcand, DevBuf &dist)
{
    const int64_t n = v.n, all = (n + DT - 1) / DT * DT;
    bool whole = n * all * 4 <= WHOLE_BYTES;
    if (whole && dist.alloc((size_t)(n * all * 4)) != hipSuccess) {
        (void)hipGetLastError();
        whole = false;
    }
    const int64_t panel = whole ? n : std::min<int64_t>(PANEL_ROWS, all);
    const int64_t ld = whole ? all : std::min<int64_t>(PANEL_COLS, all);
    DevBuf state;
    if (!whole) BTRY(dist.alloc((size_t)(panel * ld * 4)));
    if (ld < n) BTRY(state.alloc((size_t)panel * (256 + 2 + KNN_LEVELS * (128 + 2)) * 8));
    for (int64_t r0 = 0; r0 < n; r0 += panel) {
        const int64_t rows = std::min<int64_t>(panel, n - r0);
        for (int64_t c0 = 0; c0 < n; c0 += ld) {
            const int64_t c1 = std::min<int64_t>(c0 + ld, n);
            const dim3 tiles((unsigned)((c1 - c0 + DT - 1) / DT), (unsigned)((rows + DT - 1) / DT));
            if (v.u8)
                hipLaunchKernelGGL(dist_u8_kernel, tiles, dim3(256), 0, 0, reinterpret_cast<const uint8_t *>(v.vectors),
                                   norms_shifted, n, v.d, r0, rows, c0, ld, dist.as<float>());
            else if (whole)
                hipLaunchKernelGGL(dist_f32_kernel<true>, tiles, dim3(256), 0, 0,
                                   reinterpret_cast<const float *>(v.vectors), n, v.d, r0, rows, c0, ld, dist.as<float>());
            else
                hipLaunchKernelGGL(dist_f32_kernel<false>, tiles, dim3(256), 0, 0,
                                   reinterpret_cast<const float *>(v.vectors), n, v.d, r0, rows, c0, ld, dist.as<float>());
            BTRY(hipGetLastError());
            SelectArgs sa{};
            sa.D = dist.as<float>();
            sa.n = n;
            sa.r0 = r0;
            sa.rows = rows;
            sa.ld = ld;
            sa.c0 = c0;
            sa.c1 = c1;
            sa.state = state.as<uint64_t>();
            sa.K = K;
            sa.Kl = Kl;
            sa.levels = levels;
            sa.m = m;
            sa.ranks = ranks;
            sa.thr = thr;
            sa.cand = cand;
            sa.lcand = lcand;
            hipLaunchKernelGGL(select_kernel, dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, 0, sa);
            BTRY(hipGetLastError());
        }
    }
    if (whole) {
        v.D = dist.as<float>();
        v.ld = ld;
    }
    return hipSuccess;
}

// Points a breadth-first search from `entry` reaches; -1 where the device's
// search is not worth its steps, each a round trip to the host of 16 us. The
// host's own search costs 4 to 16 ns an entry of the adjacency with its copies, so
// the steps may take up to 2 ns an entry: rows of 16 and more of clustered and
// random points (n = 1,000 to 60,000) need 4 to 19 steps, points along a line
// thousands (a build of n = 10,000, R = 4: 91 ms with them, 1.9 without). Rows of
// less than 8 entries leave points out of reach nearly always, which the host has
// to repair (scattered points, n = 1,000, R = 4: 1.1 ms with the steps, 0.5 without).
hipError_t count_reached(const uint32_t *adj, int64_t n, int R, uint32_t entry, int64_t *reached)
{
    *reached = -1;
    const int64_t max_steps = R < 8 ? 0 : n * R / 8192;
    if (max_steps == 0) return hipSuccess;
    DevBuf seen, list, count;
    BTRY(seen.alloc((size_t)n * 4));
    BTRY(list.alloc((size_t)n * 2 * 4));
    BTRY(count.alloc(4));
    BTRY(hipMemset(seen.p, 0, (size_t)n * 4));
    const uint32_t one = 1;
    BTRY(hipMemcpy(seen.as<uint32_t>() + entry, &one, 4, hipMemcpyHostToDevice));
    BTRY(hipMemcpy(list.p, &entry, 4, hipMemcpyHostToDevice));
    uint32_t *in = list.as<uint32_t>(), *out = in + n;
    uint32_t n_in = 1;
    int64_t listed = 0;
    for (int64_t step = 0; n_in > 0; ++step) {
        if (step == max_steps) return hipSuccess;
        listed += n_in;
        BTRY(hipMemset(count.p, 0, 4));
        hipLaunchKernelGGL(bfs_kernel, dim3((n_in + 3) / 4), dim3(256), 0, 0, adj, R, seen.as<uint32_t>(), in, n_in, out,
                           count.as<uint32_t>());
        BTRY(hipGetLastError());
        BTRY(hipMemcpy(&n_in, count.p, 4, hipMemcpyDeviceToHost));
        std::swap(in, out);
    }
    *reached = listed;
    return hipSuccess;
}

}  // namespace

hipError_t build_graph(const void *d_vectors, int64_t n, int32_t d, int vec_dtype, int32_t R, uint32_t entry,
                       const int32_t *h_attrs, int32_t m, uint32_t f32_mask, float alpha, int32_t attr_levels,
                       uint32_t *d_adj, BuildStats *stats)
{
    const bool u8 = vec_dtype == BOA_VEC_U8;
    const float alpha2 = alpha * alpha;
    // budgets: each attribute level R/8 edges, the vector pass the rest but
    // one (the free slot the connectivity repair may take)
    static const double kLevelQ[4] = {0.001, 0.01, 0.05, 0.2};
    const int levels = (h_attrs && m > 0 && R >= 8) ? std::min(attr_levels, 4) : 0;
    const int b_lvl = std::max(1, R / 8);
    const int budget = std::max(1, R - 1 - levels * b_lvl);
    const int K = (int)std::min<int64_t>(std::min(2 * R, KNN_LIST), n - 1);
    DevBuf norms, norms2;
    BuildView v{d_vectors, nullptr, n, d, u8 ? 1 : 0, nullptr, 0};
    if (u8) {
        BTRY(norms.alloc((size_t)n * 4));
        BTRY(norms2.alloc((size_t)n * 4));
        hipLaunchKernelGGL(norms_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, 0, v, norms.as<uint32_t>(),
                           norms2.as<int32_t>());
        BTRY(hipGetLastError());
        v.norms = norms.as<uint32_t>();
    }
    if (K < 1) {   // a single point: no edges
        BTRY(hipMemset(d_adj, 0xFF, (size_t)n * R * 4));
        return hipSuccess;
    }
    // 2. candidates by vector distance, for all attribute levels too (JAG
    // threshold pruning, Sec. II "Graph construction": per level, the nearest
    // vectors among the points within the point's attribute threshold, where
    // the capped attribute distance is zero)
    const int Kl = (int)std::min<int64_t>(std::min(4 * b_lvl, KNN_LEVEL_LIST), n - 1);
    DevBuf cand, lcand, ranks, thr, dist;
    BTRY(cand.alloc((size_t)n * K * 4));
    if (levels > 0) {
        BTRY(ranks.alloc((size_t)n * m * 4));
        BTRY(thr.alloc((size_t)n * levels * 4));
        BTRY(lcand.alloc((size_t)n * Kl * levels * 4));
        BTRY(ranks_and_thresholds(h_attrs, n, m, f32_mask, kLevelQ, levels, ranks.as<int32_t>(), thr.as<int32_t>()));
    }
    BTRY(find_candidates(v, norms2.as<int32_t>(), K, Kl, levels, m, ranks.as<int32_t>(), thr.as<int32_t>(),
                         cand.as<uint32_t>(), lcand.as<uint32_t>(), dist));
    // 3. forward prune
    DevBuf fwd, lrow;
    BTRY(fwd.alloc((size_t)n * R * 4));
    {
        PruneArgs pa{};
        pa.v = v;
        pa.cand = cand.as<uint32_t>();
        pa.K = K;
        pa.R = R;
        pa.budget = budget;
        pa.alpha2 = alpha2;
        pa.out = fwd.as<uint32_t>();
        hipLaunchKernelGGL(prune_fwd_kernel, dim3((unsigned)((n + 3) / 4)), dim3(256), 0, 0, pa);
        BTRY(hipGetLastError());
    }
    if (levels > 0) {   // the levels' b_lvl edges per point
        BTRY(lrow.alloc((size_t)n * b_lvl * levels * 4));
        PruneArgs pa{};
        pa.v = v;
        pa.cand = lcand.as<uint32_t>();
        pa.K = Kl;
        pa.R = b_lvl;
        pa.budget = b_lvl;
        pa.alpha2 = alpha2;
        pa.out = lrow.as<uint32_t>();
        hipLaunchKernelGGL(prune_fwd_kernel, dim3((unsigned)((n + 3) / 4), (unsigned)levels), dim3(256), 0, 0, pa);
        BTRY(hipGetLastError());
    }
    // 4. reverse edges (CSR), then the union re-pruned
    DevBuf indeg, off, cursor, rev;
    BTRY(indeg.alloc((size_t)n * 4));
    BTRY(hipMemset(indeg.p, 0, (size_t)n * 4));
    const unsigned eb = (unsigned)((n * R + 255) / 256);
    hipLaunchKernelGGL(count_in_kernel, dim3(eb), dim3(256), 0, 0, fwd.as<uint32_t>(), n, R, indeg.as<uint32_t>());
    BTRY(hipGetLastError());
    std::vector<uint32_t> h_in((size_t)n), h_off((size_t)n + 1);
    BTRY(hipMemcpy(h_in.data(), indeg.p, (size_t)n * 4, hipMemcpyDeviceToHost));
    h_off[0] = 0;
    for (int64_t i = 0; i < n; ++i) h_off[i + 1] = h_off[i] + h_in[i];
    BTRY(off.alloc(((size_t)n + 1) * 4));
    BTRY(cursor.alloc((size_t)n * 4));
    BTRY(rev.alloc((size_t)h_off[n] * 4));
    BTRY(hipMemcpy(off.p, h_off.data(), ((size_t)n + 1) * 4, hipMemcpyHostToDevice));
    BTRY(hipMemset(cursor.p, 0, (size_t)n * 4));
    hipLaunchKernelGGL(scatter_rev_kernel, dim3(eb), dim3(256), 0, 0, fwd.as<uint32_t>(), n, R, off.as<uint32_t>(),
                       cursor.as<uint32_t>(), rev.as<uint32_t>());
    BTRY(hipGetLastError());
    {
        PruneArgs pa{};
        pa.v = v;
        pa.fwd = fwd.as<uint32_t>();
        pa.rev_off = off.as<uint32_t>();
        pa.rev = rev.as<uint32_t>();
        pa.R = R;
        pa.budget = budget;
        pa.alpha2 = alpha2;
        pa.out = d_adj;
        hipLaunchKernelGGL(prune_union_kernel, dim3((unsigned)((n + 3) / 4)), dim3(256), 0, 0, pa);
        BTRY(hipGetLastError());
    }
    // 5. the levels' edges appended to the rows
    DevBuf added;
    BTRY(added.alloc(16));
    BTRY(hipMemset(added.p, 0, 16));
    hipLaunchKernelGGL(append_levels_kernel, dim3((unsigned)((n + 3) / 4)), dim3(256), 0, 0, d_adj, lrow.as<uint32_t>(), n,
                       R, levels, b_lvl, added.as<unsigned long long>());
    BTRY(hipGetLastError());
    unsigned long long h_added[2] = {0, 0};
    BTRY(hipMemcpy(h_added, added.p, 16, hipMemcpyDeviceToHost));
    int64_t reached = 0;
    BTRY(count_reached(d_adj, n, R, entry, &reached));
    if (stats) {
        stats->K = K;
        stats->repaired = 0;
        stats->repair_fallback = 0;
        stats->attr_edges = (int64_t)h_added[0];
        stats->edges = (int64_t)h_added[1];
    }
    if (reached == n) return hipSuccess;
    std::vector<uint32_t> adj((size_t)n * R), hc((size_t)n * K);
    BTRY(hipMemcpy(adj.data(), d_adj, adj.size() * 4, hipMemcpyDeviceToHost));
    BTRY(hipMemcpy(hc.data(), cand.p, hc.size() * 4, hipMemcpyDeviceToHost));
    // 6. connectivity repair from s (host, unless the device's search found
    // every point within reach): breadth-first search, then each unreached
    // point (ascending id) gets an in-edge from its nearest reached kNN
    // candidate with a free slot; the search then continues from it
    std::vector<uint8_t> seen((size_t)n, 0);
    std::vector<uint32_t> queue;
    queue.reserve((size_t)n);
    auto bfs_from = [&](uint32_t s) {
        size_t h = queue.size();
        seen[s] = 1;
        queue.push_back(s);
        while (h < queue.size()) {
            const uint32_t x = queue[h++];
            for (int r = 0; r < R; ++r) {
                const uint32_t y = adj[(size_t)x * R + r];
                if (y != BOA_PAD && !seen[y]) {
                    seen[y] = 1;
                    queue.push_back(y);
                }
            }
        }
    };
    bfs_from(entry);
    int64_t repaired = 0, fallback = 0;
    auto free_slot = [&](uint32_t w) -> int {
        for (int r = 0; r < R; ++r)
            if (adj[(size_t)w * R + r] == BOA_PAD) return r;
        return -1;
    };
    for (int64_t u = 0; u < n; ++u) {
        if (seen[u]) continue;
        int64_t w = -1;
        for (int c = 0; c < K; ++c) {   // candidates are nearest first
            const uint32_t x = hc[(size_t)u * K + c];
            if (x != BOA_PAD && seen[x] && free_slot(x) >= 0) {
                w = x;
                break;
            }
        }
        if (w < 0) {
            // no reached candidate with room: the first reached point (in
            // search order) with a free slot (every row keeps one)
            for (size_t q = 0; q < queue.size() && w < 0; ++q)
                if (free_slot(queue[q]) >= 0) w = queue[q];
            ++fallback;
        }
        if (w < 0) return hipErrorUnknown;   // cannot happen: s itself has a free slot
        adj[(size_t)w * R + free_slot((uint32_t)w)] = (uint32_t)u;
        ++repaired;
        bfs_from((uint32_t)u);
    }
    BTRY(hipMemcpy(d_adj, adj.data(), adj.size() * 4, hipMemcpyHostToDevice));
    if (stats) {
        stats->repaired = repaired;
        stats->repair_fallback = fallback;
        stats->edges += repaired;
    }
    return hipSuccess;
}

}  // namespace boa
