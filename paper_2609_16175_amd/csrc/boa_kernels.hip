// Device side of the BOA filtered beam search for gfx950 (CDNA4).
//
// One 64-lane wavefront runs one query at a time: a persistent grid of
// waves pulls query slots from a per-launch atomic counter. Per expansion
// (Alg. 2, one node per iteration):
//   1. select the smallest not-yet-expanded key of the worklist;
//   2. gather its adjacency row, one neighbour per lane (one coalesced load);
//   3. test-and-insert every neighbour into the query's visited set: a
//      two-choice bucketed table of 16-bit entries in LDS whose overflow
//      goes to a per-wave bitmap over all points in HBM, or an LDS bitmap over
//      all ids (teams, and the escalation launch of a split search, where it
//      fits and still lets every query be resident);
//   4. for the unseen neighbours: gather the attribute cells and count the
//      violated range predicates (phi, Eq. 2), gather the vector and compute
//      the squared L2 distance with a 16-lane (float32) or G-lane (uint8)
//      group per candidate and a butterfly reduction;
//   5. pack (phi, distance, id) into one 64-bit key and drop keys that cannot
//      enter the worklist. The rest wait, one per lane, beside the sorted
//      worklist in LDS (WaveList); when the next batch does not fit, they are
//      sorted by counting (each key's rank is the number of keys below it)
//      and merged: each key's rank in the list by an eight-way search, its
//      output slot marked in a bitmap, and the suffix rebuilt backwards in
//      64-entry chunks where a popcount of the bitmap tells every output
//      slot where its entry comes from.
// The epilogue writes the first k filter-valid entries, the phase width,
// and the Eq. 3 confidence flag.
//
// Launches of few queries give each a team of waves instead (team_kernel,
// below): one owns the worklist and the visited set, the others run the row,
// gathers and scoring of the nodes next in order.
//
// Worklist key (unsigned 64-bit, compared as an integer):
//   bits 63..60 phi (violations, <= 8), bits 59..28 float32 bits of the
//   squared distance (non-negative floats order like their bit patterns),
//   bits 27..4 point id (< 2^24), bit 0 expanded flag. Distinct ids make
//   distinct keys, so the flag bits never decide an order.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "boa_internal.h"

namespace boa {

// Optional per-stage cycle accounting (build with -DBOA_STAGE_PROFILE): each
// wave adds the shader-clock cycles of every stage of every expansion to its
// slot's row of PhaseArgs::prof. Off in the product build.
#ifdef BOA_STAGE_PROFILE
#define PROF_T(var) const uint64_t var = __builtin_amdgcn_s_memtime()
#define PROF_ADD(i, v) (prof_acc[(i)] += (v))
#else
#define PROF_T(var)
#define PROF_ADD(i, v)
#endif

static constexpr uint64_t KEY_NONE = ~0ull;
static constexpr uint64_t KEY_PHI1 = 1ull << 60;  // smallest key with phi >= 1

__device__ __forceinline__ uint64_t make_key(uint32_t phi, float d, uint32_t id)
{
    return ((uint64_t)phi << 60) | ((uint64_t)__float_as_uint(d) << 28) | ((uint64_t)id << 4);
}
__device__ __forceinline__ uint32_t key_id(uint64_t k) { return (uint32_t)(k >> 4) & 0xFFFFFFu; }
__device__ __forceinline__ float key_dist(uint64_t k) { return __uint_as_float((uint32_t)(k >> 28)); }

__device__ __forceinline__ int lane_id() { return __lane_id(); }

// Compiler-level ordering point for LDS data exchanged between lanes of one
// wave (the wave executes in lockstep; this keeps the compiler from caching
// or reordering the shared accesses across it).
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ uint32_t bcast0(uint32_t v) { return __builtin_amdgcn_readfirstlane(v); }

// value of lane l (wave-uniform l) in every lane, without an LDS round trip
__device__ __forceinline__ uint64_t readlane64(uint64_t v, int l)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, l);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), l);
    return ((uint64_t)hi << 32) | lo;
}

__device__ __forceinline__ uint32_t lanes_below(uint64_t mask)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// first index i in [0, n) with a[i] >= key (a sorted ascending)
__device__ __forceinline__ uint32_t lower_bound64(const uint64_t *a, uint32_t n, uint64_t key)
{
    uint32_t lo = 0, hi = n;
    while (lo < hi) {
        uint32_t mid = (lo + hi) >> 1;
        if (a[mid] < key) lo = mid + 1; else hi = mid;
    }
    return lo;
}
// The same index in a[0, P) for a power of two P whose entries from n on
// hold KEY_NONE (greater than any key), by eight-way steps: seven
// independent LDS reads per step at shifted offsets, the same number of
// steps in every lane (512 entries: three eight-way steps and one compare).
// The answer stays in [b, b + s]; pivot j of a step (stride s / 8) is below
// the key exactly when at least j s / 8 entries from b are.
__device__ __forceinline__ uint32_t lower_bound64_p2(const uint64_t *a, uint32_t P, uint64_t key)
{
    uint32_t b = 0, sh = 31u - (uint32_t)__clz(P);   // s = 2^sh = P
    while (sh >= 3u) {   // uniform
        sh -= 3u;
        uint32_t below = 0;
#pragma unroll
        for (uint32_t j = 1; j <= 7; ++j) below += a[b + (j << sh) - 1u] < key ? 1u : 0u;
        b += below << sh;
    }
    while (sh > 0u) {    // s in {2, 4}: halve
        sh -= 1u;
        if (a[b + (1u << sh) - 1u] < key) b += 1u << sh;
    }
    return b + (a[b] < key ? 1u : 0u);
}

// Cross-lane move inside a 16-lane row by DPP (no LDS round trip):
// row_shr:J gives lane i the value of lane i-J; lanes whose source falls
// outside the row receive 0.
template <int J>
__device__ __forceinline__ uint32_t from_lane_minus(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x110 + J, 0xF, 0xF, false);
}
template <int J>
__device__ __forceinline__ float from_lane_minus_f(float v)
{
    return __uint_as_float(from_lane_minus<J>(__float_as_uint(v)));
}
// ---------------------------------------------------------------------------
// Distance policies. Each lane group computes one candidate's distance per
// round; rounds are unrolled by RU so that RU rows of loads are in flight.

// W = 2 is the variant for launches that hold few waves per CU (the
// escalation of a split search, and fused launches whose LDS admits no more
// waves than it does): twice the rows in flight per round trip and more, paid
// for in registers that such launches do not need for occupancy. W = 3 is the
// one of a team's helpers, between the two.
template <int T, int W = 1>
struct F32Scorer {
    // lane p = lane & 15 accumulates float4 chunks p, p+16, p+32, ...
    static constexpr bool kSpec = false;
    static constexpr int kSpecMaxR = 0;
    struct RowGather {};
    __device__ __forceinline__ void gather_row(const void *, int, uint32_t, int, int, RowGather &) const {}
    __device__ __forceinline__ void score_row(const RowGather &, int, int, float *, int) const {}
    // rows of more than 320 dimensions keep the query in LDS rather than in
    // 4T registers (every 16-lane group reads the same chunks: broadcasts)
    static constexpr bool kQueryLds = T >= 6;
    static constexpr int kLdsBytes = kQueryLds ? 16 * T * 16 : 0;
    static constexpr bool kPQ = false;
    float4 q[kQueryLds ? 1 : T];
    float4 *ql = nullptr;

    __device__ __forceinline__ void bind_lds(void *buf) { ql = reinterpret_cast<float4 *>(buf); }

    __device__ __forceinline__ float4 qchunk(int t, int p) const
    {
        if constexpr (kQueryLds) return ql[p + 16 * t];
        else return q[t];
    }

    __device__ __forceinline__ void load_query(const void *Q, uint32_t qi, int d, int lane)
    {
        const float4 *qq = reinterpret_cast<const float4 *>(reinterpret_cast<const float *>(Q) + (size_t)qi * d);
        int p = lane & 15, nch = d >> 2;
        if constexpr (kQueryLds) {
            // chunks 0 .. 16T-1, zero past the row (the caller's wave_sync
            // orders these writes before the reads)
            for (int cc = lane; cc < 16 * T; cc += 64) ql[cc] = cc < nch ? qq[cc] : make_float4(0.f, 0.f, 0.f, 0.f);
        } else {
#pragma unroll
            for (int t = 0; t < T; ++t) {
                int cc = p + 16 * t;
                q[t] = cc < nch ? qq[cc] : make_float4(0.f, 0.f, 0.f, 0.f);
            }
        }
    }

    // rows in flight per round trip: the narrow variant keeps registers for
    // occupancy; the wide one covers most expansions in one round trip
    static constexpr int RU = W == 1 ? (T <= 2 ? 4 : (T <= 4 ? 2 : 1))
                              : W == 3 ? (T <= 2 ? 8 : (T <= 4 ? 4 : 2))
                                       : (T <= 2 ? 16 : (T <= 4 ? 8 : (T <= 6 ? 4 : (T <= 12 ? 2 : 1))));
    // waves per SIMD a team launch's registers leave room for
    static constexpr int kTeamWaves = T <= 4 ? 4 : 2;
    // ... and a launch with one wave per query
    static constexpr int kWaves = W == 1 ? (T <= 8 ? 3 : 2) : 1;
    struct Ids {
        uint32_t v[RU];
    };

    // candidate ids of the round starting at r0 (independent LDS reads; a
    // lane past the candidates takes candidate 0)
    __device__ __forceinline__ void read_ids(const uint32_t *cid, int c, int r0, int lane, Ids &ids) const
    {
        const int g = lane >> 4;
#pragma unroll
        for (int u = 0; u < RU; ++u) {
            const int cj = r0 + 4 * u + g;
            ids.v[u] = cid[cj < c ? cj : 0];
        }
    }

    // `first` holds the ids of the first round, read by the caller together
    // with its own reads of the candidate list
    __device__ __forceinline__ void score(const void *V, int d, const uint32_t *cid, int c, float *cd, int lane,
                                          const Ids &first)
    {
        const float *vec = reinterpret_cast<const float *>(V);
        const int g = lane >> 4, p = lane & 15, nch = d >> 2;
        for (int r0 = 0; r0 < c; r0 += 4 * RU) {
            // the rows: unconditional loads from valid global addresses (a
            // chunk past the row end re-reads its last chunk), masked afterwards
            Ids ids = first;
            if (r0 > 0) read_ids(cid, c, r0, lane, ids);
            const uint32_t *idv = ids.v;
            float4 x[RU][T];
#pragma unroll
            for (int u = 0; u < RU; ++u) {
                if (r0 + 4 * u < c) {   // uniform: a candidate left in this round
                    const float4 *row = reinterpret_cast<const float4 *>(vec + (size_t)idv[u] * d);
#pragma unroll
                    for (int t = 0; t < T; ++t) {
                        const int cc = p + 16 * t;
                        x[u][t] = row[cc < nch ? cc : nch - 1];
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < RU; ++u) {
                if (r0 + 4 * u >= c) break;   // uniform: no candidate left in this round
                const float acc = dist(x[u], p, nch);
                const int cj = r0 + 4 * u + g;
                if (p == 15 && cj < c) cd[cj] = acc;
            }
        }
    }

    // squared distance of one row held by a 16-lane group (chunk p + 16 t in
    // x[t]); lane 15 of the group returns it
    __device__ __forceinline__ float dist(float4 (&x)[T], int p, int nch) const
    {
        float acc = 0.0f;
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const float4 qv = qchunk(t, p);
            if (p + 16 * t >= nch) x[t] = qv;   // past the row end: adds zero
            float a0 = x[t].x - qv.x;
            acc = __builtin_fmaf(a0, a0, acc);
            float a1 = x[t].y - qv.y;
            acc = __builtin_fmaf(a1, a1, acc);
            float a2 = x[t].z - qv.z;
            acc = __builtin_fmaf(a2, a2, acc);
            float a3 = x[t].w - qv.w;
            acc = __builtin_fmaf(a3, a3, acc);
        }
        // pairwise tree over the 16 partials (p += p+8, +4, +2, +1), mirrored
        // onto the row's top lanes: lane 15 ends with the same sums in the
        // same order (each add is commutative)
        acc = acc + from_lane_minus_f<8>(acc);
        acc = acc + from_lane_minus_f<4>(acc);
        acc = acc + from_lane_minus_f<2>(acc);
        acc = acc + from_lane_minus_f<1>(acc);
        return acc;
    }
};

template <int G, int W = 1>
struct U8Scorer {
    // lane p = lane % G holds the query's 16-byte chunk p (p < d/16); the
    // exact int32 sum is order-free. Per chunk, |x - q|^2 = x.x - 2 x.q + q.q
    // from unsigned 4-byte dot products: every term is an exact integer
    // (at most 16 * 255^2 per lane), so the result is the exact sum of
    // squared differences.
    // rows of at most 128 bytes gather every neighbour of an expanded node
    // before its visited test (gather_row / score_row below)
    static constexpr bool kSpec = G <= 8;
    static constexpr int kTeamWaves = G <= 16 ? 4 : 2;
    static constexpr int kWaves = W == 1 || G <= 8 ? 3 : 1;
    static constexpr int kLdsBytes = 0;
    static constexpr bool kPQ = false;
    uint4 q;
    uint32_t qq;   // q.q of this lane's chunk

    __device__ __forceinline__ void bind_lds(void *) {}

    __device__ __forceinline__ void load_query(const void *Q, uint32_t qi, int d, int lane)
    {
        const uint8_t *qb = reinterpret_cast<const uint8_t *>(Q) + (size_t)qi * d;
        int p = lane % G;
        q = p < (d >> 4) ? reinterpret_cast<const uint4 *>(qb)[p] : make_uint4(0, 0, 0, 0);
        qq = dot16(q, q);
    }

    static __device__ __forceinline__ uint32_t dot16(const uint4 &a, const uint4 &b)
    {
        uint32_t s = __builtin_amdgcn_udot4(a.x, b.x, 0u, false);
        s = __builtin_amdgcn_udot4(a.y, b.y, s, false);
        s = __builtin_amdgcn_udot4(a.z, b.z, s, false);
        return __builtin_amdgcn_udot4(a.w, b.w, s, false);
    }

    static constexpr int PER = 64 / G;   // candidates per round
    // rows in flight per round trip of score(); with row gathers it scores
    // only the entry point and rows longer than the gathers cover
    static constexpr int RU = (W == 1 || G <= 8) ? (G <= 8 ? 2 : 4) : (G <= 16 ? G : 16);
    struct Ids {
        uint32_t v[RU];
    };

    __device__ __forceinline__ void read_ids(const uint32_t *cid, int c, int r0, int lane, Ids &ids) const
    {
        const int g = lane / G;
#pragma unroll
        for (int u = 0; u < RU; ++u) {
            const int cj = r0 + PER * u + g;
            ids.v[u] = cid[cj < c ? cj : 0];
        }
    }

    __device__ __forceinline__ void score(const void *V, int d, const uint32_t *cid, int c, float *cd, int lane,
                                          const Ids &first)
    {
        const uint8_t *vec = reinterpret_cast<const uint8_t *>(V);
        const int g = lane / G, p = lane % G, nch = d >> 4;
        for (int r0 = 0; r0 < c; r0 += PER * RU) {
            // unconditional loads from valid addresses, masked afterwards (as
            // in F32Scorer)
            Ids ids = first;
            if (r0 > 0) read_ids(cid, c, r0, lane, ids);
            const uint32_t *idv = ids.v;
            uint4 x[RU];
#pragma unroll
            for (int u = 0; u < RU; ++u) {
                if (r0 + PER * u < c)   // uniform
                    x[u] = reinterpret_cast<const uint4 *>(vec + (size_t)idv[u] * d)[p < nch ? p : nch - 1];
            }
#pragma unroll
            for (int u = 0; u < RU; ++u) {
                if (r0 + PER * u >= c) break;   // uniform: no candidate left in this round
                const int32_t acc = dist(x[u], p, nch);
                const int cj = r0 + PER * u + g;
                if (p == G - 1 && cj < c) cd[cj] = (float)acc;
            }
        }
    }

    // Every neighbour of an expanded node, before its visited test: lane j
    // holds row entry j (padding replaced by a valid id), and round u's
    // G-lane group g loads chunk p of entry PER u + g. All rounds' loads are
    // issued together; score_row waits for them.
    static constexpr int RS_ALL = (BOA_MAX_R + PER - 1) / PER;
    static constexpr int RS = !kSpec ? 1 : (RS_ALL < 4 ? RS_ALL : 4);
    static constexpr int kSpecMaxR = kSpec ? PER * RS : 0;   // longer rows take the other path
    struct RowGather {
        uint4 x[RS];
    };

    __device__ __forceinline__ void gather_row(const void *V, int d, uint32_t v, int R, int lane,
                                               RowGather &rg) const
    {
        const uint8_t *vec = reinterpret_cast<const uint8_t *>(V);
        const int g = lane / G, p = lane % G, nch = d >> 4;
        // every round's id first (cross-lane reads in flight together), then
        // the loads
        uint32_t id[RS];
#pragma unroll
        for (int u = 0; u < RS; ++u) id[u] = (uint32_t)__shfl((int)v, (PER * u + g) & 63);
#pragma unroll
        for (int u = 0; u < RS; ++u) {
            if (PER * u < R)   // uniform
                rg.x[u] = reinterpret_cast<const uint4 *>(vec + (size_t)id[u] * d)[p < nch ? p : nch - 1];
        }
    }

    // distances of the gathered entries: cd[j] for j < R
    __device__ __forceinline__ void score_row(const RowGather &rg, int d, int R, float *cd, int lane) const
    {
        const int g = lane / G, p = lane % G, nch = d >> 4;
#pragma unroll
        for (int u = 0; u < RS; ++u) {
            if (PER * u >= R) break;   // uniform
            const int32_t acc = dist(rg.x[u], p, nch);
            const int cj = PER * u + g;
            if (p == G - 1) cd[cj] = (float)acc;   // (cj < 64: slots past R are not read)
        }
    }

    // exact squared distance of one row held by a G-lane group (16-byte
    // chunk p in x); the group's top lane returns it
    __device__ __forceinline__ int32_t dist(uint4 x, int p, int nch) const
    {
        int32_t acc = (int32_t)(dot16(x, x) + qq - 2u * dot16(x, q));
        if (nch < G) {         // (uniform) lanes past the row add zero
            if (p >= nch) acc = 0;
        }
        // exact integer sum over the group; the group's top lane holds it
#pragma unroll
        for (int s = G >> 1; s >= 16; s >>= 1) acc += __shfl_xor(acc, s);
        if (G >= 16) acc += (int32_t)from_lane_minus<8>((uint32_t)acc);
        if (G >= 8) acc += (int32_t)from_lane_minus<4>((uint32_t)acc);
        if (G >= 4) acc += (int32_t)from_lane_minus<2>((uint32_t)acc);
        if (G >= 2) acc += (int32_t)from_lane_minus<1>((uint32_t)acc);
        return acc;
    }
};

// Product-quantised asymmetric distance (Alg. 2 "PQDist"): 4-bit codes, 16
// centroids per subspace. The query's distance table (M x 16 float32) lives
// in LDS; a 16-lane group scores one candidate, lane p adding the entries of
// subspaces p, p+16, ... in increasing order (nibble (p + 16t) of the packed
// code), then the same pairwise tree as the exact float32 distance.
//
// A code is read as 16-byte chunks (rows are padded to whole ones), chunk c by
// lane c of the group, in one load per candidate and 32 candidates per round
// trip; the nibbles then reach their lanes by row broadcasts, two per 16
// subspaces. (A byte load per 16 subspaces and lane, eight candidates per
// round trip, took 11,800 cycles of an expansion at M = 192.)
template <int T>
struct PQScorer {
    static constexpr bool kSpec = false;
    static constexpr int kSpecMaxR = 0;
    static constexpr int kTeamWaves = 4;
    static constexpr int kWaves = 2;
    struct RowGather {};
    __device__ __forceinline__ void gather_row(const void *, int, uint32_t, int, int, RowGather &) const {}
    __device__ __forceinline__ void score_row(const RowGather &, int, int, float *, int) const {}
    static constexpr bool kPQ = true;
    static constexpr int kLdsBytes = 16 * T * 16 * 4;   // the table of up to 16 T subspaces
    float *lut = nullptr;
    const uint8_t *codes = nullptr;
    const float *cb = nullptr;
    int M = 0, row = 0, ds = 0, u8 = 0;

    __device__ __forceinline__ void bind_lds(void *buf) { lut = reinterpret_cast<float *>(buf); }
    __device__ __forceinline__ void bind_pq(const uint8_t *c, int m, const float *codebook, int d, int vec_u8)
    {
        codes = c;
        M = m;
        row = pq_row_bytes(m);
        cb = codebook;
        ds = d / m;
        u8 = vec_u8;
    }

    // table entry (m, c): fma chain over the subspace's dimensions from +0;
    // zero past the M-th subspace, which adds nothing (the caller orders
    // these writes before the reads). Entries first, first + step, ...
    __device__ __forceinline__ void load_table(const void *Q, uint32_t qi, int d, int first, int step)
    {
        for (int e = first; e < 16 * T * 16; e += step) {
            const int m = e >> 4, c = e & 15;
            float acc = 0.0f;
            for (int j = 0; m < M && j < ds; ++j) {
                const size_t qo = (size_t)qi * d + m * ds + j;
                const float qv = u8 ? (float)reinterpret_cast<const uint8_t *>(Q)[qo]
                                    : reinterpret_cast<const float *>(Q)[qo];
                const float diff = qv - cb[((size_t)m * 16 + c) * ds + j];
                acc = __builtin_fmaf(diff, diff, acc);
            }
            lut[e] = acc;
        }
    }
    __device__ __forceinline__ void load_query(const void *Q, uint32_t qi, int d, int lane)
    {
        load_table(Q, qi, d, lane, 64);
    }

    static constexpr int RU = 8;   // rounds of 4 candidates per round trip
    struct Ids {
        uint32_t v[RU];
    };

    __device__ __forceinline__ void read_ids(const uint32_t *cid, int c, int r0, int lane, Ids &ids) const
    {
        const int g = lane >> 4;
#pragma unroll
        for (int u = 0; u < RU; ++u) {
            const int cj = r0 + 4 * u + g;
            ids.v[u] = cid[cj < c ? cj : 0];
        }
    }

    // the t-th term of the lane's sum: dword 2 t + (p >> 3) of the code holds
    // its nibble, in chunk t / 2
    template <int TT>
    __device__ __forceinline__ void add_terms(const uint4 &x, const float *mine, int shift, float &acc) const
    {
        if constexpr (TT < T) {
            const uint32_t lo = (TT & 1) ? x.z : x.x, hi = (TT & 1) ? x.w : x.y;
            int w = __builtin_amdgcn_update_dpp(0, (int)lo, 0x150 + TT / 2, 0xF, 0xF, false);   // row_newbcast
            w = __builtin_amdgcn_update_dpp(w, (int)hi, 0x150 + TT / 2, 0xF, 0xC, false);       // (lanes 8-15)
            acc = acc + mine[TT * 256 + (((uint32_t)w >> shift) & 15u)];
            add_terms<TT + 1>(x, mine, shift, acc);
        }
    }

    __device__ __forceinline__ void score(const void *, int, const uint32_t *cid, int c, float *cd, int lane,
                                          const Ids &first)
    {
        const int g = lane >> 4, p = lane & 15;
        const float *mine = lut + p * 16;
        const int shift = 4 * (p & 7);
        const int chunk = 16 * min(p, (row >> 4) - 1);
        for (int r0 = 0; r0 < c; r0 += 4 * RU) {
            Ids ids = first;
            if (r0 > 0) read_ids(cid, c, r0, lane, ids);
            uint4 x[RU];
#pragma unroll
            for (int u = 0; u < RU; ++u)
                if (r0 + 4 * u < c)   // uniform
                    x[u] = *reinterpret_cast<const uint4 *>(codes + (size_t)ids.v[u] * row + chunk);
#pragma unroll
            for (int u = 0; u < RU; ++u) {
                if (r0 + 4 * u >= c) break;   // uniform
                float acc = 0.0f;
                add_terms<0>(x[u], mine, shift, acc);
                acc = acc + from_lane_minus_f<8>(acc);
                acc = acc + from_lane_minus_f<4>(acc);
                acc = acc + from_lane_minus_f<2>(acc);
                acc = acc + from_lane_minus_f<1>(acc);
                const int cj = r0 + 4 * u + g;
                if (p == 15 && cj < c) cd[cj] = acc;
            }
        }
    }
};

// The re-rank of a product-quantised search: keys (exact distance bits, id) of
// the worklist's first n entries, by 16-lane groups in the fixed order of the
// float32 path (lane p: chunks p, p+16, ..., then pairwise), or exactly in
// int32 for uint8 vectors; 16 entries at a time, each row read in whole lines.
__device__ __forceinline__ void exact_keys(const PhaseArgs &a, uint32_t qi, const uint64_t *beam, uint32_t n,
                                           uint64_t *out, int lane)
{
    const int d = a.ix.d, g = lane >> 4, p = lane & 15;
    constexpr int RU = 4;
    for (uint32_t e0 = 0; e0 < n; e0 += 4 * RU) {
        uint32_t id[RU];
#pragma unroll
        for (int u = 0; u < RU; ++u) id[u] = key_id(beam[min(e0 + 4u * u + (uint32_t)g, n - 1u)]);
        float dist[RU];
        if (a.vec_u8) {
            const uint8_t *V = reinterpret_cast<const uint8_t *>(a.ix.vectors);
            const uint4 *q4 = reinterpret_cast<const uint4 *>(reinterpret_cast<const uint8_t *>(a.queries) + (size_t)qi * d);
            const int nch = d >> 4;
            uint32_t acc[RU] = {};
            for (int c0 = 0; c0 < nch; c0 += 16) {
                const int c = min(c0 + p, nch - 1);
                const uint4 qv = q4[c];
                const uint32_t qq = U8Scorer<1>::dot16(qv, qv);
#pragma unroll
                for (int u = 0; u < RU; ++u) {
                    const uint4 x = reinterpret_cast<const uint4 *>(V + (size_t)id[u] * d)[c];
                    const uint32_t t = U8Scorer<1>::dot16(x, x) + qq - 2u * U8Scorer<1>::dot16(x, qv);
                    acc[u] += c0 + p < nch ? t : 0u;
                }
            }
#pragma unroll
            for (int u = 0; u < RU; ++u) {
                acc[u] += from_lane_minus<8>(acc[u]);
                acc[u] += from_lane_minus<4>(acc[u]);
                acc[u] += from_lane_minus<2>(acc[u]);
                acc[u] += from_lane_minus<1>(acc[u]);
                dist[u] = (float)(int32_t)acc[u];
            }
        } else {
            const float *V = reinterpret_cast<const float *>(a.ix.vectors);
            const float4 *q4 = reinterpret_cast<const float4 *>(reinterpret_cast<const float *>(a.queries) + (size_t)qi * d);
            const int nch = d >> 2;
            float acc[RU] = {};
#pragma unroll 2
            for (int c0 = 0; c0 < nch; c0 += 16) {
                const int c = min(c0 + p, nch - 1);
                const float4 qv = q4[c];
#pragma unroll
                for (int u = 0; u < RU; ++u) {
                    float4 x = reinterpret_cast<const float4 *>(V + (size_t)id[u] * d)[c];
                    if (c0 + p >= nch) x = qv;   // past the row end: adds zero
                    float t = x.x - qv.x;
                    acc[u] = __builtin_fmaf(t, t, acc[u]);
                    t = x.y - qv.y;
                    acc[u] = __builtin_fmaf(t, t, acc[u]);
                    t = x.z - qv.z;
                    acc[u] = __builtin_fmaf(t, t, acc[u]);
                    t = x.w - qv.w;
                    acc[u] = __builtin_fmaf(t, t, acc[u]);
                }
            }
#pragma unroll
            for (int u = 0; u < RU; ++u) {
                acc[u] = acc[u] + from_lane_minus_f<8>(acc[u]);
                acc[u] = acc[u] + from_lane_minus_f<4>(acc[u]);
                acc[u] = acc[u] + from_lane_minus_f<2>(acc[u]);
                acc[u] = acc[u] + from_lane_minus_f<1>(acc[u]);
                dist[u] = acc[u];
            }
        }
#pragma unroll
        for (int u = 0; u < RU; ++u) {
            const uint32_t e = e0 + 4u * u + (uint32_t)g;
            if (p == 15 && e < n) out[e] = ((uint64_t)__float_as_uint(dist[u]) << 32) | id[u];
        }
    }
}

__device__ __forceinline__ uint64_t wave_min64(uint64_t v)
{
#pragma unroll
    for (int s = 32; s >= 1; s >>= 1) {
        const uint64_t o = ((uint64_t)(uint32_t)__shfl_xor((int)(uint32_t)(v >> 32), s) << 32) |
                           (uint32_t)__shfl_xor((int)(uint32_t)v, s);
        v = o < v ? o : v;
    }
    return v;
}

// ---------------------------------------------------------------------------
// Attribute filter (Eq. 2). A point's record is m_pad cells, loaded as one
// aligned vector load (int4 halves w0, w1). The index holds float32 cells
// as order-preserving integers (f32_ord), and RangeTest maps each query's
// bounds the same way, so a cell satisfies its range [lo, hi] exactly when
// (uint32)(x - lo) <= hi - lo. A range that nothing satisfies (lo > hi, or a
// NaN bound of a float32 column, which fails every comparison) counts in
// phi0 for every point; its cell, like a padding cell, then passes.

__device__ __forceinline__ void load_attr_record(const IndexView &ix, uint32_t id, int4 &w0, int4 &w1)
{
    const int32_t *ar = ix.attrs + (size_t)id * ix.m_pad;
    if (ix.m_pad >= 4) {
        w0 = reinterpret_cast<const int4 *>(ar)[0];
        if (ix.m_pad == 8) w1 = reinterpret_cast<const int4 *>(ar)[1];
    } else if (ix.m_pad == 2) {
        const int2 t2 = reinterpret_cast<const int2 *>(ar)[0];
        w0.x = t2.x;
        w0.y = t2.y;
    } else {
        w0.x = ar[0];
    }
}

// The bounds stay in lane j of two registers, column j's, and are read back as
// scalars where a cell is tested (held in all lanes they take 16 registers, and
// as scalars across the search they spill).
struct RangeTest {
    int32_t l;
    uint32_t s;
    uint32_t phi0;

    // query qi's m ranges (row-major nq x m x 2 cells)
    __device__ __forceinline__ void set(const int32_t *ranges, uint32_t qi, int m, uint32_t f32_mask)
    {
        const int lane = lane_id();
        l = 0;
        s = 0xFFFFFFFFu;   // (padding cells pass)
        bool none = false;
        if (lane < m) {
            const int32_t *r = ranges + ((size_t)qi * m + lane) * 2;
            int32_t lo = r[0], hi = r[1];
            if ((f32_mask >> lane) & 1u) {
                none = ((uint32_t)lo & 0x7FFFFFFFu) > 0x7F800000u || ((uint32_t)hi & 0x7FFFFFFFu) > 0x7F800000u;
                lo = f32_ord((uint32_t)lo);
                hi = f32_ord((uint32_t)hi);
            }
            none |= lo > hi;
            if (!none) {
                l = lo;
                s = (uint32_t)hi - (uint32_t)lo;
            }
        }
        phi0 = (uint32_t)__popcll(__ballot(none));
    }

    // phi of a record: its m_pad cells (one uniform dispatch, no per-cell tests)
    __device__ __forceinline__ uint32_t phi(const int4 &w0, const int4 &w1, int m_pad) const
    {
        const int32_t av[BOA_MAX_M] = {w0.x, w0.y, w0.z, w0.w, w1.x, w1.y, w1.z, w1.w};
        auto cells = [&](auto nc_tag) -> uint32_t {
            constexpr int NC = decltype(nc_tag)::value;
            uint32_t p = phi0;
#pragma unroll
            for (int j = 0; j < NC; ++j) {
                const int32_t lj = __builtin_amdgcn_readlane(l, j);
                const uint32_t sj = (uint32_t)__builtin_amdgcn_readlane((int)s, j);
                p += (uint32_t)(av[j] - lj) > sj ? 1u : 0u;
            }
            return p;
        };
        switch (m_pad) {
        case 1: return cells(std::integral_constant<int, 1>{});
        case 2: return cells(std::integral_constant<int, 2>{});
        case 4: return cells(std::integral_constant<int, 4>{});
        default: return cells(std::integral_constant<int, 8>{});
        }
    }
};

// ---------------------------------------------------------------------------
// Visited set (exact). LDS part: a two-choice bucketed table of 16-bit
// entries. A bijective mix of the id's B bits gives h; its top bits select
// the home bucket b1, the low r = B - log2(buckets) <= 15 bits are stored.
// The alternate bucket is b2 = b1 ^ alt(r) (alt odd, so b2 != b1). An entry
// is r in b1 or 0x8000 | r in b2, so (bucket, entry) identifies the id
// uniquely; 0xFFFF marks a free slot, so an id whose r is 0x7FFF has no
// alternate bucket. A bucket holds 8 entries (16 bytes, one LDS read).
// Insert goes to the emptier bucket through a 32-bit CAS on the word that
// holds the slot. When both buckets are full the id goes to the wave slot's
// bitmap over all points in HBM (cleared when a query first overflows).
// Buckets only fill up, so an id absent from a bucket pair that still has
// room has never been inserted anywhere: the bitmap is consulted only when
// both buckets are full.
// The bitmap keeps a log of the ids whose bits were set since it was last
// clear, so that the clear rewrites only their words; when the log is full
// (or its state unknown, header BOA_LOG_DIRTY) the whole bitmap is cleared.
// The wave holds the log's length in a register and writes it back to the
// header when it exits.

struct Visited {
    uint32_t *words;     // LDS table, 2 entries per word, 4 words per bucket
    uint32_t bmask;      // buckets - 1
    uint32_t rbits;      // stored bits per id
    uint32_t idbits;     // B
    uint32_t *bits;      // this wave slot's HBM bitmap, words32 words
    uint32_t words32;
    uint32_t *log;       // its log: header word, then (after BOA_LOG_HDR words) log_cap ids
    uint32_t log_cap;
    uint32_t *status;
};

// ids have at most 24 bits (BOA_MAX_N), so 24-bit multiplies (full rate)
// by odd constants are bijections modulo 2^B
__device__ __forceinline__ uint32_t mix_id(uint32_t v, uint32_t B)
{
    const uint32_t mask = (1u << B) - 1u;
    uint32_t h = __umul24(v, 0x3779B1u) & mask;
    h ^= h >> ((B + 1u) >> 1);
    return __umul24(h, 0xEBCA6Bu) & mask;
}

// smaller of each pair of 16-bit halves (one packed instruction; written as
// vector arithmetic the compiler splits it into scalar halves)
__device__ __forceinline__ uint32_t pk_min_u16(uint32_t a, uint32_t b)
{
    uint32_t r;
    asm("v_pk_min_u16 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// whether one of the bucket's eight halves is e
__device__ __forceinline__ bool has16(const uint4 &b, uint32_t e)
{
    const uint32_t ee = e * 0x00010001u;
    const uint32_t m = pk_min_u16(pk_min_u16(b.x ^ ee, b.y ^ ee), pk_min_u16(b.z ^ ee, b.w ^ ee));
    return (m & 0xFFFFu) == 0u || m < 0x10000u;
}

// A bucket fills from its first half-word on and entries are never removed,
// so the free slots (0xFFFF) are a suffix: a word has a free slot when its
// upper half is one.
__device__ __forceinline__ bool word_free(uint32_t w) { return w >= 0xFFFF0000u; }
// wholly free words of a bucket (how empty it is, to two slots)
__device__ __forceinline__ uint32_t free_words(const uint4 &b)
{
    return (b.x == 0xFFFFFFFFu ? 1u : 0u) + (b.y == 0xFFFFFFFFu ? 1u : 0u) + (b.z == 0xFFFFFFFFu ? 1u : 0u) +
           (b.w == 0xFFFFFFFFu ? 1u : 0u);
}

// the two buckets an id may be in, and its stored bits
__device__ __forceinline__ void visit_slots(const Visited &s, uint32_t v, uint32_t &b1, uint32_t &b2, uint32_t &r)
{
    const uint32_t h = mix_id(v, s.idbits);
    r = h & ((1u << s.rbits) - 1u);
    b1 = h >> s.rbits;
    b2 = (b1 ^ (((__umul24(r, 0xD1E995u) + 0x7F4A7C15u) >> 7) | 1u)) & s.bmask;
}

// 1: v was not in the set and now is (in LDS); 0: v was already there;
// -1: both buckets full and v not in them (the caller consults the bitmap).
__device__ __forceinline__ int visit_lds(const Visited &s, uint32_t v)
{
    uint32_t b1, b2, r;
    visit_slots(s, v, b1, b2, r);
    const uint32_t e1 = r, e2 = 0x8000u | r;
    const bool alt_ok = e2 != 0xFFFFu;
    const uint4 *bk = reinterpret_cast<const uint4 *>(s.words);
    for (int attempt = 0; attempt < 256; ++attempt) {
        // both buckets read before either is tested: one LDS round trip
        const uint4 B1 = bk[b1], B2 = bk[b2];
        if (has16(B1, e1) || (alt_ok && has16(B2, e2))) return 0;
        const bool room1 = word_free(B1.w), room2 = alt_ok && word_free(B2.w);
        if (!room1 && !room2) return -1;
        // the emptier bucket, the home bucket when they are equally so
        const bool use1 = room1 && (!room2 || free_words(B1) >= free_words(B2));
        const uint4 Bc = use1 ? B1 : B2;
        const uint32_t e = use1 ? e1 : e2;
        const uint32_t bi = use1 ? b1 : b2;
        // the first free half: in the first word with one, its low half when
        // that one is free
        uint32_t wi = 3, old = Bc.w;
        if (word_free(Bc.z)) { wi = 2; old = Bc.z; }
        if (word_free(Bc.y)) { wi = 1; old = Bc.y; }
        if (word_free(Bc.x)) { wi = 0; old = Bc.x; }
        const uint32_t neu = old == 0xFFFFFFFFu ? (0xFFFF0000u | e) : ((old & 0xFFFFu) | (e << 16));
        if (atomicCAS(&s.words[bi * 4u + wi], old, neu) == old) return 1;
        // another lane changed that word: look again
    }
    atomicOr(s.status, BOA_STATUS_OVERFLOW);
    return 0;
}

__device__ __forceinline__ bool visit_bits(const Visited &s, uint32_t v)
{
    uint32_t bit = 1u << (v & 31u);
    uint32_t old = atomicOr(&s.bits[v >> 5], bit);
    return (old & bit) == 0u;
}

// Clear the bitmap before a query's first spill: the words of the n_log
// logged ids, or every word when the log does not cover the set bits.
__device__ __forceinline__ void clear_bits(const Visited &s, uint32_t n_log, int lane)
{
    if (n_log <= s.log_cap) {
        const uint32_t *ids = s.log + BOA_LOG_HDR;
        uint32_t i = lane;
        for (; i + 192 < n_log; i += 256) {   // four loads in flight, then their stores
            const uint32_t v0 = ids[i], v1 = ids[i + 64], v2 = ids[i + 128], v3 = ids[i + 192];
            s.bits[v0 >> 5] = 0u;
            s.bits[v1 >> 5] = 0u;
            s.bits[v2 >> 5] = 0u;
            s.bits[v3 >> 5] = 0u;
        }
        for (; i < n_log; i += 64) s.bits[ids[i] >> 5] = 0u;
    } else {
        uint4 z = make_uint4(0, 0, 0, 0);
        uint4 *b4 = reinterpret_cast<uint4 *>(s.bits);
        for (uint32_t i = lane; i < (s.words32 >> 2); i += 64) b4[i] = z;
    }
    // the stores must land before this wave's atomics on the same words
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
}

// The visited set of one query, written by one wave: the hashed table with its
// HBM bitmap, or (bitmap != 0) one LDS bit per id.
struct VisitSet {
    Visited s;
    uint32_t bitmap;
    uint32_t table_words;   // LDS words of either kind
    bool spill;             // this query has used the HBM bitmap
    uint32_t n_log;         // ids logged in this wave slot's HBM bitmap (its header,
                            // in a register: no other wave uses the slot meanwhile)

    __device__ __forceinline__ void bind(const PhaseArgs &a, uint32_t *lds, uint32_t slot)
    {
        s.words = lds;
        s.bmask = (1u << (a.h_log2 - 3)) - 1u;       // 8 slots per bucket
        s.idbits = a.id_bits;
        s.rbits = a.id_bits > (uint32_t)(a.h_log2 - 3) ? a.id_bits - (uint32_t)(a.h_log2 - 3) : 0u;
        s.words32 = a.bits_words;
        s.bits = a.bits + (size_t)slot * a.slot_words;
        s.log = s.bits + a.bits_words;
        s.log_cap = a.log_cap;
        s.status = a.status;
        bitmap = a.vis_bitmap;
        table_words = a.vis_bitmap ? a.vis_words : (1u << a.h_log2) >> 1;
        spill = false;
        n_log = 0;
    }
    __device__ __forceinline__ void open() { n_log = bitmap ? 0u : bcast0(s.log[0]); }
    __device__ __forceinline__ void close(int lane) const
    {
        if (!bitmap && lane == 0) s.log[0] = n_log;
    }
    // empty set: the bitmap with no bit set, the table with every slot free
    __device__ __forceinline__ void clear(int lane)
    {
        const uint32_t f = bitmap ? 0u : 0xFFFFFFFFu;
        const uint4 z = make_uint4(f, f, f, f);
        uint4 *h4 = reinterpret_cast<uint4 *>(s.words);
        for (uint32_t i = lane; i < table_words >> 2; i += 64) h4[i] = z;
    }
    // the entry point, by one lane
    __device__ __forceinline__ void enter(uint32_t v) const
    {
        if (bitmap) s.words[v >> 5] |= 1u << (v & 31u);
        else visit_lds(s, v);
    }
    // test-and-insert of this lane's id: 1 new, 0 seen (or padding)
    __device__ __forceinline__ int test(uint32_t v, int lane)
    {
        if (bitmap) {   // one bit per id: a single LDS atomic
            if (v == BOA_PAD) return 0;
            const uint32_t bit = 1u << (v & 31u);
            return (atomicOr(&s.words[v >> 5], bit) & bit) ? 0 : 1;
        }
        int vst = 0;
        if (v != BOA_PAD) vst = visit_lds(s, v);
        if (__ballot(vst < 0) != 0ull) {
            if (!spill) {          // first overflow of this query: reset the bitmap
                spill = true;
                clear_bits(s, n_log, lane);
                n_log = 0;
            }
            const bool to_bits = vst < 0;
            if (to_bits) vst = visit_bits(s, v) ? 1 : 0;
            // log the ids whose bits this wave has just set
            const uint64_t lm = __ballot(to_bits && vst > 0);
            if (lm) {
                const uint32_t cnt = (uint32_t)__popcll(lm);
                if (n_log <= s.log_cap && cnt <= s.log_cap - n_log) {
                    if (to_bits && vst > 0) s.log[BOA_LOG_HDR + n_log + lanes_below(lm)] = v;
                    n_log += cnt;
                } else {
                    n_log = BOA_LOG_DIRTY;
                }
            }
        }
        return vst;
    }
    // Whether the LDS part holds an id: true only for ids in the set, also
    // while the set's own wave inserts others (an entry is written as a whole
    // word and never changes until the set is cleared).
    __device__ __forceinline__ bool holds(uint32_t v) const
    {
        if (bitmap) return (s.words[v >> 5] >> (v & 31u)) & 1u;
        uint32_t b1, b2, r;
        visit_slots(s, v, b1, b2, r);
        const uint4 *bk = reinterpret_cast<const uint4 *>(s.words);
        const uint4 B1 = bk[b1], B2 = bk[b2];
        return has16(B1, r) || (r != 0x7FFFu && has16(B2, 0x8000u | r));
    }
};

// ---------------------------------------------------------------------------
// The worklist of Alg. 2, held by one wave: a sorted list in LDS and up to 64
// pending keys, one per lane, not yet merged into it.
//
// The worklist at any time is the Lcap smallest keys entered so far, so it is
// the same whenever the merge into the sorted list happens, and a key that
// has Lcap smaller ones can be dropped at any later time. The next node to
// expand is the smallest unexpanded key of both parts, provided fewer than L
// keys are smaller (else every entry among the first L is expanded and the
// phase has converged). So the pending keys are merged only when the next
// batch does not fit the 64 lanes, or when that count cannot be told without
// it. A merge (sort by counting, search, rebuild of up to Lcap entries) costs
// several times a selection, and at widths of 100 and more it is needed once
// in 4 to 15 expansions instead of at every one.

// Smallest of 64 lanes' values: DPP steps inside the rows of 16, then across
// the rows; a lane without a source keeps its own value, lane 63 ends with the
// result. (In one block: each step reads what the one before wrote, two wait
// states later, and the compiler's own form of it takes a move more per step.)
__device__ __forceinline__ uint32_t wave_min32(uint32_t v)
{
    asm("s_nop 1\n\t"
        "v_min_u32_dpp %0, %0, %0 row_shr:1 row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1\n\t"
        "v_min_u32_dpp %0, %0, %0 row_shr:2 row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1\n\t"
        "v_min_u32_dpp %0, %0, %0 row_shr:4 row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1\n\t"
        "v_min_u32_dpp %0, %0, %0 row_shr:8 row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1\n\t"
        "v_min_u32_dpp %0, %0, %0 row_bcast:15 row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1\n\t"
        "v_min_u32_dpp %0, %0, %0 row_bcast:31 row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1"
        : "+v"(v));
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}
// The smallest key without the expanded flag (KEY_NONE, which has it set, if
// there is none). The upper halves decide unless they tie.
__device__ __forceinline__ uint64_t wave_min_open(uint64_t key)
{
    const uint32_t hi = (key & 1ull) ? 0xFFFFFFFFu : (uint32_t)(key >> 32);
    const uint32_t m = wave_min32(hi);
    if (m == 0xFFFFFFFFu) return KEY_NONE;
    const uint64_t eq = __ballot(hi == m);
    uint32_t lo;
    if ((eq & (eq - 1ull)) == 0ull)
        lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)key, __ffsll((unsigned long long)eq) - 1);
    else
        lo = wave_min32(hi == m ? (uint32_t)key : 0xFFFFFFFFu);
    return ((uint64_t)m << 32) | lo;
}

static constexpr int NEXT_NONE = 0, NEXT_FOUND = 1, NEXT_MERGE = 2;

struct WaveList {
    uint64_t *beam;      // sorted entries [0, len), KEY_NONE up to the next power of two
    uint64_t *nkey;      // 64
    uint64_t *posbm;     // output-slot bitmap of a merge
    uint32_t len, L, Lcap;
    uint64_t thr;        // with len == Lcap: the last entry, which a new key must beat
    uint32_t pn;         // pending keys: lanes [0, pn) of pend, KEY_NONE in the others
    uint64_t pend;
    uint64_t pmin;       // the smallest unexpanded one
    // window on the sorted list: win = beam[wb + lane], wmask its unexpanded
    // lanes; every entry below wb and below the first set bit is expanded
    uint32_t wb;
    uint64_t win, wmask;

    __device__ __forceinline__ uint32_t limit() const { return min(len, L); }
    __device__ __forceinline__ void clear(int Lb, int lane)
    {
        for (int i = lane; i < Lb; i += 64) beam[i] = KEY_NONE;
        len = 0;
    }
    // start of a phase on a list without pending keys
    __device__ __forceinline__ void begin(int L_, int Lcap_, int lane)
    {
        L = (uint32_t)L_;
        Lcap = (uint32_t)Lcap_;
        len = bcast0(len);
        pn = 0;
        pend = KEY_NONE;
        pmin = KEY_NONE;
        set_thr();
        scan(0, lane);
    }
    __device__ __forceinline__ void set_thr()
    {
        thr = len == Lcap ? readlane64(beam[Lcap - 1u], 0) : KEY_NONE;
    }
    __device__ __forceinline__ void scan(uint32_t from, int lane)
    {
        const uint32_t lim = limit();
        wmask = 0ull;
        for (wb = from; wb < lim; wb += 64) {
            const uint32_t i = wb + lane;
            win = i < lim ? beam[i] : 1ull;
            wmask = __ballot(!(win & 1ull));
            if (wmask) break;
        }
    }
    // first unexpanded sorted entry (its index: the limit if there is none)
    __device__ __forceinline__ uint32_t first_index() const
    {
        return wmask ? wb + (uint32_t)__ffsll((unsigned long long)wmask) - 1u : limit();
    }
    __device__ __forceinline__ uint64_t first_key() const
    {
        return wmask ? readlane64(win, __ffsll((unsigned long long)wmask) - 1) : KEY_NONE;
    }
    // new keys that can still enter
    __device__ __forceinline__ uint64_t filter(uint64_t key) const { return key < thr ? key : KEY_NONE; }

    // The next node to expand (its key in x), marked as expanded in its place:
    // the pending keys, the sorted list, or the caller's new keys nk (not yet
    // added). NEXT_NONE: converged. NEXT_MERGE: not known before a merge.
    __device__ __forceinline__ int next(uint64_t &nk, uint64_t &x, int lane)
    {
        const uint64_t m = wave_min_open(nk);
        const uint64_t s = first_key();
        x = s < pmin ? s : pmin;
        x = m < x ? m : x;
        if (x == KEY_NONE) return NEXT_NONE;
        const uint32_t j = first_index();
        if (j + pn >= L) {
            // smaller keys: j sorted ones (an upper bound unless the node is
            // the sorted list's own) and the expanded pending ones
            const uint32_t below = j + (uint32_t)__popcll(__ballot(pend < x));
            if (below >= L) return x == s ? NEXT_NONE : NEXT_MERGE;
        }
        if (x == s) {
            const int l = __ffsll((unsigned long long)wmask) - 1;
            wave_sync();
            if (lane == 0) beam[wb + (uint32_t)l] = x | 1ull;
            wave_sync();
            wmask &= wmask - 1ull;
            if (!wmask) scan(wb + 64u, lane);
        }
        if (pend == x) pend |= 1ull;
        if (nk == x) nk |= 1ull;
        return NEXT_FOUND;
    }
    // Enter the new keys (one per lane, KEY_NONE elsewhere; none kept after),
    // merging the pending ones first if they do not fit beside them; flush:
    // merge in any case (pn > 0 afterwards: flush again).
    __device__ __forceinline__ void add(uint64_t &nk, bool flush, int lane)
    {
        bool full = false;
        for (;;) {
            const uint64_t am = __ballot(nk != KEY_NONE);
            const uint32_t cnt = (uint32_t)__popcll(am);
            if (!full && (pn + cnt > 64u || (flush && cnt == 0u))) {
                merge(lane);
                nk = filter(nk);
                full = true;
                continue;
            }
            if (cnt != 0u) {
                if (nk != KEY_NONE) nkey[pn + lanes_below(am)] = nk;
                wave_sync();
                if ((uint32_t)lane - pn < cnt) pend = nkey[lane];
                wave_sync();
                pn += cnt;
                nk = KEY_NONE;
                if (flush && !full) continue;
            }
            pmin = wave_min_open(pend);
            return;
        }
    }
    // merge the pending keys into the sorted list
    __device__ __forceinline__ void merge(int lane)
    {
        uint64_t key = filter(pend);
        pn = 0;
        pend = KEY_NONE;
        const uint64_t keep = __ballot(key != KEY_NONE);
        const uint32_t kept = __popcll(keep);
        if (kept == 0) return;
        const uint32_t cursor = first_index();
        // sort the keys: each one's rank is the number of keys below it (they
        // are distinct), read back from LDS as broadcasts, two keys per read;
        // the other lanes' KEY_NONE after them, so that reads past the keys
        // compare false
        nkey[key != KEY_NONE ? lanes_below(keep) : kept + lanes_below(~keep)] = key;
        wave_sync();
        uint32_t rank = 0;
        {
            // eight keys per step: four independent LDS reads in flight
            const ulonglong2 *nk2 = reinterpret_cast<const ulonglong2 *>(nkey);
            for (uint32_t i = 0; i < kept; i += 8) {
                const ulonglong2 a0 = nk2[(i >> 1) + 0], a1 = nk2[(i >> 1) + 1];
                const ulonglong2 a2 = nk2[(i >> 1) + 2], a3 = nk2[(i >> 1) + 3];
                rank += (a0.x < key ? 1u : 0u) + (a0.y < key ? 1u : 0u);
                rank += (a1.x < key ? 1u : 0u) + (a1.y < key ? 1u : 0u);
                rank += (a2.x < key ? 1u : 0u) + (a2.y < key ? 1u : 0u);
                rank += (a3.x < key ? 1u : 0u) + (a3.y < key ? 1u : 0u);
            }
        }
        wave_sync();
        if (key != KEY_NONE) nkey[rank] = key;
        wave_sync();
        key = lane < (int)kept ? nkey[lane] : KEY_NONE;
        // rank of each new key in the list and its output slot
        uint32_t f = 0xFFFFFFFFu;
        uint32_t pos = 0;
        if (lane < (int)kept) {
            pos = lower_bound64_p2(beam, (uint32_t)beam_slots((int32_t)len), key);
            f = pos + lane;
        }
        const uint32_t p0 = bcast0(pos);
        const uint32_t newlen = min(Lcap, len + kept);
        const uint32_t w_lo = bcast0(p0 >> 6), w_hi = bcast0((newlen - 1u) >> 6);
        for (uint32_t w = w_lo + lane; w <= w_hi; w += 64) posbm[w] = 0ull;
        wave_sync();
        const bool placed = f < Lcap;
        if (placed) atomicOr(reinterpret_cast<unsigned long long *>(&posbm[f >> 6]), 1ull << (f & 63u));
        const uint32_t n_placed = __popcll(__ballot(placed));
        wave_sync();
        // rebuild [p0, newlen) from the last 64-slot chunk down
        uint64_t word = posbm[w_hi];
        uint32_t below = n_placed - (uint32_t)__popcll(word);   // new keys before the chunk
        for (int w = (int)w_hi; w >= (int)w_lo; --w) {
            const uint32_t o = ((uint32_t)w << 6) + lane;
            const bool act = o >= p0 && o < newlen;
            const bool isnew = (word >> lane) & 1ull;
            const uint32_t cnt = below + (uint32_t)__popcll(word & ((1ull << lane) - 1ull));
            uint64_t val = 0;
            if (act) val = isnew ? nkey[cnt] : beam[o - cnt];
            wave_sync();
            if (act) beam[o] = val;
            if (w > (int)w_lo) {
                word = posbm[w - 1];
                below -= (uint32_t)__popcll(word);
            }
            wave_sync();
        }
        len = bcast0(newlen);
        set_thr();
        scan(min(p0, cursor), lane);
    }
};

// ---------------------------------------------------------------------------

// The launch's arguments where they are needed once per query or phase: read
// again from the kernel's argument segment (a scalar load) instead of being
// held in scalar registers across the search, which spill.
__device__ __forceinline__ const PhaseArgs &cold_args()
{
    auto p = (const PhaseArgs __attribute__((address_space(4))) *)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return *(const PhaseArgs *)p;
}

// The end of a query's phase: Eq. 3 on its n_valid valid entries (d_k, d_max:
// squared distances of the k-th and the last), statistics, and the result if
// the phase is the query's last. result(q, id, dist) gives this lane the q-th
// valid entry.
template <class Result>
__device__ __forceinline__ bool end_phase(const PhaseArgs &a, int lane, int p, uint32_t qi, uint32_t t, int L,
                                          uint32_t n_valid, float d_k, float d_max, uint32_t E, uint32_t S,
                                          bool spill, Result &&result)
{
    const int k = a.k;
    uint32_t conf = 0;
    if (n_valid > (uint32_t)k) {
        const double dk = sqrt((double)d_k);
        const double dmax = sqrt((double)d_max);
        const double gamma = dmax == 0.0 ? 0.0 : (dmax - dk) / dmax;
        // (uniform, also for the compiler: a phase loop that lanes could
        // leave one by one would put every value it carries in vector
        // registers and every test on them under an execution mask)
        conf = bcast0(gamma <= a.eps ? 1u : 0u);
    }
    const bool last = conf != 0u || p + 1 == a.p_end;
    if (lane == 0) {
        const size_t ps = (size_t)p * a.nq + qi;
        if (a.qstat) {   // per-phase statistics (absent in the allocation-free search)
            a.qstat[ps] = (uint8_t)(1u + conf + (spill ? 4u : 0u));
            a.qE[ps] = E;
            a.qS[ps] = S;
        }
        if (a.user_E) a.user_E[qi] += E;
        if (a.user_S) a.user_S[qi] += S;
        if (a.write_conf) a.conf[t] = (uint8_t)conf;
        if (last) a.final_L[qi] = L;
    }
    if (last) {
        for (int q = lane; q < k; q += 64) {
            uint32_t id = BOA_PAD;
            float dd = __int_as_float(0x7f800000);
            if ((uint32_t)q < n_valid) result(q, id, dd);
            a.ids[(size_t)qi * k + q] = id;
            a.dists[(size_t)qi * k + q] = dd;
        }
    }
    return last;
}

// What the end of a phase reads of its worklist: the number of valid entries,
// the squared distances of the k-th and of the last, and the entries (lane q
// mod 64 holds the q-th of a re-ranked list).
template <class Scorer>
struct PhaseResult {
    uint32_t n_valid;
    float d_k, d_max;
    uint64_t key[2];
    const uint64_t *beam;

    // rrk: LDS for the exact keys of a product-quantised search (its distance
    // table's place: the table is loaded again if another phase follows)
    __device__ __forceinline__ void read(const PhaseArgs &a, const WaveList &wl, uint32_t qi, uint64_t *rrk, int lane)
    {
        beam = wl.beam;
        n_valid = bcast0(lower_bound64(beam, min(wl.len, wl.L), KEY_PHI1));
        const int k = a.k;
        d_k = d_max = 0.f;
        key[0] = key[1] = KEY_NONE;
        if constexpr (Scorer::kPQ) {
            // re-rank the valid entries by exact distance (Sec. III-B step 8):
            // keys (exact distance bits, id); the k smallest in order by k
            // rounds of a wave minimum, the largest by one wave maximum
            exact_keys(a, qi, beam, n_valid, rrk, lane);
            wave_sync();
            uint64_t prev = 0, mx = 0;
            for (uint32_t i = lane; i < n_valid; i += 64) mx = max(mx, rrk[i]);
            mx = ~wave_min64(~mx);
            const int kk = min(k, (int)n_valid);
            for (int q = 0; q < kk; ++q) {
                uint64_t mn = KEY_NONE;
                for (uint32_t i = lane; i < n_valid; i += 64) {
                    const uint64_t x = rrk[i];
                    if ((q == 0 || x > prev) && x < mn) mn = x;
                }
                mn = wave_min64(mn);
                if (q == lane) key[0] = mn;
                if (q == lane + 64) key[1] = mn;
                prev = mn;
            }
            if (kk > 0) d_k = __uint_as_float((uint32_t)(prev >> 32));
            d_max = __uint_as_float((uint32_t)(mx >> 32));
        } else if (n_valid > (uint32_t)k) {
            d_k = key_dist(beam[k - 1]);
            d_max = key_dist(beam[n_valid - 1]);
        }
    }
    __device__ __forceinline__ void entry(int q, uint32_t &id, float &dd) const
    {
        if constexpr (Scorer::kPQ) {
            const uint64_t kk = q < 64 ? key[0] : key[1];
            id = (uint32_t)kk;
            dd = __uint_as_float((uint32_t)(kk >> 32));
        } else {
            const uint64_t kk = beam[q];
            id = key_id(kk);
            dd = key_dist(kk);
        }
    }
};

template <class Scorer>
__global__ void __launch_bounds__(256, Scorer::kWaves) phase_kernel(PhaseArgs a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = lane_id();
    const int wid = threadIdx.x >> 6;
    const uint32_t slot = a.slot_base + blockIdx.x * a.waves_per_block + wid;

    // per-wave LDS: worklist, sorted new keys, output-slot bitmap, candidate
    // ids and distances, visited table; sized for the widest phase of the launch
    unsigned char *mine = smem + (size_t)wid * a.lds_per_wave;
    // (sizes keep every array 16-byte aligned: Lb and the bitmap word count are even)
    const int Lb = beam_slots(a.L_alloc);
    const int pw = ((a.L_alloc >> 6) + 3) & ~1;
    uint64_t *beam = reinterpret_cast<uint64_t *>(mine);         // Lb
    uint64_t *nkey = beam + Lb;                                  // 64
    uint64_t *posbm = nkey + 64;                                 // pw >= L/64 + 2
    uint32_t *cid = reinterpret_cast<uint32_t *>(posbm + pw);   // 64
    float *cd = reinterpret_cast<float *>(cid + 64);             // 64
    unsigned char *qlds = reinterpret_cast<unsigned char *>(cd + 64);   // the scorer's query copy or table
    // the exact re-rank keys of a product-quantised search (Lb entries), over
    // its table, which the re-rank does not need
    uint64_t *rrk = reinterpret_cast<uint64_t *>(qlds);
    uint32_t *htab = reinterpret_cast<uint32_t *>(
        qlds + (Scorer::kPQ ? max(Scorer::kLdsBytes, 8 * Lb) : Scorer::kLdsBytes));   // H/2 words (H 16-bit slots)

    const IndexView ix = a.ix;
    int R = ix.R;   // (made opaque once per expansion, see there)
    const int d = ix.d;
    // row gathers ahead of the visited test (scorers that have them, rows they cover)
    const bool spec = Scorer::kSpec && R <= Scorer::kSpecMaxR;

    const uint32_t n_in = bcast0(*a.n_active);
    if (n_in <= a.tau_count || n_in <= a.min_active || n_in > a.max_active) return;   // (tau: the loop of Alg. 1 has stopped)

    VisitSet vs;
    vs.bind(a, htab, slot);
    vs.open();

    Scorer sc;
    sc.bind_lds(qlds);
    if constexpr (Scorer::kPQ) sc.bind_pq(a.pq_codes, a.pq_m, a.pq_cb, d, a.vec_u8);
    // one point's attribute record (m_pad cells) and its violation count (Eq. 2)
    auto load_attrs = [&](uint32_t id, int4 &w0, int4 &w1) { load_attr_record(ix, id, w0, w1); };
    RangeTest rt;
    auto count_phi = [&](const int4 &w0, const int4 &w1) -> uint32_t { return rt.phi(w0, w1, ix.m_pad); };
    // keys of the c candidates listed in cid[0, c), one per lane. Attribute
    // records first, then the vectors, so that both gathers are in flight
    // together; phi is counted afterwards. This lane's candidate (for its
    // attribute record) and the scorer's first round of ids are LDS reads
    // issued together.
    auto score_listed = [&](uint32_t c) -> uint64_t {
        if (c == 0) return KEY_NONE;
        wave_sync();
        const uint32_t my_id = cid[lane];
        typename Scorer::Ids ids0;
        sc.read_ids(cid, (int)c, 0, lane, ids0);
        int4 w0 = make_int4(0, 0, 0, 0), w1 = make_int4(0, 0, 0, 0);
        if (lane < (int)c) load_attrs(my_id, w0, w1);
        sc.score(ix.vectors, d, cid, (int)c, cd, lane, ids0);
        const uint32_t phi = count_phi(w0, w1);
        wave_sync();
        return lane < (int)c ? make_key(phi, cd[lane], cid[lane]) : KEY_NONE;
    };
    WaveList wl;
    wl.beam = beam;
    wl.nkey = nkey;
    wl.posbm = posbm;
    wl.len = 0;
#ifdef BOA_STAGE_PROFILE
    uint64_t prof_acc[BOA_PROF_SLOTS] = {};
#endif
    for (;;) {
        const PhaseArgs &aq = cold_args();
        uint32_t t = 0;
        if (lane == 0) t = atomicAdd(aq.queue, 1u);
        t = bcast0(t) + aq.t_begin;
        if (t >= min(aq.t_end, n_in)) break;
        const uint32_t qi = bcast0(aq.active[t]);

        sc.load_query(aq.queries, qi, d, lane);
        rt.set(aq.ranges, qi, aq.ix.m, aq.ix.f32_mask);
        // the phases of this launch: each restarts the search from the entry
        // point at its own width (Alg. 1 calls Alg. 2 afresh)
        // search state; in the warm-start mode it carries over from phase to
        // phase (the worklist, its expanded flags and the visited set)
        for (int p = aq.p_begin; p < cold_args().p_end; ++p) {
        const PhaseArgs &ap = cold_args();
        const int L = ap.sched[p];
        // warm start: the list keeps up to the next phase's width while only
        // its first L entries are expanded (the last phase keeps L)
        const int Lcap = (ap.warm && p + 1 < ap.p_end) ? ap.sched[p + 1] : L;
        const bool fresh = !ap.warm || p == ap.p_begin;
        if (fresh) {
            vs.clear(lane);
            wl.clear(Lb, lane);
            vs.spill = false;
        }
        vs.spill = bcast0(vs.spill ? 1u : 0u) != 0u;
        wave_sync();

        uint32_t E = 0, S = bcast0(fresh ? 1u : 0u);
        wl.begin(L, Lcap, lane);
        // adjacency row already in flight for the node expected next
        uint32_t pf_id = BOA_PAD;
        uint32_t pf_row = BOA_PAD;
        // keys of the last expansion's new nodes, not yet in the worklist
        uint64_t nk = KEY_NONE;

        // the entry point is scored before the first expansion (a warm phase
        // continues with nothing new to score)
        if (fresh) {
            if (lane == 0) {
                vs.enter(ix.entry);
                cid[0] = ix.entry;
            }
            nk = score_listed(1u);
        }

        for (;;) {
            // Row-gather scorers re-read the row length as an opaque (uniform)
            // value at every expansion, so that tests on it (lane < R, the
            // number of gather rounds) are recomputed where they are used
            // instead of being hoisted out of the loop as lane masks, which
            // would not fit the scalar registers and would be reloaded from
            // spill lanes at every use. (The other scorers spill more with it.
            // The same for the lane number moves waits for the prefetched row
            // earlier.)
            if constexpr (Scorer::kSpec) {
                int r = R;
                asm volatile("" : "+v"(r));
                R = __builtin_amdgcn_readfirstlane(r);
            }
            // ---- the nearest unexpanded node, also among the keys just scored
            PROF_T(t_sel0);
            uint64_t ku;
            const int found = wl.next(nk, ku, lane);
            PROF_T(t_sel1);
            PROF_ADD(0, t_sel1 - t_sel0);
            if (found != NEXT_FOUND) {
                wl.add(nk, true, lane);
                // converged (every entry among the first L expanded), and the
                // list in order for what reads it
                if (found == NEXT_NONE && wl.pn == 0) break;
                continue;
            }
            const uint32_t u = key_id(ku);
            E += 1;

            // ---- adjacency row (prefetched if predicted)
            uint32_t v;
            if (u == pf_id) {
                v = lane < R ? pf_row : BOA_PAD;
                PROF_ADD(8, 1);
            } else {
                v = lane < R ? ix.adj[(size_t)u * R + lane] : BOA_PAD;
            }
            PROF_ADD(10, 1);
            // (the row is waited for here, on every path: a wait that only one
            // of the paths below needs would be placed where they join, and
            // would hold the visited test back until the gathers are done)
            asm volatile("" : "+v"(v));
            PROF_T(t_row);
            PROF_ADD(12, t_row - t_sel1);

            // row-gather scorers: every neighbour's attribute record and
            // vector requested now, so that the gathers overlap the visited
            // test; only the new neighbours' keys are entered (the same
            // candidates, distances and keys as scoring after the test)
            typename Scorer::RowGather rg;
            int4 aw0 = make_int4(0, 0, 0, 0), aw1 = make_int4(0, 0, 0, 0);
            if (spec) {
                const uint32_t vv = v != BOA_PAD ? v : ix.entry;   // padding: any valid row, unused
                if (lane < R) load_attrs(vv, aw0, aw1);
                sc.gather_row(ix.vectors, d, vv, R, lane, rg);
            }

            // ---- test-and-insert into the visited set
            const int vst = vs.test(v, lane);
            PROF_T(t_vl);
            PROF_ADD(13, t_vl - t_row);
            const bool is_new = vst > 0;
            const uint64_t nm = __ballot(is_new);
            const uint32_t c = __popcll(nm);
            PROF_ADD(14, c == 0 ? 1 : 0);
            if (!spec && is_new) cid[lanes_below(nm)] = v;
            S += c;
            // ---- the previous expansion's keys enter the worklist while the
            // gathers are in flight
            wl.add(nk, false, lane);
            PROF_T(t_add);
            PROF_ADD(3, t_add - t_vl);
            // the row of the entry expected next is requested only now: a
            // load issued before the visited test would be waited for there
            // (loads retire in order), while from here it overlaps the gathers.
            // It is requested on every path (the entry's row when nothing is
            // predicted), so that waiting for the gathers is one fixed count.
            {
                // (every lane loads, lanes past R from the row's last slot:
                // a load under a branch would leave the count unknown; the
                // row is masked where it is used, since a select here would
                // wait for the load at once)
                const uint64_t kn = min(wl.first_key(), wl.pmin);
                const uint32_t pid = kn != KEY_NONE ? key_id(kn) : ix.entry;
                pf_id = kn != KEY_NONE ? pid : BOA_PAD;
                pf_row = ix.adj[(size_t)pid * R + (lane < R ? lane : R - 1)];
            }
            PROF_T(t_vis1);
            PROF_ADD(1, t_vis1 - t_sel1);
            PROF_ADD(6, vs.spill ? 1 : 0);
            // ---- the new nodes' keys (one per lane)
            if (spec) {
                const uint32_t phi = count_phi(aw0, aw1);
                sc.score_row(rg, d, R, cd, lane);
                wave_sync();
                nk = is_new ? make_key(phi, cd[lane], v) : KEY_NONE;
            } else {
                nk = score_listed(c);
            }
            nk = wl.filter(nk);
            PROF_T(t_sc1);
            PROF_ADD(2, t_sc1 - t_vis1);
        }

        // ---- epilogue: confidence (Eq. 3) over the phase's worklist (its
        // first L entries); the result is written by the last phase the
        // query runs in this launch
        wave_sync();
        const PhaseArgs &ae = cold_args();
        PhaseResult<Scorer> res;
        res.read(ae, wl, qi, rrk, lane);
        const bool last = end_phase(ae, lane, p, qi, t, L, res.n_valid, res.d_k, res.d_max, E, S, vs.spill,
                                    [&](int q, uint32_t &id, float &dd) { res.entry(q, id, dd); });
        wave_sync();
        if (last) break;
        if constexpr (Scorer::kPQ) sc.load_query(ae.queries, qi, d, lane);
        }   // phases
    }       // queries
    vs.close(lane);
#ifdef BOA_STAGE_PROFILE
    if (lane == 0 && a.prof) {
        for (int i = 0; i < BOA_PROF_SLOTS; ++i) a.prof[(size_t)slot * BOA_PROF_SLOTS + i] += prof_acc[i];
    }
#endif
}

// ---------------------------------------------------------------------------
// A team of waves per query, for launches with few queries: one wave (wave 0
// of the block) owns the worklist and the visited set; the others (helpers)
// expand nodes it names, ahead of their turn.
//
// With one wave per query, an expansion is a chain of memory round trips (the
// row, the gathers) and of the wave's own work, one after the other: 8 to 11
// thousand cycles, while a launch of a few hundred queries leaves most of the
// chip idle. What an expansion reads does not depend on the worklist: a
// helper loads the node's row, leaves out the neighbours that the visited set
// already holds, and computes the others' keys. The worklist wave names the
// unexpanded entries next in order before they are selected, so that the keys
// are usually there when their node's turn comes; it then makes the one
// authoritative test-and-insert of each neighbour, enters the new keys and
// selects. The expansions stay one node at a time in the order of Alg. 2, the
// visited set sees the same inserts in the same order, and a key is dropped
// only where the set held its id at the helper's look, which it then holds
// for good (sets are cleared between phases, while every helper is idle): the
// results and counts are those of the one-wave launch.
//
// Measured, before (two waves in lock step in a split search's escalation, else
// one wave) and with teams: 64 queries (uint8, d = 128, widths 16 and 512) 1.63
// and 1.05 ms; 239 queries at width 512 (float32, d = 128, R = 64, in a split
// search of 10,000) 3.79 and 3.13 ms; 777 at width 500 (d = 100) 2.35 and 1.31
// ms; 2,000 with d = 768 up to width 1024 in BOA+ mode 23.7 and 17.0 ms, there
// bound by memory. An expansion takes the worklist wave 3,000 cycles of its own
// work; 60 to 70 of 100 nodes have been named ahead.
//
// Orders are passed through LDS: the worklist wave writes a helper's request
// word (a sequence number, a kind and a payload); the helper answers with the
// sequence number once its keys are written. A helper waits only for a
// request, and one follows on every path (the last is TEAM_EXIT); the
// worklist wave waits only for a helper that holds a request, which ends
// without waiting for anybody.
enum : uint32_t { TEAM_EXPAND = 0, TEAM_SCORE = 1, TEAM_QUERY = 2, TEAM_EXIT = 3 };
struct TeamWave {        // one helper
    uint64_t req;        // sequence number << 34 | kind << 32 | payload
    uint32_t done;       // upper half of the last request answered
    uint32_t pad;
    uint32_t cid[64];    // its candidates and their distances
    float cd[64];
};

// P helpers share a node: part q takes the row's slice of W = ceil(R / P)
// entries from q W on, and answers in the same entries of the group's keys.
template <class Scorer, int P>
__device__ __forceinline__ void team_helper(const PhaseArgs &a, TeamWave *me, int helper, uint64_t *group_keys,
                                            int part, const VisitSet &vs, unsigned char *qlds, int lane)
{
    const IndexView ix = a.ix;
    const int d = ix.d;
    const int W = (ix.R + P - 1) / P, row0 = part * W;
    const int R = min(W, ix.R - row0);   // (0 or less: nothing for this part)
    uint64_t *keys = group_keys + row0;
    const bool spec = Scorer::kSpec && R <= Scorer::kSpecMaxR;
    auto row_of = [&](uint32_t u) -> uint32_t {
        return ix.adj[(size_t)u * ix.R + max(0, min(row0 + lane, row0 + R - 1))];
    };
    Scorer sc;
    sc.bind_lds(qlds);
    if constexpr (Scorer::kPQ) sc.bind_pq(a.pq_codes, a.pq_m, a.pq_cb, d, a.vec_u8);
    RangeTest rt;
    uint32_t *cid = me->cid;
    float *cd = me->cd;
    uint32_t last = 0;
    // the row of the nearest node this helper found last, requested while
    // the worklist wave selects: a node found just now is the next one in 30
    // to 40 of 100 expansions, and is then asked of the helper that found it
    uint32_t pf_id = BOA_PAD, pf_row = BOA_PAD;
    for (;;) {
        uint64_t r;
        for (;;) {
            r = readlane64(__hip_atomic_load(&me->req, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP), 0);
            if ((uint32_t)(r >> 32) != last) break;
            __builtin_amdgcn_s_sleep(1);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
        last = (uint32_t)(r >> 32);
        const uint32_t kind = last & 3u, what = (uint32_t)r;
        if (kind == TEAM_EXIT) return;
        if (kind == TEAM_QUERY) {
            const PhaseArgs &aq = cold_args();
            // (the helpers share a table; each has its own copy of a query)
            if constexpr (Scorer::kPQ)
                sc.load_table(aq.queries, what, d, lane + 64 * helper, 64 * TEAM_GROUPS * P);
            else
                sc.load_query(aq.queries, what, d, lane);
            rt.set(aq.ranges, what, aq.ix.m, aq.ix.f32_mask);
        } else {
            uint64_t key = KEY_NONE;
            uint32_t v = lane == 0 && part == 0 ? what : BOA_PAD;
            if (kind == TEAM_EXPAND) {
                v = what == pf_id ? pf_row : row_of(what);
                if (lane >= R) v = BOA_PAD;
            }
            asm volatile("" : "+v"(v));
            if (spec && kind == TEAM_EXPAND) {
                const uint32_t vv = v != BOA_PAD ? v : ix.entry;   // padding: any valid row, unused
                typename Scorer::RowGather rg;
                int4 w0 = make_int4(0, 0, 0, 0), w1 = make_int4(0, 0, 0, 0);
                if (lane < R) load_attr_record(ix, vv, w0, w1);
                sc.gather_row(ix.vectors, d, vv, R, lane, rg);
                const bool open = v != BOA_PAD && !vs.holds(vv);
                const uint32_t phi = rt.phi(w0, w1, ix.m_pad);
                sc.score_row(rg, d, R, cd, lane);
                wave_sync();
                if (open) key = make_key(phi, cd[lane], v);
            } else {
                bool open = v != BOA_PAD;
                if (open && kind == TEAM_EXPAND) open = !vs.holds(v);
                const uint64_t om = __ballot(open);
                const uint32_t c = (uint32_t)__popcll(om);
                if (open) cid[lanes_below(om)] = v;
                if (c > 0) {
                    wave_sync();
                    const uint32_t my_id = cid[lane];
                    typename Scorer::Ids ids0;
                    sc.read_ids(cid, (int)c, 0, lane, ids0);
                    int4 w0 = make_int4(0, 0, 0, 0), w1 = make_int4(0, 0, 0, 0);
                    if (lane < (int)c) load_attr_record(ix, my_id, w0, w1);
                    sc.score(ix.vectors, d, cid, (int)c, cd, lane, ids0);
                    const uint32_t phi = rt.phi(w0, w1, ix.m_pad);
                    wave_sync();
                    if (lane < (int)c) key = make_key(phi, cd[lane], my_id);
                }
            }
            if (lane < W && row0 + lane < 64) keys[lane] = key;
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
            __builtin_amdgcn_wave_barrier();
            if (lane == 0) __hip_atomic_store(&me->done, last, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            const uint64_t near = wave_min_open(key);
            if (near != KEY_NONE) {
                pf_id = key_id(near);
                pf_row = row_of(pf_id);
            }
            continue;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_wave_barrier();
        if (lane == 0) __hip_atomic_store(&me->done, last, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
}

template <class Scorer, int P>
__global__ void __launch_bounds__(64 * (1 + TEAM_GROUPS * P), Scorer::kTeamWaves) team_kernel(PhaseArgs a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = lane_id();
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int Lb = beam_slots(a.L_alloc);
    const int pw = ((a.L_alloc >> 6) + 3) & ~1;
    uint64_t *beam = reinterpret_cast<uint64_t *>(smem);          // Lb
    uint64_t *nkey = beam + Lb;                                     // 64
    uint64_t *posbm = nkey + 64;                                    // pw
    uint64_t *keys = posbm + pw;                                    // 64 per group
    TeamWave *wv = reinterpret_cast<TeamWave *>(keys + 64 * TEAM_GROUPS);   // one per helper
    unsigned char *qlds = reinterpret_cast<unsigned char *>(wv + TEAM_GROUPS * P);
    uint32_t *vis = reinterpret_cast<uint32_t *>(
        qlds + (Scorer::kPQ ? max(Scorer::kLdsBytes, 8 * Lb) : Scorer::kLdsBytes));

    const uint32_t n_in = bcast0(*a.n_active);
    // (the same for every wave of the block)
    if (n_in <= a.tau_count || n_in <= a.min_active || n_in > a.max_active) return;
    VisitSet vs;
    vs.bind(a, vis, a.slot_base + blockIdx.x);
    if (threadIdx.x < TEAM_GROUPS * P) {
        wv[threadIdx.x].req = 0;
        wv[threadIdx.x].done = 0;
    }
    // (entries past a row's parts stay empty)
    for (int i = threadIdx.x; i < 64 * TEAM_GROUPS; i += blockDim.x) keys[i] = KEY_NONE;
    __syncthreads();
    if (wid > 0) {
        const int h = (wid - 1) / P;
        team_helper<Scorer, P>(a, wv + (wid - 1), wid - 1, keys + 64 * h, (wid - 1) - h * P, vs, qlds, lane);
        return;
    }
    __builtin_amdgcn_s_setprio(2);   // the helpers wait for this wave
    vs.open();
    const IndexView ix = a.ix;
    WaveList wl;
    wl.beam = beam;
    wl.nkey = nkey;
    wl.posbm = posbm;
    wl.len = 0;
    // group h's state in lane h: the node it holds (or works on), its last
    // request's upper half
    uint32_t hnode = BOA_PAD, hseq = 0;
    uint32_t seq = 0;
    auto order = [&](int h, uint32_t kind, uint32_t what) {
        seq = (seq + 1u) & 0x3FFFFFFFu;
        const uint32_t hi = seq << 2 | kind;
        if (lane == h) {
            hseq = hi;
            hnode = kind == TEAM_EXPAND ? what : BOA_PAD;
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
#pragma unroll
            for (int q = 0; q < P; ++q)
                __hip_atomic_store(&wv[h * P + q].req, (uint64_t)hi << 32 | what, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_WORKGROUP);
        }
    };
    // groups whose last request is answered by every part
    auto idle = [&]() -> uint64_t {
        bool is = false;
        if (lane < TEAM_GROUPS) {
            is = true;
#pragma unroll
            for (int q = 0; q < P; ++q)
                is &= __hip_atomic_load(&wv[lane * P + q].done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) == hseq;
        }
        return __ballot(is);
    };
    constexpr uint64_t ALL = (1ull << TEAM_GROUPS) - 1ull;
    auto wait_for = [&](uint64_t which) {
        while ((idle() & which) != which) __builtin_amdgcn_s_sleep(1);
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    };
#ifdef BOA_STAGE_PROFILE
    // 0 select, 3 enter the keys, 1 name the next nodes, 2 wait for the
    // helper, 13 read and test its keys; 8 nodes named ahead, 10 expansions,
    // 12 keys ready without a wait
    uint64_t prof_acc[BOA_PROF_SLOTS] = {};
#endif
    for (;;) {
        const PhaseArgs &aq = cold_args();
        uint32_t t = 0;
        if (lane == 0) t = atomicAdd(aq.queue, 1u);
        t = bcast0(t) + aq.t_begin;
        if (t >= min(aq.t_end, n_in)) break;
        const uint32_t qi = bcast0(aq.active[t]);
        for (int h = 0; h < TEAM_GROUPS; ++h) order(h, TEAM_QUERY, qi);
        for (int p = aq.p_begin; p < cold_args().p_end; ++p) {
            const PhaseArgs &ap = cold_args();
            const int L = ap.sched[p];
            const int Lcap = (ap.warm && p + 1 < ap.p_end) ? ap.sched[p + 1] : L;
            const bool fresh = !ap.warm || p == ap.p_begin;
            // every helper idle: the set may be cleared, and what they hold
            // (looked up in the set before) is forgotten
            wait_for(ALL);
            hnode = BOA_PAD;
            if (fresh) {
                vs.clear(lane);
                wl.clear(Lb, lane);
                vs.spill = false;
            }
            vs.spill = bcast0(vs.spill ? 1u : 0u) != 0u;
            wave_sync();
            uint32_t E = 0, S = bcast0(fresh ? 1u : 0u);
            wl.begin(L, Lcap, lane);
            uint64_t nk = KEY_NONE;
            int hl = 0;   // the helper read last: idle and holding nothing
            if (fresh) {
                // the entry point is scored before the first expansion
                if (lane == 0) vs.enter(ix.entry);
                wave_sync();
                order(0, TEAM_SCORE, ix.entry);
                wait_for(1ull);
                nk = keys[lane];
            }
            for (;;) {
                PROF_T(t0);
                uint64_t ku;
                const int found = wl.next(nk, ku, lane);
                if (found != NEXT_FOUND) {
                    wl.add(nk, true, lane);
                    if (found == NEXT_NONE && wl.pn == 0) break;
                    continue;
                }
                const uint32_t u = key_id(ku);
                E += 1;
                // ---- the helper that holds the node, or one to expand it now
                uint64_t hm = __ballot(hnode == u);
                if (hm == 0ull) {
                    // one that holds nothing, at best the helper read last
                    // (it may have the node's row); else one that is done with
                    // a node named ahead, which is then named again later
                    uint64_t fr = __ballot(hnode == BOA_PAD) & ALL;
                    if (fr == 0ull)
                        while ((fr = idle()) == 0ull) __builtin_amdgcn_s_sleep(1);
                    const int hn = ((fr >> hl) & 1ull) ? hl : __ffsll((unsigned long long)fr) - 1;
                    order(hn, TEAM_EXPAND, u);
                    hm = 1ull << hn;
                } else {
                    PROF_ADD(8, 1);
                }
                const int h = __ffsll((unsigned long long)hm) - 1;
                PROF_T(t1);
                PROF_ADD(0, t1 - t0);
                // ---- the previous expansion's keys enter the worklist
                wl.add(nk, false, lane);
                PROF_T(t2);
                PROF_ADD(3, t2 - t1);
                // ---- the two entries next in order (of the nearest pending
                // one and the first two of the sorted list) are named to
                // helpers that hold nothing, or neither of them
                {
                    const uint64_t s1 = wl.first_key();
                    const uint64_t wm = wl.wmask & (wl.wmask - 1ull);
                    const uint64_t s2 = wm ? readlane64(wl.win, __ffsll((unsigned long long)wm) - 1) : KEY_NONE;
                    const bool pf = wl.pmin < s1;
                    const uint64_t c0 = pf ? wl.pmin : s1, c1 = pf ? s1 : min(wl.pmin, s2);
                    const uint64_t m0 = __ballot(hnode == key_id(c0)), m1 = __ballot(hnode == key_id(c1));
                    const bool n0 = c0 != KEY_NONE && m0 == 0ull, n1 = c1 != KEY_NONE && m1 == 0ull;
                    if (n0 || n1) {
                        uint64_t av = __ballot(hnode == BOA_PAD) & ALL & ~hm;
                        if (__popcll(av) < (n0 && n1 ? 2 : 1)) av |= idle() & ~(hm | m0 | m1);
                        if (n0 && av) {
                            order(__ffsll((unsigned long long)av) - 1, TEAM_EXPAND, key_id(c0));
                            av &= av - 1ull;
                        }
                        if (n1 && av) order(__ffsll((unsigned long long)av) - 1, TEAM_EXPAND, key_id(c1));
                    }
                }
                PROF_T(t3);
                PROF_ADD(1, t3 - t2);
                // ---- its keys
#ifdef BOA_STAGE_PROFILE
                if (idle() & hm) PROF_ADD(12, 1);
#endif
                wait_for(hm);
                PROF_T(t4);
                PROF_ADD(2, t4 - t3);
                const uint64_t key = keys[64 * h + lane];
                if (lane == h) hnode = BOA_PAD;
                hl = h;
                const bool is_new = vs.test(key != KEY_NONE ? key_id(key) : BOA_PAD, lane) > 0;
                S += (uint32_t)__popcll(__ballot(is_new));
                nk = wl.filter(is_new ? key : KEY_NONE);
                PROF_T(t5);
                PROF_ADD(13, t5 - t4);
                PROF_ADD(10, 1);
            }
            // ---- end of the phase
            const PhaseArgs &ae = cold_args();
            if constexpr (Scorer::kPQ) wait_for(ALL);   // (the table's place is about to be used)
            PhaseResult<Scorer> res;
            res.read(ae, wl, qi, reinterpret_cast<uint64_t *>(qlds), lane);
            const bool last = end_phase(ae, lane, p, qi, t, L, res.n_valid, res.d_k, res.d_max, E, S, vs.spill,
                                        [&](int q, uint32_t &id, float &dd) { res.entry(q, id, dd); });
            if constexpr (Scorer::kPQ) {
                if (!last)
                    for (int h = 0; h < TEAM_GROUPS; ++h) order(h, TEAM_QUERY, qi);
            }
            wave_sync();
            if (last) break;
        }   // phases
        // (no helper reads the query any more)
        wait_for(ALL);
    }       // queries
    for (int h = 0; h < TEAM_GROUPS; ++h) order(h, TEAM_EXIT, 0u);
    vs.close(lane);
#ifdef BOA_STAGE_PROFILE
    if (lane == 0 && a.prof) {
        for (int i = 0; i < BOA_PROF_SLOTS; ++i) a.prof[(size_t)blockIdx.x * BOA_PROF_SLOTS + i] += prof_acc[i];
    }
#endif
}

// Stable compaction of the active list (Alg. 1: survivors escalate). One
// block: flags -> ballot prefix within waves -> wave totals in LDS.
__global__ void __launch_bounds__(1024) compact_kernel(CompactArgs a)
{
    __shared__ uint32_t wsum[16];
    __shared__ uint32_t base_s;
    const uint32_t n_in = *a.n_in;
    const bool stopped = n_in <= a.tau_count;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
    if (threadIdx.x == 0) base_s = 0;
    __syncthreads();
    for (uint32_t b0 = 0; !stopped && b0 < n_in; b0 += blockDim.x) {
        uint32_t t = b0 + threadIdx.x;
        bool keep = t < n_in && a.conf[t] == 0;
        uint64_t mk = __ballot(keep);
        if (lane == 0) wsum[w] = __popcll(mk);
        __syncthreads();
        uint32_t off = base_s;
        for (int i = 0; i < w; ++i) off += wsum[i];
        if (keep) a.out[off + lanes_below(mk)] = a.in[t];
        __syncthreads();
        if (threadIdx.x == 0) {
            uint32_t tot = 0;
            for (int i = 0; i < nw; ++i) tot += wsum[i];
            base_s += tot;
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) *a.n_out = stopped ? 0u : base_s;
}

// BOA+ survivor pooling: append the non-confident entries of one phase-0
// sub-batch (a slice of the active list) to a pool, stably, after the
// pool's current entries; then publish the new count. One block.
__global__ void __launch_bounds__(1024) append_kernel(AppendArgs a)
{
    __shared__ uint32_t wsum[16];
    __shared__ uint32_t base_s;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
    if (threadIdx.x == 0) base_s = *a.pool_count;
    __syncthreads();
    for (uint32_t b0 = 0; b0 < a.n; b0 += blockDim.x) {
        uint32_t t = b0 + threadIdx.x;
        bool keep = t < a.n && a.conf[t] == 0;
        uint64_t mk = __ballot(keep);
        if (lane == 0) wsum[w] = __popcll(mk);
        __syncthreads();
        uint32_t off = base_s;
        for (int i = 0; i < w; ++i) off += wsum[i];
        if (keep) a.pool[off + lanes_below(mk)] = a.in[t];
        __syncthreads();
        if (threadIdx.x == 0) {
            uint32_t tot = 0;
            for (int i = 0; i < nw; ++i) tot += wsum[i];
            base_s += tot;
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) *a.pool_count = base_s;
}

__global__ void init_kernel(InitArgs a)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < (size_t)a.nq) {
        a.active0[i] = (uint32_t)i;
        if (a.user_E) a.user_E[i] = 0;
        if (a.user_S) a.user_S[i] = 0;
    }
    if (a.qstat && i < (size_t)a.nq * a.n_phases) a.qstat[i] = 0;
    if (i < (size_t)a.n_counters) a.counters[i] = 0;
    if (i < a.reset_slots) a.bits[i * a.slot_words + a.bits_words] = BOA_LOG_DIRTY;
    if (i == 0) {
        a.n_active[0] = (uint32_t)a.nq;
        // later phases' counts and the BOA+ pool counts
        for (int p = 1; p < 2 * (BOA_MAX_PHASES + 1); ++p) a.n_active[p] = 0;
        *a.status = 0;
    }
}

// ---------------------------------------------------------------------------
// launch helpers (host)

template <class Scorer>
static hipError_t launch_phase_t(const PhaseArgs &a, int blocks, hipStream_t st)
{
    size_t lds = (size_t)a.lds_per_wave * a.waves_per_block;
    hipLaunchKernelGGL(phase_kernel<Scorer>, dim3(blocks), dim3(64 * a.waves_per_block), lds, st, a);
    return hipGetLastError();
}

template <class Scorer>
static int occupancy_t(int wpb, size_t lds)
{
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, phase_kernel<Scorer>, 64 * wpb, lds) != hipSuccess)
        return 0;
    return nb;
}

#define BOA_DISPATCH_W(VEC, DIM, W, CALL)                                    \
    do {                                                                     \
        if ((VEC) == BOA_VEC_F32) {                                          \
            int T_ = ((DIM) + 63) / 64;                                      \
            if (T_ <= 1) { using S_ = F32Scorer<1, W>; CALL; }               \
            else if (T_ <= 2) { using S_ = F32Scorer<2, W>; CALL; }          \
            else if (T_ <= 3) { using S_ = F32Scorer<3, W>; CALL; }          \
            else if (T_ <= 4) { using S_ = F32Scorer<4, W>; CALL; }          \
            else if (T_ <= 6) { using S_ = F32Scorer<6, W>; CALL; }          \
            else if (T_ <= 8) { using S_ = F32Scorer<8, W>; CALL; }          \
            else if (T_ <= 12) { using S_ = F32Scorer<12, W>; CALL; }        \
            else { using S_ = F32Scorer<16, W>; CALL; }                      \
        } else {                                                             \
            int G_ = (DIM) / 16;                                             \
            if (G_ <= 1) { using S_ = U8Scorer<1, W>; CALL; }                \
            else if (G_ <= 2) { using S_ = U8Scorer<2, W>; CALL; }           \
            else if (G_ <= 4) { using S_ = U8Scorer<4, W>; CALL; }           \
            else if (G_ <= 8) { using S_ = U8Scorer<8, W>; CALL; }           \
            else if (G_ <= 16) { using S_ = U8Scorer<16, W>; CALL; }         \
            else if (G_ <= 32) { using S_ = U8Scorer<32, W>; CALL; }         \
            else { using S_ = U8Scorer<64, W>; CALL; }                       \
        }                                                                    \
    } while (0)

#define BOA_DISPATCH_PQ(PQM, CALL)                                           \
    do {                                                                     \
        int T_ = ((PQM) + 15) / 16;                                          \
        if (T_ <= 1) { using S_ = PQScorer<1>; CALL; }                       \
        else if (T_ <= 2) { using S_ = PQScorer<2>; CALL; }                  \
        else if (T_ <= 4) { using S_ = PQScorer<4>; CALL; }                  \
        else if (T_ <= 8) { using S_ = PQScorer<8>; CALL; }                  \
        else if (T_ <= 12) { using S_ = PQScorer<12>; CALL; }                \
        else { using S_ = PQScorer<16>; CALL; }                              \
    } while (0)

// product-quantised searches (PQM > 0) take the PQ scorer, which has no
// wide variant; the others the exact scorer of the vector type
#define BOA_DISPATCH(VEC, DIM, WIDE, CALL, PQM)                              \
    do {                                                                     \
        if ((PQM) > 0) BOA_DISPATCH_PQ(PQM, CALL);                           \
        else if (WIDE) BOA_DISPATCH_W(VEC, DIM, 2, CALL);                    \
        else BOA_DISPATCH_W(VEC, DIM, 1, CALL);                              \
    } while (0)

template <class Scorer, int P>
static hipError_t launch_team_t(const PhaseArgs &a, int blocks, hipStream_t st)
{
    hipLaunchKernelGGL((team_kernel<Scorer, P>), dim3(blocks), dim3(64 * (1 + TEAM_GROUPS * P)),
                       (size_t)a.lds_per_wave, st, a);
    return hipGetLastError();
}

template <class Scorer, int P>
static int team_occupancy_t(size_t lds)
{
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, team_kernel<Scorer, P>, 64 * (1 + TEAM_GROUPS * P), lds) !=
        hipSuccess)
        return 0;
    return nb;
}

// the launch with a team of waves per query (lds_per_wave is the block's LDS)
hipError_t launch_team(const PhaseArgs &a, int vec_dtype, int parts, int blocks, hipStream_t st)
{
    hipError_t e = hipSuccess;
    if (a.pq) BOA_DISPATCH_PQ(a.pq_m, e = (launch_team_t<S_, 1>(a, blocks, st)));
    else if (parts == 2) BOA_DISPATCH_W(vec_dtype, a.ix.d, 3, e = (launch_team_t<S_, 2>(a, blocks, st)));
    else BOA_DISPATCH_W(vec_dtype, a.ix.d, 3, e = (launch_team_t<S_, 1>(a, blocks, st)));
    return e;
}

int team_occupancy(int vec_dtype, int d, int parts, size_t lds, int pq_m)
{
    int r = 0;
    if (pq_m > 0) BOA_DISPATCH_PQ(pq_m, r = (team_occupancy_t<S_, 1>(lds)));
    else if (parts == 2) BOA_DISPATCH_W(vec_dtype, d, 3, r = (team_occupancy_t<S_, 2>(lds)));
    else BOA_DISPATCH_W(vec_dtype, d, 3, r = (team_occupancy_t<S_, 1>(lds)));
    return r;
}

size_t team_lds_bytes(int32_t L, int parts, uint32_t vis_words, int scorer_lds)
{
    const int32_t Lb = beam_slots(L), pw = ((L >> 6) + 3) & ~1;
    return (size_t)8 * Lb + 8 * 64 + 8 * (size_t)pw + TEAM_GROUPS * (8 * 64 + parts * sizeof(TeamWave)) +
           (size_t)scorer_lds + 4 * (size_t)vis_words;
}

hipError_t launch_phase(const PhaseArgs &a, int vec_dtype, int blocks, hipStream_t st, bool wide)
{
    hipError_t e = hipSuccess;
    BOA_DISPATCH(vec_dtype, a.ix.d, wide, e = launch_phase_t<S_>(a, blocks, st), a.pq ? a.pq_m : 0);
    return e;
}

template <class Scorer>
static int scorer_lds_t()
{
    return Scorer::kLdsBytes;
}

int scorer_lds_bytes(int vec_dtype, int d, bool wide, int pq_m)
{
    int r = 0;
    BOA_DISPATCH(vec_dtype, d, wide, r = scorer_lds_t<S_>(), pq_m);
    return r;
}

int phase_occupancy(int vec_dtype, int d, int wpb, size_t lds, bool wide, int pq_m)
{
    int r = 0;
    BOA_DISPATCH(vec_dtype, d, wide, r = occupancy_t<S_>(wpb, lds), pq_m);
    return r;
}

hipError_t launch_compact(const CompactArgs &a, hipStream_t st)
{
    hipLaunchKernelGGL(compact_kernel, dim3(1), dim3(1024), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_append(const AppendArgs &a, hipStream_t st)
{
    hipLaunchKernelGGL(append_kernel, dim3(1), dim3(1024), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_init(const InitArgs &a, hipStream_t st)
{
    size_t n = (size_t)a.nq * (a.n_phases > 1 ? a.n_phases : 1);
    if ((size_t)a.n_counters > n) n = a.n_counters;
    if (a.reset_slots > n) n = (size_t)a.reset_slots;
    if (n == 0) n = 1;
    unsigned blocks = (unsigned)((n + 255) / 256);
    hipLaunchKernelGGL(init_kernel, dim3(blocks), dim3(256), 0, st, a);
    return hipGetLastError();
}

}  // namespace boa
