// Link-prediction evaluation ("Evaluation Metrics" section): filtered ranks of DistMult scores (Eq. 4),
// MRR (Eq. 5) and Hits@k (Eq. 6).
//
// A query (fixed entity f, relation r, answer a) scores every entity e as  sum_k (H[f][k] M[r][k]) H[e][k]:
// with the query vectors Q = H[f] * M[r] gathered once, all scores are the product Q H^T.  That
// (queries x entities) matrix is never stored: k_eval_count computes it tile by tile on the matrix cores and
// keeps, per query, only how many entries lie above / exactly at the answer's score.
// What the filtered setting removes - the known answers of the same (f, r), from none to thousands per query - is
// scored again by k_eval_pairs and subtracted.  Both kernels build a score from the same sequence of steps (k ascending,
// 16 k per step, fp32 accumulator starting at zero; a step is three products of two fp16 parts, split_f16.h, or, in small
// evaluations and for queries whose numbers do not allow that, six products of three bf16 parts, split_bf16.h, and then a score
// that is not finite comes from v_mfma_f32_32x32x2_f32 steps, two k each), so a pair gets the same bits in both and the subtraction is exact.
// The same per-query kernel ranks against explicit candidate lists.
#include "common.h"
#include "split_f16.h"

#include <algorithm>
#include <cmath>
#include <mutex>
#include <type_traits>
#include <vector>

// Scratch of kge_eval_rank_all_static: device memory that lives in the library's code object, one copy
// per GPU, held until the process ends.  In host code this name is only a handle for
// hipGetSymbolAddress; the address kernels and fills may use is static_scratch_ptr()'s result.
static __device__ __align__(256) unsigned char scratch[KGE_EVAL_STATIC_BYTES];

struct kge_eval_filter {
    int device;
    int32_t n_entities, n_relations;
    // table 0: known tails of (head, rel); table 1: known heads of (tail, rel).
    // key = (fixed * R + rel) * N + other, ascending, unique; val = other
    int64_t n[2];
    int64_t *key[2];
    int32_t *val[2];
};

namespace {

// What k_eval_range found of H and of Q, numbers as the bits of their absolute values: the largest ones and the smallest one of
// H that is not zero, less one, in four places that the blocks of k_eval_range share out.  n_three (the first one's): the
// queries that k_eval_pairs found to need three parts.
struct EvalRange { struct alignas(64) Place { uint32_t max_h, least_h, max_q, n_three; } at[4]; };
static_assert(sizeof(EvalRange) == 256, "what one query's share of the workspace is rounded up to");

// tail queries of all test triples first, then the head queries; their query vectors Q[q][:] = H[fixed][:] * M[rel][:]
// (one thread per 4 columns) and cleared counters
__global__ void k_eval_queries(const int32_t *__restrict__ th, const int32_t *__restrict__ tr,
                               const int32_t *__restrict__ tt, int64_t n_test, const float4 *__restrict__ H,
                               const float4 *__restrict__ M, int32_t d4, int32_t *__restrict__ fixed,
                               int32_t *__restrict__ rel, int32_t *__restrict__ answer, float4 *__restrict__ Q,
                               unsigned *__restrict__ cnt_gt, EvalRange *__restrict__ range)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < 4) range->at[t] = EvalRange::Place{0u, 0xffffffffu, 0u, 0u};
    if (t >= 2 * n_test * d4) return;
    const int64_t i = t / d4;
    const int32_t c = (int32_t)(t - i * d4);
    const bool head_query = i >= n_test;
    const int64_t j = head_query ? i - n_test : i;
    const int32_t f = head_query ? tt[j] : th[j], r = tr[j];
    const float4 h = H[(int64_t)f * d4 + c], m = M[(int64_t)r * d4 + c];
    Q[t] = make_float4(h.x * m.x, h.y * m.y, h.z * m.z, h.w * m.w);
    if (c == 0) {
        fixed[i] = f;
        rel[i] = r;
        answer[i] = head_query ? th[j] : tt[j];
        cnt_gt[i] = 0u;
    }
}

// Q[q][:] = H[fixed[q]][:] * M[rel[q]][:], one thread per 4 columns
__global__ void k_eval_qvec(const float4 *__restrict__ H, const float4 *__restrict__ M,
                            const int32_t *__restrict__ fixed, const int32_t *__restrict__ rel, int64_t nq,
                            int32_t d4, float4 *__restrict__ Q)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= nq * d4) return;
    const int64_t q = t / d4;
    const int32_t c = (int32_t)(t - q * d4);
    const float4 h = H[(int64_t)fixed[q] * d4 + c], m = M[(int64_t)rel[q] * d4 + c];
    Q[t] = make_float4(h.x * m.x, h.y * m.y, h.z * m.z, h.w * m.w);
}

// 8 consecutive k of a row from k (past the width: the row's last ones; no condition stands around the loads, so that
// they can be in flight together), and their parts, scaled by sx and sy
struct Row8 { float4 x, y; };
__device__ __forceinline__ Row8 row_of(const float *__restrict__ row, int32_t k, int32_t d)
{
    Row8 r;
    r.x = *reinterpret_cast<const float4 *>(row + (k < d ? k : d - 4));
    r.y = *reinterpret_cast<const float4 *>(row + (k + 4 < d ? k + 4 : d - 4));
    return r;
}
template <int NP> struct Parts8 { uint4 p[NP]; };
template <int NP>
__device__ __forceinline__ Parts8<NP> parts_of(const Row8 &r, float sx, float sy)
{
    const auto a = split_parts<NP>(r.x.x * sx, r.x.y * sx), b = split_parts<NP>(r.x.z * sx, r.x.w * sx);
    const auto c = split_parts<NP>(r.y.x * sy, r.y.y * sy), e = split_parts<NP>(r.y.z * sy, r.y.w * sy);
    Parts8<NP> q;
#pragma unroll
    for (int p = 0; p < NP; ++p) q.p[p] = make_uint4(a.w[p], b.w[p], c.w[p], e.w[p]);
    return q;
}

// Whether scores are formed from two fp16 parts, and the powers of two that bring the largest numbers of H and of Q to
// 2^14 .. 2^15.  Below 80 columns three bf16 parts are the more accurate (relative error at 64: 1.12e-7 against 1.15e-7, at 128
// 1.66e-7 against 1.44e-7).  With both exponents within 24 no score or threshold can leave fp32's normal range on the way;
// infinities and NaN lie above every exponent that is let through.
constexpr int HALF_FROM = 80;
struct EvalScale { bool half = false, h_loses = false; float h = 1.f, q = 1.f, inv = 1.f; uint32_t q_small = 0u; };
__device__ __forceinline__ EvalScale eval_scale(const EvalRange *__restrict__ range)
{
    EvalScale c;
    uint32_t max_h = 0u, least_h = 0xffffffffu, max_q = 0u;
#pragma unroll
    for (int i = 0; i < 4; ++i) { max_h = max(max_h, range->at[i].max_h); least_h = min(least_h, range->at[i].least_h); max_q = max(max_q, range->at[i].max_q); }
    const int eh = (int)(max_h >> 23) - 127, eq = (int)(max_q >> 23) - 127;
    c.half = abs(eh) <= 24 && abs(eq) <= 24;
    auto two_to = [](int e) { return __uint_as_float((uint32_t)__builtin_amdgcn_readfirstlane((e + 127) << 23)); };
    if (c.half) {
        c.h = two_to(14 - eh); c.q = two_to(14 - eq); c.inv = two_to(eh + eq - 28);
        c.h_loses = least_h + 1u < (uint32_t)(eh + 111) << 23;       // LossBound
        c.q_small = (uint32_t)(eq + 111) << 23;
    }
    return c;
}

// Numbers that scale to less than 2^-2 lose bits to fp16's smallest numbers, 2^-25 each at most, so a score may be off by
//   2^-25 (sum_k |q_k| where h_k loses bits + sum_k |h_k| where q_k does),   |h_k| < 2^15.
// That is nothing where the columns that make up a score are of the largest ones' size, and all of it where they are far
// below: a column of H that is large where every relation is zero, rows of very different size.  A query takes two parts if
// twice that bound (the answer's score has its own) is at most 2^-25 of sum_k |q_k h_k| over its answer's row, half of
// what rounding each of the answer's terms to fp32 may move; else all its scores are formed from three parts.  Scores far
// from the answer's may still have lost bits: they lie on the same side of it.  In ordinary embeddings no query needs three
// parts, and finding that out costs nothing that can be measured: 20,000 queries x 1 M entities, d = 256, 28.6 ms with and
// without; 40,932 x 14,541, d = 200, 1005 and 1001 us.
struct LossBound {
    float q_sum = 0.f, terms = 0.f;
    int32_t q_small = 0;
    __device__ __forceinline__ void add(float q, float h, const EvalScale &sc)
    {
        q_sum += __builtin_fabsf(q * sc.q);
        terms += __builtin_fabsf((q * sc.q) * (h * sc.h));
        q_small += (__float_as_uint(q) & 0x7fffffffu) - 1u < sc.q_small - 1u ? 1 : 0;       // not zero
    }
    __device__ __forceinline__ bool too_large(const EvalScale &sc) const        // 1.01: the sums' own rounding
    {
        return terms < 2.02f * ((sc.h_loses ? q_sum : 0.f) + 32768.f * (float)q_small);
    }
};

// Scores of 32 (query, entity) pairs: lane l and lane l + 32 name pair l (qrow its query vector, ent its entity; ent < 0:
// no pair, any score).  Row l of the matrix-core tile is the pair's query and column l its entity, so the scores lie on the
// diagonal; the rest of the tile is not used.  Lanes 0..31 supply k = 16 s .. 16 s + 7 of step s and lanes 32..63 the
// next 8, as in k_eval_count; every lane gets its pair's score.
__device__ __forceinline__ float diagonal(const split_floatx16 &acc, int lane)
{
    const int c = lane & 31, v = (c >> 3) * 4 + (c & 3);       // register v of the half (c / 4) % 2 is row c
    float s = acc[0];
#pragma unroll
    for (int u = 1; u < 16; ++u) s = v == u ? acc[u] : s;
    return __shfl(s, c + 32 * ((c >> 2) & 1), 64);
}
// NP parts per number; sh, sq: scales of entities and queries (the score comes times their product)
template <int NP>
__device__ __forceinline__ float pair_scores(const float *__restrict__ qrow, const float *__restrict__ H,
                                             int32_t ent, int32_t d, int lane, float sh, float sq)
{
    split_floatx16 acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.f;
    const int half = lane >> 5;
    const float *hb = H + (int64_t)(ent < 0 ? 0 : ent) * d;
    // two steps in flight ahead of the one being multiplied: the rows are gathered, and a tile is one chain
    Row8 q0 = row_of(qrow, 8 * half, d), h0 = row_of(hb, 8 * half, d);
    Row8 q1 = row_of(qrow, 16 + 8 * half, d), h1 = row_of(hb, 16 + 8 * half, d);
    for (int32_t k0 = 0; k0 < d; k0 += 16) {
        const int32_t k = k0 + 8 * half;
        const Parts8<NP> q = parts_of<NP>(q0, sq, sq), h = parts_of<NP>(h0, k < d ? sh : 0.f, k + 4 < d ? sh : 0.f);
        q0 = q1; h0 = h1;
        q1 = row_of(qrow, k + 32, d);
        h1 = row_of(hb, k + 32, d);
#pragma unroll
        for (int p = 0; p < split_terms<NP>(); ++p) acc = split_product<NP>(q.p[split_b<NP>(p)], h.p[split_a<NP>(p)], acc);
    }
    float s = diagonal(acc, lane);
    if (NP == 3 && __any(ent >= 0 && split_not_finite(s))) {
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[v] = 0.f;
        for (int32_t k0 = 0; k0 < d; k0 += 2)
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(qrow[k0 + half], hb[k0 + half], acc, 0, 0, 0);
        const float f = diagonal(acc, lane);
        if (split_not_finite(s)) s = f;
    }
    return s;
}

__device__ __forceinline__ int64_t lower_bound_i64(const int64_t *__restrict__ a, int64_t n, int64_t x)
{
    int64_t lo = 0, hi = n;
    while (lo < hi) {
        const int64_t mid = lo + ((hi - lo) >> 1);
        if (a[mid] < x) lo = mid + 1; else hi = mid;
    }
    return lo;
}

struct FilterTables {
    const int64_t *key[2]; const int32_t *val[2]; int64_t n[2]; int64_t N; int32_t R;
};

constexpr int PQ = 32, PW = 8;             // queries and wavefronts of a block of k_eval_pairs

// The known answers of a block's PQ queries laid end to end, query i's from place ptr[i] on: the query at place `at`.
// A place past the last one (the rest of the last tile, whose rows are read all the same) has the block's first query: the
// block may hold fewer than PQ.
using PairPlace = int64_t;                  // 32 lists of up to 2^31 entities
__host__ __device__ __forceinline__ int query_at(const PairPlace *ptr, PairPlace at)
{
    int i = 0;                             // the last query that starts at or before `at`
#pragma unroll
    for (int step = PQ / 2; step > 0; step >>= 1) if (ptr[i + step] <= at) i += step;
    return at < ptr[PQ] ? i : 0;
}

// The answers' scores and, among the known answers of each query's (fixed entity, relation), how many others score
// above / exactly at them.  A block takes PQ queries.  Their answers are one matrix-core tile of 32 pairs; the known
// answers of all its queries are laid end to end and cut into such tiles, dealt out over the block's wavefronts: most
// lists hold a handful of entities (a tile of their own would be nearly empty) and a hub's hundreds are not one
// wavefront's chain.  A block's queries lie a grid apart: neighbours in a test file often share a hub, whose list is as long
// for each of them.  Bound by the gathered rows (a load touches 32 of them).  40,932 queries of the 14,541-entity graph at
// width 200: 676 us with one wavefront and one tile per query and fp32 steps, 187 with three bf16 parts, 207 with two
// fp16 parts and the bounds on what they lose (545 with conditions around the row loads: each then waits for the last).  HALF = false: three bf16 parts only, for
// narrow rows and small evaluations; both forms in one kernel take 94 registers and leave two blocks per compute unit, this one 78 and three.
template <bool HALF>
__global__ __launch_bounds__(64 * PW) void k_eval_pairs(const float *__restrict__ Q, const float *__restrict__ H,
                                                    int32_t d, int64_t nq, int64_t n_test,
                                                    int32_t *fixed, const int32_t *__restrict__ rel,
                                                    const int32_t *__restrict__ answer, FilterTables ft,
                                                    EvalRange *range,
                                                    float *__restrict__ s_answer, int32_t *__restrict__ out_gt,
                                                    unsigned *__restrict__ cnt_eq)
{
    __shared__ int64_t bound[2 * PQ];
    __shared__ PairPlace ptr[PQ + 1];
    __shared__ int32_t gt_s[PQ], eq_s[PQ];
    __shared__ float thr[PQ];
    __shared__ bool three[PQ];                              // the query needs three parts
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int64_t step = gridDim.x;                         // the block's queries: blockIdx.x, and every step-th after it
    auto query = [&](int i) { return (int64_t)blockIdx.x + i * step; };
    const int n_here = (int)((nq - 1 - blockIdx.x) / step) + 1;
    EvalScale sc;
    if constexpr (HALF) sc = eval_scale(range);
    auto scores = [&](const float *qrow, int32_t ent, bool by_three) __attribute__((always_inline)) {
        if constexpr (HALF)
            if (sc.half) {
                float s = pair_scores<2>(qrow, H, ent, d, lane, sc.h, sc.q) * sc.inv;
                if (__any(by_three)) {
                    const float x = pair_scores<3>(qrow, H, ent, d, lane, 1.f, 1.f);
                    if (by_three) s = x;
                }
                return s;
            }
        return pair_scores<3>(qrow, H, ent, d, lane, 1.f, 1.f);
    };
    if (t < 2 * PQ) {                                       // ends of the queries' ranges in the tables, by wavefront 0
        const int i = t >> 1;
        int64_t pos = 0;
        if (i < n_here) {
            const int64_t q = query(i);
            const int side = q >= n_test ? 1 : 0;
            const int64_t base = ((int64_t)fixed[q] * ft.R + rel[q]) * ft.N;
            pos = lower_bound_i64(ft.key[side], ft.n[side], (t & 1) ? base + ft.N : base);
        }
        bound[t] = pos;
    } else if (w == 1) {                                    // the answers' scores, by wavefront 1
        const int i = lane & 31;
        const int64_t q = query(i < n_here ? i : 0);
        const float s = scores(Q + q * d, i < n_here ? answer[q] : -1, false);
        if (lane < n_here) { thr[lane] = s; s_answer[q] = s; }
    } else {
        if (w == 2 && lane < PQ) { gt_s[lane] = 0; eq_s[lane] = 0; }
        if (HALF && sc.half)                                // which queries need three parts, by the others
            for (int i = w - 2; i < n_here; i += PW - 2) {
                const int64_t q = query(i);
                const float4 *qr = reinterpret_cast<const float4 *>(Q + q * d), *hr = reinterpret_cast<const float4 *>(H + (int64_t)answer[q] * d);
                LossBound b;
                for (int32_t c = lane; c < d / 4; c += 64) {
                    const float4 x = qr[c], y = hr[c];
                    b.add(x.x, y.x, sc); b.add(x.y, y.y, sc); b.add(x.z, y.z, sc); b.add(x.w, y.w, sc);
                }
                for (int off = 32; off > 0; off >>= 1) {
                    b.q_sum += __shfl_xor(b.q_sum, off, 64); b.terms += __shfl_xor(b.terms, off, 64); b.q_small += __shfl_xor(b.q_small, off, 64);
                }
                if (lane == 0) three[i] = b.too_large(sc);
            }
    }
    __syncthreads();
    if (HALF && sc.half && w == 1) {
        const int i = lane & 31;
        const int64_t q = query(i < n_here ? i : 0);
        const bool by_three = i < n_here && three[i];
        if (__any(by_three)) {
            const float s = pair_scores<3>(Q + q * d, H, by_three ? answer[q] : -1, d, lane, 1.f, 1.f);
            if (lane < n_here && by_three) { thr[lane] = s; s_answer[q] = s; }
            const int n = __popcll(__ballot(lane < n_here && by_three));
            if (lane == 0) atomicAdd(&range->at[0].n_three, (uint32_t)n);
        }
        // k_eval_count finds it where the query's entity was, which only this block reads and wavefront 0 has read
        if (lane < n_here) fixed[q] = by_three ? 1 : 0;
    }
    if (w == 0) {                                           // where each query's known answers start in the block's row
        PairPlace x = lane < PQ ? (PairPlace)(bound[2 * lane + 1] - bound[2 * lane]) : 0;
        const PairPlace own = x;
        for (int off = 1; off < PQ; off <<= 1) { const PairPlace y = __shfl_up(x, off, 64); if (lane >= off) x += y; }
        if (lane < PQ) { ptr[lane] = x - own; if (lane == PQ - 1) ptr[PQ] = x; }
    }
    __syncthreads();
    const PairPlace n_pairs = ptr[PQ];
    for (PairPlace b = w * 32; b < n_pairs; b += PW * 32) {  // bounds are the same in every lane
        const PairPlace at = b + (lane & 31);
        const int i = query_at(ptr, at);
        const int64_t q = query(i);
        int32_t e = -1;
        if (at < n_pairs) {
            e = ft.val[q >= n_test ? 1 : 0][bound[2 * i] + (at - ptr[i])];
            if (e == answer[q]) e = -1;
        }
        const float s = scores(Q + q * d, e, HALF && sc.half && e >= 0 && three[i]);
        if (lane < 32 && e >= 0) {
            if (s > thr[i]) atomicAdd(gt_s + i, 1);
            if (s == thr[i]) atomicAdd(eq_s + i, 1);
        }
    }
    __syncthreads();
    if (t < n_here) { out_gt[query(t)] = gt_s[t]; cnt_eq[query(t)] = 0u - (unsigned)eq_s[t]; }
}

// Candidate lists: one wavefront per query, LPR lanes per entity row (LPR * 4 >= min(d, 256) columns at a
// time), 64 / LPR rows side by side and UN such groups in flight.  A score is the row's fp32 dot product
// with the query vector summed in a fixed order (per lane over its column pieces, then a butterfly over the
// row's lanes), the answer's score included, so equal rows give equal scores.
//
// A lane past the row's width loads nothing: the first-level cache hands out 64 bytes per cycle, lanes that only repeat
// a column included (3000 queries x 200 candidates at d = 200: 134 us, 98 without them).  Rows of a part of the
// wavefront's lanes stand under one condition per round (d = 36: 26.4 us, 29.0 under one each); a row of all 64, and an
// index of its list, under its own (150,000 entities, 5000 queries x 500 at d = 200: 305 us, 323 under one per round, 310
// with the indices under one each and the rows under one; d = 132: 240, 248, 246).
template <int LPR, int NP, int UN, bool FULL>
__device__ __forceinline__ void row_dots(const float4 *__restrict__ H, const int32_t (&e)[UN], const float4 (&q4)[NP], int32_t d4,
                                         int sub, float (&s)[UN])
{
    float4 h[NP][UN];
    if constexpr (!FULL && LPR == 64) {
#pragma unroll
        for (int u = 0; u < UN; ++u)
#pragma unroll
            for (int j = 0; j < NP; ++j)
                h[j][u] = sub + j * LPR < d4 ? H[(int64_t)(e[u] < 0 ? 0 : e[u]) * d4 + sub + j * LPR] : make_float4(0.f, 0.f, 0.f, 0.f);
    } else {
#pragma unroll
        for (int j = 0; j < NP; ++j) {
#pragma unroll
            for (int u = 0; u < UN; ++u) h[j][u] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (FULL || sub + j * LPR < d4)
#pragma unroll
                for (int u = 0; u < UN; ++u) h[j][u] = H[(int64_t)(e[u] < 0 ? 0 : e[u]) * d4 + sub + j * LPR];
        }
    }
#pragma unroll
    for (int u = 0; u < UN; ++u) {
        s[u] = 0.f;
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            s[u] = fmaf(h[j][u].x, q4[j].x, s[u]); s[u] = fmaf(h[j][u].y, q4[j].y, s[u]);
            s[u] = fmaf(h[j][u].z, q4[j].z, s[u]); s[u] = fmaf(h[j][u].w, q4[j].w, s[u]);
        }
    }
}

// NP: column pieces per lane, LPR * NP * 4 >= d; FULL: equal (no condition at all: 93 us at d = 256, 100 with it)
template <int LPR, int NP, bool FULL>
__global__ __launch_bounds__(256) void k_eval_candidates(const float4 *__restrict__ Q, const float4 *__restrict__ H,
                                                         int32_t d4, int64_t nq, const int32_t *__restrict__ answer,
                                                         const int32_t *__restrict__ cand, int32_t n_cand,
                                                         int32_t *__restrict__ out_gt, int32_t *__restrict__ out_eq)
{
    constexpr int RPP = 64 / LPR, UN = NP > 2 ? 2 : 4;         // rows per pass, passes in flight
    const int lane = threadIdx.x & 63, sub = lane % LPR, grp = lane / LPR;
    const int64_t q = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (q >= nq) return;                                    // whole wavefronts leave
    float4 q4[NP];
#pragma unroll
    for (int j = 0; j < NP; ++j) q4[j] = sub + j * LPR < d4 ? Q[q * d4 + sub + j * LPR] : make_float4(0.f, 0.f, 0.f, 0.f);
    const int32_t ans = answer[q];
    auto reduce = [&](float s) {
#pragma unroll
        for (int off = LPR / 2; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
        return s;
    };
    const int32_t own[1] = {ans};
    float st[1];
    row_dots<LPR, NP, 1, FULL>(H, own, q4, d4, sub, st);
    st[0] = reduce(st[0]);
    const int32_t *list = cand + q * n_cand;
    int gt = 0, eq = 0;
    for (int32_t b = 0; b < n_cand; b += RPP * UN) {         // bounds are the same in every lane
        int32_t e[UN];
        float s[UN];
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const int32_t i = b + u * RPP + grp;
            if constexpr (!FULL && LPR == 64) e[u] = i < n_cand ? list[i] : -1;
            else e[u] = list[i < n_cand ? i : n_cand - 1];
            if (i >= n_cand || e[u] == ans) e[u] = -1;
        }
        row_dots<LPR, NP, UN, FULL>(H, e, q4, d4, sub, s);
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const float r = reduce(s[u]);
            if (sub == 0 && e[u] >= 0) { gt += r > st[0] ? 1 : 0; eq += r == st[0] ? 1 : 0; }
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) { gt += __shfl_xor(gt, off, 64); eq += __shfl_xor(eq, off, 64); }
    if (lane == 0) { out_gt[q] = gt; out_eq[q] = eq; }
}

// ---- all entities.  A block of 8 wavefronts takes QN queries and walks `tiles_per_block` consecutive tiles of EM
// entities; a wavefront owns WI x WJ accumulators of 32 entities x 32 queries, the wavefronts 2 x 4 of those.  The query
// is the accumulator's column, so a lane has one threshold and one pair of counts per 32 queries, kept in registers over
// all tiles.  16-deep steps: a step's rows are split into LDS ([part][row][k]; three parts: two buffers, two parts: three) one
// step ahead, with two parts two ahead, their loads issued one step before that, one barrier per step, also from one tile to the next.
// Bound by the matrix cores, which run at 1.7 GHz under this load and are 61 % busy; the rest goes to the barrier of a step
// and to what no product covers.  20,000 queries x 1 M entities at width 256, NP = 2: 27.6 ms (371 TFLOP/s, 1.1 PFLOP/s of
// fp16 products); NP = 3, six products per term: 49 (208); fp32 steps: 88.6.  40,932 x 14,541 at width 200: 0.83 ms, 1.34
// with NP = 3.
constexpr int ELP = 48;                       // bytes per LDS row: 16 bf16 and 16 of padding (an odd multiple of 16)


// Blocks of a count over row_tiles x col_tiles tiles: about 2048 (8 rounds of one per compute unit) when there is that much
// work, the chunk count a multiple of the patch width when it exceeds it
struct CountGrid { int32_t tiles_per_block, col_tiles, row_tiles, col_chunks; int64_t blocks; };
__host__ __device__ inline CountGrid count_grid(int64_t row_tiles, int64_t col_tiles)
{
    int64_t col_chunks = cdiv(2048, row_tiles);
    if (col_chunks > 4) col_chunks = cdiv(col_chunks, 4) * 4;
    if (col_chunks > col_tiles) col_chunks = col_tiles;
    const int64_t tpb = cdiv(col_tiles, col_chunks);
    col_chunks = cdiv(col_tiles, tpb);
    const int64_t patches = cdiv(row_tiles, 8) * cdiv(col_chunks, 4);
    return CountGrid{(int32_t)tpb, (int32_t)col_tiles, (int32_t)row_tiles, (int32_t)col_chunks, cdiv(patches, 8) * 8 * 32};     // whole rounds of 8 patches, 32 blocks each
}

// block id -> (query tile, chunk of entity tiles); false: a padding block of the edge patches.  Workgroup i runs on XCD i % 8,
// each with its own L2.  The (query tile, chunk) space is cut into 8 x 4 patches; a patch goes to one XCD and is what that XCD
// runs at a time (32 blocks), so its L2 holds 8 query tiles, re-read at every entity tile, and 4 streams of entity tiles, each
// shared by 8 blocks.
__device__ __forceinline__ bool count_place(const CountGrid &g, int64_t block, int64_t &row_tile, int64_t &chunk)
{
    const int64_t slot = block / 8, xcd = block % 8;
    const int64_t patch = (slot / 32) * 8 + xcd;
    const int r32 = (int)(slot % 32);
    const int64_t patches_r = (g.row_tiles + 7) / 8;
    row_tile = (patch % patches_r) * 8 + r32 % 8;
    chunk = (patch / patches_r) * 4 + r32 / 8;
    return row_tile < g.row_tiles && chunk < g.col_chunks;
}

// The block's queries are those from q0 on, or, with `ids`, those named there.  three (NP = 2): queries that three parts rank
template <int WI, int WJ, bool DUMP, int NP, bool IDS>
__device__ __forceinline__ void count_tiles(unsigned char *lds, const EvalScale sc, int64_t row_tile, int64_t chunk,
                                            const int32_t *ids, const int32_t *__restrict__ three, const float *__restrict__ Q, int64_t nq,
                                            const float *__restrict__ H, int64_t N, int32_t d,
                                            const float *__restrict__ s_answer, int32_t tiles_per_block, int32_t n_col_tiles,
                                            unsigned *__restrict__ cnt_gt, unsigned *__restrict__ cnt_eq,
                                            float *__restrict__ dump)
{
    constexpr int EM = 64 * WI, QN = 128 * WJ, NA = EM / 128, NB = QN / 128;
    constexpr int PA = EM * ELP, PB = QN * ELP, BUF = NP * (PA + PB);      // bytes of a part of either operand, of a buffer
    const int t = threadIdx.x, lane = t & 63, half = lane >> 5;
    const int w = __builtin_amdgcn_readfirstlane(t >> 6), we = w >> 2, wq = w & 3;
    const int64_t q0 = row_tile * QN;
    const int32_t ct_beg = (int32_t)chunk * tiles_per_block;
    const int32_t ct_end = ct_beg + tiles_per_block < n_col_tiles ? ct_beg + tiles_per_block : n_col_tiles;

    // rows r_ld + 128 * pass of either operand, 4 consecutive k; rows and k past the end repeat the last ones (such
    // rows are not counted, such k are zeroed in the entities)
    const int r_ld = t >> 2, k_ld = (t & 3) * 4;
    const float *qb = Q + (IDS ? 0 : q0 * d);
    const uint32_t q_last = (uint32_t)(nq - 1 - q0 < QN - 1 ? nq - 1 - q0 : QN - 1);
    const float sq = NP == 2 ? sc.q : 1.f;
    auto query = [&](int c) __attribute__((always_inline)) { return IDS ? (int64_t)ids[c] : q0 + c; };     // column c of the tile
    int32_t id_ld[NB];
#pragma unroll
    for (int ps = 0; ps < NB; ++ps) id_ld[ps] = IDS ? ids[min((uint32_t)(r_ld + ps * 128), q_last)] : 0;
    float4 ra[NA], rb[NB];
    int32_t lt = ct_beg, lk = 0, sk = 0;                    // tile and k of the next load, k of the next staging
    auto load = [&]() __attribute__((always_inline)) {
        const uint32_t k = (uint32_t)(lk + k_ld < d ? lk + k_ld : d - 4);
        const float *hb = H + (int64_t)lt * EM * d;
        const int64_t more = N - 1 - (int64_t)lt * EM;
        const uint32_t e_last = (uint32_t)(more < EM - 1 ? more : EM - 1);
#pragma unroll
        for (int ps = 0; ps < NA; ++ps)
            ra[ps] = *reinterpret_cast<const float4 *>(hb + (min((uint32_t)(r_ld + ps * 128), e_last) * (uint32_t)d + k));
#pragma unroll
        for (int ps = 0; ps < NB; ++ps)
            if constexpr (IDS) rb[ps] = *reinterpret_cast<const float4 *>(qb + (int64_t)id_ld[ps] * d + k);
            else rb[ps] = *reinterpret_cast<const float4 *>(qb + (min((uint32_t)(r_ld + ps * 128), q_last) * (uint32_t)d + k));
        lk += 16;
        if (lk >= d) { lk = 0; if (lt + 1 < ct_end) ++lt; }
    };
    // the two operands' rows of the next staging; entities' k past the width are zeroed
    auto stage_a = [&](unsigned char *L) __attribute__((always_inline)) {
        const float on = sk + k_ld < d ? sc.h : 0.f;
        unsigned char *at = L + r_ld * ELP + k_ld * 2;
#pragma unroll
        for (int ps = 0; ps < NA; ++ps) {
            const auto x = split_parts<NP>(ra[ps].x * on, ra[ps].y * on), y = split_parts<NP>(ra[ps].z * on, ra[ps].w * on);
#pragma unroll
            for (int p = 0; p < NP; ++p) *reinterpret_cast<uint2 *>(at + p * PA + ps * 128 * ELP) = make_uint2(x.w[p], y.w[p]);
        }
        sk = sk + 16 < d ? sk + 16 : 0;
    };
    auto stage_b = [&](unsigned char *L) __attribute__((always_inline)) {
        unsigned char *at = L + r_ld * ELP + k_ld * 2;
#pragma unroll
        for (int ps = 0; ps < NB; ++ps) {
            const auto x = split_parts<NP>(rb[ps].x * sq, rb[ps].y * sq), y = split_parts<NP>(rb[ps].z * sq, rb[ps].w * sq);
#pragma unroll
            for (int p = 0; p < NP; ++p) *reinterpret_cast<uint2 *>(at + NP * PA + p * PB + ps * 128 * ELP) = make_uint2(x.w[p], y.w[p]);
        }
    };
    auto stage = [&](unsigned char *L) __attribute__((always_inline)) { stage_a(L); stage_b(L); };

    float thr[WJ];
    unsigned gt[WJ], eq[WJ];
#pragma unroll
    for (int j = 0; j < WJ; ++j) {
        const int c = (wq * WJ + j) * 32 + (lane & 31);
        // two parts: scores come times a power of two, and so does what they are compared with (no bit is lost either way:
        // a sum of fp16 products is no smaller than 2^-48, and the powers are limited); nothing is above or at infinity
        thr[j] = q0 + c < nq && !(NP == 2 && three[q0 + c]) ? s_answer[query(c)] * (NP == 2 ? sc.h * sc.q : 1.f) : INFINITY;
        gt[j] = eq[j] = 0u;
    }
    if constexpr (NP == 2) {
        bool any = false;
#pragma unroll
        for (int j = 0; j < WJ; ++j) any |= thr[j] != INFINITY;
        if (!__syncthreads_or(any)) return;
    }
    split_floatx16 acc[WI][WJ];
    auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < WI; ++i)
#pragma unroll
            for (int j = 0; j < WJ; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
    };
    // the tile's scores are complete: compare and count.  Register v of lane l: entity 8 (v / 4) + 4 (l / 32) + v % 4
    // of 32, query l % 32 of 32
    auto count = [&](int32_t ct) __attribute__((always_inline)) {
        const int64_t e0 = (int64_t)ct * EM + we * WI * 32;
        if constexpr (NP == 3) {
            float most = 0.f;          // v_maximum3_f32: two scores per instruction, a NaN stays
#pragma unroll
            for (int i = 0; i < WI; ++i)
#pragma unroll
                for (int j = 0; j < WJ; ++j)
#pragma unroll
                    for (int v = 0; v < 16; ++v) most = __builtin_elementwise_maximum(most, __builtin_fabsf(acc[i][j][v]));
            if (__any(split_not_finite(most))) {          // an infinity, a NaN or an overflow among the terms: such scores again, in fp32
#pragma unroll
                for (int i = 0; i < WI; ++i)
#pragma unroll
                    for (int j = 0; j < WJ; ++j) {
                        split_floatx16 f;
#pragma unroll
                        for (int v = 0; v < 16; ++v) f[v] = 0.f;
                        const int64_t e = e0 + i * 32 + (lane & 31);
                        const float *hp = H + (e < N ? e : N - 1) * d, *qr = Q + query(min((wq * WJ + j) * 32 + (lane & 31), (int)q_last)) * d;
                        for (int32_t k = half; k < d; k += 2) f = __builtin_amdgcn_mfma_f32_32x32x2f32(hp[k], qr[k], f, 0, 0, 0);
#pragma unroll
                        for (int v = 0; v < 16; ++v) if (split_not_finite(acc[i][j][v])) acc[i][j][v] = f[v];
                    }
            }
        }
        int32_t left = N - e0 < (int64_t)WI * 32 ? (int32_t)(N - e0) : WI * 32;            // entities of this wavefront's part
        if (NP == 2 && !DUMP && left == WI * 32) {
            // thr - s has its sign bit where s lies above (a difference of fp32 numbers is zero only if they are equal): the
            // signs are shifted into a word and counted 32 at a time, 2 instructions per score where a compare and an add
            // with carry wait for each other.  An equal score (a difference of +0 bits) is rare: one minimum over all.
            uint32_t least = 0xffffffffu;
#pragma unroll
            for (int j = 0; j < WJ; ++j)
#pragma unroll
                for (int i2 = 0; i2 < WI; i2 += 2) {
                    uint32_t above = 0u;
#pragma unroll
                    for (int v = 0; v < 32; v += 2) {
                        const uint32_t u = __float_as_uint(thr[j] - acc[i2 + v / 16][j][v % 16]);
                        const uint32_t x = __float_as_uint(thr[j] - acc[i2 + v / 16][j][v % 16 + 1]);
                        above = __builtin_amdgcn_alignbit(__builtin_amdgcn_alignbit(above, u, 31), x, 31);
                        asm("v_min3_u32 %0, %0, %1, %2" : "+v"(least) : "v"(u), "v"(x));      // one chain: a tree keeps them all
                    }
                    gt[j] += __popc(above);
                    asm volatile("" : "+v"(gt[j]));       // counted here, not behind the branch below
                }
            if (__any(least == 0u)) {
#pragma unroll
                for (int j = 0; j < WJ; ++j) {
                    float x = thr[j];
                    asm volatile("" : "+v"(x));           // keeps the comparisons in this branch
#pragma unroll
                    for (int i = 0; i < WI; ++i)
#pragma unroll
                        for (int v = 0; v < 16; ++v) eq[j] += acc[i][j][v] == x ? 1u : 0u;
                }
            }
        } else {
            asm volatile("" : "+s"(left));        // keeps the rows' conditions in this branch
#pragma unroll
            for (int i = 0; i < WI; ++i)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int row = i * 32 + 8 * (v >> 2) + 4 * half + (v & 3);
                    const bool in = row < left;
#pragma unroll
                    for (int j = 0; j < WJ; ++j) {
                        gt[j] += in && acc[i][j][v] > thr[j] ? 1u : 0u;
                        eq[j] += in && acc[i][j][v] == thr[j] ? 1u : 0u;
                        if (DUMP) {
                            const int c = (wq * WJ + j) * 32 + (lane & 31);
                            if (in && q0 + c < nq && !(NP == 2 && thr[j] == INFINITY))
                                dump[query(c) * N + e0 + row] = acc[i][j][v] * (NP == 2 ? sc.inv : 1.f);
                        }
                    }
                }
        }
        if (NP == 3) clear();
    };

    if (NP == 3 && ct_beg < ct_end) {
        load();
        stage(lds);
        load();
        clear();
        __syncthreads();
        const int off_a = (we * WI * 32 + (lane & 31)) * ELP + half * 16, off_b = NP * PA + (wq * WJ * 32 + (lane & 31)) * ELP + half * 16;
        int32_t ct = ct_beg, kc = 0;
        int cur = 0;
        while (true) {
            const unsigned char *L = lds + cur;
            cur ^= BUF;
            uint4 a[WI][NP], b[WJ][NP];
#pragma unroll
            for (int p = 0; p < NP; ++p) {
#pragma unroll
                for (int i = 0; i < WI; ++i) a[i][p] = *reinterpret_cast<const uint4 *>(L + off_a + p * PA + i * 32 * ELP);
#pragma unroll
                for (int j = 0; j < WJ; ++j) b[j][p] = *reinterpret_cast<const uint4 *>(L + off_b + p * PB + j * 32 * ELP);
            }
            stage(lds + cur);
            load();
#pragma unroll
            for (int p = 0; p < split_terms<NP>(); ++p)
#pragma unroll
                for (int i = 0; i < WI; ++i)
#pragma unroll
                    for (int j = 0; j < WJ; ++j) acc[i][j] = split_product<NP>(a[i][split_a<NP>(p)], b[j][split_b<NP>(p)], acc[i][j]);
            kc += 16;
            if (kc >= d) {
                count(ct);
                kc = 0;
                if (++ct == ct_end) break;
            }
            __syncthreads();
        }
    }
    if (NP == 2 && ct_beg < ct_end) {
        // Three buffers: while a step is multiplied, the one after next is split into LDS and the next one's operands are
        // read into the registers that the step no longer needs, so that no product waits for LDS.  The barrier stands
        // where the writes before it are long done and the reads behind it are needed eight products later.  A step's
        // three rounds of products are spread among the other instructions by hand (mix): clustered, they and the
        // splitting take turns, because all wavefronts keep the same step.
        const int off_a = (we * WI * 32 + (lane & 31)) * ELP + half * 16, off_b = NP * PA + (wq * WJ * 32 + (lane & 31)) * ELP + half * 16;
        uint4 ah[WI], al[WI], bh[WJ], bl[WJ];
        auto read_a = [&](const unsigned char *L, int p, uint4 (&x)[WI]) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < WI; ++i) x[i] = *reinterpret_cast<const uint4 *>(L + off_a + p * PA + i * 32 * ELP);
        };
        auto read_b = [&](const unsigned char *L, int p, uint4 (&x)[WJ]) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < WJ; ++j) x[j] = *reinterpret_cast<const uint4 *>(L + off_b + p * PB + j * 32 * ELP);
        };
        const split_floatx16 zero = {};
        auto multiply = [&](const uint4 (&x)[WI], const uint4 (&y)[WJ], auto fresh) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < WI; ++i)
#pragma unroll
                for (int j = 0; j < WJ; ++j) acc[i][j] = split_product<2>(x[i], y[j], decltype(fresh)::value ? zero : acc[i][j]);
        };
        auto mix = [&](auto valu) __attribute__((always_inline)) {
#pragma unroll
            for (int m = 0; m < WI * WJ; ++m) {
                __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);                      // one product
                __builtin_amdgcn_sched_group_barrier(0x2, decltype(valu)::value, 0);  // vector instructions
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        int nxt = BUF, after = 2 * BUF;
        auto step = [&](auto fresh) __attribute__((always_inline)) {
            const std::false_type more{};
            stage_a(lds + after);
            multiply(al, bh, fresh);
            mix(std::integral_constant<int, 4>{});
            read_a(lds + nxt, 1, al);
            stage_b(lds + after);
            multiply(ah, bh, more);
            mix(std::integral_constant<int, 4>{});
            __syncthreads();
            read_b(lds + nxt, 0, bh);
            load();
            multiply(ah, bl, more);
            mix(std::integral_constant<int, 3>{});
            read_a(lds + nxt, 0, ah);
            read_b(lds + nxt, 1, bl);
            nxt = after;
            after = after == 2 * BUF ? 0 : after + BUF;
        };
        load();
        stage(lds);
        load();
        stage(lds + BUF);
        load();
        __syncthreads();
        read_a(lds, 1, al); read_b(lds, 0, bh); read_a(lds, 0, ah); read_b(lds, 1, bl);
        for (int32_t ct = ct_beg; ct < ct_end; ++ct) {
            step(std::true_type{});
            for (int32_t kc = 16; kc < d; kc += 16) step(std::false_type{});
            count(ct);
        }
    }
#pragma unroll
    for (int j = 0; j < WJ; ++j) {
        gt[j] += __shfl_xor(gt[j], 32, 64);
        eq[j] += __shfl_xor(eq[j], 32, 64);
        const int c = (wq * WJ + j) * 32 + (lane & 31);
        if (lane < 32 && q0 + c < nq) {
            if (gt[j]) atomicAdd(cnt_gt + query(c), gt[j]);
            if (eq[j]) atomicAdd(cnt_eq + query(c), eq[j]);
        }
    }
}

// Numbers first .. first + QN - 1 of the queries that `three` marks, or of all of them, into ids (past the last one: any query)
template <int QN>
__device__ __forceinline__ void pick_queries(const int32_t *__restrict__ three, int64_t nq, bool marked, int64_t first, int32_t *ids)
{
    __shared__ int32_t before[8];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    if (!marked) {
        for (int i = t; i < QN; i += 512) ids[i] = (int32_t)(first + i < nq ? first + i : nq - 1);
        __syncthreads();
        return;
    }
    for (int i = t; i < QN; i += 512) ids[i] = 0;
    const int64_t per = cdiv(nq, 512), beg = t * per < nq ? t * per : nq, end = beg + per < nq ? beg + per : nq;
    int32_t n = 0;
    for (int64_t q = beg; q < end; ++q) n += three[q] ? 1 : 0;
    int32_t x = n;
    for (int off = 1; off < 64; off <<= 1) { const int32_t y = __shfl_up(x, off, 64); if (lane >= off) x += y; }
    if (lane == 63) before[w] = x;
    __syncthreads();
    int64_t at = x - n - first;
    for (int i = 0; i < w; ++i) at += before[i];
    for (int64_t q = beg; q < end; ++q)
        if (three[q]) { if (at >= 0 && at < QN) ids[at] = (int32_t)q; ++at; }
    __syncthreads();
}

// HALF: blocks [0, g.blocks) rank all queries by two parts; those that need three are left to the rest of the grid, which
// walks its own, smaller space of tiles.  Where no query can take two parts, the first blocks rank all of them by three.
// HALF = false: three parts (narrow rows, small evaluations).
template <int WI, int WJ, bool DUMP, bool HALF>
__global__ __launch_bounds__(512, 2) void k_eval_count(const EvalRange *__restrict__ range, const int32_t *__restrict__ three,
                                                    const float *__restrict__ Q,
                                                    int64_t nq, const float *__restrict__ H, int64_t N, int32_t d,
                                                    const float *__restrict__ s_answer, CountGrid g,
                                                    unsigned *__restrict__ cnt_gt,
                                                    unsigned *__restrict__ cnt_eq, float *__restrict__ dump)
{
    // two buffers of three parts or three of two
    __shared__ __attribute__((aligned(16))) unsigned char lds[6 * (64 * WI + 128 * WJ) * ELP];
    int64_t row_tile, chunk;
    if constexpr (!HALF) {
        if (count_place(g, blockIdx.x, row_tile, chunk))
            count_tiles<WI, WJ, DUMP, 3, false>(lds, EvalScale{}, row_tile, chunk, nullptr, nullptr, Q, nq, H, N, d, s_answer,
                                                g.tiles_per_block, g.col_tiles, cnt_gt, cnt_eq, dump);
    } else {
        __shared__ int32_t ids[128 * WJ];
        const EvalScale sc = eval_scale(range);
        const bool rest = blockIdx.x >= g.blocks;
        if (sc.half && !rest) {
            if (count_place(g, blockIdx.x, row_tile, chunk))
                count_tiles<WI, WJ, DUMP, 2, false>(lds, sc, row_tile, chunk, nullptr, three, Q, nq, H, N, d, s_answer,
                                                    g.tiles_per_block, g.col_tiles, cnt_gt, cnt_eq, dump);
            return;
        }
        const int64_t n = sc.half ? range->at[0].n_three : nq;
        if (sc.half != rest || n == 0) return;
        const CountGrid own = rest ? count_grid(cdiv(n, 128 * WJ), g.col_tiles) : g;
        const int64_t first = rest ? blockIdx.x - g.blocks : blockIdx.x, step = rest ? gridDim.x - g.blocks : own.blocks;
        for (int64_t block = first; block < own.blocks; block += step) {
            if (!count_place(own, block, row_tile, chunk)) continue;
            __syncthreads();                              // the block before has read its operands
            pick_queries<128 * WJ>(three, nq, rest, row_tile * (128 * WJ), ids);
            count_tiles<WI, WJ, DUMP, 3, true>(lds, EvalScale{}, row_tile, chunk, ids, nullptr, Q, n, H, N, d, s_answer,
                                               own.tiles_per_block, own.col_tiles, cnt_gt, cnt_eq, dump);
        }
    }
}

// EvalRange of H (blocks [0, h_blocks)) and of Q (the rest), as bits of absolute values: ordered as the numbers are, infinities
// above them and NaN above those.  n4: pieces of 4 numbers.  `out` comes initialised.
// Bound by a launch and the atomics, which take turns where they meet: few large blocks, eight loads of a thread in flight, and
// four places for them.  60,000 x 80: 8 us, 28 with 1024 blocks of four loads on one place; 1 M x 256: 174 us, 5.9 TB/s.
constexpr int RANGE_T = 1024, RANGE_BLOCKS = 256;
__global__ __launch_bounds__(RANGE_T) void k_eval_range(const uint4 *__restrict__ H, int64_t h_n4, const uint4 *__restrict__ Q, int64_t q_n4,
                                                        int32_t h_blocks, EvalRange *__restrict__ out)
{
    constexpr int U = 8, NW = RANGE_T / 64;
    __shared__ uint32_t red[2][NW];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const bool is_h = (int)blockIdx.x < h_blocks;
    const uint4 *X = is_h ? H : Q;
    const int64_t n = is_h ? h_n4 : q_n4;
    const int64_t block = is_h ? blockIdx.x : blockIdx.x - h_blocks, step = (is_h ? h_blocks : gridDim.x - h_blocks) * (int64_t)RANGE_T;
    uint32_t most = 0u, least = 0xffffffffu;
    for (int64_t c0 = block * RANGE_T + threadIdx.x; c0 < n; c0 += U * step) {
        uint4 x[U];
#pragma unroll
        for (int u = 0; u < U; ++u) { const int64_t c = c0 + u * step; x[u] = X[c < n ? c : c0]; }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t y[4] = {x[u].x & 0x7fffffffu, x[u].y & 0x7fffffffu, x[u].z & 0x7fffffffu, x[u].w & 0x7fffffffu};
            most = max(most, max(max(y[0], y[1]), max(y[2], y[3])));
            least = min(least, min(min(y[0] - 1u, y[1] - 1u), min(y[2] - 1u, y[3] - 1u)));      // a zero: the largest there is
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        most = max(most, (uint32_t)__shfl_xor((int)most, off, 64));
        least = min(least, (uint32_t)__shfl_xor((int)least, off, 64));
    }
    if (lane == 0) { red[0][w] = most; red[1][w] = least; }
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int i = 1; i < NW; ++i) { most = max(most, red[0][i]); least = min(least, red[1][i]); }
        EvalRange::Place *at = &out->at[block & 3];
        uint32_t *hi = is_h ? &at->max_h : &at->max_q;
        if (most > __hip_atomic_load(hi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(hi, most);
        if (is_h && least < __hip_atomic_load(&at->least_h, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMin(&at->least_h, least);
    }
}

// higher = above - above among the filtered; equal = equal - equal among the filtered (where the counter started) - the
// answer itself
__global__ void k_eval_finish(const unsigned *__restrict__ cnt_gt, const unsigned *__restrict__ cnt_eq,
                              const int32_t *__restrict__ sub_gt, int64_t nq,
                              int32_t *__restrict__ higher, int32_t *__restrict__ equal)
{
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= nq) return;
    const int64_t g = (int64_t)cnt_gt[q] - sub_gt[q], e = (int64_t)(int32_t)cnt_eq[q] - 1;
    higher[q] = (int32_t)(g > 0 ? g : 0);
    equal[q] = (int32_t)(e > 0 ? e : 0);
}

struct Ks { int32_t k[8]; int32_t n; };

// One block: the sum of 1 / rank in double, in a fixed order, and the numbers of ranks up to each k.  Bound by one compute
// unit's instructions and a few memory round trips: 8 queries of a thread in flight, ranks doubled so that they are whole
// numbers r < 2^33, the reciprocal from v_rcp_f64 and two Newton steps, which round as a division does: the first leaves a
// relative error below 2^-46, the second rounds a value within 2^-91 of 1 / r, and no point halfway between two doubles lies
// within 2^-87 of it, being m / 2^k with k <= 54 + 33 and m r a whole number other than 2^k.  (The full division takes twice
// the instructions.)  40,932 queries: 22 us, 32 with divisions, conditions per k and 4 in flight.
__global__ __launch_bounds__(1024) void k_eval_metrics(const int32_t *__restrict__ higher,
                                                       const int32_t *__restrict__ equal, int64_t nq, Ks ks,
                                                       double *__restrict__ out)
{
    constexpr int UN = 8;
    __shared__ double red[16];
    __shared__ uint32_t hits[16][8];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    double s = 0.0;
    uint32_t n[8], k2[8];                                   // 2 k; a k below 1, or none: no rank is that small
#pragma unroll
    for (int j = 0; j < 8; ++j) { n[j] = 0u; k2[j] = j < ks.n && ks.k[j] > 0 ? 2u * (uint32_t)ks.k[j] : 0u; }
    for (int64_t q0 = threadIdx.x; q0 < nq; q0 += UN * 1024) {
        int32_t h[UN], e[UN];
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const int64_t q = q0 + u * 1024 < nq ? q0 + u * 1024 : nq - 1;
            h[u] = higher[q];
            e[u] = equal[q];
        }
        uint32_t c2[UN];                                    // twice the rank; past the last query: above every 2 k
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const bool in = q0 + u * 1024 < nq;
            const int64_t r2 = 2 + 2 * (int64_t)h[u] + e[u];
            c2[u] = !in || r2 > 0xffffffffll ? 0xffffffffu : r2 < 1 ? 1u : (uint32_t)r2;
            const double r = (double)r2;
            double x = __builtin_amdgcn_rcp(r);
            x = __builtin_fma(__builtin_fma(-r, x, 1.0), x, x);
            x = __builtin_fma(__builtin_fma(-r, x, 1.0), x, x);
            if (r2 <= 0) x = 1.0 / r;                       // no counts of a ranking
            s += in ? x : 0.0;
        }
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (j < ks.n)
#pragma unroll
                for (int u = 0; u < UN; ++u) n[j] += c2[u] <= k2[j] ? 1u : 0u;
    }
    s *= 2.0;
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
    if (lane == 0) red[w] = s;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        for (int off = 32; off > 0; off >>= 1) n[j] += __shfl_xor(n[j], off, 64);
        if (lane == 0) hits[w][j] = n[j];
    }
    __syncthreads();
    const int t = (int)threadIdx.x;
    if (t <= ks.n) {
        double x = 0.0;
        if (t == 0) for (int i = 0; i < 16; ++i) x += red[i];
        else for (int i = 0; i < 16; ++i) x += (double)hits[i][t - 1];
        out[t] = nq > 0 ? x / (double)nq : 0.0;
    }
}

struct EvalWs {
    size_t off_fixed, off_rel, off_answer, off_Q, off_s, off_sub_gt, off_range, off_cnt_gt, off_cnt_eq, total;
};

EvalWs eval_layout(int64_t nq, int32_t d)
{
    EvalWs w;
    size_t cur = 0;
    const size_t n = (size_t)(nq > 0 ? nq : 1);
    auto take = [&](size_t bytes) { size_t o = cur; cur = align_up(cur + bytes, 256); return o; };
    w.off_fixed = take(n * 4); w.off_rel = take(n * 4); w.off_answer = take(n * 4);
    w.off_Q = take(n * (size_t)d * 4); w.off_s = take(n * 4);
    w.off_sub_gt = take(n * 4); w.off_range = take(n * 4);      // 256 bytes are used
    w.off_cnt_gt = take(n * 4); w.off_cnt_eq = take(n * 4);
    w.total = cur;
    return w;
}

int check_model(const float *H, int64_t n_entities, int32_t d, const float *M, int32_t n_relations)
{
    KGE_REQUIRE(H && M, KGE_EINVAL, "H or M is NULL");
    KGE_REQUIRE(n_entities > 0 && n_entities <= 0x7FFFFFFFll && n_relations > 0, KGE_EINVAL,
                "n_entities must be in [1, 2^31) and n_relations positive");
    KGE_REQUIRE(d > 0 && d % 4 == 0 && d <= 1024, KGE_EINVAL, "d must be a multiple of 4 in [4, 1024]");
    KGE_REQUIRE(((uintptr_t)H % 16) == 0 && ((uintptr_t)M % 16) == 0, KGE_EINVAL, "H and M must be 16-byte aligned");
    return KGE_OK;
}

int check_ws(void *workspace, size_t ws_bytes, int64_t nq, int32_t d, EvalWs *w)
{
    *w = eval_layout(nq, d);
    KGE_REQUIRE(workspace && ((uintptr_t)workspace % 256) == 0, KGE_EINVAL, "workspace must be 256-byte aligned");
    KGE_REQUIRE(ws_bytes >= w->total, KGE_ENOMEM, "workspace has %zu bytes, %zu needed", ws_bytes, w->total);
    return KGE_OK;
}

template <int WI, int WJ>
int launch_count_tiles(const EvalRange *range, const int32_t *three, const float *Q, int64_t nq, const float *H, int64_t N, int32_t d,
                       const float *s_answer, unsigned *cnt_gt, unsigned *cnt_eq, float *dump, hipStream_t st)
{
    const CountGrid g = count_grid(cdiv(nq, 128 * WJ), cdiv(N, 64 * WI));
    const int64_t blocks = g.blocks + (range ? 256 : 0);     // one per compute unit for queries that need three parts
    KGE_REQUIRE(blocks <= 0x7FFFFFFFll, KGE_ERANGE, "evaluation grid too large");
#define EC_CALL(DUMPV, HALFV)                                                                                             \
    k_eval_count<WI, WJ, DUMPV, HALFV><<<(unsigned)blocks, 512, 0, st>>>(range, three, Q, nq, H, N, d, s_answer, g, cnt_gt, cnt_eq, dump)
    if (range) { if (dump) EC_CALL(true, true); else EC_CALL(false, true); }
    else { if (dump) EC_CALL(true, false); else EC_CALL(false, false); }
#undef EC_CALL
    KGE_LAUNCH_CHECK();
    return KGE_OK;
}

int launch_count(const EvalRange *range, const int32_t *three, const float *Q, int64_t nq, const float *H, int64_t N, int32_t d, const float *s_answer,
                 unsigned *cnt_gt, unsigned *cnt_eq, float *dump, hipStream_t st)
{
    // 256 x 256 tiles halve the splitting per product; with fewer of them than compute units (256) most of the chip
    // would wait for them, and 128 x 128 tiles spread the work
    if (cdiv(nq, 256) * cdiv(N, 256) >= 256) return launch_count_tiles<4, 2>(range, three, Q, nq, H, N, d, s_answer, cnt_gt, cnt_eq, dump, st);
    return launch_count_tiles<2, 1>(range, three, Q, nq, H, N, d, s_answer, cnt_gt, cnt_eq, dump, st);
}

// Two fp16 parts cost a launch that looks at the range, and k_eval_pairs blocks that hold both forms, two per compute unit
// instead of three; what they save grows with the products and, as each tile starts its chain of steps anew, with the width.
// Whole evaluations, us, three bf16 parts / two fp16 parts where possible: 5000 entities, d = 80, 5000 queries 78 / 85, 10,000
// queries 124 / 125; d = 128, 1000 queries 58 / 60, 3200 queries 85 / 83; d = 200, 1000 queries 74 / 72; 14,541 entities,
// d = 80, 2000 queries 79 / 82, 4000 queries 127 / 119; d = 96, 2000 queries 87 / 88; d = 128, 1000 queries 86 / 88, 2000
// queries 105 / 98; 60,000 entities, d = 80, 1000 queries 143 / 134.
bool two_parts_pay(int64_t nq, int64_t N, int32_t d) { return d >= HALF_FROM && (double)nq * (double)N * d * d >= 3.4e11; }

// Queries per block of k_eval_pairs: the most that leave 1024 blocks (four of them fill a compute unit), but no fewer than a
// block's wavefronts, so that long lists never get fewer wavefronts than queries.  2000 queries, half of them with
// 50,000 known answers, d = 64: 2.1 ms; one wavefront per query 5.7; always 32 neighbouring queries per block 19.2.  200
// queries with short lists at d = 200: 32 us, 48 with 32 per block.
int64_t pair_queries(int64_t nq) { return nq >= 1024 * PQ ? PQ : nq >= 1024 * PW ? nq / 1024 : PW; }

int rank_all(const kge_eval_filter *f, const float *H, int64_t N, int32_t d, const float *M, int32_t R,
             const int32_t *test_h, const int32_t *test_r, const int32_t *test_t, int64_t n_test, void *workspace,
             size_t ws_bytes, int32_t *higher, int32_t *equal, float *dump, float *dump_answer, hipStream_t st)
{
    int rc = check_model(H, N, d, M, R);
    if (rc != KGE_OK) return rc;
    KGE_REQUIRE(n_test >= 0 && n_test <= 0x3FFFFFFFll, KGE_EINVAL, "n_test out of range");
    KGE_REQUIRE(!f || (f->n_entities == N && f->n_relations == R), KGE_EINVAL,
                "the filter was built for other entity / relation counts");
    const int64_t nq = 2 * n_test;
    EvalWs w;
    rc = check_ws(workspace, ws_bytes, nq, d, &w);
    if (rc != KGE_OK) return rc;
    if (n_test == 0) return KGE_OK;
    KGE_REQUIRE(test_h && test_r && test_t && (dump || (higher && equal)), KGE_EINVAL, "NULL array");
    char *ws = (char *)workspace;
    int32_t *fixed = (int32_t *)(ws + w.off_fixed), *rel = (int32_t *)(ws + w.off_rel), *answer = (int32_t *)(ws + w.off_answer);
    float *Q = (float *)(ws + w.off_Q), *s = (float *)(ws + w.off_s);
    int32_t *sub_gt = (int32_t *)(ws + w.off_sub_gt);
    EvalRange *range = (EvalRange *)(ws + w.off_range);
    EvalRange *half_range = two_parts_pay(nq, N, d) ? range : nullptr;      // else three bf16 parts without a look
    unsigned *cnt_gt = (unsigned *)(ws + w.off_cnt_gt), *cnt_eq = (unsigned *)(ws + w.off_cnt_eq);
    {
        KGE_PROF("eval_queries", st);
        k_eval_queries<<<(unsigned)cdiv(nq * (d / 4), 256), 256, 0, st>>>(test_h, test_r, test_t, n_test, (const float4 *)H,
                                                                         (const float4 *)M, d / 4, fixed, rel, answer,
                                                                         (float4 *)Q, cnt_gt, range);
        KGE_LAUNCH_CHECK();
        if (half_range) {
            const int64_t h_n4 = N * (d / 4), q_n4 = nq * (d / 4);
            const int32_t h_blocks = (int32_t)std::min<int64_t>(cdiv(h_n4, RANGE_T), RANGE_BLOCKS), q_blocks = (int32_t)std::min<int64_t>(cdiv(q_n4, RANGE_T), RANGE_BLOCKS);
            k_eval_range<<<h_blocks + q_blocks, RANGE_T, 0, st>>>((const uint4 *)H, h_n4, (const uint4 *)Q, q_n4, h_blocks, range);
            KGE_LAUNCH_CHECK();
        }
    }
    {
        KGE_PROF("eval_pairs", st);
        FilterTables ft;
        for (int sde = 0; sde < 2; ++sde) {
            ft.key[sde] = f ? f->key[sde] : nullptr; ft.val[sde] = f ? f->val[sde] : nullptr; ft.n[sde] = f ? f->n[sde] : 0;
        }
        ft.N = N; ft.R = R;
        (half_range ? k_eval_pairs<true> : k_eval_pairs<false>)<<<(unsigned)cdiv(nq, pair_queries(nq)), 64 * PW, 0, st>>>(
            Q, H, d, nq, n_test, fixed, rel, answer, ft, half_range, dump_answer ? dump_answer : s, sub_gt, cnt_eq);
        KGE_LAUNCH_CHECK();
    }
    {
        KGE_PROF("eval_count", st);
        rc = launch_count(half_range, fixed, Q, nq, H, N, d, dump_answer ? dump_answer : s, cnt_gt, cnt_eq, dump, st);
        if (rc != KGE_OK) return rc;
    }
    if (higher && equal) {
        k_eval_finish<<<(unsigned)cdiv(nq, 256), 256, 0, st>>>(cnt_gt, cnt_eq, sub_gt, nq, higher, equal);
        KGE_LAUNCH_CHECK();
    }
    return KGE_OK;
}

}  // namespace

extern "C" int kge_eval_filter_create(const int32_t *head, const int32_t *rel, const int32_t *tail, int64_t n_known,
                                      int32_t n_entities, int32_t n_relations, kge_eval_filter **out)
{
    KGE_REQUIRE(out, KGE_EINVAL, "NULL argument");
    *out = nullptr;
    KGE_REQUIRE(n_known >= 0 && (n_known == 0 || (head && rel && tail)), KGE_EINVAL, "NULL triple arrays");
    KGE_REQUIRE(n_entities > 0 && n_relations > 0, KGE_EINVAL, "n_entities and n_relations must be positive");
    KGE_REQUIRE((double)n_entities * (double)n_relations * (double)n_entities < 9.0e18, KGE_ERANGE,
                "entity and relation counts too large for a 64-bit key");
    for (int64_t i = 0; i < n_known; ++i)
        KGE_REQUIRE(head[i] >= 0 && head[i] < n_entities && tail[i] >= 0 && tail[i] < n_entities && rel[i] >= 0 &&
                        rel[i] < n_relations, KGE_ERANGE, "known triple %lld has an id out of range", (long long)i);
    kge_eval_filter *f = new kge_eval_filter();
    f->n_entities = n_entities; f->n_relations = n_relations;
    for (int sde = 0; sde < 2; ++sde) { f->key[sde] = nullptr; f->val[sde] = nullptr; f->n[sde] = 0; }
    hipError_t e = hipGetDevice(&f->device);
    std::vector<int64_t> keys((size_t)n_known);
    std::vector<int32_t> vals;
    for (int sde = 0; sde < 2 && e == hipSuccess; ++sde) {
        const int32_t *fx = sde ? tail : head, *ot = sde ? head : tail;
        for (int64_t i = 0; i < n_known; ++i)
            keys[(size_t)i] = ((int64_t)fx[i] * n_relations + rel[i]) * n_entities + ot[i];
        std::sort(keys.begin(), keys.end());
        const size_t n = (size_t)(std::unique(keys.begin(), keys.end()) - keys.begin());
        vals.resize(n);
        for (size_t i = 0; i < n; ++i) vals[i] = (int32_t)(keys[i] % n_entities);
        f->n[sde] = (int64_t)n;
        e = hipMalloc((void **)&f->key[sde], (n ? n : 1) * sizeof(int64_t));
        if (e == hipSuccess) e = hipMalloc((void **)&f->val[sde], (n ? n : 1) * sizeof(int32_t));
        if (e == hipSuccess && n) e = hipMemcpy(f->key[sde], keys.data(), n * sizeof(int64_t), hipMemcpyHostToDevice);
        if (e == hipSuccess && n) e = hipMemcpy(f->val[sde], vals.data(), n * sizeof(int32_t), hipMemcpyHostToDevice);
        keys.resize((size_t)n_known);
    }
    if (e != hipSuccess) {
        kge_set_error("building the evaluation filter failed: %s", hipGetErrorString(e));
        kge_eval_filter_destroy(f);
        return KGE_EHIP;
    }
    *out = f;
    return KGE_OK;
}

extern "C" void kge_eval_filter_destroy(kge_eval_filter *f)
{
    if (!f) return;
    for (int sde = 0; sde < 2; ++sde) {
        if (f->key[sde]) (void)hipFree(f->key[sde]);
        if (f->val[sde]) (void)hipFree(f->val[sde]);
    }
    delete f;
}

extern "C" size_t kge_eval_workspace_bytes(int64_t n_queries, int32_t d)
{
    if (n_queries < 0 || d <= 0) { kge_set_error("negative query count or bad d"); return 0; }
    return eval_layout(n_queries, d).total;
}

extern "C" int kge_eval_rank_all(const kge_eval_filter *filter, const float *H, int64_t n_entities, int32_t d,
                                 const float *M, int32_t n_relations, const int32_t *test_h, const int32_t *test_r,
                                 const int32_t *test_t, int64_t n_test, void *workspace, size_t ws_bytes,
                                 int32_t *higher, int32_t *equal, void *stream)
{
    KGE_REQUIRE(n_test <= 0 || (higher && equal), KGE_EINVAL, "higher or equal is NULL");
    return rank_all(filter, H, n_entities, d, M, n_relations, test_h, test_r, test_t, n_test, workspace, ws_bytes,
                    higher, equal, nullptr, nullptr, (hipStream_t)stream);
}

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices];      // per device: where that GPU's copy of `scratch` lives

// Address of the current device's copy of `scratch`, looked up once per device with that device current.
int static_scratch_ptr(void **out)
{
    int dev = -1;
    KGE_HIP(hipGetDevice(&dev));
    KGE_REQUIRE(dev >= 0 && dev < kMaxDevices, KGE_EINVAL, "device index %d is outside [0, %d)", dev, kMaxDevices);
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        KGE_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
        KGE_REQUIRE(ptr && ((uintptr_t)ptr % 256) == 0, KGE_EHIP, "the static scratch array has no usable device address");
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return KGE_OK;
}
}  // namespace

extern "C" int kge_eval_rank_all_static(const kge_eval_filter *filter, const float *H, int64_t n_entities, int32_t d,
                                        const float *M, int32_t n_relations, const int32_t *test_h,
                                        const int32_t *test_r, const int32_t *test_t, int64_t n_test,
                                        int32_t *higher, int32_t *equal, void *stream)
{
    KGE_REQUIRE(n_test <= 0 || (higher && equal), KGE_EINVAL, "higher or equal is NULL");
    KGE_REQUIRE(n_test >= 0 && n_test <= 0x3FFFFFFFll && d > 0, KGE_EINVAL, "n_test or d out of range");
    const size_t need = eval_layout(2 * n_test, d).total;
    KGE_REQUIRE(need <= (size_t)KGE_EVAL_STATIC_BYTES, KGE_ENOMEM,
                "%lld test triples of width %d need %zu bytes of scratch; the static buffer holds %zu "
                "(use kge_eval_rank_all with a workspace)", (long long)n_test, d, need, (size_t)KGE_EVAL_STATIC_BYTES);
    void *ptr = nullptr;
    int rc = static_scratch_ptr(&ptr);
    if (rc != KGE_OK) return rc;
    return rank_all(filter, H, n_entities, d, M, n_relations, test_h, test_r, test_t, n_test, ptr,
                    (size_t)KGE_EVAL_STATIC_BYTES, higher, equal, nullptr, nullptr, (hipStream_t)stream);
}

extern "C" int32_t kge_test_pair_query(const int64_t *n_known, int32_t n_queries, int64_t at, int64_t *n_pairs)
{
    if (!n_known || !n_pairs || n_queries < 1 || n_queries > PQ) return -1;
    PairPlace ptr[PQ + 1] = {0};
    for (int i = 0; i < PQ; ++i) ptr[i + 1] = ptr[i] + (PairPlace)(i < n_queries ? n_known[i] : 0);
    *n_pairs = ptr[PQ];
    return query_at(ptr, (PairPlace)at);
}

extern "C" int kge_eval_debug_scores(const float *H, int64_t n_entities, int32_t d, const float *M, int32_t n_relations,
                                     const int32_t *test_h, const int32_t *test_r, const int32_t *test_t, int64_t n_test,
                                     void *workspace, size_t ws_bytes, float *scores, float *answer_score, void *stream)
{
    KGE_REQUIRE(scores && answer_score, KGE_EINVAL, "scores or answer_score is NULL");
    return rank_all(nullptr, H, n_entities, d, M, n_relations, test_h, test_r, test_t, n_test, workspace, ws_bytes,
                    nullptr, nullptr, scores, answer_score, (hipStream_t)stream);
}

extern "C" int kge_eval_rank_candidates(const float *H, int64_t n_entities, int32_t d, const float *M,
                                        int32_t n_relations, const int32_t *fixed, const int32_t *rel,
                                        const int32_t *answer, int64_t n_queries, const int32_t *cand, int32_t n_cand,
                                        void *workspace, size_t ws_bytes, int32_t *higher, int32_t *equal, void *stream)
{
    int rc = check_model(H, n_entities, d, M, n_relations);
    if (rc != KGE_OK) return rc;
    KGE_REQUIRE(n_queries >= 0 && n_queries <= 0x7FFFFFFFll && n_cand >= 0, KGE_EINVAL, "negative count");
    EvalWs w;
    rc = check_ws(workspace, ws_bytes, n_queries, d, &w);
    if (rc != KGE_OK) return rc;
    if (n_queries == 0) return KGE_OK;
    KGE_REQUIRE(fixed && rel && answer && higher && equal && (n_cand == 0 || cand), KGE_EINVAL, "NULL array");
    hipStream_t st = (hipStream_t)stream;
    char *ws = (char *)workspace;
    float *Q = (float *)(ws + w.off_Q);
    {
        KGE_PROF("eval_queries", st);
        k_eval_qvec<<<(unsigned)cdiv(n_queries * (d / 4), 256), 256, 0, st>>>((const float4 *)H, (const float4 *)M, fixed, rel,
                                                                             n_queries, d / 4, (float4 *)Q);
        KGE_LAUNCH_CHECK();
    }
    KGE_PROF("eval_cand", st);
    const unsigned grid = (unsigned)cdiv(n_queries, 4);
    const int32_t d4 = d / 4;
    const float4 *Q4 = (const float4 *)Q, *H4 = (const float4 *)H;
#define CAND_CALL(LPRV, NPV)                                                                                              \
    do {                                                                                                                 \
        if (d4 == LPRV * NPV) k_eval_candidates<LPRV, NPV, true><<<grid, 256, 0, st>>>(Q4, H4, d4, n_queries, answer, cand, n_cand, higher, equal); \
        else k_eval_candidates<LPRV, NPV, false><<<grid, 256, 0, st>>>(Q4, H4, d4, n_queries, answer, cand, n_cand, higher, equal); \
    } while (0)
    if (d4 <= 8) CAND_CALL(8, 1);
    else if (d4 <= 16) CAND_CALL(16, 1);
    else if (d4 <= 32) CAND_CALL(32, 1);
    else if (d4 <= 64) CAND_CALL(64, 1);
    else if (d4 <= 128) CAND_CALL(64, 2);
    else CAND_CALL(64, 4);
#undef CAND_CALL
    KGE_LAUNCH_CHECK();
    return KGE_OK;
}

extern "C" int kge_eval_metrics(const int32_t *higher, const int32_t *equal, int64_t n_queries, const int32_t *ks,
                                int32_t n_ks, double *out, void *stream)
{
    KGE_REQUIRE(out && n_queries >= 0 && (n_queries == 0 || (higher && equal)), KGE_EINVAL, "NULL array or negative count");
    KGE_REQUIRE(n_ks >= 0 && n_ks <= 8 && (n_ks == 0 || ks), KGE_EINVAL, "n_ks must be in [0, 8]");
    KGE_REQUIRE(((uintptr_t)out % 8) == 0, KGE_EINVAL, "out must be 8-byte aligned");
    Ks k;
    k.n = n_ks;
    for (int j = 0; j < 8; ++j) k.k[j] = j < n_ks ? ks[j] : 0;
    k_eval_metrics<<<1, 1024, 0, (hipStream_t)stream>>>(higher, equal, n_queries, k, out);
    KGE_LAUNCH_CHECK();
    return KGE_OK;
}
