// Neighbour aggregation of the RGCN layer (Eq. 1 with W_r = sum_b a_rb V_b, Eq. 2) and
// its backward counterparts.  All kernels here are bandwidth bound: they stream rows of
// the projected messages P[j][b][:] (or of the upstream gradient G) with 128-bit loads and do
// a handful of fp32 FMAs per loaded element.
//
// Work decomposition.  One wavefront per row (destination, source, or (relation, destination)
// run).  Rows with >= KGE_HEAVY edges are cut into units of KGE_HEAVY edges, one wavefront
// each, placed first in the grid; a unit writes a partial sum and a small finishing kernel adds
// the partials of a row in unit order.  No atomics, bit-reproducible results - but for the coefficient gradient's dot
// products of k_source_backward.
//
// Lane layout.  A row of `d` elements is covered by LPR lanes, each holding VEC consecutive
// elements (VEC = 4 for fp32, 8 for bf16: one 16-byte load).  The 64 / LPR lane groups of a
// wavefront work on different (edge, basis) pairs in parallel: GB of them across bases,
// GE = groups / GB across edges.
#include "common.h"

#include <algorithm>
#include <type_traits>

namespace {

constexpr int WPB = 4;                 // wavefronts per block

template <bool BF16> struct MsgRow;
template <> struct MsgRow<false> {
    static constexpr int VEC = 4;
    static __device__ __forceinline__ uint4 load_raw(const void *base, int64_t off)
    {
        return *reinterpret_cast<const uint4 *>(reinterpret_cast<const float *>(base) + off);
    }
    static __device__ __forceinline__ void unpack(const uint4 &x, float (&v)[4])
    {
        v[0] = __uint_as_float(x.x); v[1] = __uint_as_float(x.y);
        v[2] = __uint_as_float(x.z); v[3] = __uint_as_float(x.w);
    }
};
template <> struct MsgRow<true> {
    static constexpr int VEC = 8;
    static __device__ __forceinline__ uint4 load_raw(const void *base, int64_t off)
    {
        return *reinterpret_cast<const uint4 *>(reinterpret_cast<const uint16_t *>(base) + off);
    }
    static __device__ __forceinline__ void unpack(const uint4 &x, float (&v)[8])
    {
        v[0] = __uint_as_float(x.x << 16); v[1] = __uint_as_float(x.x & 0xffff0000u);
        v[2] = __uint_as_float(x.y << 16); v[3] = __uint_as_float(x.y & 0xffff0000u);
        v[4] = __uint_as_float(x.z << 16); v[5] = __uint_as_float(x.z & 0xffff0000u);
        v[6] = __uint_as_float(x.w << 16); v[7] = __uint_as_float(x.w & 0xffff0000u);
    }
};

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi)   // two fp32 -> packed bf16x2, nearest even
{
    // one v_cvt_pk_bf16_f32 on gfx950
    typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
    typedef float floatx2_t __attribute__((ext_vector_type(2)));
    const floatx2_t v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}

__device__ __forceinline__ float act_apply(int act, float x) { return act == KGE_ACT_RELU ? fmaxf(x, 0.f) : x; }

// Which row and edge range a wavefront works on.  Wavefronts [0, n_units) take the units of heavy
// rows; wavefront n_units + r takes light row r (and leaves at once if r is heavy).
struct RowWork {
    int64_t row;       // row id, or -1: nothing to do
    int32_t beg, end;  // edge range
    int32_t unit;      // >= 0: partial result goes to slot `unit`; -1: the row is finished here
};
__device__ __forceinline__ RowWork row_work(int64_t wid, const int32_t *__restrict__ ptr, int64_t n_rows,
                                            int32_t n_units, const int32_t *__restrict__ hv_row,
                                            const int32_t *__restrict__ hv_unit_ptr,
                                            const int32_t *__restrict__ unit_hv, int32_t heavy = KGE_HEAVY)
{
    RowWork w;
    if (wid < n_units) {
        const int32_t h = unit_hv[wid];
        w.row = hv_row[h];
        w.unit = (int32_t)wid;
        w.beg = ptr[w.row] + (int32_t)(wid - hv_unit_ptr[h]) * heavy;
        w.end = min(w.beg + heavy, ptr[w.row + 1]);
        return w;
    }
    w.row = wid - n_units;
    w.unit = -1;
    if (w.row >= n_rows) { w.row = -1; w.beg = w.end = 0; return w; }
    w.beg = ptr[w.row];
    w.end = ptr[w.row + 1];
    if (w.end - w.beg >= heavy) w.row = -1;
    return w;
}

// A sub-graph's size is known on the device only: of two forms of a sum that are both launched, one runs if the sub-graph has
// more than `at` edges and the other if not.  count null: always.
struct EdgeGate {
    const unsigned long long *count;
    unsigned long long at;
    __device__ __forceinline__ bool shut(bool above) const { return count && (*count > at) != above; }
};

// ------------------------------------------------------------------ forward
//   out[i][:] = act( sum_e invc_e sum_b a[rel_e][b] P[src_e][b][:] + Self[i][:] )
// PLAIN (B = 1, no coefficient table, dm_rel unused): out[i] = act( sum_e w_e P[idx_e] + Self[i] ),
// w = 1 if dm_invc is null.
template <bool BF16, int LPR, bool PLAIN>
__global__ __launch_bounds__(64 * WPB) void k_gather_fwd(
    const int32_t *__restrict__ dm_ptr, const int32_t *__restrict__ dm_src,
    const int32_t *__restrict__ dm_rel, const float *__restrict__ dm_invc, int64_t N,
    int32_t n_units, const int32_t *__restrict__ hv_row, const int32_t *__restrict__ hv_unit_ptr,
    const int32_t *__restrict__ unit_hv,
    const void *__restrict__ P, const float *__restrict__ a, int32_t B, int32_t d, int32_t gb_count,
    const float *__restrict__ Self, int act, float *__restrict__ out, float *__restrict__ out2,
    uint16_t *__restrict__ outbf, float *__restrict__ partial, const uint8_t *__restrict__ active, EdgeGate gate)
{
    if (gate.shut(PLAIN)) return;
    // outbf (optional): a bf16 copy of the output rows (the next layer's bf16 input, written here instead of by a
    // conversion pass over `out`)
    constexpr int VEC = MsgRow<BF16>::VEC;
    constexpr int G = 64 / LPR;
    constexpr int U = 8;
    const int lane = threadIdx.x & 63;
    const int64_t wid = (int64_t)blockIdx.x * WPB + (threadIdx.x >> 6);
    const int kl = lane % LPR, g = lane / LPR;
    if (active && wid >= n_units && wid - n_units < N && !active[wid - n_units]) {
        // a row outside the batch's sub-graph, seen before its edge range is even fetched: a zero row
        // (a heavy row's zeros are written once more by the finishing kernel)
        if (g == 0 && kl * VEC < d) {
            const int64_t o = (wid - n_units) * d + kl * VEC;
#pragma unroll
            for (int v4 = 0; v4 < VEC; v4 += 4) {
                *reinterpret_cast<float4 *>(out + o + v4) = make_float4(0.f, 0.f, 0.f, 0.f);
                if (out2) *reinterpret_cast<float4 *>(out2 + o + v4) = make_float4(0.f, 0.f, 0.f, 0.f);
                if (outbf) *reinterpret_cast<uint2 *>(outbf + o + v4) = make_uint2(0u, 0u);
            }
        }
        return;
    }
    const RowWork rw = row_work(wid, dm_ptr, N, n_units, hv_row, hv_unit_ptr, unit_hv);
    if (rw.row < 0) return;                             // whole wavefront leaves together
    if (active && !active[rw.row]) {                    // a unit of a heavy row outside the sub-graph
        if (rw.unit < 0 && g == 0 && kl * VEC < d) {
            const int64_t o = rw.row * d + kl * VEC;
#pragma unroll
            for (int v4 = 0; v4 < VEC; v4 += 4) {
                *reinterpret_cast<float4 *>(out + o + v4) = make_float4(0.f, 0.f, 0.f, 0.f);
                if (out2) *reinterpret_cast<float4 *>(out2 + o + v4) = make_float4(0.f, 0.f, 0.f, 0.f);
                if (outbf) *reinterpret_cast<uint2 *>(outbf + o + v4) = make_uint2(0u, 0u);
            }
        }
        return;
    }
    const int GB = gb_count, GE = G / GB;
    const int gb = g % GB, ge = g / GB;
    const bool kact = kl * VEC < d;
    const int nb = (B + GB - 1) / GB;                   // basis slots per edge for this group

    float acc[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) acc[v] = 0.f;
    // the row's self-loop part is fetched ahead of the edges (it is only needed at the end; loaded there it would
    // add one more memory round trip to every wavefront)
    float4 selfv[VEC / 4];
#pragma unroll
    for (int v4 = 0; v4 < VEC / 4; ++v4) selfv[v4] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (g == 0 && kact && rw.unit < 0) {
#pragma unroll
        for (int v4 = 0; v4 < VEC / 4; ++v4)
            selfv[v4] = *reinterpret_cast<const float4 *>(Self + rw.row * d + kl * VEC + 4 * v4);
    }

    for (int32_t e0 = rw.beg; e0 < rw.end; e0 += 64) {
        const int cnt = min(64, rw.end - e0);
        int32_t my_src = 0, my_rel = 0;
        float my_w = 0.f;
        if (lane < cnt) {
            my_src = dm_src[e0 + lane];
            if (PLAIN) {
                my_w = dm_invc ? dm_invc[e0 + lane] : 1.f;
            } else {
                my_rel = dm_rel[e0 + lane];
                my_w = dm_invc[e0 + lane];
            }
        }
        const int erounds = (cnt + GE - 1) / GE;        // uniform trip counts for all lanes
        const int items = erounds * nb;
        int er = 0, bi = 0;                             // current (edge round, basis slot)
        for (int q0 = 0; q0 < items; q0 += U) {
            float coef[U];
            uint4 raw[U];
            // Plain sums with several lane groups load no more rows than there are (a vertex with two runs two, not
            // 16: sum_runs of 5.8 M runs into 2.9 M rows of 128 floats 2.07 -> 1.42 ms); with one group, or several
            // bases per edge, the slots are nearly always full and the bound costs more (1.42 -> 2.00 ms for 544 k edges
            // x 10 bases x 200 floats).  Uniform over the wavefront.
            const int slots = PLAIN && G > 1 ? min(U, items - q0) : U;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (u >= slots) break;
                const int el = er * GE + ge;
                const int b = bi * GB + gb;
                // a slot past the end repeats the chunk's first edge with coefficient 0, and a lane past the
                // row's width reads its start: every load is unconditional (no divergent branch around it)
                const bool ok = q0 + u < items && el < cnt && b < B;
                const int els = ok ? el : 0, bs = ok ? b : 0;
                const int32_t src = __shfl(my_src, els, 64);
                const int32_t rel = __shfl(my_rel, els, 64);
                const float w = __shfl(my_w, els, 64);
                const float cf = PLAIN ? w : a[(int64_t)rel * B + bs] * w;
                coef[u] = ok ? cf : 0.f;
                raw[u] = MsgRow<BF16>::load_raw(P, ((int64_t)src * B + bs) * d + (kact ? kl * VEC : 0));
                if (++bi == nb) { bi = 0; ++er; }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (u >= slots) break;
                float val[VEC];
                MsgRow<BF16>::unpack(raw[u], val);
#pragma unroll
                for (int v = 0; v < VEC; ++v) acc[v] = fmaf(coef[u], val[v], acc[v]);
            }
        }
    }
    // fold the lane groups together (fixed order: deterministic)
#pragma unroll
    for (int off = LPR; off < 64; off <<= 1)
#pragma unroll
        for (int v = 0; v < VEC; ++v) acc[v] += __shfl_xor(acc[v], off, 64);

    if (g == 0 && kact) {
        if (rw.unit >= 0) {
            float *q = partial + (int64_t)rw.unit * d + kl * VEC;
#pragma unroll
            for (int v4 = 0; v4 < VEC; v4 += 4)
                *reinterpret_cast<float4 *>(q + v4) = make_float4(acc[v4], acc[v4 + 1], acc[v4 + 2], acc[v4 + 3]);
            return;
        }
        const int64_t o = rw.row * d + kl * VEC;
#pragma unroll
        for (int v4 = 0; v4 < VEC; v4 += 4) {
            const float4 s = selfv[v4 / 4];
            float4 r = make_float4(act_apply(act, acc[v4] + s.x), act_apply(act, acc[v4 + 1] + s.y),
                                   act_apply(act, acc[v4 + 2] + s.z), act_apply(act, acc[v4 + 3] + s.w));
            *reinterpret_cast<float4 *>(out + o + v4) = r;
            if (out2) *reinterpret_cast<float4 *>(out2 + o + v4) = r;
            if (outbf) *reinterpret_cast<uint2 *>(outbf + o + v4) = make_uint2(pack_bf16x2(r.x, r.y), pack_bf16x2(r.z, r.w));
        }
    }
}

// The rows that the edges of one (source, relation) pair share:
//   Q[g][:] = sum_b a[rel_g][b] P[src_g][b][:]        (fp32, [n_sgrp][d])
// for every group g of the source-major view, after which the forward sum over edges gathers one row per edge instead of B.
// One wavefront per source (per 64 groups of one with more); a row is covered by LPR lanes, the 64 / LPR lane groups take
// different groups, U each at a time.  A lane holds the coefficients of one of the 64 groups and hands them out (a scalar
// where a wavefront has one lane group, else by a shuffle), so that no memory round trip stands between the groups.  The
// source's P rows and the coefficients stay in registers if it has at most NB bases, else they pass NB at a time per round.
// Bound by writing Q and by the latency of a source's chain.  544 k edges, 355 k groups, 10 bases of 200 floats: 87 us and
// the gather of one row per edge 94, where gathering ten took 723; 2 M edges, 1.16 M groups, 16 bases of 128 bf16: 209 + 190,
// 1036.  (The loop over the bases has to be unrolled in full: with P indexed in scratch memory 185 and 596 us.)
template <bool BF16, int LPR, int NB>
__global__ __launch_bounds__(64 * WPB) void k_relation_rows(
    const int32_t *__restrict__ sg_ptr, const int32_t *__restrict__ sg_rel, int64_t N,
    int32_t n_units, const int32_t *__restrict__ hv_row, const int32_t *__restrict__ hv_unit_ptr,
    const int32_t *__restrict__ unit_hv, const void *__restrict__ P, const float *__restrict__ a, int32_t B, int32_t d,
    float *__restrict__ Q, const uint8_t *__restrict__ active, EdgeGate gate)
{
    if (gate.shut(true)) return;
    constexpr int VEC = MsgRow<BF16>::VEC, NG = 64 / LPR, U = NG > 1 ? 4 : 8;
    const int lane = threadIdx.x & 63;
    const RowWork rw = row_work((int64_t)blockIdx.x * WPB + (threadIdx.x >> 6), sg_ptr, N, n_units, hv_row, hv_unit_ptr, unit_hv,
                                KGE_HEAVY_GROUPS);
    if (rw.row < 0) return;                              // whole wavefronts leave
    if (active && !active[rw.row]) return;               // no active destination has an edge from here
    const int kl = lane % LPR, g = lane / LPR;
    const bool kact = kl * VEC < d;
    const int64_t col = kact ? kl * VEC : 0;
    const int64_t prow = rw.row * B;
    uint4 p[NB];
    float c[NB];                                         // of the lane's group
    auto fetch = [&](int b0) __attribute__((always_inline)) {
#pragma unroll
        for (int n = 0; n < NB; ++n) p[n] = MsgRow<BF16>::load_raw(P, (prow + min(b0 + n, B - 1)) * d + col);
    };
    if (B <= NB) fetch(0);
    for (int32_t g0 = rw.beg; g0 < rw.end; g0 += 64) {
        const int cnt = min(64, rw.end - g0);
        const float *ar = a + (int64_t)sg_rel[g0 + min(lane, cnt - 1)] * B;
        auto coefs = [&](int b0) __attribute__((always_inline)) {
#pragma unroll
            for (int n = 0; n < NB; ++n) c[n] = ar[min(b0 + n, B - 1)];
        };
        if (B <= NB) coefs(0);
        for (int q0 = 0; q0 < cnt; q0 += NG * U) {
            float acc[U][VEC];
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int v = 0; v < VEC; ++v) acc[u][v] = 0.f;
            for (int b0 = 0; b0 < B; b0 += NB) {
                if (B > NB) { fetch(b0); coefs(b0); }
#pragma unroll
                for (int n = 0; n < NB; ++n)
                    if (b0 + n < B) {                    // uniform
                        float val[VEC];
                        MsgRow<BF16>::unpack(p[n], val);
#pragma unroll
                        for (int u = 0; u < U; ++u) {    // a slot past the last group: sums that nothing stores
                            float x;
                            if constexpr (NG > 1) x = __shfl(c[n], (q0 + u * NG + g) & 63, 64);
                            else x = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(c[n]), (q0 + u) & 63));
#pragma unroll
                            for (int v = 0; v < VEC; ++v) acc[u][v] = fmaf(x, val[v], acc[u][v]);
                        }
                    }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int q = q0 + u * NG + g;
                if (q >= cnt || !kact) continue;
                float *o = Q + (int64_t)(g0 + q) * d + col;
#pragma unroll
                for (int v4 = 0; v4 < VEC; v4 += 4)
                    *reinterpret_cast<float4 *>(o + v4) = make_float4(acc[u][v4], acc[u][v4 + 1], acc[u][v4 + 2], acc[u][v4 + 3]);
            }
        }
    }
}

// Heavy destinations: out[i] = act(sum of the row's unit partials + Self[i]).  One thread per float4.
__global__ void k_gather_fwd_finish(int32_t n_hv, const int32_t *__restrict__ hv_row,
                                    const int32_t *__restrict__ hv_unit_ptr, const float *__restrict__ partial,
                                    int32_t d, const float *__restrict__ Self, int act,
                                    float *__restrict__ out, float *__restrict__ out2,
                                    uint16_t *__restrict__ outbf, const uint8_t *__restrict__ active)
{
    const int d4 = d >> 2;
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (int64_t)n_hv * d4) return;
    const int32_t h = (int32_t)(idx / d4);
    const int k4 = (int)(idx - (int64_t)h * d4) * 4;
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    if (active && !active[hv_row[h]]) {
        const int64_t oz = (int64_t)hv_row[h] * d + k4;
        *reinterpret_cast<float4 *>(out + oz) = s;
        if (out2) *reinterpret_cast<float4 *>(out2 + oz) = s;
        if (outbf) *reinterpret_cast<uint2 *>(outbf + oz) = make_uint2(0u, 0u);
        return;
    }
    for (int32_t u = hv_unit_ptr[h]; u < hv_unit_ptr[h + 1]; ++u) {
        const float4 x = *reinterpret_cast<const float4 *>(partial + (int64_t)u * d + k4);
        s.x += x.x; s.y += x.y; s.z += x.z; s.w += x.w;
    }
    const int64_t o = (int64_t)hv_row[h] * d + k4;
    const float4 sf = *reinterpret_cast<const float4 *>(Self + o);
    const float4 r = make_float4(act_apply(act, s.x + sf.x), act_apply(act, s.y + sf.y),
                                 act_apply(act, s.z + sf.z), act_apply(act, s.w + sf.w));
    *reinterpret_cast<float4 *>(out + o) = r;
    if (out2) *reinterpret_cast<float4 *>(out2 + o) = r;
    if (outbf) *reinterpret_cast<uint2 *>(outbf + o) = make_uint2(pack_bf16x2(r.x, r.y), pack_bf16x2(r.z, r.w));
}

// ------------------------------------------------------------------ activation backward
__global__ void k_act_backward(const float4 *__restrict__ dH, const float4 *__restrict__ Hout, int act,
                               int64_t n4, float4 *__restrict__ G)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (; i < n4; i += stride) {
        float4 g = dH[i];
        if (act == KGE_ACT_RELU) {
            float4 h = Hout[i];
            g.x = h.x > 0.f ? g.x : 0.f; g.y = h.y > 0.f ? g.y : 0.f;
            g.z = h.z > 0.f ? g.z : 0.f; g.w = h.w > 0.f ? g.w : 0.f;
        }
        G[i] = g;
    }
}

// ------------------------------------------------------------------ backward pass of the neighbour sum, by source
// One wavefront per (source row work, chunk of bases) on the source-major view, whose edges are grouped by relation.
// With y = sum over the edges of one relation out of source j of (1/c_e) G[dst_e][:],
//   dP[j][b][:] += a[rel][b] y       and       da[rel][b] += < P[j][b][:], y >,
// so the gathered rows are read once for both, P[j] once per source (not once per edge out of it), and a relation's edges
// cost one product per basis.  The dot products of a group go to the scratch row of the run that its first edge lies in
// (atomically: another source's group may use the same row; runs are sorted by relation and k_coeff_reduce adds up a
// relation's rows), after a chunk of 64 edges, so that no atomic stands between the gathered loads.
// A row is covered by LPR lanes of 4 columns, the 64 / LPR lane groups take NB bases each (16 per wavefront at most).
// DP = false: the dot products only (dP comes from k_gather_t_bf16).
// SPREAD: with few bases and narrow rows most lane groups would hold no base; they share a relation's edges instead, all of
// them with the same NB bases, and their sums meet in a butterfly per relation.
// Bound by the vector instructions of the groups (most sources have one edge of a relation), the rows coming from the
// caches: 544 k edges, 4 bases, d = 200, fp32: 149 us; for more bases the matrix-core form below takes over (10 bases 365
// against 211 us).
template <int OFF> __device__ __forceinline__ float lane_xor(float x)
{
    if constexpr (OFF == 1) return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0xb1, 0xf, 0xf, true));
    else if constexpr (OFF == 2) return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x4e, 0xf, 0xf, true));
    else return __shfl_xor(x, OFF, 64);
}
// sums of K per-lane values (a power of two, at most LPR) over LPR consecutive lanes: lane l gets sum l % K
template <int K, int LPR, int OFF = 1> __device__ __forceinline__ float sums_over_lanes(const float *v, int lane)
{
    if constexpr (K > 1) {
        float h[K / 2];
#pragma unroll
        for (int i = 0; i < K / 2; ++i) {
            const bool odd = (lane & OFF) != 0;
            h[i] = (odd ? v[2 * i + 1] : v[2 * i]) + lane_xor<OFF>(odd ? v[2 * i] : v[2 * i + 1]);
        }
        return sums_over_lanes<K / 2, LPR, OFF * 2>(h, lane);
    } else if constexpr (OFF < LPR) {
        const float s = v[0] + lane_xor<OFF>(v[0]);
        return sums_over_lanes<1, LPR, OFF * 2>(&s, lane);
    } else {
        return v[0];
    }
}

template <bool BF16, int LPR, int NB, bool DP, bool SPREAD, bool FULL>
__global__ __launch_bounds__(64 * WPB) void k_source_backward(
    const int32_t *__restrict__ sm_ptr, const int32_t *__restrict__ sm_dst, const int32_t *__restrict__ sm_rel,
    const float *__restrict__ sm_invc, const int32_t *__restrict__ sm_seg, int64_t N,
    int32_t n_units, const int32_t *__restrict__ hv_row, const int32_t *__restrict__ hv_unit_ptr,
    const int32_t *__restrict__ unit_hv, const float *__restrict__ G, const float *__restrict__ a,
    const void *__restrict__ P, int32_t B, int32_t d, int32_t n_chunks, void *__restrict__ dP, int64_t ld,
    float *__restrict__ partial, float *__restrict__ seg_out, const uint8_t *__restrict__ active)
{
    constexpr int NG = 64 / LPR, NBT = SPREAD ? NB : NG * NB, U = 4;
    __shared__ float dots[WPB][64][NBT];
    __shared__ int32_t dot_seg[WPB][64];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t wid_all = (int64_t)blockIdx.x * WPB + wv;
    const int64_t wid = wid_all / n_chunks;
    const int b0 = (int)(wid_all - wid * n_chunks) * NBT;
    const RowWork rw = row_work(wid, sm_ptr, N, n_units, hv_row, hv_unit_ptr, unit_hv);
    if (rw.row < 0) return;                              // whole wavefronts leave; the kernel has no block barrier
    const int kl = lane % LPR, g = lane / LPR, first_b = SPREAD ? 0 : g * NB;      // of this lane's bases in the chunk
    const bool kact = kl * 4 < d;
    const int col = kact ? kl * 4 : 0;
    const int nbs = B - b0 < NBT ? B - b0 : NBT;         // bases of this chunk

    float pv[NB][4], acc[NB][4];
#pragma unroll
    for (int n = 0; n < NB; ++n) {
        const int b = b0 + first_b + n;
        const int64_t o = (rw.row * B + (b < B ? b : B - 1)) * d + col;
        float4 x;
        if (BF16) {
            const uint2 r = *reinterpret_cast<const uint2 *>(reinterpret_cast<const uint16_t *>(P) + o);
            x = make_float4(__uint_as_float(r.x << 16), __uint_as_float(r.x & 0xffff0000u),
                            __uint_as_float(r.y << 16), __uint_as_float(r.y & 0xffff0000u));
        } else {
            x = *reinterpret_cast<const float4 *>(reinterpret_cast<const float *>(P) + o);
        }
        pv[n][0] = kact ? x.x : 0.f; pv[n][1] = kact ? x.y : 0.f; pv[n][2] = kact ? x.z : 0.f; pv[n][3] = kact ? x.w : 0.f;
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[n][v] = 0.f;
    }

    for (int32_t e0 = rw.beg; e0 < rw.end; e0 += 64) {
        const int cnt = min(64, rw.end - e0);
        int32_t my_dst = 0, my_rel = 0, my_seg = 0;
        float my_w = 0.f;
        if (lane < cnt) {
            my_dst = sm_dst[e0 + lane]; my_rel = sm_rel[e0 + lane]; my_w = sm_invc[e0 + lane]; my_seg = sm_seg[e0 + lane];
            if (active && !active[my_dst]) my_dst = -1;   // destination outside the sub-graph: G row is zero
        }
        int n_grp = 0;
        int32_t cur_rel = -1, cur_seg = 0;               // uniform over the wavefront
        float4 y = make_float4(0.f, 0.f, 0.f, 0.f);
        auto flush = [&]() __attribute__((always_inline)) {
            const float *ar = a + (int64_t)cur_rel * B;
            // a lane past the width has read column 0, and an infinity there times its zero of P would be NaN (a condition
            // around the loads instead: 1 to 2 % slower at all widths).  FULL: there is none
            if (!FULL && !kact) y = make_float4(0.f, 0.f, 0.f, 0.f);
            if (SPREAD)                                  // the lane groups' shares of the edges
#pragma unroll
                for (int off = LPR; off < 64; off <<= 1) {
                    y.x += __shfl_xor(y.x, off, 64); y.y += __shfl_xor(y.y, off, 64);
                    y.z += __shfl_xor(y.z, off, 64); y.w += __shfl_xor(y.w, off, 64);
                }
            float part[NB];
#pragma unroll
            for (int n = 0; n < NB; ++n) {
                if (DP) {
                    float c = ar[min(b0 + n, B - 1)];    // scalar loads: every lane group's coefficients, then its own
#pragma unroll
                    for (int h = 1; h < NG && !SPREAD; ++h) c = g == h ? ar[min(b0 + h * NB + n, B - 1)] : c;
                    acc[n][0] = fmaf(c, y.x, acc[n][0]); acc[n][1] = fmaf(c, y.y, acc[n][1]);
                    acc[n][2] = fmaf(c, y.z, acc[n][2]); acc[n][3] = fmaf(c, y.w, acc[n][3]);
                }
                part[n] = fmaf(pv[n][3], y.w, fmaf(pv[n][2], y.z, fmaf(pv[n][1], y.y, pv[n][0] * y.x)));
            }
            const float s = sums_over_lanes<NB, LPR>(part, lane);
            if (kl < NB && (!SPREAD || g == 0)) dots[wv][n_grp][first_b + kl] = s;
            if (lane == 0) dot_seg[wv][n_grp] = cur_seg;
            ++n_grp;
        };
        if constexpr (SPREAD) {
            const bool live = lane < cnt && my_dst >= 0;
            const uint64_t lives = __ballot(live);
            const int32_t before = __shfl_up(my_rel, 1, 64);
            uint64_t starts = __ballot(lane < cnt && (lane == 0 || my_rel != before));
            while (starts) {                             // uniform: one relation's edges [s, t) of the chunk
                const int s = __builtin_ctzll(starts);
                starts &= starts - 1;
                const int t = starts ? __builtin_ctzll(starts) : cnt;
                if (!(lives >> s & (t - s == 64 ? ~0ull : (1ull << (t - s)) - 1ull))) continue;
                cur_rel = __builtin_amdgcn_readlane(my_rel, s);
                cur_seg = __builtin_amdgcn_readlane(my_seg, s);
                y = make_float4(0.f, 0.f, 0.f, 0.f);
                for (int q0 = s; q0 < t; q0 += NG * U) {
                    float4 row[U];
                    float w[U];
                    bool on[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) {        // a slot past the end or outside the sub-graph: a row that is dropped
                        const int el = min(q0 + u * NG + g, t - 1);
                        const int32_t dst = __shfl(my_dst, el, 64);
                        on[u] = q0 + u * NG + g < t && dst >= 0 && kact;
                        w[u] = __shfl(my_w, el, 64);
                        row[u] = *reinterpret_cast<const float4 *>(G + (int64_t)(dst < 0 ? 0 : dst) * d + col);
                    }
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        if (!on[u]) row[u] = make_float4(0.f, 0.f, 0.f, 0.f);
                        y.x = fmaf(w[u], row[u].x, y.x); y.y = fmaf(w[u], row[u].y, y.y);
                        y.z = fmaf(w[u], row[u].z, y.z); y.w = fmaf(w[u], row[u].w, y.w);
                    }
                }
                flush();
                cur_rel = -1;
            }
        } else {
            float4 nxt[U];
            auto fetch = [&](int q0) __attribute__((always_inline)) {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int32_t dst = __builtin_amdgcn_readlane(my_dst, min(q0 + u, cnt - 1));
                    nxt[u] = *reinterpret_cast<const float4 *>(G + (int64_t)(dst < 0 ? 0 : dst) * d + col);
                }
            };
            fetch(0);
            for (int q0 = 0; q0 < cnt; q0 += U) {
                float4 row[U];
#pragma unroll
                for (int u = 0; u < U; ++u) row[u] = nxt[u];
                fetch(q0 + U);                               // past the chunk: its last edge again
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int el = q0 + u;
                    if (el >= cnt || __builtin_amdgcn_readlane(my_dst, el) < 0) continue;
                    const int32_t rel = __builtin_amdgcn_readlane(my_rel, el);
                    const float w = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(my_w), el));
                    if (rel != cur_rel) {
                        if (cur_rel >= 0) flush();
                        cur_rel = rel;
                        cur_seg = __builtin_amdgcn_readlane(my_seg, el);
                        y = make_float4(0.f, 0.f, 0.f, 0.f);
                    }
                    y.x = fmaf(w, row[u].x, y.x); y.y = fmaf(w, row[u].y, y.y);
                    y.z = fmaf(w, row[u].z, y.z); y.w = fmaf(w, row[u].w, y.w);
                }
            }
        }
        if (cur_rel >= 0) flush();
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        for (int i = lane; i < n_grp * nbs; i += 64) {
            const int q = i / nbs, n = i - q * nbs;
            unsafeAtomicAdd(seg_out + (int64_t)dot_seg[wv][q] * B + b0 + n, dots[wv][q][n]);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
    if (!DP || !kact || (SPREAD && g != 0)) return;
#pragma unroll
    for (int n = 0; n < NB; ++n) {
        const int b = b0 + first_b + n;
        if (b >= B) continue;
        if (rw.unit >= 0) {
            *reinterpret_cast<float4 *>(partial + ((int64_t)rw.unit * B + b) * d + kl * 4) =
                make_float4(acc[n][0], acc[n][1], acc[n][2], acc[n][3]);
        } else {
            const int64_t o = (int64_t)rw.row * ld + (int64_t)b * d + kl * 4;
            if (BF16) {
                uint2 x;
                x.x = pack_bf16x2(acc[n][0], acc[n][1]); x.y = pack_bf16x2(acc[n][2], acc[n][3]);
                *reinterpret_cast<uint2 *>(reinterpret_cast<uint16_t *>(dP) + o) = x;
            } else {
                *reinterpret_cast<float4 *>(reinterpret_cast<float *>(dP) + o) =
                    make_float4(acc[n][0], acc[n][1], acc[n][2], acc[n][3]);
            }
        }
    }
}

// The same on the fp32 matrix cores (v_mfma_f32_16x16x4_f32), for several bases.  A wavefront takes a source (or a unit of a
// heavy one) and 16 bases.  It adds up the rows y of up to 16 (source, relation) groups as above, but leaves them in LDS,
// [group][column], and then forms
//   dots[group][base] = Y P^T        (16 x W)(W x 16): both operands 16 bytes per lane, P[j] in registers for the whole source
//   dP[base][column] += A Y          (16 x 16)(16 x W): A[base][group] = a[rel][base], Y read by columns
// so that a product and a sum over lanes per group, base and column turn into 8 W / 16 matrix-core instructions per 16 groups,
// and the dots leave as 64-byte rows of atomics straight from the accumulators.  All fp32, as before.
// The lane groups of a narrow row take consecutive edges of a pass each; a group of edges cut by that, or by a unit, has two
// rows.  Unused rows and the columns past the width are zeros (an infinity times a zero would be NaN).
// W = 16 NBLK >= d columns.  A block is one wavefront (its LDS is what limits their number), 8 rows of G in flight per lane.
// Bound by the latency of a source's chain at two wavefronts per SIMD: 544 k edges, 355 k groups, 10 bases, d = 200, fp32: 211
// us, 365 on the vector units; 2 M edges, 16 bases, d = 128, bf16 messages: 443, 754.  (Four wavefronts per block and 4 rows in
// flight 407 and 542; three wavefronts per SIMD by fewer registers 330 and 560.)
typedef float sb_f32x4 __attribute__((ext_vector_type(4)));

template <bool BF16, int NBLK, bool DP>
__global__ __launch_bounds__(64, 2) void k_source_cores(
    const int32_t *__restrict__ sm_ptr, const int32_t *__restrict__ sm_dst, const int32_t *__restrict__ sm_rel,
    const float *__restrict__ sm_invc, const int32_t *__restrict__ sm_seg, int64_t N,
    int32_t n_units, const int32_t *__restrict__ hv_row, const int32_t *__restrict__ hv_unit_ptr,
    const int32_t *__restrict__ unit_hv, const float *__restrict__ G, const float *__restrict__ a,
    const void *__restrict__ P, int32_t B, int32_t d, int32_t n_chunks, void *__restrict__ dP, int64_t ld,
    float *__restrict__ partial, float *__restrict__ seg_out, const uint8_t *__restrict__ active)
{
    constexpr int W = 16 * NBLK, LPR = W > 128 ? 64 : W > 64 ? 32 : 16, NG = 64 / LPR;
    constexpr int RPG = NG == 4 ? 4 : 8, SUB = NG * RPG;              // edges per lane group and per pass (16 at most)
    constexpr int SUM = NBLK <= 8 ? 4 : (NBLK + 1) / 2;               // blocks of 16 columns that a dot product sums in one go
    constexpr bool NARROW = NG == 4;      // rows of up to four lane groups per pass, more of them: each 16 have a sum of their own in dP
    constexpr int PITCH = W + 4;                                      // 4 rows apart: 16 banks; one: an odd number of 16 bytes
    __shared__ __attribute__((aligned(16))) float Y[16 * PITCH];
    __shared__ __attribute__((aligned(16))) int32_t slot_rel[16], slot_seg[16];
    const int lane = threadIdx.x;
    const int64_t wid = (int64_t)blockIdx.x / n_chunks;
    const int b0 = (int)((int64_t)blockIdx.x - wid * n_chunks) * 16;
    const RowWork rw = row_work(wid, sm_ptr, N, n_units, hv_row, hv_unit_ptr, unit_hv);
    if (rw.row < 0) return;                              // a block is one wavefront
    const int kl = lane % LPR, g = lane / LPR;           // of the row phase: column quad, lane group
    const int l16 = lane & 15, l4 = lane >> 4;           // of the products
    const bool kact = kl * 4 < d;
    const int col = kact ? kl * 4 : 0;

    float p[NBLK][4];                                    // P[row][b0 + l16][16 t + 4 l4 ..]
    sb_f32x4 acc[NBLK];
    {
        const int64_t prow = (rw.row * B + min(b0 + l16, B - 1)) * d;
#pragma unroll
        for (int t = 0; t < NBLK; ++t) {
            const int c = 16 * t + 4 * l4;
            const int64_t o = prow + (c < d ? c : 0);
            float4 x;
            if (BF16) {
                const uint2 r = *reinterpret_cast<const uint2 *>(reinterpret_cast<const uint16_t *>(P) + o);
                x = make_float4(__uint_as_float(r.x << 16), __uint_as_float(r.x & 0xffff0000u),
                                __uint_as_float(r.y << 16), __uint_as_float(r.y & 0xffff0000u));
            } else {
                x = *reinterpret_cast<const float4 *>(reinterpret_cast<const float *>(P) + o);
            }
            p[t][0] = c < d ? x.x : 0.f; p[t][1] = c < d ? x.y : 0.f; p[t][2] = c < d ? x.z : 0.f; p[t][3] = c < d ? x.w : 0.f;
            acc[t] = sb_f32x4{0.f, 0.f, 0.f, 0.f};
        }
    }
    auto zero_rows = [&](int from) __attribute__((always_inline)) {
        for (int r = from + g; r < 16; r += NG)
            if (kl * 4 < W) *reinterpret_cast<float4 *>(Y + r * PITCH + kl * 4) = make_float4(0.f, 0.f, 0.f, 0.f);
    };
    zero_rows(0);                                        // the columns past the width stay zeros from here on
    int used = 0;                                        // rows of Y in use; uniform
    auto flush = [&]() __attribute__((always_inline)) {
        zero_rows(used);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        const int4 rel4 = *reinterpret_cast<const int4 *>(&slot_rel[4 * l4]), seg4 = *reinterpret_cast<const int4 *>(&slot_seg[4 * l4]);
        const int32_t rel[4] = {rel4.x, rel4.y, rel4.z, rel4.w}, seg[4] = {seg4.x, seg4.y, seg4.z, seg4.w};
        float c[4];
        if (DP)
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const float x = a[(int64_t)(4 * l4 + s < used ? rel[s] : 0) * B + min(b0 + l16, B - 1)];
                c[s] = 4 * l4 + s < used ? x : 0.f;
            }
        // four chains for every SUM blocks: with two chains over all blocks dots, and with them da, are up to 30 % further off than
        // the vector form's (5001 entities, d = 200, relative to 64 bits: 2.5e-7, 1.9e-7 there, 2.0e-7 so).  Kernel, us, two chains / a
        // sum for every 4 blocks / so: step of 8192 triples, d = 200: 206 / 216 / 211; d = 256: 301 / 238 / 230
        const sb_f32x4 zero = {0.f, 0.f, 0.f, 0.f};
        sb_f32x4 dots = zero;
#pragma unroll
        for (int t0 = 0; t0 < NBLK; t0 += SUM) {
            sb_f32x4 dot[4];
#pragma unroll
            for (int t = t0; t < t0 + SUM && t < NBLK; ++t) {
                const float4 y = *reinterpret_cast<const float4 *>(Y + l16 * PITCH + 16 * t + 4 * l4);
                dot[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(y.x, p[t][0], t == t0 ? zero : dot[0], 0, 0, 0);
                dot[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(y.y, p[t][1], t == t0 ? zero : dot[1], 0, 0, 0);
                dot[2] = __builtin_amdgcn_mfma_f32_16x16x4f32(y.z, p[t][2], t == t0 ? zero : dot[2], 0, 0, 0);
                dot[3] = __builtin_amdgcn_mfma_f32_16x16x4f32(y.w, p[t][3], t == t0 ? zero : dot[3], 0, 0, 0);
            }
            dot[0] = (dot[0] + dot[1]) + (dot[2] + dot[3]);
            dots = t0 == 0 ? dot[0] : dots + dot[0];
        }
        if (DP)
#pragma unroll
            for (int t = 0; t < NBLK; ++t) {
                sb_f32x4 sum = NARROW ? zero : acc[t];
#pragma unroll
                for (int s = 0; s < 4; ++s)              // groups 4 k + s of the four lane quarters k
                    sum = __builtin_amdgcn_mfma_f32_16x16x4f32(c[s], Y[(4 * l4 + s) * PITCH + 16 * t + l16], sum, 0, 0, 0);
                acc[t] = NARROW ? acc[t] + sum : sum;
            }
#pragma unroll
        for (int v = 0; v < 4; ++v)
            if (4 * l4 + v < used && b0 + l16 < B) unsafeAtomicAdd(seg_out + (int64_t)seg[v] * B + b0 + l16, dots[v]);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        used = 0;
    };

    for (int32_t e0 = rw.beg; e0 < rw.end; e0 += 64) {
        int cnt = min(64, rw.end - e0);
        const int mine = e0 + min(lane, cnt - 1);
        int32_t my_dst = sm_dst[mine], my_rel = sm_rel[mine], my_seg = sm_seg[mine];
        float my_w = sm_invc[mine];
        if (active) {                                    // edges into the sub-graph only, moved together
            const bool live = lane < cnt && active[my_dst];
            const uint64_t lives = __ballot(live);
            cnt = __popcll(lives);
            if (cnt == 0) continue;
            const int before = __popcll(lives & ((1ull << lane) - 1ull));
            const int to = (live ? before : cnt + lane - before) * 4;         // the others fill the rest
            my_dst = __builtin_amdgcn_ds_permute(to, my_dst);
            my_rel = __builtin_amdgcn_ds_permute(to, my_rel);
            my_seg = __builtin_amdgcn_ds_permute(to, my_seg);
            my_w = __int_as_float(__builtin_amdgcn_ds_permute(to, __float_as_int(my_w)));
        }
        const int32_t prev_rel = __shfl_up(my_rel, 1, 64);
        float4 row[RPG];
        auto fetch = [&](int e) __attribute__((always_inline)) {     // edge e of the page; past its end the last one again
            int32_t dst;
            if constexpr (NG == 1) dst = __builtin_amdgcn_readlane(my_dst, min(e, cnt - 1));
            else dst = __shfl(my_dst, min(e, cnt - 1), 64);
            return *reinterpret_cast<const float4 *>(G + (int64_t)dst * d + col);
        };
#pragma unroll
        for (int u = 0; u < RPG; ++u) row[u] = fetch(g * RPG + u);
        for (int q0 = 0; q0 < cnt; q0 += SUB) {
            const int end = min(q0 + SUB, cnt);
            const bool in = lane >= q0 && lane < end;
            const uint64_t starts = __ballot(in && ((lane - q0) % RPG == 0 || my_rel != prev_rel));
            const int n_new = __popcll(starts);
            if (used + n_new > 16) flush();
            const int slot = used + __popcll(starts & ((2ull << lane) - 1ull)) - 1;
            const bool first = starts >> lane & 1, last = lane + 1 == end || (lane < 63 && (starts >> (lane + 1) & 1));
            if (in && first) { slot_rel[slot] = my_rel; slot_seg[slot] = my_seg; }
            const int info = slot | (first ? 32 : 0) | (last ? 64 : 0);
            float4 y = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
            for (int u = 0; u < RPG; ++u) {
                const int e = q0 + g * RPG + u;
                int f;
                float w;
                if constexpr (NG == 1) {
                    f = __builtin_amdgcn_readlane(info, min(e, 63));
                    w = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(my_w), min(e, 63)));
                } else {
                    f = __shfl(info, min(e, 63), 64);
                    w = __shfl(my_w, min(e, 63), 64);
                }
                if (f & 32) y = make_float4(0.f, 0.f, 0.f, 0.f);
                y.x = fmaf(w, row[u].x, y.x); y.y = fmaf(w, row[u].y, y.y);
                y.z = fmaf(w, row[u].z, y.z); y.w = fmaf(w, row[u].w, y.w);
                row[u] = fetch(e + SUB);
                if ((f & 64) && e < end && kact) *reinterpret_cast<float4 *>(Y + (f & 15) * PITCH + kl * 4) = y;
            }
            used += n_new;
        }
    }
    if (used) flush();
    if (!DP) return;
    // the sums through LDS, so that a lane stores four consecutive columns
#pragma unroll
    for (int t = 0; t < NBLK; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) Y[(4 * l4 + v) * PITCH + 16 * t + l16] = acc[t][v];
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    if (!kact) return;
    for (int m = g; m < 16 && b0 + m < B; m += NG) {
        const float4 x = *reinterpret_cast<const float4 *>(Y + m * PITCH + kl * 4);
        if (rw.unit >= 0) {
            *reinterpret_cast<float4 *>(partial + ((int64_t)rw.unit * B + b0 + m) * d + kl * 4) = x;
        } else {
            const int64_t o = (int64_t)rw.row * ld + (int64_t)(b0 + m) * d + kl * 4;
            if (BF16) *reinterpret_cast<uint2 *>(reinterpret_cast<uint16_t *>(dP) + o) = make_uint2(pack_bf16x2(x.x, x.y), pack_bf16x2(x.z, x.w));
            else *reinterpret_cast<float4 *>(reinterpret_cast<float *>(dP) + o) = x;
        }
    }
}

// dP with bf16 messages and many bases, a small dense product per source, on v_mfma_f32_32x32x16_bf16:
//   dP[j] (B x d, bf16) = W^T (B x deg) * Gg (deg x d),  W[e][b] = a[rel_e][b] invc_e (rounded to bf16),  Gg[e] = Gbf[dst_e].
// One block of four wavefronts per (source or heavy unit, chunk of 64 bases, chunk of 256 columns).  The block
// stages up to 32 edges at a time in LDS, as they lie in memory and with 16-byte loads: the gathered rows of G
// ([edge][column]) and the coefficient rows ([edge][base], multiplied by 1/c and rounded on the way).  The edge is
// the contraction index of both, so the matrix-core operands are fetched with the transposing LDS read, two per
// operand; wavefront w owns bases 32 (w / 2) .. and columns 128 (w % 2) ..: one coefficient operand feeds four
// products.  Sixteen edges per matrix-core instruction instead of two, and the gathered rows are read once per
// block instead of once per wavefront.
typedef float gt_floatx16 __attribute__((ext_vector_type(16)));
constexpr int GTB_EP = 32;                 // edges per pass
constexpr int GTB_PG = 256 + 32;           // LDS pitches, elements: 64 bytes modulo 256 (the four rows that 16
constexpr int GTB_PC = 64 + 96;            // lanes read at once fall in different quarters of the banks)

__global__ __launch_bounds__(256) void k_gather_t_bf16(
    const int32_t *__restrict__ sm_ptr, const int32_t *__restrict__ sm_dst,
    const int32_t *__restrict__ sm_rel, const float *__restrict__ sm_invc, int64_t N,
    int32_t n_units, const int32_t *__restrict__ hv_row, const int32_t *__restrict__ hv_unit_ptr,
    const int32_t *__restrict__ unit_hv,
    const uint16_t *__restrict__ Gbf, int64_t ldg, const float *__restrict__ a, int32_t B, int32_t d,
    int32_t n_bchunks, int32_t n_cchunks, uint16_t *__restrict__ dP, int64_t ld, float *__restrict__ partial,
    const uint8_t *__restrict__ active)
{
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    typedef __bf16 gtb_bf16x8 __attribute__((ext_vector_type(8)));
    __shared__ __attribute__((aligned(16))) uint16_t Gs[GTB_EP * GTB_PG];     // 18,432 B; the epilogue's staging too
    __shared__ __attribute__((aligned(16))) uint16_t Cs[GTB_EP * GTB_PC];     // 10,240 B
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int n_chunks = n_bchunks * n_cchunks;
    const int64_t wid = (int64_t)blockIdx.x / n_chunks;
    const int chunk = (int)((int64_t)blockIdx.x - wid * n_chunks);
    const int bbase = (chunk / n_cchunks) * 64, cbase = (chunk % n_cchunks) * 256;
    const RowWork rw = row_work(wid, sm_ptr, N, n_units, hv_row, hv_unit_ptr, unit_hv);
    if (rw.row < 0) return;                               // uniform over the block
    const int wm = w >> 1, wn = w & 1;

    gt_floatx16 acc[4];
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[c][v] = 0.f;

    // this thread's part of a pass: edge t / 8; of its G row the 16-byte chunks (t % 8) + 8 p, of its coefficient
    // row the 8 bases from 8 (t % 8)
    const int el = t >> 3, sub = t & 7;
    const int l16 = lane & 15, kr0 = 8 * (lane >> 5) + (l16 >> 2), mc = 16 * ((lane >> 4) & 1) + 4 * (l16 & 3);
    auto frag = [&](const uint16_t *tile, int pitch, int kr, int col) __attribute__((always_inline)) {
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (s16x4 __attribute__((address_space(3))) *)(tile + kr * pitch + col));
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (s16x4 __attribute__((address_space(3))) *)(tile + (kr + 4) * pitch + col));
        return __builtin_bit_cast(gtb_bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };

    for (int32_t e0 = rw.beg; e0 < rw.end; e0 += GTB_EP) {
        const int cnt = min(GTB_EP, rw.end - e0);
        int32_t dst = -1, rel = 0;
        float wgt = 0.f;
        if (el < cnt) {
            dst = sm_dst[e0 + el]; rel = sm_rel[e0 + el]; wgt = sm_invc ? sm_invc[e0 + el] : 1.f;
            if (active && !active[dst]) dst = -1;         // destination outside the sub-graph: its G row is zero
        }
        uint4 gq[4];
        float cf[8];
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const int col = cbase + 8 * (sub + 8 * p);
            gq[p] = make_uint4(0u, 0u, 0u, 0u);
            if (dst >= 0 && col < d) gq[p] = *reinterpret_cast<const uint4 *>(Gbf + (int64_t)dst * ldg + col);
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int b = bbase + 8 * sub + q;
            cf[q] = (dst >= 0 && b < B) ? a[(int64_t)rel * B + b] * wgt : 0.f;
        }
        __syncthreads();                                  // the previous pass's operands are consumed
#pragma unroll
        for (int p = 0; p < 4; ++p)
            *reinterpret_cast<uint4 *>(&Gs[el * GTB_PG + 8 * (sub + 8 * p)]) = gq[p];
        *reinterpret_cast<uint4 *>(&Cs[el * GTB_PC + 8 * sub]) =
            make_uint4(pack_bf16x2(cf[0], cf[1]), pack_bf16x2(cf[2], cf[3]), pack_bf16x2(cf[4], cf[5]), pack_bf16x2(cf[6], cf[7]));
        __syncthreads();
        if (bbase + 32 * wm < B) {                        // uniform per wavefront
#pragma unroll
            for (int ks = 0; ks < GTB_EP; ks += 16) {
                if (ks >= cnt) break;                     // uniform
                const gtb_bf16x8 af = frag(Cs, GTB_PC, ks + kr0, 32 * wm + mc);
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    if (cbase + 128 * wn + 32 * c >= d) continue;     // uniform
                    const gtb_bf16x8 bfr = frag(Gs, GTB_PG, ks + kr0, 128 * wn + 32 * c + mc);
                    acc[c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af, bfr, acc[c], 0, 0, 0);
                }
            }
        }
    }
    __syncthreads();                                      // Gs is free: each wavefront stages its tiles in its quarter
    // D register v of lane l: base 8*(v/4) + 4*(l/32) + v%4, column l%32 of its tile
    const int h = lane >> 5, l32 = lane & 31;
    float (*stage)[36] = reinterpret_cast<float (*)[36]>(reinterpret_cast<float *>(Gs) + w * 32 * 36);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const int tb = bbase + 32 * wm, tc = cbase + 128 * wn + 32 * c;
        if (tb >= B || tc >= d) continue;                 // uniform
        if (rw.unit >= 0) {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int b = tb + 8 * (v >> 2) + 4 * h + (v & 3);
                if (b < B) partial[((int64_t)rw.unit * B + b) * d + tc + l32] = acc[c][v];
            }
        } else {
            // through LDS so that each lane writes 16 consecutive bf16 of one base row
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int v = 0; v < 16; ++v) stage[8 * (v >> 2) + 4 * h + (v & 3)][l32] = acc[c][v];
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            const int br = lane >> 1, c16 = (lane & 1) * 16;
            const float4 x0 = *reinterpret_cast<const float4 *>(&stage[br][c16]);
            const float4 x1 = *reinterpret_cast<const float4 *>(&stage[br][c16 + 4]);
            const float4 x2 = *reinterpret_cast<const float4 *>(&stage[br][c16 + 8]);
            const float4 x3 = *reinterpret_cast<const float4 *>(&stage[br][c16 + 12]);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            if (tb + br < B) {
                uint16_t *q = dP + (int64_t)rw.row * ld + (int64_t)(tb + br) * d + tc + c16;
                *reinterpret_cast<uint4 *>(q) = make_uint4(pack_bf16x2(x0.x, x0.y), pack_bf16x2(x0.z, x0.w),
                                                           pack_bf16x2(x1.x, x1.y), pack_bf16x2(x1.z, x1.w));
                *reinterpret_cast<uint4 *>(q + 8) = make_uint4(pack_bf16x2(x2.x, x2.y), pack_bf16x2(x2.z, x2.w),
                                                               pack_bf16x2(x3.x, x3.y), pack_bf16x2(x3.z, x3.w));
            }
        }
    }
}

// Heavy sources: dP[j] = sum of the row's unit partials.  One thread per float4 of a [B*d] row.
template <bool BF16>
__global__ void k_gather_t_finish(int32_t n_hv, const int32_t *__restrict__ hv_row,
                                  const int32_t *__restrict__ hv_unit_ptr, const float *__restrict__ partial,
                                  int32_t bd, void *__restrict__ dP, int64_t ld)
{
    const int bd4 = bd >> 2;
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (int64_t)n_hv * bd4) return;
    const int32_t h = (int32_t)(idx / bd4);
    const int k4 = (int)(idx - (int64_t)h * bd4) * 4;
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int32_t u = hv_unit_ptr[h]; u < hv_unit_ptr[h + 1]; ++u) {
        const float4 x = *reinterpret_cast<const float4 *>(partial + (int64_t)u * bd + k4);
        s.x += x.x; s.y += x.y; s.z += x.z; s.w += x.w;
    }
    const int64_t o = (int64_t)hv_row[h] * ld + k4;
    if (BF16) {
        uint2 x;
        x.x = pack_bf16x2(s.x, s.y); x.y = pack_bf16x2(s.z, s.w);
        *reinterpret_cast<uint2 *>(reinterpret_cast<uint16_t *>(dP) + o) = x;
    } else {
        *reinterpret_cast<float4 *>(reinterpret_cast<float *>(dP) + o) = s;
    }
}

// ------------------------------------------------------------------ run means
// One wavefront per (relation, destination) run s (or per unit of a long run):
//   Z[s][:] = invc_s * sum_{j in run s} H[j][:]
// the normalised neighbour sum of Eq. 1 for one relation, before any weight is applied.
// BF16: the input rows and Z are bf16 (sums stay fp32).
template <bool BF16, int LPR>
__global__ __launch_bounds__(64 * WPB) void k_run_mean(
    const int32_t *__restrict__ seg_ptr, const int32_t *__restrict__ seg_dst,
    const float *__restrict__ inv_c, const int32_t *__restrict__ col_src, int64_t S,
    int32_t n_units, const int32_t *__restrict__ hv_row, const int32_t *__restrict__ hv_unit_ptr,
    const int32_t *__restrict__ unit_hv, const void *__restrict__ H, int32_t d,
    void *__restrict__ Z, float *__restrict__ partial, const uint8_t *__restrict__ active, int skip_single)
{
    constexpr int VEC = MsgRow<BF16>::VEC;
    constexpr int NG = 64 / LPR;
    constexpr int U = (NG >= 8) ? 2 : (NG >= 2 ? 4 : 8);     // row loads in flight per lane
    const int lane = threadIdx.x & 63;
    const int64_t wid = (int64_t)blockIdx.x * WPB + (threadIdx.x >> 6);
    const RowWork rw = row_work(wid, seg_ptr, S, n_units, hv_row, hv_unit_ptr, unit_hv);
    if (rw.row < 0) return;
    if (skip_single && rw.unit < 0 && rw.end - rw.beg == 1) return;    // read in place by the consumer
    const int kl = lane % LPR, g = lane / LPR;
    const bool kact = kl * VEC < d;
    float acc[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) acc[v] = 0.f;
    const bool skip = active && !active[seg_dst[rw.row]];     // destination outside the sub-graph: zeros
    if (skip && rw.unit >= 0) return;
    const int len = skip ? 0 : rw.end - rw.beg;
    // 64 sources at a time, a lane each, handed out by shuffles; rounds of NG * U rows, the last one as many as there are.
    // No per-lane condition around a row's load (the loads of a round would wait for each other): a slot past the end
    // repeats the last row and is replaced by zeros, a lane past the width reads the row's start.  60 M edges into 5.8 M runs
    // of 128 floats: 5.22 ms with an index and a condition per load, 4.16 now (7.4 TB/s of rows)
    const int64_t col = kact ? kl * VEC : 0;
    for (int e0 = 0; e0 < len; e0 += 64) {
        const int cnt = min(64, len - e0);
        const int32_t mine = col_src[rw.beg + e0 + min(lane, cnt - 1)];
        for (int j0 = 0; j0 < cnt; j0 += NG * U) {
            const int slots = min(U, (cnt - j0 + NG - 1) / NG);          // uniform
            uint4 x[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int32_t src = __shfl(mine, min(j0 + u * NG + g, cnt - 1), 64);
                if (u < slots) x[u] = MsgRow<BF16>::load_raw(H, (int64_t)src * d + col);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (u >= slots) break;
                if (j0 + u * NG + g >= cnt) x[u] = make_uint4(0u, 0u, 0u, 0u);
                float val[VEC];
                MsgRow<BF16>::unpack(x[u], val);
#pragma unroll
                for (int v = 0; v < VEC; ++v) acc[v] += val[v];
            }
        }
    }
#pragma unroll
    for (int off = LPR; off < 64; off <<= 1)
#pragma unroll
        for (int v = 0; v < VEC; ++v) acc[v] += __shfl_xor(acc[v], off, 64);
    if (g != 0 || !kact) return;
    if (rw.unit >= 0) {
#pragma unroll
        for (int v4 = 0; v4 < VEC; v4 += 4)
            *reinterpret_cast<float4 *>(partial + (int64_t)rw.unit * d + kl * VEC + v4) =
                make_float4(acc[v4], acc[v4 + 1], acc[v4 + 2], acc[v4 + 3]);
        return;
    }
    const float w = skip ? 0.f : inv_c[rw.row];
#pragma unroll
    for (int v = 0; v < VEC; ++v) acc[v] *= w;
    if (BF16) {
        *reinterpret_cast<uint4 *>(reinterpret_cast<uint16_t *>(Z) + rw.row * d + kl * VEC) =
            make_uint4(pack_bf16x2(acc[0], acc[1]), pack_bf16x2(acc[2], acc[3]),
                       pack_bf16x2(acc[4 % VEC], acc[5 % VEC]), pack_bf16x2(acc[6 % VEC], acc[7 % VEC]));
    } else {
        typedef float rm_f32x4 __attribute__((ext_vector_type(4)));
        __builtin_nontemporal_store(rm_f32x4{acc[0], acc[1], acc[2], acc[3]},
                                    reinterpret_cast<rm_f32x4 *>(reinterpret_cast<float *>(Z) + rw.row * d + kl * VEC));
    }
}

// The same run means when most runs are very short (many relations: a run is often a single edge).
// One wavefront takes RPW consecutive runs; each lane group owns every NG-th of them and has the
// first source row of all its runs in flight at once, which is the whole sum for most.  Runs of
// KGE_HEAVY edges or more are left to the unit wavefronts of k_run_mean and k_run_mean_finish.
template <bool BF16, int LPR, int RPW>
__global__ __launch_bounds__(64 * WPB) void k_run_mean_multi(
    const int32_t *__restrict__ seg_ptr, const int32_t *__restrict__ seg_dst,
    const float *__restrict__ inv_c, const int32_t *__restrict__ col_src, int64_t S,
    const void *__restrict__ H, int32_t d, void *__restrict__ Z, const uint8_t *__restrict__ active, int skip_single,
    const int32_t *__restrict__ run_list)
{
    // run_list (optional): the wavefronts walk runs run_list[0 .. S) instead of runs 0 .. S
    constexpr int VEC = MsgRow<BF16>::VEC;
    constexpr int NG = 64 / LPR;
    constexpr int PER = RPW / NG;                          // runs per lane group
    static_assert(RPW % NG == 0 && RPW < 64, "runs per wavefront must be a multiple of the lane groups");
    const int lane = threadIdx.x & 63;
    const int64_t s0 = ((int64_t)blockIdx.x * WPB + (threadIdx.x >> 6)) * RPW;
    if (s0 >= S) return;
    const int kl = lane % LPR, g = lane / LPR;
    const bool kact = kl * VEC < d;
    // bounds of the RPW runs: lanes 0 .. RPW hold seg_ptr[s0 + lane]; with a list, lane r holds its run's
    // id and both of its bounds
    int32_t pv = 0, pe = 0, pid = 0;
    if (run_list) {
        if (lane < RPW && s0 + lane < S) { pid = run_list[s0 + lane]; pv = seg_ptr[pid]; pe = seg_ptr[pid + 1]; }
    } else if (lane <= RPW) {
        pv = seg_ptr[min(s0 + lane, S)];
    }
    int32_t beg[PER], len[PER], src0[PER], rid[PER];
    float w[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int r = i * NG + g;
        const int32_t b = __shfl(pv, r, 64), e1 = __shfl(pv, r + 1, 64), e2 = __shfl(pe, r, 64), id = __shfl(pid, r, 64);
        const int32_t e = run_list ? e2 : e1;
        const bool exists = s0 + r < S;
        const int64_t sr = run_list ? (int64_t)id : s0 + r;
        rid[i] = (int32_t)sr;
        beg[i] = b;
        len[i] = exists ? e - b : -1;                      // -1: no such run
        w[i] = 0.f;
        src0[i] = 0;
        if (len[i] >= KGE_HEAVY) len[i] = -1;              // written by the finishing kernel
        if (skip_single && len[i] == 1) len[i] = -1;       // read in place by the consumer
        if (len[i] > 0) {
            if (active && !active[seg_dst[sr]]) len[i] = 0;            // outside the sub-graph: a zero row
            else { w[i] = inv_c[sr]; src0[i] = col_src[b]; }
        }
    }
    // no condition stands around the rows' loads (each would wait for the one before): a run without edges reads row 0 and
    // drops it, a lane past the width the row's start
    const int64_t col = kact ? kl * VEC : 0;
    uint4 x0[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) x0[i] = MsgRow<BF16>::load_raw(H, (int64_t)src0[i] * d + col);
#pragma unroll
    for (int i = 0; i < PER; ++i) if (len[i] <= 0) x0[i] = make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        if (len[i] < 0) continue;
        float acc[VEC];
        MsgRow<BF16>::unpack(x0[i], acc);
        // the rest of a longer run, two rows at a time and, from the fourth edge on, four: the sources of the next rows are
        // fetched with these, so that a step is one memory round trip
        const int32_t last = beg[i] + (len[i] > 0 ? len[i] - 1 : 0);
        int32_t nx[4];
        if (len[i] > 1) {
#pragma unroll
            for (int u = 0; u < 4; ++u) nx[u] = col_src[min(beg[i] + 1 + u, last)];
        }
        for (int el = 1; el < len[i]; el += 4) {
            uint4 x[4];
            const bool more = el + 2 < len[i];
            x[0] = MsgRow<BF16>::load_raw(H, (int64_t)nx[0] * d + col);
            x[1] = MsgRow<BF16>::load_raw(H, (int64_t)nx[1] * d + col);
            if (more) {
                x[2] = MsgRow<BF16>::load_raw(H, (int64_t)nx[2] * d + col);
                x[3] = MsgRow<BF16>::load_raw(H, (int64_t)nx[3] * d + col);
#pragma unroll
                for (int u = 0; u < 4; ++u) nx[u] = col_src[min(beg[i] + el + 4 + u, last)];
            } else {
                x[2] = x[3] = make_uint4(0u, 0u, 0u, 0u);
            }
#pragma unroll
            for (int u = 1; u < 4; ++u) if (el + u >= len[i]) x[u] = make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
            for (int h = 0; h < 4; h += 2) {
                float va[VEC], vb[VEC];
                MsgRow<BF16>::unpack(x[h], va);
                MsgRow<BF16>::unpack(x[h + 1], vb);
#pragma unroll
                for (int v = 0; v < VEC; ++v) acc[v] += va[v] + vb[v];
            }
        }
        if (!kact) continue;
        const int64_t o = (int64_t)rid[i] * d + kl * VEC;
#pragma unroll
        for (int v = 0; v < VEC; ++v) acc[v] *= w[i];
        if (BF16) {
            typedef uint32_t rm_u32x4 __attribute__((ext_vector_type(4)));
            __builtin_nontemporal_store(rm_u32x4{pack_bf16x2(acc[0], acc[1]), pack_bf16x2(acc[2], acc[3]),
                                                 pack_bf16x2(acc[4 % VEC], acc[5 % VEC]), pack_bf16x2(acc[6 % VEC], acc[7 % VEC])},
                                        reinterpret_cast<rm_u32x4 *>(reinterpret_cast<uint16_t *>(Z) + o));
        } else {
            *reinterpret_cast<float4 *>(reinterpret_cast<float *>(Z) + o) = make_float4(acc[0], acc[1], acc[2], acc[3]);
        }
    }
}

// Long runs: Z[s] = invc_s * sum of the run's unit partials.  One thread per float4.
template <bool BF16>
__global__ void k_run_mean_finish(int32_t n_hv, const int32_t *__restrict__ hv_row,
                                  const int32_t *__restrict__ hv_unit_ptr, const float *__restrict__ partial,
                                  const float *__restrict__ inv_c, int32_t d, void *__restrict__ Z,
                                  const int32_t *__restrict__ seg_dst, const uint8_t *__restrict__ active)
{
    const int d4 = d >> 2;
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (int64_t)n_hv * d4) return;
    const int32_t h = (int32_t)(idx / d4);
    const int k4 = (int)(idx - (int64_t)h * d4) * 4;
    const int64_t row = hv_row[h];
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    if (!(active && !active[seg_dst[row]])) {
        for (int32_t u = hv_unit_ptr[h]; u < hv_unit_ptr[h + 1]; ++u) {
            const float4 x = *reinterpret_cast<const float4 *>(partial + (int64_t)u * d + k4);
            s.x += x.x; s.y += x.y; s.z += x.z; s.w += x.w;
        }
        const float w = inv_c[row];
        s.x *= w; s.y *= w; s.z *= w; s.w *= w;
    }
    if (BF16)
        *reinterpret_cast<uint2 *>(reinterpret_cast<uint16_t *>(Z) + row * d + k4) =
            make_uint2(pack_bf16x2(s.x, s.y), pack_bf16x2(s.z, s.w));
    else
        *reinterpret_cast<float4 *>(reinterpret_cast<float *>(Z) + row * d + k4) = s;
}

// ------------------------------------------------------------------ coefficient gradient
// da[r][b] += sum of seg_out[s][b] over one chunk of relation r's runs (the partition's chunk list: every chunk lies
// in one relation).  A run's B values are covered by TPR threads of V floats each (V = 4 when B is a multiple
// of 4); the block's 256 / TPR run slots walk the chunk with four rows in flight per thread.
template <int V>
__global__ __launch_bounds__(256) void k_coeff_reduce(const int32_t *__restrict__ c_rel, const int32_t *__restrict__ c_beg,
                                                      const int32_t *__restrict__ c_end,
                                                      const float *__restrict__ seg_out, int32_t B, int32_t TPR,
                                                      float *__restrict__ da)
{
    __shared__ float red[256 * V];
    const int r = c_rel[blockIdx.x];
    const int64_t beg = c_beg[blockIdx.x], end = c_end[blockIdx.x];
    const int slots = 256 / TPR;
    const int b = (threadIdx.x % TPR) * V, slot = threadIdx.x / TPR;
    float acc[V];
#pragma unroll
    for (int v = 0; v < V; ++v) acc[v] = 0.f;
    if (b < B) {
        int64_t s = beg + slot;
        for (; s + 3 * slots < end; s += 4 * slots) {
            float x[4][V];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const float *q = seg_out + (s + (int64_t)u * slots) * B + b;
                if (V == 4) { const float4 t4 = *reinterpret_cast<const float4 *>(q); x[u][0] = t4.x; x[u][1 % V] = t4.y; x[u][2 % V] = t4.z; x[u][3 % V] = t4.w; }
                else x[u][0] = q[0];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int v = 0; v < V; ++v) acc[v] += x[u][v];
        }
        for (; s < end; s += slots)
#pragma unroll
            for (int v = 0; v < V; ++v) acc[v] += seg_out[s * B + b + v];
    }
#pragma unroll
    for (int v = 0; v < V; ++v) red[threadIdx.x * V + v] = acc[v];
    __syncthreads();
    if (slot == 0 && b < B) {
#pragma unroll
        for (int v = 0; v < V; ++v) {
            float t = 0.f;
            for (int k = 0; k < slots; ++k) t += red[(k * TPR + threadIdx.x) * V + v];
            if (t != 0.f) unsafeAtomicAdd(&da[(int64_t)r * B + b + v], t);
        }
    }
}

int pow2_at_least(int x) { int p = 1; while (p < x) p <<= 1; return p; }
int largest_pow2_dividing(int x, int cap) { int p = 1; while (p * 2 <= cap && x % (p * 2) == 0) p <<= 1; return p; }

}  // namespace

// ------------------------------------------------------------------ launchers
#define DISPATCH_LPR(LPRV, CALL)                                                        \
    switch (LPRV) {                                                                     \
    case 1: { constexpr int L = 1; CALL; } break;                                       \
    case 2: { constexpr int L = 2; CALL; } break;                                       \
    case 4: { constexpr int L = 4; CALL; } break;                                       \
    case 8: { constexpr int L = 8; CALL; } break;                                       \
    case 16: { constexpr int L = 16; CALL; } break;                                     \
    case 32: { constexpr int L = 32; CALL; } break;                                     \
    default: { constexpr int L = 64; CALL; } break;                                     \
    }

// out[i] = act( sum_{q in row i of the view} w_q X[idx_q][:] + Self[i] ),  X rows of d elements (fp32 or bf16)
static int launch_row_sum(const int32_t *ptr, const int32_t *idx, const float *w, int64_t n_rows,
                          const kge_heavy_index &hx, const char *name, const void *X, int x_bf16, int32_t d,
                          const float *Self, int act, float *out, float *out2, uint16_t *outbf, float *partial,
                          const uint8_t *active, hipStream_t st, EdgeGate gate = {nullptr, 0}, bool finish = true)
{
    if (n_rows == 0) return KGE_OK;
    const int vec = x_bf16 ? 8 : 4;
    const int lpr = pow2_at_least((d + vec - 1) / vec);
    KGE_REQUIRE(lpr <= 64, KGE_EINVAL, "feature width %d too large for the aggregation kernel", d);
    const unsigned grid = (unsigned)cdiv(n_rows + hx.n_units, WPB);
    {
        KGE_PROF(name, st);
#define RS_ARGS ptr, idx, nullptr, w, n_rows, hx.n_units, hx.hv_row, hx.hv_unit_ptr, hx.unit_hv, X, nullptr, 1, d, 1, \
                Self, act, out, out2, outbf, partial, active, gate
        if (x_bf16) { DISPATCH_LPR(lpr, (k_gather_fwd<true, L, true><<<grid, 64 * WPB, 0, st>>>(RS_ARGS))); }
        else { DISPATCH_LPR(lpr, (k_gather_fwd<false, L, true><<<grid, 64 * WPB, 0, st>>>(RS_ARGS))); }
#undef RS_ARGS
    }
    KGE_LAUNCH_CHECK();
    if (finish && hx.n_hv > 0) {
        KGE_PROF("gather_fwd_fin", st);
        const int64_t n = (int64_t)hx.n_hv * (d / 4);
        k_gather_fwd_finish<<<(unsigned)cdiv(n, 256), 256, 0, st>>>(hx.n_hv, hx.hv_row, hx.hv_unit_ptr, partial, d,
                                                                   Self, act, out, out2, outbf, active);
        KGE_LAUNCH_CHECK();
    }
    return KGE_OK;
}

// Bytes: the form with a row per (source, relation) reads P once, writes and reads fp32 rows of the groups and gathers one
// fp32 row per edge; the other one gathers B rows per edge.  What has to be saved pays for the launches (about 5 us each at
// the rate of the gathers): one more, and two where both forms are launched and a sub-graph's size decides.
// Whole forward passes, us, a row per pair / B rows per edge: 14,541 entities x 272,115 triples, d = 64: 3 bases 70 / 81, 4
// bases 73 / 100; d = 200: 3 bases 193 / 257; one relation, 1 M triples, d = 128, 2 bases 274 / 302; 50,021 entities x
// 1 M triples, 128 bf16: 6 bases 457 / 477, 8 bases 458 / 593.
static double relation_rows_fixed(const kge_partition *p, int32_t B, int32_t d, int msg_bf16)
{
    return d * ((double)p->n_vert * B * (msg_bf16 ? 2 : 4) + 8.0 * (double)p->n_sgrp);
}
static double relation_rows_per_edge(int32_t B, int32_t d, int msg_bf16) { return (double)d * (B * (msg_bf16 ? 2 : 4) - 4); }
// Bytes do not cost the same, though: rows of P, few bases of it above all, come from caches that a larger Q does not fit.  So
// the form has to pay as well when a gathered byte of an array of 256 MB (the last-level cache) or more counts 1.75, of a
// smaller one in proportion less, a byte of Q that is written 1.75 and one of P that is read once 1.  Forward passes, us, a row per pair / B rows per edge: 20,000 entities x 1.5
// M triples, 237 relations, 2.4 edges per pair: d = 64, 2 bases 210 / 151, d = 200, 2 bases 648 / 542, d = 128, 4 bases of
// bf16 437 / 322; 50,021 entities x 1 M triples, 40 relations, 4 bases of 128 bf16 332 / 294.  Of 1615 shapes that the bytes alone
// take, 43 were more than 2 % slower so (at most 1.39), with both conditions 16 (at most 1.17); 2 lose what they gained (8 %).
struct RelationRowsCost { double per_edge, fixed; };
static RelationRowsCost relation_rows_cached(const kge_partition *p, int32_t B, int32_t d, int msg_bf16)
{
    const double P = (double)p->n_vert * d * B * (msg_bf16 ? 2 : 4), Q = 4.0 * d * (double)p->n_sgrp;
    auto weight = [](double bytes) { return 1.0 + 0.75 * std::min(1.0, bytes / 2.56e8); };
    return {d * (B * (msg_bf16 ? 2 : 4) * weight(P) - 4 * weight(Q)), P + 1.75 * Q};
}
static bool relation_rows_pay(const kge_partition *p, int32_t B, int32_t d, int msg_bf16, double least)
{
    const RelationRowsCost c = relation_rows_cached(p, B, d, msg_bf16);
    return p->n_edge * relation_rows_per_edge(B, d, msg_bf16) > relation_rows_fixed(p, B, d, msg_bf16) + least &&
           p->n_edge * c.per_edge > c.fixed + least;
}
// edges of a sub-graph from which it pays
static unsigned long long relation_rows_edges(const kge_partition *p, int32_t B, int32_t d, int msg_bf16)
{
    const RelationRowsCost c = relation_rows_cached(p, B, d, msg_bf16);
    return (unsigned long long)std::max(relation_rows_fixed(p, B, d, msg_bf16) / relation_rows_per_edge(B, d, msg_bf16), c.fixed / c.per_edge);
}
constexpr double ONE_LAUNCH = 3.2e7;
bool gather_by_relation(const kge_partition *p, int32_t B, int32_t d, int msg_bf16)
{
    return relation_rows_pay(p, B, d, msg_bf16, ONE_LAUNCH);
}

template <bool BF16>
static int launch_relation_rows(const kge_partition *p, const void *P, const float *a, int32_t B, int32_t d, float *Q,
                                const uint8_t *src_active, EdgeGate gate, hipStream_t st)
{
    const kge_heavy_index &hx = p->hv_sg;
    const int lpr = pow2_at_least((d + MsgRow<BF16>::VEC - 1) / MsgRow<BF16>::VEC);
    const unsigned grid = (unsigned)cdiv(p->n_vert + hx.n_units, WPB);
    KGE_PROF("gather_rows", st);
#define RR_ARGS p->sg_ptr, p->sg_rel, p->n_vert, hx.n_units, hx.hv_row, hx.hv_unit_ptr, hx.unit_hv, P, a, B, d, Q, src_active, gate
    if (B <= 4) { DISPATCH_LPR(lpr, (k_relation_rows<BF16, L, 4><<<grid, 64 * WPB, 0, st>>>(RR_ARGS))); }
    else if (B <= 8) { DISPATCH_LPR(lpr, (k_relation_rows<BF16, L, 8><<<grid, 64 * WPB, 0, st>>>(RR_ARGS))); }
    else if (B <= 12) { DISPATCH_LPR(lpr, (k_relation_rows<BF16, L, 12><<<grid, 64 * WPB, 0, st>>>(RR_ARGS))); }
    else { DISPATCH_LPR(lpr, (k_relation_rows<BF16, L, 16><<<grid, 64 * WPB, 0, st>>>(RR_ARGS))); }
#undef RR_ARGS
    KGE_LAUNCH_CHECK();
    return KGE_OK;
}

int launch_gather_forward(const kge_partition *p, const void *P, int msg_bf16, const float *a,
                          int32_t B, int32_t d, const float *Self, int act, float *out, float *out2,
                          float *partial, float *rel_rows, const uint8_t *active, const uint8_t *src_active,
                          const unsigned long long *n_active_edges, hipStream_t st)
{
    const int64_t N = p->n_vert;
    if (N == 0) return KGE_OK;
    const int vec = msg_bf16 ? 8 : 4;
    const int lpr = pow2_at_least((d + vec - 1) / vec);
    KGE_REQUIRE(lpr <= 64, KGE_EINVAL, "feature width %d too large for the aggregation kernel", d);
    const int gbc = largest_pow2_dividing(B, 64 / lpr);
    const kge_heavy_index &hx = p->hv_dm;
    EdgeGate gate = {nullptr, 0};
    if (relation_rows_pay(p, B, d, msg_bf16, active ? 4 * ONE_LAUNCH : ONE_LAUNCH)) {
        // with a sub-graph: only if it has the edges that pay for all groups' rows
        if (active) gate = {n_active_edges, relation_rows_edges(p, B, d, msg_bf16)};
        int rc = msg_bf16 ? launch_relation_rows<true>(p, P, a, B, d, rel_rows, src_active, gate, st)
                          : launch_relation_rows<false>(p, P, a, B, d, rel_rows, src_active, gate, st);
        if (rc != KGE_OK) return rc;
        rc = launch_row_sum(p->dm_ptr, p->dm_grp, p->dm_invc, N, hx, "gather_fwd", rel_rows, 0, d, Self, act, out, out2, nullptr,
                            partial, active, st, gate, !gate.count);
        if (rc != KGE_OK || !gate.count) return rc;
    }
    const unsigned grid = (unsigned)cdiv(N + hx.n_units, WPB);
    {
        KGE_PROF("gather_fwd", st);
#define GF_ARGS p->dm_ptr, p->dm_src, p->dm_rel, p->dm_invc, N, hx.n_units, hx.hv_row, hx.hv_unit_ptr, hx.unit_hv, \
                P, a, B, d, gbc, Self, act, out, out2, nullptr, partial, active, gate
        if (msg_bf16) { DISPATCH_LPR(lpr, (k_gather_fwd<true, L, false><<<grid, 64 * WPB, 0, st>>>(GF_ARGS))); }
        else { DISPATCH_LPR(lpr, (k_gather_fwd<false, L, false><<<grid, 64 * WPB, 0, st>>>(GF_ARGS))); }
#undef GF_ARGS
    }
    KGE_LAUNCH_CHECK();
    if (hx.n_hv > 0) {
        KGE_PROF("gather_fwd_fin", st);
        const int64_t n = (int64_t)hx.n_hv * (d / 4);
        k_gather_fwd_finish<<<(unsigned)cdiv(n, 256), 256, 0, st>>>(hx.n_hv, hx.hv_row, hx.hv_unit_ptr, partial, d,
                                                                   Self, act, out, out2, nullptr, active);
        KGE_LAUNCH_CHECK();
    }
    return KGE_OK;
}

// out[i] = act( sum over the runs (r, i) of destination i of U[run][:] + Self[i] )
int launch_sum_runs(const kge_partition *p, const void *U, int u_bf16, int32_t d, const float *Self, int act,
                    float *out, float *out2, void *out_bf16, float *partial, const uint8_t *active, hipStream_t st)
{
    return launch_row_sum(p->dr_ptr, p->dr_seg, nullptr, p->n_vert, p->hv_dr, "sum_runs", U, u_bf16, d, Self, act,
                          out, out2, reinterpret_cast<uint16_t *>(out_bf16), partial, active, st);
}

// dH[j] = sum over the edges e out of j of invc_e dZ[run(e)][:] + Self[j]
int launch_sum_edges_out(const kge_partition *p, const void *dZ, int z_bf16, int32_t d, const float *Self,
                         float *out, float *partial, const uint8_t *active, hipStream_t st)
{
    return launch_row_sum(p->sm_ptr, p->sm_seg, p->sm_invc, p->n_vert, p->hv_sm, "sum_edges_out", dZ, z_bf16, d, Self,
                          KGE_ACT_IDENTITY, out, nullptr, nullptr, partial, active, st);
}

int launch_act_backward(const float *dHout, const float *Hout, int act, int64_t n, float *G, hipStream_t st)
{
    if (n == 0) return KGE_OK;
    int64_t n4 = n / 4;
    int64_t blocks = cdiv(n4, 256);
    if (blocks > 65536) blocks = 65536;
    KGE_PROF("act_bwd", st);
    k_act_backward<<<(unsigned)blocks, 256, 0, st>>>(reinterpret_cast<const float4 *>(dHout),
                                                    reinterpret_cast<const float4 *>(Hout), act, n4,
                                                    reinterpret_cast<float4 *>(G));
    KGE_LAUNCH_CHECK();
    return KGE_OK;
}

// rows of dP whose edges were cut into units: their partial sums added up
static int launch_gather_t_finish(const kge_heavy_index &hx, const float *partial, int32_t bd, void *dP, int64_t ld, bool bf16,
                                  hipStream_t st)
{
    if (hx.n_hv == 0) return KGE_OK;
    KGE_PROF("gather_t_fin", st);
    const int64_t n = (int64_t)hx.n_hv * (bd / 4);
    if (bf16) k_gather_t_finish<true><<<(unsigned)cdiv(n, 256), 256, 0, st>>>(hx.n_hv, hx.hv_row, hx.hv_unit_ptr, partial, bd, dP, ld);
    else k_gather_t_finish<false><<<(unsigned)cdiv(n, 256), 256, 0, st>>>(hx.n_hv, hx.hv_row, hx.hv_unit_ptr, partial, bd, dP, ld);
    KGE_LAUNCH_CHECK();
    return KGE_OK;
}

template <bool BF16, int LPR, int NB, bool DP, bool SPREAD = false>
static int launch_source_backward_nb(const kge_partition *p, const float *G, const float *a, const void *P, int32_t B, int32_t d,
                                     void *dP, int64_t ld, float *partial, float *seg_scratch, const uint8_t *active, hipStream_t st)
{
    const kge_heavy_index &hx = p->hv_sm;
    const int n_chunks = (int)cdiv(B, SPREAD ? NB : 64 / LPR * NB);
    const int64_t blocks = cdiv((p->n_vert + hx.n_units) * n_chunks, WPB);
    KGE_REQUIRE(blocks < 0x7fffffffLL, KGE_ERANGE, "grid too large");
    KGE_PROF(DP ? "gather_t" : "coeff_seg", st);
    auto run = [&](auto full) {
        k_source_backward<BF16, LPR, NB, DP, SPREAD, decltype(full)::value><<<(unsigned)blocks, 64 * WPB, 0, st>>>(
            p->sm_ptr, p->sm_dst, p->sm_rel, p->sm_invc, p->sm_seg, p->n_vert, hx.n_units, hx.hv_row, hx.hv_unit_ptr, hx.unit_hv, G, a,
            P, B, d, n_chunks, dP, ld, partial, seg_scratch, active);
    };
    if (SPREAD || d == 4 * LPR) run(std::true_type{});
    else run(std::false_type{});
    KGE_LAUNCH_CHECK();
    return KGE_OK;
}

template <bool BF16, int NBLK, bool DP>
static int launch_source_cores(const kge_partition *p, const float *G, const float *a, const void *P, int32_t B, int32_t d,
                               void *dP, int64_t ld, float *partial, float *seg_scratch, const uint8_t *active, hipStream_t st)
{
    const kge_heavy_index &hx = p->hv_sm;
    const int n_chunks = (int)cdiv(B, 16);
    const int64_t blocks = (p->n_vert + hx.n_units) * n_chunks;
    KGE_REQUIRE(blocks < 0x7fffffffLL, KGE_ERANGE, "grid too large");
    KGE_PROF(DP ? "gather_t" : "coeff_seg", st);
    k_source_cores<BF16, NBLK, DP><<<(unsigned)blocks, 64, 0, st>>>(
        p->sm_ptr, p->sm_dst, p->sm_rel, p->sm_invc, p->sm_seg, p->n_vert, hx.n_units, hx.hv_row, hx.hv_unit_ptr, hx.unit_hv, G, a,
        P, B, d, n_chunks, dP, ld, partial, seg_scratch, active);
    KGE_LAUNCH_CHECK();
    return KGE_OK;
}

// The vector form: the fewest bases per lane that cover B in one chunk, 16 per wavefront at most; the dot products alone (at 32
// columns, beyond them the matrix cores): always those 16.
// At most 4 bases of rows of at most 16 lanes, six edges or more per relation of a source on average: shared edges (2 M
// edges of 20,000 sources, one relation: d = 16, 2 bases 128 -> 65 us, d = 64, 4 bases 131 -> 74; 6.3 edges per relation:
// 141 -> 114 and 146 -> 144; 4.2 edges: 152 -> 161 and 160 -> 200).
template <bool BF16, bool DP>
static int launch_source_backward(const kge_partition *p, const float *G, const float *a, const void *P, int32_t B, int32_t d,
                                  void *dP, int64_t ld, float *partial, float *seg_scratch, const uint8_t *active, hipStream_t st)
{
#define SB_CALL(LPRV, NBV) return launch_source_backward_nb<BF16, LPRV, NBV, DP>(p, G, a, P, B, d, dP, ld, partial, seg_scratch, active, st)
    if constexpr (DP)
        if (d <= 64 && B <= 4 && p->n_edge >= 6 * p->n_seg) {      // lane groups without a basis, and edges to share
#define SB_SPREAD(LPRV, NBV) return launch_source_backward_nb<BF16, LPRV, NBV, DP, true>(p, G, a, P, B, d, dP, ld, partial, seg_scratch, active, st)
            if (d > 32) {
                if (B == 1) SB_SPREAD(16, 1);
                if (B == 2) SB_SPREAD(16, 2);
                SB_SPREAD(16, 4);
            }
            if (B == 1) SB_SPREAD(8, 1);
            if (B == 2) SB_SPREAD(8, 2);
            SB_SPREAD(8, 4);
#undef SB_SPREAD
        }
    // The matrix cores' tiles are 16 groups x 16 bases: from 9 bases on they are well enough filled (whole backward passes, us,
    // cores / not: 14,541 entities x 272,115 triples, d = 200, 10 bases 315 / 470, d = 256, 9 bases 398 / 466, d = 128, 9 bases
    // 228 / 338; 50,000 entities with 8 groups each, d = 128, 10 bases 392 / 425).  With fewer bases where sources have enough
    // relations: up to 64 columns 6 on average (d = 64, 1 to 8 bases 115 / 144 to 153 / 190; 4 groups each: 424 / 387 at 5
    // bases), up to 208 columns 16 and 5 bases (d = 200, 5 bases 296 / 359, 4 bases 308 / 269; d = 128, 6 bases 209 / 222,
    // with 8 groups each 329 / 267; d = 256, 8 bases 394 / 383)
    const int64_t per_source = p->n_sgrp / (p->n_vert > 0 ? p->n_vert : 1);
    const bool cores = d > 32 && (B >= 9 || (d <= 64 ? per_source >= 6 : d <= 208 && B >= 5 && per_source >= 16));
#define SB_CORES(NBLKV) return launch_source_cores<BF16, NBLKV, DP>(p, G, a, P, B, d, dP, ld, partial, seg_scratch, active, st)
    if (cores) {
        if (d <= 64) SB_CORES(4);
        if (d <= 128) SB_CORES(8);
        if (d <= 208) SB_CORES(13);
        SB_CORES(16);
    }
#undef SB_CORES
    if constexpr (DP) {                                  // 8 bases at most beyond 32 columns
        if (d > 128) {
            if (B <= 2) SB_CALL(64, 2);
            if (B <= 4) SB_CALL(64, 4);
            SB_CALL(64, 8);
        }
        if (d > 64) {
            if (B <= 2) SB_CALL(32, 1);
            if (B <= 4) SB_CALL(32, 2);
            SB_CALL(32, 4);
        }
        if (d > 32) {
            if (B <= 4) SB_CALL(16, 1);
            SB_CALL(16, 2);
        }
        if (B <= 8) SB_CALL(8, 1);
    }
    SB_CALL(8, 2);
#undef SB_CALL
}

int launch_project_first_backward(const kge_partition *p, const void *P, int msg_bf16, const float *G, const float *a,
                                  int32_t B, int32_t d, float *seg_scratch, float *partial, float *da, void *dP, int64_t ld,
                                  const uint8_t *active, hipStream_t st)
{
    KGE_REQUIRE(B <= 256 && d <= 256, KGE_EINVAL, "more than 256 bases or a wider row than 256 are not supported");
    if (p->n_vert == 0) return KGE_OK;
    int rc;
    if (!dP) rc = launch_source_backward<true, false>(p, G, a, P, B, d, dP, ld, partial, seg_scratch, active, st);
    else if (msg_bf16) rc = launch_source_backward<true, true>(p, G, a, P, B, d, dP, ld, partial, seg_scratch, active, st);
    else rc = launch_source_backward<false, true>(p, G, a, P, B, d, dP, ld, partial, seg_scratch, active, st);
    if (rc == KGE_OK && dP) rc = launch_gather_t_finish(p->hv_sm, partial, B * d, dP, ld, msg_bf16 != 0, st);
    if (rc != KGE_OK || p->n_relc == 0) return rc;
    KGE_PROF("coeff_reduce", st);
    if (B % 4 == 0) k_coeff_reduce<4><<<(unsigned)p->n_relc, 256, 0, st>>>(p->relc_rel, p->relc_beg, p->relc_end, seg_scratch, B,
                                                                    pow2_at_least(B / 4), da);
    else k_coeff_reduce<1><<<(unsigned)p->n_relc, 256, 0, st>>>(p->relc_rel, p->relc_beg, p->relc_end, seg_scratch, B,
                                                                pow2_at_least(B), da);
    KGE_LAUNCH_CHECK();
    return KGE_OK;
}

// The bf16 form of dP: Gbf = the bf16 copy of G, rows `ldg` elements apart.  For layers with at least 32 bases and a width
// that is a multiple of 32; other shapes go the general way from the fp32 G.
bool gather_transpose_bf16_supported(int32_t B, int32_t d) { return B >= 32 && d % 32 == 0 && d >= 32; }

int launch_gather_transpose_bf16(const kge_partition *p, const void *Gbf, int64_t ldg, const float *a, int32_t B,
                                 int32_t d, void *dP, int64_t ld, float *partial, const uint8_t *active, hipStream_t st)
{
    KGE_REQUIRE(gather_transpose_bf16_supported(B, d), KGE_EINVAL, "transposed aggregation: shape not supported by the bf16 kernel");
    KGE_REQUIRE(ldg % 8 == 0 && ((uintptr_t)Gbf % 16) == 0 && ld % 8 == 0 && ((uintptr_t)dP % 16) == 0, KGE_EINVAL,
                "transposed aggregation: rows must be 16-byte aligned");
    const kge_heavy_index &hx = p->hv_sm;
    if (p->n_vert == 0) return KGE_OK;
    const int n_bchunks = (B + 63) / 64, n_cchunks = (d + 255) / 256;
    const int64_t blocks = ((int64_t)p->n_vert + hx.n_units) * n_bchunks * n_cchunks;
    KGE_REQUIRE(blocks < 0x7fffffffLL, KGE_ERANGE, "grid too large");
    {
        KGE_PROF("gather_t", st);
        k_gather_t_bf16<<<(unsigned)blocks, 256, 0, st>>>(p->sm_ptr, p->sm_dst, p->sm_rel, p->sm_invc, p->n_vert, hx.n_units,
                                                         hx.hv_row, hx.hv_unit_ptr, hx.unit_hv,
                                                         reinterpret_cast<const uint16_t *>(Gbf), ldg, a, B, d, n_bchunks,
                                                         n_cchunks, reinterpret_cast<uint16_t *>(dP), ld, partial, active);
        KGE_LAUNCH_CHECK();
    }
    return launch_gather_t_finish(p->hv_sm, partial, B * d, dP, ld, true, st);
}

// Z[s][:] = invc_s * sum_{j in run s} H[j][:]; H and Z fp32, or both bf16; `partial`: [hv_seg.n_units][d] floats
int launch_run_mean(const kge_partition *p, const void *H, int32_t d, void *Z, int bf16, float *partial,
                    const uint8_t *active, int skip_single, hipStream_t st)
{
    const int64_t S = p->n_seg;
    if (S == 0) return KGE_OK;
    // single-edge runs skipped: only the listed runs of two or more edges are visited
    const int32_t *run_list = skip_single && p->mrun ? p->mrun : nullptr;
    const int64_t n_visit = run_list ? p->n_mrun : S;
    const int vec = bf16 ? 8 : 4;
    const int lpr = pow2_at_least((d + vec - 1) / vec);
    KGE_REQUIRE(lpr <= 64, KGE_EINVAL, "feature width %d too large for the run-mean kernel", d);
    const kge_heavy_index &hx = p->hv_seg;
    if (p->n_edge < 3 * S && lpr >= 8) {
        // mostly very short runs: several runs per wavefront; the unit wavefronts of the general kernel
        // still take the heavy runs (it is launched with no light rows)
        constexpr int RPW = 8;
        KGE_PROF("run_mean", st);
        const unsigned gridm = (unsigned)cdiv(cdiv(n_visit, RPW), WPB);
#define RMM_ARGS p->seg_ptr, p->seg_dst, p->inv_c, p->col_src, n_visit, H, d, Z, active, skip_single, run_list
        if (bf16) { DISPATCH_LPR(lpr, (k_run_mean_multi<true, (L < 8 ? 8 : L), RPW><<<gridm, 64 * WPB, 0, st>>>(RMM_ARGS))); }
        else { DISPATCH_LPR(lpr, (k_run_mean_multi<false, (L < 8 ? 8 : L), RPW><<<gridm, 64 * WPB, 0, st>>>(RMM_ARGS))); }
#undef RMM_ARGS
        KGE_LAUNCH_CHECK();
        if (hx.n_units > 0) {
            const unsigned gridu = (unsigned)cdiv(hx.n_units, WPB);
#define RMU_ARGS p->seg_ptr, p->seg_dst, p->inv_c, p->col_src, (int64_t)0, hx.n_units, hx.hv_row, hx.hv_unit_ptr, hx.unit_hv, \
                 H, d, Z, partial, active, 0
            if (bf16) { DISPATCH_LPR(lpr, (k_run_mean<true, L><<<gridu, 64 * WPB, 0, st>>>(RMU_ARGS))); }
            else { DISPATCH_LPR(lpr, (k_run_mean<false, L><<<gridu, 64 * WPB, 0, st>>>(RMU_ARGS))); }
#undef RMU_ARGS
            KGE_LAUNCH_CHECK();
        }
    } else {
    const unsigned grid = (unsigned)cdiv(S + hx.n_units, WPB);
    {
        KGE_PROF("run_mean", st);
#define RM_ARGS p->seg_ptr, p->seg_dst, p->inv_c, p->col_src, S, hx.n_units, hx.hv_row, hx.hv_unit_ptr, hx.unit_hv, \
                H, d, Z, partial, active, skip_single
        if (bf16) { DISPATCH_LPR(lpr, (k_run_mean<true, L><<<grid, 64 * WPB, 0, st>>>(RM_ARGS))); }
        else { DISPATCH_LPR(lpr, (k_run_mean<false, L><<<grid, 64 * WPB, 0, st>>>(RM_ARGS))); }
#undef RM_ARGS
    }
    KGE_LAUNCH_CHECK();
    }
    if (hx.n_hv > 0) {
        KGE_PROF("run_mean_fin", st);
        const int64_t n = (int64_t)hx.n_hv * (d / 4);
        if (bf16) k_run_mean_finish<true><<<(unsigned)cdiv(n, 256), 256, 0, st>>>(hx.n_hv, hx.hv_row, hx.hv_unit_ptr, partial,
                                                                                p->inv_c, d, Z, p->seg_dst, active);
        else k_run_mean_finish<false><<<(unsigned)cdiv(n, 256), 256, 0, st>>>(hx.n_hv, hx.hv_row, hx.hv_unit_ptr, partial,
                                                                             p->inv_c, d, Z, p->seg_dst, active);
        KGE_LAUNCH_CHECK();
    }
    return KGE_OK;
}
