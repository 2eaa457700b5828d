// Dense contractions of the encoder (Eq. 2 applied to every vertex, and its two
// transposes for the backward pass) on the gfx950 matrix cores.
//
//   project      P = H [V_1 .. V_B | W_0]                      (N x d_in) (d_in x (B+1)d_out)
//   weight_grad  d[V_1 .. V_B | W_0] = H^T [dP | G]            (d_in x N) (N x (B+1)d_out)
//   input_grad   dH = [dP | G] [V_1 .. V_B | W_0]^T            (N x (B+1)d_out) ((B+1)d_out x d_in)
//
// and, for layers that apply W_r per (relation, destination) run,
//
//   rel_outer    C_r = sum_{runs s of r} Z_s^T G_{dst(s)}        grouped over relations, (d_in x d_out) each
//   coeff        da = C Vflat^T                                  (2R x d_in d_out) (d_in d_out x B)
//
// One kernel template: 128x128 block tile, 4 wavefronts in a 2x2 grid, each wavefront owns a 64x64 sub-tile as
// 2x2 accumulators of 32x32.  The fp32 operands are split into three bf16 parts each on their way into LDS and
// multiplied on the bf16 matrix cores (split_bf16.h: six products per term, fp32 accuracy).  Operand loaders and the
// epilogue are small functors, so the concatenated operands ([V|W0], [dP|G]) are never materialised.  This file is
// the fp32 path; workloads with bf16 messages use the bf16 matrix-core kernels of gemm_bf16.hip.
#include "common.h"
#include "split_bf16.h"

#include <type_traits>

namespace {

constexpr int BM = 128, BN = 128, BK = 16, GT = 256;
constexpr int LP = 48;                      // bytes per row of a part in LDS: 16 bf16 and 16 bytes of padding, an odd
                                            // multiple of 16, so that 16-byte reads of 8 rows touch every bank once
constexpr int PLANE = 128 * LP;             // one part of a 128-row operand tile
constexpr int FLUSH = 8;                    // steps after which the matrix cores' sums move to a second set (below)

// ---- operands.  An operand is seen as rows x (rows of the output for A, its columns for B) times the contraction
// index k, and its memory is contiguous either along k (KC) or along x.  Extents along the contiguous index are
// multiples of 4.  bind(g) selects group g's matrix.
//   KC:  start(c, ps, x) sets up row x (in range) as piece ps of cursor c; at(c, ps, k) is where its k.. lie; k does not
//        decrease from call to call
//   !KC: start(c, x) sets up columns x..; row(k) is the stored row of contraction index k; at(c, row)
// Cursors hold addresses, so that a step's loads cost an addition each.  el(x, k): one element.

struct RowsK {                  // KC: rows of p, ld apart, optionally picked through a list
    static constexpr bool KC = true;
    const float *__restrict__ p; int64_t ld; const int32_t *__restrict__ idx; int64_t gstride;
    struct Cur { const float *q[2]; };
    __device__ __forceinline__ void bind(int32_t g) { p += g * gstride; }
    __device__ __forceinline__ void start(Cur &c, int ps, int64_t x) const { c.q[ps] = p + (idx ? (int64_t)idx[x] : x) * ld; }
    __device__ __forceinline__ const float *at(Cur &c, int ps, int32_t k) const { return c.q[ps] + k; }
    __device__ __forceinline__ float el(int64_t x, int64_t k) const { return p[(idx ? (int64_t)idx[x] : x) * ld + k]; }
};
struct XcatK {                  // KC: row x of [dP | G]
    static constexpr bool KC = true;
    const float *dP, *G; int32_t d_out, bd;
    struct Cur { const float *a[2], *g[2]; };
    __device__ __forceinline__ void bind(int32_t) {}
    __device__ __forceinline__ void start(Cur &c, int ps, int64_t x) const { c.a[ps] = dP + x * bd; c.g[ps] = G + x * d_out - bd; }
    __device__ __forceinline__ const float *at(Cur &c, int ps, int32_t k) const { return (k < bd ? c.a[ps] : c.g[ps]) + k; }
    __device__ __forceinline__ float el(int64_t x, int64_t k) const { return k < bd ? dP[x * bd + k] : G[x * d_out + k - bd]; }
};
struct WcatK {                  // KC: row x of every V_b, then of W_0, end to end
    static constexpr bool KC = true;
    const float *V, *W0; int32_t d_in, d_out, B;
    struct Cur { int64_t x[2]; int32_t b, kb; };
    __device__ __forceinline__ void bind(int32_t) {}
    __device__ __forceinline__ void start(Cur &c, int ps, int64_t x) const { c.x[ps] = x * d_out; c.b = 0; c.kb = 0; }
    __device__ __forceinline__ const float *at(Cur &c, int ps, int32_t k) const
    {
        while (k - c.kb >= d_out) { c.kb += d_out; ++c.b; }
        return (c.b < B ? V + (int64_t)c.b * d_in * d_out : W0) + c.x[ps] + (k - c.kb);
    }
    __device__ __forceinline__ float el(int64_t x, int64_t k) const
    {
        const int64_t b = k / d_out;
        return (b < B ? V + b * d_in * d_out : W0)[x * d_out + k - b * d_out];
    }
};
struct RowsX {                  // x-contiguous: row k of p, ld apart, optionally picked through a list
    static constexpr bool KC = false;
    const float *__restrict__ p; int64_t ld; const int32_t *__restrict__ idx; int64_t gstride;
    struct Cur { const float *q; };
    __device__ __forceinline__ void bind(int32_t g) { p += g * gstride; }
    __device__ __forceinline__ void start(Cur &c, int32_t x) const { c.q = p + x; }
    __device__ __forceinline__ int32_t row(int64_t k) const { return idx ? idx[k] : (int32_t)k; }
    __device__ __forceinline__ const float *at(const Cur &c, int32_t row) const { return c.q + row * ld; }
    __device__ __forceinline__ float el(int64_t x, int64_t k) const { return p[row(k) * ld + x]; }
};
struct XcatX {                  // x-contiguous: row k of [dP | G]
    static constexpr bool KC = false;
    const float *dP, *G; int32_t d_out, bd;
    struct Cur { const float *q; int32_t ld; };
    __device__ __forceinline__ void bind(int32_t) {}
    __device__ __forceinline__ void start(Cur &c, int32_t x) const { c.q = x < bd ? dP + x : G + (x - bd); c.ld = x < bd ? bd : d_out; }
    __device__ __forceinline__ int32_t row(int64_t k) const { return (int32_t)k; }
    __device__ __forceinline__ const float *at(const Cur &c, int32_t row) const { return c.q + (int64_t)row * c.ld; }
    __device__ __forceinline__ float el(int64_t x, int64_t k) const { return x < bd ? dP[k * bd + x] : G[k * d_out + x - bd]; }
};
struct WcatX {                  // x-contiguous: row k of [V_1 .. V_B | W_0]
    static constexpr bool KC = false;
    const float *V, *W0; int32_t d_in, d_out, B;
    struct Cur { const float *q; };
    __device__ __forceinline__ void bind(int32_t) {}
    __device__ __forceinline__ void start(Cur &c, int32_t x) const
    {
        const int32_t b = x / d_out;
        c.q = (b < B ? V + (int64_t)b * d_in * d_out : W0) + (x - b * d_out);
    }
    __device__ __forceinline__ int32_t row(int64_t k) const { return (int32_t)k; }
    __device__ __forceinline__ const float *at(const Cur &c, int32_t row) const { return c.q + (int64_t)row * d_out; }
    __device__ __forceinline__ float el(int64_t x, int64_t k) const
    {
        const int64_t b = x / d_out;
        return (b < B ? V + b * d_in * d_out : W0)[k * d_out + x - b * d_out];
    }
};

// ---- outputs: column n's address in row 0 and its row pitch; bind(g) selects the group of a grouped launch
struct EpiProject {             // columns < B*d_out go to P, the rest to Self
    float *P, *Self; int32_t d_out, bd;
    __device__ __forceinline__ void bind(int32_t, bool) {}
    __device__ __forceinline__ float *column(int32_t n, int64_t &ld) const { ld = n < bd ? bd : d_out; return n < bd ? P + n : Self + (n - bd); }
    __device__ __forceinline__ void put(float *q, float v) const { *q = v; }
};
struct EpiWeightGrad {          // atomic accumulation of split-K partial tiles
    float *dV, *dW0; int32_t d_in, d_out, B;
    __device__ __forceinline__ void bind(int32_t, bool) {}
    __device__ __forceinline__ float *column(int32_t n, int64_t &ld) const
    {
        const int32_t b = n / d_out;
        ld = d_out;
        return (b < B ? dV + (int64_t)b * d_in * d_out : dW0) + (n - b * d_out);
    }
    __device__ __forceinline__ void put(float *q, float v) const { unsafeAtomicAdd(q, v); }
};
struct EpiRows {                // streamed out: the next kernel reads it once
    float *out; int64_t cols;
    __device__ __forceinline__ void bind(int32_t, bool) {}
    __device__ __forceinline__ float *column(int32_t n, int64_t &ld) const { ld = cols; return out + n; }
    __device__ __forceinline__ void put(float *q, float v) const { __builtin_nontemporal_store(v, q); }
};
struct EpiRowsAtomic {          // split-K partial tiles; one matrix per group, gstride apart; a group's only part is stored
    float *out; int64_t cols, gstride; bool sole;
    __device__ __forceinline__ void bind(int32_t g, bool only) { out += g * gstride; sole = only; }
    __device__ __forceinline__ float *column(int32_t n, int64_t &ld) const { ld = cols; return out + n; }
    __device__ __forceinline__ void put(float *q, float v) const { if (sole) *q = v; else unsafeAtomicAdd(q, v); }
};

// A launch is (row tiles) x (column tiles) x (splits) blocks in one dimension.  Row tile x holds rows x * BM.. or, with
// a tile list (mt_beg non-null), rows [mt_beg[x], mt_end[x]) of group mt_id[x] (at most BM rows): A and the output are
// cut at the tile's end, B is the group's matrix.  The contraction range of split z is [z*kchunk, min((z+1)*kchunk, K)),
// or, in a grouped launch (g_beg non-null), [g_beg[z], g_end[z]) with the epilogue bound to group g_id[z].
struct GemmGrid {
    int32_t tiles_m, tiles_n, splits;
    int64_t K, kchunk;
    const int32_t *g_id, *g_beg, *g_end, *mt_id, *mt_beg, *mt_end;
};
__host__ __device__ __forceinline__ bool gemm_by_cols(const GemmGrid &g)
{
    return g.splits <= 1 && !g.g_beg && !g.mt_beg && g.tiles_m < 8 && g.tiles_n > g.tiles_m;
}

// C (+)= A B^T, A (M x K), B (N x K).
// Steps of 16 k: a step's operands are split into LDS ([part][row][k]) one step ahead of their use, their loads are issued
// two steps further ahead into registers (two sets, used in turn; past the range's end the last step is loaded again, so
// that nothing in the loop is conditional and the waits for one set leave the other in flight).  Two LDS buffers, one
// barrier per step; 74 KB, two blocks per compute unit.
// A wavefront leaves out the 32-wide parts of its sub-tile that lie past the operands' ends (width 200 is 7 such parts,
// not 8; a relation with 30 runs one of 4).
// What the matrix cores cut off when they add products to a larger sum is cut off downwards, whatever the signs: over
// thousands of steps and blocks it adds up (3e-6 in the weight gradients of 5.8 M rows, where fp32 steps give 1e-6).
// Every FLUSH steps (half of a short contraction's) the sums therefore move to a second set by an ordinary addition and
// start again from zero, and every other such group is formed with A negated and subtracted, so that what is cut off
// cancels.
// What bounds it: with rows of 128 floats the bytes moved (60 M edges, 5.8 M runs: a layer's six products take 7.0 ms at
// about 4 TB/s; with fp32 matrix-core steps they took 8.6); with wider rows what a wavefront issues around the
// matrix-core steps (splitting, addresses, the sums' moves: 9 vector instructions for each, where up to 6 would hide).
// 352 k runs of 474 relations at width 200, microseconds with fp32 steps / now: rel_outer 570 / 335, apply_rel 427 /
// 319, apply_rel_t 406 / 270; against fp64 the gradients are off by 3e-7 there, 5e-7 before.
struct GemmLds { unsigned char buf[2][6 * PLANE]; };                              // [buffer][A's parts, B's parts]

template <class SA, class SB, class EPI>
__device__ __forceinline__ void gemm_tile(GemmLds &shared, uint32_t block, SA A, SB B, EPI epi, int32_t M_, int32_t N_, const GemmGrid &g)
{
    auto &lds = shared.buf;
    const int t = threadIdx.x, lane = t & 63, half = lane >> 5;
    const int w = __builtin_amdgcn_readfirstlane(t >> 6), wm = w >> 1, wn = w & 1;
    // block id -> (row tile, column tile, split).  Workgroup i runs on XCD i % 8: the tiles that read the same rows of
    // a long operand (the column tiles of a row tile; all tiles of a split) run on one XCD one after another, and the
    // rows come from its L2 all but once.  With fewer row tiles than XCDs the column tiles go round them instead.
    const bool by_split = g.splits > 1 || g.g_beg, by_cols = gemm_by_cols(g);
    const int32_t per = by_split ? g.tiles_m * g.tiles_n : by_cols ? g.tiles_m : g.tiles_n;
    const int32_t slot = block / 8, unit = slot / per * 8 + block % 8, in_unit = slot % per;
    const int32_t tn = by_cols ? unit : in_unit % g.tiles_n, sp = by_split ? unit : 0;
    const int32_t tm = by_split ? in_unit / g.tiles_n : by_cols ? in_unit : unit;
    if (tm >= g.tiles_m || tn >= g.tiles_n || sp >= g.splits) return;       // padding blocks of the last units
    int64_t m0 = (int64_t)tm * BM, m_end = M_;
    if (g.mt_beg) { m0 = g.mt_beg[tm]; m_end = g.mt_end[tm]; B.bind(g.mt_id[tm]); }
    const int32_t n0 = tn * BN;
    int64_t kbeg = sp * g.kchunk;
    int64_t kend = (kbeg + g.kchunk < g.K) ? kbeg + g.kchunk : g.K;
    if (g.g_beg) {
        kbeg = g.g_beg[sp];
        kend = g.g_end[sp];
        const int32_t id = g.g_id[sp];
        epi.bind(id, (sp == 0 || g.g_id[sp - 1] != id) && (sp + 1 == g.splits || g.g_id[sp + 1] != id));
    }
    if (kbeg >= kend) return;
    const int64_t klast = kbeg + (kend - 1 - kbeg) / BK * BK;         // the last step's first k

    // ---- global -> registers -> LDS.  k-contiguous operands: 4 lanes share a row's 16 k, a thread takes two rows 64
    // apart.  x-contiguous operands: a wavefront takes 4 consecutive k, a lane 2 columns of each, so that a lane ends
    // up with runs of 4 k as the matrix cores want them (one column and 8 k per lane: twice the loads, 20 % slower).
    // Rows, columns and k past the operands' ends repeat the last ones; such rows only feed results that are dropped,
    // such k are zeroed on the way into LDS.
    typename SA::Cur ca;
    typename SB::Cur cb;
    int32_t rowa[2][4], rowb[2][4];      // by the parity of the step they belong to
    auto pick = [&](auto &S, int32_t (&row)[4], int64_t k0) __attribute__((always_inline)) {
        if constexpr (!std::decay_t<decltype(S)>::KC) {
#pragma unroll
            for (int q = 0; q < 4; ++q) { const int64_t k = k0 + w * 4 + q; row[q] = S.row(k < kend ? k : kend - 1); }
        }
    };
    auto start = [&](auto &S, auto &c, int64_t x0, int64_t x_last) __attribute__((always_inline)) {
        if constexpr (std::decay_t<decltype(S)>::KC) {
#pragma unroll
            for (int ps = 0; ps < 2; ++ps) {
                const int64_t x = x0 + (t >> 2) + ps * 64;
                S.start(c, ps, x < x_last ? x : x_last);
            }
        } else {
            const int32_t x = (int32_t)x0 + lane * 2;
            S.start(c, x < (int32_t)x_last ? x : (int32_t)x_last - 1);
        }
    };
    auto load = [&](auto &S, auto &c, const int32_t (&row)[4], float4 (&r)[2], int64_t k0) __attribute__((always_inline)) {
        if constexpr (std::decay_t<decltype(S)>::KC) {
            int32_t k = (int32_t)k0 + (t & 3) * 4;
            if (k > (int32_t)kend - 4) k = (int32_t)kend - 4;
#pragma unroll
            for (int ps = 0; ps < 2; ++ps) r[ps] = *reinterpret_cast<const float4 *>(S.at(c, ps, k));
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float2 v = *reinterpret_cast<const float2 *>(S.at(c, row[q]));
                if (q & 1) { r[q >> 1].z = v.x; r[q >> 1].w = v.y; }
                else { r[q >> 1].x = v.x; r[q >> 1].y = v.y; }
            }
        }
    };
    auto stage = [&](auto &S, unsigned char *L, const float4 (&r)[2], int64_t k0, float sign) __attribute__((always_inline)) {
        if constexpr (std::decay_t<decltype(S)>::KC) {
            const float on = k0 + (t & 3) * 4 < kend ? sign : 0.f;
#pragma unroll
            for (int ps = 0; ps < 2; ++ps) {
                const Split3 lo = split_pair(r[ps].x * on, r[ps].y * on), hi = split_pair(r[ps].z * on, r[ps].w * on);
#pragma unroll
                for (int p = 0; p < 3; ++p)
                    *reinterpret_cast<uint2 *>(L + p * PLANE + ((t >> 2) + ps * 64) * LP + (t & 3) * 8) = make_uint2(lo.w[p], hi.w[p]);
            }
        } else {
            const int64_t left = kend - k0 - w * 4;         // of this wavefront's 4 k
            const float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
            float4 u = r[0], v = r[1];
            if (left < 4) {
                if (left < 1) u = z; else if (left < 2) { u.z = 0.f; u.w = 0.f; }
                if (left < 3) v = z; else { v.z = 0.f; v.w = 0.f; }
            }
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const Split3 lo = c ? split_pair(u.y * sign, u.w * sign) : split_pair(u.x * sign, u.z * sign);
                const Split3 hi = c ? split_pair(v.y * sign, v.w * sign) : split_pair(v.x * sign, v.z * sign);
#pragma unroll
                for (int p = 0; p < 3; ++p)
                    *reinterpret_cast<uint2 *>(L + p * PLANE + (lane * 2 + c) * LP + w * 8) = make_uint2(lo.w[p], hi.w[p]);
            }
        }
    };
    auto at_most = [&](int64_t k) { return k < klast ? k : klast; };
    float4 ra[2][2], rb[2][2];
    // step number j's loads; its rows were picked with step j - 1's, ahead of those loads: a wavefront's memory operations
    // retire in order, and waiting for an index behind them would wait for them too
    auto load_step = [&](int par, int64_t k0) __attribute__((always_inline)) {
        pick(A, rowa[par ^ 1], at_most(k0 + BK));
        pick(B, rowb[par ^ 1], at_most(k0 + BK));
        load(A, ca, rowa[par], ra[par], at_most(k0));
        load(B, cb, rowb[par], rb[par], at_most(k0));
    };
    start(A, ca, m0, m_end - 1);
    start(B, cb, n0, N_ - 1);
    pick(A, rowa[0], kbeg);
    pick(B, rowb[0], kbeg);
    load_step(0, kbeg);
    load_step(1, kbeg + BK);
    stage(A, lds[0], ra[0], kbeg, 1.f);
    stage(B, lds[0] + 3 * PLANE, rb[0], kbeg, 1.f);
    load_step(0, kbeg + 2 * BK);
    __syncthreads();

    const int off_a = (wm * 64 + (lane & 31)) * LP + half * 16, off_b = 3 * PLANE + (wn * 64 + (lane & 31)) * LP + half * 16;
    split_floatx16 tot[2][2], acc[2][2];
    const int64_t n_steps = (kend - kbeg + BK - 1) / BK;
    const int group = n_steps <= 2 * FLUSH ? (int)(n_steps + 1) / 2 : FLUSH;      // steps per group, two groups at least
    // NI, NJ: 32-wide parts of this wavefront's sub-tile that hold rows (columns) of the output
    auto contract = [&](auto ni, auto nj) __attribute__((always_inline)) {
        constexpr int NI = decltype(ni)::value, NJ = decltype(nj)::value;
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) { tot[i][j][v] = 0.f; acc[i][j][v] = 0.f; }
        auto step = [&](int64_t k0, int cur, float next_sign) __attribute__((always_inline)) {
            const unsigned char *L = lds[cur];
            uint4 a[2][3], b[2][3];
#pragma unroll
            for (int p = 0; p < 3; ++p) {
#pragma unroll
                for (int i = 0; i < NI; ++i) a[i][p] = *reinterpret_cast<const uint4 *>(L + off_a + p * PLANE + i * 32 * LP);
#pragma unroll
                for (int j = 0; j < NJ; ++j) b[j][p] = *reinterpret_cast<const uint4 *>(L + off_b + p * PLANE + j * 32 * LP);
            }
            stage(A, lds[cur ^ 1], ra[cur ^ 1], k0 + BK, next_sign);
            stage(B, lds[cur ^ 1] + 3 * PLANE, rb[cur ^ 1], k0 + BK, 1.f);
            load_step(cur ^ 1, k0 + 3 * BK);
#pragma unroll
            for (int p = 0; p < SPLIT_TERMS; ++p)
#pragma unroll
                for (int i = 0; i < NI; ++i)
#pragma unroll
                    for (int j = 0; j < NJ; ++j) acc[i][j] = split_mfma(a[i][split_pa(p)], b[j][split_pb(p)], acc[i][j]);
            __syncthreads();
        };
        float sign = 1.f;
        auto flush = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < NI; ++i)
#pragma unroll
                for (int j = 0; j < NJ; ++j)
#pragma unroll
                    for (int v = 0; v < 16; ++v) { tot[i][j][v] = fmaf(sign, acc[i][j][v], tot[i][j][v]); acc[i][j][v] = 0.f; }
        };
        int left = group;
        auto one = [&](int64_t k0, int cur) __attribute__((always_inline)) {
            step(k0, cur, left == 1 ? -sign : sign);
            if (--left == 0) { flush(); left = group; sign = -sign; }
        };
        int64_t k0 = kbeg;
        for (; k0 + BK < kend; k0 += 2 * BK) {
            one(k0, 0);
            one(k0 + BK, 1);
        }
        if (k0 < kend) one(k0, 0);
        if (left != group) flush();
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    const int64_t m_left = m_end - m0 - wm * 64;
    const int32_t n_left = N_ - n0 - wn * 64;
    const int mi = m_left > 32 ? 2 : m_left > 0 ? 1 : 0, nj = n_left > 32 ? 2 : n_left > 0 ? 1 : 0;
    if (mi == 0 || nj == 0) contract(I0{}, I0{});        // every wavefront moves operands and meets the barriers
    else if (mi == 2 && nj == 2) contract(I2{}, I2{});
    else if (mi == 2) contract(I2{}, I1{});
    else if (nj == 2) contract(I1{}, I2{});
    else contract(I1{}, I1{});

    // ---- epilogue.  D register v of lane l is row 8*(v/4) + 4*(l/32) + v%4, column l%32.
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            if (i >= mi || j >= nj) continue;
            const int64_t mb = m0 + wm * 64 + i * 32;
            const int32_t n = n0 + wn * 64 + j * 32 + (lane & 31);
            bool odd = false;
#pragma unroll
            for (int v = 0; v < 16; ++v) odd |= split_not_finite(tot[i][j][v]);
            if (__any(odd)) {        // an infinity, a NaN or an overflow among the terms: these sums again, in fp32
                split_floatx16 f;
#pragma unroll
                for (int v = 0; v < 16; ++v) f[v] = 0.f;
                const int64_t m = mb + (lane & 31);
                for (int64_t k = kbeg + half; k - half < kend; k += 2) {
                    const float x = m < m_end && k < kend ? A.el(m, k) : 0.f, y = n < N_ && k < kend ? B.el(n, k) : 0.f;
                    f = __builtin_amdgcn_mfma_f32_32x32x2f32(x, y, f, 0, 0, 0);
                }
#pragma unroll
                for (int v = 0; v < 16; ++v) if (split_not_finite(tot[i][j][v])) tot[i][j][v] = f[v];
            }
            if (n >= N_) continue;
            int64_t ld;
            float *q = epi.column(n, ld);
            q += (mb + 4 * half) * ld;
            if (mb + 32 <= m_end) {
#pragma unroll
                for (int v = 0; v < 16; ++v) epi.put(q + (8 * (v >> 2) + (v & 3)) * ld, tot[i][j][v]);
            } else {
                const int32_t left = (int32_t)(m_end - mb) - 4 * half;
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    if (8 * (v >> 2) + (v & 3) < left) epi.put(q + (8 * (v >> 2) + (v & 3)) * ld, tot[i][j][v]);
            }
        }
}

template <class SA, class SB, class EPI>
__global__ __launch_bounds__(GT, 2) void k_gemm(SA A, SB B, EPI epi, int32_t M_, int32_t N_, GemmGrid g)
{
    __shared__ __attribute__((aligned(16))) GemmLds lds;
    gemm_tile(lds, blockIdx.x, A, B, epi, M_, N_, g);
}

// a product and its blocks: row tiles x column tiles x splits, numbered as gemm_tile reads them (a multiple of 8, so that
// several products behind one another keep their tiles on the XCDs that the numbers name)
template <class SA, class SB, class EPI>
struct GemmJob { SA a; SB b; EPI e; int32_t M, N; GemmGrid g; uint32_t blocks; };

template <class SA, class SB, class EPI>
int gemm_job(const SA &sa, const SB &sb, const EPI &ep, int64_t rows, int32_t cols, GemmGrid g, GemmJob<SA, SB, EPI> *job)
{
    if (!g.mt_beg) g.tiles_m = (int32_t)cdiv(rows, BM);
    g.tiles_n = (int32_t)cdiv(cols, BN);
    const bool by_split = g.splits > 1 || g.g_beg;
    const bool by_cols = gemm_by_cols(g);
    const int64_t per = by_split ? (int64_t)g.tiles_m * g.tiles_n : by_cols ? g.tiles_m : g.tiles_n;
    const int64_t units = by_split ? g.splits : by_cols ? g.tiles_n : g.tiles_m;
    const int64_t blocks = g.splits == 0 ? 0 : cdiv(units, 8) * 8 * per;     // no splits: nothing to sum, as in a graph without edges
    KGE_REQUIRE(rows <= 0x7fffffffLL && blocks <= 0x7fffffffLL, KGE_ERANGE, "too many tiles for one launch");
    *job = GemmJob<SA, SB, EPI>{sa, sb, ep, (int32_t)rows, cols, g, (uint32_t)blocks};
    return KGE_OK;
}

template <class SA, class SB, class EPI>
int run_job(const GemmJob<SA, SB, EPI> &j, hipStream_t st)
{
    k_gemm<SA, SB, EPI><<<j.blocks, GT, 0, st>>>(j.a, j.b, j.e, j.M, j.N, j.g);
    KGE_LAUNCH_CHECK();
    return KGE_OK;
}

template <class SA, class SB, class EPI>
int run_gemm(const SA &sa, const SB &sb, const EPI &ep, int64_t rows, int32_t cols, GemmGrid g, hipStream_t st)
{
    GemmJob<SA, SB, EPI> job;
    int rc = gemm_job(sa, sb, ep, rows, cols, g, &job);
    return rc != KGE_OK ? rc : run_job(job, st);
}

// Several products that do not depend on one another in one launch, one behind the other: the blocks of the next start as
// those of the one before run out.  In a small graph each product fills a part of the chip for the 7 to 10 us that its few
// steps take, most of them latency; in a large one the last wave of a launch leaves compute units idle.  Microseconds of a
// training step's layers with a launch for each product / with two launches in all: 1000 vertices, 10 relations, 5000 edges,
// width 32: 197 / 146; 14541 vertices, 237 relations, 272 k edges, width 200: 3194 / 3015, width 64: 1132 / 1038; 40000, 200
// relations, width 256: 5025 / 4806; one layer over 200 k vertices, 2 relations, 2 M edges, width 64: 1097 / 1024; 100 k, 237
// relations, 1 M edges, width 200: 4484 / 4422; 300 k, 1000 relations, 3 M edges, width 64: 3464 / 3356.  No size tried lost.
template <class... JOBS>
__global__ __launch_bounds__(GT, 2) void k_gemm_jobs(JOBS... jobs)
{
    __shared__ __attribute__((aligned(16))) GemmLds lds;
    uint32_t block = blockIdx.x;
    auto one = [&](const auto &j) __attribute__((always_inline)) {
        if (block >= j.blocks) { block -= j.blocks; return false; }
        gemm_tile(lds, block, j.a, j.b, j.e, j.M, j.N, j.g);
        return true;
    };
    (void)(one(jobs) || ...);
}
template <class... JOBS> int run_jobs(hipStream_t st, const JOBS &...jobs)
{
    const int64_t blocks = (int64_t(0) + ... + jobs.blocks);
    if (blocks == 0) return KGE_OK;
    KGE_REQUIRE(blocks <= 0x7fffffffLL, KGE_ERANGE, "too many tiles for one launch");
    k_gemm_jobs<JOBS...><<<(uint32_t)blocks, GT, 0, st>>>(jobs...);
    KGE_LAUNCH_CHECK();
    return KGE_OK;
}

__global__ void k_zero16(float4 *p, int64_t n4)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (; i < n4; i += stride) p[i] = make_float4(0.f, 0.f, 0.f, 0.f);
}

__global__ void k_zero4(uint32_t *p, int64_t n)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) p[i] = 0u;
}

struct ZeroSpans { uint32_t *p[4]; int64_t first[5]; };      // span k: words [first[k], first[k + 1]) of the whole

__global__ __launch_bounds__(256) void k_zero_spans(ZeroSpans s)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < s.first[4]; i += stride) {
        const int k = i < s.first[1] ? 0 : i < s.first[2] ? 1 : i < s.first[3] ? 2 : 3;
        s.p[k][i - s.first[k]] = 0u;
    }
}

}  // namespace

// Several small buffers in one launch (a launch and its gap cost 5 us, the fills of a small graph a fraction of that); a
// big one among them gets a launch of its own with 16-byte stores.
int launch_fill_zero_spans(const kge_span *spans, int n, hipStream_t st)
{
    KGE_REQUIRE(n >= 0 && n <= 4, KGE_EINVAL, "at most four buffers");
    ZeroSpans z{};
    int64_t words = 0;
    for (int k = 0; k < 4; ++k) {
        z.first[k] = words;
        if (k >= n || spans[k].bytes == 0) continue;
        KGE_REQUIRE(((uintptr_t)spans[k].ptr % 4) == 0 && spans[k].bytes % 4 == 0, KGE_EINVAL,
                    "zero fill needs a 4-byte aligned buffer and size");
        if (spans[k].bytes > ((size_t)4 << 20)) {
            int rc = launch_fill_zero(spans[k].ptr, spans[k].bytes, st);
            if (rc != KGE_OK) return rc;
            continue;
        }
        z.p[k] = (uint32_t *)spans[k].ptr;
        words += (int64_t)(spans[k].bytes / 4);
    }
    z.first[4] = words;
    if (words == 0) return KGE_OK;
    KGE_PROF("zero", st);
    int64_t blocks = cdiv(words, 256);
    if (blocks > 2048) blocks = 2048;
    k_zero_spans<<<(unsigned)blocks, 256, 0, st>>>(z);
    KGE_LAUNCH_CHECK();
    return KGE_OK;
}

// Zero `bytes` bytes (a multiple of 4, 4-byte aligned) with a fill kernel; no memset nodes,
// so callers may capture the step in a HIP graph.
int launch_fill_zero(void *ptr, size_t bytes, hipStream_t st)
{
    if (bytes == 0) return KGE_OK;
    KGE_REQUIRE(((uintptr_t)ptr % 4) == 0 && bytes % 4 == 0, KGE_EINVAL,
                "zero fill needs a 4-byte aligned buffer and size");
    KGE_PROF("zero", st);
    if (((uintptr_t)ptr % 16) == 0 && bytes % 16 == 0) {
        int64_t n4 = (int64_t)(bytes / 16);
        int64_t blocks = cdiv(n4, 256);
        if (blocks > 65536) blocks = 65536;
        k_zero16<<<(unsigned)blocks, 256, 0, st>>>(reinterpret_cast<float4 *>(ptr), n4);
    } else {
        int64_t n = (int64_t)(bytes / 4);
        int64_t blocks = cdiv(n, 256);
        if (blocks > 65536) blocks = 65536;
        k_zero4<<<(unsigned)blocks, 256, 0, st>>>(reinterpret_cast<uint32_t *>(ptr), n);
    }
    KGE_LAUNCH_CHECK();
    return KGE_OK;
}

namespace {
using ProjectJob = GemmJob<RowsK, WcatX, EpiProject>;
using WeightGradJob = GemmJob<RowsX, XcatX, EpiWeightGrad>;
using InputGradJob = GemmJob<XcatK, WcatK, EpiRows>;
using RelOuterJob = GemmJob<RowsX, RowsX, EpiRowsAtomic>;
using ApplyJob = GemmJob<RowsK, RowsX, EpiRows>;
using ApplyTJob = GemmJob<RowsK, RowsK, EpiRows>;

int project_job(const float *H, int64_t N, int32_t d_in, int32_t d_out, int32_t B, const float *V, const float *W0, float *P,
                float *Self, ProjectJob *job)
{
    return gemm_job(RowsK{H, d_in, nullptr, 0}, WcatX{V, W0, d_in, d_out, B}, EpiProject{P, Self, d_out, B * d_out}, N,
                    (B + 1) * d_out, GemmGrid{0, 0, 1, d_in, d_in}, job);
}
int weight_grad_job(const float *H, int64_t N, int32_t d_in, int32_t d_out, int32_t B, const float *dP, const float *G, float *dV,
                    float *dW0, WeightGradJob *job)
{
    int32_t nc = (B + 1) * d_out;
    int64_t tiles = cdiv(d_in, BM) * cdiv(nc, BN);
    // split the N-long contraction so that roughly 2048 blocks are in flight
    int64_t splits = cdiv(2048, tiles);
    int64_t kchunk = cdiv(cdiv(N, splits), BK) * BK;
    if (kchunk < 4 * BK) kchunk = 4 * BK;
    splits = cdiv(N, kchunk);
    return gemm_job(RowsX{H, d_in, nullptr, 0}, XcatX{dP, G, d_out, B * d_out}, EpiWeightGrad{dV, dW0, d_in, d_out, B}, d_in, nc,
                    GemmGrid{0, 0, (int32_t)splits, N, kchunk}, job);
}
int input_grad_job(const float *dP, const float *G, int64_t N, int32_t d_in, int32_t d_out, int32_t B, const float *V, const float *W0,
                   float *dH, InputGradJob *job)
{
    int32_t nc = (B + 1) * d_out;
    return gemm_job(XcatK{dP, G, d_out, B * d_out}, WcatK{V, W0, d_in, d_out, B}, EpiRows{dH, d_in}, N, d_in,
                    GemmGrid{0, 0, 1, nc, nc}, job);
}
int rel_outer_job(const kge_partition *p, const float *Z, const float *G, int32_t d_in, int32_t d_out, float *C, RelOuterJob *job)
{
    return gemm_job(RowsX{Z, d_in, nullptr, 0}, RowsX{G, d_out, p->seg_dst, 0}, EpiRowsAtomic{C, d_out, (int64_t)d_in * d_out, false},
                    d_in, d_out, GemmGrid{0, 0, p->n_relc, p->n_seg, 0, p->relc_rel, p->relc_beg, p->relc_end}, job);
}
// the row tiles of the per-run products: <= 128 consecutive runs of one relation each
GemmGrid rel_tiles(const kge_partition *p, int32_t K)
{
    return GemmGrid{p->n_relt, 0, 1, K, K, nullptr, nullptr, nullptr, p->relt_rel, p->relt_beg, p->relt_end};
}
int apply_job(const kge_partition *p, const float *Z, const float *Wrel, int32_t d_in, int32_t d_out, float *U, ApplyJob *job)
{
    return gemm_job(RowsK{Z, d_in, nullptr, 0}, RowsX{Wrel, d_out, nullptr, (int64_t)d_in * d_out}, EpiRows{U, d_out}, p->n_seg, d_out,
                    rel_tiles(p, d_in), job);
}
int apply_t_job(const kge_partition *p, const float *G, const float *Wrel, int32_t d_in, int32_t d_out, float *dZ, ApplyTJob *job)
{
    return gemm_job(RowsK{G, d_out, p->seg_dst, 0}, RowsK{Wrel, d_out, nullptr, (int64_t)d_in * d_out}, EpiRows{dZ, d_in}, p->n_seg, d_in,
                    rel_tiles(p, d_out), job);
}
}  // namespace

int launch_project(const float *H, int64_t N, int32_t d_in, int32_t d_out, int32_t B, const float *V,
                   const float *W0, float *P, float *Self, hipStream_t st)
{
    if (N == 0) return KGE_OK;
    KGE_PROF("project", st);
    ProjectJob job;
    int rc = project_job(H, N, d_in, d_out, B, V, W0, P, Self, &job);
    return rc != KGE_OK ? rc : run_job(job, st);
}

int launch_weight_grad(const float *H, int64_t N, int32_t d_in, int32_t d_out, int32_t B,
                       const float *dP, const float *G, float *dV, float *dW0, hipStream_t st)
{
    if (N == 0) return KGE_OK;
    KGE_PROF("weight_grad", st);
    WeightGradJob job;
    int rc = weight_grad_job(H, N, d_in, d_out, B, dP, G, dV, dW0, &job);
    return rc != KGE_OK ? rc : run_job(job, st);
}

int launch_input_grad(const float *dP, const float *G, int64_t N, int32_t d_in,
                      int32_t d_out, int32_t B, const float *V, const float *W0, float *dH,
                      hipStream_t st)
{
    if (N == 0) return KGE_OK;
    KGE_PROF("input_grad", st);
    InputGradJob job;
    int rc = input_grad_job(dP, G, N, d_in, d_out, B, V, W0, dH, &job);
    return rc != KGE_OK ? rc : run_job(job, st);
}

int launch_coeff_contract(const kge_partition *p, const float *C, const float *V, int32_t d_in, int32_t d_out,
                          int32_t B, float *da, hipStream_t st)
{
    const int64_t R2 = 2 * (int64_t)p->n_relations;
    const int64_t dd = (int64_t)d_in * d_out;
    if (p->n_seg == 0) return KGE_OK;
    {
        const int64_t tiles = cdiv(R2, BM) * cdiv(B, BN);
        int64_t splits = cdiv(512, tiles);
        int64_t kchunk = cdiv(cdiv(dd, splits), BK) * BK;
        if (kchunk < 4 * BK) kchunk = 4 * BK;
        splits = cdiv(dd, kchunk);
        RowsK sa{C, dd, nullptr, 0};
        RowsK sb{V, dd, nullptr, 0};
        EpiRowsAtomic ep{da, B, 0, false};
        KGE_PROF("coeff_contract", st);
        return run_gemm(sa, sb, ep, R2, B, GemmGrid{0, 0, (int32_t)splits, dd, kchunk}, st);
    }
}

// ---- relation-weight order ------------------------------------------------------------------
namespace {

// out[i][x] = sum_k c[i][k] M[k][x]   (c is [ni][nk])
// One block: 16 rows i, 1024 columns x (4 per thread); M is read once per 16 rows.
__global__ __launch_bounds__(256) void k_lincomb(const float *__restrict__ c, int32_t ni, int32_t nk,
                                                 const float *__restrict__ M, int64_t nx, float *__restrict__ out)
{
    __shared__ float sc[16][64];
    const int i0 = blockIdx.y * 16;
    const int64_t x = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
    float4 acc[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) acc[j] = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int k0 = 0; k0 < nk; k0 += 64) {
        __syncthreads();
        for (int q = threadIdx.x; q < 16 * 64; q += 256) {
            const int j = q >> 6, kk = q & 63;
            const int i = i0 + j, k = k0 + kk;
            sc[j][kk] = (i < ni && k < nk) ? c[(int64_t)i * nk + k] : 0.f;
        }
        __syncthreads();
        const int kn = min(64, nk - k0);
        if (x < nx)
            for (int kk = 0; kk < kn; ++kk) {
                const float4 m = *reinterpret_cast<const float4 *>(M + (int64_t)(k0 + kk) * nx + x);
#pragma unroll
                for (int j = 0; j < 16; ++j) {
                    const float w = sc[j][kk];
                    acc[j].x = fmaf(w, m.x, acc[j].x); acc[j].y = fmaf(w, m.y, acc[j].y);
                    acc[j].z = fmaf(w, m.z, acc[j].z); acc[j].w = fmaf(w, m.w, acc[j].w);
                }
            }
    }
    if (x < nx)
#pragma unroll
        for (int j = 0; j < 16; ++j)
            if (i0 + j < ni) *reinterpret_cast<float4 *>(out + (int64_t)(i0 + j) * nx + x) = acc[j];
}

}  // namespace

// Wrel[r] = sum_b a[r][b] V_b   ([2R][d_in*d_out] floats): Eq. 2 written out for every relation
int launch_relation_weights(const float *a, int32_t R2, int32_t B, const float *V, int64_t dd, float *Wrel,
                            hipStream_t st)
{
    if (R2 == 0) return KGE_OK;
    dim3 grid((unsigned)cdiv(dd, 1024), (unsigned)cdiv(R2, 16), 1);
    KGE_PROF("rel_weights", st);
    k_lincomb<<<grid, 256, 0, st>>>(a, R2, B, V, dd, Wrel);
    KGE_LAUNCH_CHECK();
    return KGE_OK;
}

namespace {

// dV[b][x] += sum_{r in this block's chunk} a[r][b] C[r][x] for BB bases b at once: the block's 256 columns of C
// are read once for all of them (C, one matrix per relation, is the big operand).  A row's BB coefficients are
// uniform over the block and contiguous: they arrive through scalar loads and enter the multiply-adds as scalar
// operands.
template <int BB>
__global__ __launch_bounds__(256) void k_basis_grad_cols(const float *__restrict__ a, int32_t R2, int32_t B,
                                                         int32_t b_base, const float *__restrict__ C, int64_t nx,
                                                         int32_t rchunk, float *__restrict__ dV)
{
    const int64_t x = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int b0 = b_base + blockIdx.z * BB;
    const int rb = blockIdx.y * rchunk, re = min(rb + rchunk, R2);
    const bool in = x < nx;
    const float *cp = C + (in ? x : 0);
    float acc[BB];
#pragma unroll
    for (int j = 0; j < BB; ++j) acc[j] = 0.f;
    int r = rb;
    for (; r + 4 <= re; r += 4) {
        float c[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) c[u] = cp[(int64_t)(r + u) * nx];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const float *ar = a + (int64_t)(r + u) * B + b0;
#pragma unroll
            for (int j = 0; j < BB; ++j) acc[j] = fmaf(ar[j], c[u], acc[j]);
        }
    }
    for (; r < re; ++r) {
        const float c = cp[(int64_t)r * nx];
        const float *ar = a + (int64_t)r * B + b0;
#pragma unroll
        for (int j = 0; j < BB; ++j) acc[j] = fmaf(ar[j], c, acc[j]);
    }
    if (in)
#pragma unroll
        for (int j = 0; j < BB; ++j) atomicAdd(dV + (int64_t)(b0 + j) * nx + x, acc[j]);
}

template <int BB>
int basis_grad_groups(const float *a, int32_t R2, int32_t B, int32_t &b_done, const float *C, int64_t dd, float *dV,
                      hipStream_t st)
{
    const int64_t zb = (B - b_done) / BB;
    if (zb == 0) return KGE_OK;
    // the sum over relations is cut into chunks so that about 1536 blocks run (six per compute unit are resident
    // at once: one round of blocks, no tail); their partial sums meet in dV
    const int64_t xb = cdiv(dd, 256);
    int64_t chunks = cdiv(1536, xb * zb);
    if (chunks > cdiv(R2, 16)) chunks = cdiv(R2, 16);
    const int32_t rchunk = (int32_t)cdiv(R2, chunks);
    KGE_REQUIRE(xb <= 0x7fffffffLL && zb <= 65535, KGE_ERANGE, "basis gradient: too many columns or bases");
    dim3 grid((unsigned)xb, (unsigned)cdiv(R2, rchunk), (unsigned)zb);
    k_basis_grad_cols<BB><<<grid, 256, 0, st>>>(a, R2, B, b_done, C, dd, rchunk, dV);
    KGE_LAUNCH_CHECK();
    b_done += (int32_t)zb * BB;
    return KGE_OK;
}

}  // namespace

// dV_b = sum_r a[r][b] C[r]   (the chain rule on Wrel[r] = sum_b a[r][b] V_b with dWrel = C)
// Many bases (multiples of 4 were measured; the operand loads take pairs of them, which have to be aligned as such) and
// columns: a product on the matrix cores, a^T C, that reads C once: 2000 relations x 65,536 columns with 64 bases 188 us,
// 359 on the vector units (whose multiply-adds bound it), with 20 bases 150, 197; 240 relations 33, 93 and 28, 43 (in a
// layer of 25 M runs, where C comes from memory: 64 bases 268, 445).  It needs one and a half tiles of 128 columns per
// compute unit: at 2000 x 50,176 with 32 bases 145, 154, but at 2000 x 40,000 145, 125.  Otherwise groups of 64, 16, 8,
// 4, 2 and 1 bases per block (10 bases as 8 + 2: 36 us at 474 x 40,000, 51 as 4 + 4 + 1 + 1).
int launch_basis_grad_from_relations(const float *a, int32_t R2, int32_t B, const float *C, int64_t dd, float *dV,
                                     hipStream_t st)
{
    if (R2 == 0 || B == 0) return KGE_OK;
    KGE_PROF("basis_grad", st);
    if (B >= 20 && B % 4 == 0 && dd >= 384 * BN && ((uintptr_t)a % 8) == 0) {
        RowsX sa{a, B, nullptr, 0};
        RowsX sb{C, dd, nullptr, 0};
        EpiRowsAtomic ep{dV, dd, 0, true};
        return run_gemm(sa, sb, ep, B, (int32_t)dd, GemmGrid{0, 0, 1, R2, R2}, st);
    }
    int32_t b_done = 0;
    int rc = basis_grad_groups<64>(a, R2, B, b_done, C, dd, dV, st);
    if (rc == KGE_OK) rc = basis_grad_groups<16>(a, R2, B, b_done, C, dd, dV, st);
    if (rc == KGE_OK) rc = basis_grad_groups<8>(a, R2, B, b_done, C, dd, dV, st);
    if (rc == KGE_OK) rc = basis_grad_groups<4>(a, R2, B, b_done, C, dd, dV, st);
    if (rc == KGE_OK) rc = basis_grad_groups<2>(a, R2, B, b_done, C, dd, dV, st);
    if (rc == KGE_OK) rc = basis_grad_groups<1>(a, R2, B, b_done, C, dd, dV, st);
    return rc;
}

// ---- a layer's products that do not depend on one another, in one launch
// U[s] = Z[s] Wrel[rel(s)] (one row tile per relation and <= 128 runs) and Self = H W_0
int launch_forward_products(const kge_partition *p, const float *Z, const float *Wrel, const float *H, const float *W0, int32_t d_in,
                            int32_t d_out, float *U, float *Self, hipStream_t st)
{
    KGE_PROF("fwd_products", st);
    ApplyJob apply;
    ProjectJob self;
    int rc = apply_job(p, Z, Wrel, d_in, d_out, U, &apply);
    if (rc == KGE_OK) rc = project_job(H, p->n_vert, d_in, d_out, 0, W0, W0, nullptr, Self, &self);
    return rc != KGE_OK ? rc : run_jobs(st, apply, self);
}

// C_r += sum of its runs' Z[s]^T G[dst(s)] and dW_0 += H^T G; with dZ also dZ[s] = G[dst(s)] Wrel[rel(s)]^T and Self = G W_0^T
int launch_backward_products(const kge_partition *p, const float *Z, const float *G, const float *Wrel, const float *H, const float *W0,
                             int32_t d_in, int32_t d_out, float *C, float *dW0, float *dZ, float *Self, hipStream_t st)
{
    KGE_PROF(dZ ? "bwd_products" : "outer_products", st);
    RelOuterJob outer;
    WeightGradJob weight;
    int rc = rel_outer_job(p, Z, G, d_in, d_out, C, &outer);
    if (rc == KGE_OK) rc = weight_grad_job(H, p->n_vert, d_in, d_out, 0, nullptr, G, nullptr, dW0, &weight);
    if (rc != KGE_OK) return rc;
    if (!dZ) return run_jobs(st, outer, weight);
    ApplyTJob apply;
    InputGradJob self;
    rc = apply_t_job(p, G, Wrel, d_in, d_out, dZ, &apply);
    if (rc == KGE_OK) rc = input_grad_job(nullptr, G, p->n_vert, d_in, d_out, 0, W0, W0, Self, &self);
    return rc != KGE_OK ? rc : run_jobs(st, outer, weight, apply, self);
}
