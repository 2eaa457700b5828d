// fp32 layers of 100 to 160 columns in the relation-weight order: rows times one matrix per group,
//
//   apply_rel     U[s]  = Z[s] W_{rel(s)}              groups: relations, rows: their runs
//   apply_rel_t   dZ[s] = G[dst(s)] W_{rel(s)}^T
//   project       Self  = H W_0                        one group
//   input_grad    dH    = G W_0^T
//
// on the fp16 matrix cores with two parts per number (split_f16.h) and all four products of them, those with a second part in
// sums of their own: a sum of K terms is then rounded K / 16 times where it matters.  A row is scaled by its own power of two,
// found when the block has the whole row in registers; a matrix by one of its own, found when k_pack_products splits it once
// for all row tiles, into the order in which a wavefront loads it.
// Second parts are kept 2^11 times as large, as large as the first ones, so that a number keeps both down to 2^-27 of the largest
// of its row or matrix.  One that is smaller still, and not zero, enters as a NaN: a sum may rest on such numbers alone (where the
// large ones meet zeros), and all sums that it reaches come from fp32 products, as those do that are not finite.
#include "common.h"
#include "split_f16.h"

#include <algorithm>

namespace {

constexpr int RT = 128;                       // rows of a tile (KGE_REL_TILE)
static_assert(RT == KGE_REL_TILE, "the partition's row tiles");
constexpr int NOT_OK = INT32_MIN;             // k_pack_products' exponent of a matrix that cannot be split

// Two parts of numbers below 2^15, the second one times 2^11; not zero, the numbers are at least SMALLEST: from there down the
// second part is below fp16's ordinary numbers
constexpr float SMALLEST = 1.220703125e-4f;    // 2^-13
__device__ __forceinline__ Split2 split_large(float x, float y)
{
    const split_floatx2 v = {x, y};
    const split_halfx2 a = __builtin_convertvector(v, split_halfx2);
    const split_floatx2 left = {__builtin_fmaf((float)a.x, -1.f, x) * 2048.f, __builtin_fmaf((float)a.y, -1.f, y) * 2048.f};
    Split2 s;
    s.w[0] = __builtin_bit_cast(uint32_t, a);
    s.w[1] = __builtin_bit_cast(uint32_t, __builtin_convertvector(left, split_halfx2));
    return s;
}
// second parts at their own size (what is lost of them here enters a product with another second part only)
__device__ __forceinline__ uint4 at_own_size(uint4 x)
{
    const _Float16 f = (_Float16)4.8828125e-4f;
    return __builtin_bit_cast(uint4, __builtin_bit_cast(split_halfx8, x) * split_halfx8{f, f, f, f, f, f, f, f});
}

// steps of 16 terms that a contraction is padded to: one kernel per class
constexpr int step_class(int32_t K) { return K <= 112 ? 7 : K <= 128 ? 8 : 10; }

// A matrix (K x N, row-major) as the two operands it is used as: `fwd` contracts over its rows k (columns n of the result),
// `back` over its columns n.  Operand block (c, s, part): 32 columns of the result from 32 c, terms 16 s .. 16 s + 15,
// 16 bytes per lane: column 32 c + l % 32, terms 16 s + 8 (l / 32) ..; zeros past either end.  Numbers are scaled so that the
// largest lies in 2^14 .. 2^15; info = the exponent by which a product with it is to be scaled back, or NOT_OK: a number
// that is not finite, or a largest one outside 2^-100 .. 2^100.
// One block of 16 wavefronts per matrix, the last group being W0.  Bound by the latency of its two passes: 10 to 18 us for
// three matrices of 128 x 32 and 128 x 128 (70 and 80 with a thread per column and 4 rows in flight).
__global__ __launch_bounds__(1024) void k_pack_products(const float *__restrict__ W, const float *__restrict__ W0, int32_t groups,
                                                        int32_t K, int32_t N, uint4 *__restrict__ fwd, uint4 *__restrict__ back,
                                                        int32_t ks_f, int32_t ks_b, int32_t *__restrict__ info)
{
    __shared__ uint32_t most_s;
    const int t = threadIdx.x, lane = t & 63, w = t >> 6, g = blockIdx.x;
    const float *M = g == groups - 1 ? W0 : W + (int64_t)g * K * N;
    if (t == 0) most_s = 0u;
    __syncthreads();
    const int col = lane * 4 < N ? lane * 4 : N - 4;         // N is a multiple of 4; lanes past the width repeat its end
    uint32_t most = 0u;
    for (int k0 = w; k0 < K; k0 += 16 * 8) {                 // a wavefront takes every 16th row, 8 in flight
        uint4 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = *reinterpret_cast<const uint4 *>(M + (int64_t)min(k0 + 16 * u, K - 1) * N + col);
#pragma unroll
        for (int u = 0; u < 8; ++u)
            most = max(most, max(max(v[u].x & 0x7fffffffu, v[u].y & 0x7fffffffu), max(v[u].z & 0x7fffffffu, v[u].w & 0x7fffffffu)));
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) most = max(most, (uint32_t)__shfl_xor((int)most, off, 64));
    if (lane == 0) atomicMax(&most_s, most);
    __syncthreads();
    const int e = (int)(most_s >> 23) - 127;
    const bool zero = most_s == 0u, ok = zero || abs(e) <= 100;
    if (t == 0) info[g] = !ok ? NOT_OK : zero ? 0 : e - 14;
    if (!ok) return;
    const float scale = zero ? 1.f : __uint_as_float((uint32_t)(127 + 14 - e) << 23);
    const int c_f = (N + 31) / 32, c_b = (K + 31) / 32;
    for (int which = 0; which < 2; ++which) {
        uint4 *out = which ? back : fwd;
        if (!out) continue;
        const int ks = which ? ks_b : ks_f, blocks = (which ? c_b : c_f) * ks;
        const int rows = which ? N : K, cols = which ? K : N;      // terms, columns of the result
        out += (int64_t)g * blocks * 128;
        for (int b = w; b < blocks; b += 16) {
            const int c = b / ks, s = b - c * ks, rc = c * 32 + (lane & 31), k = s * 16 + 8 * (lane >> 5);
            float x[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int kk = min(k + j, rows - 1), cc = min(rc, cols - 1);
                const float y = which ? M[(int64_t)cc * N + kk] : M[(int64_t)kk * N + cc];
                x[j] = y != 0.f && __builtin_fabsf(y * scale) < SMALLEST ? __builtin_nanf("") : y * scale;
                x[j] = k + j < rows && rc < cols ? x[j] : 0.f;
            }
            const Split2 p0 = split_large(x[0], x[1]), p1 = split_large(x[2], x[3]), p2 = split_large(x[4], x[5]), p3 = split_large(x[6], x[7]);
            out[(int64_t)b * 128 + lane] = make_uint4(p0.w[0], p1.w[0], p2.w[0], p3.w[0]);
            out[(int64_t)b * 128 + 64 + lane] = make_uint4(p0.w[1], p1.w[1], p2.w[1], p3.w[1]);
        }
    }
}

struct RowTiles { const int32_t *id, *beg, *end; int32_t n; int64_t rows; };     // id null: one group, 128 rows each

// A block of 8 wavefronts walks consecutive row tiles.  A tile's rows are loaded while the tile before it is multiplied, scaled
// and split into LDS in one piece ([part][row][k], an odd number of 16 bytes per row), and stay there; the matrix stays in
// operand registers for as long as its group's tiles last, so that no product waits for memory.  Wavefronts stand WN across
// the columns, 32 each, and share the rows (WN = 4: 64 each, 2 and 1: 32, those past the rows only load and split).
// Bound by the bytes of the rows.  5.3 M runs of 128 floats (a layer of 60 M edges): the four products 4.09 ms, 4.89 with six
// bf16 products per term in tiles of 128 x 128 x 16, whose operands are split once per column tile; 73 % of the rate of a
// copy.  With the matrix loaded for every tile, four steps ahead, behind the next tile's rows: 4.43.
template <int KS, int WN>
__global__ __launch_bounds__(512, 2) void k_row_products(const float *__restrict__ A, int64_t lda, const int32_t *__restrict__ aidx,
                                                         RowTiles tiles, int32_t K, int32_t N, const uint4 *__restrict__ pack,
                                                         const int32_t *__restrict__ info, const float *__restrict__ W,
                                                         int32_t w_k, int32_t w_n, float *__restrict__ out)
{
    static_assert(WN == 1 || WN == 2 || WN == 4, "the rows of a tile are covered");
    constexpr int WM = WN == 4 ? 2 : 4, RB = 4 / WM, NI = (KS * 4 + 7) / 8;
    constexpr int PITCH = KS * 32 + 16, PLANE = RT * PITCH;
    __shared__ __attribute__((aligned(16))) unsigned char lds[2 * PLANE];
    __shared__ __attribute__((aligned(16))) int32_t row_exp[RT];
    const int t = threadIdx.x, lane = t & 63, half = lane >> 5;
    const int w = __builtin_amdgcn_readfirstlane(t >> 6), wn = w % WN, wm = w / WN;
    const bool multiplies = wm < 4 / RB && wn * 32 < N;
    const int32_t t_beg = (int32_t)((int64_t)blockIdx.x * tiles.n / gridDim.x), t_end = (int32_t)((int64_t)(blockIdx.x + 1) * tiles.n / gridDim.x);
    if (t_beg >= t_end) return;
    const int32_t k4 = K >> 2, cols32 = (N + 31) / 32;

    auto bounds = [&](int32_t tile, int64_t &m0, int64_t &m_end, int32_t &g) __attribute__((always_inline)) {
        if (tiles.id) { m0 = tiles.beg[tile]; m_end = tiles.end[tile]; g = tiles.id[tile]; }
        else { m0 = (int64_t)tile * RT; m_end = m0 + RT < tiles.rows ? m0 + RT : tiles.rows; g = 0; }
    };
    // 8 lanes per row, rows t / 8 and 64 further; past a tile's end its last row, past the width its last numbers again
    float4 ra[2][NI];
    auto load = [&](int32_t tile) __attribute__((always_inline)) {
        int64_t m0, m_end;
        int32_t g;
        bounds(tile, m0, m_end, g);
#pragma unroll
        for (int ps = 0; ps < 2; ++ps) {
            int64_t x = m0 + (t >> 3) + 64 * ps;
            x = x < m_end ? x : m_end - 1;
            const float4 *q = reinterpret_cast<const float4 *>(A + (aidx ? (int64_t)aidx[x] : x) * lda);
#pragma unroll
            for (int i = 0; i < NI; ++i) ra[ps][i] = q[min(8 * i + (t & 7), k4 - 1)];
        }
    };
    auto stage = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int ps = 0; ps < 2; ++ps) {
            const int row = (t >> 3) + 64 * ps;
            uint32_t m = 0u, least = 0xffffffffu;        // least: of twice the bits, less one: the smallest number that is not zero
            auto bits = [](float x) { return __float_as_uint(x) & 0x7fffffffu; };
            auto low = [](float x) { return (__float_as_uint(x) << 1) - 1u; };
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                m = max(m, max(max(bits(ra[ps][i].x), bits(ra[ps][i].y)), max(bits(ra[ps][i].z), bits(ra[ps][i].w))));
                least = min(least, min(min(low(ra[ps][i].x), low(ra[ps][i].y)), min(low(ra[ps][i].z), low(ra[ps][i].w))));
            }
#pragma unroll
            for (int off = 1; off < 8; off <<= 1) m = max(m, (uint32_t)__shfl_xor((int)m, off, 64));
            // an infinity or a NaN: any scale, its results are formed again
            const int e = min(max((int)(m >> 23), 27), 254);
            // 2^(14 - (e - 127)), or NaN if one of the lane's numbers would scale to less than SMALLEST (2^(e - 154) before)
            const uint32_t smallest = e > 27 ? (uint32_t)(e - 27) << 23 : 0x00400000u;
            const float scale = least < 2u * smallest - 1u ? __builtin_nanf("") : __uint_as_float((uint32_t)(268 - e) << 23);
            if ((t & 7) == 0) row_exp[row] = e - 141;
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const int c = 8 * i + (t & 7);
                const float s = c < k4 ? scale : 0.f;
                const Split2 lo = split_large(ra[ps][i].x * s, ra[ps][i].y * s), hi = split_large(ra[ps][i].z * s, ra[ps][i].w * s);
                if (c >= KS * 4) continue;
#pragma unroll
                for (int p = 0; p < 2; ++p) *reinterpret_cast<uint2 *>(lds + p * PLANE + row * PITCH + c * 8) = make_uint2(lo.w[p], hi.w[p]);
            }
        }
    };
    // LDS only: loads and stores of rows stay in flight
    auto barrier = [&]() __attribute__((always_inline)) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    };

    uint4 bh[KS], bl[KS];                                // the group's matrix, this wavefront's columns
    int32_t have = -1;
    load(t_beg);
    for (int32_t tile = t_beg; tile < t_end; ++tile) {
        int64_t m0, m_end;
        int32_t g;
        bounds(tile, m0, m_end, g);
        stage();
        barrier();
        if (multiplies && g != have) {                   // ahead of the next tile's rows: loads retire in order
            const uint4 *b = pack + ((int64_t)g * cols32 + wn) * KS * 128 + lane;
#pragma unroll
            for (int s = 0; s < KS; ++s) { bh[s] = b[s * 128]; bl[s] = b[s * 128 + 64]; }
            have = g;
        }
        if (tile + 1 < t_end) load(tile + 1);
        if (multiplies) {
            const bool again = info[g] == NOT_OK;        // nothing was packed: all of it in fp32
            const int32_t w_exp = again ? 0 : info[g];
            const unsigned char *a = lds + (wm * RB * 32 + (lane & 31)) * PITCH + half * 16;
            split_floatx16 acc[RB], low[RB];             // products of the first parts; 2^11 times those with a second part
#pragma unroll
            for (int i = 0; i < RB; ++i)
#pragma unroll
                for (int v = 0; v < 16; ++v) { acc[i][v] = 0.f; low[i][v] = 0.f; }
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                uint4 ah[RB], al[RB];
#pragma unroll
                for (int i = 0; i < RB; ++i) {
                    al[i] = *reinterpret_cast<const uint4 *>(a + PLANE + i * 32 * PITCH + s * 32);
                    ah[i] = *reinterpret_cast<const uint4 *>(a + i * 32 * PITCH + s * 32);
                }
#pragma unroll
                for (int i = 0; i < RB; ++i) low[i] = split_product<2>(at_own_size(al[i]), bl[s], low[i]);
#pragma unroll
                for (int i = 0; i < RB; ++i) low[i] = split_product<2>(al[i], bh[s], low[i]);
#pragma unroll
                for (int i = 0; i < RB; ++i) low[i] = split_product<2>(ah[i], bl[s], low[i]);
#pragma unroll
                for (int i = 0; i < RB; ++i) acc[i] = split_product<2>(ah[i], bh[s], acc[i]);
            }
            // D register v of lane l is row 8 (v / 4) + 4 (l / 32) + v % 4, column l % 32
            const int n = wn * 32 + (lane & 31);
#pragma unroll
            for (int i = 0; i < RB; ++i) {
                const int r0 = (wm * RB + i) * 32;
                bool odd = false;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int4 e = *reinterpret_cast<const int4 *>(&row_exp[r0 + 8 * q + 4 * half]);
                    const int ex[4] = {e.x, e.y, e.z, e.w};
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        acc[i][4 * q + v] = __builtin_amdgcn_ldexpf(__builtin_fmaf(low[i][4 * q + v], 4.8828125e-4f, acc[i][4 * q + v]), ex[v] + w_exp);
                        odd |= split_not_finite(acc[i][4 * q + v]);
                    }
                }
                const int64_t mb = m0 + r0;
                if (mb >= m_end) continue;
                if (again || __any(odd)) {               // these sums again, in fp32
                    split_floatx16 f;
#pragma unroll
                    for (int v = 0; v < 16; ++v) f[v] = 0.f;
                    const int64_t m = mb + (lane & 31) < m_end ? mb + (lane & 31) : m_end - 1;
                    const float *q = A + (aidx ? (int64_t)aidx[m] : m) * lda;
                    const float *y = W + (int64_t)g * K * N + (int64_t)(n < N ? n : N - 1) * w_n;
                    for (int32_t k = half; k < K; k += 2) f = __builtin_amdgcn_mfma_f32_32x32x2f32(q[k], y[(int64_t)k * w_k], f, 0, 0, 0);
#pragma unroll
                    for (int v = 0; v < 16; ++v) if (again || split_not_finite(acc[i][v])) acc[i][v] = f[v];
                }
                if (n >= N) continue;
                float *o = out + (mb + 4 * half) * N + n;
                const int32_t left = (int32_t)(m_end - mb < 32 ? m_end - mb : 32) - 4 * half;
#pragma unroll
                for (int v = 0; v < 16; ++v) {           // streamed out: the next kernel reads it once
                    const int r = 8 * (v >> 2) + (v & 3);
                    if (r < left) __builtin_nontemporal_store(acc[i][v], o + (int64_t)r * N);
                }
            }
        }
        barrier();
    }
}

template <int KS>
int launch_class(const float *A, int64_t lda, const int32_t *aidx, const RowTiles &tiles, int32_t K, int32_t N, const uint4 *pack,
                 const int32_t *info, const float *W, bool transposed, float *out, hipStream_t st)
{
    const unsigned grid = (unsigned)std::min<int32_t>(tiles.n, 256);
    const int32_t w_k = transposed ? 1 : N, w_n = transposed ? K : 1;
#define RP_CALL(WNV) k_row_products<KS, WNV><<<grid, 512, 0, st>>>(A, lda, aidx, tiles, K, N, pack, info, W, w_k, w_n, out)
    if (N <= 32) RP_CALL(1);
    else if (N <= 64) RP_CALL(2);
    else RP_CALL(4);
#undef RP_CALL
    KGE_LAUNCH_CHECK();
    return KGE_OK;
}

int launch_products(const float *A, int64_t lda, const int32_t *aidx, const RowTiles &tiles, int32_t K, int32_t N, const void *pack,
                    const int32_t *info, const float *W, bool transposed, float *out, hipStream_t st)
{
    if (tiles.n == 0) return KGE_OK;
    const uint4 *pk = reinterpret_cast<const uint4 *>(pack);
    switch (step_class(K)) {
    case 7: return launch_class<7>(A, lda, aidx, tiles, K, N, pk, info, W, transposed, out, st);
    case 8: return launch_class<8>(A, lda, aidx, tiles, K, N, pk, info, W, transposed, out, st);
    default: return launch_class<10>(A, lda, aidx, tiles, K, N, pk, info, W, transposed, out, st);
    }
}

}  // namespace

size_t row_products_bytes(int32_t K, int32_t N) { return (size_t)step_class(K) * ((N + 31) / 32) * 2048; }

// From 100 terms on the results are closer to 64 bits than six bf16 products (relative error of a layer's output, 10^-7: 100
// columns 1.10 / 1.15, 128: 1.13 / 1.22, 160: 1.22 / 1.39; with 96 and three products 1.16 / 1.06); beyond 160 x 128 operands and sums
// do not fit the registers.  The matrices are split anew for every pass: 256 runs per relation pay for that (whole layers, us:
// 3000 entities, 50 relations, 276 runs each, 128 x 128: 228, 232 without; 100 relations, 201 runs each: 242, 249).
bool row_products_pay(const kge_partition *p, int32_t K, int32_t N)
{
    return K >= 100 && K <= 160 && N <= 128 && p->n_seg >= 256 * 2 * (int64_t)p->n_relations;
}

int launch_pack_products(const float *Wrel, const float *W0, int32_t R2, int32_t d_in, int32_t d_out, void *fwd, void *back,
                         int32_t *info, hipStream_t st)
{
    KGE_PROF("pack_weights", st);
    k_pack_products<<<(unsigned)(R2 + 1), 1024, 0, st>>>(Wrel, W0, R2 + 1, d_in, d_out, reinterpret_cast<uint4 *>(fwd),
                                                        reinterpret_cast<uint4 *>(back), step_class(d_in), step_class(d_out), info);
    KGE_LAUNCH_CHECK();
    return KGE_OK;
}

// one row tile per (relation, <= 128 runs)
int launch_apply_relation_products(const kge_partition *p, const float *rows, const int32_t *ridx, int32_t K, int32_t N, const void *pack,
                                   const int32_t *info, const float *Wrel, bool transposed, float *out, hipStream_t st)
{
    KGE_PROF(transposed ? "apply_rel_t" : "apply_rel", st);
    return launch_products(rows, K, ridx, RowTiles{p->relt_rel, p->relt_beg, p->relt_end, p->n_relt, p->n_seg}, K, N, pack, info, Wrel,
                           transposed, out, st);
}

int launch_self_products(const float *rows, int64_t n_rows, int32_t K, int32_t N, const void *pack, const int32_t *info, const float *W0,
                         bool transposed, float *out, hipStream_t st)
{
    KGE_PROF(transposed ? "input_grad" : "project", st);
    return launch_products(rows, K, nullptr, RowTiles{nullptr, nullptr, nullptr, (int32_t)cdiv(n_rows, RT), n_rows}, K, N, pack, info, W0,
                           transposed, out, st);
}
