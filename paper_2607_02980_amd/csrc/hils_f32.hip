// HiLS attention for fp32 storage on the fp32 matrix instruction, gfx950: the
// attention of the prefill (the selection is in hils_fwd.hip) and its backward.
//
// v_mfma_f32_16x16x4_f32 (A 16x4, B 4x16, D 16x16; fp32 products and sums), lane l:
//   A: A[m = l%16][k = l/16]   B: B[k = l/16][n = l%16]   D: D[m = (l/16)*4 + i][n = l%16]
// The contraction index may be dealt to the lane groups in any order as long as A and
// B agree, which makes every operand a 16-byte load of a row-major tensor and every
// product's accumulators the next product's operand:
//   over the head dim, k-step (t, j) of group lg = l/16 is dim 16 t + 4 lg + j, so a
//     float4 of row l%16 holds four k-steps ("row" operand);
//   over 16 rows, k-step i of group lg is row 4 lg + i, exactly where accumulators hold
//     them; the other operand takes output dim 4 (l%16) + j of 64-wide block dd as
//     product j, so a float4 of row 4 lg + i feeds four products ("column" operand), and
//     accumulator [4 dd + j][i] is dim 64 dd + 16 lg + 4 i + j.
// fp32 sequences are short and few, so the work is cut fine: a wave owns 16 (row, head)
// columns against one 64-key part at a time, and the waves of a block (forward, dq) or
// several blocks (dk, dv) share a tile's parts and add their sums in a fixed order.
//
// Gradients as in hils_bwd.hip's head comment.
#include "hils_device.hpp"
#include "hils_dispatch.hpp"
#include "hils_internal.hpp"
#include "hils_mfma.hpp"

namespace hils {

namespace {

constexpr int kW = 4;                    // waves per block of the backward
constexpr int kThreads = kW * kWave;
constexpr int kAttnW = 8;                // waves per block of the forward
constexpr int kCols = 16;                // (query, head) columns of a block: 16 / G queries x G heads
constexpr int kMaxItems = kCols * 64;    // entries of 16 / G queries' selections (K <= 64)

__device__ __forceinline__ f32x4 mfma_f32(float a, float b, const f32x4& c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
// Four floats of global memory, of which only the alignment of a float is known (a caller's
// array may begin anywhere; one instruction takes it all the same), and of LDS.
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ f32x4 ld4(const float* p) { return *reinterpret_cast<const f32x4u*>(p); }
__device__ __forceinline__ void st4(float* p, const f32x4& x) { *reinterpret_cast<f32x4u*>(p) = x; }
__device__ __forceinline__ f32x4 lds4(const float* p) { return *reinterpret_cast<const f32x4*>(p); }
__device__ __forceinline__ void to_lds4(float* p, const f32x4& x) { *reinterpret_cast<f32x4*>(p) = x; }

// The parts of a tile of queries q0 .. q0 + 16/G - 1 of one KV group: the 64-key pieces
// of their local windows, then the union of the chunks they retrieved, each with the
// queries that did.
struct __align__(16) TileParts {
    int sel[kMaxItems];               // [query][K, a multiple of 4] the rows' valid entries, else -1
    int chunk[kMaxItems];             // union, in order of (first query, slot)
    unsigned short users[kMaxItems];  // its queries, one bit each
    int wave_n[kAttnW];
    int len[kCols];                   // entries up to the query's last valid one
    int n;                            // union size
    int bad;                          // a result of the tile is not finite
};

// Fills sel, chunk, users and n; called by the whole block, ends with a barrier.  Every valid
// entry counts its chunk in all the queries' lists, four entries per LDS read and no further
// than each list's last valid entry (all entries one by one, with a division for the query:
// 142 us for 200 tokens, 4 heads in groups of 1, d = 64, K = 64, W = 64).
template <int NW>
__device__ inline void build_parts(TileParts& tp, const int32_t* idx, int N, int K, int W, int q0, int nq) {
    const int tid = threadIdx.x, lane = tid % kWave, w = wave_id();
    const int K4 = (K + 3) & ~3;
    if (tid < nq) tp.len[tid] = 0;
    if (tid == 0) tp.bad = 0;
    __syncthreads();
    for (int e = tid; e < nq * K4; e += NW * kWave) {
        const int q = e / K4, slot = e % K4, n = q0 + q;
        int v = -1;
        if (n < N && slot < K) {
            const int32_t* row = idx + (size_t)n * K;
            if (idx_entry_valid(row, slot, n_candidates(n, W))) v = row[slot];
        }
        tp.sel[e] = v;
        if (v >= 0) atomicMax(&tp.len[q], slot + 1);
    }
    __syncthreads();
    auto times = [&](int i, int c, int upto) {  // how often query i names c before slot upto
        const int4* row = reinterpret_cast<const int4*>(tp.sel + i * K4);
        int t = 0;
        for (int s = 0; s < upto; s += 4) {
            const int4 v = row[s / 4];
            t += (int)(v.x == c) + (int)(v.y == c) + (int)(v.z == c) + (int)(v.w == c);
        }
        return t;
    };
    int base = 0;
    for (int e0 = 0; e0 < nq * K4; e0 += NW * kWave) {
        const int e = e0 + tid;
        const int c = e < nq * K4 ? tp.sel[e] : -1;
        // the m-th time that a query names the chunk (a given row out of order may name it more
        // than once): used by the queries that name it as often, listed by the first of them
        const int q = e / K4;
        unsigned users = 0;
        if (__ballot(c >= 0) != 0ull) {  // uniform over the wave
            int m = 1;
            for (int t = q * K4; t < e && c >= 0; ++t) m += tp.sel[t] == c;
            for (int i = 0; i < nq; ++i)
                users |= (unsigned)(times(i, c, __builtin_amdgcn_readfirstlane(tp.len[i])) >= m) << i;
        }
        const bool lead = c >= 0 && (users & ((1u << q) - 1u)) == 0;
        const uint64_t bal = __ballot(lead);
        if (lane == 0) tp.wave_n[w] = popc64(bal);
        __syncthreads();
        int pos = base + popc64(bal & ((1ull << lane) - 1ull));
        int all = 0;
        for (int i = 0; i < NW; ++i) {
            pos += i < w ? tp.wave_n[i] : 0;
            all += tp.wave_n[i];
        }
        if (lead) {
            tp.chunk[pos] = c;
            tp.users[pos] = (unsigned short)users;
        }
        base += all;
        __syncthreads();
    }
    if (tid == 0) tp.n = base;
    __syncthreads();
}

// x . y of two rows, the lane's dims (both pointers at dim 4 lg), summed over the lane groups.
template <int D>
__device__ __forceinline__ float row_dot(const float* x, const float* y) {
    float acc = 0.f;
#pragma unroll
    for (int t = 0; t < D / 16; ++t) {
        const f32x4 u = ld4(x + 16 * t), v = ld4(y + 16 * t);
#pragma unroll
        for (int j = 0; j < 4; ++j) acc = fmaf(u[j], v[j], acc);
    }
    return group4_sum(acc);
}

// A 64-row block of X as row operands (16 rows k, k-steps t) or as column operands
// (rows 16 k + 4 lg + i, 64-wide dim block dd), in registers: 64 or, d = 128, 128 of them.
template <int D>
struct RowOps {
    f32x4 x[4][D / 16];
    __device__ __forceinline__ void load(const float* X, int lane) {
        const float* p = X + (size_t)(lane % 16) * D + 4 * (lane / 16);
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int t = 0; t < D / 16; ++t) x[k][t] = ld4(p + (size_t)16 * k * D + 16 * t);
    }
    // acc[k][row 16 k + 4 lg + i][column l%16] of the block against the columns' y
    __device__ __forceinline__ void times(const f32x4* y, f32x4* acc) const {
#pragma unroll
        for (int k = 0; k < 4; ++k) acc[k] = zero4();
#pragma unroll
        for (int t = 0; t < D / 16; ++t)
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int k = 0; k < 4; ++k) acc[k] = mfma_f32(x[k][t][j], y[t][j], acc[k]);
    }
};
template <int D>
struct ColOps {
    f32x4 x[4][4][D / 64];
    __device__ __forceinline__ void load(const float* X, int lane) {
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int dd = 0; dd < D / 64; ++dd)
                    x[k][i][dd] = ld4(X + (size_t)(16 * k + 4 * (lane / 16) + i) * D + 64 * dd + 4 * (lane % 16));
    }
    // o[dims][column] += X^T p; rows at or past `rows` count as zero (their bytes may be
    // anything, and 0 * NaN would reach every column)
    __device__ __forceinline__ void add(int rows, const f32x4* p, f32x4* o, int lane) {
        if (rows < kChunk) {
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int dd = 0; dd < D / 64; ++dd)
                        if (16 * k + 4 * (lane / 16) + i >= rows) x[k][i][dd] = zero4();
        }
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int dd = 0; dd < D / 64; ++dd)
#pragma unroll
                    for (int j = 0; j < 4; ++j) o[4 * dd + j] = mfma_f32(x[k][i][dd][j], p[k][i], o[4 * dd + j]);
    }
};

// The items of a wave's tile: pieces 0 .. npiece - 1, then the union's chunks; the first
// one from `it` on (in steps of the waves) that a query of `mine` uses.
__device__ __forceinline__ int next_item(const TileParts& tp, int it, int npiece, int items, unsigned mine) {
    while (it >= npiece && it < items && (__builtin_amdgcn_readfirstlane(tp.users[it - npiece]) & mine) == 0u) it += kW;
    return it;
}

// acc[key 4 lg + i][column l%16] of 16 rows of X (from `row0`) against the columns' x.
template <int D>
__device__ __forceinline__ f32x4 rows_times(const float* row0, const f32x4* x, int lane) {
    const float* p = row0 + (size_t)(lane % 16) * D + 4 * (lane / 16);
    f32x4 acc = zero4();
#pragma unroll
    for (int t = 0; t < D / 16; ++t) {
        const f32x4 y = ld4(p + 16 * t);
#pragma unroll
        for (int j = 0; j < 4; ++j) acc = mfma_f32(y[j], x[t][j], acc);
    }
    return acc;
}

// o[dims][column] += X^T p over 16 rows of X; rows at or past `rows` count as zero
// (their bytes may be anything, and 0 * NaN would reach every column).
template <int D>
__device__ __forceinline__ void add_columns(const float* row0, int rows, const f32x4& p, f32x4* o, int lane) {
    const int lg = lane / 16;
#pragma unroll
    for (int dd = 0; dd < D / 64; ++dd)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int r = 4 * lg + i;
            f32x4 y = ld4(row0 + (size_t)r * D + 64 * dd + 4 * (lane % 16));
            if (r >= rows) y = zero4();
#pragma unroll
            for (int j = 0; j < 4; ++j) o[4 * dd + j] = mfma_f32(y[j], p[i], o[4 * dd + j]);
        }
}

// ---------------------------------------------------------------------------
// Forward: local window, retrieved chunks and their fusion (Eqs. (1), (10))
// ---------------------------------------------------------------------------
// One block per 16 / G queries x G heads of one KV group; wave w takes parts w, w + 8,
// ... and keeps a running maximum M, denominator Z and numerator o per column (a window
// piece enters with its exponentials, a chunk with e^{s^} times its own softmax), merged
// over the waves at the end.  K and V come straight from L2: a wave shares them with no
// other.  A value of V that is not finite reaches every column of the tile through a
// product with zero, so a tile with such a result is done again one query at a time.
//
// Bound: the fp32 matrix rate (157 TFLOP/s) where the union is dense, load latency at two
// waves per SIMD in short sequences.  2048 queries, 4 heads over 1 KV head, d = 64,
// K = 4: one block per query with scalar dot products from LDS took 119 us.
template <int D, int G>
__global__ __launch_bounds__(kAttnW * kWave, D == 64 ? 4 : 2) void k_attn_f32(FwdArgs a) {
    constexpr int T = D / 16, DB = D / 16, NQ = kCols / G;
    __shared__ TileParts tp;
    __shared__ __align__(16) float s_o[kAttnW][kCols][D + 4];
    __shared__ float s_m[kAttnW][kCols], s_z[kAttnW][kCols];
    const int tid = threadIdx.x, w = wave_id(), lane = tid % kWave, lg = lane / 16, col = lane % 16;
    const int q0 = blockIdx.x * NQ, g = blockIdx.y, b = blockIdx.z;
    const int nC = a.L / kChunk;
    const size_t bg = (size_t)b * a.Hkv + g;
    const float* kb = as<float>(a.k) + bg * a.L * D;
    const float* vb = as<float>(a.v) + bg * a.L * D;
    const int hh = col % G, qi = col / G, n = min(q0 + qi, a.N - 1);
    const int hl = (a.Hl == a.Hq) ? g * G + hh : g;
    const size_t row = ((size_t)b * a.Hq + g * G + hh) * a.N + n;
    const float* lrows = as<float>(a.lmk) + ((size_t)b * a.Hl + hl) * nC * D;
    const float* lbias = a.bias ? a.bias + ((size_t)b * a.Hl + hl) * nC : nullptr;
    f32x4 q[T];
#pragma unroll
    for (int t = 0; t < T; ++t) q[t] = ld4(as<float>(a.q) + row * D + 16 * t + 4 * lg);
    const float* qrow = as<float>(a.q_route ? a.q_route : a.q) + row * D + 4 * lg;
    build_parts<kAttnW>(tp, a.idx + bg * a.N * a.K, a.N, a.K, a.W, q0, NQ);

    // one pass over the parts of the queries first .. last; writes those rows
    auto pass = [&](int first, int last) {
        const int nlast = min(q0 + last, a.N - 1);
        const int c0 = n_candidates(min(q0 + first, a.N - 1), a.W), npiece = nlast / kChunk - c0 + 1;
        const int ell = n_candidates(n, a.W) * kChunk;
        const unsigned mine = ((2u << last) - 1u) & ~((1u << first) - 1u);
        f32x4 o[DB];
#pragma unroll
        for (int db = 0; db < DB; ++db) o[db] = zero4();
        float M = -INFINITY, Z = 0.f;
        const int items = npiece + __builtin_amdgcn_readfirstlane(tp.n);  // scalar: MFMAs ignore the lane mask
        for (int it = w; it < items; it += kAttnW) {
            const bool piece = it < npiece;
            const unsigned users =
                piece ? 0u : __builtin_amdgcn_readfirstlane(tp.users[piece ? 0 : it - npiece]) & mine;
            if (!piece && users == 0u) continue;  // uniform over the wave
            const int c = __builtin_amdgcn_readfirstlane(piece ? c0 + it : tp.chunk[piece ? 0 : it - npiece]);
            const float* kc = kb + (size_t)c * kChunk * D;
            const float* vc = vb + (size_t)c * kChunk * D;
            f32x4 s[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) s[k] = rows_times<D>(kc + 16 * k * D, q, lane);
            const int j0 = c * kChunk;
            float mx = -INFINITY;
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int j = j0 + 16 * k + 4 * lg + i;
                    s[k][i] = (!piece || (j <= n && j >= ell)) ? a.scale * s[k][i] : -INFINITY;
                    mx = fmaxf(mx, s[k][i]);
                }
            mx = group4_max(mx);
            const float ms = mx == -INFINITY ? 0.f : mx;
            float l = 0.f;
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    s[k][i] = fexp(s[k][i] - ms);
                    l += s[k][i];
                }
            l = group4_sum(l);
            // the part's logit (log of the mass it enters with) and the factor of its exponentials
            const bool on = piece ? mx != -INFINITY : (users >> qi) & 1u;
            const float z = piece ? mx : a.scale * row_dot<D>(qrow, lrows + (size_t)c * D + 4 * lg) + (lbias ? lbias[c] : 0.f);
            const float Mn = on ? fmaxf(M, z) : M;
            const float Mu = Mn == -INFINITY ? 0.f : Mn;
            const float rs = fexp(M - Mu);
            const float e = on ? fexp(z - Mu) : 0.f;
            Z = Z * rs + (piece ? l * e : e);
            const float f = piece ? e : e / l;
            M = Mn;
            f32x4 oc[DB];
#pragma unroll
            for (int db = 0; db < DB; ++db) oc[db] = zero4();
#pragma unroll
            for (int k = 0; k < 4; ++k) add_columns<D>(vc + 16 * k * D, nlast + 1 - j0 - 16 * k, s[k], oc, lane);
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int i = 0; i < 4; ++i) o[db][i] = on ? o[db][i] * rs + f * oc[db][i] : o[db][i];
        }
        if (lg == 0) {
            s_m[w][col] = M;
            s_z[w][col] = Z;
        }
#pragma unroll
        for (int dd = 0; dd < D / 64; ++dd)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                to_lds4(&s_o[w][col][64 * dd + 16 * lg + 4 * i],
                    f32x4{o[4 * dd][i], o[4 * dd + 1][i], o[4 * dd + 2][i], o[4 * dd + 3][i]});
        __syncthreads();
        // (the results are stored after all of the tile's are known to be finite or the pass
        // is one query's, and the queries are read for s^: out may take their place)
        static_assert(kCols * D / 4 <= kAttnW * kWave, "one piece of the results per thread");
        const int cc = tid / (D / 4), d4 = (tid % (D / 4)) * 4, qq = cc / G, nn = q0 + qq;
        const bool stores = cc < kCols && nn < a.N && qq >= first && qq <= last;
        float mm = 0.f, zz = 0.f;
        f32x4 acc = zero4();
        if (stores) {
            mm = s_m[0][cc];
#pragma unroll
            for (int i = 1; i < kAttnW; ++i) mm = fmaxf(mm, s_m[i][cc]);
#pragma unroll
            for (int i = 0; i < kAttnW; ++i) {
                const float x = fexp(s_m[i][cc] - mm);
                zz += s_z[i][cc] * x;
                acc += lds4(&s_o[i][cc][d4]) * x;
            }
            acc *= 1.f / zz;
            const float t = acc[0] + acc[1] + acc[2] + acc[3];
            if (NQ > 1 && !(fabsf(t) < INFINITY)) tp.bad = 1;
        }
        __syncthreads();
        if (stores && (first == last || !tp.bad)) {
            const size_t orow = ((size_t)b * a.Hq + g * G + cc % G) * a.N + nn;
            st4(as_mut<float>(a.out) + orow * D + d4, acc);
            if (d4 == 0) a.lse[orow] = mm + __logf(zz);
        }
    };
    pass(0, NQ - 1);
    if (NQ > 1 && tp.bad)
        for (int i = 0; i < NQ; ++i) pass(i, i);
}

// ---------------------------------------------------------------------------
// Backward, query-major: dq, dq^ and u = dO . out
// ---------------------------------------------------------------------------
// The forward's tile and split of the parts.  Per part S^T = K Q^T, GV^T = V dO^T, ds and
// dq^T += K^T ds^T; a retrieved chunk adds ds^_c k'_c.  The waves' sums are added at the
// end.  Also clears the inverse index's counters, which the next launch uses.  (One block
// per query with scalar dot products: 145 us at 2048 queries, 4 heads.)
template <int D, int G>
__global__ __launch_bounds__(kThreads, D == 64 ? 2 : 1) void k_bwd_dq_f32(BwdArgs a, float* u, int* counts, size_t nclear) {
    constexpr int T = D / 16, DB = D / 16, NQ = kCols / G;
    __shared__ TileParts tp;
    __shared__ __align__(16) float s_o[kW][kCols][D + 4];
    __shared__ __align__(16) float s_r[kW][kCols][D + 4];  // dq^ (routing queries given)
    const int tid = threadIdx.x, w = wave_id(), lane = tid % kWave, lg = lane / 16, col = lane % 16;
    const int q0 = blockIdx.x * NQ, g = blockIdx.y, b = blockIdx.z;
    const int nC = a.L / kChunk;
    const size_t bg = (size_t)b * a.Hkv + g;
    for (size_t i = (bg * gridDim.x + blockIdx.x) * kThreads + tid; i < nclear;
         i += (size_t)gridDim.x * gridDim.y * gridDim.z * kThreads)
        counts[i] = 0;
    const float* kb = as<float>(a.k) + bg * a.L * D;
    const float* vb = as<float>(a.v) + bg * a.L * D;
    const int hh = col % G, qi = col / G, n = min(q0 + qi, a.N - 1);
    const int hl = (a.Hl == a.Hq) ? g * G + hh : g;
    const size_t row = ((size_t)b * a.Hq + g * G + hh) * a.N + n;
    const float* lrows = as<float>(a.lmk) + ((size_t)b * a.Hl + hl) * nC * D;
    const float* lbias = a.bias ? a.bias + ((size_t)b * a.Hl + hl) * nC : nullptr;
    const bool route = a.q_route != nullptr;
    const float* qrow = as<float>(route ? a.q_route : a.q) + row * D + 4 * lg;
    f32x4 q[T], go[T];
    float ub = 0.f;
#pragma unroll
    for (int t = 0; t < T; ++t) {
        q[t] = ld4(as<float>(a.q) + row * D + 16 * t + 4 * lg);
        go[t] = ld4(as<float>(a.dout) + row * D + 16 * t + 4 * lg);
        const f32x4 y = ld4(as<float>(a.out) + row * D + 16 * t + 4 * lg);
#pragma unroll
        for (int j = 0; j < 4; ++j) ub = fmaf(go[t][j], y[j], ub);
    }
    ub = group4_sum(ub);
    const float L = a.lse[row];
    if (w == 0 && lg == 0 && q0 + qi < a.N) u[row] = ub;
    build_parts<kW>(tp, a.idx + bg * a.N * a.K, a.N, a.K, a.W, q0, NQ);

    auto pass = [&](int first, int last) {
        const int nlast = min(q0 + last, a.N - 1);
        const int c0 = n_candidates(min(q0 + first, a.N - 1), a.W), npiece = nlast / kChunk - c0 + 1;
        const int ell = n_candidates(n, a.W) * kChunk;
        const unsigned mine = ((2u << last) - 1u) & ~((1u << first) - 1u);
        f32x4 dq[DB], dr[DB];  // dr in the lane's dims of dq: [4 dd + j][i]
#pragma unroll
        for (int db = 0; db < DB; ++db) dq[db] = dr[db] = zero4();
        const int items = npiece + __builtin_amdgcn_readfirstlane(tp.n);  // scalar: MFMAs ignore the lane mask
        auto chunk_of = [&](int i) {
            return __builtin_amdgcn_readfirstlane(i < npiece ? c0 + i : tp.chunk[max(i - npiece, 0)]);
        };
        int it = next_item(tp, w, npiece, items, mine);
        int c = it < items ? chunk_of(it) : 0;
        while (it < items) {
            const bool piece = it < npiece;
            const unsigned users = piece ? 0u : __builtin_amdgcn_readfirstlane(tp.users[max(it - npiece, 0)]);
            const int j0 = c * kChunk;
            // V's rows in flight during S, K's columns during the softmax terms
            RowOps<D> kr, vr;
            kr.load(kb + (size_t)j0 * D, lane);
            vr.load(vb + (size_t)j0 * D, lane);
            f32x4 s[4], gv[4];
            kr.times(q, s);
            vr.times(go, gv);
            __builtin_amdgcn_sched_barrier(0);
            ColOps<D> kc;
            kc.load(kb + (size_t)j0 * D, lane);
            const int nit = next_item(tp, it + kW, npiece, items, mine);
            const int cn = nit < items ? chunk_of(nit) : c;
            if (piece) {
#pragma unroll
                for (int k = 0; k < 4; ++k)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int j = j0 + 16 * k + 4 * lg + i;
                        s[k][i] = (j <= n && j >= ell) ? fexp(a.scale * s[k][i] - L) * (gv[k][i] - ub) : 0.f;
                    }
            } else {
                const bool on = (users >> qi) & 1u;
                float mx = -INFINITY;
#pragma unroll
                for (int k = 0; k < 4; ++k)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        s[k][i] *= a.scale;
                        mx = fmaxf(mx, s[k][i]);
                    }
                mx = group4_max(mx);
                float l = 0.f;
#pragma unroll
                for (int k = 0; k < 4; ++k)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        s[k][i] = fexp(s[k][i] - mx);
                        l += s[k][i];
                    }
                const float inv = 1.f / group4_sum(l);
                float uc = 0.f;
#pragma unroll
                for (int k = 0; k < 4; ++k)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        s[k][i] *= inv;
                        uc = fmaf(s[k][i], gv[k][i], uc);
                    }
                uc = group4_sum(uc);
                const float* lrow = lrows + (size_t)c * D;
                const float sh = a.scale * row_dot<D>(qrow, lrow + 4 * lg) + (lbias ? lbias[c] : 0.f);
                const float al = fexp(sh - L);
                const float dsh = on ? al * (uc - ub) : 0.f;
#pragma unroll
                for (int k = 0; k < 4; ++k)
#pragma unroll
                    for (int i = 0; i < 4; ++i) s[k][i] = on ? al * s[k][i] * (gv[k][i] - uc) : 0.f;
#pragma unroll
                for (int dd = 0; dd < D / 64; ++dd)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const f32x4 y = ld4(lrow + 64 * dd + 16 * lg + 4 * i);
#pragma unroll
                        for (int j = 0; j < 4; ++j) dr[4 * dd + j][i] += on ? dsh * y[j] : 0.f;
                    }
            }
            kc.add(nlast + 1 - j0, s, dq, lane);
            it = nit;
            c = cn;
        }
#pragma unroll
        for (int dd = 0; dd < D / 64; ++dd)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int d0 = 64 * dd + 16 * lg + 4 * i;
                f32x4 x = {dq[4 * dd][i], dq[4 * dd + 1][i], dq[4 * dd + 2][i], dq[4 * dd + 3][i]};
                const f32x4 y = {dr[4 * dd][i], dr[4 * dd + 1][i], dr[4 * dd + 2][i], dr[4 * dd + 3][i]};
                if (route)
                    to_lds4(&s_r[w][col][d0], y);
                else
                    x += y;
                to_lds4(&s_o[w][col][d0], x);
            }
        __syncthreads();
        for (int e = tid; e < kCols * D / 4; e += kThreads) {
            const int cc = e / (D / 4), d4 = (e % (D / 4)) * 4, qq = cc / G, nn = q0 + qq;
            if (nn >= a.N || qq < first || qq > last) continue;
            const size_t orow = ((size_t)b * a.Hq + g * G + cc % G) * a.N + nn;
            f32x4 x = zero4(), y = zero4();
#pragma unroll
            for (int i = 0; i < kW; ++i) {
                x += lds4(&s_o[i][cc][d4]);
                if (route) y += lds4(&s_r[i][cc][d4]);
            }
            x *= a.scale;
            st4(as_mut<float>(a.dq) + orow * D + d4, x);
            if (route) st4(as_mut<float>(a.dq_route) + orow * D + d4, y * a.scale);
            const float t = x[0] + x[1] + x[2] + x[3];
            if (NQ > 1 && !(fabsf(t) < INFINITY)) tp.bad = 1;
        }
        __syncthreads();
    };
    pass(0, NQ - 1);
    if (NQ > 1 && tp.bad)
        for (int i = 0; i < NQ; ++i) pass(i, i);
}

// ---------------------------------------------------------------------------
// Backward, key-major: dk, dv of one chunk and dk', db' of its landmarks
// ---------------------------------------------------------------------------
// The pairs (row, head) of chunk c, 16 / G rows x G heads per tile: first the rows whose
// window covers keys of c, then the rows that retrieved it (sorted).  The tiles are dealt
// over nsplit blocks of 4 waves per chunk (a 2K sequence has 32 chunks for 256 CUs), each
// wave with its own dK^T, dV^T of all 64 keys; the block adds its waves' sums through LDS
// and k_bwd_sum_f32 the blocks', both in a fixed order.  S = Q K^T here (pairs on the M
// side), so that the weights are the operands of dV^T += dO^T P and dK^T += Q^T dS.
//
// Bound: the fp32 matrix rate (1 us of it per 16 pairs and wave at d = 64) and, at 1 or 2
// waves per SIMD, the loads of each tile's rows.  One block per chunk taking one row at a
// time: 4006 us at 2048 queries, 4 heads over 1 KV head, d = 64, K = 4.
template <int D, int G>
struct SumLayout {  // floats of one block's sums: dK, dV [64][D], dK' [G][D], db' [G]
    static constexpr int dk = 0, dv = kChunk * D, dl = 2 * kChunk * D, db = dl + G * D, n = (db + G + 3) / 4 * 4;
};

// Max / sum over the 16 lanes l%16 of a lane group.
__device__ __forceinline__ float max16(float x) {
    x = fmaxf(x, dpp<0xB1>(x));
    x = fmaxf(x, dpp<0x4E>(x));
    x = fmaxf(x, dpp<0x141>(x));
    return fmaxf(x, dpp<0x140>(x));
}

template <int D, int G>
__global__ __launch_bounds__(kThreads, D == 64 ? 2 : 1) void k_bwd_keys_f32(BwdArgs a, const int* offsets,
                                                                           const int* sorted, const float* u,
                                                                           float* sums, int nsplit) {
    constexpr int T = D / 16, DB = D / 16, RT = kCols / G, ROW = D + 4;
    using SL = SumLayout<D, G>;
    __shared__ __align__(16) float s_kv[2][kChunk][ROW];
    __shared__ __align__(16) float s_dl[kW][G][D];
    __shared__ float s_db[kW][G];
    const int tid = threadIdx.x, w = wave_id(), lane = tid % kWave, lg = lane / 16, col = lane % 16;
    const int c = blockIdx.x / nsplit, split = blockIdx.x % nsplit, g = blockIdx.y, b = blockIdx.z;
    const int nC = a.L / kChunk, j0 = c * kChunk;
    const size_t bg = (size_t)b * a.Hkv + g;
    const bool route = a.q_route != nullptr, per_head = a.Hl == a.Hq;
    const float* q = as<float>(a.q);
    const float* qr = as<float>(route ? a.q_route : a.q);
    const float* go = as<float>(a.dout);
    for (int e = tid; e < 2 * kChunk * D / 4; e += kThreads) {
        const int m = e / (kChunk * D / 4), r = e % (kChunk * D / 4) / (D / 4), d4 = (e % (D / 4)) * 4;
        to_lds4(&s_kv[m][r][d4], ld4(as<float>(m ? a.v : a.k) + (bg * a.L + j0 + r) * D + d4));
    }
    __syncthreads();
    const int n_hi = min(a.N - 1, j0 + kChunk + a.W - 2);
    const int nlocal = max(0, n_hi - j0 + 1);
    int beg = 0, nret = 0;
    if (offsets) {
        beg = __builtin_amdgcn_readfirstlane(offsets[bg * (nC + 1) + c]);
        nret = __builtin_amdgcn_readfirstlane(offsets[bg * (nC + 1) + c + 1]) - beg;
    }
    const int* seg = sorted + bg * a.N * a.K + beg;
    const int tloc = (nlocal + RT - 1) / RT, tiles = tloc + (nret + RT - 1) / RT;

    f32x4 dk[DB][4], dv[DB][4], dl[4][D / 64];
    float db[4];
#pragma unroll
    for (int x = 0; x < DB; ++x)
#pragma unroll
        for (int k = 0; k < 4; ++k) dk[x][k] = dv[x][k] = zero4();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        db[i] = 0.f;
#pragma unroll
        for (int dd = 0; dd < D / 64; ++dd) dl[i][dd] = zero4();
    }
    // row of pair p = (row p / G, head p % G) of tile t, or -1
    auto pair_row = [&](int t, int p) {
        const bool ret = t >= tloc;
        const int e = (ret ? t - tloc : t) * RT + p / G;
        if (e >= (ret ? nret : nlocal)) return -1;
        return ret ? seg[e] >> 6 : j0 + e;
    };
    const size_t hrow = (size_t)b * a.Hq + g * G;
    const int cl = per_head ? g * G + col % G : g;
    const float* lrow = as<float>(a.lmk) + (((size_t)b * a.Hl + cl) * nC + c) * D;
    const float lbias = a.bias ? a.bias[((size_t)b * a.Hl + cl) * nC + c] : 0.f;
    for (int t = split * kW + w; t < tiles; t += nsplit * kW) {
        const bool ret = t >= tloc;  // uniform over the wave
        asm volatile("" ::: "memory");  // K and V are read from LDS in every tile, not kept in registers
        f32x4 s[4], gv[4];
        float sh_row = 0.f;  // s^_c of pair l%16
        {
            const int n = pair_row(t, col);
            const size_t r = (hrow + col % G) * a.N + max(n, 0);
            f32x4 x[T], y[T];
#pragma unroll
            for (int k = 0; k < T; ++k) {
                x[k] = ld4(q + r * D + 16 * k + 4 * lg);
                y[k] = ld4(go + r * D + 16 * k + 4 * lg);
            }
            if (ret) {
                sh_row = a.scale * row_dot<D>(qr + r * D + 4 * lg, lrow + 4 * lg) + lbias;
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                s[k] = gv[k] = zero4();
#pragma unroll
                for (int tt = 0; tt < T; ++tt) {
                    const f32x4 kk = lds4(&s_kv[0][16 * k + col][16 * tt + 4 * lg]);
                    const f32x4 vv = lds4(&s_kv[1][16 * k + col][16 * tt + 4 * lg]);
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        s[k] = mfma_f32(x[tt][j], kk[j], s[k]);
                        gv[k] = mfma_f32(y[tt][j], vv[j], gv[k]);
                    }
                }
            }
        }
        asm volatile("" ::: "memory");
        // pair 4 lg + i against key 16 k + l%16: the weight of dV and ds, then the pair's
        // rows as column operands (an empty pair's count as zero)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int p = 4 * lg + i, n = pair_row(t, p);
            const bool on = n >= 0;
            const size_t r = (hrow + p % G) * a.N + max(n, 0);
            f32x4 gt[D / 64], qt[D / 64];
#pragma unroll
            for (int dd = 0; dd < D / 64; ++dd) {
                gt[dd] = ld4(go + r * D + 64 * dd + 4 * col);
                qt[dd] = ld4(q + r * D + 64 * dd + 4 * col);
                if (!on) gt[dd] = qt[dd] = zero4();
            }
            const float L = a.lse[r], ub = u[r];
            float wt[4], ds[4];
            if (!ret) {
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const bool sees = j0 + 16 * k + col <= n;  // (keys past it may hold anything)
                    wt[k] = sees ? fexp(a.scale * s[k][i] - L) : 0.f;
                    ds[k] = sees ? wt[k] * (gv[k][i] - ub) : 0.f;
                }
            } else {
                float mx = -INFINITY;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    wt[k] = a.scale * s[k][i];
                    mx = fmaxf(mx, wt[k]);
                }
                mx = max16(mx);
                float l = 0.f;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    wt[k] = fexp(wt[k] - mx);
                    l += wt[k];
                }
                const float inv = 1.f / group_sum<16>(l);
                float uc = 0.f;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    wt[k] *= inv;
                    uc = fmaf(wt[k], gv[k][i], uc);
                }
                uc = group_sum<16>(uc);
                const float al = fexp(__shfl(sh_row, p, kWave) - L);
                const float dsh = on ? al * (uc - ub) : 0.f;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    wt[k] = on ? al * wt[k] : 0.f;
                    ds[k] = on ? wt[k] * (gv[k][i] - uc) : 0.f;
                }
                db[i] += dsh;
#pragma unroll
                for (int dd = 0; dd < D / 64; ++dd) {
                    f32x4 y = qt[dd];
                    if (route) y = ld4(qr + r * D + 64 * dd + 4 * col);
                    if (on) dl[i][dd] += dsh * y;
                }
            }
#pragma unroll
            for (int dd = 0; dd < D / 64; ++dd)
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        dv[4 * dd + j][k] = mfma_f32(gt[dd][j], wt[k], dv[4 * dd + j][k]);
                        dk[4 * dd + j][k] = mfma_f32(qt[dd][j], ds[k], dk[4 * dd + j][k]);
                    }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    // dk' and db': pair 4 lg + i is head (4 lg + i) % G; sum the lanes and the i of a head
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        auto over_groups = [&](float x) {
            if constexpr (G == 8) return x + __shfl_xor(x, 32, kWave);  // groups lg and lg + 2 hold the same head
            return group4_sum(x);
        };
        db[i] = over_groups(db[i]);
#pragma unroll
        for (int dd = 0; dd < D / 64; ++dd)
#pragma unroll
            for (int j = 0; j < 4; ++j) dl[i][dd][j] = over_groups(dl[i][dd][j]);
    }
    if (lg < (G == 8 ? 2 : 1)) {
#pragma unroll
        for (int h = 0; h < (G < 4 ? G : 4); ++h) {
            float x = 0.f;
            f32x4 y[D / 64];
#pragma unroll
            for (int dd = 0; dd < D / 64; ++dd) y[dd] = zero4();
#pragma unroll
            for (int i = h; i < 4; i += (G < 4 ? G : 4)) {
                x += db[i];
#pragma unroll
                for (int dd = 0; dd < D / 64; ++dd) y[dd] += dl[i][dd];
            }
            const int hd = G == 8 ? 4 * lg + h : h;
            if (col == 0) s_db[w][hd] = x;
#pragma unroll
            for (int dd = 0; dd < D / 64; ++dd) to_lds4(&s_dl[w][hd][64 * dd + 4 * col], y[dd]);
        }
    }
    // dK, dV: the waves add their sums one after another
    for (int ww = 0; ww < kW; ++ww) {
        __syncthreads();
        if (w == ww)
#pragma unroll
            for (int dd = 0; dd < D / 64; ++dd)
#pragma unroll
                for (int k = 0; k < 4; ++k)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        float* pk = &s_kv[0][16 * k + col][64 * dd + 16 * lg + 4 * i];
                        float* pv = &s_kv[1][16 * k + col][64 * dd + 16 * lg + 4 * i];
                        f32x4 x = {dk[4 * dd][k][i], dk[4 * dd + 1][k][i], dk[4 * dd + 2][k][i], dk[4 * dd + 3][k][i]};
                        f32x4 y = {dv[4 * dd][k][i], dv[4 * dd + 1][k][i], dv[4 * dd + 2][k][i], dv[4 * dd + 3][k][i]};
                        if (ww > 0) {
                            x += lds4(pk);
                            y += lds4(pv);
                        }
                        to_lds4(pk, x);
                        to_lds4(pv, y);
                    }
    }
    __syncthreads();
    float* out = sums + ((bg * nC + c) * nsplit + split) * (size_t)SL::n;
    for (int e = tid; e < 2 * kChunk * D / 4; e += kThreads) {
        const int m = e / (kChunk * D / 4), r = e % (kChunk * D / 4) / (D / 4), d4 = (e % (D / 4)) * 4;
        st4(out + (m ? SL::dv : SL::dk) + r * D + d4, lds4(&s_kv[m][r][d4]));
    }
    for (int e = tid; e < G * D + G; e += kThreads) {
        float x = 0.f;
        for (int i = 0; i < kW; ++i) x += e < G * D ? s_dl[i][e / D][e % D] : s_db[i][e - G * D];
        out[SL::dl + e] = x;
    }
}

// The blocks' sums of every chunk, added in order and written as dk, dv, dk', db'.
template <int D, int G>
__global__ __launch_bounds__(kThreads) void k_bwd_sum_f32(BwdArgs a, const float* sums, int nsplit) {
    using SL = SumLayout<D, G>;
    constexpr int per = SL::n / 4, blocks = (per + kThreads - 1) / kThreads;  // blocks per chunk
    const int nC = a.L / kChunk, e = (blockIdx.x % blocks) * kThreads + threadIdx.x;
    const int c = blockIdx.x / blocks, g = blockIdx.y, b = blockIdx.z;
    const size_t bg = (size_t)b * a.Hkv + g, bc = bg * nC + c;
    if (e >= per) return;
    const float* src = sums + bc * nsplit * (size_t)SL::n + 4 * e;
    f32x4 x = zero4();
    for (int i = 0; i < nsplit; ++i) x += ld4(src + (size_t)i * SL::n);
    const int o = 4 * e;
    const bool per_head = a.Hl == a.Hq;
    if (o < SL::dv) {
        st4(as_mut<float>(a.dk) + (bg * a.L + (size_t)c * kChunk) * D + o, x * a.scale);
    } else if (o < SL::dl) {
        st4(as_mut<float>(a.dv) + (bg * a.L + (size_t)c * kChunk) * D + o - SL::dv, x);
    } else if (o < SL::db) {
        const int h = (o - SL::dl) / D, d = (o - SL::dl) % D;
        if (per_head) {
            st4(as_mut<float>(a.dlmk) + (((size_t)b * a.Hl + g * G + h) * nC + c) * D + d, x * a.scale);
        } else if (h == 0) {  // one landmark for the group: the heads' sums together
            for (int hh = 1; hh < G; ++hh)
                for (int i = 0; i < nsplit; ++i) x += ld4(src + (size_t)i * SL::n + hh * D);
            st4(as_mut<float>(a.dlmk) + (((size_t)b * a.Hl + g) * nC + c) * D + d, x * a.scale);
        }
    } else if (a.dbias && o == SL::db) {
        for (int h = 0; h < G; ++h) {
            float y = 0.f;
            for (int i = 0; i < nsplit; ++i) y += src[(size_t)i * SL::n + h];
            if (per_head)
                a.dbias[((size_t)b * a.Hl + g * G + h) * nC + c] = y;
            else
                x[0] = h ? x[0] + y : y;
        }
        if (!per_head) a.dbias[((size_t)b * a.Hl + g) * nC + c] = x[0];
    }
}

// Blocks per chunk of the key-major pass: enough for two blocks on each of the 256 CUs,
// but no more than give every wave a tile of the window's rows, and at most 16 (the sums
// of a block take 64 x 2 d floats).
int key_splits_most(int G, int N, int W) {
    const int rows = (int)std::min<long>(N, (long)kChunk + W);
    return std::max(1, std::min(16, rows * G / (kCols * kW)));
}
int key_splits(size_t chunks, int most) {
    return (int)std::min<size_t>(most, std::max<size_t>(1, 512 / chunks));
}

struct F32Layout {
    size_t u, sorted, sums, inv_base;
    InvLayout inv;
    int nsplit;
    size_t total;
};
F32Layout f32_layout(int B, int Hq, int Hkv, int N, int L, int d, int K, int W) {
    F32Layout w;
    const int G = Hq / Hkv;
    const size_t chunks = (size_t)B * Hkv * (L / kChunk);
    const int most = key_splits_most(G, N, W);
    w.nsplit = key_splits(chunks, most);
    // (chunks * nsplit blocks at most, and a bound that never falls as the call grows: a
    // workspace of the largest call serves every smaller one)
    const size_t blocks = std::max(chunks, std::min<size_t>(512, chunks * most));
    w.u = 0;
    w.sorted = align256(w.u + (size_t)B * Hq * N * sizeof(float));
    w.sums = align256(w.sorted + (size_t)B * Hkv * N * K * sizeof(int));
    const size_t n = ((size_t)(2 * kChunk + G) * d + G + 3) / 4 * 4;
    w.inv_base = align256(w.sums + blocks * n * sizeof(float));
    w.inv = inv_layout(B, Hkv, N, L, K, w.inv_base);
    w.total = w.inv.end;
    return w;
}

struct AttnRun {
    template <int D, int G>
    static hipError_t run(const FwdArgs& a, hipStream_t s) {
        constexpr int NQ = kCols / G;
        HILS_LAUNCH("k_attn_f32", (k_attn_f32<D, G>), dim3((a.N + NQ - 1) / NQ, a.Hkv, a.B), dim3(kAttnW * kWave), 0, s,
                    a);
        return hipGetLastError();
    }
};

struct BwdRun {
    template <int D, int G>
    static hipError_t run(const BwdArgs& a, hipStream_t s) {
        constexpr int NQ = kCols / G;
        using SL = SumLayout<D, G>;
        const F32Layout ly = f32_layout(a.B, a.Hq, a.Hkv, a.N, a.L, D, a.K, a.W);
        char* ws = static_cast<char*>(a.ws);
        float* u = reinterpret_cast<float*>(ws + ly.u);
        float* sums = reinterpret_cast<float*>(ws + ly.sums);
        int* sorted = reinterpret_cast<int*>(ws + ly.sorted);
        const int nC = a.L / kChunk;
        // Sequences so short that no row has a candidate need no index: 1 to 6 tokens took 37 to
        // 58 us with its four launches, 24 to 49 by the kernels
        // of one block per row; without them 30 (d = 64) and 46 to 54 (d = 128).
        const bool retrieves = n_candidates(a.N - 1, a.W) > 0;
        const int* offsets = retrieves ? reinterpret_cast<const int*>(ws + ly.inv.offsets) : nullptr;
        HILS_LAUNCH("k_bwd_dq_f32", (k_bwd_dq_f32<D, G>), dim3((a.N + NQ - 1) / NQ, a.Hkv, a.B), dim3(kThreads), 0, s,
                    a, u, reinterpret_cast<int*>(ws + ly.inv.counts),
                    retrieves ? inv_count_words(a.B, a.Hkv, a.L, ly.inv) : 0);
        if (retrieves) {
            const InvArgs ia{a.idx, a.B, a.Hkv, a.N, a.K, a.W, a.L, 0, a.N};
            launch_inverse_index(ia, ly.inv, a.ws, s, false, true);
            launch_inv_sort(ia, ly.inv, a.ws, sorted, s);
        }
        HILS_LAUNCH("k_bwd_keys_f32", (k_bwd_keys_f32<D, G>), dim3(nC * ly.nsplit, a.Hkv, a.B), dim3(kThreads), 0, s,
                    a, offsets, (const int*)sorted, (const float*)u, sums, ly.nsplit);
        HILS_LAUNCH("k_bwd_sum_f32", (k_bwd_sum_f32<D, G>), dim3((SL::n / 4 + kThreads - 1) / kThreads * nC, a.Hkv, a.B),
                    dim3(kThreads), 0, s, a, (const float*)sums, ly.nsplit);
        return hipGetLastError();
    }
};

}  // namespace

size_t bwd_f32_workspace_bytes(int B, int Hq, int Hkv, int N, int L, int d, int K, int W) {
    return f32_layout(B, Hq, Hkv, N, L, d, K, W).total;
}

hipError_t launch_attn_f32(const FwdArgs& a, hipStream_t s) { return dispatch_f32<AttnRun>(a.d, a.Hq / a.Hkv, a, s); }

hipError_t launch_bwd_f32(const BwdArgs& a, hipStream_t s) { return dispatch_f32<BwdRun>(a.d, a.Hq / a.Hkv, a, s); }

}  // namespace hils
