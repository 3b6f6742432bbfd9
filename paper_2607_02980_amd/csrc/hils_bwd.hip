// The gradient of HiLS attention, and the inverse index that the backward and the bf16
// prefill share, gfx950.  (The kernels of the backward are in hils_bwd_mfma.hip, bf16
// storage, and hils_f32.hip.)
//
// With g = dO and u = g . out for a (row, head), and L its fusion LSE:
//   local key j:     w_j = exp(s_j - L);  dv_j += w_j g;  ds_j = w_j (g.v_j - u)
//   chunk c, key j:  p_j = exp(s_j - log Z_c), a_c = exp(s^_c - L), u_c = g . o_c
//                    dv_j += a_c p_j g;  ds_j = a_c p_j (g.v_j - u_c)
//   retrieval score: ds^_c = a_c (u_c - u)
//   dq += scale ds_j k_j;  dk_j += scale ds_j q;  dq^ += scale ds^_c k'_c;
//   dk'_c += scale ds^_c q^;  db'_c += ds^_c
// (Eq. (10) differentiated with the selection fixed; selection gets no gradient.)
//
// Inverse index (k_inv_*): for each (b, group, chunk) the rows that selected it.
#include "hils_device.hpp"
#include "hils_dispatch.hpp"
#include "hils_internal.hpp"

namespace hils {

constexpr int kBlock = 256;

// ---------------------------------------------------------------------------
// Inverse index: (b, g, c) -> rows n whose selection holds c.
// ---------------------------------------------------------------------------
__global__ void k_fill_i32(int* p, size_t n, int v) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// Entries are processed per (b, g) in blocks of kInvRows rows; a block first
// counts its entries per chunk in LDS and then touches each global counter
// once, so global atomics scale with (blocks x chunks touched), not entries.
// Counters are kept per (chunk, row bucket): every list is the concatenation of
// its buckets' sub-lists in bucket order, so a consumer can take the entries of
// one chunk that fall in one range of rows (the chunk pass walks the buckets in
// order, so the query rows it gathers stay in L2).
// List entries are (n << 6) | slot (slot < K <= 64).
constexpr int kInvRows = 256;
constexpr int kInvHist = 8192;  // chunks counted in LDS; larger L falls back to global atomics
static_assert(kInvBucketRows % kInvRows == 0, "a block of rows lies in one bucket");

// (n: the row relative to a.n0)
__device__ __forceinline__ bool entry_valid(const InvArgs& a, const int32_t* irow, int slot, int n, int* c) {
    if (!idx_entry_valid(irow, slot, n_candidates(a.n0 + n, a.W))) return false;
    *c = irow[slot];
    return true;
}

// grid (ceil(N / kInvRows), B*Hkv); counts [bg][nR][nC] (a block's counters are
// contiguous: one bucket)
__global__ __launch_bounds__(kBlock) void k_inv_count(InvArgs a, int nR, int brows, int* counts) {
    __shared__ int s_hist[kInvHist];
    const int bg = blockIdx.y, n0 = blockIdx.x * kInvRows, tid = threadIdx.x;
    const int nC = a.L / kChunk, R = n0 / brows;
    const bool lds = nC <= kInvHist;
    int* gcnt = counts + (size_t)bg * nC * nR;
    if (lds)
        for (int c = tid; c < nC; c += kBlock) s_hist[c] = 0;
    __syncthreads();
    const int rows = min(kInvRows, a.N - n0);
    for (int e = tid; e < rows * a.K; e += kBlock) {
        const int n = n0 + e / a.K, slot = e % a.K;
        const int32_t* irow = a.idx + ((size_t)bg * a.Nrow + a.n0 + n) * a.K;
        int c;
        if (!entry_valid(a, irow, slot, n, &c)) continue;
        if (lds)
            atomicAdd(&s_hist[c], 1);
        else
            atomicAdd(&gcnt[R * nC + c], 1);
    }
    __syncthreads();
    if (lds)
        for (int c = tid; c < nC; c += kBlock)
            if (s_hist[c]) atomicAdd(&gcnt[R * nC + c], s_hist[c]);
}

__global__ __launch_bounds__(kBlock) void k_inv_fill(InvArgs a, int nR, int brows, const int* boff, int* cursor,
                                                     int* list) {
    __shared__ int s_hist[kInvHist];
    const int bg = blockIdx.y, n0 = blockIdx.x * kInvRows, tid = threadIdx.x;
    const int nC = a.L / kChunk, R = n0 / brows;
    const bool lds = nC <= kInvHist;
    int* gcur = cursor + (size_t)bg * nC * nR;
    const int* off = boff + (size_t)bg * (nC * nR + 1);
    int* lst = list + (size_t)bg * a.N * a.K;
    const int rows = min(kInvRows, a.N - n0);
    if (lds) {
        for (int c = tid; c < nC; c += kBlock) s_hist[c] = 0;
        __syncthreads();
        for (int e = tid; e < rows * a.K; e += kBlock) {
            const int n = n0 + e / a.K, slot = e % a.K;
            int c;
            if (entry_valid(a, a.idx + ((size_t)bg * a.Nrow + a.n0 + n) * a.K, slot, n, &c)) atomicAdd(&s_hist[c], 1);
        }
        __syncthreads();
        // reserve this block's range of every chunk it touches; s_hist becomes the running position
        for (int c = tid; c < nC; c += kBlock)
            if (s_hist[c]) s_hist[c] = off[c * nR + R] + atomicAdd(&gcur[R * nC + c], s_hist[c]);
        __syncthreads();
    }
    for (int e = tid; e < rows * a.K; e += kBlock) {
        const int n = n0 + e / a.K, slot = e % a.K;
        int c;
        if (!entry_valid(a, a.idx + ((size_t)bg * a.Nrow + a.n0 + n) * a.K, slot, n, &c)) continue;
        const int pos = lds ? atomicAdd(&s_hist[c], 1) : off[c * nR + R] + atomicAdd(&gcur[R * nC + c], 1);
        lst[pos] = (n << 6) | slot;
    }
}

// Exclusive prefix sum of one int per thread over a kBlock-thread block (wave
// scans by shuffles, then the wave totals); every thread gets the block total.
// Contains barriers: called by every thread of the block.
__device__ __forceinline__ int block_exclusive_scan(int x, int* s_wave, int* total) {
    const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave;
    int incl = x;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const int y = __shfl_up(incl, o, kWave);
        if (lane >= o) incl += y;
    }
    if (lane == kWave - 1) s_wave[w] = incl;
    __syncthreads();
    int before = 0, all = 0;
#pragma unroll
    for (int i = 0; i < kBlock / kWave; ++i) {
        const int t = s_wave[i];
        before += i < w ? t : 0;
        all += t;
    }
    __syncthreads();  // s_wave may be reused by the caller
    *total = all;
    return before + incl - x;
}

// one block per (b, g): exclusive scan of the nR x nC counts in chunk-major order
// into boff[nC * nR + 1], and each chunk's whole list into offsets[nC + 1]
__global__ __launch_bounds__(kBlock) void k_inv_scan(const int* counts, int* boff, int* offsets, int nC, int nR) {
    __shared__ int s_part[kBlock / kWave];
    const int bg = blockIdx.x, tid = threadIdx.x;
    const int M = nC * nR;
    const int per = (M + kBlock - 1) / kBlock;
    const int lo = min(M, tid * per), hi = min(M, lo + per);
    const int* cnt = counts + (size_t)bg * M;
    int* bo = boff + (size_t)bg * (M + 1);
    int* off = offsets + (size_t)bg * (nC + 1);
    int sum = 0;
    auto count = [&](int i) { return cnt[(i % nR) * nC + i / nR]; };  // i = c * nR + R
    for (int i = lo; i < hi; ++i) sum += count(i);
    int total;
    int run = block_exclusive_scan(sum, s_part, &total);
    if (tid == 0) {
        bo[M] = total;
        off[nC] = total;
    }
    for (int i = lo; i < hi; ++i) {
        bo[i] = run;
        if (i % nR == 0) off[i / nR] = run;
        run += count(i);
    }
}

InvLayout inv_layout(int B, int Hkv, int N, int L, int K, size_t base, int row_end) {
    const size_t bg = (size_t)B * Hkv, nC = (size_t)L / kChunk;
    InvLayout w;
    w.brows = kInvBucketRows;
    while ((size_t)w.brows * K < 64 * nC && w.brows < N) w.brows *= 2;
    w.nR = (N + w.brows - 1) / w.brows;
    const size_t M = nC * (size_t)w.nR;
    w.counts = align256(base);
    w.offsets = align256(w.counts + bg * M * sizeof(int));
    w.boff = align256(w.offsets + bg * (nC + 1) * sizeof(int));
    w.cursor = align256(w.boff + bg * (M + 1) * sizeof(int));
    w.list = align256(w.cursor + bg * M * sizeof(int));
    // A (chunk, bucket) sub-list of len entries makes ceil(len / kInvSeg) <= len / kInvSeg
    // + 1 items, and only the chunks c < n / kChunk of a bucket's last row n can
    // have entries there (a candidate chunk ends before the query): at most
    // (R + 1) * brows / kChunk sub-lists of bucket R are not empty; for a segment of
    // rows that starts later, bucket R's rows lie below row_end, whose candidate
    // chunks number at most row_end / kChunk + 1.
    size_t subl = 0;
    for (int R = 0; R < w.nR; ++R)
        subl += row_end < 0 ? std::min(nC, (size_t)(R + 1) * (w.brows / kChunk))
                            : std::min(nC, (size_t)row_end / kChunk + 1);
    w.max_work_bg = (size_t)N * K / kInvSeg + subl;
    w.work = align256(w.list + bg * (size_t)N * K * sizeof(int));
    w.nwork = align256(w.work + bg * w.max_work_bg * sizeof(int4));
    w.end = align256(w.nwork + bg * sizeof(int));
    return w;
}

// Work items of one (b, g) (one block each): its (chunk, bucket) sub-lists cut into
// segments of kInvSeg entries, bucket-major, so that the items in flight together
// work on one range of rows.
__global__ __launch_bounds__(kBlock) void k_inv_work(const int* boff, int nC, int nR, size_t max_work_bg, int4* work,
                                                     int* nwork) {
    __shared__ int s_part[kBlock / kWave];
    const int bg = blockIdx.x, tid = threadIdx.x;
    const int M = nC * nR;
    const int* bo = boff + (size_t)bg * (M + 1);
    int4* wk = work + (size_t)bg * max_work_bg;
    const int per = (M + kBlock - 1) / kBlock;
    const int lo = min(M, tid * per), hi = min(M, lo + per);
    auto nseg = [&](int i) {  // i = R * nC + c
        const int j = (i % nC) * nR + i / nC;
        return (bo[j + 1] - bo[j] + kInvSeg - 1) / kInvSeg;
    };
    int sum = 0;
    for (int i = lo; i < hi; ++i) sum += nseg(i);
    int total;
    int run = block_exclusive_scan(sum, s_part, &total);
    if (tid == 0) nwork[bg] = total;
    for (int i = lo; i < hi; ++i) {
        const int ns = nseg(i);
        for (int sgi = 0; sgi < ns; ++sgi) wk[run + sgi] = make_int4(i / nC, i % nC, sgi, 0);
        run += ns;
    }
}

void launch_inverse_index(const InvArgs& a, const InvLayout& w, void* ws, hipStream_t s, bool work_list) {
    char* base = static_cast<char*>(ws);
    int* counts = reinterpret_cast<int*>(base + w.counts);
    int* offsets = reinterpret_cast<int*>(base + w.offsets);
    int* boff = reinterpret_cast<int*>(base + w.boff);
    int* cursor = reinterpret_cast<int*>(base + w.cursor);
    int* list = reinterpret_cast<int*>(base + w.list);
    const int nC = a.L / kChunk;
    const size_t ncnt = (size_t)a.B * a.Hkv * nC * w.nR;
    const unsigned gc = (unsigned)((ncnt + kBlock - 1) / kBlock);
    const dim3 grows((a.N + kInvRows - 1) / kInvRows, a.B * a.Hkv);
    HILS_LAUNCH("k_fill_i32", k_fill_i32, dim3(gc), dim3(kBlock), 0, s, counts, ncnt, 0);
    HILS_LAUNCH("k_fill_i32", k_fill_i32, dim3(gc), dim3(kBlock), 0, s, cursor, ncnt, 0);
    HILS_LAUNCH("k_inv_count", k_inv_count, grows, dim3(kBlock), 0, s, a, w.nR, w.brows, counts);
    HILS_LAUNCH("k_inv_scan", k_inv_scan, dim3(a.B * a.Hkv), dim3(kBlock), 0, s, (const int*)counts, boff, offsets,
                nC, w.nR);
    HILS_LAUNCH("k_inv_fill", k_inv_fill, grows, dim3(kBlock), 0, s, a, w.nR, w.brows, (const int*)boff, cursor,
                list);
    if (work_list)
        HILS_LAUNCH("k_inv_work", k_inv_work, dim3(a.B * a.Hkv), dim3(kBlock), 0, s, (const int*)boff, nC, w.nR,
                    w.max_work_bg, reinterpret_cast<int4*>(base + w.work), reinterpret_cast<int*>(base + w.nwork));
}

hipError_t launch_bwd(const BwdArgs& a, hipStream_t s) { return a.bf16 ? launch_bwd_mfma(a, s) : launch_bwd_f32(a, s); }

}  // namespace hils
