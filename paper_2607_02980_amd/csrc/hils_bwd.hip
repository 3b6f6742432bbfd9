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
constexpr int kInvRows = 128;
static_assert(kInvBucketRows % kInvRows == 0, "a block of rows lies in one bucket");
static_assert(kInvRows % 128 == 0 && kInvRows <= 32 * 16, "tiles of 16 to 128 rows do not straddle blocks");

// The entries of rows n0 .. n0 + rows - 1, kPer per thread and round with their loads in
// flight together: f(chunk, entry, gap) for the valid ones; gap: the entry before it in
// the row is not one.
template <typename F>
__device__ __forceinline__ void for_entries(const InvArgs& a, int bg, int n0, int rows, F&& f) {
    constexpr int kPer = 4;
    const int32_t* idx = a.idx + ((size_t)bg * a.Nrow + a.n0 + n0) * a.K;
    const int total = rows * a.K;
    for (int e0 = threadIdx.x; e0 < total; e0 += kPer * kBlock) {
        int c[kPer], before[kPer], before2[kPer];
#pragma unroll
        for (int t = 0; t < kPer; ++t) {
            const int e = min(e0 + t * kBlock, total - 1);
            c[t] = idx[e];
            before[t] = idx[max(e - 1, 0)];
            before2[t] = idx[max(e - 2, 0)];
        }
#pragma unroll
        for (int t = 0; t < kPer; ++t) {
            const int e = e0 + t * kBlock;
            if (e >= total) break;
            // (as idx_entry_valid)
            const int n = n0 + e / a.K, slot = e % a.K;
            const int nc = n_candidates(a.n0 + n, a.W);
            if (c[t] >= 0 && c[t] < nc && (slot == 0 || c[t] > before[t]))
                f(c[t], (n << 6) | slot,
                  slot > 0 && !(before[t] >= 0 && before[t] < nc && (slot == 1 || before[t] > before2[t])));
        }
    }
}

// grid (ceil(N / kInvRows), B*Hkv); counts [bg][nR][nC] (a block's counters are
// contiguous: one bucket)
__global__ __launch_bounds__(kBlock) void k_inv_count(InvArgs a, int nR, int brows, int* counts) {
    __shared__ int s_hist[kInvHist];
    const int bg = blockIdx.y, n0 = blockIdx.x * kInvRows, tid = threadIdx.x;
    const int nC = a.L / kChunk, R = n0 / brows;
    const bool lds = nC <= kInvHist;
    int* gcnt = counts + (size_t)bg * nC * nR + (size_t)R * nC;
    const int rows = min(kInvRows, a.N - n0);
    __shared__ unsigned s_uni, s_gap;  // bit t: tile t of the block is flagged; has a row with gaps
    if (tid == 0) s_uni = s_gap = 0u;
    if (a.flags) {
        // the unions of the block's tiles: their chunks' bitmaps in the histogram's place,
        // as many tiles at once as fit
        const int ntile = (rows + a.QT - 1) / a.QT, nw = (nC + 31) / 32, fit = min(ntile, kInvHist / nw);
        for (int t0 = 0; t0 < ntile; t0 += fit) {
            __syncthreads();
            for (int i = tid; i < fit * nw; i += kBlock) s_hist[i] = 0;
            __syncthreads();
            for_entries(a, bg, n0, rows, [&](int c, int ent, bool gap) {
                const int t = ((ent >> 6) - n0) / a.QT - t0;
                if (t >= 0 && t < fit) atomicOr(&s_hist[t * nw + (c >> 5)], 1 << (c & 31));
                if (gap && t >= 0 && t < fit) atomicOr(&s_gap, 1u << (t0 + t));
            });
            __syncthreads();
            for (int t = tid / kWave; t < fit && t0 + t < ntile; t += kBlock / kWave) {
                int u = 0;
                for (int i = tid % kWave; i < nw; i += kWave) u += __popc((unsigned)s_hist[t * nw + i]);
#pragma unroll
                for (int o = 32; o >= 1; o >>= 1) u += __shfl_xor(u, o, kWave);
                if (tid % kWave == 0) {
                    const bool f = u <= a.umax && !(s_gap >> (t0 + t) & 1u);
                    if (f) atomicOr(&s_uni, 1u << (t0 + t));
                    a.flags[(size_t)bg * ((a.N + a.QT - 1) / a.QT) + n0 / a.QT + t0 + t] = f;
                }
            }
        }
        __syncthreads();
    }
    if (lds)
        for (int c = tid; c < nC; c += kBlock) s_hist[c] = 0;
    __syncthreads();
    const unsigned uni = s_uni;
    for_entries(a, bg, n0, rows, [&](int c, int ent, bool) {
        if (uni && (uni >> (((ent >> 6) - n0) / a.QT) & 1u)) return;
        if (lds)
            atomicAdd(&s_hist[c], 1);
        else
            atomicAdd(&gcnt[c], 1);
    });
    __syncthreads();
    if (lds)
        for (int c = tid; c < nC; c += kBlock)
            if (s_hist[c]) atomicAdd(&gcnt[c], s_hist[c]);
}

// cursor [bg][nR][nC]: the next free list position of every (bucket, chunk)
__global__ __launch_bounds__(kBlock) void k_inv_fill(InvArgs a, int nR, int brows, int* cursor, int* list) {
    __shared__ int s_hist[kInvHist];
    const int bg = blockIdx.y, n0 = blockIdx.x * kInvRows, tid = threadIdx.x;
    const int nC = a.L / kChunk, R = n0 / brows;
    const bool lds = nC <= kInvHist;
    int* gcur = cursor + (size_t)bg * nC * nR + (size_t)R * nC;
    int* lst = list + (size_t)bg * a.N * a.K;
    const int rows = min(kInvRows, a.N - n0);
    unsigned uni = 0u;  // bit t: tile t of the block is flagged, its rows left out
    if (a.flags)
        for (int t = 0; t * a.QT < rows; ++t)
            uni |= (unsigned)(a.flags[(size_t)bg * ((a.N + a.QT - 1) / a.QT) + n0 / a.QT + t] != 0) << t;
    auto left_out = [&](int ent) { return uni && (uni >> (((ent >> 6) - n0) / a.QT) & 1u); };
    if (lds) {
        for (int c = tid; c < nC; c += kBlock) s_hist[c] = 0;
        __syncthreads();
        for_entries(a, bg, n0, rows, [&](int c, int ent, bool) {
            if (!left_out(ent)) atomicAdd(&s_hist[c], 1);
        });
        __syncthreads();
        // reserve this block's range of every chunk it touches; s_hist becomes the running position
        for (int c = tid; c < nC; c += kBlock)
            if (s_hist[c]) s_hist[c] = atomicAdd(&gcur[c], s_hist[c]);
        __syncthreads();
    }
    for_entries(a, bg, n0, rows, [&](int c, int ent, bool) {
        if (left_out(ent)) return;
        const int pos = lds ? atomicAdd(&s_hist[c], 1) : atomicAdd(&gcur[c], 1);
        lst[pos] = ent;
    });
}

// Exclusive prefix sum of one int per thread over a kScan-thread block (wave
// scans by shuffles, then the wave totals); every thread gets the block total.
// Contains barriers: called by every thread of the block.
constexpr int kScan = 1024;
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
    for (int i = 0; i < kScan / kWave; ++i) {
        const int t = s_wave[i];
        before += i < w ? t : 0;
        all += t;
    }
    __syncthreads();  // s_wave may be reused by the caller
    *total = all;
    return before + incl - x;
}

// One block per (b, g): from the nR x nC counts, in chunk-major order, the sub-lists'
// starts boff[nC * nR + 1] and each chunk's whole list offsets[nC + 1]; in the counts' own
// bucket-major order the fill's cursors and (work != null) the work items, one block of the
// chunk pass each: the (chunk, bucket) sub-lists cut into segments of kInvSeg entries, so
// that the items in flight together work on one range of rows.  Both orders read the
// counts from LDS while they fit (48 KB: 12288 of them; two launches of 256 threads
// striding through global memory took 43 us at 8192 counts, 32K tokens).
constexpr int kScanCounts = 12288;
__global__ __launch_bounds__(kScan) void k_inv_scan(const int* counts, int* boff, int* offsets, int* cursor, int nC,
                                                    int nR, size_t max_work_bg, int4* work, int* nwork) {
    extern __shared__ int s_cnt[];
    __shared__ int s_part[kScan / kWave];
    const int bg = blockIdx.x, tid = threadIdx.x;
    const int M = nC * nR;
    const int* cnt = counts + (size_t)bg * M;
    int* bo = boff + (size_t)bg * (M + 1);
    int* off = offsets + (size_t)bg * (nC + 1);
    int* cur = cursor + (size_t)bg * M;
    if (M <= kScanCounts) {
        for (int i = tid; i < M; i += kScan) s_cnt[i] = cnt[i];
        __syncthreads();
        cnt = s_cnt;
    }
    const int per = (M + kScan - 1) / kScan;
    const int lo = min(M, tid * per), hi = min(M, lo + per);
    int total, sum = 0;
    for (int i = lo; i < hi; ++i) sum += cnt[(i % nR) * nC + i / nR];  // i = c * nR + R
    int run = block_exclusive_scan(sum, s_part, &total);
    if (tid == 0) {
        bo[M] = total;
        off[nC] = total;
    }
    for (int i = lo; i < hi; ++i) {
        const int c = i / nR, j = (i % nR) * nC + c;
        bo[i] = run;
        cur[j] = run;
        if (i % nR == 0) off[c] = run;
        run += cnt[j];
    }
    if (!work) return;
    int4* wk = work + (size_t)bg * max_work_bg;
    sum = 0;
    for (int i = lo; i < hi; ++i) sum += (cnt[i] + kInvSeg - 1) / kInvSeg;  // i = R * nC + c
    run = block_exclusive_scan(sum, s_part, &total);
    if (tid == 0) nwork[bg] = total;
    for (int i = lo; i < hi; ++i) {
        const int ns = (cnt[i] + kInvSeg - 1) / kInvSeg;
        for (int sgi = 0; sgi < ns; ++sgi) wk[run + sgi] = make_int4(i / nC, i % nC, sgi, 0);
        run += ns;
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

void launch_inverse_index(const InvArgs& a, const InvLayout& w, void* ws, hipStream_t s, bool work_list, bool cleared) {
    char* base = static_cast<char*>(ws);
    int* counts = reinterpret_cast<int*>(base + w.counts);
    int* offsets = reinterpret_cast<int*>(base + w.offsets);
    int* boff = reinterpret_cast<int*>(base + w.boff);
    int* cursor = reinterpret_cast<int*>(base + w.cursor);
    int* list = reinterpret_cast<int*>(base + w.list);
    const int nC = a.L / kChunk;
    const dim3 grows((a.N + kInvRows - 1) / kInvRows, a.B * a.Hkv);
    if (!cleared) {
        const size_t ncnt = inv_count_words(a.B, a.Hkv, a.L, w);
        HILS_LAUNCH("k_fill_i32", k_fill_i32, dim3((unsigned)((ncnt + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, counts,
                    ncnt, 0);
    }
    HILS_LAUNCH("k_inv_count", k_inv_count, grows, dim3(kBlock), 0, s, a, w.nR, w.brows, counts);
    const size_t M = (size_t)nC * w.nR;
    HILS_LAUNCH("k_inv_scan", k_inv_scan, dim3(a.B * a.Hkv), dim3(kScan), M <= kScanCounts ? M * sizeof(int) : 0, s,
                (const int*)counts, boff, offsets, cursor, nC, w.nR, w.max_work_bg,
                work_list ? reinterpret_cast<int4*>(base + w.work) : nullptr, reinterpret_cast<int*>(base + w.nwork));
    HILS_LAUNCH("k_inv_fill", k_inv_fill, grows, dim3(kBlock), 0, s, a, w.nR, w.brows, cursor, list);
}

hipError_t launch_bwd(const BwdArgs& a, hipStream_t s) { return a.bf16 ? launch_bwd_mfma(a, s) : launch_bwd_f32(a, s); }

}  // namespace hils
