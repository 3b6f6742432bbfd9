// HiLS attention prefill forward, fp32 storage, gfx950 (the bf16 path runs on
// MFMA in hils_prefill.hip).
//
// One wavefront scores and selects for one (b, KV group, query) row; the attention
// over the selection is in hils_f32.hip.
#include "hils_device.hpp"
#include "hils_dispatch.hpp"
#include "hils_internal.hpp"

namespace hils {

constexpr int kBlock = 256;
constexpr int kSlice = 1024;  // candidates scored per selection round of one wave

// ---------------------------------------------------------------------------
// Landmark scoring + group max + top-K (Eq. (9), Sec. 4.1 / App. C).
// Grid: ceil(rows / 4) blocks of 4 waves; wave w owns row blockIdx.x*4 + w,
// rows ordered (b, g, n).  The candidates C_i are scored in slices of kSlice;
// each slice is merged with the running top-K by an exact wave radix select.
// ---------------------------------------------------------------------------
template <typename T, int D, int G>
__global__ __launch_bounds__(kBlock) void k_score_topk_rows(FwdArgs a) {
    __shared__ float s_q[4][G][D];
    __shared__ float s_sc[4][kSlice + 64];
    __shared__ int s_id[4][kSlice + 64];
    __shared__ int s_bid[4][64];
    __shared__ float s_bsc[4][64];
    __shared__ int s_tid[4][64];
    __shared__ float s_tsc[4][64];

    const int wave = wave_id(), lane = threadIdx.x % kWave;
    const long row = (long)blockIdx.x * 4 + wave;
    if (row >= (long)a.B * a.Hkv * a.N) return;  // whole wave leaves; no block barriers below
    const int n = (int)(row % a.N);
    const int g = (int)((row / a.N) % a.Hkv);
    const int b = (int)(row / ((long)a.N * a.Hkv));
    const int pos = n;
    const int ncand = n_candidates(pos, a.W);
    const int nC = a.L / kChunk;

    const T* qr = as<T>(a.q_route ? a.q_route : a.q);
    for (int e = lane; e < G * D; e += kWave) {
        const int hh = e / D, dd = e % D;
        s_q[wave][hh][dd] = to_f32(qr[(((size_t)b * a.Hq + g * G + hh) * a.N + n) * D + dd]);
    }
    __builtin_amdgcn_wave_barrier();

    // s^ of head hh for chunk c (Eq. (9) with Eq. (11))
    auto score = [&](int hh, int c) {
        const int hl = (a.Hl == a.Hq) ? g * G + hh : g;
        const T* lr = as<T>(a.lmk) + (((size_t)b * a.Hl + hl) * nC + c) * D;
        float acc = 0.f;
#pragma unroll 4
        for (int dd = 0; dd < D; dd += 8) {
            float x[8];
            load8(lr + dd, x);
#pragma unroll
            for (int t = 0; t < 8; ++t) acc += s_q[wave][hh][dd + t] * x[t];
        }
        float sv = a.scale * acc;
        if (a.bias) sv += a.bias[((size_t)b * a.Hl + hl) * nC + c];
        return sv;
    };
    // per-head normalised ranking: each head's log-sum-exp over C_i first
    float lse[G];
#pragma unroll
    for (int hh = 0; hh < G; ++hh) lse[hh] = 0.f;
    if (a.head_norm && ncand > 0) {
#pragma unroll 1
        for (int hh = 0; hh < G; ++hh) {
            float m = -INFINITY, sum = 0.f;
            for (int c = lane; c < ncand; c += kWave) {
                const float sv = score(hh, c);
                const float nm = fmaxf(m, sv);
                sum = sum * fexp(m - nm) + fexp(sv - nm);
                m = nm;
            }
            const float M = wave_max(m);
            const float S = wave_sum(m == -INFINITY ? 0.f : sum * fexp(m - M));
            lse[hh] = M + __logf(S);
        }
    }

    int nbest = 0;
    for (int s0 = 0; s0 < ncand; s0 += kSlice) {
        const int len = min(kSlice, ncand - s0);
        for (int e = lane; e < len; e += kWave) {
            const int c = s0 + e;
            float best = -INFINITY;
#pragma unroll
            for (int hh = 0; hh < G; ++hh) best = fmaxf(best, score(hh, c) - lse[hh]);
            s_sc[wave][e] = best;
            s_id[wave][e] = c;
        }
        for (int t = lane; t < nbest; t += kWave) {
            s_sc[wave][len + t] = s_bsc[wave][t];
            s_id[wave][len + t] = s_bid[wave][t];
        }
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        nbest = wave_topk(s_sc[wave], s_id[wave], len + nbest, a.K, s_bid[wave], s_bsc[wave], s_tid[wave],
                          s_tsc[wave]);
    }
    int32_t* orow = a.idx + (((size_t)b * a.Hkv + g) * a.N + n) * a.K;
    for (int t = lane; t < a.K; t += kWave) orow[t] = t < nbest ? s_bid[wave][t] : -1;
}

struct ScoreRun {
    template <int D, int G>
    static hipError_t run(const FwdArgs& a, hipStream_t s) {
        const long rows = (long)a.B * a.Hkv * a.N;
        HILS_LAUNCH("k_score_topk_rows", (k_score_topk_rows<float, D, G>), dim3((unsigned)((rows + 3) / 4)),
                    dim3(kBlock), 0, s, a);
        return hipGetLastError();
    }
};

hipError_t launch_prefill_rows(const FwdArgs& a, hipStream_t s) {
    if (!a.given_idx) {
        const hipError_t e = dispatch_f32<ScoreRun>(a.d, a.Hq / a.Hkv, a, s);
        if (e != hipSuccess) return e;
    }
    return launch_attn_f32(a, s);
}

}  // namespace hils
