// Layout of the decode workspace, shared by the kernels and the host.
#pragma once

#include <algorithm>

#include "../../include/hils.h"
#include "hils_device.hpp"
#include "hils_internal.hpp"

namespace hils {

constexpr int kSlice = 256;       // candidate chunks per scan workgroup, at most
constexpr int kMaxLocalPieces = 64;  // local window pieces per row (W <= 4032)

struct DecLayout {
    int nC, nslices, nlocal, nparts;  // nparts = K + nlocal records per (b, g)
    int slice;                        // candidate chunks per scan workgroup
    int mq_umax;                      // union chunks per multi-query workgroup (at most)
    int hn_words;                     // 4-byte words of one (row, slice) record of hn
    size_t cand, parts, lse, mq, hn, total;  // byte offsets
};

inline int local_pieces_max(int W) { return (W + 62) / 64 + 1; }

// R = B * N rows; with N > 1 also the records of the multi-query pass
// (k_dec_mq: per workgroup mq_umax union chunks x 16 tile rows); under the per-head
// normalised ranking (HN) also, per (row, slice), the union of the G heads' top-K
// chunks of the slice by raw score: its size, ids and G raw scores each.
inline DecLayout dec_layout(int B, int N, int Hkv, int G, int d, int L, int K, int W, int HN,
                            bool shared = false) {
    const int R = B * N;
    DecLayout o;
    o.nC = L / kChunk;
    o.nlocal = local_pieces_max(W);
    o.nparts = K + o.nlocal;
    const size_t bg = (size_t)R * Hkv;
    const int nq = 16 / G < 8 ? 16 / G : 8;  // queries per multi-query workgroup
    o.mq_umax = nq * K + o.nlocal + 1;
    const size_t mq_groups = N > 1 ? (size_t)B * ((N + nq - 1) / nq) * Hkv : 0;
    o.hn_words = (1 + G * K * (1 + G) + 3) & ~3;
    const size_t parts = (bg * o.nparts * G * (4 + d) * 4 + 255) & ~(size_t)255;
    const size_t mq = (mq_groups * o.mq_umax * 16 * (4 + d) * 4 + 255) & ~(size_t)255;
    auto cand = [&](int slice) { return (bg * ((o.nC + slice - 1) / slice) * K * 8 + 255) & ~(size_t)255; };
    // Slices of 256 chunks, halved to 128 or 64 while fewer than 4 workgroups per CU would
    // scan (a wave keeps at most 16 KB of landmarks in flight, and a ragged batch leaves
    // many slices empty), the row's survivors stay within one selection of a wave (4 per
    // lane) and the workspace within the fixed array of the call without one.  Scan of 8
    // sequences of 64K, 4 new tokens: 28.6 us with 256 workgroups of 256 chunks.  With one
    // landmark head per KV group a slice's read is a quarter or less and its selection is
    // not, so one workgroup per CU is enough (steps with 1024 and 256, shared landmarks: 16
    // sequences of 100K, d = 64, 39.1 and 35.2 us; 24 of 60K, d = 128, 46.9 and 43.4; 8 of
    // 100K 31.1 and 30.7).
    o.slice = kSlice;
    const long sgroups = (long)B * ((N + 3) / 4) * Hkv, full = shared && N == 1 ? 256 : 1024;
    while (!HN && o.slice > 64 && sgroups * ((o.nC + o.slice - 1) / o.slice) < full &&
           (o.nC + o.slice / 2 - 1) / (o.slice / 2) * K <= 4 * kWave &&
           cand(o.slice / 2) + parts + mq <= HILS_DECODE_NOALLOC_SCRATCH_BYTES)
        o.slice /= 2;
    o.nslices = (o.nC + o.slice - 1) / o.slice;
    o.cand = 0;
    o.parts = cand(o.slice);
    // per-head (max, sum of exp) of each slice's scores, for the normalised ranking
    o.lse = o.parts + parts;
    o.mq = o.lse + (HN ? (bg * o.nslices * G * 2 * 4 + 255) & ~(size_t)255 : 0);
    o.hn = o.mq + mq;
    o.total = o.hn + (HN ? ((bg * o.nslices * o.hn_words * 4 + 255) & ~(size_t)255) : 0);
    // The size never falls as B, N or L grow, so that a workspace of the largest call serves
    // every smaller one, whichever slices it takes: room for the survivors of 64-chunk slices
    // up to 4 * kWave per row (the limit above) where that stays within the fixed array, and
    // never less than the slices of 256 need.
    const size_t most = std::min<size_t>((size_t)((o.nC + 63) / 64) * K, 4 * kWave);
    const size_t coarse = cand(kSlice) + parts + mq;
    const size_t fine = std::max(cand(kSlice), (bg * most * 8 + 255) & ~(size_t)255) + parts + mq;
    o.total = std::max({o.total, coarse, std::min<size_t>(fine, HILS_DECODE_NOALLOC_SCRATCH_BYTES)});
    return o;
}

}  // namespace hils
