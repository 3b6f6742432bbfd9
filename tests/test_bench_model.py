"""The work model behind bench.py's roofline figures, checked against sums written
out row by row (no GPU): the method FLOPs of the chunk pass (QK^T and PV over the
S keys of every selected chunk, 4dS, plus the surrogate score, 2d, per (row,
query head, selected chunk)), of the local pass (4d per window key) and of the
scorers (2d per (head, candidate)), the records the chunk pass writes, and the
decode step's bytes.  Row i's candidates are the chunks that end before its
window starts, C_i = {c : 64 (c + 1) <= i - W + 1} (Sec. 2.1), and its window
the keys from chunk |C_i| on up to i."""
import subprocess
import sys

import numpy as np

import bench


def per_row(N, S, W, K):
    rows = []
    for i in range(N):
        nc = max(0, (i - W + 1) // S)
        rows.append((nc, min(K, nc), i - nc * S + 1))
    return rows


def test_prefill_model_matches_row_sums():
    B, Hq, Hkv, N, d, S, K, W = 1, 32, 8, 32768, 128, 64, 16, 512
    rows = per_row(N, S, W, K)
    sel = sum(r[1] for r in rows)
    cand = sum(r[0] for r in rows)
    win = sum(r[2] for r in rows)
    m = bench.prefill_kernel_model(B, Hq, Hkv, N, N, d, S, K, W)
    assert m["k_pf_chunks"]["flop"] == B * Hq * (4 * d * S + 2 * d) * sel
    assert m["k_pf_local"]["flop"] == B * Hq * 4 * d * win
    assert m["k_pf_score"]["flop"] == m["k_pf_sigma"]["flop"] == B * Hq * 2 * d * cand
    assert m["k_pf_select"]["flop"] == 0
    # records: a bf16 d-vector and an fp32 score per (row, query head, selected chunk)
    assert m["k_pf_chunks"]["design_bytes"] == B * Hq * sel * (2 * d + 4)
    # the headline figure quoted in the measurement notes: 536.2 GFLOP per chunk pass
    assert abs(m["k_pf_chunks"]["flop"] / 1e9 - 536.2) < 0.1
    attn, score = bench.prefill_work(B, Hq, Hkv, N, d, S, K, W)
    assert attn == B * Hq * 4 * d * (win + S * sel) and score == B * Hq * 2 * d * cand


def test_union_share_counts_tiles_and_pairs():
    # two tiles of 32 rows (groups of 4), 3 slots: the first's rows retrieve chunks {0, 1}
    # (one slot empty), the second's 32 different pairs and chunk 9
    idx = np.full((1, 1, 64, 3), -1, np.int32)
    idx[0, 0, :32, :2] = [0, 1]
    idx[0, 0, 32:, 0] = 9
    idx[0, 0, 32:, 1] = 10 + np.arange(32)
    idx[0, 0, 32:, 2] = 50 + np.arange(32)
    assert bench.union_share(idx, 4, 1) == (0.0, 0.0)
    assert bench.union_share(idx, 4, 2) == (0.5, 64 / (64 + 96))
    assert bench.union_share(idx, 4, 65) == (1.0, 1.0)


def test_union_split_keeps_the_work():
    m = bench.prefill_kernel_model(1, 32, 8, 8192, 8192, 128, 64, 16, 512)
    tiles, pairs = 0.25, 0.125
    s = bench.split_union(m, tiles, pairs)
    assert (bench.union_limit(4, 16), bench.union_limit(8, 16)) == (40, 64)
    names = ("k_pf_chunks", "k_pf_local", "k_pf_union")
    assert sum(s[n]["flop"] for n in names) == m["k_pf_chunks"]["flop"] + m["k_pf_local"]["flop"]
    assert s["k_pf_local"]["bytes"] + s["k_pf_union"]["bytes"] == m["k_pf_local"]["bytes"]
    assert s["k_pf_chunks"]["design_bytes"] == s["k_pf_local"]["design_bytes"] == 0.875 * m["k_pf_chunks"]["design_bytes"]
    assert bench.split_union(m, 0.0, 0.0)["k_pf_chunks"] == m["k_pf_chunks"]


def test_decode_bytes_match_the_step():
    # one new token at position ctx of each of 32 sequences: the candidates'
    # landmarks once, the K selected chunks and the window's K/V, q in and out + lse
    B, Hq, Hkv, ctx, d, S, K, W = 32, 32, 8, 131072, 128, 64, 16, 512
    nc = max(0, (ctx - W + 1) // S)
    nloc = ctx - nc * S + 1
    total, parts = bench.decode_bytes(B, Hq, Hkv, Hq, ctx, d, S, K, W)
    assert parts["landmarks"] == B * Hq * nc * d * 2
    assert parts["kv"] == B * Hkv * (min(K, nc) * S + nloc) * d * 2 * 2
    assert parts["q_out"] == B * Hq * d * 2 * 2 + B * Hq * 4
    assert total == sum(parts.values())


def test_bench_refuses_more_than_one_gpu():
    r = subprocess.run([sys.executable, bench.__file__, "--gpus", "2"], capture_output=True, text=True, timeout=120)
    assert r.returncode != 0
    assert "--gpus 2 is not supported" in r.stderr
