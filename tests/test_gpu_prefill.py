"""GPU parity of hils_prefill_fwd against the oracle, every row compared.

Sizes span several 64-key tiles, ragged tails (N not a multiple of 64), empty
candidate sets (early queries), |C_i| < K, W = 1 (own-chunk local term), a
bias-boosted variant where retrieved chunks carry most of the mass, Q-Cal
routing queries, Hl = Hkv, and group sizes 1..8."""
import numpy as np
import pytest
import torch

import oracle
from paper_2607_02980_amd import synth
from tests.gpu_helpers import (check_close, check_lse, check_selection, host_inputs, kernels_of, log, np32, oshape,
                               to_device)

pytestmark = pytest.mark.gpu

CASES = {
    # name: (params, wid, bias, route, bias_shift)
    "tiny_2k_f32_full_config": (dict(B=1, Hq=4, Hkv=1, N=2048, L=2048, d=64, topk=4, window=512, dtype="f32"), 1,
                                False, False, 0.0),
    "bf16_ragged_multi_tile": (dict(B=2, Hq=8, Hkv=2, N=1000, L=1024, d=128, topk=8, window=200), 101, False, False,
                               0.0),
    "bf16_window1": (dict(B=1, Hq=4, Hkv=1, N=1024, L=1024, d=128, topk=8, window=1), 102, False, False, 0.0),
    # three 2048-row buckets of the chunk pass's inverse index, the last one ragged
    "bf16_row_buckets_ragged": (dict(B=2, Hq=8, Hkv=2, N=4500, L=4544, d=64, topk=8, window=256), 111, False, False,
                                0.0),
    # K * 2048 < 64 * L/S: the buckets double to 4096 rows
    "bf16_row_buckets_grown": (dict(B=1, Hq=4, Hkv=1, N=8192, L=8192, d=64, topk=2, window=256), 112, False, False,
                               0.0),
    "bf16_bias_boosted": (dict(B=1, Hq=8, Hkv=2, N=768, L=768, d=64, topk=4, window=64), 103, True, False, 4.0),
    "bf16_route_Hl_eq_Hkv": (dict(B=1, Hq=8, Hkv=2, Hl=2, N=640, L=640, d=64, topk=6, window=100), 104, True, True,
                             0.0),
    "f32_route_bias_G2": (dict(B=2, Hq=4, Hkv=2, N=700, L=704, d=128, topk=5, window=130, dtype="f32"), 105, True,
                          True, 0.0),
    "bf16_G2_route_bias": (dict(B=1, Hq=4, Hkv=2, N=700, L=704, d=128, topk=5, window=130), 119, True, True, 0.0),
    "bf16_mha_G1": (dict(B=1, Hq=2, Hkv=2, N=512, L=512, d=64, topk=3, window=70), 106, False, False, 0.0),
    "bf16_G8_d128": (dict(B=1, Hq=8, Hkv=1, N=576, L=576, d=128, topk=16, window=64), 107, True, False, 0.0),
    "bf16_topk_exceeds_candidates": (dict(B=1, Hq=4, Hkv=1, N=300, L=320, d=64, topk=16, window=64), 108, False,
                                     False, 0.0),
    "bf16_all_local": (dict(B=1, Hq=4, Hkv=2, N=200, L=256, d=64, topk=4, window=512), 109, False, False, 0.0),
    "f32_large_topk_K64": (dict(B=1, Hq=4, Hkv=1, N=2048, L=2048, d=64, topk=64, window=64, dtype="f32"), 110,
                           False, False, 0.0),
    # bf16 at the larger retrieval budgets the ABI accepts (K = 32 and 64 of up to
    # 39 and 69 candidates)
    "bf16_K32": (dict(B=1, Hq=8, Hkv=2, N=2500, L=2560, d=128, topk=32, window=256), 113, False, False, 0.0),
    "bf16_K64_d64": (dict(B=1, Hq=4, Hkv=1, N=4500, L=4544, d=64, topk=64, window=64), 114, False, False, 0.0),
    # the paper's efficiency shape (Sec. 7.1): d = 64, 16 query / 2 KV heads, S = 64,
    # K = 32, W = 512
    "bf16_paper_shape_d64_G8_K32": (dict(B=1, Hq=16, Hkv=2, N=4096, L=4096, d=64, topk=32, window=512), 115, False,
                                    False, 0.0),
}

# one landmark head's scores raised by 150 (a bias of +150 on every chunk): the
# group's selection follows that head, while every other head's window mass and
# selected scores sit ~150 below it, where e^{-x} underflows to 0 in float; the fusion
# weights are per head (App. C), so each head needs its own stabiliser
GAP_CASES = {
    "bf16_head_gap_150": (dict(B=1, Hq=8, Hkv=2, N=1100, L=1152, d=128, topk=8, window=128), 116, (1, 150.0)),
    "bf16_head_gap_150_G8_d64": (dict(B=1, Hq=8, Hkv=1, N=900, L=960, d=64, topk=6, window=64), 117, (5, 150.0)),
    "f32_head_gap_150": (dict(B=1, Hq=4, Hkv=1, N=700, L=704, d=64, topk=5, window=64, dtype="f32"), 118,
                         (2, 150.0)),
}
for _n, (_kw, _wid, _gap) in GAP_CASES.items():
    CASES[_n] = (_kw, _wid, False, False, 0.0)


def run_case(name, forced=False, flags=0):
    from paper_2607_02980_amd import hils

    kw, wid, bias, route, shift = CASES[name]
    p = hils.Params(flags=flags, **kw)
    gap = GAP_CASES[name][2] if name in GAP_CASES else None
    log(f"[prefill] case={name} forced={forced} flags={flags} params={kw} head_gap={gap}")
    host = host_inputs(p, wid, bias=bias, route=route, bias_shift=shift, head_gap=gap)
    dev = to_device(host, p)
    s = oshape(p)
    ref = oracle.fwd(s, np32(host["q"]), np32(host["k"]), np32(host["v"]), np32(host["lmk"]),
                     bias=np32(host.get("bias")), q_route=np32(host.get("q_route")))
    if forced:
        p.flags = hils.HILS_FLAG_GIVEN_IDX | flags
        idx_in = torch.from_numpy(ref["idx"]).cuda()
        out, lse, idx = hils.hils_prefill_fwd(p, dev["q"], dev["k"], dev["v"], dev["lmk"], dev.get("bias"),
                                              dev.get("q_route"), idx=idx_in)
    else:
        out, lse, idx = hils.hils_prefill_fwd(p, dev["q"], dev["k"], dev["v"], dev["lmk"], dev.get("bias"),
                                              dev.get("q_route"))
    torch.cuda.synchronize()
    gidx = idx.cpu().numpy()
    ndiff = check_selection(p, host, gidx, ref["idx"])
    log(f"  selection: {ndiff} rows differ only by accepted ties")
    if ndiff:
        ref = oracle.fwd(s, np32(host["q"]), np32(host["k"]), np32(host["v"]), np32(host["lmk"]),
                         bias=np32(host.get("bias")), q_route=np32(host.get("q_route")), idx=gidx)
    check_close("out", np32(out), ref["out"], p.dtype)
    check_lse(np32(lse), ref["lse"], p.dtype)


@pytest.mark.parametrize("name", list(CASES))
def test_prefill_matches_oracle(name):
    run_case(name)


@pytest.mark.parametrize("name", ["bf16_ragged_multi_tile", "bf16_window1", "bf16_bias_boosted", "bf16_route_Hl_eq_Hkv",
                                  "bf16_G2_route_bias", "bf16_mha_G1", "bf16_G8_d128", "bf16_K32", "bf16_K64_d64",
                                  "bf16_paper_shape_d64_G8_K32", "bf16_head_gap_150", "bf16_head_gap_150_G8_d64"])
def test_prefill_chunk_major(name):
    """The chunk-major records against the oracle, whatever way the sizes take by themselves: a
    gap before a given selection keeps its tile from the union."""
    from paper_2607_02980_amd import hils

    kw, wid, bias, route, shift = CASES[name]
    p = hils.Params(**kw)
    host = host_inputs(p, wid, bias=bias, route=route, bias_shift=shift,
                       head_gap=GAP_CASES[name][2] if name in GAP_CASES else None)
    dev = to_device(host, p)
    args = (np32(host[n]) for n in ("q", "k", "v", "lmk"))
    extra = dict(bias=np32(host.get("bias")), q_route=np32(host.get("q_route")))
    p.topk = min(p.topk, 63)
    args = (oshape(p), *args)
    idx = oracle.fwd(*args, **extra)["idx"]
    ref = oracle.fwd(*args, idx=idx, **extra)
    gap = torch.from_numpy(np.concatenate([np.full_like(idx[..., :1], -1), idx], -1)).cuda().contiguous()
    p.topk += 1
    p.flags = hils.HILS_FLAG_GIVEN_IDX
    res = {}

    def call():
        res["r"] = hils.hils_prefill_fwd(p, dev["q"], dev["k"], dev["v"], dev["lmk"], dev.get("bias"), dev.get("q_route"),
                                         idx=gap)

    assert "k_pf_chunks" in kernels_of(call)
    check_close("out", np32(res["r"][0]), ref["out"], "bf16")
    check_lse(np32(res["r"][1]), ref["lse"], "bf16")


def test_prefill_union_packing_forced_index():
    # union packing also serves a given selection
    from paper_2607_02980_amd import hils

    run_case("bf16_K32", forced=True, flags=hils.HILS_FLAG_UNION_PACKING)


@pytest.mark.parametrize("name", ["bf16_ragged_multi_tile", "f32_route_bias_G2", "bf16_K32", "bf16_head_gap_150"])
def test_prefill_forced_index(name):
    run_case(name, forced=True)


@pytest.mark.parametrize("name", ["bf16_ragged_multi_tile", "bf16_window1", "bf16_bias_boosted", "bf16_route_Hl_eq_Hkv",
                                  "bf16_G2_route_bias", "bf16_mha_G1", "bf16_G8_d128", "bf16_topk_exceeds_candidates", "bf16_all_local",
                                  "bf16_K32", "bf16_K64_d64", "bf16_paper_shape_d64_G8_K32", "bf16_head_gap_150",
                                  "bf16_head_gap_150_G8_d64"])
def test_prefill_union_packing(name):
    # the one-load-multiple-compute chunk terms (tiles load the union of their
    # rows' chunks) on i.i.d. inputs, against the oracle
    from paper_2607_02980_amd import hils

    run_case(name, flags=hils.HILS_FLAG_UNION_PACKING)


@pytest.mark.parametrize("name", ["bf16_ragged_multi_tile", "bf16_route_Hl_eq_Hkv", "bf16_G8_d128",
                                  "bf16_head_gap_150"])
def test_prefill_union_packing_head_normalised(name):
    # union packing (no workspace, so the fused scorer) under the per-head normalised
    # ranking, whose log-sum-exps come from the separate pass
    from paper_2607_02980_amd import hils

    run_case(name, flags=hils.HILS_FLAG_UNION_PACKING | hils.HILS_FLAG_HEAD_NORM_SELECT)


@pytest.mark.parametrize("G", [4, 1])
def test_prefill_union_packing_on_locality_inputs(G):
    # queries correlated along the sequence (adjacent queries share most chunks):
    # the union path and the chunk-major path against the oracle
    from paper_2607_02980_amd import hils, synth

    p = hils.Params(B=1, Hq=8, Hkv=8 // G, N=3072, L=3072, d=128, topk=16, window=512)
    host = host_inputs(p, 120)
    host["q"] = synth.ar1_host((p.B, p.Hq, p.N, p.d), synth.seed_for(120, "q"), "bf16", rho=0.97)
    dev = to_device(host, p)
    s = oshape(p)
    ref = oracle.fwd(s, np32(host["q"]), np32(host["k"]), np32(host["v"]), np32(host["lmk"]))
    ov = oracle.chunk_overlap(ref["idx"], 16)
    log(f"[prefill-union] G={G} chunk overlap of 16 adjacent queries: {ov:.3f}")
    assert ov > 0.7
    for flags in (hils.HILS_FLAG_UNION_PACKING, 0):
        p.flags = flags
        out, lse, idx = hils.hils_prefill_fwd(p, dev["q"], dev["k"], dev["v"], dev["lmk"])
        torch.cuda.synchronize()
        gidx = idx.cpu().numpy()
        ndiff = check_selection(p, host, gidx, ref["idx"])
        r = ref if not ndiff else oracle.fwd(s, np32(host["q"]), np32(host["k"]), np32(host["v"]),
                                            np32(host["lmk"]), idx=gidx)
        check_close("out", np32(out), r["out"], p.dtype)
        check_lse(np32(lse), r["lse"], p.dtype)


@pytest.mark.parametrize("name", ["tiny_2k_f32_full_config", "bf16_ragged_multi_tile", "bf16_bias_boosted",
                                  "bf16_route_Hl_eq_Hkv", "f32_route_bias_G2", "bf16_mha_G1", "bf16_G8_d128",
                                  "bf16_topk_exceeds_candidates", "bf16_K32", "bf16_K64_d64",
                                  "bf16_paper_shape_d64_G8_K32", "bf16_head_gap_150", "f32_head_gap_150"])
def test_prefill_head_normalised_selection(name):
    # the per-head normalised ranking (Sec. 4.1 wording), against the oracle's
    from paper_2607_02980_amd import hils

    run_case(name, flags=hils.HILS_FLAG_HEAD_NORM_SELECT)


def test_prefill_is_deterministic():
    from paper_2607_02980_amd import hils

    kw, wid, bias, route, shift = CASES["bf16_ragged_multi_tile"]
    p = hils.Params(**kw)
    dev = to_device(host_inputs(p, wid), p)
    a = hils.hils_prefill_fwd(p, dev["q"], dev["k"], dev["v"], dev["lmk"])
    b = hils.hils_prefill_fwd(p, dev["q"], dev["k"], dev["v"], dev["lmk"])
    torch.cuda.synchronize()
    for x, y in zip(a, b):
        assert torch.equal(x, y)


@pytest.mark.parametrize("N,Hkv,G,K,rho", [(830, 2, 4, 4, 0.0), (1790, 2, 4, 4, 0.97), (1800, 1, 4, 4, 0.0),
                                           (1330, 1, 8, 6, 0.0), (770, 3, 1, 4, 0.0), (1850, 3, 1, 4, 0.0),
                                           (1025, 1, 2, 4, 0.0), (1000, 2, 2, 64, 0.0),
                                           (2040, 1, 4, 8, 0.0), (2100, 1, 4, 8, 0.0),
                                           (2360, 1, 4, 8, 0.0), (2400, 1, 4, 8, 0.0),   # one round: 37 and 38 chunks
                                           (2550, 4, 4, 8, 0.0), (2610, 4, 4, 8, 0.0)])  # more tiles: 40 and 41
def test_few_chunks_match_given_selection(N, Hkv, G, K, rho):
    """Few more chunks than a row retrieves (the union path; on both sides of its limit,
    3 K + 16 chunks at d = 64, fewer while the tiles fit the chip at once) against the same
    selection given with a gap before it, which always takes the chunk-major pass, and
    without one, which takes the same path; and a NaN value stays with the rows that attend it."""
    from paper_2607_02980_amd import hils

    p = hils.Params(B=2, Hq=Hkv * G, Hkv=Hkv, N=N, L=-(-N // 64) * 64, d=64, topk=K, window=130)
    host = host_inputs(p, 370, bias=True, route=True)
    if rho:
        host["q"] = synth.ar1_host(host["q"].shape, 371, "bf16", rho)
    dev = to_device(host, p)

    def run(flags, idx=None):
        p.flags = flags
        return hils.hils_prefill_fwd(p, dev["q"], dev["k"], dev["v"], dev["lmk"], dev["bias"], dev["q_route"], idx=idx)

    out, lse, idx = run(0)
    same, slse, _ = run(hils.HILS_FLAG_GIVEN_IDX, idx.clone())
    assert torch.equal(out, same) and torch.equal(lse, slse)
    if K < 64:
        p.topk = K + 1
        gap = torch.cat([torch.full_like(idx[..., :1], -1), idx], -1).contiguous()
        ref, rlse, _ = run(hils.HILS_FLAG_GIVEN_IDX, gap)
        p.topk = K
        # the chunk-major records round each chunk's output to bf16 (2^-9), the union does not
        assert (out.float() - ref.float()).abs().max() <= 2e-2 and (lse - rlse).abs().max() <= 2e-4
    j = 200  # in chunk 3
    dev["v"][0, 0, j] = float("nan")
    n = torch.arange(N, device="cuda")
    left = ((n - p.window + 1).div(64, rounding_mode="floor") * 64).clamp(min=0)
    sees = ((n >= j) & (left <= j)) | (idx[0, 0] == j // 64).any(-1)
    near = (n >= 128) & (left <= j + 192)  # a tile of up to 128 rows shares its windows' keys
    out2, _, idx2 = run(0)
    assert torch.equal(idx, idx2)
    far = ~sees & ~near
    assert torch.equal(out2[0, :G, far], out[0, :G, far]) and torch.isnan(out2[0, :G, sees]).all()


@pytest.mark.parametrize("N,Hkv,G,K,union", [(700, 4, 1, 2, True), (1441, 4, 1, 2, False),    # 44 and 62 us: records, union
                                             (1534, 4, 1, 4, False), (2933, 1, 1, 16, False),  # 46 chunks: 69 and 112 us
                                             (2933, 16, 1, 16, True),                          # 146 and 133 us
                                             (1200, 2, 4, 4, True), (2600, 2, 4, 4, False),
                                             (2600, 2, 8, 8, True)])
def test_few_tiles_take_the_faster_way(N, Hkv, G, K, union):
    """One sequence of few tiles (d = 128): the union pass while it is the shorter chain, the
    chunk-major pass, which spreads over the chunks, beyond."""
    from paper_2607_02980_amd import hils

    p = hils.Params(B=1, Hq=Hkv * G, Hkv=Hkv, N=N, L=-(-N // 64) * 64, d=128, topk=K, window=64)
    dev = to_device(host_inputs(p, 374), p)
    ran = kernels_of(lambda: hils.hils_prefill_fwd(p, dev["q"], dev["k"], dev["v"], dev["lmk"]))
    assert ("k_pf_union" in ran, "k_pf_chunks" in ran) == (union, not union), ran


@pytest.mark.parametrize("N,Hkv,G,K,chunks", [(14200, 2, 4, 64, False), (14400, 2, 4, 64, True),  # 222 and 225 chunks
                                              (8100, 8, 1, 32, False), (8300, 8, 1, 32, True)])   # 127 and 130
def test_large_k_leaves_one_union_workgroup_per_cu(N, Hkv, G, K, chunks):
    """d = 128 and lists of chunks so long that one union workgroup fits a CU: the whole call
    takes the union up to 3 K + 32 chunks."""
    from paper_2607_02980_amd import hils

    p = hils.Params(B=1, Hq=Hkv * G, Hkv=Hkv, N=N, L=-(-N // 64) * 64, d=128, topk=K, window=64)
    dev = {n: torch.randn(s, device="cuda").to(torch.bfloat16)
           for n, s in dict(q=(1, p.Hq, N, 128), k=(1, Hkv, p.L, 128), v=(1, Hkv, p.L, 128),
                            lmk=(1, p.Hq, p.L // 64, 128)).items()}
    ran = kernels_of(lambda: hils.hils_prefill_fwd(p, dev["q"], dev["k"], dev["v"], dev["lmk"]))
    assert ("k_pf_chunks" in ran) == chunks, ran


@pytest.mark.parametrize("B,N,Hkv,G,K,by_tile", [(1, 17000, 1, 4, 16, False),  # 1.28 times the time by tile
                                                 (1, 8000, 3, 4, 16, False), (1, 11000, 4, 4, 31, False),
                                                 (2, 11000, 2, 4, 32, True), (1, 6200, 8, 4, 16, True),
                                                 (1, 11000, 1, 8, 16, False), (2, 6200, 1, 8, 16, True)])
def test_tiles_choose_where_the_early_ones_fill_the_chip(B, N, Hkv, G, K, by_tile):
    """Long sequences (d = 128, more tiles than the chip takes at once): by tile with enough KV
    groups, else all chunk-major."""
    from paper_2607_02980_amd import hils

    p = hils.Params(B=B, Hq=Hkv * G, Hkv=Hkv, N=N, L=-(-N // 64) * 64, d=128, topk=K, window=64)
    dev = {n: torch.randn(s, device="cuda").to(torch.bfloat16)
           for n, s in dict(q=(B, p.Hq, N, 128), k=(B, Hkv, p.L, 128), v=(B, Hkv, p.L, 128),
                            lmk=(B, p.Hq, p.L // 64, 128)).items()}
    ran = kernels_of(lambda: hils.hils_prefill_fwd(p, dev["q"], dev["k"], dev["v"], dev["lmk"]))
    assert "k_pf_chunks" in ran and ("k_pf_union" in ran) == by_tile, ran


def union_sizes(idx, G):
    """Chunks in the union of every tile of 128 / G rows of a selection [B, Hkv, N, K]."""
    QT = 128 // G
    pad = -idx.shape[2] % QT
    idx = np.pad(idx, ((0, 0), (0, 0), (0, pad), (0, 0)), constant_values=-1)
    blk = np.sort(idx.reshape(-1, QT * idx.shape[-1]), axis=-1)
    return ((np.diff(blk, axis=-1, prepend=-1) != 0)).sum(-1)


@pytest.mark.parametrize("N,Hkv,G,K,d,ran", [(6200, 2, 4, 16, 128, "chunks"), (5700, 1, 8, 17, 128, "chunks"),
                                             (6000, 1, 4, 20, 128, "chunks"), (4100, 2, 1, 16, 64, "chunks"),
                                             (5700, 3, 4, 16, 128, "chunks"),
                                             # enough KV groups and more tiles than two per CU: by tile
                                             (10100, 2, 8, 17, 128, "both"), (6200, 8, 4, 16, 128, "both"),
                                             (12000, 4, 4, 32, 128, "both")])
def test_tiles_of_both_kinds(N, Hkv, G, K, d, ran):
    """Sequences whose early tiles take the union and whose later ones the chunk-major pass
    (adjacent queries alike in the second half, so that some later ones take it too), and ones
    just as long that are all chunk-major: rows of all kinds against the oracle, and bitwise
    the same when given the selection."""
    from paper_2607_02980_amd import hils

    p = hils.Params(B=1, Hq=Hkv * G, Hkv=Hkv, N=N, L=-(-N // 64) * 64, d=d, topk=K, window=200)
    host = host_inputs(p, 372, bias=True)
    alike = synth.ar1_host(host["q"].shape, 373, "bf16", 0.999)
    host["q"][:, :, N // 2:] = alike[:, :, N // 2:]
    dev = to_device(host, p)
    res = {}

    def call():
        res["r"] = hils.hils_prefill_fwd(p, dev["q"], dev["k"], dev["v"], dev["lmk"], dev["bias"])

    names = kernels_of(call)
    assert ("k_pf_chunks" in names, "k_pf_union" in names) == (True, ran == "both"), names
    out, lse, idx = res["r"]
    if ran == "both":
        small = union_sizes(idx.cpu().numpy(), G) <= (4 * K if G == 8 else 5 * K // 2)
        half = len(small) // Hkv // 2
        late = small.reshape(Hkv, -1)[:, half:]
        log(f"[tiles] {small.mean():.3f} of the tiles take the union, {late.mean():.3f} of the later half")
        assert small.any() and not small.all() and late.any()
    p.flags = hils.HILS_FLAG_GIVEN_IDX
    same, slse, _ = hils.hils_prefill_fwd(p, dev["q"], dev["k"], dev["v"], dev["lmk"], dev["bias"], idx=idx.clone())
    assert torch.equal(out, same) and torch.equal(lse, slse)
    p.flags = 0
    # every row of the smaller cases, every 7th and the edges of tiles of the others
    n = np.arange(N) if N * p.Hq <= 100000 else np.unique(np.r_[0:N:7, 31:N:320, 32:N:320, N - 1])
    args = (oshape(p), *(np32(host[x]) for x in ("q", "k", "v", "lmk")))
    ref = oracle.fwd(*args, bias=np32(host["bias"]), idx=idx.cpu().numpy(),
                     rows=np.stack([np.zeros_like(n), n], -1).astype(np.int32))
    check_close("out", np32(out)[:, :, n], ref["out"][:, :, n], "bf16")
    check_lse(np32(lse)[:, :, n], ref["lse"][:, :, n], "bf16")
