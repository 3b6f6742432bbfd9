"""GPU parity of the fp32-storage prefill and backward kernels at the edges of their
tiles (16 / G queries x G heads per block, 64-key parts, blocks per chunk): one query,
odd lengths, every group size and head dim, shared landmarks, more slots than candidates;
and that what a row does not attend never reaches it."""
import numpy as np
import pytest
import torch

import oracle
from tests.gpu_helpers import (check_close, check_lse, check_selection, host_inputs, kernels_of, log, np32, oshape,
                               to_device)

pytestmark = pytest.mark.gpu

# (B, Hq, Hkv, Hl, N, L, d, K, W, bias, route)
CASES = [
    # (not one query: its one key makes dq exactly 0, and the bar is relative to |dq|, while
    # the fp32 rounding of g.v - u, 2^-24 |g||v| per term, stays)
    (1, 4, 1, 4, 2, 64, 64, 4, 512, False, False),
    (2, 4, 4, 4, 333, 384, 64, 16, 64, True, True),     # G = 1: 16 queries per block
    (1, 8, 4, 4, 257, 320, 128, 3, 1, False, True),     # G = 2, shared landmarks, W = 1
    (1, 4, 1, 1, 700, 704, 64, 64, 100, True, False),   # K above every candidate count
    (2, 8, 1, 8, 450, 512, 128, 7, 200, True, True),    # G = 8: 2 queries per block
    (1, 16, 2, 2, 321, 384, 64, 5, 64, True, True),     # G = 8, shared landmarks
    (1, 2, 1, 2, 1500, 1536, 64, 4, 256, False, False),
    # up to 112 queries: a block per query while about a round of them fits the chip, or tiles
    (1, 4, 4, 4, 64, 64, 128, 3, 1, True, True),
    (3, 8, 1, 1, 64, 128, 64, 3, 1, True, False),
    (1, 4, 2, 4, 112, 128, 128, 5, 1, True, True),
    (1, 4, 2, 2, 113, 128, 64, 5, 1, False, True),
    (5, 16, 4, 16, 79, 128, 64, 2, 1, False, False),    # 1580 rows: tiles
    (9, 16, 4, 16, 79, 128, 64, 2, 1, False, False),    # 2844: blocks
    # no row has a candidate, and the first length at which one has
    (2, 8, 4, 4, 3, 64, 128, 4, 256, True, True),
    (1, 4, 2, 4, 64, 64, 64, 3, 1, True, False),
    (1, 4, 2, 4, 65, 128, 64, 3, 1, True, True),
]


def params(case):
    from paper_2607_02980_amd import hils

    B, Hq, Hkv, Hl, N, L, d, K, W, bias, route = case
    return hils.Params(B=B, Hq=Hq, Hkv=Hkv, Hl=Hl, N=N, L=L, d=d, topk=K, window=W, dtype="f32"), bias, route


def poisoned(p, op):
    """A workspace whose every byte is set (floats read as NaN): all that is read must be written first."""
    from paper_2607_02980_amd import hils

    return torch.full((max(1, hils.hils_workspace_size(p, op)),), 255, dtype=torch.uint8, device="cuda")


def step(p, dev):
    from paper_2607_02980_amd import hils

    out, lse, idx = hils.hils_prefill_fwd(p, dev["q"], dev["k"], dev["v"], dev["lmk"], dev.get("bias"),
                                          dev.get("q_route"))
    g = hils.hils_bwd(p, dev["dout"], dev["q"], dev["k"], dev["v"], dev["lmk"], out, lse, idx, dev.get("bias"),
                      dev.get("q_route"), workspace=poisoned(p, hils.HILS_OP_BWD))
    torch.cuda.synchronize()
    return out, lse, idx, g


@pytest.mark.parametrize("case", CASES, ids=str)
def test_f32_matches_oracle(case):
    p, bias, route = params(case)
    log(f"[f32] {case}")
    host = host_inputs(p, 340 + CASES.index(case), bias=bias, route=route, dout=True)
    dev = to_device(host, p)
    if p.L > p.N:  # keys past the last query are nobody's: anything may be there
        for name in ("k", "v"):
            dev[name][:, :, p.N:] = float("nan")
    out, lse, idx, g = step(p, dev)
    s, h = oshape(p), {n: np32(t) for n, t in host.items()}
    args = (s, h["q"], h["k"], h["v"], h["lmk"])
    kw = dict(bias=h.get("bias"), q_route=h.get("q_route"))
    check_selection(p, host, idx.cpu().numpy(), oracle.fwd(*args, **kw)["idx"])
    ref = oracle.fwd(*args, idx=idx.cpu().numpy(), **kw)
    check_close("out", np32(out), ref["out"], "f32")
    check_lse(np32(lse), ref["lse"], "f32")
    rb = oracle.bwd(s, h["dout"], *args[1:], idx.cpu().numpy(), **kw)
    for key, rkey in (("dq", "dq"), ("dk", "dk"), ("dv", "dv"), ("dlmk", "dlmk"), ("dlmk_bias", "dbias"),
                      ("dq_route", "dq_route")):
        if rb[rkey] is not None:
            check_close(key, np32(g[key]), rb[rkey], "f32", rel=True)


@pytest.mark.parametrize("N,W,index", [(3, 256, False), (64, 1, False), (65, 1, True), (575, 512, False), (576, 512, True)])
def test_f32_backward_indexes_only_where_rows_retrieve(N, W, index):
    from paper_2607_02980_amd import hils

    p, _, _ = params((1, 4, 1, 4, N, -(-N // 64) * 64, 64, 4, W, False, False))
    dev = to_device(host_inputs(p, 354, dout=True), p)
    out, lse, idx = hils.hils_prefill_fwd(p, dev["q"], dev["k"], dev["v"], dev["lmk"])
    ran = kernels_of(lambda: hils.hils_bwd(p, dev["dout"], dev["q"], dev["k"], dev["v"], dev["lmk"], out, lse, idx))
    assert ("k_inv_count" in ran, "k_inv_sort" in ran) == (index, index), ran


def test_f32_is_deterministic():
    p, bias, route = params(CASES[4])
    dev = to_device(host_inputs(p, 350, bias=bias, route=route, dout=True), p)
    a, b = step(p, dev), step(p, dev)
    assert all(torch.equal(x, y) for x, y in zip(a[:3], b[:3]))
    for key in a[3]:
        assert torch.equal(a[3][key], b[3][key]), key


def test_f32_values_stay_with_the_rows_that_attend_them():
    """A NaN in one value row reaches the rows that attend it and no other, though they
    share tiles with rows that do; an infinite key likewise in dq."""
    p, _, _ = params((1, 4, 1, 4, 400, 448, 64, 2, 64, False, False))
    host = host_inputs(p, 351, dout=True)
    dev = to_device(host, p)
    out, lse, idx, g = step(p, dev)
    j = 130  # in chunk 2
    n = torch.arange(p.N, device="cuda")
    left = ((n - p.window + 1).div(64, rounding_mode="floor") * 64).clamp(min=0)
    sees = ((n >= j) & (left <= j)) | (idx[0, 0] == j // 64).any(-1)
    dev["v"][0, 0, j] = float("nan")
    out2, _, idx2, _ = step(p, dev)
    assert torch.equal(idx, idx2)
    assert torch.isnan(out2[:, :, sees]).all() and not torch.isnan(out2[:, :, ~sees]).any()
    check_close("out", np32(out2[:, :, ~sees]), np32(out[:, :, ~sees]), "f32")
    dev["v"] = to_device(host, p)["v"]
    dev["k"][0, 0, j, 5] = float("inf")
    _, _, _, g2 = step(p, dev)
    check_close("dq", np32(g2["dq"][:, :, ~sees]), np32(g["dq"][:, :, ~sees]), "f32", rel=True)


@pytest.mark.parametrize("G,d", [(1, 64), (2, 128), (4, 64)])
def test_f32_a_row_out_of_order_changes_no_other(G, d):
    """A given row that names a chunk twice (entries must ascend, so its own result is nobody's
    business) leaves the rows of its tile that hold the chunk as they were."""
    from paper_2607_02980_amd import hils

    p, _, _ = params((1, 2 * G, 2, 2 * G, 900, 960, d, 4, 64, False, False))
    dev = to_device(host_inputs(p, 352, dout=True), p)
    out, lse, idx, g = step(p, dev)
    n = 704  # first of its tile
    bad = idx.clone()
    bad[0, 0, n] = torch.tensor([idx[0, 0, n + 16 // G - 1, 0], -1, idx[0, 0, n + 16 // G - 1, 0], -1])
    p.flags = hils.HILS_FLAG_GIVEN_IDX
    out2, lse2, _ = hils.hils_prefill_fwd(p, dev["q"], dev["k"], dev["v"], dev["lmk"], idx=bad)
    p.flags = 0
    g2 = hils.hils_bwd(p, dev["dout"], dev["q"], dev["k"], dev["v"], dev["lmk"], out, lse, bad)
    torch.cuda.synchronize()
    rest = torch.ones(p.N, dtype=torch.bool, device="cuda")
    rest[n] = False
    # (the union's order follows the rows, so the sums of the tile may run in another order)
    for x, y, name in ((out2, out, "out"), (lse2, lse, "lse"), (g2["dq"], g["dq"], "dq")):
        check_close(name, np32(x[:, :G, rest]), np32(y[:, :G, rest]), "f32", rel=True)


def test_f32_prefill_in_place():
    """Outputs in the place of the queries: the bits of a separate output, also in tiles that
    are computed again because a value they share is not finite."""
    from paper_2607_02980_amd import hils

    p, _, _ = params((1, 8, 2, 8, 700, 704, 64, 4, 64, False, False))
    dev = to_device(host_inputs(p, 353), p)
    dev["v"][0, 0, 130] = float("nan")
    a = hils.hils_prefill_fwd(p, dev["q"], dev["k"], dev["v"], dev["lmk"])
    b = hils.hils_prefill_fwd(p, dev["q"], dev["k"], dev["v"], dev["lmk"], out=dev["q"])
    torch.cuda.synchronize()
    assert torch.isnan(a[0]).any() and torch.equal(a[2], b[2])
    same = torch.equal(torch.nan_to_num(a[0], nan=1e9), torch.nan_to_num(b[0], nan=1e9)), torch.equal(a[1], b[1])
    assert same == (True, True)
