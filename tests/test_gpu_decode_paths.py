"""GPU parity of the bf16 decode step where its paths meet: one launch per step up to 256
chunks in the caches, scan slices of 64 to 256 chunks, the merge of the survivors by one
wave (64, 256 or 512 of them) or by a workgroup, and the multi-query pass split over
workgroups.  Against the oracle, from a workspace whose every byte is set."""
import numpy as np
import pytest
import torch

import oracle
from tests.gpu_helpers import check_close, check_lse, check_selection, host_inputs, log, np32, oshape, to_device

pytestmark = pytest.mark.gpu

# (B, Hq, Hkv, Hl, N, chunks, d, K, W, bias, route, paged, seqlens or None)
CASES = [
    (1, 8, 1, 8, 1, 255, 64, 16, 512, True, False, False, None),
    (1, 8, 1, 1, 1, 256, 64, 64, 64, True, True, True, None),         # the last size of one launch
    (2, 2, 2, 2, 1, 257, 128, 7, 100, False, False, False, [16448, 12000]),
    (3, 4, 1, 4, 1, 40, 128, 4, 300, False, True, True, [2560, 1, 400]),
    (2, 8, 2, 8, 1, 700, 128, 16, 512, True, False, True, [44800, 9000]),  # 64-chunk slices, 176 survivors
    (2, 4, 1, 1, 1, 1100, 64, 32, 512, False, False, False, None),    # 128-chunk slices, 288 survivors
    (1, 2, 1, 2, 1, 1100, 64, 64, 512, False, False, False, None),    # 256-chunk slices, 320 survivors
    (1, 4, 1, 4, 1, 2400, 64, 64, 64, False, False, False, None),     # 640 survivors: merged by the workgroup
    (2, 8, 2, 8, 4, 300, 128, 16, 512, False, False, False, [19200, 5000]),  # multi-query, 8 workgroups a group
    (1, 2, 2, 2, 9, 300, 64, 5, 64, True, True, True, None),          # G = 1: groups of 8 and 1 queries
    (2, 16, 2, 2, 5, 70, 64, 16, 128, True, False, False, [4480, 6]),  # G = 8: groups of 2, 2 and 1
    (33, 8, 4, 8, 2, 40, 64, 3, 200, False, False, False, None),      # 132 groups: not split
]


@pytest.mark.parametrize("case", CASES, ids=str)
def test_decode_paths_match_oracle(case):
    from paper_2607_02980_amd import hils

    B, Hq, Hkv, Hl, N, nc, d, K, W, bias, route, paged, lens = case
    p = hils.Params(B=B, Hq=Hq, Hkv=Hkv, Hl=Hl, N=N, L=nc * 64, d=d, topk=K, window=W)
    log(f"[decode paths] {case}")
    host = host_inputs(p, 360 + CASES.index(case), bias=bias, route=route)
    dev = to_device(host, p)
    lens = lens or [p.L] * B
    qpos = np.array([[n - N + i for i in range(N)] for n in lens], np.int32)
    sl = torch.tensor(lens, dtype=torch.int32, device="cuda")
    ws = torch.full((max(1, hils.hils_workspace_size(p, hils.HILS_OP_DECODE)),), 255, dtype=torch.uint8, device="cuda")
    if paged:
        g = torch.Generator().manual_seed(5)
        table = torch.randperm(B * nc + 3, generator=g)[:B * nc].to(torch.int32)

        def pool(t, *shape):  # [B, H, nc, ...] -> [pages, H, ...]
            x = torch.zeros((B * nc + 3, *shape), dtype=t.dtype, device="cuda")
            x[table.long().cuda()] = t.transpose(1, 2).reshape(B * nc, *shape)
            return x

        k, v = (pool(dev[n].view(B, Hkv, nc, 64, d), Hkv, 64, d) for n in ("k", "v"))
        lmk = pool(dev["lmk"], Hl, d)
        bp = pool(dev["bias"], Hl) if bias else None
        out, lse, idx = hils.hils_decode_paged_fwd(p, dev["q"], k, v, lmk, table.view(B, nc).cuda(), bp,
                                                   dev.get("q_route"), sl, workspace=ws)
    else:
        out, lse, idx = hils.hils_decode_fwd(p, dev["q"], dev["k"], dev["v"], dev["lmk"], dev.get("bias"),
                                             dev.get("q_route"), sl, workspace=ws)
    torch.cuda.synchronize()
    s, h = oshape(p), {n: np32(t) for n, t in host.items()}
    args = (s, h["q"], h["k"], h["v"], h["lmk"])
    kw = dict(bias=h.get("bias"), q_route=h.get("q_route"), qpos=qpos)
    gidx = idx.cpu().numpy()
    check_selection(p, host, gidx, oracle.fwd(*args, **kw)["idx"], qpos=qpos)
    ref = oracle.fwd(*args, idx=gidx, **kw)
    check_close("out", np32(out), ref["out"], "bf16")
    check_lse(np32(lse), ref["lse"], "bf16")


def test_finer_slices_stay_within_the_fixed_array():
    """Finer slices never push a call over the fixed array of the call without a workspace."""
    from paper_2607_02980_amd import hils

    for B, L, K in ((1, 1 << 20, 64), (4, 1 << 20, 32), (15, 65536, 64), (60, 32768, 16), (112, 16384, 16)):
        p = hils.Params(B=B, Hq=32, Hkv=8, N=1, L=L, d=128, topk=K)
        nloc, rows = (512 + 62) // 64 + 1, B * 8
        al = lambda x: (x + 255) & ~255  # noqa: E731
        ns = (L // 64 + 255) // 256
        coarse = al(rows * ns * K * 8) + al(rows * (K + nloc) * 4 * 132 * 4) + al(rows * ns * 4 * 8)
        size = hils.hils_workspace_size(p, hils.HILS_OP_DECODE)
        assert size <= max(coarse, hils.HILS_DECODE_NOALLOC_SCRATCH_BYTES), (B, L, K, size, coarse)


@pytest.mark.parametrize("B,Hkv,ctx,d", [(1, 2, 4095, 64), (16, 8, 20000, 64), (3, 8, 20000, 128), (36, 8, 17000, 64)])
def test_shared_landmarks_match_repeated_ones(B, Hkv, ctx, d):
    """One landmark head per KV group against the same landmarks given for every query head, at
    slices of 64 to 256 chunks (the shared scan takes longer ones): the same selection and, to
    the rounding of the scores' sums, the same outputs."""
    from paper_2607_02980_amd import hils

    G, L = 4, -(-(ctx + 1) // 64) * 64
    g = torch.Generator(device="cuda").manual_seed(5)
    t = lambda *s: torch.randn(s, device="cuda", generator=g).to(torch.bfloat16)
    q, k, v, lmk = t(B, Hkv * G, 1, d), t(B, Hkv, L, d), t(B, Hkv, L, d), t(B, Hkv, L // 64, d)
    res = []
    for Hl, lm in ((Hkv, lmk), (Hkv * G, lmk.repeat_interleave(G, 1).contiguous())):
        p = hils.Params(B=B, Hq=Hkv * G, Hkv=Hkv, Hl=Hl, N=1, L=L, d=d, topk=8, window=128)
        ws = torch.full((hils.hils_workspace_size(p, hils.HILS_OP_DECODE),), 255, dtype=torch.uint8, device="cuda")
        res.append(hils.hils_decode_fwd(p, q, k, v, lm, workspace=ws))
    (o1, l1, i1), (o2, l2, i2) = res
    same = (i1 == i2).all(-1)  # (a tie in the last bits of two scores may go either way)
    assert same.float().mean() > 0.99
    rows = same.repeat_interleave(G, 1)
    assert (o1.float() - o2.float())[rows].abs().max() <= 2e-2 and (l1 - l2)[rows].abs().max() <= 2e-4
