"""Scoring: one, two and four tiles of 32 blocks per workgroup, wavefronts that take the blocks of query rows in turns, and
`last` with its node's rows in one block of 32 rows or on both sides of an edge, against the oracle, both head dims."""
import numpy as np
import pytest
import torch

import oracle
from helpers import check_selection, say

pytestmark = pytest.mark.gpu

CASES = [  # ctx, B, M, Hq, Hkv, last node
    ([16 * 33], 16, 1, 8, 8, 0),                  # one row block, one block in the second tile
    ([16 * 1500], 16, 20, 16, 2, 7),              # five row blocks
    ([61437], 16, 60, 32, 8, 59),                 # two tiles
    ([32 * 640] * 6 + [33], 32, 64, 32, 8, 8),    # four tiles, one short sequence
    ([64 * 700, 64 * 300, 1], 64, 64, 40, 8, 51), # ten row blocks in turns, the node's rows across an edge
    ([64 * 200] * 12, 64, 50, 80, 8, 3),          # sixteen row blocks in turns, an edge again
    ([16 * 300], 16, 80, 64, 4, 79),              # more than sixteen row blocks
]


@pytest.mark.parametrize("D", [128, 64])
@pytest.mark.parametrize("reduce", ["mean", "max", "last"])
@pytest.mark.parametrize("ctx,B,M,Hq,Hkv,last", CASES)
def test_against_the_oracle(gpu_lib, ctx, B, M, Hq, Hkv, last, reduce, D):
    sp, ns, nr, k = gpu_lib, 1, 4, 40
    say("case", ctx, B, M, Hq, Hkv, reduce, D)
    batch, nbm, G = len(ctx), (max(ctx) + B - 1) // B, Hq // Hkv
    gen = torch.Generator(device="cuda").manual_seed(61)
    rows = torch.empty((batch, Hkv, nbm * B, D), dtype=torch.bfloat16, device="cuda")   # never read
    kv = sp.KV(rows, rows, torch.tensor(ctx, dtype=torch.int32, device="cuda"), B, nbm)
    kmax = torch.randn((batch, Hkv, nbm, D), generator=gen, device="cuda").to(torch.bfloat16)
    kmin = kmax - torch.rand((batch, Hkv, nbm, D), generator=gen, device="cuda").to(torch.bfloat16)
    q = torch.randn((batch, M, Hq, D), generator=gen, device="cuda").to(torch.bfloat16)
    tree, cfg = sp.Tree(q, last_node=last), sp.SelectCfg(ns, nr, k, reduce)
    ws = torch.zeros((sp.specpv_workspace_bytes(kv, tree, cfg),), dtype=torch.uint8, device="cuda")
    idx = torch.full((batch, Hkv, cfg.n_sel), -7, dtype=torch.int32, device="cuda")
    cnt = torch.full((batch, Hkv), -7, dtype=torch.int32, device="cuda")
    scores = torch.full((batch, Hkv, nbm), -7.0, device="cuda")
    sp.specpv_select_blocks(kv, tree, kmax, kmin, cfg, idx, cnt, scores, ws)
    torch.cuda.synchronize()
    for b, g in ((0, 0), (batch - 1, Hkv - 1), (batch // 2, Hkv // 2)):
        nb = (ctx[b] + B - 1) // B
        sc = oracle.block_scores(q[b].cpu()[:, g * G:(g + 1) * G], kmax[b, g:g + 1, :nb].permute(1, 0, 2).cpu(),
                                 kmin[b, g:g + 1, :nb].permute(1, 0, 2).cpu(), reduce, last, "eq2")
        got = scores[b, g].cpu().numpy()
        # sums of up to 1280 rows and of 128 products in fp32, in blocks of 16: 1e-5 of the largest term or less
        np.testing.assert_allclose(got[:nb], sc[0], atol=1e-5 * float(np.abs(sc).max()) + 1e-5 * D ** 0.5, rtol=1e-5)
        assert (got[nb:] == -7.0).all(), "scores behind the sequence's last block are written"
        ridx, rcnt = oracle.select_blocks(sc, ns, nr, k)
        check_selection(idx[b, g:g + 1].cpu().numpy(), cnt[b, g:g + 1].cpu().numpy(), ridx, rcnt, sc, ns, nr, k, "%d %d" % (b, g))
