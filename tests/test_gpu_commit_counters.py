"""The counters of a commit are moved by whichever workgroup of a sequence is last to have read them: numbers of workgroups on
either side of what is counted on one level, words of a sequence with and without lines of their own, several launches for
layers and for sequences, lists, buffers and caches without room, three commits in a row with the same words, and replays of a graph of one."""
import numpy as np
import pytest
import torch

from helpers import say

pytestmark = pytest.mark.gpu


def _expect(ctx, pend, acc, free, P, cap, B, to_cache):
    """(lengths, pending, dropped, new list entries per sequence) after a commit; free: the fewest free entries of a list row"""
    total = pend + acc
    stored = np.minimum(total, np.maximum(cap - ctx, 0)) if to_cache else np.minimum(total, P)
    if not to_cache:
        return ctx, stored, np.stack([total - stored, np.zeros_like(total)], 1), np.zeros_like(total)
    blocks = np.where(stored > 0, (ctx + stored - 1) // B - ctx // B + 1, 0)   # none of them is listed yet
    return ctx + stored, np.zeros_like(pend), np.stack([total - stored, np.maximum(blocks - free, 0)], 1), blocks


@pytest.mark.parametrize("batch,Hkv,layers,graph", [(1, 1, 1, False), (1, 16, 1, True), (1, 17, 1, False), (3, 8, 5, True), (28, 2, 3, False), (29, 2, 3, True),
                                                    (911, 1, 2, False), (2, 8, 33, False), (5, 3, 32, True)])
@pytest.mark.parametrize("mode_name", ["partial", "refresh"])
def test_counters_move_once(gpu_lib, batch, Hkv, layers, graph, mode_name):
    sp, dev = gpu_lib, torch.device("cuda")
    say("case", batch, Hkv, layers, graph, mode_name)
    D, B, nb, P, Mt, n_sel = 64, 16, 8, 20, 12, 3
    to_cache = mode_name == "refresh"
    rng = np.random.default_rng(5)
    ctx = rng.integers(0, nb * B + 1, batch).astype(np.int64)
    pend = rng.integers(0, P + 1, batch).astype(np.int64)
    acc = rng.integers(0, 9, batch).astype(np.int64)
    free = rng.integers(0, n_sel + 1, (batch, Hkv, layers))
    t = lambda x: torch.tensor(x, dtype=torch.int32, device=dev)
    ctx_d, pend_d, acc_d = t(ctx), t(pend), t(acc)
    path = torch.arange(8, dtype=torch.int32, device=dev).repeat(batch, 1)
    ks, vs = ([torch.randn((batch, Hkv, nb * B, D), device=dev).bfloat16() for _ in range(layers)] for _ in range(2))
    bk, bv = ([torch.randn((batch, P + Mt, Hkv, D), device=dev).bfloat16() for _ in range(layers)] for _ in range(2))
    kvs = [sp.KV(ks[l], vs[l], ctx_d, B, nb) for l in range(layers)]
    idx = [torch.full((batch, Hkv, n_sel), -5, dtype=torch.int32, device=dev) for _ in range(layers)]   # (no block's number)
    cnt = [t(n_sel - free[:, :, l]) for l in range(layers)]
    dropped = torch.full((batch, 2), -1, dtype=torch.int32, device=dev)
    ws = torch.zeros((sp.specpv_workspace_bytes(kvs[0]),), dtype=torch.uint8, device=dev)
    start = [x.clone() for x in (ctx_d, pend_d, acc_d)] + [x.clone() for x in cnt] + [x.clone() for x in idx]

    def call():
        sp.specpv_commit_accepted_layers(kvs, bk, bv, P, Mt, pend_d, path, acc_d, sp.MODE_REFRESH if to_cache else sp.MODE_PARTIAL, workspace=ws,
                                         sel_idxs=idx, sel_counts=cnt, dropped=dropped)

    def check(c, p, fr):
        c2, p2, d2, blocks = _expect(c, p, acc, fr.min((1, 2)), P, nb * B, B, to_cache)
        torch.cuda.synchronize()
        assert np.array_equal(ctx_d.cpu().numpy(), c2) and np.array_equal(pend_d.cpu().numpy(), p2)
        assert np.array_equal(dropped.cpu().numpy(), d2)
        fr2 = np.maximum(fr - blocks[:, None, None], 0)
        for l in range(layers):
            assert np.array_equal(cnt[l].cpu().numpy(), n_sel - fr2[:, :, l]), l
        assert int(ws[:65536].sum()) == 0
        return c2, p2, fr2

    def reset():
        for x, s in zip([ctx_d, pend_d, acc_d] + cnt + idx, start):
            x.copy_(s)

    c, p, fr = ctx, pend, free
    for _ in range(3):
        call()
        c, p, fr = check(c, p, fr)
        for x in idx:
            x.fill_(-5)   # (the next commit's first block may be this one's last)
    if graph:
        reset()
        call()
        reset()
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            call()
        for _ in range(3):
            reset()
            dropped.fill_(-1)
            g.replay()
            check(ctx, pend, free)
