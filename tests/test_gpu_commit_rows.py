"""Rows and summaries of a commit to the cache, bit for bit: numbers of rows on either side of what the small variant keeps and of
what is read at once, one and several blocks, older rows from none to many trips, more blocks than wavefronts."""
import numpy as np
import pytest
import torch

from helpers import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("P,most,B", [(28, 4, 64), (29, 4, 64), (20, 8, 5), (95, 28, 16), (119, 4, 250), (0, 3, 1)])
def test_rows_and_summaries(gpu_lib, dtype, D, P, most, B):
    sp, dev = gpu_lib, torch.device("cuda")
    say("case", dtype, D, P, most, B)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    Hkv, Mt, nb, layers = 3, most + 5, 900 // B, 2
    ctx = np.array([0, B, B + 1, 4 * B - 1, 3 * B + B // 2, nb * B - 2, nb * B], dtype=np.int64)
    batch = len(ctx)
    rng = np.random.default_rng(P + D + B)
    pend = rng.integers(0, P + 1, batch)
    pend[1], pend[2] = P, 0
    acc = rng.integers(0, most + 1, batch)
    acc[1], acc[4] = most, most
    path = np.sort(np.stack([rng.permutation(Mt)[:most] for _ in range(batch)]), 1)
    t = lambda x: torch.tensor(x, dtype=torch.int32, device=dev)
    ks, vs = ([torch.randn((batch, Hkv, nb * B, D), device=dev).to(dt) for _ in range(layers)] for _ in range(2))
    bk, bv = ([torch.randn((batch, P + Mt, Hkv, D), device=dev).to(dt) for _ in range(layers)] for _ in range(2))
    kx, kn = ([torch.full((batch, Hkv, nb, D), 7.0, device=dev, dtype=dt) for _ in range(layers)] for _ in range(2))
    want = [[x.clone() for x in y] for y in (ks, vs, kx, kn)]
    for b in range(batch):
        rows = [P - pend[b] + i for i in range(pend[b])] + [P + path[b, i] for i in range(acc[b])]
        rows = rows[:max(0, nb * B - ctx[b])]
        n = len(rows)
        for l in range(layers):
            if n == 0:
                continue
            want[0][l][b, :, ctx[b]:ctx[b] + n] = bk[l][b, rows].transpose(0, 1)
            want[1][l][b, :, ctx[b]:ctx[b] + n] = bv[l][b, rows].transpose(0, 1)
            for i in range(ctx[b] // B, (ctx[b] + n - 1) // B + 1):
                block = want[0][l][b, :, i * B:min((i + 1) * B, ctx[b] + n)]
                want[2][l][b, :, i], want[3][l][b, :, i] = block.amax(1), block.amin(1)
    ctx_d, pend_d = t(ctx), t(pend)
    kvs = [sp.KV(ks[l], vs[l], ctx_d, B, nb) for l in range(layers)]
    ws = torch.zeros((sp.specpv_workspace_bytes(kvs[0]),), dtype=torch.uint8, device=dev)
    sp.specpv_commit_accepted_layers(kvs, bk, bv, P, Mt, pend_d, t(path), t(acc), sp.MODE_REFRESH, kmaxs=kx, kmins=kn, workspace=ws)
    torch.cuda.synchronize()
    for l in range(layers):
        for got, ref in zip((ks[l], vs[l], kx[l], kn[l]), (w[l] for w in want)):
            assert torch.equal(got, ref), l


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("P,most", [(28, 5), (31, 1), (32, 1), (32, 9), (33, 4), (64, 40)])
def test_rows_within_the_buffer(gpu_lib, dtype, D, P, most):
    sp, dev = gpu_lib, torch.device("cuda")
    say("case", dtype, D, P, most)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    Hkv, Mt, layers = 3, most + 5, 2
    pend = np.array([0, P, P - 1, P // 2, max(0, P - most), 3])
    acc = np.array([most, most, most, 0, most, 1])
    batch = len(pend)
    rng = np.random.default_rng(P + D + most)
    path = np.sort(np.stack([rng.permutation(Mt)[:most] for _ in range(batch)]), 1)
    t = lambda x: torch.tensor(x, dtype=torch.int32, device=dev)
    cache = torch.zeros((batch, Hkv, 16, D), device=dev, dtype=dt)
    bk, bv = ([torch.randn((batch, P + Mt, Hkv, D), device=dev).to(dt) for _ in range(layers)] for _ in range(2))
    want = [[x.clone() for x in y] for y in (bk, bv)]
    stored = []
    for b in range(batch):
        rows = ([P - pend[b] + i for i in range(pend[b])] + [P + path[b, i] for i in range(acc[b])])[:P]
        stored.append(len(rows))
        for w, src in zip(want, (bk, bv)):
            for l in range(layers):
                w[l][b, P - len(rows):P] = src[l][b, rows]
    pend_d, ctx_d = t(pend), t([0] * batch)
    kvs = [sp.KV(cache, cache.clone(), ctx_d, 16, 1) for _ in range(layers)]
    ws = torch.zeros((sp.specpv_workspace_bytes(kvs[0]),), dtype=torch.uint8, device=dev)
    sp.specpv_commit_accepted_layers(kvs, bk, bv, P, Mt, pend_d, t(path), t(acc), sp.MODE_PARTIAL, workspace=ws)
    torch.cuda.synchronize()
    assert pend_d.tolist() == stored
    for l in range(layers):
        assert torch.equal(bk[l], want[0][l]) and torch.equal(bv[l], want[1][l]), l
