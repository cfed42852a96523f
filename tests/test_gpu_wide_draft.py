"""Draft K / V of one sequence beyond what 32 bits address: nodes behind that line attend their own rows."""
import pytest
import torch

from helpers import say

pytestmark = pytest.mark.gpu


def test_nodes_behind_the_line(gpu_lib):
    sp, dev = gpu_lib, torch.device("cuda")
    M, H, D, L = 128, 66100, 128, 3   # 127 * 66100 * 512 bytes > 2^32
    say("case", M, H, D)
    gen = torch.Generator(device=dev).manual_seed(3)
    rnd = lambda *shape: torch.randn(shape, generator=gen, device=dev)
    k, v, kd, vd, q = rnd(1, H, L, D), rnd(1, H, L, D), rnd(1, M, H, D), rnd(1, M, H, D), rnd(1, M, H, D)
    parent = [-1] + [i - 1 if i % 40 else 0 for i in range(1, M)]   # paths of up to 41 nodes, the last ones behind the line
    kv = sp.KV(k, v, torch.tensor([L], dtype=torch.int32, device=dev), 1, L)
    tree = sp.Tree(q, kd, vd, torch.tensor([parent], dtype=torch.int32, device=dev))
    ws = torch.zeros((sp.specpv_workspace_bytes(kv, tree, None),), dtype=torch.uint8, device=dev)
    out = torch.zeros_like(q)
    sp.specpv_partial_verify_attn(kv, tree, None, None, out, None, ws)
    torch.cuda.synchronize()
    heads = [0, 1, 33000, H - 2, H - 1]
    f = lambda x: x.double().cpu()
    for j in (0, 5, 63, 64, 119, 126, 127):
        path, at = [], j
        while at >= 0:
            path.append(at)
            at = parent[at]
        for h in heads:
            kk, vv = torch.cat([f(k[0, h]), f(kd[0, path, h])]), torch.cat([f(v[0, h]), f(vd[0, path, h])])
            want = torch.softmax(kk @ f(q[0, j, h]) / D ** 0.5, 0) @ vv
            assert (f(out[0, j, h]) - want).abs().max() <= 1e-5, (j, h)   # (the fp32 bar)
