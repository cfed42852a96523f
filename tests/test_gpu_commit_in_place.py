"""A commit whose buffer lies in the cache it goes to: one sequence, token-major, the pending rows and the candidates written where the
cache goes on, so that rows move up within one array.  Rows and summaries bit for bit those of a commit from a buffer elsewhere."""
import numpy as np
import pytest
import torch

from helpers import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("P,pend,Mt,most,B,L", [(0, 0, 60, 8, 16, 130), (20, 18, 60, 6, 64, 250), (0, 0, 128, 128, 16, 5), (90, 90, 38, 38, 1, 77), (20, 3, 40, 40, 250, 249)])
@pytest.mark.parametrize("ahead", [0, 3])   # rows between the cache's end and the buffer
def test_buffer_at_the_cache_s_end(gpu_lib, dtype, D, P, pend, Mt, most, B, L, ahead):
    sp, dev = gpu_lib, torch.device("cuda")
    say("case", dtype, D, P, pend, Mt, most, B, L, ahead)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    Hkv, layers = 5, 3
    nb = (L + ahead + P + Mt + B) // B + 1
    gen = torch.Generator(device=dev).manual_seed(P + Mt + B)
    path = torch.randperm(Mt, generator=gen, device=dev)[:most].sort().values.to(torch.int32).view(1, most)
    t = lambda x: torch.tensor([x], dtype=torch.int32, device=dev)

    def state():
        gen.manual_seed(9)
        ks, vs = ([torch.randn((1, nb * B, Hkv, D), generator=gen, device=dev).to(dt) for _ in range(layers)] for _ in range(2))
        kx, kn = ([torch.full((1, Hkv, nb, D), 7.0, device=dev, dtype=dt) for _ in range(layers)] for _ in range(2))
        return ks, vs, kx, kn

    got = []
    for in_place in (False, True):
        ks, vs, kx, kn = state()
        at = slice(L + ahead, L + ahead + P + Mt)
        bk, bv = [[x[:, at] if in_place else x[:, at].clone() for x in y] for y in (ks, vs)]
        ctx, n_pending, n_acc = t(L), t(pend), t(most)
        kvs = [sp.KV(ks[l], vs[l], ctx, B, nb, "bthd") for l in range(layers)]
        ws = torch.zeros((sp.specpv_workspace_bytes(kvs[0]),), dtype=torch.uint8, device=dev)
        sp.specpv_commit_accepted_layers(kvs, bk, bv, P, Mt, n_pending, path, n_acc, sp.MODE_REFRESH, kmaxs=kx, kmins=kn, workspace=ws)
        torch.cuda.synchronize()
        n = L + pend + most
        assert int(ctx) == n and int(n_pending) == 0
        used = slice((L // B), (n - 1) // B + 1)
        got.append([[x[:, :n] for x in ks], [x[:, :n] for x in vs], [x[:, :, used] for x in kx], [x[:, :, used] for x in kn]])
    start = state()
    rows = [L + ahead + P - pend + i for i in range(pend)] + [L + ahead + P + int(i) for i in path[0]]
    for l in range(layers):
        for x in range(2):
            want = torch.cat([start[x][l][:, :L], start[x][l][:, rows]], 1)
            assert torch.equal(got[0][x][l], want) and torch.equal(got[1][x][l], want), (l, x)
        for x in (2, 3):
            assert torch.equal(got[0][x][l], got[1][x][l]), (l, x)
