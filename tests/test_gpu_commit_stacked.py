"""A commit of layers whose tensors lie at one distance from each other (slices of one tensor, in order or backwards) against the same
layers one by one, and against layers that lie anywhere or of which one does: caches, buffers, summaries, lists and counters the same."""
import pytest
import torch

from helpers import say

pytestmark = pytest.mark.gpu

NAMES = ("k", "v", "bk", "bv", "kx", "kn", "idx", "cnt")


def _tensors(layers, batch, Hkv, D, B, nb, P, Mt, n_sel):
    g = torch.Generator(device="cuda").manual_seed(3)
    r = lambda *s: torch.randn(s, generator=g, device="cuda").bfloat16()
    x = dict(k=r(layers, batch, Hkv, nb * B, D), v=r(layers, batch, Hkv, nb * B, D), bk=r(layers, batch, P + Mt, Hkv, D), bv=r(layers, batch, P + Mt, Hkv, D),
             kx=r(layers, batch, Hkv, nb, D), kn=r(layers, batch, Hkv, nb, D))
    x["idx"] = torch.full((layers, batch, Hkv, n_sel), -1, dtype=torch.int32, device="cuda")
    x["idx"][..., :2] = torch.arange(2, dtype=torch.int32, device="cuda")
    x["cnt"] = torch.full((layers, batch, Hkv), 2, dtype=torch.int32, device="cuda")
    return x


@pytest.mark.parametrize("layers", [1, 2, 3, 33, 40])
@pytest.mark.parametrize("to_cache", [True, False])
@pytest.mark.parametrize("how", ["stacked", "backwards", "every second", "one apart", "apart"])
def test_against_layer_by_layer(gpu_lib, layers, to_cache, how):
    sp = gpu_lib
    say("case", layers, to_cache, how)
    batch, Hkv, D, B, nb, P, Mt, n_sel = 2, 3, 64, 16, 6, 9, 7, 5
    base = _tensors(2 * layers, batch, Hkv, D, B, nb, P, Mt, n_sel)
    i32 = lambda v: torch.tensor(v, dtype=torch.int32, device="cuda")
    results = []
    for together in (True, False):
        x = {n: t.clone() for n, t in base.items()}
        order = list(range(layers))[::-1] if how == "backwards" else (list(range(0, 2 * layers, 2)) if how == "every second" else list(range(layers)))
        t = {n: [x[n][i] for i in order] for n in NAMES}
        if how == "apart":
            between = []   # allocations of growing size, so that the clones are at no one distance
            for n, v in t.items():
                for i in range(layers):
                    between.append(torch.empty(1 + 4096 * i * i, device="cuda"))
                    v[i] = v[i].clone()
        if how == "one apart":
            t["v"][-1] = t["v"][-1].clone()
        ctx, pend, dropped = i32([37, 60]), i32([5, 0]), torch.zeros((batch, 2), dtype=torch.int32, device="cuda")
        kvs = [sp.KV(t["k"][l], t["v"][l], ctx, B, nb) for l in range(layers)]
        ws = torch.zeros((sp.specpv_workspace_bytes(kvs[0]),), dtype=torch.uint8, device="cuda")
        acc, n_acc, mode = i32([[0, 2, 5], [1, 3, 6]]), i32([3, 2]), sp.MODE_REFRESH if to_cache else sp.MODE_PARTIAL
        if together:
            sp.specpv_commit_accepted_layers(kvs, t["bk"], t["bv"], P, Mt, pend, acc, n_acc, mode, t["kx"], t["kn"], ws, t["idx"], t["cnt"], dropped)
        else:
            for l in range(layers):   # the counters move with every call: put back for all but the last
                if l:
                    ctx.copy_(i32([37, 60])); pend.copy_(i32([5, 0]))
                sp.specpv_commit_accepted(kvs[l], t["bk"][l], t["bv"][l], P, Mt, pend, acc, n_acc, mode, t["kx"][l], t["kn"][l], ws, t["idx"][l], t["cnt"][l], dropped)
        torch.cuda.synchronize()
        results.append([torch.stack(t[n]) for n in NAMES] + [ctx, pend, dropped, ws] + ([x[n] for n in NAMES] if how != "apart" else []))
    for a, b in zip(*results):
        assert torch.equal(a, b)
