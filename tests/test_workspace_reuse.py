"""One workspace for the trees of a decode loop: sized for the largest, it serves every smaller tree, batch and cache."""
import ctypes
import random

import numpy as np
import pytest
import torch

import oracle
import paper_2512_02337_amd as specpv
import workloads
from helpers import ATOL, GpuRun, say
from test_abi_cpu import _cfg, _kv, _tree

EWORKSPACE = -2


def _calls(kv, tree, cfg, nbytes, pending):
    """Statuses of the full pass, the refresh (scores in the workspace) and the partial step; pointers are never followed:
    without a GPU the calls end at their first launch."""
    lib, B, vp = specpv.load(), ctypes.byref, ctypes.c_void_p
    ws = (vp(0x100000), nbytes, None)
    n_sel = cfg.n_sink_blocks + cfg.n_recent_blocks + cfg.k_blocks + cfg.n_extra_slots
    keys = _tree(M=tree.M + pending, n_q_heads=tree.n_q_heads, n_key_only=pending, last_node=pending)
    return (lib.specpv_partial_verify_attn(B(kv), B(tree), None, None, 0, vp(0x300), None, *ws),
            lib.specpv_full_verify_refresh(B(kv), B(tree), vp(16), vp(32), -1, B(cfg), vp(0x300), None, vp(0x100), vp(0x200), None, *ws),
            lib.specpv_partial_verify_attn(B(kv), B(keys), vp(0x100), vp(0x200), n_sel, vp(0x300), None, *ws))


def _shape(Hkv, G, nb, B=64, D=128, dtype=1, batch=1):
    return _kv(n_kv_heads=Hkv, head_dim=D, block_size=B, max_blocks=nb, batch=batch, dtype=dtype, stride_t=D, stride_h=nb * B * D, stride_b=Hkv * nb * B * D)


def _bytes(kv, tree, cfg):
    return specpv.load().specpv_workspace_bytes(ctypes.byref(kv), ctypes.byref(tree), ctypes.byref(cfg))


no_gpu = pytest.mark.skipif(torch.cuda.is_available(), reason="made-up addresses: only where no kernel can be launched")


@no_gpu
@pytest.mark.parametrize("ctx,Hkv,G", [(16384, 8, 4), (4096, 8, 5), (65536, 2, 8), (4096, 8, 4), (131072, 8, 4)])
def test_smaller_trees_fit(ctx, Hkv, G):
    kv, cfg = _shape(Hkv, G, ctx // 64), _cfg(n_recent_blocks=8, k_blocks=55, n_extra_slots=2)
    sized = _bytes(kv, _tree(M=64, n_q_heads=Hkv * G), cfg)
    with_pending = _bytes(kv, _tree(M=84, n_q_heads=Hkv * G), cfg)   # sized for a refresh with 20 pending tokens
    for M in range(1, 65):
        assert EWORKSPACE not in _calls(kv, _tree(M=M, n_q_heads=Hkv * G), cfg, sized, 0), (ctx, Hkv, G, M)
        assert EWORKSPACE not in _calls(kv, _tree(M=M, n_q_heads=Hkv * G), cfg, with_pending, 20), (ctx, Hkv, G, M)


@no_gpu
def test_any_smaller_shape_fits():
    rnd = random.Random(11)
    for _ in range(1500):
        Hkv, G, D, dtype = rnd.choice([1, 2, 4, 8]), rnd.choice([1, 2, 4, 5, 8]), rnd.choice([64, 128]), rnd.choice([0, 1, 1])
        B, nb, batch, M = rnd.choice([7, 16, 32, 64]), rnd.choice([8, 64, 500, 2048, 8192]), rnd.choice([1, 2, 4, 16]), rnd.randint(2, 128)
        cfg = _cfg(n_recent_blocks=8, k_blocks=rnd.choice([4, 55, 246]))
        sized = _bytes(_shape(Hkv, G, nb, B, D, dtype, batch), _tree(M=M, n_q_heads=Hkv * G), cfg)
        less = dict(nb=rnd.randint(1, nb), batch=rnd.randint(1, batch), M=rnd.randint(1, M))
        kv, tree = _shape(Hkv, G, less["nb"], B, D, dtype, less["batch"]), _tree(M=less["M"], n_q_heads=Hkv * G)
        assert EWORKSPACE not in _calls(kv, tree, cfg, sized, 0), (Hkv, G, D, dtype, B, nb, batch, M, less)
    # what cannot hold one split is still refused
    kv, tree = _shape(8, 4, 256), _tree()
    one = 65536 + 8 * 4 * 60 * (128 * 2 + 8)
    assert EWORKSPACE not in _calls(kv, tree, _cfg(), one + 512, 0)
    assert _calls(kv, tree, _cfg(), one - 256, 0) == (EWORKSPACE,) * 3


@no_gpu
@pytest.mark.parametrize("Hkv,G,D,B,nb,batch,M", [(1, 4, 128, 64, 261, 9, 60), (8, 1, 128, 64, 775, 65, 18), (4, 4, 128, 7, 1735, 2, 60),
                                                  (1, 4, 128, 64, 236, 9, 60), (1, 1, 64, 7, 7228, 100, 60), (2, 1, 64, 32, 6242, 100, 60)])
def test_full_passes_that_fit_the_static_array(Hkv, G, D, B, nb, batch, M):
    """Long full passes over batches whose partials fit the library's own array with the splits of equally long
    sequences: what is done about uneven lengths does not take them beyond it."""
    lib, vp = specpv.load(), ctypes.c_void_p
    rc = lib.specpv_partial_verify_attn_static(ctypes.byref(_shape(Hkv, G, nb, B, D, 1, batch)), ctypes.byref(_tree(M=M, n_q_heads=Hkv * G)),
                                               None, None, 0, vp(0x300), None, None)
    assert rc == -4, rc   # as far as the first launch; -3: the array is too small


SHAPE = dict(Hq=16, Hkv=2, D=128, dtype="bf16", B=64, M=40, tree="bounded", ns=1, nr=4, k=27, beta=1.5, layers=1, name="reuse")


@pytest.mark.gpu
@pytest.mark.parametrize("over", [dict(ctx=[9000]), dict(ctx=[700], M=1), dict(ctx=[9000, 3000, 60]), dict(ctx=[9000, 3000, 60], D=64),
                                  dict(ctx=[2500], D=64, M=7), dict(ctx=[1500], dtype="f32", D=64)])
@pytest.mark.parametrize("splits", [1, 3, 1000])
def test_results_and_bounds_in_a_small_workspace(gpu_lib, over, splits):
    """A workspace with room for that many splits (1000: the plan's own): the oracle's results, and not a byte behind it."""
    c = dict(SHAPE, **over)
    c["rho"] = [0.1] * len(c["ctx"])
    case = workloads.to_device(workloads.make_case(c, seed=7), "cuda")
    run = GpuRun(gpu_lib, case)
    rows = len(c["ctx"]) * c["Hq"] * c["M"]
    row = c["D"] * (2 if c["D"] == 128 and c["dtype"] == "bf16" else 4) + 8
    # (in a batch, room for the shares of a few workgroups as well)
    scores = 65536 + ((len(c["ctx"]) * c["Hkv"] * run.kv.max_blocks * 4 + 255) & ~255)
    size = max(65536 + 512 + splits * rows * row, scores)
    size = min(size, run.ws.numel()) & ~255
    buf = torch.zeros((size + 4096,), dtype=torch.uint8, device="cuda")
    buf[size:] = 0x5a
    run.ws = buf[:size]
    for full in (False, True):
        if full:   # scores in the workspace, where the partials were
            want = run.sel_idx.clone(), run.sel_count.clone()
            run.sel_idx.fill_(-7)
            gpu_lib.specpv_full_verify_refresh(run.kv, run.tree, run.kmax, run.kmin, 0, run.cfg, run.out, run.lse, run.sel_idx, run.sel_count, None, run.ws)
            assert torch.equal(run.sel_idx, want[0]) and torch.equal(run.sel_count, want[1])
        else:
            run.summarize(); run.select(); run.attend()
        torch.cuda.synchronize()
        worst = 0.0
        for b in range(case["batch"]):
            o = workloads.oracle_views(case, b)
            idx, cnt = (None, None) if full else (run.sel_idx.cpu().numpy()[b], run.sel_count.cpu().numpy()[b])
            O, _, _ = oracle.tree_attention(o["Q"], o["K"], o["V"], o["Kd"], o["Vd"], o["parent"], case["B"], idx, cnt)
            worst = max(worst, np.abs(run.out[b].float().cpu().numpy() - O).max())
        say("   %s, room for %d splits, %s: max-abs err %.3g" % (over, splits, "full" if full else "partial", worst))
        assert worst <= ATOL[c["dtype"]], (over, splits, full, worst)
        assert bool((buf[size:] == 0x5a).all()) and int(buf[:65536].sum()) == 0
