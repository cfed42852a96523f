"""How a short call's workgroups find their (sequence, KV head): by shifts with 8, 16, 32, ... KV heads, by division with any
other number of them, with one and with several sequences, with lists and without, query heads of every group size."""
import ctypes

import numpy as np
import pytest
import torch

import workloads
from paper_2512_02337_amd import binding
from helpers import GpuRun, say
from test_gpu_parity import SMALL, _check_attn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("G,M", [(1, 17), (4, 16), (5, 60)])
@pytest.mark.parametrize("ctx", [[1500], [1500, 33, 700]])
@pytest.mark.parametrize("Hkv", [4, 7, 8, 16, 24, 32])
def test_heads_and_sequences(gpu_lib, Hkv, ctx, G, M):
    cfg = dict(SMALL, ctx=ctx, B=32, M=M, Hq=G * Hkv, Hkv=Hkv, rho=[0.1] * len(ctx))
    say("case", cfg)
    case = workloads.to_device(workloads.make_case(cfg, seed=47), "cuda")
    run = GpuRun(gpu_lib, case)
    run.summarize(); run.select(); run.attend()
    torch.cuda.synchronize()
    sel = [(run.sel_idx.cpu().numpy()[b], run.sel_count.cpu().numpy()[b]) for b in range(case["batch"])]
    tag = "%d KV heads, G = %d, %d nodes, %s" % (Hkv, G, M, ctx)
    _check_attn(run, case, sel, tag + " kept")
    run.out.zero_()
    run.attend(None, None)
    torch.cuda.synchronize()
    _check_attn(run, case, None, tag + " all")


@pytest.mark.parametrize("Hkv", [4, 8])
@pytest.mark.parametrize("M", [16, 60])
def test_list_without_room(gpu_lib, M, Hkv):
    """Lists of no entries (n_sel = 0, whatever the counts say): the draft tree alone, and nothing read from the lists."""
    cfg = dict(SMALL, ctx=[1500], B=32, M=M, Hq=4 * Hkv, Hkv=Hkv)
    say("case", cfg)
    case = workloads.to_device(workloads.make_case(cfg, seed=47), "cuda")
    run = GpuRun(gpu_lib, case)
    run.sel_count.fill_(3)
    ptr = lambda t: ctypes.c_void_p(t.data_ptr())
    rc = binding.load().specpv_partial_verify_attn(ctypes.byref(run.kv.c), ctypes.byref(run.tree.c), ptr(run.sel_idx), ptr(run.sel_count), 0,
                                                   ptr(run.out), ptr(run.lse), ptr(run.ws), run.ws.numel(),
                                                   ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0
    torch.cuda.synchronize()
    none = (np.zeros((Hkv, run.sel_idx.shape[-1]), np.int32), np.zeros(Hkv, np.int32))
    _check_attn(run, case, [none], "no entries, %d KV heads" % Hkv)
