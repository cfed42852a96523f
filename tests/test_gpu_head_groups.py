"""How a short call's workgroups find their (sequence, KV head): by shifts with 8, 16, 32, ... KV heads, by division with any
other number of them, with one and with several sequences, with lists and without, query heads of every group size."""
import pytest
import torch

import workloads
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
