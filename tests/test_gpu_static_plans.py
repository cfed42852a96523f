"""specpv_partial_verify_attn_static runs the plan of the call with a workspace, also where its partial results take more than the
bytes by which it takes calls: bit-identical results, by splits and by shares.  Splits and shares of a full pass over sequences of very
different lengths on either side of where the plan changes from one to the other, against the oracle."""
import numpy as np
import pytest
import torch

import workloads
from helpers import GpuRun, say
from test_gpu_parity import SMALL, _check_attn

pytestmark = pytest.mark.gpu

LARGE = [dict(ctx=[30011, 15005], D=64, B=32, M=37, Hq=32, Hkv=8), dict(ctx=[16000], dtype="f32", B=64, M=37, Hq=32, Hkv=8), dict(ctx=[60000, 90, 31000], D=64, B=64, M=37, Hq=32, Hkv=8),
         dict(ctx=[9000], dtype="f32", B=64, M=60, Hq=16, Hkv=4), dict(ctx=[9000, 7000], B=64, M=37, Hq=32, Hkv=8)]


@pytest.mark.parametrize("over", LARGE, ids=["-".join(str(v) for v in o.values()) for o in LARGE])
def test_large_partials_in_the_array(gpu_lib, over):
    say("case", over)
    cfg = dict(SMALL)
    cfg.update(over, rho=[0.1] * len(over["ctx"]))
    run = GpuRun(gpu_lib, workloads.make_case(cfg, seed=3, device=torch.device("cuda")))
    run.attend(None, None)
    out, lse = torch.zeros_like(run.out), torch.zeros_like(run.lse)
    gpu_lib.specpv_partial_verify_attn_static(run.kv, run.tree, None, None, out, lse)
    torch.cuda.synchronize()
    assert torch.equal(out, run.out) and torch.equal(lse, run.lse)


UNEVEN = [  # on either side: 48 chunks of 32 tokens to a split (64 channels: 32), and a round of workgroups more or less
    dict(ctx=[3000, 180, 2999, 1, 0, 3000, 64, 1500], M=30, Hq=10, Hkv=2), dict(ctx=[6200, 0, 370, 6200], M=24, Hq=8, Hkv=2), dict(ctx=[9000, 500], M=37, Hq=16, Hkv=2),
    dict(ctx=[9000, 8999], M=3, Hq=8, Hkv=8), dict(ctx=[1100, 70, 1025, 33], D=64, M=37, Hq=8, Hkv=2), dict(ctx=[9000, 40, 0, 4000], D=64, M=5, Hq=10, Hkv=2)]


@pytest.mark.parametrize("over", UNEVEN, ids=["-".join(str(v) for v in o.values()) for o in UNEVEN])
def test_lengths_of_every_kind(gpu_lib, over):
    say("case", over)
    cfg = dict(SMALL)
    cfg.update(over, rho=[0.1] * len(over["ctx"]))
    case = workloads.to_device(workloads.make_case(cfg, seed=5), "cuda")
    run = GpuRun(gpu_lib, case)
    run.refresh(stale=0)
    torch.cuda.synchronize()
    _check_attn(run, case, None, "full")
    assert int(run.ws[:65536].sum()) == 0
