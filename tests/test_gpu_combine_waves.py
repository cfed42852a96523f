"""The merge of the partials with one and with two wavefronts per four rows: on both sides of each line between the two (rows,
query heads per KV head, up to eight splits and more, shares of a batch, partially verified tokens that it attends itself),
against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from helpers import ATOL, GpuRun, say, with_pending
from test_gpu_parity import SMALL

pytestmark = pytest.mark.gpu

CASES = [  # (over, partially verified tokens); workgroups are sequences * KV heads * nodes, the lines at 256 and 512 of them
    (dict(ctx=[300], M=32, Hq=32, Hkv=8), 0), (dict(ctx=[300], M=33, Hq=32, Hkv=8), 0), (dict(ctx=[300, 290], M=17, Hq=24, Hkv=8), 0),
    (dict(ctx=[300], M=64, Hq=40, Hkv=8), 0), (dict(ctx=[300], M=65, Hq=40, Hkv=8), 0), (dict(ctx=[200], M=128, Hq=64, Hkv=4), 0),
    (dict(ctx=[300], M=128, Hq=4, Hkv=2), 0), (dict(ctx=[300], M=129 // 3, Hq=18, Hkv=6), 9),
    (dict(ctx=[9000], M=33, Hq=32, Hkv=8), 0), (dict(ctx=[4000], M=16, Hq=32, Hkv=2), 0), (dict(ctx=[9000], M=65, Hq=40, Hkv=8), 11),
    (dict(ctx=[6000, 33, 3000], M=60, Hq=32, Hkv=8), 0), (dict(ctx=[3000, 2999], M=37, Hq=40, Hkv=8, D=64), 0),
    (dict(ctx=[500], M=32, Hq=32, Hkv=8, D=64, dtype="f32"), 0), (dict(ctx=[500], M=33, Hq=32, Hkv=8, dtype="f32"), 0),
    (dict(ctx=[500, 200], M=64, Hq=32, Hkv=8, D=64, dtype="f32"), 16), (dict(ctx=[300, 200], M=65, Hq=32, Hkv=8, dtype="f32"), 16),
    (dict(ctx=[2500, 200], M=65, Hq=32, Hkv=8, D=64, dtype="f32"), 20)]


@pytest.mark.parametrize("over,n_key", CASES, ids=["-".join(str(v) for v in o.values()) + "-%d" % n for o, n in CASES])
def test_either_form_against_the_oracle(gpu_lib, over, n_key):
    say("case", over, n_key)
    cfg = dict(SMALL, B=32, name="waves")
    cfg.update(over, rho=[0.1] * len(over["ctx"]))
    case = workloads.make_case(cfg, seed=71)
    if n_key:
        case = with_pending(case, n_key, seed=72)
    case = workloads.to_device(case, "cuda")
    run = GpuRun(gpu_lib, case)
    run.attend(None, None)
    torch.cuda.synchronize()
    worst = 0.0
    for b in range(case["batch"]):
        o = workloads.oracle_views(case, b)
        O, LSE, _ = oracle.tree_attention(o["Q"], o["K"], o["V"], o["Kd"], o["Vd"], o["parent"], case["B"], None, None, n_key_only=n_key)
        worst = max(worst, np.abs(run.out[b].float().cpu().numpy() - O).max())
        np.testing.assert_allclose(run.lse[b].cpu().numpy(), LSE, atol=2e-5 if case["dtype"] == "f32" else 2e-3, rtol=1e-5)
    say("   max-abs err %.3g" % worst)
    assert worst <= ATOL[case["dtype"]]
