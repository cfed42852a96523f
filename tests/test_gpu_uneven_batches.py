"""Full passes over batches whose sequences differ in length, on either side of where the plan turns to the group kernel
(256 chunks of 32 tokens; one KV head keeps the tile kernel, whose ranges are short there) and of where it deals shares of the
chunks (64 sequences).  test_plans_cpu.py holds which of them go by shares."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from helpers import ATOL, GpuRun, say

pytestmark = pytest.mark.gpu

BASE = dict(Hq=4, Hkv=1, D=128, dtype="bf16", B=32, M=9, tree="bounded", ns=1, nr=2, k=5, beta=1.5, layers=1, name="uneven")
CASES = [
    (dict(ctx=[8192, 500, 31]), "256 chunks"),
    (dict(ctx=[8193, 500, 31]), "257, one head"),
    (dict(ctx=[8300, 0, 4000], M=1), "one head, one node, an empty sequence"),
    (dict(ctx=[8192, 500, 31], Hq=32, Hkv=8), "256, eight heads"),
    (dict(ctx=[8193, 500, 31], Hq=32, Hkv=8), "257, eight heads: shares"),
    (dict(ctx=[8193, 500, 31], Hq=32, Hkv=8, M=60), "257, eight row blocks: shares"),
    (dict(ctx=[8300, 0, 4000], M=1, Hq=32, Hkv=8), "one node, an empty sequence: shares"),
    (dict(ctx=[8500] + [40 + 3 * i for i in range(64)], M=3), "65 sequences: splits"),
    (dict(ctx=[8500] + [40 + 3 * i for i in range(63)], M=3), "64 sequences: shares"),
    (dict(ctx=[8500] + [40 + 3 * i for i in range(64)], M=3, D=64), "65 sequences, 64 channels"),
]


@pytest.mark.parametrize("over,tag", CASES)
def test_against_the_oracle(gpu_lib, over, tag):
    c = dict(BASE, **over)
    c["rho"] = [0.1] * len(c["ctx"])
    case = workloads.to_device(workloads.make_case(c, seed=5), "cuda")
    run = GpuRun(gpu_lib, case)
    run.summarize()
    for _ in range(2):   # the workspace as the first pass left it
        run.out.fill_(7.0)
        run.attend(None, None)
        torch.cuda.synchronize()
        worst = 0.0
        for b in range(case["batch"]):
            o = workloads.oracle_views(case, b)
            O, lse, _ = oracle.tree_attention(o["Q"], o["K"], o["V"], o["Kd"], o["Vd"], o["parent"], case["B"])
            worst = max(worst, np.abs(run.out[b].float().cpu().numpy() - O).max())
            np.testing.assert_allclose(run.lse[b].cpu().numpy(), lse, atol=2e-3, rtol=1e-5)
        say("   %s: max-abs err %.3g" % (tag, worst))
        assert worst <= ATOL[c["dtype"]], (tag, worst)
