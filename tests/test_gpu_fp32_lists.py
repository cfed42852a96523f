"""The fp32 attention over lists that it keeps in registers (up to 256 entries), reads from memory (more), and over lists whose
tokens it counts in 64 bits, against the oracle; full lists, short counts and entries that name no block."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from helpers import ATOL, GpuRun, say
from test_gpu_parity import SMALL

pytestmark = pytest.mark.gpu

CASES = [  # (over, entries of a list row, entries that count)
    (dict(ctx=[700], B=7, M=5), 1, 1), (dict(ctx=[1300], B=16, M=16, D=64), 64, 61), (dict(ctx=[1500, 900], B=5, M=9), 65, 65),
    (dict(ctx=[5000], B=16, M=24, D=64), 256, 256), (dict(ctx=[5000], B=16, M=24), 257, 257), (dict(ctx=[4000], B=9, M=7, D=64), 300, 40),
    (dict(ctx=[600], B=16, M=3), 200, 0), (dict(ctx=[700], B=1 << 19, M=4, Hq=2, Hkv=1, D=64), 4096, 2)]


@pytest.mark.parametrize("over,n_row,count", CASES)
def test_lists(gpu_lib, over, n_row, count):
    say("case", over, n_row, count)
    cfg = dict(SMALL, dtype="f32", name="f32 lists", ns=0, nr=0)
    cfg.update(over, rho=[0.0] * len(over["ctx"]))
    case = workloads.make_case(cfg, seed=51, device="cuda")
    run = GpuRun(gpu_lib, case)
    rng = np.random.default_rng(3)
    lists = np.full((case["batch"], case["Hkv"], n_row), -1, dtype=np.int32)
    for b, L in enumerate(over["ctx"]):
        nb = (L + case["B"] - 1) // case["B"]
        for g in range(case["Hkv"]):
            own = np.sort(rng.permutation(nb)[:count]).astype(np.int32)
            lists[b, g, :len(own)] = own
            if len(own) > 3:
                lists[b, g, 1] = -1      # names no block
    counts = np.full((case["batch"], case["Hkv"]), count, dtype=np.int32)
    run.attend(torch.from_numpy(lists).cuda(), torch.from_numpy(counts).cuda())
    torch.cuda.synchronize()
    for b in range(case["batch"]):
        o = workloads.oracle_views(case, b)
        kept = [lists[b, g][lists[b, g] >= 0] for g in range(case["Hkv"])]
        idx = np.full((case["Hkv"], max(1, max(len(x) for x in kept))), -1, dtype=np.int32)
        for g, x in enumerate(kept):
            idx[g, :len(x)] = x
        O, LSE, _ = oracle.tree_attention(o["Q"], o["K"], o["V"], o["Kd"], o["Vd"], o["parent"], case["B"], idx, np.array([len(x) for x in kept], dtype=np.int32))
        worst = np.abs(run.out[b].cpu().numpy() - O).max()
        say("   max-abs err %.3g" % worst)
        assert worst <= ATOL["f32"]
        np.testing.assert_allclose(run.lse[b].cpu().numpy(), LSE, atol=2e-5, rtol=1e-5)
