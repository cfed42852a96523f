"""Draft rows that are not finite: a path whose products all overflow to minus infinity weighs nothing beside a finite context, and an
infinity in a V row reaches the rows that descend from its node and no other, whether the path fills its last four slots or not.
One wavefront and two per four rows, rows by node and packed, every form of partials, and the merge beside the scores of a refresh."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from helpers import ATOL, GpuRun, say
from test_gpu_parity import SMALL

pytestmark = pytest.mark.gpu

CASES = [  # two wavefronts that share the tree, one, packed, more than eight / sixteen partials, shares, fp32, 64 channels
    dict(ctx=[700], M=24), dict(ctx=[700] * 8, M=60, Hq=32, Hkv=8), dict(ctx=[900], M=33, Hq=40, Hkv=8), dict(ctx=[700] * 11, M=60, Hq=40, Hkv=8),
    dict(ctx=[4000], M=60, Hq=32, Hkv=8), dict(ctx=[30000], M=60, Hq=32, Hkv=8), dict(ctx=[9000, 300], M=37, Hq=32, Hkv=8), dict(ctx=[300], M=9, dtype="f32"),
    dict(ctx=[300] * 40, M=60, Hq=32, Hkv=8, dtype="f32", D=64), dict(ctx=[2000, 900], M=37, Hq=16, Hkv=4, D=64), dict(ctx=[900], M=70, Hq=10, Hkv=2, D=64)]


def _run(sp, over, tree, full, change):
    say("case", over, tree, full)
    cfg = dict(SMALL, B=32, name="infinite", tree=tree)
    cfg.update(over, rho=[0.1] * len(over["ctx"]))
    case = workloads.make_case(cfg, seed=71)
    change(case)
    case = workloads.to_device(case, "cuda")
    run = GpuRun(sp, case)
    if full:
        run.refresh()
    else:
        run.attend(None, None)
    torch.cuda.synchronize()
    return case, run.out.float().cpu().numpy(), run.lse.cpu().numpy()


@pytest.mark.parametrize("full", [False, True], ids=["attention", "refresh"])
@pytest.mark.parametrize("tree", ["chain", "bounded"])
@pytest.mark.parametrize("over", CASES, ids=["-".join(str(v) for v in o.values()) for o in CASES])
def test_products_of_minus_infinity(gpu_lib, over, tree, full):
    def change(case):
        case["q"][..., 0] = 4.0
        case["kd"][..., 0] = -3e38   # (the product is beyond fp32's range)
    case, out, lse = _run(gpu_lib, over, tree, full, change)
    for b in range(case["batch"]):
        o = workloads.oracle_views(case, b)
        O, LSE, _ = oracle.tree_attention(o["Q"], o["K"], o["V"], o["Kd"], o["Vd"], o["parent"], case["B"], None, None)
        assert np.abs(out[b] - O).max() <= ATOL[case["dtype"]]
        np.testing.assert_allclose(lse[b], LSE, atol=2e-3 if case["dtype"] == "bf16" else 1e-5, rtol=1e-5)


@pytest.mark.parametrize("full", [False, True], ids=["attention", "refresh"])
@pytest.mark.parametrize("over", CASES, ids=["-".join(str(v) for v in o.values()) for o in CASES])
def test_infinity_in_a_v_row(gpu_lib, over, full):
    M, chan = over["M"], 5

    def forest(case):   # a second root, and the infinities in the first and in one of its children's rows (another channel)
        case["parent"][:, M // 2] = -1

    def change(case):
        forest(case)
        case["vd"][:, 0, :, chan] = float("inf")
        case["vd"][:, 1, :, chan + 1] = float("-inf")

    _, plain, lse0 = _run(gpu_lib, over, "bounded", full, forest)
    case, out, lse = _run(gpu_lib, over, "bounded", full, change)
    par = case["parent"].cpu().numpy()
    for b in range(case["batch"]):
        under = np.zeros((2, M), dtype=bool)
        for i in range(M):
            for x in range(2):
                under[x, i] = i == x or (par[b, i] >= 0 and under[x, par[b, i]])
        assert under[0].any() and not under[0].all()
        want = plain[b].copy()
        want[under[0], :, chan], want[under[1], :, chan + 1] = np.inf, -np.inf
        assert np.array_equal(out[b], want)
    assert np.array_equal(lse, lse0)
