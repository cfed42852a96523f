"""The merge of the partials with the rows of a KV head packed into fours (group sizes that are no multiple of four): one and two
wavefronts per four rows, rows that do not fill the last four, one and two registers of parents, root paths beyond the first
eight nodes and beyond 64, every count of partials that has a kernel of its own, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from helpers import ATOL, GpuRun, say, with_pending
from test_gpu_parity import SMALL

pytestmark = pytest.mark.gpu

CASES = [  # (over, partially verified tokens); fours of rows are sequences * KV heads * ceil(nodes * G / 4), the line at 2048 of them
    (dict(ctx=[300], M=1, Hq=4, Hkv=4), 0), (dict(ctx=[40], M=7, Hq=10, Hkv=2), 0), (dict(ctx=[500], M=33, Hq=6, Hkv=2, tree="chain"), 0),
    (dict(ctx=[900], M=65, Hq=40, Hkv=8, tree="chain"), 0), (dict(ctx=[900], M=127, Hq=6, Hkv=2, tree="chain"), 0), (dict(ctx=[300], M=60, Hq=40, Hkv=8), 13),
    (dict(ctx=[4000], M=60, Hq=40, Hkv=8), 0), (dict(ctx=[16000], M=17, Hq=5, Hkv=1, tree="uniform"), 0), (dict(ctx=[9000, 33, 5000], M=60, Hq=40, Hkv=8), 7),
    (dict(ctx=[700] * 11, M=38, Hq=40, Hkv=8), 0), (dict(ctx=[700] * 11, M=37, Hq=40, Hkv=8), 0), (dict(ctx=[700] * 8, M=96, Hq=14, Hkv=2, tree="chain"), 0),
    (dict(ctx=[2500, 2600], M=37, Hq=24, Hkv=8, D=64), 0), (dict(ctx=[300], M=70, Hq=7, Hkv=1, D=64, tree="star"), 5),
    (dict(ctx=[12000], M=60, Hq=20, Hkv=4, D=64), 0)]


@pytest.mark.parametrize("over,n_key", CASES, ids=["-".join(str(v) for v in o.values()) + "-%d" % n for o, n in CASES])
def test_packed_rows_against_the_oracle(gpu_lib, over, n_key):
    say("case", over, n_key)
    cfg = dict(SMALL, B=32, name="packed")
    cfg.update(over, rho=[0.1] * len(over["ctx"]))
    case = workloads.make_case(cfg, seed=81)
    if n_key:
        case = with_pending(case, n_key, seed=82)
    case = workloads.to_device(case, "cuda")
    run = GpuRun(gpu_lib, case)
    run.attend(None, None)
    torch.cuda.synchronize()
    worst = 0.0
    for b in range(case["batch"]):
        o = workloads.oracle_views(case, b)
        O, LSE, _ = oracle.tree_attention(o["Q"], o["K"], o["V"], o["Kd"], o["Vd"], o["parent"], case["B"], None, None, n_key_only=n_key)
        worst = max(worst, np.abs(run.out[b].float().cpu().numpy() - O).max())
        np.testing.assert_allclose(run.lse[b].cpu().numpy(), LSE, atol=2e-3, rtol=1e-5)   # (bf16's bar, see test_gpu_combine_waves)
    say("   max-abs err %.3g" % worst)
    assert worst <= ATOL["bf16"]
