"""The kernel for long token ranges: row block counts of every workgroup shape (those shared by two wavefronts among them), with
even, odd and single chunks per workgroup, one sequence and a ragged batch, against the oracle."""
import pytest
import torch

import workloads
from helpers import GpuRun, say
from test_gpu_parity import SMALL, _check_attn

pytestmark = pytest.mark.gpu

CASES = [
    (dict(ctx=[40000], B=64, M=16, Hq=8, Hkv=4), "128 channels, one row block"),
    (dict(ctx=[33000, 999], B=64, M=33, Hq=4, Hkv=4), "128 channels, two row blocks, one row in the second"),
    (dict(ctx=[20000, 64], B=32, M=35, Hq=16, Hkv=4), "128 channels, five row blocks"),
    (dict(ctx=[20033], B=16, M=47, Hq=16, Hkv=4), "128 channels, six row blocks, chunks across blocks"),
    (dict(ctx=[20000, 7001, 33], B=64, M=52, Hq=20, Hkv=4), "128 channels, nine row blocks"),
    (dict(ctx=[15000], B=64, M=64, Hq=20, Hkv=4), "128 channels, ten row blocks"),
    (dict(ctx=[9000, 3001], B=32, M=88, Hq=16, Hkv=4, tree="uniform"), "128 channels, eleven row blocks"),
    (dict(ctx=[5000, 321], B=32, M=33, Hq=4, Hkv=4, D=64), "64 channels, two row blocks"),
    (dict(ctx=[4001], B=16, M=37, Hq=16, Hkv=4, D=64), "64 channels, five row blocks"),
    (dict(ctx=[2999, 3000], B=64, M=64, Hq=20, Hkv=4, D=64), "64 channels, ten row blocks"),
]


@pytest.mark.parametrize("over,tag", CASES, ids=[c[1] for c in CASES])
def test_full_pass_against_the_oracle(gpu_lib, over, tag):
    say("case", tag)
    cfg = dict(SMALL)
    cfg.update(over)
    cfg["rho"] = [0.1] * len(cfg["ctx"])
    case = workloads.to_device(workloads.make_case(cfg, seed=41), "cuda")
    for layout in ("bhtd", "bthd"):
        run = GpuRun(gpu_lib, case, layout=layout)
        run.attend(None, None)
        torch.cuda.synchronize()
        _check_attn(run, case, None, tag + " " + layout)
