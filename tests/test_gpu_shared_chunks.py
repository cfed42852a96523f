"""Full passes over batches, where the workgroups take equal shares of the chunks of all sequences: empty and one-token
sequences, one that holds nearly everything, more sequences than shares, against the oracle."""
import pytest
import torch

import workloads
from helpers import GpuRun, say
from test_gpu_parity import SMALL, _check_attn

pytestmark = pytest.mark.gpu

CASES = [
    (dict(ctx=[0, 40000, 1, 70, 0, 12000], G=4), "empty sequences first and between"),
    (dict(ctx=[60000, 0, 1], G=5), "one sequence holds all"),
    (dict(ctx=[3000] * 9 + [0], G=4, M=64), "ten sequences, one row block per wavefront"),
    (dict(ctx=[9000, 14000, 31, 32, 33], G=4, B=16), "chunks across blocks"),
    (dict(ctx=[20000, 5000, 12000], G=4, D=64), "64 channels"),
    (dict(ctx=[700 * ((7 * i) % 11) for i in range(64)], G=2, M=64), "64 sequences"),
    (dict(ctx=[700 * ((7 * i) % 11) for i in range(65)], G=2, M=64), "65: back to splits"),
    (dict(ctx=[400 * ((7 * i) % 11) for i in range(16)], G=4, Hkv=8), "eight heads: few shares to a pair"),
    (dict(ctx=[4000] + [40] * 14 + [0], G=4, Hkv=8), "eight heads, one long"),
    (dict(ctx=[400 * ((7 * i) % 11) for i in range(16)], G=4, Hkv=8, D=64, M=16), "eight heads, 64 channels"),
]


@pytest.mark.parametrize("over,tag", CASES, ids=[c[1] for c in CASES])
def test_against_the_oracle(gpu_lib, over, tag):
    say("case", tag)
    cfg = dict(SMALL)
    over = dict(over)
    G = over.pop("G")
    cfg.update(B=64, M=60, Hkv=2)
    cfg.update(over)
    cfg["Hq"] = G * cfg["Hkv"]
    cfg["rho"] = [0.1] * len(cfg["ctx"])
    case = workloads.to_device(workloads.make_case(cfg, seed=41), "cuda")
    for layout in ("bhtd", "bthd"):
        run = GpuRun(gpu_lib, case, layout=layout)
        for _ in range(2):   # the second call finds what the first left in the workspace
            run.out.zero_()
            run.attend(None, None)
            torch.cuda.synchronize()
            _check_attn(run, case, None, tag + " " + layout)
