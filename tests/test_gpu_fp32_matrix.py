"""The fp32 kernels (scoring and attention on the fp32 matrix instructions) at the edges of their 16-row and 16-token
tiles, with 16 and with 32 rows per wavefront, against the oracle: 1e-5 on the outputs, lists exact."""
import numpy as np
import pytest
import torch

import workloads
from helpers import GpuRun, check_selection, oracle_select, say
from test_gpu_parity import SMALL, _check_attn

pytestmark = pytest.mark.gpu

CASES = [
    (dict(ctx=[257], B=16, M=1, Hq=2, Hkv=2), "one row; one token in the last tile"),
    (dict(ctx=[511], B=7, M=17, Hq=2, Hkv=2), "17 rows; odd block size, tiles across blocks"),
    (dict(ctx=[1030, 15, 1], B=32, M=33, Hq=8, Hkv=2, rho=[0.1] * 3), "132 rows; sequences of 15 tokens and of one"),
    (dict(ctx=[9001], B=64, M=60, Hq=16, Hkv=4, D=64), "64 channels, 240 rows, 32 per wavefront"),
    (dict(ctx=[9001], B=64, M=61, Hq=16, Hkv=4), "128 channels, 244 rows, 32 per wavefront"),
    (dict(ctx=[700], B=16, M=128, Hq=16, Hkv=1, tree="chain"), "2048 rows, G=16"),
]


@pytest.mark.parametrize("over,tag", CASES, ids=[c[1] for c in CASES])
def test_against_the_oracle(gpu_lib, over, tag):
    say("case", tag)
    cfg = dict(SMALL)
    cfg.update(dtype="f32")
    cfg.update(over)
    case = workloads.to_device(workloads.make_case(cfg, seed=31), "cuda")
    for layout, reduce, score in (("bhtd", "mean", "eq2"), ("bthd", "max", "channel_bound"), ("bhtd", "last", "eq2")):
        run = GpuRun(gpu_lib, case, layout=layout, reduce=reduce, last_node=cfg["M"] // 2, score=score)
        run.refresh(stale=0)
        torch.cuda.synchronize()
        _check_attn(run, case, None, tag + " full " + layout)
        sel = []
        for b in range(case["batch"]):
            got_idx, got_cnt = run.sel_idx.cpu().numpy()[b], run.sel_count.cpu().numpy()[b]
            o, kmax, kmin, sc, idx, cnt = oracle_select(case, b, reduce, cfg["M"] // 2, score=score)
            tol = 2e-5 * max(1.0, float(np.abs(sc).max()))
            np.testing.assert_allclose(run.scores.cpu().numpy()[b][:, :sc.shape[1]], sc, rtol=2e-5, atol=tol)
            check_selection(got_idx, got_cnt, idx, cnt, sc, case["ns"], case["nr"], case["k_blocks"], tag)
            sel.append((got_idx, got_cnt))
        run.out.zero_()
        run.attend()
        torch.cuda.synchronize()
        _check_attn(run, case, sel, tag + " partial " + layout)
