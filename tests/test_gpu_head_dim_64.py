"""The matrix-core kernels at 64 channels (scoring and attention), and the query rows of a KV head packed over its heads:
shapes at the edges of the 32-row blocks, of the 32-token chunks and of the workgroup sizes, against the oracle."""
import numpy as np
import pytest
import torch

import workloads
from helpers import GpuRun, check_selection, oracle_select, say
from test_gpu_parity import SMALL, _check_attn

pytestmark = pytest.mark.gpu

CASES = [
    (dict(ctx=[40000], B=64, M=60, Hq=8, Hkv=2), "G=4, 240 rows: eight wavefronts, the last with a half-filled block"),
    (dict(ctx=[36001], B=16, M=37, Hq=8, Hkv=2, tree="uniform"), "148 rows on six wavefronts, one idle; block 16; one token in the last chunk"),
    (dict(ctx=[9000, 31, 1], B=32, M=1, Hq=6, Hkv=2, rho=[0.1] * 3), "three rows; sequences of 31 tokens and of one"),
    (dict(ctx=[34000], B=64, M=100, Hq=10, Hkv=2, tree="uniform"), "500 rows: two workgroups of eight"),
    (dict(ctx=[2000, 900], B=7, M=33, Hq=8, Hkv=8, rho=[0.1] * 2), "G=1, 33 rows: one row in the second block; odd block size"),
    (dict(ctx=[1000], B=16, M=128, Hq=16, Hkv=1, tree="chain"), "2048 rows, G=16"),
    (dict(ctx=[36000], B=64, M=78, Hq=8, Hkv=2, D=128), "128 channels, 312 rows: ten wavefronts where heads of their own would need twelve"),
    (dict(ctx=[36000], B=32, M=3, Hq=16, Hkv=2, D=128), "128 channels, 24 rows in one block"),
]


@pytest.mark.parametrize("over,tag", CASES, ids=[c[1] for c in CASES])
def test_against_the_oracle(gpu_lib, over, tag):
    say("case", tag)
    cfg = dict(SMALL)
    cfg.update(D=64)
    cfg.update(over)
    case = workloads.to_device(workloads.make_case(cfg, seed=29), "cuda")
    for layout in ("bhtd", "bthd"):
        run = GpuRun(gpu_lib, case, layout=layout)
        run.refresh(stale=0)
        torch.cuda.synchronize()
        _check_attn(run, case, None, tag + " full " + layout)
        sel = []
        for b in range(case["batch"]):
            got_idx, got_cnt = run.sel_idx.cpu().numpy()[b], run.sel_count.cpu().numpy()[b]
            o, kmax, kmin, sc, idx, cnt = oracle_select(case, b)
            tol = 2e-5 * max(1.0, float(np.abs(sc).max()))
            np.testing.assert_allclose(run.scores.cpu().numpy()[b][:, :sc.shape[1]], sc, rtol=2e-5, atol=tol)
            check_selection(got_idx, got_cnt, idx, cnt, sc, case["ns"], case["nr"], case["k_blocks"], tag)
            sel.append((got_idx, got_cnt))
        run.out.zero_()
        run.attend()
        torch.cuda.synchronize()
        _check_attn(run, case, sel, tag + " partial " + layout)


def test_pending_tokens(gpu_lib):
    """64 channels: pending tokens in front of the tree as extra chunks, one full and one ragged."""
    import test_gpu_parity
    test_gpu_parity.test_pending_tokens_go_with_the_cache_tokens(gpu_lib, dict(ctx=[5000, 700], rho=[0.1] * 2, D=64, B=32, M=50), 39, "64 channels")
