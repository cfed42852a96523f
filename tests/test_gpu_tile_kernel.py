"""The kernel for short token ranges and the combine kernel behind it: query-row counts around the tile sizes (32, 64, 128
packed rows), numbers of (sequence, KV head) pairs that are and are not a multiple of the XCDs, chunk counts from one
up, one and many splits, against the oracle."""
import pytest
import torch

import workloads
from helpers import GpuRun, say
from test_gpu_parity import SMALL, _check_attn

pytestmark = pytest.mark.gpu

CASES = [
    (dict(ctx=[2048], B=64, M=8, Hq=32, Hkv=8), "32 rows: eight token groups"),
    (dict(ctx=[2048], B=64, M=33, Hq=8, Hkv=8), "33 rows: one over a tile of 32"),
    (dict(ctx=[4096], B=32, M=16, Hq=32, Hkv=8), "64 rows"),
    (dict(ctx=[4096, 4096], B=32, M=65, Hq=16, Hkv=16, rho=[0.1] * 2), "65 rows, 32 pairs"),
    (dict(ctx=[8000], B=64, M=32, Hq=32, Hkv=8), "128 rows: two token groups, ragged end"),
    (dict(ctx=[8000], B=16, M=43, Hq=9, Hkv=3, tree="uniform"), "129 rows, three pairs, chunks across blocks"),
    (dict(ctx=[33], B=32, M=1, Hq=4, Hkv=1), "two chunks, one token in the second"),
    (dict(ctx=[6000] * 9, B=64, M=5, Hq=4, Hkv=1, rho=[0.1] * 9), "nine pairs"),
    (dict(ctx=[12000], B=64, M=60, Hq=10, Hkv=2, k=180), "a list of 180 blocks, two pairs, many splits"),
    (dict(ctx=[3000], B=64, M=128, Hq=32, Hkv=2, tree="chain"), "2048 rows"),
]


@pytest.mark.parametrize("over,tag", CASES, ids=[c[1] for c in CASES])
def test_against_the_oracle(gpu_lib, over, tag):
    say("case", tag)
    cfg = dict(SMALL)
    cfg.update(k=40)
    cfg.update(over)
    case = workloads.to_device(workloads.make_case(cfg, seed=37), "cuda")
    for layout in ("bhtd", "bthd"):
        run = GpuRun(gpu_lib, case, layout=layout)
        run.summarize(); run.select(); run.attend()
        torch.cuda.synchronize()
        sel = [(run.sel_idx.cpu().numpy()[b], run.sel_count.cpu().numpy()[b]) for b in range(case["batch"])]
        _check_attn(run, case, sel, tag + " kept " + layout)
        run.out.zero_()
        run.attend(None, None)
        torch.cuda.synchronize()
        _check_attn(run, case, None, tag + " all " + layout)


@pytest.mark.parametrize("M,Hq,Hkv", [(4, 32, 8), (20, 16, 4), (60, 32, 8)])
def test_pending_tokens(gpu_lib, M, Hq, Hkv):
    """Each tile size with pending tokens in front of the tree, one full and one ragged chunk of them."""
    import test_gpu_parity
    test_gpu_parity.test_pending_tokens_go_with_the_cache_tokens(gpu_lib, dict(ctx=[4000], B=64, M=M, Hq=Hq, Hkv=Hkv), 37, "M=%d, %d heads on %d" % (M, Hq, Hkv))
