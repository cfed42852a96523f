"""Block sizes that are and are not a multiple of 16 and of 32, over lists and over all blocks: the rows of a 32-token chunk are
one run, two, or any, and the kernels for short and for long token ranges each have a path for that."""
import numpy as np
import pytest
import torch

import workloads
from helpers import GpuRun, say
from test_gpu_parity import SMALL, _check_attn

pytestmark = pytest.mark.gpu

SHAPES = [(dict(ctx=[1500], M=60, Hq=16, Hkv=4), "two token groups"),
          (dict(ctx=[1500], M=16, Hq=16, Hkv=4), "four token groups"),
          (dict(ctx=[1500], M=3, Hq=8, Hkv=4), "eight token groups"),
          (dict(ctx=[14000], M=60, Hq=16, Hkv=4), "eight row blocks"),
          (dict(ctx=[9001, 4000, 77], M=60, Hq=20, Hkv=4), "ten row blocks, three sequences"),
          (dict(ctx=[5003, 2000], M=37, Hq=16, Hkv=4, D=64), "64 channels")]


@pytest.mark.parametrize("B", [8, 16, 24, 48, 80])
@pytest.mark.parametrize("over,tag", SHAPES, ids=[c[1] for c in SHAPES])
def test_against_the_oracle(gpu_lib, over, tag, B):
    say("case", tag, "blocks of", B)
    cfg = dict(SMALL)
    cfg.update(over)
    cfg.update(B=B, rho=[0.1] * len(over["ctx"]))
    case = workloads.to_device(workloads.make_case(cfg, seed=47), "cuda")
    run = GpuRun(gpu_lib, case)
    run.attend(None, None)
    torch.cuda.synchronize()
    _check_attn(run, case, None, tag + " all")
    # a list in any order, with -1 in front and in the middle, of whole and of ragged blocks, longer than the registers hold
    rs, nbs = np.random.RandomState(B), [(L + B - 1) // B for L in over["ctx"]]
    n = min(700, max(nbs) + 2)
    idx = np.full((case["batch"], case["Hkv"], n), -1, dtype=np.int32)
    cnt = np.zeros((case["batch"], case["Hkv"]), dtype=np.int32)
    for b, nb in enumerate(nbs):
        for g in range(case["Hkv"]):
            take = min(nb, n - 2)
            row = np.concatenate([[-1], rs.permutation(nb)[:take], [-1]])
            row[take // 3] = -1
            idx[b, g, :take + 2], cnt[b, g] = row, take + 2
    sel = torch.from_numpy(idx).cuda(), torch.from_numpy(cnt).cuda()
    run.out.zero_()
    run.attend(*sel)
    torch.cuda.synchronize()

    def valid(b):   # the oracle's list: the entries that count
        out = np.full_like(idx[b], -1)
        c = np.zeros_like(cnt[b])
        for g in range(case["Hkv"]):
            v = [i for i in idx[b, g, :cnt[b, g]] if i >= 0]
            out[g, :len(v)], c[g] = v, len(v)
        return out, c
    _check_attn(run, case, [valid(b) for b in range(case["batch"])], tag + " listed")


@pytest.mark.parametrize("B", [16, 24, 64])
def test_lengths_beyond_the_last_block(gpu_lib, B):
    """A cache whose block count stops short of the sequence: what lies behind it is not attended."""
    say("case blocks of", B)
    cfg = dict(SMALL)
    for ctx, M in ((1501, 60), (9001, 60), (700, 3)):
        cfg.update(ctx=[ctx], B=B, M=M, Hq=16, Hkv=4)
        case = workloads.to_device(workloads.make_case(cfg, seed=53), "cuda")
        keep = case["max_blocks"] - 3
        run = GpuRun(gpu_lib, case)
        run.kv = gpu_lib.KV(run.k, run.v, case["ctx_len"], B, keep)
        run.attend(None, None)
        torch.cuda.synchronize()
        idx = np.tile(np.arange(keep, dtype=np.int32), (case["Hkv"], 1))
        _check_attn(run, case, [(idx, np.full((case["Hkv"],), keep, dtype=np.int32))], "%d tokens" % ctx)
