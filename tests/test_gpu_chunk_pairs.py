"""Chunks taken two at a time (128 channels, bf16): even and odd numbers of them per wavefront, a last one by itself, ends inside
the first and the second chunk of a pair, in the kernels for short and for long token ranges; and rows whose maximum jumps by
more than the exponent range of fp32 from one chunk to the next."""
import pytest
import torch

import workloads
from helpers import GpuRun, say
from test_gpu_parity import SMALL, _check_attn

pytestmark = pytest.mark.gpu

LENGTHS = [1, 32, 33, 64, 65, 96, 128, 129, 161, 1000, 2048, 4100]


def _case(seed=43, **over):
    cfg = dict(SMALL)
    cfg.update(over)
    cfg["rho"] = [0.1] * len(cfg["ctx"])
    return workloads.to_device(workloads.make_case(cfg, seed=seed), "cuda")


@pytest.mark.parametrize("M,Hq,Hkv", [(16, 16, 4), (32, 16, 4), (60, 16, 4)])   # tiles of 64 and of 128 rows
def test_short_ranges(gpu_lib, M, Hq, Hkv):
    say("case %d nodes, lengths" % M, LENGTHS)
    for B in (64, 16):
        for L in LENGTHS:
            case = _case(ctx=[L], B=B, M=M, Hq=Hq, Hkv=Hkv)
            run = GpuRun(gpu_lib, case)
            run.attend(None, None)
            torch.cuda.synchronize()
            _check_attn(run, case, None, "%d nodes, %d tokens, blocks of %d" % (M, L, B))


@pytest.mark.parametrize("M", [32, 60])   # four and eight row blocks
@pytest.mark.parametrize("ctx", [[20000], [20033], [12345, 64, 33, 4097]])
def test_long_ranges(gpu_lib, M, ctx):
    say("case %d nodes" % M, ctx)
    for B in (64, 16):
        case = _case(ctx=ctx, B=B, M=M, Hq=16, Hkv=4)
        run = GpuRun(gpu_lib, case)
        run.attend(None, None)
        torch.cuda.synchronize()
        _check_attn(run, case, None, "%d nodes, %s, blocks of %d" % (M, ctx, B))


@pytest.mark.parametrize("ctx,M,Hq,D", [([700], 3, 8, 128), ([4096], 24, 8, 128), ([4096], 60, 8, 128), ([30000], 60, 8, 128),
                                        ([30000], 64, 10, 128), ([8000], 24, 8, 64)])
def test_maxima_that_jump(gpu_lib, ctx, M, Hq, D):
    """Scores rise by 160 powers of two every 48 tokens, twice, then fall back: what came before weighs nothing."""
    say("case", ctx, M, Hq, D)
    case = _case(ctx=ctx, B=64, M=M, Hq=Hq, Hkv=2, D=D)
    level = (torch.arange(case["k"].shape[2], device="cuda") // 48) % 3
    case["q"] = (0.1 * case["q"].float() + 1.0).to(torch.bfloat16)
    case["k"] = (0.1 * case["k"].float() + (112.0 / D ** 0.5) * level[None, None, :, None]).to(torch.bfloat16)
    run = GpuRun(gpu_lib, case)
    run.attend(None, None)
    torch.cuda.synchronize()
    _check_attn(run, case, None, "%s tokens, %d nodes" % (ctx, M))
