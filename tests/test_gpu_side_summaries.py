"""A full pass that recomputes summaries with some of its own workgroups: the summaries are those of the summary kernel to the
bit, nothing in front of the stale range is touched, and the pass gives what it gives with summaries that are up to date."""
import pytest
import torch

import workloads
from helpers import GpuRun, say
from test_gpu_parity import SMALL

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ctx,B,M,Hq,Hkv", [([65536], 64, 60, 32, 8),              # eight row blocks
                                            ([50001], 64, 60, 16, 4),              # a ragged last block
                                            ([40000], 128, 75, 16, 4),             # ten row blocks, blocks of 128
                                            ([32768, 777, 20000, 1], 64, 60, 32, 8),   # shares over a batch
                                            ([60000], 64, 64, 64, 4)])             # thirty-two row blocks: four workgroups
@pytest.mark.parametrize("part", [0.0, 0.4, 0.97])
def test_against_the_summary_kernel(gpu_lib, ctx, B, M, Hq, Hkv, part):
    say("case", ctx, B, M, Hq, Hkv, part)
    cfg = dict(SMALL)
    cfg.update(ctx=ctx, B=B, M=M, Hq=Hq, Hkv=Hkv, k=20, rho=[0.1] * len(ctx))
    case = workloads.make_case(cfg, seed=59, device=torch.device("cuda"))
    run = GpuRun(gpu_lib, case)
    run.summarize()
    run.refresh(-1)
    torch.cuda.synchronize()
    want = [x.clone() for x in (run.kmax, run.kmin, run.out, run.lse, run.sel_idx, run.sel_count)]
    begin = int(part * case["max_blocks"])
    for x in (run.kmax, run.kmin):
        x[:, :, begin:] = -7.0
    run.out.zero_()
    run.refresh(begin)
    torch.cuda.synchronize()
    for b, L in enumerate(ctx):
        nb = (L + B - 1) // B
        assert torch.equal(run.kmax[b, :, :nb], want[0][b, :, :nb]) and torch.equal(run.kmin[b, :, :nb], want[1][b, :, :nb]), "summaries differ"
        assert (run.kmax[b, :, max(nb, begin):] == -7.0).all(), "written behind the last block"
    # another number of splits: other sums in fp32 and roundings of the partials to fp16 (2^-11), far below the output's bf16,
    # so results differ by a unit in their last place at most, which is up to 2^-7 of a value
    assert (run.out.float() - want[2].float()).abs().max() <= 2.0 ** -7 * want[2].float().abs().max()
    # (a row's sum runs over weights rounded to bf16, 2^-8, against a reference that follows the splits; that no token is lost
    # or taken twice, which is less than that, is the next test's)
    assert (run.lse - want[3]).abs().max() <= 2.0 ** -8
    assert torch.equal(run.sel_idx, want[4]) and torch.equal(run.sel_count, want[5])


@pytest.mark.parametrize("ctx,B,M,Hq,Hkv", [([65536], 64, 60, 32, 8),                  # eight row blocks
                                            ([50001], 128, 64, 20, 4),                 # ten, a ragged end
                                            ([32768, 777, 20000, 1], 64, 60, 32, 8),   # shares over a batch
                                            ([30000, 29999, 4096], 64, 64, 40, 8),     # ... of ten
                                            ([60000], 64, 64, 64, 4)])                 # thirty-two: four workgroups
def test_every_token_once(gpu_lib, ctx, B, M, Hq, Hkv):
    """Queries of zeros weigh every token alike: lse counts the tokens, and with rows of V that name their chunk (chunk c is
    channel c % 128) so does every output channel the tokens of its chunks, wherever the pass is cut."""
    say("case", ctx, B, M, Hq, Hkv)
    cfg = dict(SMALL)
    cfg.update(ctx=ctx, B=B, M=M, Hq=Hq, Hkv=Hkv, k=20, rho=[0.1] * len(ctx))
    case = workloads.make_case(cfg, seed=67, device=torch.device("cuda"))
    case["q"].zero_()
    case["vd"].zero_()
    chunk = torch.arange(case["v"].shape[2], device="cuda") // 32 % 128
    case["v"].copy_(torch.nn.functional.one_hot(chunk, 128).to(case["v"].dtype))
    run = GpuRun(gpu_lib, case)
    # weights, sums and counts are whole numbers, exact in fp32: what is left is log2 (a unit of 2^-19 below 2^17 tokens) and
    # the product with ln 2 (half a unit of 2^-20); of an output its bf16 (half of a unit of 2^-7), the partials' fp16 (half
    # of 2^-10) and a few roundings of fp32.  One chunk less, or more, is far beyond both.
    lse_bound, out_bound = 2.0 ** -18, 2.0 ** -8 + 2.0 ** -11 + 2.0 ** -20
    depth = torch.zeros((len(ctx), M), dtype=torch.float64)   # nodes of a root path
    for b, par in enumerate(case["parent"].tolist()):
        for j, p in enumerate(par):
            depth[b, j] = 1 + (depth[b, p] if p >= 0 else 0)
    tokens = torch.tensor(ctx, dtype=torch.float64)[:, None] + depth
    assert (torch.log(tokens) - torch.log(tokens - 1)).min() > 2 * lse_bound   # a single token shows
    count = torch.stack([torch.bincount(chunk[:L].cpu(), minlength=128) for L in ctx]).double()
    assert 32 / count.max() > 4 * out_bound
    want = count[:, None, None, :] / tokens[:, :, None, None]
    for stale in (-1, 0, int(0.4 * case["max_blocks"]), case["max_blocks"] - 1):
        run.out.fill_(7.0)
        run.lse.zero_()
        run.refresh(stale)
        torch.cuda.synchronize()
        lse, out = run.lse.cpu().double(), run.out.cpu().double()
        say("   stale from", stale, "lse off by %.2g, outputs by %.2g of themselves" % (
            (lse - torch.log(tokens)[:, :, None]).abs().max(), ((out - want).abs() / want.clamp_min(1e-9)).max()))
        assert ((lse - torch.log(tokens)[:, :, None]).abs() <= lse_bound).all(), stale
        assert ((out - want).abs() <= out_bound * want).all(), stale


@pytest.mark.parametrize("over", [dict(ctx=[65536]), dict(ctx=[30000, 777, 20000, 1]), dict(ctx=[9001], B=32, M=37, D=64),
                                  dict(ctx=[2048], B=16, M=16, Hq=4, Hkv=1, D=64, dtype="f32")], ids=["long", "batch", "64 channels", "fp32"])
def test_a_refresh_and_the_calls_it_stands_for(gpu_lib, over):
    """Without stale summaries every result has the bits of the separate calls; with them, everything but out and lse."""
    say("case", over)
    cfg = dict(SMALL, B=64, M=60, Hq=32, Hkv=8, k=20)
    cfg.update(over, rho=[0.1] * len(over["ctx"]))
    case = workloads.make_case(cfg, seed=61, device=torch.device("cuda"))
    run = GpuRun(gpu_lib, case)
    run.summarize(); run.attend(None, None); run.select()
    torch.cuda.synchronize()
    results = lambda: [x.clone() for x in (run.kmax, run.kmin, run.scores, run.sel_idx, run.sel_count, run.out, run.lse)]
    want = results()
    for stale in (-1, 0, case["max_blocks"] // 2):
        for x in (run.out, run.lse, run.scores, run.sel_idx, run.sel_count):
            x.zero_()
        run.refresh(stale)
        torch.cuda.synchronize()
        got = results()
        for a, b in zip(got if stale < 0 else got[:5], want):
            assert torch.equal(a, b), (stale, a.shape)
