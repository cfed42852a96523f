"""Block summaries against torch's amax / amin, bit for bit, where the kernel takes another course: several small blocks to a
wavefront and one, every count of passes, ragged last blocks, ranges of blocks that begin and end anywhere, both layouts and types;
and small blocks that a full pass summarises on the side."""
import pytest
import torch

import workloads
from helpers import GpuRun, say
from test_gpu_parity import SMALL

pytestmark = pytest.mark.gpu


def _check(sp, dt, D, Hkv, lens, B, layout, lo, hi, extra=0):
    batch, nb = len(lens), max(1, (max(lens) + B - 1) // B) + extra
    gen = torch.Generator(device="cuda").manual_seed(7)
    k = torch.randn((batch, Hkv, nb * B, D), generator=gen, device="cuda", dtype=dt)
    for b, L in enumerate(lens):
        k[b, :, L:] = float("nan")   # rows behind a sequence's end
    stored = k if layout == "bhtd" else k.permute(0, 2, 1, 3).contiguous()
    kv = sp.KV(stored, stored, torch.tensor(lens, dtype=torch.int32, device="cuda"), B, nb, layout)
    mx = torch.full((batch, Hkv, nb, D), -7.0, dtype=dt, device="cuda")
    mn = torch.full_like(mx, -7.0)
    sp.specpv_block_summarize(kv, lo, hi, mx, mn)
    torch.cuda.synchronize()
    for b, L in enumerate(lens):
        rows = k[b].view(Hkv, nb, B, D)
        valid = (torch.arange(nb * B, device="cuda") < L).view(1, nb, B, 1)
        want_x = torch.where(valid, rows, torch.full_like(rows, float("-inf"))).amax(2)
        want_n = torch.where(valid, rows, torch.full_like(rows, float("inf"))).amin(2)
        i = torch.arange(nb, device="cuda")
        mine = (i >= lo) & (i < ((L + B - 1) // B if hi < 0 else min(hi, (L + B - 1) // B)))
        assert torch.equal(mx[b][:, mine], want_x[:, mine]) and torch.equal(mn[b][:, mine], want_n[:, mine])
        assert (mx[b][:, ~mine] == -7.0).all() and (mn[b][:, ~mine] == -7.0).all()


@pytest.mark.parametrize("dt,D", [(torch.bfloat16, 128), (torch.bfloat16, 64), (torch.float32, 128), (torch.float32, 64)])
@pytest.mark.parametrize("B", [1, 4, 7, 8, 16, 24, 32, 33, 48, 64, 100, 128, 300])
def test_every_count_of_passes(gpu_lib, dt, D, B):
    say("case", dt, D, B)
    for layout in ("bhtd", "bthd"):
        _check(gpu_lib, dt, D, 2, [5 * B + 1, 0, 3 * B - 1 if B > 1 else 2, 1], B, layout, 0, -1)
        _check(gpu_lib, dt, D, 3, [9 * B], B, layout, 2, 7, extra=3)


@pytest.mark.parametrize("dt,D,B", [(torch.bfloat16, 128, 16), (torch.bfloat16, 64, 32), (torch.bfloat16, 64, 16), (torch.float32, 64, 16), (torch.float32, 128, 8)])
@pytest.mark.parametrize("lo,hi", [(0, -1), (3, -1), (5, 1022)])
def test_several_blocks_to_a_wavefront(gpu_lib, dt, D, B, lo, hi):
    say("case", dt, D, B, lo, hi)   # 8192 blocks and more
    _check(gpu_lib, dt, D, 8, [1030 * B - 5, 1027 * B + 1], B, "bhtd", lo, hi)


@pytest.mark.parametrize("ctx,B,M,Hq,Hkv", [([30000], 16, 60, 32, 8), ([29999], 32, 60, 32, 8), ([20001, 77, 9000], 16, 60, 32, 8), ([24007], 32, 75, 16, 4)])
@pytest.mark.parametrize("part", [0.0, 0.5, 0.97])
def test_small_blocks_on_the_side(gpu_lib, ctx, B, M, Hq, Hkv, part):
    say("case", ctx, B, M, Hq, Hkv, part)
    cfg = dict(SMALL)
    cfg.update(ctx=ctx, B=B, M=M, Hq=Hq, Hkv=Hkv, k=20, rho=[0.1] * len(ctx))
    run = GpuRun(gpu_lib, workloads.make_case(cfg, seed=59, device=torch.device("cuda")))
    run.summarize()
    run.refresh(-1)
    torch.cuda.synchronize()
    want = [x.clone() for x in (run.kmax, run.kmin, run.sel_idx, run.sel_count, run.out, run.lse)]
    begin = int(part * run.case["max_blocks"])
    for x in (run.kmax, run.kmin):
        x[:, :, begin:] = -7.0
    run.refresh(begin)
    torch.cuda.synchronize()
    for b, L in enumerate(ctx):
        nb = (L + B - 1) // B
        assert torch.equal(run.kmax[b, :, :nb], want[0][b, :, :nb]) and torch.equal(run.kmin[b, :, :nb], want[1][b, :, :nb])
        assert (run.kmax[b, :, max(nb, begin):] == -7.0).all()
    assert torch.equal(run.sel_idx, want[2]) and torch.equal(run.sel_count, want[3])
    # another number of splits: a unit in the last place of a bf16 value at most (test_gpu_side_summaries.py)
    assert ((run.out.float() - want[4].float()).abs() <= 2.0 ** -7 * want[4].float().abs() + 1e-3).all()
    assert (run.lse - want[5]).abs().max() <= 2.0 ** -8


@pytest.mark.parametrize("dt,D,B", [(torch.bfloat16, 128, 16), (torch.bfloat16, 128, 32), (torch.bfloat16, 64, 16), (torch.float32, 64, 16)])
@pytest.mark.parametrize("short", [1, 2, 3])
def test_sequences_longer_than_the_cache_has_blocks(gpu_lib, dt, D, B, short):
    """The summaries of the blocks that are there, and nothing behind them."""
    say("case", dt, D, B, short)
    Hkv, all_blocks = 8, 1032
    nb = all_blocks - short
    gen = torch.Generator(device="cuda").manual_seed(7)
    k = torch.randn((1, Hkv, all_blocks * B, D), generator=gen, device="cuda", dtype=dt)
    k[:, :, nb * B:] = float("nan")
    kv = gpu_lib.KV(k, k, torch.tensor([all_blocks * B], dtype=torch.int32, device="cuda"), B, nb)
    mx = torch.full((1, Hkv, all_blocks, D), -7.0, dtype=dt, device="cuda")   # (the kernel's arrays are its first nb * Hkv rows)
    mn = torch.full_like(mx, -7.0)
    gpu_lib.specpv_block_summarize(kv, 0, -1, mx.view(-1)[:Hkv * nb * D].view(1, Hkv, nb, D), mn.view(-1)[:Hkv * nb * D].view(1, Hkv, nb, D))
    torch.cuda.synchronize()
    rows = k[:, :, :nb * B].view(1, Hkv, nb, B, D)
    assert torch.equal(mx.view(-1)[:Hkv * nb * D].view(1, Hkv, nb, D), rows.amax(3)) and torch.equal(mn.view(-1)[:Hkv * nb * D].view(1, Hkv, nb, D), rows.amin(3))
    assert (mx.view(-1)[Hkv * nb * D:] == -7.0).all() and (mn.view(-1)[Hkv * nb * D:] == -7.0).all()


@pytest.mark.parametrize("B,short", [(16, 1), (16, 2), (16, 3), (32, 1)])
def test_side_summaries_of_sequences_longer_than_the_cache(gpu_lib, B, short):
    say("case", B, short)
    cfg = dict(SMALL)
    cfg.update(ctx=[30000], B=B, M=60, Hq=32, Hkv=8, k=20, rho=[0.1])
    case = workloads.make_case(cfg, seed=59, device=torch.device("cuda"))
    nb = case["max_blocks"] // 4 * 4 - short
    case = dict(case, max_blocks=nb)
    run = GpuRun(gpu_lib, case)
    run.kv = gpu_lib.KV(run.k, run.v, case["ctx_len"], B, nb)
    run.refresh(0)
    torch.cuda.synchronize()
    rows = case["k"][:, :, :nb * B].view(1, 8, nb, B, -1)
    assert torch.equal(run.kmax, rows.amax(3)) and torch.equal(run.kmin, rows.amin(3))
