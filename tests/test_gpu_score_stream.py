"""Scores by streams (a workgroup goes through several groups of tiles with its query rows in registers) against scoring and selection in
one launch, which takes its tiles at once: scores, lists and counts bit for bit.  One group to a workgroup and many, last groups and
last tiles that are not full, sequences that end in front of a workgroup's first group, 2 to 16 blocks of query rows, rows that do not
fill the last block, every reducer, KV heads in eights and not, both head dims; and against 64 bits."""
import pytest
import torch

import workloads
from helpers import GpuRun, say
from test_gpu_parity import SMALL

pytestmark = pytest.mark.gpu

CASES = [  # (over, reducer)
    (dict(ctx=[16 * 2100], B=16, M=60, Hq=40, Hkv=8), "mean"), (dict(ctx=[8 * 4096], B=8, M=60, Hq=32, Hkv=8), "max"), (dict(ctx=[8 * 4001] * 3, B=8, M=33, Hq=32, Hkv=8), "mean"),
    (dict(ctx=[8 * 3000, 8 * 33, 0, 8 * 1500], B=8, M=60, Hq=40, Hkv=8), "max"), (dict(ctx=[16 * 1025, 16 * 700], B=16, M=64, Hq=32, Hkv=4), "last"),
    (dict(ctx=[8 * 2000] * 9, B=8, M=31, Hq=12, Hkv=3), "mean"), (dict(ctx=[8 * 4090, 8 * 2047], B=8, M=128, Hq=16, Hkv=4), "mean"),
    (dict(ctx=[8 * 1999] * 5, B=8, M=37, Hq=32, Hkv=8, D=64), "mean"), (dict(ctx=[8 * 4000, 40], B=8, M=60, Hq=40, Hkv=8, D=64), "max"), (dict(ctx=[8 * 4000] * 4, B=8, M=26, Hq=40, Hkv=8, D=64), "mean")]


@pytest.fixture
def routes(gpu_lib):
    yield gpu_lib
    gpu_lib.specpv_debug_set_select_route(0)


@pytest.mark.parametrize("over,reduce", CASES, ids=["-".join(str(v) for v in o.values()) + "-" + r for o, r in CASES])
def test_same_bits_as_tiles_at_once(routes, over, reduce):
    sp = routes
    say("case", over, reduce)
    cfg = dict(SMALL)
    cfg.update(over, rho=[0.1] * len(over["ctx"]))
    case = workloads.make_case(cfg, seed=13, device=torch.device("cuda"))
    run = GpuRun(sp, case, reduce=reduce, last_node=case["M"] // 2)
    run.summarize()
    results = []
    for route in (0, 1):
        sp.specpv_debug_set_select_route(route)
        for x in (run.scores, run.sel_idx, run.sel_count):
            x.zero_()
        run.select()
        torch.cuda.synchronize()
        results.append([x.clone() for x in (run.scores, run.sel_idx, run.sel_count)])
    for a, b in zip(*results):
        assert torch.equal(a, b)
    G, last = case["Hq"] // case["Hkv"], case["M"] // 2
    for b, n in enumerate(case["ctx_len"].tolist()):
        nb = (n + case["B"] - 1) // case["B"]
        q = case["q"][b].double().view(case["M"], case["Hkv"], G, case["D"])
        for g in range(case["Hkv"]):
            rows = (q[last, g] if reduce == "last" else q[:, g].reshape(-1, case["D"]))
            s = torch.maximum(rows @ run.kmax[b, g, :nb].double().T, rows @ run.kmin[b, g, :nb].double().T)
            want = s.amax(0) if reduce == "max" else s.mean(0)
            # 128 products of a row, then up to 512 rows, in fp32: 640 roundings of 2^-24 against the largest sum of magnitudes
            bound = 640 * 2.0 ** -24 * float((rows.abs() @ torch.maximum(run.kmax[b, g, :nb].abs(), run.kmin[b, g, :nb].abs()).double().T).max()) if nb else 0.0
            assert nb == 0 or float((results[0][0][b, g, :nb].double() - want).abs().max()) <= bound
