"""Scores by streams (a workgroup goes through several groups of tiles with its query rows in registers) against scoring and selection in
one launch, which takes its tiles at once (four blocks of query rows and more): scores, lists and counts bit for bit.  One group to a
workgroup and many, last groups and last tiles that are not full, workgroups dealt to sequences of all lengths, empty ones among them, up
to the 64 that a wavefront deals to, sequences longer than the blocks that the cache has, 2 to 16 blocks of query rows, rows that do not
fill the last block, every reducer, KV heads in eights and not, both head dims; and against 64 bits.  That a case goes by streams is
worked out here once more (256 CUs)."""
import pytest
import torch

import workloads
from helpers import GpuRun, say
from test_gpu_parity import SMALL

pytestmark = pytest.mark.gpu

CASES = [  # (over, reducer); `last` at node M / 2
    (dict(ctx=[16 * 3100], B=16, M=60, Hq=40, Hkv=8), "mean"), (dict(ctx=[8 * 4096], B=8, M=60, Hq=32, Hkv=8), "max"), (dict(ctx=[8 * 4001] * 3, B=8, M=33, Hq=32, Hkv=8), "mean"),
    (dict(ctx=[8 * 3000, 8 * 33, 0, 8 * 1500], B=8, M=60, Hq=40, Hkv=8), "max"), (dict(ctx=[8 * 4090, 8 * 700], B=8, M=39, Hq=40, Hkv=8), "last"),   # (rows 95 .. 99, in two blocks)
    (dict(ctx=[8 * 2000] * 9, B=8, M=31, Hq=24, Hkv=3), "mean"), (dict(ctx=[8 * 4090, 8 * 2047], B=8, M=128, Hq=16, Hkv=4), "mean"),
    (dict(ctx=[8 * 2299] * 5, B=8, M=37, Hq=32, Hkv=8, D=64), "mean"), (dict(ctx=[8 * 4096, 40], B=8, M=60, Hq=32, Hkv=8, D=64), "max"), (dict(ctx=[8 * 4000] * 4, B=8, M=26, Hq=40, Hkv=8, D=64), "mean"),
    # 2, 3 and 16 blocks of query rows
    (dict(ctx=[8 * 4096] * 2, B=8, M=16, Hq=32, Hkv=8), "mean"), (dict(ctx=[8 * 4000, 8 * 77, 8 * 3999], B=8, M=23, Hq=32, Hkv=8), "max"), (dict(ctx=[8 * 4000], B=8, M=64, Hq=64, Hkv=8), "mean"),
    (dict(ctx=[8 * 4096, 8 * 50], B=8, M=9, Hq=64, Hkv=8, D=64), "max"),
    # one long sequence first, last and among others, and as many as there are lanes
    (dict(ctx=[8 * 2048] + [8 * 128] * 15, B=8, M=60, Hq=40, Hkv=8), "mean"), (dict(ctx=[8] * 15 + [8 * 2048], B=8, M=60, Hq=32, Hkv=8), "max"), (dict(ctx=[0, 8 * 900, 0, 0, 8 * 4096, 1, 8 * 64], B=8, M=60, Hq=32, Hkv=8), "mean"),
    (dict(ctx=[8 * (17 * i % 301) for i in range(63)] + [8 * 600], B=8, M=60, Hq=16, Hkv=4), "mean"), (dict(ctx=[8 * 1400 * (i + 1) // 16 for i in range(16)], B=8, M=37, Hq=16, Hkv=2), "max")]
CAP = [(dict(ctx=[8 * 4096, 8 * 900, 8 * 3500], B=8, M=60, Hq=32, Hkv=8), 3300)]   # blocks that the cache has


def by_streams(c, blocks):
    """score_stream_plan (csrc/score_mfma.hip)."""
    D, batch, Hkv, rows, cus = c["D"], len(c["ctx"]), c["Hkv"], c["M"] * c["Hq"] // c["Hkv"], 256
    if c.get("reduce") == "last":
        G, node = c["Hq"] // Hkv, c["M"] // 2
        rows = (node + 1) * G - node * G // 32 * 32
    r32 = (rows + 31) // 32
    if not 2 <= r32 <= 16:
        return False
    T = (r32 * 4096 + 128 * D - 1) // (128 * D)
    per_cu = min(16 // r32, 160 * 1024 // (2 * T * (128 * D + r32 * 256)))
    groups, phases = per_cu * cus // Hkv, ((blocks + 31) // 32 + T - 1) // T
    if batch > 64 or groups < batch or phases < groups // batch:
        return False
    rounds = -(-phases // (groups // batch))
    if batch > 1 and ((D == 64 and groups < 4 * batch) or (rounds > 1 and (groups < 2 * batch or phases * batch * Hkv < (0.72 if D == 128 else 0.85) * rounds * per_cu * cus))):
        return False
    return True


@pytest.fixture
def routes(gpu_lib):
    yield gpu_lib
    gpu_lib.specpv_debug_set_select_route(0)


@pytest.mark.parametrize("over,reduce,cap", [(o, r, None) for o, r in CASES] + [(o, "mean", n) for o, n in CAP],
                         ids=["-".join(str(v) for v in o.values()) + "-" + r for o, r in CASES] + ["cap-%d" % n for _, n in CAP])
def test_same_bits_as_tiles_at_once(routes, over, reduce, cap):
    sp = routes
    say("case", over, reduce, cap)
    cfg = dict(SMALL)
    cfg.update(over, rho=[0.1] * len(over["ctx"]))
    case = workloads.make_case(cfg, seed=13, device=torch.device("cuda"))
    assert by_streams(dict(cfg, reduce=reduce), cap or case["max_blocks"]) or torch.cuda.get_device_properties(0).multi_processor_count != 256
    if cap:
        k, v = case["k"], case["v"]
        case = dict(case, max_blocks=cap)
    run = GpuRun(sp, case, reduce=reduce, last_node=case["M"] // 2)
    if cap:
        run.kv = sp.KV(k, v, case["ctx_len"], case["B"], cap)
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
        nb = min((n + case["B"] - 1) // case["B"], case["max_blocks"])
        q = case["q"][b].double().view(case["M"], case["Hkv"], G, case["D"])
        for g in range(case["Hkv"]):
            rows = (q[last, g] if reduce == "last" else q[:, g].reshape(-1, case["D"]))
            s = torch.maximum(rows @ run.kmax[b, g, :nb].double().T, rows @ run.kmin[b, g, :nb].double().T)
            want = s.amax(0) if reduce == "max" else s.mean(0)
            # 128 products of a row, then up to 512 rows, in fp32: 640 roundings of 2^-24 against the largest sum of magnitudes
            bound = 640 * 2.0 ** -24 * float((rows.abs() @ torch.maximum(run.kmax[b, g, :nb].abs(), run.kmin[b, g, :nb].abs()).double().T).max()) if nb else 0.0
            assert nb == 0 or float((results[0][0][b, g, :nb].double() - want).abs().max()) <= bound
