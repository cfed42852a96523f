"""A refresh whose merge and scores go out as one launch against the same as two launches (select route 2): attention, lse,
scores, lists and counts the same bit for bit, with the scores in the caller's array and behind the partials of the workspace
(and, where they have no room there, in their place: the two launches again), every reducer, every count of partials that has a kernel of
its own, rows by node and packed, KV heads in eights and not, more wavefronts than blocks of query rows and the reverse.  The
first route's attention is checked against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from helpers import ATOL, GpuRun, say
from test_gpu_parity import SMALL

pytestmark = pytest.mark.gpu

CASES = [  # (over, reducer)
    (dict(ctx=[100], M=1, Hq=8, Hkv=8), "mean"), (dict(ctx=[700], M=24), "max"), (dict(ctx=[3000], M=60, Hq=32, Hkv=8), "last"),
    (dict(ctx=[9001], M=60, Hq=32, Hkv=8), "mean"), (dict(ctx=[20000], M=78, Hq=32, Hkv=8, B=64), "mean"), (dict(ctx=[33000], M=60, Hq=32, Hkv=8), "max"),
    (dict(ctx=[4000], M=60, Hq=40, Hkv=8), "mean"), (dict(ctx=[9000, 200, 5000], M=60, Hq=40, Hkv=8), "mean"), (dict(ctx=[9000, 0, 5000], M=60, Hq=32, Hkv=8), "last"),
    (dict(ctx=[5000], M=128, Hq=32, Hkv=2), "mean"), (dict(ctx=[5000], M=3, Hq=48, Hkv=3), "mean"), (dict(ctx=[2000] * 5, M=17, Hq=6, Hkv=3), "max"),
    (dict(ctx=[6000, 3000], M=37, Hq=32, Hkv=8, D=64), "mean"), (dict(ctx=[900], M=5, Hq=10, Hkv=2, D=64), "last"), (dict(ctx=[12000], M=64, Hq=16, Hkv=4, D=64), "max")]


@pytest.fixture
def routes(gpu_lib):
    yield gpu_lib
    gpu_lib.specpv_debug_set_select_route(0)


@pytest.mark.parametrize("over,reduce", CASES, ids=["-".join(str(v) for v in o.values()) + "-" + r for o, r in CASES])
def test_one_launch_equals_two(routes, over, reduce):
    sp = routes
    say("case", over, reduce)
    cfg = dict(SMALL, name="tail")
    cfg.update(over, rho=[0.1] * len(over["ctx"]))
    case = workloads.to_device(workloads.make_case(cfg, seed=91), "cuda")
    run = GpuRun(sp, case, reduce=reduce, last_node=case["M"] // 2 if reduce == "last" else 0)
    run.summarize()
    scores_bytes = (run.scores.numel() * 4 + 255) & ~255
    results = []
    for route in (0, 2):
        for place in ("array", "workspace", "small workspace"):
            sp.specpv_debug_set_select_route(route)
            ws = run.ws
            if place == "small workspace":   # room for the scores in the place of the partials, and for the partials
                rows = case["batch"] * case["Hq"] * case["M"]
                ws = run.ws[:max(65536 + 1024 + 64 * rows * (264 if case["D"] == 64 else 136), 65536 + scores_bytes) & ~255]
                if ws.numel() >= run.ws.numel():
                    continue
            for x in (run.out, run.lse, run.scores):
                x.zero_()
            run.sel_idx.fill_(-7)
            sp.specpv_full_verify_refresh(run.kv, run.tree, run.kmax, run.kmin, -1, run.cfg, run.out, run.lse, run.sel_idx, run.sel_count,
                                          run.scores if place == "array" else None, ws)
            torch.cuda.synchronize()
            results.append((route, place, run.out.clone(), run.lse.clone(), run.sel_idx.clone(), run.sel_count.clone(), run.scores.clone()))
            assert int(run.ws[:65536].sum()) == 0
    first = results[0]
    for r in results[1:]:
        names = ["out", "lse", "lists", "counts"] + (["scores"] if r[1] == "array" else [])
        if r[1] == "small workspace":
            names = ["lists", "counts"]   # (fewer splits may fit: other last bits)
        for n, a, b in zip(["out", "lse", "lists", "counts", "scores"], first[2:], r[2:]):
            if n in names:
                assert torch.equal(a, b), (r[:2], n)
    for b in range(case["batch"]):
        o = workloads.oracle_views(case, b)
        O, _, _ = oracle.tree_attention(o["Q"], o["K"], o["V"], o["Kd"], o["Vd"], o["parent"], case["B"], None, None)
        worst = np.abs(first[2][b].float().cpu().numpy() - O).max()
        assert worst <= ATOL["bf16"], (b, worst)
