"""A refresh whose merge and scores go out as one launch against the same as two launches (select route 2): attention, lse,
scores, lists and counts the same bit for bit, with the scores in the caller's array and behind the partials of the workspace,
every reducer, every count of partials that has a kernel of its own, rows by node and packed, KV heads in eights and not, more wavefronts
than blocks of query rows and the reverse, key-only nodes in front of the tree, summaries that are recomputed.  The first route's
attention is checked against the oracle.  In a workspace without room for the scores behind the partials they take the partials'
place, in two launches: sizes on either side of that line, told apart by where the scores are found, with nothing written behind."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from helpers import ATOL, GpuRun, say, with_pending
from test_gpu_parity import SMALL

pytestmark = pytest.mark.gpu

CASES = [  # (over, reducer)
    (dict(ctx=[100], M=1, Hq=8, Hkv=8), "mean"), (dict(ctx=[700], M=24), "max"), (dict(ctx=[3000], M=60, Hq=32, Hkv=8), "last"),
    (dict(ctx=[9001], M=60, Hq=32, Hkv=8), "mean"), (dict(ctx=[20000], M=78, Hq=32, Hkv=8, B=64), "mean"), (dict(ctx=[33000], M=60, Hq=32, Hkv=8), "max"),
    (dict(ctx=[4000], M=60, Hq=40, Hkv=8), "mean"), (dict(ctx=[9000, 200, 5000], M=60, Hq=40, Hkv=8), "mean"), (dict(ctx=[9000, 0, 5000], M=60, Hq=32, Hkv=8), "last"),
    (dict(ctx=[3480, 2610, 1740, 870], M=66, Hq=32, Hkv=8, B=64), "max"), (dict(ctx=[5000], M=128, Hq=32, Hkv=2), "mean"), (dict(ctx=[5000], M=3, Hq=48, Hkv=3), "mean"), (dict(ctx=[2000] * 5, M=17, Hq=6, Hkv=3), "max"),
    (dict(ctx=[6000, 3000], M=37, Hq=32, Hkv=8, D=64), "mean"), (dict(ctx=[900], M=5, Hq=10, Hkv=2, D=64), "last"), (dict(ctx=[12000], M=64, Hq=16, Hkv=4, D=64), "max")]


@pytest.fixture
def routes(gpu_lib):
    yield gpu_lib
    gpu_lib.specpv_debug_set_select_route(0)


PENDING = [  # (over, reducer, key-only nodes, stale from)
    (dict(ctx=[9001], M=60, Hq=32, Hkv=8), "last", 16, -1), (dict(ctx=[9000, 200, 5000], M=37, Hq=40, Hkv=8), "last", 7, -1), (dict(ctx=[700], M=24), "mean", 20, 3),
    (dict(ctx=[6000, 3000], M=37, Hq=32, Hkv=8, D=64), "last", 9, -1), (dict(ctx=[20000], M=60, Hq=32, Hkv=8, B=64), "max", 18, 0),
    (dict(ctx=[9000, 200, 5000], M=60, Hq=40, Hkv=8), "mean", 0, 0), (dict(ctx=[30000, 9000, 20000], M=60, Hq=40, Hkv=8, B=64), "mean", 0, 0),
    (dict(ctx=[20000, 30000], M=60, Hq=40, Hkv=8, B=64), "last", 5, 17), (dict(ctx=[9000, 4000, 5000], M=30, Hq=40, Hkv=8, D=64), "max", 0, 0)]


def _setup(sp, over, reduce, n_key=0, keep=None):
    cfg = dict(SMALL, name="tail")
    cfg.update(over, rho=[0.1] * len(over["ctx"]))
    case = workloads.make_case(cfg, seed=91)
    if n_key:
        case = with_pending(case, n_key, seed=92)
    case = workloads.to_device(case, "cuda")
    return case, GpuRun(sp, case, reduce=reduce, last_node=n_key + case["M"] // 2 if reduce == "last" else n_key, cfg=keep)


def _refresh(sp, run, scores, ws, stale=-1):
    for x in (run.out, run.lse, run.scores):
        x.zero_()
    run.sel_idx.fill_(-7)
    sp.specpv_full_verify_refresh(run.kv, run.tree, run.kmax, run.kmin, stale, run.cfg, run.out, run.lse, run.sel_idx, run.sel_count, scores, ws)
    torch.cuda.synchronize()


def _against_the_oracle(case, out, n_key=0):
    for b in range(case["batch"]):
        o = workloads.oracle_views(case, b)
        O, _, _ = oracle.tree_attention(o["Q"], o["K"], o["V"], o["Kd"], o["Vd"], o["parent"], case["B"], None, None, n_key_only=n_key)
        worst = np.abs(out[b].float().cpu().numpy() - O).max()
        assert worst <= ATOL["bf16"], (b, worst)


@pytest.mark.parametrize("over,reduce", CASES, ids=["-".join(str(v) for v in o.values()) + "-" + r for o, r in CASES])
def test_one_launch_equals_two(routes, over, reduce):
    sp = routes
    say("case", over, reduce)
    case, run = _setup(sp, over, reduce)
    run.summarize()
    results = []
    for route in (0, 2):
        for place in ("array", "workspace"):
            sp.specpv_debug_set_select_route(route)
            _refresh(sp, run, run.scores if place == "array" else None, run.ws)
            results.append((route, place, run.out.clone(), run.lse.clone(), run.sel_idx.clone(), run.sel_count.clone(), run.scores.clone()))
            assert int(run.ws[:65536].sum()) == 0
    first = results[0]
    for r in results[1:]:
        names = ["out", "lse", "lists", "counts"] + (["scores"] if r[1] == "array" else [])
        for n, a, b in zip(["out", "lse", "lists", "counts", "scores"], first[2:], r[2:]):
            if n in names:
                assert torch.equal(a, b), (r[:2], n)
    _against_the_oracle(case, first[2])


@pytest.mark.parametrize("over,reduce,n_key,stale", PENDING, ids=["-".join(str(v) for v in o.values()) + "-%s-%d-%d" % (r, k, t) for o, r, k, t in PENDING])
def test_pending_nodes_and_stale_summaries(routes, over, reduce, n_key, stale):
    sp = routes
    say("case", over, reduce, n_key, stale)
    case, run = _setup(sp, over, reduce, n_key)
    run.summarize()
    sums = run.kmax.clone(), run.kmin.clone()
    results = []
    for route in (0, 2):
        sp.specpv_debug_set_select_route(route)
        if stale >= 0:
            run.kmax[:, :, stale:] = 0
            run.kmin[:, :, stale:] = 0
        _refresh(sp, run, run.scores, run.ws, stale)
        results.append([x.clone() for x in (run.out, run.lse, run.sel_idx, run.sel_count, run.scores, run.kmax, run.kmin)])
    for a, b in zip(*results):
        assert torch.equal(a, b)
    assert torch.equal(results[0][5], sums[0]) and torch.equal(results[0][6], sums[1])
    _against_the_oracle(case, results[0][0], n_key)
    select = GpuRun(sp, case, reduce=reduce, last_node=run.tree.c.last_node)   # the selection as a call of its own
    select.summarize()
    sp.specpv_debug_set_select_route(0)
    select.select()
    torch.cuda.synchronize()
    assert torch.equal(select.scores, results[0][4]) and torch.equal(select.sel_idx, results[0][2]) and torch.equal(select.sel_count, results[0][3])


@pytest.mark.parametrize("over,reduce", CASES, ids=["-".join(str(v) for v in o.values()) + "-" + r for o, r in CASES])
def test_room_behind_the_partials(routes, over, reduce):
    sp = routes
    say("case", over, reduce)
    # (lists that keep every block need no scores)
    case, run = _setup(sp, over, reduce, keep=(1, 1, 3) if max(over["ctx"]) <= 14 * 16 else None)
    run.summarize()
    sp.specpv_debug_set_select_route(0)
    head, need = 65536, (run.scores.numel() * 4 + 255) & ~255
    _refresh(sp, run, run.scores, run.ws)
    want = [x.clone() for x in (run.out, run.lse, run.sel_idx, run.sel_count)]
    scores = run.scores.clone().view(case["batch"], case["Hkv"], -1)
    blocks = [(L + case["B"] - 1) // case["B"] for L in case["ctx_len"].tolist()]

    def found(ws, at):
        if at + scores.numel() * 4 > ws.numel():
            return False
        got = ws[at:at + scores.numel() * 4].view(torch.float32).view(scores.shape)
        return all(torch.equal(got[b, :, :n], scores[b, :, :n]) for b, n in enumerate(blocks))

    run.ws.zero_()
    _refresh(sp, run, None, run.ws)
    first = int(next(b for b, n in enumerate(blocks) if n > 0)) * scores.stride(0)   # a score that is written, and where it may be
    words = run.ws.view(torch.float32)
    behind = [at for at in (((words == scores.flatten()[first]).nonzero().flatten() - first) * 4).tolist() if at >= head and at % 256 == 0 and found(run.ws, at)]
    assert len(behind) == 1 and behind[0] > head, "the scores are not behind the partials"
    edge = behind[0] + need
    buf = torch.zeros((edge + 4096,), dtype=torch.uint8, device="cuda")
    # (a plan asks for 512 bytes over its rows, and with fewer it takes a split less: other places, other last bits)
    smaller = [size for size in (edge - 1, edge - 256, behind[0] + 512) if max(behind[0] + 512, head + need) <= size < edge]
    assert smaller or need < 1024
    for size, at in ([(edge, behind[0])] if need >= 512 else []) + [(size, head) for size in smaller]:
        buf.zero_()
        buf[size:] = 0xa5
        _refresh(sp, run, None, buf[:size])
        assert bool((buf[size:] == 0xa5).all()), "written behind the workspace"
        assert found(buf[:size], at), (size, at)
        assert int(buf[:head].sum()) == 0
        for a, b in zip(want, (run.out, run.lse, run.sel_idx, run.sel_count)):
            assert torch.equal(a, b), size
