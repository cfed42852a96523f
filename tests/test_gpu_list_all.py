"""Lists that keep every block there can be (max_blocks <= ns + k + nr): selection and refresh take no scores that nobody asked
for, and write the lists beside the merge.  The same lists, counts, attention and (where asked for) scores as with the scores in an
array and as two launches, on either side of the line, for empty and short sequences, entries behind the count, both types, both
score kinds and tile counts."""
import numpy as np
import pytest
import torch

import workloads
from helpers import GpuRun, say
from test_gpu_parity import SMALL

pytestmark = pytest.mark.gpu

CASES = [  # (over, kept less max_blocks, entries for later commits, score)
    (dict(ctx=[1000]), 0, 0, "eq2"), (dict(ctx=[1000]), -1, 3, "eq2"), (dict(ctx=[1000]), 70, 300, "eq2"),
    (dict(ctx=[9000, 0, 31], M=60, Hq=40, Hkv=8), 5, 2, "eq2"), (dict(ctx=[128], M=1, Hq=32, Hkv=8), 9, 0, "eq2"), (dict(ctx=[129], M=1, Hq=32, Hkv=8), 0, 1, "eq2"),
    (dict(ctx=[700, 3000], M=24), 1, 0, "channel_bound"), (dict(ctx=[1500, 600], M=37, Hq=6, Hkv=3, D=64, B=32), 3, 4, "eq2"),
    (dict(ctx=[800, 1, 430], D=64, dtype="f32", B=7), 2, 1, "eq2"), (dict(ctx=[2000], dtype="f32", M=5), 0, 5, "eq2")]


@pytest.fixture
def routes(gpu_lib):
    yield gpu_lib
    gpu_lib.specpv_debug_set_select_route(0)


@pytest.mark.parametrize("over,spare,extra,score", CASES, ids=["-".join(str(v) for v in o.values()) + "-%d-%d-%s" % (p, e, s) for o, p, e, s in CASES])
def test_every_block_is_listed(routes, over, spare, extra, score):
    sp = routes
    say("case", over, spare, extra, score)
    cfg = dict(SMALL, name="all")
    cfg.update(over, rho=[0.1] * len(over["ctx"]))
    case = workloads.to_device(workloads.make_case(cfg, seed=5), "cuda")
    run = GpuRun(sp, case, cfg=(2, 3, case["max_blocks"] + spare - 5), score=score)
    run.cfg = sp.SelectCfg(2, 3, case["max_blocks"] + spare - 5, "mean", score, extra)
    run.sel_idx = torch.zeros((case["batch"], case["Hkv"], run.cfg.n_sel), dtype=torch.int32, device="cuda")
    run.summarize()
    results = []
    for route in (0, 2):
        sp.specpv_debug_set_select_route(route)
        for scores in (run.scores, None):
            for call in ("select", "refresh"):
                run.scores.zero_()
                run.sel_idx.fill_(-7)
                run.sel_count.fill_(-7)
                if call == "select":
                    sp.specpv_select_blocks(run.kv, run.tree, run.kmax, run.kmin, run.cfg, run.sel_idx, run.sel_count, scores, run.ws)
                else:
                    run.out.zero_()
                    sp.specpv_full_verify_refresh(run.kv, run.tree, run.kmax, run.kmin, -1, run.cfg, run.out, run.lse, run.sel_idx, run.sel_count, scores, run.ws)
                torch.cuda.synchronize()
                assert int(run.ws[:65536].sum()) == 0
                results.append((call, scores is not None, run.sel_idx.clone(), run.sel_count.clone(), run.scores.clone(), run.out.clone(), run.lse.clone()))
    for call, scored, idx, count, sc, out, lse in results:
        assert torch.equal(idx, results[0][2]) and torch.equal(count, results[0][3])
        assert not scored or torch.equal(sc, results[0][4])
        assert call == "select" or (torch.equal(out, results[1][5]) and torch.equal(lse, results[1][6]))
    if spare >= 0:
        blocks = [(n + case["B"] - 1) // case["B"] for n in case["ctx_len"].tolist()]
        entry = np.arange(run.cfg.n_sel)
        for b, nb in enumerate(blocks):
            assert (results[0][2][b].cpu().numpy() == np.where(entry < nb, entry, -1)).all() and (results[0][3][b] == nb).all()


@pytest.mark.parametrize("ctx", [100, 128, 129, 700])
def test_no_scores_that_nobody_asked_for(routes, ctx):
    """A refresh whose lists keep every block leaves the place behind the partials as it was, whatever the number of blocks."""
    sp = routes
    say("case", ctx)
    cfg = dict(SMALL, name="all")
    cfg.update(ctx=[ctx], rho=[0.1])
    case = workloads.to_device(workloads.make_case(cfg, seed=5), "cuda")
    run = GpuRun(sp, case, cfg=(2, 3, case["max_blocks"]))
    run.summarize()
    left = []
    for scores in (None, run.scores):
        run.ws.zero_()
        sp.specpv_full_verify_refresh(run.kv, run.tree, run.kmax, run.kmin, -1, run.cfg, run.out, run.lse, run.sel_idx, run.sel_count, scores, run.ws)
        torch.cuda.synchronize()
        left.append(run.ws.clone())
    assert torch.equal(left[0], left[1])
