"""What the binding's extension module does where torch itself fails: an error that torch reports by a C++ exception
reaches the caller as the Python error of the same request, for every call (in a process of its own: an exception that
got away would end it)."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# tensors that claim to live on a GPU and have no memory: descriptors can be made of them, their checks pass, the
# addresses are never used
PROGRAM = r"""
import sys
import torch
from torch._subclasses.fake_tensor import FakeTensorMode
import paper_2512_02337_amd as sp
how = sys.argv[1]
FIRST = dict(summarize="summary", select="summary", partial="out", partial_static="out", refresh="out", gather="gathered", commit="buf",
             commit_layers="buf")   # the argument that is not an ordinary tensor under vmap
fake = FakeTensorMode(allow_non_fake_inputs=True)
bf, i4 = torch.bfloat16, torch.int32
with fake:
    new = lambda dt, *shape: torch.empty(shape, device="cuda", dtype=dt)
    k, kd, q = new(bf, 1, 2, 64, 64), new(bf, 1, 3, 2, 64), new(bf, 1, 3, 4, 64)
    kv = sp.KV(k, k, new(i4, 1), 16)
    tree = sp.Tree(q, kd, kd, new(i4, 1, 3))
    summary, idx, cnt, out = new(bf, *kv.summary_shape()), new(i4, 1, 2, 3), new(i4, 1, 2), new(bf, *q.shape)
    gathered, buf, per_seq, acc, ws = new(bf, 1, 2, 48, 64), new(bf, 1, 7, 2, 64), new(i4, 1), new(i4, 1, 2), new(torch.uint8, 1 << 20)
cfg = sp.SelectCfg(1, 1, 1)
last = dict(out=out, summary=summary, gathered=gathered, buf=buf)


def run(call, x):
    t = dict(last, **{FIRST[call]: x})
    if call == "summarize":
        sp.specpv_block_summarize(kv, 0, -1, t["summary"], summary)
    elif call == "select":
        sp.specpv_select_blocks(kv, tree, t["summary"], summary, cfg, idx, cnt, None, ws)
    elif call == "partial":
        sp.specpv_partial_verify_attn(kv, tree, idx, cnt, t["out"], None, ws)
    elif call == "partial_static":
        sp.specpv_partial_verify_attn_static(kv, tree, idx, cnt, t["out"], None)
    elif call == "refresh":
        sp.specpv_full_verify_refresh(kv, tree, summary, summary, -1, cfg, t["out"], None, idx, cnt, None, ws)
    elif call == "gather":
        sp.specpv_gather_blocks(kv, idx, cnt, t["gathered"], gathered)
    elif call == "commit":
        sp.specpv_commit_accepted(kv, t["buf"], buf, 4, 3, per_seq, acc, per_seq, sp.MODE_PARTIAL, workspace=ws)
    else:
        sp.specpv_commit_accepted_layers([kv], [t["buf"]], [buf], 4, 3, per_seq, acc, per_seq, sp.MODE_PARTIAL, workspace=ws)
    return x


sp.load()
for call, which in FIRST.items():
    try:
        if how == "vmap":
            with fake:
                torch.func.vmap(lambda x: run(call, x))(new(last[which].dtype, 2, *last[which].shape))
        else:
            run(call, last[which])
    except RuntimeError as e:
        print(call, "raised", str(e).replace("\n", " ")[:200], flush=True)
if how == "vmap":   # a query tensor that throws when it is asked for its address is let go of again
    from paper_2512_02337_amd import _native

    def tree_of(x):
        class Other:
            c, q, kd = tree.c, x, None
        before = sys.getrefcount(x)
        for _ in range(5):
            assert _native.partial(kv, Other, idx, cnt, out, None, ws) is None
        print("references", sys.getrefcount(x) - before, flush=True)
        return x
    with fake:
        torch.func.vmap(tree_of)(new(bf, 2, *q.shape))
"""


@pytest.mark.parametrize("how,says", [("vmap", "storage"), ("no GPU", "GPU")])
def test_errors_of_torch_are_python_errors(how, says):
    env = dict(os.environ, HIP_VISIBLE_DEVICES="-1", PYTHONPATH=ROOT)
    p = subprocess.run([sys.executable, "-c", PROGRAM, how], capture_output=True, text=True, timeout=300, env=env)
    assert p.returncode == 0, p.stdout + p.stderr[-2000:]
    lines = p.stdout.splitlines()
    calls = ["summarize", "select", "partial", "partial_static", "refresh", "gather", "commit", "commit_layers"]
    assert [l.split()[0] for l in lines[:len(calls)]] == calls, p.stdout
    assert all("raised" in l and says in l for l in lines[:len(calls)]), p.stdout
    assert lines[len(calls):] == (["references 0"] if how == "vmap" else []), p.stdout
