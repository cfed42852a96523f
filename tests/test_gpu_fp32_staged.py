"""fp32 attention with K and V rows by way of LDS (attn_f32.hip) against the oracle at 1e-5: rows on either side of a tile and of a
workgroup, tokens on either side of where the kernel takes over and of a chunk, 16 and 32 tokens a chunk, block sizes that chunks cut
through, both layouts, batches with an empty and a short sequence, lists that are not full; rows that no list names hold infinities."""
import numpy as np
import pytest
import torch

import workloads
from helpers import GpuRun, say
from test_gpu_parity import SMALL, _check_attn

pytestmark = pytest.mark.gpu

CASES = [  # (over, kept blocks)
    (dict(ctx=[1025], B=16, M=49, Hq=1, Hkv=1), 65), (dict(ctx=[2049], B=64, M=17, Hq=2, Hkv=2), 33), (dict(ctx=[2090], B=7, M=64, Hq=2, Hkv=2), 290),
    (dict(ctx=[4100], B=16, M=65, Hq=4, Hkv=2), 200), (dict(ctx=[3000, 0, 40, 2500], B=33, M=60, Hq=8, Hkv=2), 60), (dict(ctx=[6000], B=64, M=60, Hq=32, Hkv=8), 40),
    (dict(ctx=[9000], B=32, M=37, Hq=32, Hkv=8), 270), (dict(ctx=[1100] * 6, B=16, M=37, Hq=8, Hkv=2), 66),
    (dict(ctx=[4097], B=16, M=17, Hq=2, Hkv=2, D=64), 258), (dict(ctx=[5000], B=25, M=33, Hq=4, Hkv=1, D=64), 190), (dict(ctx=[8200, 31, 0], B=64, M=60, Hq=8, Hkv=2, D=64), 128),
    (dict(ctx=[2048] * 4, B=32, M=60, Hq=32, Hkv=8, D=64), 50)]


@pytest.mark.parametrize("over,kept", CASES, ids=["-".join(str(v) for v in o.values()) for o, _ in CASES])
def test_against_the_oracle(gpu_lib, over, kept):
    say("case", over, kept)
    cfg = dict(SMALL, dtype="f32")
    cfg.update(over, rho=[0.1] * len(over["ctx"]))
    case = workloads.to_device(workloads.make_case(cfg, seed=37), "cuda")
    rs = np.random.RandomState(3)
    lists = np.full((case["batch"], case["Hkv"], kept), -1, dtype=np.int32)
    counts = np.zeros((case["batch"], case["Hkv"]), dtype=np.int32)
    B = case["B"]
    for layout in ("bhtd", "bthd"):
        run = GpuRun(gpu_lib, case, layout=layout)
        run.attend(None, None)
        torch.cuda.synchronize()
        _check_attn(run, case, None, "every block, " + layout)
    for b in range(case["batch"]):
        nb = (int(case["ctx_len"][b]) + B - 1) // B
        named = np.sort(rs.choice(np.arange(1, nb), min(max(nb - 3, 0), kept), replace=False)) if nb > 1 else np.zeros(0, int)   # not block 0
        for g in range(case["Hkv"]):
            counts[b, g] = max(0, len(named) - g)   # one entry less from head to head
            lists[b, g, :counts[b, g]] = named[:counts[b, g]]
        for name in ("k", "v"):
            rows = case[name][b].view(case["Hkv"], -1, B, case["D"])
            for g in range(case["Hkv"]):
                other = np.setdiff1d(np.arange(rows.shape[1]), lists[b, g, :counts[b, g]])
                rows[g, torch.as_tensor(other, device="cuda")] = float("inf")
    for layout in ("bhtd", "bthd"):
        run = GpuRun(gpu_lib, case, layout=layout)
        run.attend(torch.as_tensor(lists, device="cuda"), torch.as_tensor(counts, device="cuda"))
        torch.cuda.synchronize()
        _check_attn(run, case, [(lists[b], counts[b]) for b in range(case["batch"])], "listed blocks, " + layout)
