"""bf16 results are rounded to nearest, ties to even, fp32 subnormals included, and infinities and NaN stay what they are: means of two
and three V rows over all bf16 bit patterns, against integer arithmetic on the same fp32 values."""
import numpy as np
import pytest
import torch

from helpers import say

pytestmark = pytest.mark.gpu


def _widen(bits):
    return (bits.astype(np.uint32) << 16).view(np.float32)


def _round(x):
    u = x.view(np.uint32)
    return np.where(np.isnan(x), (u >> 16) | 0x40, (u + 0x7fff + ((u >> 16) & 1)) >> 16).astype(np.uint16)


@pytest.mark.parametrize("D,Hkv,G", [(128, 512, 1), (128, 512, 4), (64, 1024, 2), (64, 1024, 4)])
@pytest.mark.parametrize("step", [(1, 1), (1, 2), (0x100, 3), (0x80, 0x4001)])   # from each row's bits to the next one's
def test_means_of_rows(gpu_lib, D, Hkv, G, step):
    sp, dev = gpu_lib, torch.device("cuda")
    say("case", D, Hkv, G, step)
    M = 3   # a chain: node j attends the rows 0 .. j, all with the same weight (queries of zeros)
    first = np.arange(65536, dtype=np.uint32)
    bits = np.stack([first, first + step[0], first + step[0] + step[1]]).astype(np.uint16).reshape(M, Hkv, D)
    vd = torch.from_numpy(bits.view(np.int16).copy()).view(torch.bfloat16).view(1, M, Hkv, D).to(dev)
    q = torch.zeros((1, M, Hkv * G, D), dtype=torch.bfloat16, device=dev)
    kd = torch.ones((1, M, Hkv, D), dtype=torch.bfloat16, device=dev)
    cache = torch.zeros((1, Hkv, 16, D), dtype=torch.bfloat16, device=dev)
    kv = sp.KV(cache, cache, torch.zeros(1, dtype=torch.int32, device=dev), 16, 1)
    tree = sp.Tree(q, kd, vd, torch.tensor([[-1, 0, 1]], dtype=torch.int32, device=dev))
    ws = torch.zeros((sp.specpv_workspace_bytes(kv, tree, None),), dtype=torch.uint8, device=dev)
    out = torch.zeros_like(q)
    sp.specpv_partial_verify_attn(kv, tree, None, None, out, None, ws)
    torch.cuda.synchronize()
    got = out.view(torch.int16).cpu().numpy().view(np.uint16).reshape(M, Hkv, G, D)
    v = _widen(bits)
    with np.errstate(all="ignore"):
        for j in range(M):
            total = np.zeros((Hkv, D), dtype=np.float32)
            for x in range(j, -1, -1):   # the node, then its ancestors
                total = total + v[x]
            mean = total * (np.float32(1) / np.float32(j + 1))
            want = _round(mean)
            for g in range(G):
                nan = np.isnan(mean)
                assert np.array_equal(np.isnan(_widen(got[j, :, g])), nan), (j, g)
                assert np.array_equal(got[j, :, g][~nan], want[~nan]), (j, g)
