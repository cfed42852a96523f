"""Precision of the sums against 64 bits.

Draft segment: its log-sum-exp alone (no context), which is not rounded to 16 bits.

bf16 at 64 channels: the softmax weights reach the second product with all of fp32's bits.

The output's own rounding (2^-9) hides what the sums lose, so the values are chosen to cancel: the last tokens of every KV
head share a key, and their values take away what all others sum up to, until the exact result is nearly 0 and the output
shows the error of the sums itself.  All rows of a head are the same (one query, trees of roots with one key and value 0),
so that every row block of every kernel variant is looked at.

Bound: relative to sum |w v|, n independent errors of the weights average to delta / sqrt(n).  In fp32 delta comes from the
scores (|z| < 8 log2(e), rounded to 2^-24 of it a few times: about 2^-21.5 measured on the vector ALU as well); weights
rounded to 16 bits have up to 2^-17, 2^-17.8 in the mean.  2^-19 stands between the two."""
import math

import pytest
import torch

from helpers import say

pytestmark = pytest.mark.gpu

CASES = [   # tokens per sequence, nodes, query heads per KV head, block size, kept list
    ([300], 1, 1, 32, True),
    ([300], 1, 1, 16, False),
    ([2048], 30, 4, 64, False),         # four row blocks
    ([2048], 37, 4, 32, True),          # six
    ([1000], 60, 4, 48, False),         # eight; blocks that are no multiple of a chunk
    ([2500, 1200], 37, 4, 32, False),   # shares of a ragged batch's chunks
    ([2500, 1200], 60, 5, 16, False),   # ... ten row blocks in two workgroups
]


def _parts(q, K, V, kd):
    """fp64 weights of the tokens (and, last, the draft node) and the output of one row; q [D], K, V [T, D], kd [D]."""
    z = torch.cat([K, kd[None]]).double() @ q.double() / math.sqrt(q.shape[0])
    w = torch.softmax(z, 0)
    return w, w[:-1] @ V.double()


@pytest.mark.parametrize("lens,M,G,B,kept", CASES)
def test_weights_keep_their_bits(gpu_lib, lens, M, G, B, kept):
    sp, dev, D, Hkv, bf = gpu_lib, "cuda", 64, 4, torch.bfloat16
    bt, nb = len(lens), (max(lens) + B - 1) // B
    g = torch.Generator(device=dev).manual_seed(M + max(lens))
    rn = lambda *s: torch.randn(s, generator=g, device=dev).to(bf)
    k, v, q1, kd1 = rn(bt, Hkv, nb * B, D), rn(bt, Hkv, nb * B, D), rn(bt, Hkv, D), rn(bt, Hkv, D)
    for b, T in enumerate(lens):
        for h in range(Hkv):
            k[b, h, T - 4:T] = k[b, h, T - 4]
            v[b, h, T - 4:T] = 0
            for t in range(T - 4, T):   # a value has 8 bits: four tokens take the sum down to about 2^-32 of itself
                w, o = _parts(q1[b, h], k[b, h, :T], v[b, h, :T], kd1[b, h])
                v[b, h, t] = (-o / w[t]).to(bf)
    q = q1[:, None, :, None, :].expand(bt, M, Hkv, G, D).reshape(bt, M, Hkv * G, D).contiguous()
    kd = kd1[:, None].expand(bt, M, Hkv, D).contiguous()
    kv = sp.KV(k, v, torch.tensor(lens, dtype=torch.int32, device=dev), B, nb)
    tree = sp.Tree(q, kd, torch.zeros_like(kd), torch.full((bt, M), -1, dtype=torch.int32, device=dev))
    out, ws = torch.zeros_like(q), torch.zeros((sp.specpv_workspace_bytes(kv, tree),), dtype=torch.uint8, device=dev)
    idx = cnt = None
    if kept:
        idx = torch.arange(nb, dtype=torch.int32, device=dev).repeat(bt, Hkv, 1).contiguous()
        cnt = torch.full((bt, Hkv), nb, dtype=torch.int32, device=dev)
    sp.specpv_partial_verify_attn(kv, tree, idx, cnt, out, None, ws)
    torch.cuda.synchronize()
    for b, T in enumerate(lens):
        err = []
        for h in range(Hkv):
            w, o = _parts(q1[b, h], k[b, h, :T], v[b, h, :T], kd1[b, h])
            mag = w[:-1] @ v[b, h, :T].double().abs()
            err.append((out[b, :, h * G:(h + 1) * G].double() - o) / mag)
        rms = torch.stack(err).pow(2).mean().sqrt().item()
        say("   %d tokens, %d nodes, G = %d, B = %d: rms error / sum |w v| = 2^%.1f / sqrt(n)" % (T, M, G, B, math.log2(rms * math.sqrt(T))))
        assert rms <= 2.0 ** -19 / math.sqrt(T), (lens, M, G, B, kept, T, rms)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_draft_scores_are_fp32(gpu_lib, D, dtype):
    """Products of 16-bit inputs are exact in fp32; what a sum of D of them loses is bounded here by eight roundings of the
    sum of their magnitudes (the vector ALU's chain of eight per lane and four more across lanes: 1.2e-6 to 2.6e-6 at
    most on these inputs, with either of its instructions for the products), and the log-sum-exp adds two of its own."""
    sp, dev, Hkv, G, M = gpu_lib, "cuda", 2, 4, 60
    g = torch.Generator(device=dev).manual_seed(D)
    rn = lambda *s: torch.randn(s, generator=g, device=dev).to(dtype)
    k, kd, vd, q = rn(1, Hkv, 64, D), rn(1, M, Hkv, D), rn(1, M, Hkv, D), 4 * rn(1, M, Hkv * G, D)
    parent = [-1] + [(j - 1) // 2 for j in range(1, M)]
    kv = sp.KV(k, k, torch.zeros((1,), dtype=torch.int32, device=dev), 64)
    tree = sp.Tree(q, kd, vd, torch.tensor([parent], dtype=torch.int32, device=dev))
    out, lse = torch.zeros_like(q), torch.zeros((1, M, Hkv * G), device=dev)
    sp.specpv_partial_verify_attn(kv, tree, None, None, out, lse, torch.zeros((sp.specpv_workspace_bytes(kv, tree),), dtype=torch.uint8, device=dev))
    torch.cuda.synchronize()
    worst = 0.0
    for j in range(M):
        path, a = [], j
        while a >= 0:
            path.append(a)
            a = parent[a]
        for h in range(Hkv * G):
            p = kd[0, path, h // G].double() * q[0, j, h].double() / math.sqrt(D)
            want, mag = torch.logsumexp(p.sum(1), 0).item(), p.abs().sum(1).max().item()
            err = abs(lse[0, j, h].item() - want)
            worst = max(worst, err)
            assert err <= 2.0 ** -24 * (8 * mag + 2 * (abs(want) + 1)), (D, dtype, j, h, err, mag, want)
    say("   D = %d, %s: max error %.3g" % (D, dtype, worst))
