"""Which way full passes over batches go, told apart on the host by what specpv_workspace_bytes asks for: equal shares of all chunks,
worked out from the lengths, take as many slots as workgroups and (sequence, KV head) pairs; splits take so many to a pair."""
import ctypes

import pytest
import torch

import paper_2512_02337_amd as sp
from test_abi_cpu import _kv, _tree

cpu_only = pytest.mark.skipif(torch.cuda.is_available(), reason="the plans follow the GPU's count of CUs, 256 without one")


def workspace(batch, Hkv, G, M, ctx, D=128, B=64, dtype=1):
    blocks = (ctx + B - 1) // B
    kv = _kv(n_kv_heads=Hkv, head_dim=D, block_size=B, max_blocks=blocks, batch=batch, dtype=dtype, stride_t=D, stride_h=blocks * B * D, stride_b=Hkv * blocks * B * D)
    return sp.load().specpv_workspace_bytes(ctypes.byref(kv), ctypes.byref(_tree(M=M, n_q_heads=Hkv * G)), None)


def splits_asked_for(batch, Hkv, G, M, ctx, D=128, B=64, dtype=1):
    """The splits whose room (fp32 partials, one slot more, the scores) the workspace has."""
    up = lambda x: (x + 255) & ~255
    scores = up(batch * Hkv * ((ctx + B - 1) // B) * 4)
    rows = batch * Hkv * G * M
    got = workspace(batch, Hkv, G, M, ctx, D, B, dtype)
    for ns in range(1, 65):
        if 65536 + up(rows * (ns + 1) * D * 4) + up(rows * (ns + 1) * 8) + scores == got:
            return ns
    raise AssertionError("no count of splits asks for %d bytes" % got)


def room_of_shares(batch, Hkv, G, M, shares, D=128):
    """The splits that hold the slots of so many shares."""
    R, pairs = M * G, batch * Hkv
    bytes_ = (shares + pairs) * R * (2 * D + 8 if D == 128 else 4 * D + 8) + 512   # (fp16 partials at 128 channels)
    slot = pairs * R * (4 * D + 8)
    return max(1, (bytes_ + slot - 1) // slot - 1)


@cpu_only
@pytest.mark.parametrize("batch,Hkv,G,M,ctx,shares", [
    (16, 8, 5, 60, 3000, 256), (16, 8, 4, 60, 2048, 256), (10, 8, 4, 60, 4096, 256), (4, 8, 4, 60, 8192, 256), (8, 1, 4, 60, 32768, 256), (8, 1, 8, 37, 49152, 256),
    (4, 2, 4, 60, 32768, 256), (5, 4, 8, 60, 8000, 128), (16, 1, 4, 60, 24321, 256), (32, 1, 8, 24, 5746, 256), (3, 8, 5, 37, 12000, 256), (8, 2, 4, 37, 23722, 256), (4, 8, 4, 46, 5400, 256)])
def test_shares_where_one_long_sequence_would_wait_for_itself(batch, Hkv, G, M, ctx, shares):
    assert splits_asked_for(batch, Hkv, G, M, ctx) == room_of_shares(batch, Hkv, G, M, shares)


@cpu_only
@pytest.mark.parametrize("batch,Hkv,G,M,ctx", [(3, 4, 4, 37, 7055), (2, 2, 8, 24, 57746), (16, 1, 8, 37, 4710), (2, 2, 8, 37, 30000), (4, 8, 4, 46, 3480), (3, 8, 4, 60, 4400)])
def test_splits_where_their_chains_are_short(batch, Hkv, G, M, ctx):
    assert splits_asked_for(batch, Hkv, G, M, ctx) > room_of_shares(batch, Hkv, G, M, 256)


@cpu_only
@pytest.mark.parametrize("batch,Hkv,G,M,ctx,shares", [(16, 1, 4, 8, 36448, 256), (24, 1, 4, 1, 22336, 256), (4, 4, 4, 16, 26752, 256), (4, 8, 4, 1, 32416, 512), (16, 8, 8, 1, 13376, 512)])
def test_shares_of_few_rows(batch, Hkv, G, M, ctx, shares):
    assert splits_asked_for(batch, Hkv, G, M, ctx) == room_of_shares(batch, Hkv, G, M, shares)


@cpu_only
@pytest.mark.parametrize("batch,Hkv,G,M,ctx,shares", [(16, 8, 4, 1, 2654, 512), (32, 8, 8, 16, 4448, 512), (8, 8, 5, 16, 2300, 512), (24, 8, 5, 60, 2976, 256), (11, 8, 8, 60, 10528, 256)])
def test_64_channels_shares(batch, Hkv, G, M, ctx, shares):
    assert splits_asked_for(batch, Hkv, G, M, ctx, 64) == room_of_shares(batch, Hkv, G, M, shares, 64)


@cpu_only
@pytest.mark.parametrize("batch,Hkv,G,M,ctx,splits", [(8, 1, 4, 16, 30902, 61), (3, 8, 5, 24, 7802, 19), (8, 2, 4, 30, 10000, 29), (100, 4, 4, 60, 8192, 5), (2, 8, 4, 37, 30011, 32)])
def test_64_channels_splits(batch, Hkv, G, M, ctx, splits):
    assert splits_asked_for(batch, Hkv, G, M, ctx, 64) >= splits


@cpu_only
@pytest.mark.parametrize("batch,Hkv,M,ctx,shares", [(3, 8, 9, 8193, 512), (3, 8, 60, 8193, 256), (3, 8, 1, 8300, 512), (64, 1, 3, 8500, 256)])
def test_the_cases_of_uneven_batches(batch, Hkv, M, ctx, shares):
    assert splits_asked_for(batch, Hkv, 4, M, ctx, B=32) == room_of_shares(batch, Hkv, 4, M, shares)


@cpu_only
@pytest.mark.parametrize("batch,Hkv,G,M,ctx,D,splits", [(72, 1, 8, 60, 16384, 128, 8), (72, 1, 8, 60, 16384, 64, 8), (128, 2, 4, 24, 16384, 128, 2), (128, 2, 4, 24, 16384, 64, 8)])
def test_more_than_64_sequences(batch, Hkv, G, M, ctx, D, splits):
    assert splits_asked_for(batch, Hkv, G, M, ctx, D) == splits


@cpu_only
@pytest.mark.parametrize("batch,Hkv,G,M,ctx,D,least,most", [
    (11, 8, 8, 60, 3296, 128, 2, 2), (24, 8, 4, 60, 1344, 128, 2, 2), (32, 8, 4, 37, 1184, 64, 2, 2), (16, 8, 4, 5, 2432, 128, 7, 12), (4, 8, 4, 8, 5888, 128, 27, 32),
    (16, 8, 4, 8, 1312, 64, 7, 8), (16, 8, 4, 5, 1500, 128, 7, 11), (16, 8, 4, 4, 1500, 128, 1, 14)])
def test_fp32_splits(batch, Hkv, G, M, ctx, D, least, most):
    assert least <= splits_asked_for(batch, Hkv, G, M, ctx, D, dtype=0) <= most


@cpu_only
@pytest.mark.parametrize("batch,Hkv,G,M,ctx", [(48, 8, 5, 37, 619), (65, 8, 4, 24, 790), (32, 8, 8, 60, 1024)])
def test_64_channels_few_splits_up_to_1024_tokens(batch, Hkv, G, M, ctx):
    assert splits_asked_for(batch, Hkv, G, M, ctx, 64) == 1
