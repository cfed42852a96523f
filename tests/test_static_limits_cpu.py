"""Full passes over more than 64 sequences that specpv_partial_verify_attn_static takes: the plan that runs them fits its array (host-only:
without a device such a call ends at its first launch, one that is too large before it)."""
import ctypes

import pytest
import torch

import paper_2512_02337_amd as sp
from test_abi_cpu import _kv, _tree

EHIP, ELIMIT = -4, -3


@pytest.mark.skipif(torch.cuda.is_available(), reason="the addresses are not memory")
@pytest.mark.parametrize("Hkv, G, D, M, B, blocks, batch, status", [
    (2, 2, 64, 64, 64, 797, 100, EHIP), (2, 4, 128, 24, 64, 256, 128, EHIP), (4, 4, 64, 37, 64, 64, 70, ELIMIT), (8, 4, 128, 60, 64, 64, 80, ELIMIT)])
def test_full_pass_over_many_sequences(Hkv, G, D, M, B, blocks, batch, status):
    kv = _kv(n_kv_heads=Hkv, head_dim=D, block_size=B, max_blocks=blocks, batch=batch, dtype=1, stride_t=D, stride_h=blocks * B * D,
             stride_b=Hkv * blocks * B * D)
    tree = _tree(M=M, n_q_heads=Hkv * G)
    assert sp.load().specpv_partial_verify_attn_static(ctypes.byref(kv), ctypes.byref(tree), None, None, 0, ctypes.c_void_p(0x300), None, None) == status
