"""The gather against the definition: block sizes around the pieces of a workgroup, lists with holes, counts below the row's
length, entries beyond the sequence, several sequences; bit for bit."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("D,Hkv,B,lengths,n_sel", [
    (128, 8, 64, [1000], 9), (128, 2, 16, [1, 513, 300], 5), (64, 1, 24, [200, 77], 1), (128, 3, 80, [0, 401], 6), (64, 8, 129, [1290], 12),
    (128, 8, 64, [1500], 64), (128, 8, 61, [900], 63),   # four passes to a workgroup
    (64, 1, 16, [300, 900], 475), (128, 3, 8, [500], 1030), (128, 1, 16, [200], 64), (64, 5, 16, [333], 129), (128, 19, 4, [90], 300),   # pieces of 64 entries dealt to four wavefronts
    (64, 20, 16, [300], 70),                              # more heads and entries than are looked at in one go for the length
    (64, 8, 16, [700, 5], 160)])                          # more workgroups than have a place at once
def test_gather_edges(gpu_lib, dtype, D, Hkv, B, lengths, n_sel):
    sp = gpu_lib
    rng = np.random.default_rng(B + n_sel)
    batch, T = len(lengths), max(lengths) + 3
    k, v = (torch.randn(batch, Hkv, T, D, generator=torch.Generator().manual_seed(s)).to(dtype).cuda() for s in (1, 2))
    most = (T + B - 1) // B
    kv = sp.KV(k, v, torch.tensor(lengths, dtype=torch.int32, device="cuda"), B, most)
    idx = rng.integers(-1, most + 2, (batch, Hkv, n_sel)).astype(np.int32)
    cnt = rng.integers(0, n_sel + 1, (batch, Hkv)).astype(np.int32)
    gk = torch.full((batch, Hkv, n_sel * B, D), 7.0, dtype=dtype, device="cuda")
    gv, glen = torch.full_like(gk, 7.0), torch.full((batch,), -5, dtype=torch.int32, device="cuda")
    sp.specpv_gather_blocks(kv, torch.from_numpy(idx).cuda(), torch.from_numpy(cnt).cuda(), gk, gv, glen)
    torch.cuda.synchronize()
    for b, L in enumerate(lengths):
        K, V = (x[b, :, :L].permute(1, 0, 2).double().cpu().numpy() for x in (k, v))
        Kg, Vg, rows = oracle.gather_blocks(K, V, B, idx[b], cnt[b])
        assert int(glen[b]) == int(rows.max())
        assert np.array_equal(gk[b].permute(1, 0, 2).double().cpu().numpy(), Kg)
        assert np.array_equal(gv[b].permute(1, 0, 2).double().cpu().numpy(), Vg)
