"""mc_zgemv_c (c = V^H w) and mc_zgemv_sub (w -= V c) called by themselves,
against numpy: one and several vectors, rows longer than their vectors, less
than one and more than one chunk of 64, and nothing to do.

Tolerance: sums of at most 20,000 terms of size at most 1 in fixed trees of under
400 additions in a row: 1e-12."""

import ctypes

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,n", [(1, 1), (1, 20000), (3, 63), (7, 1000), (40, 4097)])
def test_projection_and_update(mc, K, n):
    from paper_2005_13679_amd import _lib as L
    lib, rng, ldv = L.load(), np.random.default_rng(K + n), n + 5
    V = rng.standard_normal((K, ldv)) + 1j * rng.standard_normal((K, ldv))
    V /= np.linalg.norm(V[:, :n], axis=1)[:, None]
    w = rng.standard_normal(n) + 1j * rng.standard_normal(n)
    w /= np.linalg.norm(w)
    P = lambda t: ctypes.c_void_p(t.data_ptr())
    st = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    Vd, wd = torch.from_numpy(V).cuda(), torch.from_numpy(w).cuda()
    c = torch.empty(K, dtype=torch.complex128, device="cuda")
    ws = torch.empty(K * 64 * 16, dtype=torch.uint8, device="cuda")
    assert lib.mc_zgemv_c(K, n, P(Vd), ldv, P(wd), P(c), P(ws), ws.numel(), st) == L.MC_OK
    ref = V[:, :n].conj() @ w
    assert np.abs(c.cpu().numpy() - ref).max() <= 1e-12
    assert lib.mc_zgemv_sub(K, n, P(Vd), ldv, P(c), P(wd), st) == L.MC_OK
    assert np.abs(wd.cpu().numpy() - (w - V[:, :n].T @ ref)).max() <= 1e-12
    before = wd.clone()
    assert lib.mc_zgemv_c(0, n, P(Vd), ldv, P(wd), P(c), P(ws), ws.numel(), st) == L.MC_OK
    assert lib.mc_zgemv_sub(0, n, P(Vd), ldv, P(c), P(wd), st) == L.MC_OK
    assert torch.equal(wd, before)
    assert lib.mc_zgemv_c(K, n, P(Vd), ldv, P(wd), P(c), P(ws), ws.numel() - 1, st) == L.MC_ENOMEM
    assert lib.mc_zgemv_sub(K, n, P(Vd), n - 1, P(c), P(wd), st) == L.MC_EINVAL
