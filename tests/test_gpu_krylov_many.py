"""mc_lanczos_reorth on many vectors: whole sets of eight, a remainder, and
both on vectors of one and of several parts, against numpy.

Tolerance: as for few vectors, 1e-12: every sum is a fixed tree over at most
5,000 terms of size at most 1."""

import ctypes

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,n", [(15, 200), (24, 700), (33, 5000), (64, 300), (100, 1001), (203, 900)])
def test_many_vectors(mc, K, n):
    from paper_2005_13679_amd import _lib as L
    rng = np.random.default_rng(K)
    V = np.linalg.qr(rng.standard_normal((n, K)) + 1j * rng.standard_normal((n, K)))[0].T.copy()
    w = rng.standard_normal(n) + 1j * rng.standard_normal(n)
    w /= np.linalg.norm(w)
    ref = w.copy()
    for _ in range(2):
        ref = ref - V.T @ (V.conj() @ ref)
    P = lambda t: ctypes.c_void_p(t.data_ptr())
    Vd, wd = torch.from_numpy(V).cuda(), torch.from_numpy(w).cuda()
    out = torch.empty_like(wd)
    ab = torch.empty(4, dtype=torch.float64, device="cuda")
    ws = torch.empty((K + 1) * (L.MC_REORTH_BLOCKS + 2) * 16, dtype=torch.uint8, device="cuda")
    st = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    L.check(L.load().mc_lanczos_reorth(K, n, P(Vd), n, P(wd), P(out), P(ab), P(ab[2:]), P(ws),
                                       ws.numel(), st), "mc_lanczos_reorth")
    a = ab.tolist()
    assert abs(complex(a[0], a[1]) - np.vdot(V[-1], w)) <= 1e-12
    assert abs(a[2] - np.linalg.norm(ref)) <= 1e-12
    assert np.max(np.abs(out.cpu().numpy() * a[2] - ref)) <= 1e-12
