"""mc_lanczos_reorth (classical Gram-Schmidt twice, norm and scaling in four
passes) against numpy: every width of the fused pass and both sides of its
limit (12 vectors), vectors shorter than one block and with ragged parts.

Tolerance: the sums have at most 70,001 terms of size at most 1 (normalised
rows) in partial sums of at most 256 threads; n eps = 1.6e-11 bounds the worst
order, 1e-12 holds for the fixed tree (under 300 additions in a row)."""

import ctypes

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _reorth(mc, V, w, K, n, ldv, in_place):
    from paper_2005_13679_amd import _lib as L
    lib = L.load()
    P = lambda t: ctypes.c_void_p(t.data_ptr())
    out = w if in_place else torch.empty_like(w)
    ab = torch.empty(4, dtype=torch.float64, device="cuda")
    ws = torch.empty((K + 1) * (L.MC_REORTH_BLOCKS + 2) * 16, dtype=torch.uint8, device="cuda")
    st = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    L.check(lib.mc_lanczos_reorth(K, n, P(V), ldv, P(w), P(out), P(ab), P(ab[2:]), P(ws),
                                  ws.numel(), st), "mc_lanczos_reorth")
    a = ab.tolist()
    return out.cpu().numpy(), complex(a[0], a[1]), a[2]


@pytest.mark.parametrize("K,n", [(1, 1), (1, 70001), (2, 255), (3, 257), (4, 3000), (5, 70001),
                                 (6, 513), (7, 1025), (8, 70001), (9, 4097), (10, 300),
                                 (11, 2000), (12, 70001), (13, 70001), (16, 5000), (21, 9999)])
def test_matches_numpy(mc, K, n):
    rng = np.random.default_rng(31 * K + n)
    ldv = n + 3
    z = lambda *s: rng.standard_normal(s) + 1j * rng.standard_normal(s)
    basis = np.linalg.qr(z(n, K))[0].T if n >= K else z(K, n)
    V = np.zeros((K, ldv), dtype=np.complex128)
    V[:, :n] = basis
    w = z(n)
    w /= np.linalg.norm(w)
    ref, alpha = w.copy(), np.vdot(V[K - 1, :n], w)
    for _ in range(2):
        ref = ref - V[:, :n].T @ (V[:, :n].conj() @ ref)
    beta = np.linalg.norm(ref)
    for in_place in (False, True):
        got, a, b = _reorth(mc, torch.from_numpy(V).cuda(), torch.from_numpy(w).cuda(), K, n, ldv,
                            in_place)
        assert abs(a - alpha) <= 1e-12
        assert abs(b - beta) <= 1e-12
        if n > K:   # otherwise nothing is left but rounding
            assert np.max(np.abs(got * b - ref)) <= 1e-12
            assert abs(np.linalg.norm(got) - 1.0) <= 1e-12


def test_zero_vector_and_arguments(mc):
    from paper_2005_13679_amd import _lib as L
    V = torch.zeros((2, 100), dtype=torch.complex128, device="cuda")
    V[0, 0] = V[1, 1] = 1.0
    got, a, b = _reorth(mc, V, torch.zeros(100, dtype=torch.complex128, device="cuda"), 2, 100, 100,
                        False)
    assert a == 0 and b == 0.0 and not got.any()
    with pytest.raises(mc.MCError):      # the output inside the basis
        _reorth(mc, V, V[1], 2, 100, 100, True)
    with pytest.raises(mc.MCError):      # rows closer than their length
        _reorth(mc, V, torch.ones(100, dtype=torch.complex128, device="cuda"), 2, 100, 99, False)
