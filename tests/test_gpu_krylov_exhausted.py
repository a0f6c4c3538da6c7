"""Time steps in spaces that a few vectors exhaust, with the number of vectors
given: the step ends there, and at most twice the vectors and one more are made.

Tolerance: the state is a sum of 1 to 3 eigenvectors, so the step is a phase on
each; 1e-12 relative as for every product."""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("parts,applies", [(1, 2), (2, 3), (3, 5)])
@pytest.mark.parametrize("k", [8, 30])
def test_exhausted_space_ends_the_step(mc, monkeypatch, parts, applies, k):
    from paper_2005_13679_amd import api
    N, M, dt = 10, 5, 0.01
    e = np.array([0.0, 1.0, 2.5, 4.0, 7.0])
    occ = [[10, 0, 0, 0, 0], [0, 10, 0, 0, 0], [2, 2, 2, 2, 2]][:parts]
    sp = mc.DirectSpace(N, M)
    C = torch.zeros(sp.dim, dtype=torch.complex128, device="cuda")
    ref = np.zeros(sp.dim, dtype=np.complex128)
    for i, n in enumerate(occ):
        C[mc.hash_occ(N, M, n)] = 0.5 + i
        ref[mc.hash_occ(N, M, n)] = (0.5 + i) * np.exp(-1j * dt * np.dot(e, n))
    made = []
    whole = api.apply_H
    monkeypatch.setattr(api, "apply_H", lambda *a, **kw: (made.append(1), whole(*a, **kw))[1])
    st = mc.SILStepper(sp, np.diag(e).astype(complex), np.zeros((M,) * 4, complex), kmax=k)
    out, m, err = st.step(C, dt, k=k)
    assert m == parts and err == 0.0 and len(made) <= applies
    assert np.abs(out.cpu().numpy() - ref).max() <= 1e-12 * np.abs(ref).max()
    zero, m, err = st.step(torch.zeros_like(C), dt, k=k)
    assert m == 0 and err == 0.0 and not zero.any()
