"""Amplitudes of the density matrices are rounded once.  For a single
configuration n with coefficient 1, <a_q+ a_l+ a_l a_q> = n_q (n_l - [q = l])
is the square of one amplitude sqrt(ab).

Tolerance, u = 2^-53: the root is off by at most u, its square by 2u and one
more rounding: 3u to first order, 3.1u with the rest."""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

TOL = 3.1 * 2.0 ** -53


@pytest.mark.parametrize("M", [2, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("space", ["direct", "reduced", "reduced_chained", "paper"])
def test_diagonal_of_one_configuration(mc, M, space):
    N = 11
    tab = mc.DirectSpace(N, M) if space == "direct" else \
        mc.build_tables(N, M, form="paper" if space == "paper" else "reduced",
                        double_jumps=space != "reduced_chained")
    rng = np.random.default_rng(M)
    for _ in range(12):
        n = rng.multinomial(N, np.full(M, 1.0 / M))
        C = torch.zeros(mc.dim(N, M), dtype=torch.complex128, device="cuda")
        C[mc.hash_occ(N, M, n.tolist())] = 1.0
        got = mc.rho2(C, tab).cpu().numpy()
        for q in range(M):
            for l in range(M):
                want = float(n[q] * (n[l] - (q == l)))
                assert abs(got[q, l, q, l] - want) <= TOL * want, (n, q, l)
        one = mc.rho1(C, tab).cpu().numpy()
        assert np.abs(np.diag(one) - n).max() <= TOL * N
