"""Table-free H.C with four rows per lane (spaces of at least 262,144 rows,
131,072 for 7 orbitals, 786,432 for 8): against the oracle at the smallest
spaces it serves, every remainder of N by 4, each orbital count, with general
inputs and the adjoint; and which rows a value that is not finite reaches.

Tolerance: 1e-12 relative to the largest element, the bar of every apply (a
row sums at most 869 products of size max|H.C| or less in double)."""

import itertools

import numpy as np
import pytest
import torch

import workloads as W
from tests.gpu_helpers import rel_inf

pytestmark = pytest.mark.gpu

TOL = 1e-12
# the smallest N served per M, its neighbours below (one row per lane) and above
SIZES = [(510, 3), (511, 3), (513, 3), (90, 4), (91, 4), (92, 4), (39, 5), (40, 5), (41, 5),
         (42, 5), (43, 5), (24, 6), (25, 6), (26, 6), (17, 7), (18, 7), (19, 8), (20, 8),
         (722, 3), (723, 3), (725, 3), (114, 4), (115, 4), (116, 4), (47, 5), (48, 5), (49, 5),
         (50, 5), (51, 5), (28, 6), (29, 6), (30, 6)]


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def general(N, M, D):
    """h, g of no symmetry, C not normalised."""
    rng = np.random.default_rng(100 * N + M)
    h = rng.standard_normal((M, M)) + 1j * rng.standard_normal((M, M))
    g = rng.standard_normal((M,) * 4) + 1j * rng.standard_normal((M,) * 4)
    return h, g, rng.standard_normal(D) + 1j * rng.standard_normal(D), rng


@pytest.mark.parametrize("N,M", SIZES)
def test_apply_and_adjoint_match_oracle(mc, oracle_native, N, M):
    D = oracle_native.dim(N, M)
    h, g, C, rng = general(N, M, D)
    rows = np.unique(np.concatenate([rng.integers(0, D, 3000), np.arange(200),
                                     D - 1 - np.arange(200)]))
    r = torch.from_numpy(rows).cuda()
    got = mc.apply_H_direct(dev(h), dev(g), dev(C), N, M)[r].cpu().numpy()
    assert rel_inf(got, oracle_native.apply_h(N, M, h, g, C, rows)) <= TOL
    adj = mc.apply_H_adjoint(dev(h), dev(g), dev(C), mc.DirectSpace(N, M))[r].cpu().numpy()
    ref = oracle_native.apply_h(N, M, h.conj().T, np.transpose(g, (3, 2, 1, 0)).conj(), C, rows)
    assert rel_inf(adj, ref) <= TOL


def coupled(mc, N, M, k):
    """Rows that H couples to row k: at most two particles moved."""
    n = mc.unhash(N, M, k)
    seen = {tuple(n)}
    for _ in range(2):
        for o in list(seen):
            for a, b in itertools.permutations(range(M), 2):
                if o[a] > 0:
                    t = list(o)
                    t[a] -= 1
                    t[b] += 1
                    seen.add(tuple(t))
    return sorted(mc.hash_occ(N, M, o) for o in seen)


@pytest.mark.parametrize("N,M", [(511, 3), (91, 4), (41, 5), (25, 6), (18, 7), (20, 8), (723, 3),
                                 (116, 4), (49, 5), (30, 6)])
def test_values_that_are_not_finite_stay_with_coupled_rows(mc, N, M):
    D = mc.dim(N, M)
    h, g, C, rng = general(N, M, D)
    sp, hd, gd = mc.DirectSpace(N, M), dev(h), dev(g)
    for k in [0, 1, D - 1, D - 2, *rng.integers(0, D, 4)]:
        Cd = dev(C)
        Cd[int(k)] = complex(float("nan"), float("inf"))
        out = mc.apply_H(hd, gd, Cd, sp)
        bad = (~torch.isfinite(torch.view_as_real(out)).all(dim=1)).nonzero().flatten().tolist()
        assert bad == coupled(mc, N, M, int(k)), (N, M, int(k))
