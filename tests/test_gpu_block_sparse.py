"""H.C over non-zero constants only, with four rows per lane (spaces of at least
131,072 rows): one constant at a time, a dense, a holed
and a momentum-conserving interaction against the oracle, and a value that is
not finite where no constant couples it.

Tolerance: 1e-12 relative to the largest element, the bar of every apply."""

import numpy as np
import pytest
import torch

from tests.gpu_helpers import rel_inf

pytestmark = pytest.mark.gpu

TOL = 1e-12
SIZES = [(513, 3), (92, 4), (41, 5), (26, 6), (18, 7), (19, 7), (15, 8), (20, 8)]


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def check(mc, oracle, N, M, h, g, C, rows, tab):
    got = mc.apply_H_sparse(dev(h), dev(g), dev(C), tab)
    got = got[torch.from_numpy(rows).cuda()].cpu().numpy()
    ref = oracle.apply_h(N, M, h, g, C, rows)
    assert rel_inf(got, ref) <= TOL if np.abs(ref).max() > 0 else np.abs(got).max() == 0


@pytest.mark.parametrize("N,M", SIZES)
def test_interactions_match_oracle(mc, oracle_native, N, M):
    rng = np.random.default_rng(N + M)
    D = oracle_native.dim(N, M)
    C = rng.standard_normal(D) + 1j * rng.standard_normal(D)
    rows = np.unique(np.concatenate([rng.integers(0, D, 1000), np.arange(64),
                                     D - 1 - np.arange(64)]))
    tab = mc.build_tables(N, M, form="reduced", double_jumps=False)
    q = np.arange(M)
    ring = q[:, None, None, None] + q[:, None, None] == q[:, None] + q   # momentum conserved
    check(mc, oracle_native, N, M, np.diag((q - 1.0) ** 2).astype(complex), 10.0 * ring + 0j, C,
          rows, tab)
    for holes in (0.0, 0.5, 0.98):
        h = rng.standard_normal((M, M)) + 1j * rng.standard_normal((M, M))
        g = rng.standard_normal((M,) * 4) + 1j * rng.standard_normal((M,) * 4)
        g[rng.random(g.shape) < holes] = 0.0
        h[rng.random(h.shape) < holes] = 0.0
        check(mc, oracle_native, N, M, h, g, C, rows, tab)
    check(mc, oracle_native, N, M, 0 * h, 0 * g, C, rows, tab)
    check(mc, oracle_native, N, M, h.conj().T, np.zeros_like(g), C, rows, tab)


@pytest.mark.parametrize("N,M", [(513, 3), (92, 4), (41, 5), (20, 8)])
def test_one_constant_at_a_time(mc, oracle_native, N, M):
    rng = np.random.default_rng(N * M)
    D = oracle_native.dim(N, M)
    C = rng.standard_normal(D) + 1j * rng.standard_normal(D)
    rows = np.unique(np.concatenate([rng.integers(0, D, 200), [0, D - 1]]))
    tab = mc.build_tables(N, M, form="reduced", double_jumps=False)
    one = [(a, b) for a in range(M) for b in range(M)]
    two = [tuple(q) for q in np.ndindex((M,) * 4)]
    if M > 4:
        two = [two[i] for i in rng.permutation(len(two))[:150]]
    for at in one + two:
        h, g = np.zeros((M, M), complex), np.zeros((M,) * 4, complex)
        (h if len(at) == 2 else g)[at] = 0.7 - 0.3j
        check(mc, oracle_native, N, M, h, g, C, rows, tab)


@pytest.mark.parametrize("N,M", [(92, 4), (41, 5)])
def test_a_value_that_nothing_couples_stays_where_it_is(mc, N, M):
    C = torch.ones(mc.dim(N, M), dtype=torch.complex128, device="cuda")
    k = 12345
    C[k] = complex(float("inf"), 0.0)
    tab = mc.build_tables(N, M, form="reduced", double_jumps=False)
    out = mc.apply_H_sparse(dev(np.eye(M, dtype=complex)), dev(np.zeros((M,) * 4, complex)), C, tab)
    bad = torch.nonzero(~torch.isfinite(out.real) | ~torch.isfinite(out.imag)).flatten()
    assert bad.tolist() == [k]
