"""Sparse apply at three orbitals: a row that cannot lose the two particles of
a jump reads nothing through it.  The elements are those that the words before
the space's tables (the last root, that of N + 6) would address from the row
(0, 0, N) if they were taken for an index."""

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,k", [(1334, 220319), (2228, 789839), (4088, 65555)])
def test_impossible_removal_reads_nothing(mc, N, k):
    M = 3
    h = torch.zeros((M, M), dtype=torch.complex128, device="cuda")
    g = torch.zeros((M,) * 4, dtype=torch.complex128, device="cuda")
    g[0, 0, 2, 2] = 1.0
    C = torch.ones(mc.dim(N, M), dtype=torch.complex128, device="cuda")
    C[k] = complex(float("nan"), 0.0)
    out = mc.apply_H_sparse(h, g, C, mc.build_tables(N, M, form="reduced", double_jumps=False))
    bad = (~torch.isfinite(torch.view_as_real(out)).all(dim=1)).nonzero().flatten().tolist()
    # the row itself, and the row with two particles more in orbital 0
    n = mc.unhash(N, M, k)
    rows = {k} | ({mc.hash_occ(N, M, [n[0] + 2, n[1], n[2] - 2])} if n[2] >= 2 else set())
    assert set(bad) <= rows and k in bad, (bad, rows)
