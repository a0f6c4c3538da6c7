"""The single-precision estimate by which the kernels invert G_m(s) = C(s+m,
m+1): the root of J (m+1)! less m/2 is within one of the largest s with
G_m(s) <= J, for every m <= 6 and every s that D < 2^31 allows, with 3e-6 of
relative error in the root to spare (CPU)."""

import math

import numpy as np
import pytest


@pytest.mark.parametrize("m", [1, 2, 3, 4, 5, 6])
def test_estimate_is_within_one(m):
    G, s = [], 0
    while math.comb(s + m, m + 1) < 2 ** 31 and s <= 65536:
        G.append(math.comb(s + m, m + 1))
        s += 1
    G = np.array(G, dtype=np.float64)
    s = np.arange(G.size - 1)
    # the first and the last J of every s
    for J in (G[:-1], G[1:] - 1.0):
        lim = (J * math.factorial(m + 1)).astype(np.float32)
        with np.errstate(divide="ignore"):
            root = np.exp2(np.log2(lim) * np.float32(1.0 / (m + 1)))
        for err in (1.0 - 3e-6, 1.0, 1.0 + 3e-6):
            est = np.maximum(np.floor(root * np.float32(err) - np.float32(0.5 * m)), 0.0)
            assert np.max(np.abs(est - s)) <= 1
