"""Short Iterative Lanczos (SIL) time steps C(t + dt) = exp(-i H dt) C(t).

Sec. II names the SIL integrator as the time-dependent use of repeated H.C
(Park and Light's method): a Krylov basis V_k = [v_0, ..., v_{k-1}] of
(H, C/|C|) is built by Lanczos with full reorthogonalisation, the projected
tridiagonal T_k gives y = exp(-i T_k dt) e_0, and C(t + dt) ~ |C| V_k y.
The basis grows until the a-posteriori error estimate
|C| beta_k |y_{k-1}| (the weight the next Krylov vector would receive) falls
below ``tol`` or ``kmax`` is reached.

Every vector operation runs in the library's kernels (mc_apply_H,
mc_lanczos_reorth, mc_normalize, mc_zgemv_n); the k x k exponential, the
scaling by |C| and the error estimate are the library's host routine
mc_sil_coefficients.  alpha and beta are read back after each Lanczos step
for the stopping test, and where the number of vectors is given after 1, 2, 4,
... of them, to end the step where they exhaust the space.
"""

from __future__ import annotations

import ctypes

import numpy as np
import torch

from . import _lib as L
from . import api


def tridiag_expv(alphas, betas, dt: float) -> np.ndarray:
    """exp(-i T dt) e_0 for the symmetric tridiagonal T (host)."""
    a = np.ascontiguousarray(alphas, dtype=np.float64)
    b = np.ascontiguousarray(betas, dtype=np.float64)
    if b.size < max(0, a.size - 1):
        raise ValueError("need K-1 off-diagonal entries")
    y = np.empty(2 * a.size, dtype=np.float64)
    L.check(L.load().mc_tridiag_expv(a.size, a.ctypes.data_as(ctypes.c_void_p),
                                     b.ctypes.data_as(ctypes.c_void_p), float(dt),
                                     y.ctypes.data_as(ctypes.c_void_p)), "mc_tridiag_expv")
    return y[0::2] + 1j * y[1::2]


def sil_coefficients(alphas, betas, beta_next: float, norm_c: float, dt: float):
    """(coefficients |C| exp(-i T dt) e_0 as complex128, error estimate,
    invariant-space flag) from the library (host routine)."""
    a = np.ascontiguousarray(alphas, dtype=np.float64)
    b = np.ascontiguousarray(betas, dtype=np.float64)
    if b.size < max(0, a.size - 1):
        raise ValueError("need K-1 off-diagonal entries")
    coef = np.empty(2 * a.size, dtype=np.float64)
    err = ctypes.c_double()
    inv = ctypes.c_int32()
    L.check(L.load().mc_sil_coefficients(a.size, a.ctypes.data_as(ctypes.c_void_p),
                                         b.ctypes.data_as(ctypes.c_void_p), float(beta_next),
                                         float(norm_c), float(dt),
                                         coef.ctypes.data_as(ctypes.c_void_p), ctypes.byref(err),
                                         ctypes.byref(inv)), "mc_sil_coefficients")
    return coef.view(np.complex128), float(err.value), bool(inv.value)


class SILStepper:
    """Reusable SIL stepper for one (tables, h, g): Krylov storage for up to
    ``kmax`` vectors is allocated once."""

    def __init__(self, tables, h, g, kmax: int = 30):
        self.t = tables
        self.dev, self.D, self.M = tables.device, tables.dim, tables.M
        self.kmax = int(max(1, min(kmax, self.D)))
        M = self.M
        self.h = api._as_dev(h, self.dev, (M, M))
        self.g = api._as_dev(g, self.dev, (M, M, M, M))
        D, k = self.D, self.kmax
        self.V = torch.empty((k + 1, D), dtype=torch.complex128, device=self.dev)
        self.w = torch.empty(D, dtype=torch.complex128, device=self.dev)
        # per vector: alpha (complex), beta; the last row: beta = |C|
        self.ab = torch.empty((k + 1, 4), dtype=torch.float64, device=self.dev)
        self.host = torch.empty((k + 1, 4), dtype=torch.float64, pin_memory=True)
        self.copied = torch.cuda.Event()
        self.ws = torch.empty((k + 1) * (L.MC_REORTH_BLOCKS + 2) * 16, dtype=torch.uint8,
                              device=self.dev)

    def step(self, C: torch.Tensor, dt: float, tol: float = 1e-12, out: torch.Tensor | None = None,
             k: int | None = None):
        """Returns (C(t+dt), krylov_dim, error_estimate).  With ``k`` given,
        exactly k Krylov vectors are used (no early stop, unless the space is
        exhausted)."""
        dev, D = self.dev, self.D
        api._require(C, "C", torch.complex128, dev, numel=D)
        if out is None:
            out = torch.empty_like(C)
        api._require(out, "out", torch.complex128, dev, numel=D)
        lib = L.load()
        stream = torch.cuda.current_stream(dev)
        st = stream.cuda_stream
        P = api._ptr
        cap = self.kmax if k is None else int(min(k, self.kmax))
        V, w, ab, ws = self.V, self.w, self.ab, self.ws
        with torch.cuda.device(dev):
            L.check(lib.mc_normalize(D, P(C), P(V[0]), P(ab[self.kmax, 2:]), P(ws), ws.numel(), st),
                    "mc_normalize")
        if (k is None or cap < 1) and float(ab[self.kmax, 2].item()) == 0.0:
            out.copy_(C)
            return out, 0, 0.0
        alphas, betas = [], []
        coef, err, m = None, float("inf"), 0

        def vector(j):
            api.apply_H(self.h, self.g, V[j], self.t, out=w)
            with torch.cuda.device(dev):
                L.check(lib.mc_lanczos_reorth(j + 1, D, P(V), D, P(w), P(V[j + 1]), P(ab[j]),
                                              P(ab[j, 2:]), P(ws), ws.numel(), st),
                        "mc_lanczos_reorth")

        made = known = 0    # vectors enqueued, vectors whose scalars are read
        for j in range(cap):
            if j == known:
                # alpha, beta and |C| from the device: after every vector where
                # the stopping test needs them; with k given after 1, 2, 4, ...
                # vectors and with the next one under way, so that the GPU does
                # not wait and an exhausted space ends the step early (a
                # stationary state at N=100, M=5 with k = 8: 0.78 ms, and 3.97
                # where they were read once at the end)
                known = j + 1 if k is None else min(cap, max(1, 2 * known))
                while made < known:
                    vector(made)
                    made += 1
                if k is None:
                    scalars = ab.tolist()
                else:
                    self.host.copy_(ab, non_blocking=True)
                    self.copied.record(stream)
                    if made < cap:
                        vector(made)
                        made += 1
                    self.copied.synchronize()
                    scalars = self.host.tolist()
                norm_c = scalars[self.kmax][2]
                if norm_c == 0.0:
                    out.copy_(C)
                    return out, 0, 0.0
            a, b = scalars[j][0], scalars[j][2]
            alphas.append(a)
            m = j + 1
            coef, err, invariant = sil_coefficients(alphas, betas, b, norm_c, dt)
            if invariant or (k is None and err < tol):
                break
            betas.append(b)
        coef = torch.from_numpy(np.ascontiguousarray(coef)).to(dev)
        with torch.cuda.device(dev):
            L.check(lib.mc_zgemv_n(m, D, P(V), D, P(coef), P(out), st), "mc_zgemv_n")
        return out, m, err


def sil_step(tables, h, g, C: torch.Tensor, dt: float, kmax: int = 30, tol: float = 1e-12,
             k: int | None = None):
    """One SIL step; see SILStepper.step."""
    return SILStepper(tables, h, g, kmax=kmax if k is None else max(kmax, k)).step(C, dt, tol, k=k)
