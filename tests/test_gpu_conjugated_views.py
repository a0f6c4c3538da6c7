"""h and g given as lazily conjugated or negated views, in their own layout and
transposed, are read with their values."""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def test_views_of_h_and_g_are_read_with_their_values(mc):
    N, M = 6, 4
    rng = np.random.default_rng(2)
    h, g = [torch.from_numpy(rng.standard_normal(s) + 1j * rng.standard_normal(s)).cuda()
            for s in ((M, M), (M,) * 4)]
    C = torch.from_numpy(rng.standard_normal(mc.dim(N, M)) + 0j).cuda()
    sp = mc.DirectSpace(N, M)
    for hv, gv in ((h.conj(), g.conj()), (h.mH, g.permute(3, 2, 1, 0).conj()),
                   (torch._neg_view(h), g)):
        assert hv.is_conj() or hv.is_neg()
        plain = [x.resolve_conj().resolve_neg().contiguous() for x in (hv, gv)]
        assert torch.equal(mc.apply_H(hv, gv, C, sp), mc.apply_H(*plain, C, sp))
        assert mc.is_hermitian(hv, gv, M, C.device) == mc.is_hermitian(*plain, M, C.device)
    s = h + h.mH      # Hermitian, and equal to its conjugate transpose only
    assert mc.is_hermitian(s.conj(), torch.zeros_like(g), M, C.device)
    b = mc.Batch([(sp, h.conj(), g.conj())])
    want = mc.apply_H(h.conj().resolve_conj(), g.conj().resolve_conj(), C, sp)
    assert torch.equal(b.apply_H(C, b.vector()), want)
