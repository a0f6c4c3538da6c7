"""Groups of many small instances, whose tiles a wavefront each takes while it
keeps the sums that the wavefronts of a block have otherwise: on both sides of
the line, in every kind and work order, beside a joint launch, each segment has
the bits of the instance alone."""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

KINDS = [("direct", False), ("reduced", True), ("reduced", False), ("paper", True), ("paper", False)]


# tiles on both sides of the lines: 664, 830, 1,494 and 1,660 at M = 5, 728, 910,
# 1,274 and 1,456 at M = 6, 1,260 and 1,386 at M = 7, 1,212 and 1,313 at M = 8, and 2,060
# of instances of 120 rows; each beside small groups of M = 3 and 4
@pytest.mark.parametrize("N,M,counts", [(20, 5, (4, 5, 9, 10)), (14, 6, (4, 5, 7, 8)),
                                        (10, 7, (10, 11)), (8, 8, (12, 13)), (3, 8, (1030,))])
@pytest.mark.parametrize("form,maps", KINDS)
def test_bits_of_the_instance_alone(mc, N, M, counts, form, maps):
    def space(n, m):
        return mc.DirectSpace(n, m) if form == "direct" else \
            mc.build_tables(n, m, form=form, double_jumps=maps)
    rng = np.random.default_rng(N + M)

    def ops(m):
        return [torch.from_numpy(rng.standard_normal(s) + 1j * rng.standard_normal(s)).cuda()
                for s in ((m, m), (m,) * 4)]
    sp, other = space(N, M), [space(9, 4), space(12, 3)]
    variants, side = [ops(M) for _ in range(3)], [ops(4), ops(3)]
    for count in counts:
        items = [(sp, *variants[i % 3]) for i in range(count)]
        items[1:1] = [(s, *o) for s, o in zip(other, side)]
        C = None
        for order in (0, 1, 2, 3):
            b = mc.Batch(items, {"order": order})
            if C is None:
                C, out = b.vector(), b.vector()
                torch.view_as_real(C).normal_()
                alone = [mc.apply_H(h, g, b.segment(C, i).contiguous(), s)
                         for i, (s, h, g) in enumerate(items)]
                alone = torch.cat(alone)
            out.fill_(complex(float("nan"), 0.0))
            b.apply_H(C, out)
            assert torch.equal(out, alone), (count, order)
