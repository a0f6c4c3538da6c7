"""Batches in which instances of the four-row kernel (launches of their own)
lie between others of their orbital count: above its upper limit of 2^27 rows,
served by it, and below its lower one.  Each segment has the bits of the
instance alone, in every work order; so do replays of a captured Lanczos graph
against the eager recurrence."""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def instances(mc, shapes):
    items = []
    for i, (N, M) in enumerate(shapes):
        rng = np.random.default_rng(1000 + i)
        h = rng.standard_normal((M, M)) + 1j * rng.standard_normal((M, M))
        g = rng.standard_normal((M,) * 4) + 1j * rng.standard_normal((M,) * 4)
        h, g = h + h.conj().T, g + np.transpose(g, (3, 2, 1, 0)).conj()
        items.append((mc.DirectSpace(N, M), torch.from_numpy(h).cuda(),
                      torch.from_numpy(np.ascontiguousarray(g)).cuda()))
    return items


def fill(x):
    gen = torch.Generator(device="cuda").manual_seed(5)
    torch.view_as_real(x).normal_(generator=gen)
    return x


# 156,340,626, 4,598,126 and 82,251 rows; 154,143,080, 10,295,472 and 346,104;
# three sizes around the lower limits of 5 and of 7 orbitals
@pytest.mark.parametrize("shapes", [[(245, 5), (100, 5), (35, 5)], [(17, 8), (46, 8), (30, 8)],
                                    [(40, 5), (52, 5), (36, 5), (50, 5), (17, 7), (20, 7)]])
def test_every_segment_is_that_of_the_instance_alone(mc, shapes):
    items = instances(mc, shapes)
    C = out = None
    for order in (0, 1, 2, 3):
        b = mc.Batch(items, {"order": order})
        if C is None:
            C, out = fill(b.vector()), b.vector()
        out.fill_(complex(float("nan"), 1.0))     # what nothing writes shows
        b.apply_H(C, out)
        for i, (sp, h, g) in enumerate(items):
            alone = mc.apply_H(h, g, b.segment(C, i).contiguous(), sp)
            assert torch.equal(b.segment(out, i), alone), (shapes[i], order)
            del alone
    del b, C, out
    torch.cuda.empty_cache()


def test_graph_replays_with_four_row_instances(mc):
    items = instances(mc, [(40, 5), (52, 5), (36, 5), (50, 5), (17, 7), (20, 7), (9, 4)])
    b = mc.Batch(items)
    v0 = fill(b.vector())
    a_e, b_e = mc.BatchedLanczos(b, 6, graph=False).run(v0)
    assert np.isfinite(a_e).all() and (b_e > 0).all()
    lz = mc.BatchedLanczos(b, 6, graph=True)
    for rep in range(3):
        # unrelated eager work between replays
        assert np.isfinite(torch.randn(1 << 20, device=b.device).sum().item())
        a_g, b_g = lz.run(v0)
        assert np.array_equal(a_g, a_e) and np.array_equal(b_g, b_e), rep
