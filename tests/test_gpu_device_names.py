"""is_hermitian takes its device as torch does: an object, a name or a number."""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("device", [torch.device("cuda", 0), torch.device("cuda"), "cuda", "cuda:0", 0])
def test_is_hermitian_takes_every_form_of_device(mc, device):
    M = 4
    rng = np.random.default_rng(1)
    h = rng.standard_normal((M, M)) + 1j * rng.standard_normal((M, M))
    g = np.zeros((M,) * 4, dtype=np.complex128)
    assert not mc.is_hermitian(h, g, M, device)
    assert mc.is_hermitian(torch.from_numpy(h + h.conj().T).cuda(), g, M, device)
