"""Rounding of the steps' building blocks: the reciprocal of a density is that
of an FP64 division."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sd():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2007_07347_amd import sdugks
    return sdugks


def test_reciprocal_of_a_density_is_the_divisions(sd):
    """Equal bit by bit to 1 / x: densities spread over (0.5, 2) and over eight
    decades, and the numbers next to powers of two -- 1 / (1 - a 2^-53) for odd a
    lies a^2 2^-54 of an ulp from the middle of two numbers, where an error
    far below an ulp already rounds the wrong way."""
    rng = np.random.default_rng(3)
    a = np.arange(1, 1 << 16)
    near = np.concatenate([1.0 - a * 2.0 ** -53, 1.0 + a * 2.0 ** -52])
    x = np.concatenate([rng.uniform(0.5, 2.0, 1 << 20), 10.0 ** rng.uniform(-4, 4, 1 << 20),
                        *(near * 2.0 ** k for k in (-40, -3, 0, 1, 40))])
    y = sd.debug_reciprocal(x)
    bad = y != 1.0 / x
    assert not bad.any(), (bad.sum(), [float(v).hex() for v in x[bad][:4]])
