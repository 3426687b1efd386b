"""The tridiagonal eigenpairs over the range of the numbers: matrices scaled close to
its ends."""
import numpy as np
import pytest

from conftest import gpu_available
from test_gpu_tridiag_edges import _check   # the bounds of the parity tests of this step

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


@pytest.mark.parametrize("scale", [1e-300, 1e-295, 1e-280, 1e155, 1e160, 1e300])
def test_scaled_far(scale):
    rng = np.random.default_rng(5)
    _check(scale * rng.standard_normal(100), scale * rng.standard_normal(99), 100, f"scale {scale}")
