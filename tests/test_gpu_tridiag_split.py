"""The tridiagonal eigenpairs of matrices that nearly fall apart: couplings from
below rounding down to subnormal numbers, diagonals that repeat, eigenvalues that
agree to rounding, entries over forty orders of magnitude.  The vectors of
eigenvalues closer than 1e-6 ||T|| are orthonormalised together, so they have to
come out of the inverse iteration independent of each other."""
import numpy as np
import pytest

from conftest import gpu_available
from test_gpu_tridiag_edges import _check   # the bounds of the parity tests of this step

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


def test_pairs_barely_coupled():
    for n in (7, 64, 65):
        e = np.where(np.arange(n - 1) % 2 == 0, 1.0, 1e-20)
        _check(np.zeros(n), e, n, "1, 1e-20 in turn")
        _check(np.full(n, -1.5), e, n, "1, 1e-20 in turn, diagonal -1.5")


@pytest.mark.parametrize("seed", range(6))
def test_identity_plus_rank_three(seed):
    """An ordinary input: A = I + U U^T reduced to tridiagonal form, eigenvalue 1
    (n - 3)-fold up to rounding."""
    import scipy.linalg as sl
    rng = np.random.default_rng(seed)
    n = 100
    U = rng.standard_normal((n, 3))
    H = sl.hessenberg(np.eye(n) + U @ U.T)
    _check(np.diag(H).copy(), np.diag(H, -1).copy(), n, "I + U U^T")
    H = sl.hessenberg(U @ U.T)
    _check(np.diag(H).copy(), np.diag(H, -1).copy(), n, "U U^T")


@pytest.mark.parametrize("c", [1e-17, 1e-18, 1e-60, 1e-100, 1e-160, 1e-200, 1e-310])
def test_equal_diagonals(c):
    _check(np.ones(12), np.full(11, c), 12, f"equal diagonals, coupling {c}")
    d = np.concatenate([np.full(20, 1.0), np.full(20, -1.0)])
    _check(d, np.where(np.arange(39) == 19, c, 0.0), 40, f"two flat blocks, coupling {c}")


@pytest.mark.parametrize("c", [1e-18, 1e-60, 1e-200])
def test_repeated_diagonals(c):
    for seed in range(3):
        rng = np.random.default_rng(seed)
        n = int(rng.integers(10, 101))
        _check(rng.integers(-2, 3, n).astype(float), np.full(n - 1, c), n, f"-2 .. 2, coupling {c}")


@pytest.mark.parametrize("seed", range(8))
def test_entries_over_many_orders(seed):
    rng = np.random.default_rng(seed)
    n = 90
    _check(10.0 ** rng.uniform(-40, 0, n) * rng.choice([-1, 1], n), 10.0 ** rng.uniform(-60, 0, n - 1),
           n, "entries 1e-40 .. 1")
    _check(10.0 ** -np.linspace(0, 30, n) * rng.standard_normal(n),
           10.0 ** -np.linspace(1, 31, n - 1) * rng.standard_normal(n - 1), n, "graded")


@pytest.mark.parametrize("seed", range(24))
def test_joined_equal_blocks(seed):
    """Four equal random blocks joined by couplings around rounding."""
    rng = np.random.default_rng(seed)
    m = 25
    d, e = rng.standard_normal(m), rng.standard_normal(m - 1)
    for c in (0.0, 1e-18, 1e-15, 1e-12, 1e-9):
        _check(np.tile(d, 4), np.concatenate([e, [c], e, [c], e, [c], e]), 4 * m, f"blocks, {c}")
