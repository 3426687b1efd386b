"""The tridiagonal eigenpairs over the range of the numbers: matrices scaled close to
its ends, zero matrices, blocks of very different size coupled to nothing."""
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


def _solve(d, e):
    import torch
    import paper_2002_10991_amd as T
    w, Z = T.tridiagonal_eigh(torch.from_numpy(d).to("cuda"), torch.from_numpy(e).to("cuda"), len(d))
    torch.cuda.synchronize()
    return w.cpu().numpy(), Z.cpu().numpy()


def test_zero_matrix():
    for n in (2, 8, 9, 40):
        w, Z = _solve(np.zeros(n), np.zeros(n - 1))
        assert np.all(w == 0.0)
        assert np.linalg.norm(Z.T @ Z - np.eye(n)) <= 1e-12 * n


def test_uncoupled_small_entries():
    """A zero off-diagonal couples nothing: each block's eigenvalues to the accuracy
    of the block's own size."""
    w, _ = _solve(np.array([1e-25, 1.0, 3e-25]), np.zeros(2))
    assert np.allclose(w, [1e-25, 3e-25, 1.0], rtol=1e-14, atol=0.0)
    rng = np.random.default_rng(8)
    for m, size in ((5, 1e-30), (20, 1e-30), (20, 1e-100), (33, 1e-18)):
        d1, e1, d2, e2 = (rng.standard_normal(k) for k in (m, m - 1, m, m - 1))
        w, _ = _solve(np.concatenate([size * d1, d2]), np.concatenate([size * e1, [0.0], e2]))
        T1, T2 = (np.linalg.eigvalsh(np.diag(d) + np.diag(e, 1) + np.diag(e, -1))
                  for d, e in ((d1, e1), (d2, e2)))
        small = np.sort(np.argsort(np.abs(w))[:m])
        assert np.max(np.abs(w[small] / size - T1)) <= 1e-13 * 4 * np.max(np.abs(T1))
        assert np.max(np.abs(np.delete(w, small) - T2)) <= 1e-13 * 4 * np.max(np.abs(T2))


@pytest.mark.parametrize("bad", [np.nan, np.inf, -np.inf])
def test_not_finite_ends(bad):
    """Input that has no eigenpairs: the call returns, and says so in its numbers."""
    rng = np.random.default_rng(4)
    for where in ("d", "e", "all"):
        d, e = rng.standard_normal(70), rng.standard_normal(69)
        if where == "d":
            d[11] = bad
        elif where == "e":
            e[40] = bad
        else:
            d[:], e[:] = bad, bad
        print(f"[gpu] tridiag {bad} in {where}", flush=True)
        w, Z = _solve(d, e)
        assert not (np.all(np.isfinite(w)) and np.all(np.isfinite(Z)))
