"""The tridiagonal eigenpairs at the sizes where the kernels can go wrong:
orders around the chunks of the Sturm count (8) and of the substitutions (16, two
to a word of pivoting bits), eigenpair counts around the lanes per eigenvalue, and
matrices scaled far from 1 (the kernels work on a scaled copy), with zero
off-diagonals or with all entries equal."""
import numpy as np
import pytest

from conftest import gpu_available

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


def _check(d, e, nev, label):
    import torch
    import paper_2002_10991_amd as T
    n = len(d)
    print(f"[gpu] tridiag edges n={n} nev={nev} {label}", flush=True)
    w, Z = T.tridiagonal_eigh(torch.from_numpy(d).to("cuda"), torch.from_numpy(e).to("cuda"), nev)
    torch.cuda.synchronize()
    w, Z = w.cpu().numpy(), Z.cpu().numpy()
    a = np.abs(np.concatenate([e, [0.0]])) + np.abs(np.concatenate([[0.0], e]))
    tn = np.max(np.abs(d) + a)
    ref = np.linalg.eigvalsh(np.diag(d / tn) + np.diag(e / tn, 1) + np.diag(e / tn, -1))[:nev]
    # the bounds of the parity tests of this step: 1e-13 ||T||, 1e-12 n
    assert np.max(np.abs(w / tn - ref)) <= 1e-13
    R = (d[:, None] * Z - Z * w) / tn
    R[:-1] += e[:, None] / tn * Z[1:]
    R[1:] += e[:, None] / tn * Z[:-1]
    assert np.max(np.linalg.norm(R, axis=0)) <= 1e-13 * max(1.0, np.sqrt(n) / 10)
    assert np.linalg.norm(Z.T @ Z - np.eye(nev)) <= 1e-12 * n


@pytest.mark.parametrize("n,nev", [(1, 1), (2, 2), (3, 3), (8, 5), (9, 9), (10, 10), (15, 3), (16, 16),
                                   (17, 17), (18, 2), (31, 31), (32, 32), (33, 33), (34, 9), (49, 48),
                                   (65, 65), (512, 512), (513, 513), (2049, 2049)])
def test_tridiag_chunk_edges(n, nev):
    rng = np.random.default_rng(n)
    _check(rng.standard_normal(n), rng.standard_normal(n - 1), nev, "random")


@pytest.mark.parametrize("scale", [1e-150, 1e-20, 1.0, 1e150])
def test_tridiag_scaled(scale):
    rng = np.random.default_rng(5)
    _check(scale * rng.standard_normal(100), scale * rng.standard_normal(99), 100, f"scale {scale}")


def test_tridiag_split_and_flat():
    rng = np.random.default_rng(6)
    d, e = rng.standard_normal(100), rng.standard_normal(99)
    e[::7] = 0.0                               # blocks of 7 rows
    _check(d, e, 60, "split")
    _check(np.full(40, 2.0), np.zeros(39), 40, "a multiple of the identity")
    d = np.concatenate([np.full(20, 1.0), np.full(20, -1.0)])
    _check(d, np.where(np.arange(39) == 19, 1e-9, 0.0), 40, "two flat blocks, barely coupled")
