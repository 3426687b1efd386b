"""The streaming form of the back-transformation (any nbw, no workspace)
against the CPU oracle at the sizes where it can go wrong: every kernel
instance's first and last band width, orders around a multiple of the 4-row
quads and of the slots in flight, ragged column strips, and entries that must
take no part (reflector entries beyond their length, rows no reflector
touches)."""
import numpy as np
import pytest

from conftest import gpu_available

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

# relative Frobenius: K <= 40 000 reflectors of rounding ~ eps each, adding
# up like a random walk over the <= n that touch one row: 1e-12 is > 10x that
TOL = 1e-12

SHAPES = [
    # (n, nbw, nev)
    (3, 2, 1), (4, 3, 4), (5, 2, 5), (9, 8, 9), (64, 8, 16), (66, 5, 15),
    (67, 6, 17), (200, 2, 33), (201, 3, 1), (202, 4, 18), (300, 7, 40), (303, 9, 48),
    (500, 20, 33), (501, 22, 16), (402, 38, 20), (403, 39, 31), (404, 40, 17), (300, 47, 16),
    (333, 55, 19), (334, 56, 5), (335, 63, 16), (336, 71, 33), (337, 72, 16), (338, 99, 17),
    (339, 100, 16), (340, 131, 9), (341, 132, 17), (450, 195, 16), (451, 196, 7),
    (600, 255, 17), (601, 256, 16), (1201, 20, 40),
]


@pytest.mark.parametrize("dtype", ["d", "z"])
@pytest.mark.parametrize("n,nbw,nev", SHAPES)
def test_stream_parity(oracle_mod, dtype, n, nbw, nev):
    import torch
    import paper_2002_10991_amd as T
    import synth
    print(f"[gpu] stream {dtype} n={n} nbw={nbw} nev={nev}", flush=True)
    assert T.trbt_workspace_bytes(n, nbw, nev, dtype == "z") == 0
    lengths = synth.reflector_lengths(n, nbw)
    V, tau = synth.unitary_reflectors(lengths, nbw, n + nbw, dtype)
    Z = synth.gaussian(n, nev, n, dtype)
    Z[0] = np.inf                      # row 0 meets no reflector
    ref = oracle_mod.back_transform(Z[:, :], V, tau, nbw)
    V[np.arange(nbw)[None, :] >= lengths[:, None]] = np.nan   # beyond the length: not read
    ldz = n + 3
    host = np.full((nev, ldz), 777.0, Z.dtype)
    host[:, :n] = Z.T
    zb = torch.from_numpy(host).to("cuda")
    T.back_transform(zb.T[:n], torch.from_numpy(V).to("cuda"), torch.from_numpy(tau).to("cuda"),
                     nbw)
    torch.cuda.synchronize()
    out = zb.cpu().numpy()
    assert np.all(out[:, n:] == 777.0)
    assert np.array_equal(out[:, 0], host[:, 0])
    got, want = out[:, 1:n].T, ref[1:]
    assert np.all(np.isfinite(got))
    assert np.linalg.norm(got - want) <= TOL * np.linalg.norm(want)
