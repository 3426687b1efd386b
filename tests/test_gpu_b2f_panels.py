"""The panel kernels of the band-to-full back-transformation at the sizes
where they can go wrong, against the CPU oracle: reflector counts around the 64
and 128 of a panel and its halves, orders and bands around the 16-row blocks,
reflectors too far apart for 32-bit offsets, an order from which workgroups
keep in step, and rows above the reflectors that must take no part."""
import numpy as np
import pytest

from conftest import gpu_available

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

TOL = 1e-12   # the oracle parity bound of this step (relative Frobenius, FP64)


def _run(oracle_mod, n, nbw, nev, dtype, ldv):
    import torch
    import paper_2002_10991_amd as T
    import synth
    print(f"[gpu] b2f panels {dtype} n={n} nbw={nbw} nev={nev} ldv={ldv}", flush=True)
    V, tau = synth.full_unitary_reflectors(n, nbw, n + nbw, dtype)
    J = V.shape[1]
    Z = synth.gaussian(n, nev, n, dtype)
    ref = oracle_mod.back_transform_full(Z, V, tau, nbw)
    Z[:nbw] = np.inf                      # rows no reflector has
    vb = torch.full((J, ldv), float("nan"), dtype=torch.complex128 if dtype == "z" else torch.float64,
                    device="cuda")
    vb[:, :n] = torch.from_numpy(np.ascontiguousarray(V.T)).to("cuda")
    for j in range(min(J, 200)):          # nor its own rows above its start
        vb[j, :j + nbw] = float("nan")
    zb = torch.from_numpy(np.ascontiguousarray(Z.T)).to("cuda")
    T.band_to_full(zb.T, vb.T[:n], torch.from_numpy(tau).to("cuda"), nbw)
    torch.cuda.synchronize()
    out = zb.cpu().numpy().T
    assert np.array_equal(out[:nbw], Z[:nbw])
    assert np.all(np.isfinite(out[nbw:]))
    assert np.linalg.norm(out[nbw:] - ref[nbw:]) <= TOL * np.linalg.norm(ref[nbw:])


@pytest.mark.parametrize("dtype", ["d", "z"])
@pytest.mark.parametrize("n,nbw,nev", [
    (18, 16, 2), (33, 16, 16), (48, 15, 17), (49, 16, 33), (81, 16, 16), (82, 17, 1), (96, 31, 15),
    (145, 16, 18), (146, 17, 16), (209, 16, 40), (210, 1, 16), (273, 16, 16), (274, 17, 31),
    (400, 15, 16), (529, 16, 16), (641, 100, 48)])
def test_b2f_panel_edges(oracle_mod, dtype, n, nbw, nev):
    _run(oracle_mod, n, nbw, nev, dtype, n + (n & 1))


@pytest.mark.parametrize("dtype", ["d", "z"])
def test_b2f_wide_leading_dimension(oracle_mod, dtype):
    _run(oracle_mod, 150, 4, 20, dtype, 1050000)


def test_b2f_workgroups_in_step(oracle_mod):
    _run(oracle_mod, 6200, 6000, 200, "z", 6200)
