"""The passes of the blocked back-transformation over the CUs: whole passes of
column strips, a rest in slot groups, a rest split in two, and one or two
column tiles per wave.  A column's result does not depend on the strip, the
pass or the tiling it falls in (the same operations in the same order), so
the whole call equals, bitwise, calls on slices of its columns."""
import pytest

from conftest import gpu_available

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

SHAPES = [
    # (n, nbw, nev, dtype): on 256 CUs
    (2300, 16, 2100, "d"),    # 132 strips: 128 in two groups, then 4 in eight
    (3000, 16, 2990, "d"),    # two column tiles per wave, a ragged last strip
    (4300, 64, 4200, "d"),    # 263 strips: a whole pass, then 7 in eight groups
    (4300, 128, 4111, "d"),   # the same with 4 waves per workgroup
    (4200, 32, 4100, "z"),    # 257 strips: a whole pass, then one
    (900, 64, 815, "z"),      # 51 strips: 5 groups each would not fit once padded
]


@pytest.mark.parametrize("n,nbw,nev,dtype", SHAPES)
def test_passes_equal_slices(n, nbw, nev, dtype):
    import torch
    import paper_2002_10991_amd as T
    import synth
    print(f"[gpu] passes {dtype} n={n} nbw={nbw} nev={nev}", flush=True)
    V, tau = synth.unitary_reflectors(synth.reflector_lengths(n, nbw), nbw, n, dtype)
    Vd, td = torch.from_numpy(V).to("cuda"), torch.from_numpy(tau).to("cuda")
    ldz = n + 5
    Z = torch.from_numpy(synth.gaussian(ldz, nev, n, dtype).T.copy()).to("cuda")
    whole = Z.clone()
    T.back_transform(whole.T[:n], Vd, td, nbw)
    assert torch.equal(whole[:, n:], Z[:, n:])
    nz, no = (torch.linalg.norm(x[:, :n], dim=1) for x in (Z, whole))
    assert float(torch.max(torch.abs(no / nz - 1))) <= 1e-12      # unitary
    for c in sorted({0, 16, nev // 2, 2047, 2048 + 31, 4095, nev - 37}):
        if c + 37 > nev:
            continue
        part = Z[c:c + 37].clone()
        T.back_transform(part.T[:n], Vd, td, nbw)
        assert torch.equal(part, whole[c:c + 37]), c
