"""Every instance of the streaming kernel, at its first and last band width, with more
slots than a workgroup has waves: the forward form, the one that stores the adjoint's
checkpoints (real), and all of them in one plan."""
import numpy as np
import pytest

from conftest import gpu_available
from test_gpu_stream import TOL, test_stream_parity as _parity
from test_gpu_adjoint import _inputs, _relerr, gpu_adjoint

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


def _class(nbw):
    """The instance a band width takes (stream_class in trbt_stream.hip)."""
    if nbw < 40:
        return 2 * (nbw // 4) + (nbw % 4 >= 2)
    if nbw < 72:
        return 20 + (nbw - 40) // 8
    return 24 if nbw < 100 else 25 if nbw < 132 else 26 if nbw < 196 else 27


def _widths():
    first, last = {}, {}
    for nbw in range(2, 257):
        if nbw % 16 or nbw > 128:          # the others take the blocked kernels
            first.setdefault(_class(nbw), nbw)
            last[_class(nbw)] = nbw
    return sorted(set(first.values())), sorted(set(first.values()) | set(last.values()))


FIRST, ENDS = _widths()


def _order(nbw):
    """More slots than waves: 16 waves at most up to nbw = 48, 8 up to 116, else 4."""
    return nbw * (17 if nbw <= 48 else 9 if nbw <= 116 else 5) + 6


@pytest.mark.parametrize("dtype", ["d", "z"])
@pytest.mark.parametrize("nbw", ENDS)
def test_stream_widths(oracle_mod, dtype, nbw):
    _parity(oracle_mod, dtype, _order(nbw), nbw, 17)


@pytest.mark.parametrize("nbw", FIRST)
def test_stream_checkpoints(oracle_mod, nbw):
    n, nev = nbw * (17 if nbw <= 12 else 4) + 6, 18
    Z, G, V, tau = _inputs(n, nbw, nev, 300 + nbw)
    rZ, rv, rt = oracle_mod.adjoint(Z, G, V, tau, nbw)
    gb, zb, dv, dt = gpu_adjoint(Z, G, V, tau, nbw)
    assert _relerr(gb[:nev, :n].T, rZ) <= TOL
    assert _relerr(dv, rv) <= TOL
    assert _relerr(dt, rt) <= TOL


@pytest.mark.parametrize("dtype", ["d", "z"])
def test_stream_widths_in_one_plan(dtype):
    """The kernel and the operations of a single call: bitwise the same."""
    import torch
    import paper_2002_10991_amd as T
    import synth
    print(f"[gpu] stream widths in one plan {dtype}", flush=True)
    probs, want = [], []
    for i, nbw in enumerate(ENDS[::-1]):
        n, nev = 3 * nbw + 40, 1 + i % 35
        V, tau = (torch.from_numpy(x).to("cuda") for x in
                  synth.unitary_reflectors(synth.reflector_lengths(n, nbw), nbw, n, dtype))
        Z = torch.from_numpy(synth.gaussian(n, nev, n, dtype).T.copy()).to("cuda")
        want.append(T.back_transform(Z.clone().T, V, tau, nbw))
        probs.append((Z.T, V, tau, nbw))
    plan = T.BatchedPlan(probs)
    plan.run()
    torch.cuda.synchronize()
    for p, y in zip(probs, want):
        assert torch.equal(p[0], y), p[3]
