"""The streaming kernel's rings, the passes of the blocked forward and the chase's early
publish on the wait-jitter build (see test_gpu_jitter.py): a pseudo-random delay in front
of every wait and publish, results against the oracle and bitwise the release build's."""
import os

import pytest

from conftest import gpu_available
from test_gpu_jitter import _child, _jitter_lib

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

DIGEST = """
import hashlib, numpy as np, torch, synth
import paper_2002_10991_amd as T
h = hashlib.sha256()
for dt, n, nbw, nev in (("z", 700, 20, 40), ("d", 500, 7, 33), ("d", 900, 55, 20), ("z", 640, 130, 18)):
    V, tau = synth.unitary_reflectors(synth.reflector_lengths(n, nbw), nbw, n, dt)
    zb = torch.from_numpy(np.ascontiguousarray(synth.gaussian(n, nev, n + 1, dt).T)).to("cuda")
    T.back_transform(zb.T, torch.from_numpy(V).to("cuda"), torch.from_numpy(tau).to("cuda"), nbw)
    h.update(zb.cpu().numpy().tobytes())
for dt, n, nbw in (("d", 900, 32), ("z", 500, 64), ("d", 300, 5), ("z", 333, 17)):
    ab = torch.from_numpy(np.ascontiguousarray(synth.band_matrix(n, nbw, 5, dt).T)).to("cuda")
    for x in T.band_to_tridiagonal(ab, nbw):
        h.update(x.cpu().numpy().tobytes())
print("DIGEST", h.hexdigest())
"""


@pytest.mark.timeout(600)
def test_stream_passes_and_chase_pass_under_wait_jitter():
    lib = _jitter_lib()
    print("[gpu] streaming / passes / chase tests on the wait-jitter build", flush=True)
    r = _child(["-m", "pytest", "-x", "-q", "-p", "no:cacheprovider", "tests/test_gpu_stream.py",
                "tests/test_gpu_passes.py", "tests/test_gpu_chase.py::test_chase_matches_oracle"], lib)
    assert r.returncode == 0, r.stdout[-4000:] + r.stderr[-4000:]


@pytest.mark.timeout(300)
def test_stream_and_chase_are_bitwise_the_release_result():
    from paper_2002_10991_amd import build
    lib = _jitter_lib()
    digests = []
    for path in (build.OUT, lib):
        print(f"[gpu] output digest with {os.path.basename(path)}", flush=True)
        r = _child(["-c", DIGEST], path)
        assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-4000:]
        digests.append([l for l in r.stdout.splitlines() if l.startswith("DIGEST")][-1])
    assert digests[0] == digests[1]
