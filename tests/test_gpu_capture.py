"""The calls in a captured graph: every replay, with other work and
synchronisations between them, gives the eager call's result bitwise.  Among them the
launches that run as cooperative kernels: slot groups of one strip, and the last pass
of more strips than CUs."""
import pytest

from conftest import gpu_available

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

FORWARD = [
    # (n, nbw, nev, dtype): on 256 CUs
    (900, 64, 815, "z"),      # 51 strips in 4 groups each
    (1100, 32, 300, "d"),     # 19 strips in 5 groups
    (2300, 16, 2100, "d"),    # 132 strips: 128 in two groups, then 4 in eight
    (4300, 64, 4200, "d"),    # 263 strips: a whole pass, then 7 in eight groups
    (4200, 32, 4100, "z"),    # 257 strips: a whole pass, then one
    (333, 55, 190, "d"),      # streaming
    (334, 21, 100, "z"),
]


def _replays(run, inputs, outputs):
    """Capture run(), which reads (and may overwrite) the tensors `inputs`, and compare
    its outputs of three replays with those of an eager call."""
    import torch
    saved = [x.clone() for x in inputs]
    run()                              # (loads kernels, looks attributes up)
    torch.cuda.synchronize()

    def restore():
        for x, s in zip(inputs, saved):
            x.copy_(s)

    restore()
    run()
    torch.cuda.synchronize()
    want = [x.clone() for x in outputs()]
    restore()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        run()
    for _ in range(3):
        restore()
        for x in outputs():
            if not any(x is y for y in inputs):
                x.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(want, outputs()))
        (saved[0] * 2).sum().item()    # the program's own work in between
    del g


@pytest.mark.parametrize("n,nbw,nev,dtype", FORWARD)
def test_capture_forward(n, nbw, nev, dtype):
    import torch
    import paper_2002_10991_amd as T
    import synth
    print(f"[gpu] capture forward {dtype} n={n} nbw={nbw} nev={nev}", flush=True)
    V, tau = (torch.from_numpy(x).to("cuda") for x in
              synth.unitary_reflectors(synth.reflector_lengths(n, nbw), nbw, n, dtype))
    Z = torch.from_numpy(synth.gaussian(n, nev, n, dtype).T.copy()).to("cuda").T
    work = T.alloc_workspace(n, nbw, nev, dtype == "z")
    _replays(lambda: T.back_transform(Z, V, tau, nbw, work=work), [Z], lambda: [Z])
    if work is not None:
        assert T.trbt_work_check(work) == 0


@pytest.mark.parametrize("n,nbw,dtype", [(600, 32, "d"), (300, 17, "z")])
def test_capture_chase(n, nbw, dtype):
    import torch
    import paper_2002_10991_amd as T
    import synth
    print(f"[gpu] capture chase {dtype} n={n} nbw={nbw}", flush=True)
    ab = torch.from_numpy(synth.band_matrix(n, nbw, 9, dtype).T.copy()).to("cuda")
    work = torch.empty(T.trbt_band_to_tridi_workspace_bytes(n, nbw, dtype == "z") + 256,
                       dtype=torch.uint8, device="cuda")
    work = work[-work.data_ptr() % 256:]
    out = []

    def run():
        out[:] = T.band_to_tridiagonal(ab, nbw, work=work)
    _replays(run, [ab], lambda: out)


def test_capture_tridiagonal():
    import torch
    import paper_2002_10991_amd as T
    print("[gpu] capture tridiagonal", flush=True)
    g = torch.Generator().manual_seed(3)
    d, e = (torch.randn(k, generator=g, dtype=torch.float64).to("cuda") for k in (700, 699))
    e[350] = 0.0
    d[351:] = d[:349].clone()          # some clusters
    e[351:] = e[:348].clone()
    out = []

    def run():
        out[:] = T.tridiagonal_eigh(d, e, 500)
    _replays(run, [d, e], lambda: out)


@pytest.mark.parametrize("n,nbw,nev,dtype", [(700, 32, 300, "d"), (6200, 64, 400, "z")])
def test_capture_band_to_full(n, nbw, nev, dtype):
    import torch
    import paper_2002_10991_amd as T
    print(f"[gpu] capture band to full {dtype} n={n} nbw={nbw} nev={nev}", flush=True)
    dt = torch.complex128 if dtype == "z" else torch.float64
    g = torch.Generator(device="cuda").manual_seed(4)
    J = n - nbw - 1
    V = torch.randn(J, n, generator=g, dtype=dt, device="cuda").T / n ** 0.5
    tau = torch.full((J,), 0.5, dtype=dt, device="cuda")
    Z = torch.randn(nev, n, generator=g, dtype=dt, device="cuda").T
    work = torch.empty(T.trbt_band_to_full_workspace_bytes(n, nbw, nev, dtype == "z") + 256,
                       dtype=torch.uint8, device="cuda")
    work = work[-work.data_ptr() % 256:]
    _replays(lambda: T.band_to_full(Z, V, tau, nbw, work=work), [Z], lambda: [Z])
