"""Performance cases of the library: what a user's program has it do, through
the public Python functions, over the range of sizes, types and options it is
used with.

Inputs are made on the GPU from the seed alone.  Reflectors have the shape of
bulge-chasing (or full-to-band) output: v[0] = 1, the other entries
N(0, 1/len), tau such that H is unitary.  Z, G: Gaussian.  Tridiagonal
matrices: the T of a dense Gaussian symmetric matrix (Dumitriu-Edelman: N(0, 2)
on the diagonal, chi of n-1 .. 1 degrees of freedom beside it).  Bands:
Gaussian.

A case is a dict: "op" and its sizes.
  forward    back_transform, in place on Z          n, nbw, nev, dtype
  batch      BatchedPlan.run, in place              count, unit, most, nbw, dtype
             (problem sizes n_p = unit * U{1..most}, a fixed draw; nev = n_p/2)
  adjoint    back_transform_autograd and gradients  n, nbw, nev, dtype
  b2f        band_to_full, in place on Z            n, nbw, nev, dtype
  tridiag    tridiagonal_eigh                       n, nev
  chase      band_to_tridiagonal                    n, nbw, dtype
"""
import math

import numpy as np
import torch

import paper_2002_10991_amd as T

DEV = "cuda"


def listed():
    return [
        # the smallest call: the size of the finite-difference check
        dict(name="fwd-d-n64", op="forward", n=64, nbw=8, nev=16, dtype="d"),
        # all eigenvectors of one small problem
        dict(name="fwd-d-n1024", op="forward", n=1024, nbw=32, nev=1024, dtype="d"),
        # half of the spectrum of a mid-size real problem
        dict(name="fwd-d-n8192", op="forward", n=8192, nbw=64, nev=4096, dtype="d"),
        # a quarter of the spectrum of a large Hermitian problem: the benchmark's shape
        dict(name="fwd-z-n32768", op="forward", n=32768, nbw=64, nev=8192, dtype="z"),
        # nothing is a multiple of anything: band width, order, columns
        dict(name="fwd-z-n1201-nbw20", op="forward", n=1201, nbw=20, nev=401, dtype="z"),
        # k-points: independent problems of uneven size in one plan
        dict(name="batch-d-20", op="batch", count=20, unit=512, most=8, nbw=32, dtype="d"),
        # differentiable use, forward and backward
        dict(name="adj-d-n4096", op="adjoint", n=4096, nbw=64, nev=2048, dtype="d"),
        dict(name="adj-z-n1500", op="adjoint", n=1500, nbw=32, nev=750, dtype="z"),
        # the step before: eigenpairs of the tridiagonal matrix
        dict(name="tridiag-n8192", op="tridiag", n=8192, nev=4096),
        # the producer of the reflectors
        dict(name="chase-d-n8192", op="chase", n=8192, nbw=64, dtype="d"),
        # the step after: band to full
        dict(name="b2f-d-n8192", op="b2f", n=8192, nbw=64, nev=4096, dtype="d"),
        dict(name="b2f-z-n16384", op="b2f", n=16384, nbw=64, nev=4096, dtype="z"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["forward", "forward", "forward", "batch", "adjoint", "tridiag", "chase", "b2f"])
    dtype = rng.choice(["d", "z"])
    common = rng.choice([16, 32, 32, 48, 64, 64])
    if op == "forward":
        if rng.random() < 0.3:   # any band width
            n = _log(rng, 50, 1500)
            nbw = rng.randint(2, min(130, n // 2))
        else:
            nbw = rng.choice([common, common, common, 96, 128])
            n = _log(rng, 2 * nbw, 20000)
        return dict(op=op, n=n, nbw=nbw, nev=max(1, int(n * rng.choice([0.1, 0.25, 0.5, 1.0]) *
                                                        (1 if n < 10000 else 0.25))), dtype=dtype)
    if op == "batch":
        return dict(op=op, count=rng.randint(3, 24), unit=_log(rng, 40, 400), most=rng.randint(1, 6),
                    nbw=common, dtype=dtype)
    if op == "adjoint":
        n, nbw = _log(rng, 100, 3000), common
        if rng.random() < 0.2:   # any band width
            n, nbw = _log(rng, 60, 400), rng.randint(2, 30)
        return dict(op=op, n=n, nbw=nbw, nev=max(1, int(n * rng.uniform(0.1, 0.6))), dtype=dtype)
    if op == "tridiag":
        n = _log(rng, 100, 12000)
        return dict(op=op, n=n, nev=max(1, int(n * rng.choice([0.1, 0.25, 0.5, 1.0]))))
    if op == "chase":
        n = _log(rng, 200, 6000)
        return dict(op=op, n=n, nbw=rng.choice([common, rng.randint(2, 64)]), dtype=dtype)
    n = _log(rng, 200, 8000)
    return dict(op=op, n=n, nbw=rng.choice([common, rng.randint(2, 100)]),
                nev=max(1, int(n * rng.uniform(0.1, 1.0))), dtype=dtype)


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------
def _torch_dtype(dtype):
    return torch.complex128 if dtype == "z" else torch.float64


def _gen(seed, k=0):
    g = torch.Generator(device=DEV)
    g.manual_seed(1000003 * int(seed) + k)
    return g


def _stages(n, nbw):
    """Sweeps of every stage s = 0 .. n-3 and the rows of its last sweep."""
    if n < 3 or nbw < 2:
        return np.zeros(0, np.int64), np.zeros(0, np.int64)
    s = np.arange(n - 2, dtype=np.int64)
    sweeps = -((-(n - s - 2)) // nbw)
    return sweeps, np.minimum(nbw, n - (s + 1 + (sweeps - 1) * nbw))


def _unit_tau(nrm2, dtype, g):
    if dtype == "d":
        return 2.0 / nrm2
    theta = (0.5 + torch.rand(nrm2.shape[0], generator=g, device=DEV, dtype=torch.float64)) * math.pi
    return (1.0 - torch.polar(torch.ones_like(theta), theta)) / nrm2


def _norm2(V, dim):
    return (torch.view_as_real(V) if V.is_complex() else V[..., None]).square().sum((dim, -1))


def _reflectors(n, nbw, dtype, seed, k=0):
    g = _gen(seed, 7 * k + 1)
    sweeps, last = _stages(n, nbw)
    K = int(sweeps.sum())
    V = torch.randn(K, nbw, generator=g, device=DEV, dtype=_torch_dtype(dtype)).div_(math.sqrt(nbw))
    V[:, 0] = 1.0
    ends = torch.from_numpy(np.cumsum(sweeps) - 1).to(DEV)
    rows = torch.from_numpy(last).to(DEV)
    V[ends] *= (torch.arange(nbw, device=DEV)[None, :] < rows[:, None]).to(torch.float64)
    tau = torch.cat([_unit_tau(_norm2(V[a:a + (1 << 20)], 1), dtype, g)
                     for a in range(0, K, 1 << 20)])
    return V, tau


def _columns(n, nev, dtype, seed, k):
    """Gaussian n x nev, column-major."""
    return torch.randn(nev, n, generator=_gen(seed, k), device=DEV, dtype=_torch_dtype(dtype)).T


def _batch_sizes(case):
    return [int(v) for v in
            case["unit"] * np.random.default_rng(1004).integers(1, case["most"] + 1, case["count"])]


def _full_reflectors(n, nbw, dtype, seed):
    g = _gen(seed, 1)
    J = max(n - nbw - 1, 0)
    V = torch.randn(J, n, generator=g, device=DEV, dtype=_torch_dtype(dtype))
    V *= (torch.arange(n, device=DEV)[None, :] >
          (torch.arange(J, device=DEV) + nbw)[:, None]).to(torch.float64)
    V /= torch.arange(n - nbw, n - nbw - J, -1, device=DEV, dtype=torch.float64).sqrt()[:, None]
    j = torch.arange(J, device=DEV)
    V[j, j + nbw] = 1.0
    return V.T, _unit_tau(_norm2(V, 1), dtype, g)


def _tridiagonal(n, seed):
    rng = np.random.default_rng(int(seed))
    d = math.sqrt(2.0) * rng.standard_normal(n)
    e = np.sqrt(rng.chisquare(np.arange(n - 1, 0, -1)))
    return d / math.sqrt(n), e / math.sqrt(n)


def _aligned(nbytes):
    if not nbytes:
        return None
    buf = torch.empty(nbytes + T.TRBT_WORK_ALIGN, dtype=torch.uint8, device=DEV)
    return buf[-buf.data_ptr() % T.TRBT_WORK_ALIGN:][:nbytes]


def prepare(case, seed):
    op, n, nbw, nev = case["op"], case.get("n"), case.get("nbw"), case.get("nev")
    dtype = case.get("dtype", "d")
    s = dict(op=op, nbw=nbw, nev=nev)
    if op == "batch":
        s["problems"] = []
        for i, m in enumerate(_batch_sizes(case)):
            V, tau = _reflectors(m, nbw, dtype, seed, i)
            s["problems"].append((_columns(m, m // 2, dtype, seed, 7 * i + 2), V, tau, nbw))
        s["plan"] = T.BatchedPlan(s["problems"])
    elif op == "tridiag":
        s["d"], s["e"] = (torch.from_numpy(v).to(DEV) for v in _tridiagonal(n, seed))
    elif op == "chase":
        ab = torch.randn(n, nbw + 1, generator=_gen(seed), device=DEV, dtype=_torch_dtype(dtype))
        if dtype == "z":
            ab[:, 0].imag.zero_()
        s["ab"] = ab
        s["work"] = _aligned(T.trbt_band_to_tridi_workspace_bytes(n, nbw, dtype == "z"))
    elif op == "b2f":
        s["V"], s["tau"] = _full_reflectors(n, nbw, dtype, seed)
        s["Z"] = _columns(n, nev, dtype, seed, 2)
        s["work"] = _aligned(T.trbt_band_to_full_workspace_bytes(n, nbw, nev, dtype == "z"))
    else:
        s["V"], s["tau"] = _reflectors(n, nbw, dtype, seed)
        s["Z"] = _columns(n, nev, dtype, seed, 2)
        if op == "forward":
            s["work"] = T.alloc_workspace(n, nbw, nev, dtype == "z")
        else:
            s["G"] = _columns(n, nev, dtype, seed, 3)
            for k in ("Z", "V", "tau"):
                s[k].requires_grad_(True)
    return s


def run(s):
    op = s["op"]
    if op == "forward":
        return T.back_transform(s["Z"], s["V"], s["tau"], s["nbw"], work=s["work"])
    if op == "batch":
        s["plan"].run()
        return [p[0] for p in s["problems"]]
    if op == "adjoint":
        out = T.back_transform_autograd(s["Z"], s["V"], s["tau"], s["nbw"])
        return out, torch.autograd.grad(out, (s["Z"], s["V"], s["tau"]), s["G"])
    if op == "tridiag":
        return T.tridiagonal_eigh(s["d"], s["e"], s["nev"])
    if op == "chase":
        return T.band_to_tridiagonal(s["ab"], s["nbw"], work=s["work"])
    return T.band_to_full(s["Z"], s["V"], s["tau"], s["nbw"], work=s["work"])


# --------------------------------------------------------------------------
# what a pass cannot do without
# --------------------------------------------------------------------------
def _rows(n, nbw):
    """(reflectors, sum of their lengths)"""
    sweeps, last = _stages(n, nbw)
    return int(sweeps.sum()), int(((sweeps - 1) * nbw + last).sum())


def work(case):
    op, n, nbw, nev = case["op"], case.get("n"), case.get("nbw"), case.get("nev")
    size, mul = (16, 4) if case.get("dtype", "d") == "z" else (8, 1)
    if op in ("forward", "batch"):
        total = {"bytes": 0, "flops": 0}
        for m, cols in ([(n, nev)] if op == "forward" else [(m, m // 2) for m in _batch_sizes(case)]):
            K, L = _rows(m, nbw)
            total["bytes"] += size * (2 * m * cols + L + K)
            total["flops"] += mul * 4 * cols * L
        return total
    if op == "adjoint":   # Z, G, V, tau in; Z_out and three gradients out; 4 + 14 flops an entry
        K, L = _rows(n, nbw)
        return {"bytes": size * (4 * n * nev + 2 * (L + K)), "flops": mul * 18 * nev * L}
    if op == "b2f":
        J = max(n - nbw - 1, 0)
        L = J * (n - nbw) - J * (J - 1) // 2
        return {"bytes": size * (2 * n * nev + L + J), "flops": mul * 4 * nev * L}
    if op == "tridiag":   # one factorisation and one solve for each vector
        return {"bytes": 8 * (n * nev + 2 * n + nev), "flops": 12 * n * nev}
    # chase: per step one reflector from the left on nbw, from the right on nbw, and two-sided
    # on the diagonal block's triangle
    K, L = _rows(n, nbw)
    return {"bytes": size * (n * (nbw + 1) + L + K), "flops": mul * 12 * nbw * L}


# --------------------------------------------------------------------------
# the same in plain torch, 64 bits
# --------------------------------------------------------------------------
def _stage_views(n, nbw, V, tau, *mats):
    """For every stage: its slice of (V, tau) and, of each row-major (n + nbw)-row matrix, the
    rows its sweeps act on as (sweeps, nbw, columns)."""
    sweeps, _ = _stages(n, nbw)
    k0 = np.cumsum(sweeps) - sweeps
    def at(s):
        S, k = int(sweeps[s]), int(k0[s])
        return (slice(k, k + S), V[k:k + S, :, None], tau[k:k + S, None, None],
                *(m[s + 1:s + 1 + S * nbw].view(S, nbw, -1) for m in mats))
    return at


def _padded(Z, nbw):
    out = torch.zeros(Z.shape[0] + nbw, Z.shape[1], dtype=Z.dtype, device=DEV)
    out[:Z.shape[0]] = Z.detach()
    return out


def _exact_forward(n, nbw, Z, V, tau):
    A = _padded(Z, nbw)
    at = _stage_views(n, nbw, V, tau, A)
    for s in range(n - 3, -1, -1):
        _, v, t, a = at(s)
        a.baddbmm_(v, t * torch.bmm(v.mH.contiguous(), a), alpha=-1.0)
    return A


def _exact_adjoint(n, nbw, Z, V, tau, G):
    A, g = _exact_forward(n, nbw, Z, V, tau), _padded(G, nbw)
    out = A[:n].clone()
    dv, dt = torch.empty_like(V), torch.empty_like(tau)
    at = _stage_views(n, nbw, V, tau, A, g)
    for s in range(n - 2):
        k, v, t, a, b = at(s)
        vh = v.mH.contiguous()
        a.baddbmm_(v, t.conj() * torch.bmm(vh, a), alpha=-1.0)   # H is unitary: the rows before it
        w, gam = torch.bmm(vh, a), torch.bmm(vh, b)
        dt[k] = -(w.conj() * gam).sum((1, 2))
        dv[k] = -(t.conj() * (b * w.conj()).sum(2, keepdim=True) +
                  t * (a * gam.conj()).sum(2, keepdim=True))[:, :, 0]
        b.baddbmm_(v, t.conj() * gam, alpha=-1.0)
    return out, (g[:n], dv, dt)


def _exact_b2f(n, nbw, Z, V, tau):
    C = Z.contiguous().clone()
    J = V.shape[1]
    for j in range((J - 1) // 64 * 64, -1, -64):
        v = V[j + nbw:, j:min(j + 64, J)].contiguous()
        vh = v.mH.contiguous()
        M = torch.triu(vh @ v, 1) + torch.diag(1.0 / tau[j:j + 64])   # inverse of the panel's factor
        C[j + nbw:] -= v @ torch.linalg.solve_triangular(M, vh @ C[j + nbw:], upper=True)
    return C


def exact(case, seed):
    op, n, nbw, nev = case["op"], case.get("n"), case.get("nbw"), case.get("nev")
    dtype = case.get("dtype", "d")
    mul = 4 if dtype == "z" else 1
    if op == "chase":
        return None   # T and the reflectors are ill-conditioned functions of the band
    if op == "tridiag":
        if n > 4096:
            return None   # a dense eigensolver takes too long
        d, e = _tridiagonal(n, seed)
        w, Q = np.linalg.eigh(np.diag(d) + np.diag(e, -1) + np.diag(e, 1)) if n <= 1500 else \
            (v.cpu().numpy() for v in torch.linalg.eigh(torch.from_numpy(
                np.diag(d) + np.diag(e, -1) + np.diag(e, 1)).to(DEV)))
        Q = Q[:, :nev] * np.sign(Q[np.abs(Q[:, :nev]).argmax(0), np.arange(nev)])
        return w[:nev], Q
    if op == "batch":
        return [_exact_forward(m, nbw, _columns(m, m // 2, dtype, seed, 7 * i + 2),
                               *_reflectors(m, nbw, dtype, seed, i))[:m]
                for i, m in enumerate(_batch_sizes(case))]
    Z = _columns(n, nev, dtype, seed, 2)
    if op == "b2f":
        return _exact_b2f(n, nbw, Z, *_full_reflectors(n, nbw, dtype, seed))
    if mul * n * n * nev > 1 << 40:
        return None   # too long, a stage at a time
    V, tau = _reflectors(n, nbw, dtype, seed)
    if op == "forward":
        return _exact_forward(n, nbw, Z, V, tau)[:n]
    return _exact_adjoint(n, nbw, Z, V, tau, _columns(n, nev, dtype, seed, 3))
