"""Workloads the solver's speed is judged on, through the package's public calls.

``listed()`` names the fixed ones, ``draw(rng)`` gives more of the same
ranges.  A case is a dict of plain values:

  path       "solve" (a density to phi and g), "backward" (cotangents to the
             density's gradient), "train" (a differentiable solve and its
             backward pass), "batch" (several fields in one plan), "particles"
             (cloud-in-cell deposit, solve, finite-difference force)
  n, p       grid cells per axis and expansion order; nmax, the multipole
             order (equal to p unless truncated)
  precision  "fp64", "fp32" or "bf16" plans; delta_l 1 or 2 (FMM-1, FMM-2)
  want_g     whether the acceleration is asked for (solve)
  fields     grid sizes of a batch, comma separated
  count      particles

The densities are sums of Plummer spheres, the inputs of this repository's
tests and benchmark.  ``exact`` evaluates the method itself (truncated
Cartesian expansions on the same levels and lists) in float64 with plain
torch operations.
"""
import math

import numpy as np
import torch

from paper_2606_13793_amd import fmm

DEV = "cuda"


def _solve_case(name, n, p, precision="fp64", nmax=None, delta_l=1, want_g=True):
    c = {"path": "solve", "n": n, "p": p, "nmax": p if nmax is None else nmax, "precision": precision,
         "delta_l": delta_l, "want_g": want_g}
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest grid: launch latency
        _solve_case("solve_8_p4_fp64", 8, 4),
        # small grids of the tests and of batches, solved one by one
        _solve_case("solve_32_p6_fp64", 32, 6),
        _solve_case("solve_64_p5_fp32", 64, 5, "fp32"),
        # potential only, as a host code that differentiates it itself asks for
        _solve_case("solve_128_p8_fp64_phi", 128, 8, want_g=False),
        # the benchmark's grid and order under each compute policy
        _solve_case("solve_256_p6_fp64", 256, 6),
        _solve_case("solve_256_p6_fp32", 256, 6, "fp32"),
        _solve_case("solve_256_p6_bf16", 256, 6, "bf16"),
        # the paper's variant with the finest expansions two levels up
        _solve_case("solve_128_p6_fmm2_fp64", 128, 6, delta_l=2),
        # gradients: a backward pass alone, and a whole differentiable step
        {"name": "backward_128_p6_fp64", "path": "backward", "n": 128, "p": 6, "nmax": 6, "precision": "fp64",
         "delta_l": 1},
        {"name": "train_64_p4_fp32", "path": "train", "n": 64, "p": 4, "nmax": 4, "precision": "fp32", "delta_l": 1},
        # an uneven batch in the benchmark batch's proportions
        {"name": "batch_14_p4_fp32", "path": "batch", "p": 4, "nmax": 4, "precision": "fp32", "delta_l": 1,
         "fields": "32,64,32,128,32,32,64,32,64,32,128,32,64,32"},
        # a particle step at the paper's orders: deposit, solve, 5-point force
        {"name": "particles_128_p3", "path": "particles", "n": 128, "p": 3, "nmax": 2, "precision": "fp64",
         "delta_l": 1, "count": 1000003},
    ]


def draw(rng):
    path = rng.choice(["solve", "solve", "solve", "backward", "train", "batch", "particles"])
    precision = rng.choice(["fp64", "fp64", "fp32", "fp32", "bf16"])
    delta_l = rng.choice([1, 1, 1, 2])
    p = rng.randint(1, 8)
    if path == "batch":
        k = rng.randint(2, 14)
        fields = [rng.choice([16, 32, 32, 32, 64, 64, 128]) for _ in range(k)]
        return {"path": path, "p": min(p, 6), "nmax": min(p, 6), "precision": precision, "delta_l": delta_l,
                "fields": ",".join(str(n) for n in fields)}
    n = 1 << rng.randint(3, 8)
    if path in ("backward", "train"):
        n = min(n, 128)
    if delta_l == 2:
        n = max(n, 16)
    if n == 256:
        p = min(p, 6)
    nmax = p if path != "particles" and rng.random() < 0.7 else rng.randint(0, p)
    c = {"path": path, "n": n, "p": p, "nmax": nmax, "precision": precision, "delta_l": delta_l}
    if path == "solve":
        c["want_g"] = rng.random() < 0.8
    if path == "particles":
        c["precision"] = "fp64"
        c["count"] = int(math.exp(rng.uniform(math.log(1000), math.log(1 << 21)))) | 1
    return c


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------
def _dtype(case):
    return torch.float64 if case["precision"] == "fp64" else torch.float32


def _density(n, seed, dtype, k=24):
    """k Plummer spheres: centres in [0.2, 0.8]^3, radii 0.005..0.05, masses 0.01..1."""
    r = np.random.default_rng(seed)
    cen = r.uniform(0.2, 0.8, (k, 3))
    rad = np.exp(r.uniform(math.log(0.005), math.log(0.05), k))
    mass = np.exp(r.uniform(math.log(1e-2), 0.0, k))
    x = (torch.arange(n, dtype=torch.float64, device=DEV) + 0.5) / n
    out = torch.zeros((n, n, n), dtype=torch.float64, device=DEV)
    for c, a, m in zip(cen, rad, mass):
        r2 = [((x - float(c[d])) / float(a)) ** 2 for d in range(3)]
        q = 1.0 + r2[0][:, None, None] + r2[1][None, :, None] + r2[2][None, None, :]
        out += 3.0 * float(m) / (4.0 * math.pi * float(a) ** 3) / (q * q * q.sqrt())
    return out.to(dtype)


def _cotangents(case, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    n = case["n"]
    dphi = torch.randn((n, n, n), dtype=_dtype(case), device=DEV, generator=g)
    dg = torch.randn((3, n, n, n), dtype=_dtype(case), device=DEV, generator=g)
    return dphi, dg


def _particles(case, seed):
    """Particles of two uniform spheres, in cell order as AMR codes keep them."""
    r = np.random.default_rng(seed)
    k, n = case["count"], case["n"]
    pos = r.standard_normal((k, 3))
    big = r.random(k) < 8.0 / 9.0
    rad = np.where(big, 0.1, 0.05) * r.random(k) ** (1.0 / 3.0)
    pos *= (rad / np.linalg.norm(pos, axis=1))[:, None]
    pos += np.where(big[:, None], np.array([[0.6, 0.5, 0.5]]), np.array([[0.35, 0.5, 0.5]]))
    lo = np.floor(pos * n - 0.5).astype(np.int64) + 1
    pos = pos[np.argsort((lo[:, 0] * (n + 2) + lo[:, 1]) * (n + 2) + lo[:, 2], kind="stable")]
    mass = np.exp(r.uniform(math.log(0.5), math.log(2.0), k)) / k
    return torch.as_tensor(pos, device=DEV), torch.as_tensor(mass, device=DEV)


def _sizes(case):
    return [int(s) for s in case["fields"].split(",")]


def prepare(case, seed):
    st = {"path": case["path"], "want_g": case.get("want_g", True)}
    if case["path"] == "batch":
        sizes, dt = _sizes(case), _dtype(case)
        st["plan"] = fmm.Batch(sizes, case["p"], case["precision"], delta_l=case["delta_l"])
        st["rho"] = [_density(n, [seed, f], dt, 12) for f, n in enumerate(sizes)]
        st["phi"] = [torch.empty_like(r) for r in st["rho"]]
        st["g"] = [torch.empty((3, *r.shape), dtype=dt, device=DEV) for r in st["rho"]]
        return st
    nmax = None if case["nmax"] == case["p"] else case["nmax"]
    st["plan"] = fmm.Plan(case["n"], case["p"], case["precision"], nmax=nmax, delta_l=case["delta_l"])
    if case["path"] == "particles":
        st["pos"], st["mass"] = _particles(case, seed)
        st["n"] = case["n"]
    if case["path"] in ("solve", "train"):
        st["rho"] = _density(case["n"], seed, _dtype(case))
    if case["path"] in ("backward", "train"):
        st["dphi"], st["dg"] = _cotangents(case, seed)
    if case["path"] == "train":
        st["rho"].requires_grad_(True)
    return st


def run(st):
    path, plan = st["path"], st["plan"]
    if path == "solve":
        phi, g = plan.solve(st["rho"], want_g=st["want_g"])
        return [phi] if g is None else [phi, g]
    if path == "backward":
        return plan.backward(st["dphi"], st["dg"])
    if path == "train":
        phi, g = fmm.solve(plan, st["rho"])
        (drho,) = torch.autograd.grad([phi, g], [st["rho"]], [st["dphi"], st["dg"]])
        return [phi.detach(), g.detach(), drho]
    if path == "batch":
        plan.solve_into(st["rho"], st["phi"], st["g"])
        return {"phi": st["phi"], "g": st["g"]}
    rho = fmm.deposit_cic(st["n"], st["pos"], st["mass"])
    phi, g = plan.solve(rho)
    return [rho, phi, g, fmm.fd_force(phi)]


# --------------------------------------------------------------------------
# the least work of a pass
# --------------------------------------------------------------------------
def _solve_flops(n, p, nmax, dl, outs):
    """Two per multiply-add.  The kernel is harmonic, so an expansion to degree
    m has (m + 1)^2 independent terms; sources and targets of an oct mirror
    each other about its centre along each axis, which leaves 1/8 of the
    products; and the sources and targets of the finest octs are the unigrid
    cells themselves where those are fewer than the terms."""
    h = lambda m: (m + 1) ** 2  # noqa: E731
    F = n.bit_length() - 1 - dl
    macs = 0.0
    pairs = sum((2 * b + 1) * h(min(nmax, p - b)) for b in range(p + 1))
    for k in range(3, F + 1):
        macs += 8 ** (k - 2) * 216 * 8 * pairs
    blocks = (n // 4) ** 3
    macs += blocks * 216 * 64 * outs
    if F >= 3:
        macs += blocks * h(p) * 64 * outs
    if dl == 2:
        macs += 8 ** (F - 1) * 216 * h(nmax) * 64 * outs
    return 2.0 * macs


def work(case):
    esz = 8 if case["precision"] == "fp64" else 4
    p, nmax, dl = case["p"], case["nmax"], case["delta_l"]
    if case["path"] == "batch":
        sizes = _sizes(case)
        return {"bytes": float(sum(5 * esz * n ** 3 for n in sizes)),
                "flops": sum(_solve_flops(n, p, nmax, dl, 4) for n in sizes)}
    n = case["n"]
    N, one = n ** 3, _solve_flops(n, p, nmax, dl, 4)
    if case["path"] == "solve":
        outs = 4 if case["want_g"] else 1
        return {"bytes": float((1 + outs) * esz * N), "flops": _solve_flops(n, p, nmax, dl, outs)}
    if case["path"] == "backward":
        return {"bytes": 5.0 * esz * N, "flops": one}
    if case["path"] == "train":
        return {"bytes": 10.0 * esz * N, "flops": 2 * one}
    return {"bytes": 8.0 * (4 * case["count"] + 8 * N), "flops": one + 24.0 * case["count"] + 21.0 * N}


# --------------------------------------------------------------------------
# the method in float64 with plain torch
# --------------------------------------------------------------------------
def _terms(P):
    return [(a, b, m - a - b) for m in range(P + 1) for a in range(m + 1) for b in range(m - a + 1)]


def _fact(e):
    return math.factorial(e[0]) * math.factorial(e[1]) * math.factorial(e[2])


def _mono(w, e):
    """prod_d w_d^e_d / e_d! for points w (k, 3)."""
    return w[:, 0] ** e[0] * w[:, 1] ** e[1] * w[:, 2] ** e[2] / _fact(e)


def _green(R, P):
    """{multi-index: -d^g (1/r)} at the points R (k, 3), to order P."""
    r2 = (R * R).sum(1)
    f = {(0, 0, 0): 1.0 / np.sqrt(r2)}
    for e in _terms(P)[1:]:
        m, s = sum(e), np.zeros(len(R))
        for d in range(3):
            if e[d] >= 1:
                lo = list(e)
                lo[d] -= 1
                s += (2 * m - 1) * e[d] * R[:, d] * f[tuple(lo)]
                if e[d] >= 2:
                    lo[d] -= 1
                    s += (m - 1) * e[d] * (e[d] - 1) * f[tuple(lo)]
        f[e] = -s / (m * r2)
    return {e: -v for e, v in f.items()}


def _bits(b):
    return np.array([[(b >> 2) & 1, (b >> 1) & 1, b & 1]], dtype=np.float64)


def _children(x, k):
    """(m k, m k, m k, T) -> (m, m, m, k^3, T), the child slow to fast along x, y, z."""
    m, T = x.shape[0] // k, x.shape[3]
    return x.reshape(m, k, m, k, m, k, T).permute(0, 2, 4, 1, 3, 5, 6).reshape(m, m, m, k ** 3, T)


def _parents(x, k):
    m, T = x.shape[0], x.shape[4]
    return x.reshape(m, m, m, k, k, k, T).permute(0, 3, 1, 4, 2, 5, 6).reshape(m * k, m * k, m * k, T)


def _lists():
    """(parity bits, offset) of every interaction-list entry."""
    for r in range(8):
        rb = ((r >> 2) & 1, (r >> 1) & 1, r & 1)
        for dd in range(343):
            d = (dd // 49 - 3, dd // 7 % 7 - 3, dd % 7 - 3)
            if all(rb[a] - 3 <= d[a] <= rb[a] + 2 for a in range(3)) and max(abs(v) for v in d) > 1:
                yield rb, d, dd


def _over_lists(M, table, cols):
    """out[P] = sum over the list of P of M[P - d] @ table[d]; (m, m, m, T) -> (m, m, m, cols)."""
    m = M.shape[0]
    pad = torch.nn.functional.pad(M, (0, 0, 3, 3, 3, 3, 3, 3))
    acc = {}
    for rb, d, dd in _lists():
        if all(abs(v) >= m for v in d):
            continue
        s = [slice(3 + rb[a] - d[a], 3 + rb[a] - d[a] + m, 2) for a in range(3)]
        x = pad[s[0], s[1], s[2]].reshape(-1, M.shape[3]) @ table[dd]
        acc[rb] = acc[rb] + x if rb in acc else x
    x = torch.stack([acc[((r >> 2) & 1, (r >> 1) & 1, r & 1)].reshape(m // 2, m // 2, m // 2, cols) for r in range(8)],
                    dim=3)
    return _parents(x, 2)


def _t(x):
    return torch.as_tensor(np.ascontiguousarray(x), dtype=torch.float64, device=DEV)


def _fmm(rho, p, nmax, dl):
    """(phi, g) of rho (n, n, n) float64."""
    n = rho.shape[0]
    F, w = n.bit_length() - 1 - dl, 1 << dl
    S, Lt = _terms(nmax), _terms(p)
    at = {e: i for i, e in enumerate(Lt)}
    sub = np.array([[i, j, k] for i in range(w) for j in range(w) for k in range(w)], dtype=np.float64)
    sub = (sub + 0.5) / w - 0.5  # unigrid centres in a finest cell, units of its size
    # multipoles (-1)^|a| sum m (x - c)^a / (a! h^|a|), m in units of dx^3
    M = {F: _children(rho[..., None], w)[..., 0] @ _t(np.stack([_mono(-sub, e) for e in S], 1))}
    for k in range(F, 2, -1):
        T = np.zeros((8, len(S), len(S)))
        for q in range(8):
            x = -(2 * _bits(q) - 1) / 4
            for j, a in enumerate(S):
                for i, b in enumerate(S):
                    g = tuple(a[d] - b[d] for d in range(3))
                    if min(g) >= 0:
                        T[q, i, j] = 0.5 ** sum(b) * _mono(x, g)[0]
        c = _children(M[k], 2)
        M[k - 1] = c.reshape(*c.shape[:3], -1) @ _t(T.reshape(8 * len(S), len(S)))
    dgrid = np.array([[dd // 49 - 3, dd // 7 % 7 - 3, dd % 7 - 3] for dd in range(343)], dtype=np.float64)
    far = np.abs(dgrid).max(1) > 1
    # locals h^(|b|+1) d^b phi, M2L and L2L
    L = None
    if F >= 3:
        tab = np.zeros((343, len(S), 8, len(Lt)))
        for q in range(8):
            D = _green(dgrid[far] + (2 * _bits(q) - 1) / 4, p)
            for i, a in enumerate(S):
                for j, b in enumerate(Lt):
                    if sum(a) + sum(b) <= p:
                        tab[far, i, q, j] = 0.5 ** (sum(b) + 1) * D[tuple(a[d] + b[d] for d in range(3))]
        tab = _t(tab.reshape(343, len(S), -1))
        shift = np.zeros((8, len(Lt), len(Lt)))
        for q in range(8):
            x = (2 * _bits(q) - 1) / 4
            for j, b in enumerate(Lt):
                for e in Lt:
                    g = tuple(e[d] - b[d] for d in range(3))
                    if min(g) >= 0:
                        shift[q, at[e], j] = 0.5 ** (sum(b) + 1) * _mono(x, g)[0]
        shift = _t(shift.transpose(1, 0, 2).reshape(len(Lt), -1))
        for k in range(3, F + 1):
            new = _over_lists(M[k - 1], tab, tab.shape[2])
            if L is not None:
                new = new + L @ shift
            L = _parents(new.reshape(*new.shape[:3], 8, len(Lt)), 2)
        del tab
    # the finest level: M2P, L2P; columns (unigrid cell, output)
    E = [(0, 0, 0), (1, 0, 0), (0, 1, 0), (0, 0, 1)]
    ns = len(sub)
    tab = np.zeros((343, len(S), ns, 4))
    for s in range(ns):
        D = _green(dgrid[far] + sub[s], nmax + 1)
        for i, a in enumerate(S):
            for o, x in enumerate(E):
                tab[far, i, s, o] = D[tuple(a[d] + x[d] for d in range(3))]
    out = _over_lists(M[F], _t(tab.reshape(343, len(S), -1)), ns * 4)
    if L is not None:
        ev = np.zeros((len(Lt), ns, 4))
        for j, b in enumerate(Lt):
            for o, x in enumerate(E):
                e = tuple(b[d] - x[d] for d in range(3))
                if min(e) >= 0:
                    ev[j, :, o] = _mono(sub, e)
        out = out + L @ _t(ev.reshape(len(Lt), -1))
    out = _parents(out.reshape(*out.shape[:3], ns, 4), w)
    dx, h = 1.0 / n, w / n
    scale = _t([dx ** 3 / h] + [-dx ** 3 / h ** 2] * 3)
    out = out * scale
    # near field: the unigrid cells of the 27 finest cells around
    near = [torch.zeros_like(rho) for _ in range(4)]
    reach = 2 * w - 1
    pos = torch.arange(n, device=DEV)
    cell = pos // w
    for i in range(-reach, reach + 1):
        ok0 = ((cell - (pos - i).div(w, rounding_mode="floor")).abs() <= 1).double()[:, None, None]
        for j in range(-reach, reach + 1):
            ok1 = ok0 * ((cell - (pos - j).div(w, rounding_mode="floor")).abs() <= 1).double()[None, :, None]
            for k in range(-reach, reach + 1):
                ok = ok1 * ((cell - (pos - k).div(w, rounding_mode="floor")).abs() <= 1).double()[None, None, :]
                src = torch.nn.functional.pad(rho, (reach,) * 6)[reach - i:reach - i + n, reach - j:reach - j + n,
                                                                 reach - k:reach - k + n] * ok
                r = math.sqrt(i * i + j * j + k * k)
                near[0] = near[0] - src * (dx * dx / max(r, 1.0))
                for o, v in enumerate((i, j, k)):
                    if v:
                        near[1 + o] = near[1 + o] - src * (dx * v / r ** 3)
    return out[..., 0] + near[0], torch.stack([out[..., 1 + o] + near[1 + o] for o in range(3)])


def _cic(n, pos, mass):
    rho = torch.zeros(n * n * n, dtype=torch.float64, device=DEV)
    x = pos * n - 0.5
    lo = x.floor().long()
    fr = x - lo
    for b in range(8):
        bit = torch.tensor([(b >> 2) & 1, (b >> 1) & 1, b & 1], device=DEV)
        c = lo + bit
        w = torch.where(bit.bool(), fr, 1.0 - fr).prod(1) * mass * float(n) ** 3
        ok = ((c >= 0) & (c < n)).all(1)
        c = c[ok]
        rho.index_add_(0, (c[:, 0] * n + c[:, 1]) * n + c[:, 2], w[ok])
    return rho.reshape(n, n, n)


def _fd(phi):
    """Fourth-order differences over 5 cells, one-sided in the two layers at each wall."""
    n = phi.shape[0]
    idx = torch.arange(n, device=DEV)
    first = (idx - 2).clamp(0, n - 5)
    W = torch.zeros((n, n), dtype=torch.float64, device=DEV)
    for s in range(5):
        pts = np.arange(5) - s
        wts = np.linalg.solve(np.vander(pts, 5, increasing=True).T.astype(np.float64), [0, 1, 0, 0, 0]) * n
        rows = idx[(idx - first) == s]
        for j in range(5):
            W[rows, first[rows] + j] = -float(wts[j])
    return torch.stack([(W @ phi.reshape(n, -1)).reshape(phi.shape), W @ phi, phi @ W.T])


def exact(case, seed):
    p, nmax, dl = case["p"], case["nmax"], case["delta_l"]
    if case["path"] == "batch":
        outs = [_fmm(_density(n, [seed, f], _dtype(case), 12).double(), p, nmax, dl)
                for f, n in enumerate(_sizes(case))]
        return {"phi": [o[0] for o in outs], "g": [o[1] for o in outs]}
    n = case["n"]
    if case["path"] == "solve":
        phi, g = _fmm(_density(n, seed, _dtype(case)).double(), p, nmax, dl)
        return [phi, g] if case["want_g"] else [phi]
    if case["path"] == "particles":
        rho = _cic(n, *_particles(case, seed))
        phi, g = _fmm(rho, p, nmax, dl)
        return [rho, phi, g, _fd(phi)]
    if case["path"] == "train":
        rho = _density(n, seed, _dtype(case)).double().requires_grad_(True)
    else:
        rho = torch.zeros((n, n, n), dtype=torch.float64, device=DEV, requires_grad=True)
    phi, g = _fmm(rho, p, nmax, dl)
    dphi, dg = (c.double() for c in _cotangents(case, seed))
    (drho,) = torch.autograd.grad([phi, g], [rho], [dphi, dg])
    return [phi.detach(), g.detach(), drho] if case["path"] == "train" else drho
