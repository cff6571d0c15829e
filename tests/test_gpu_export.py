"""Expansions that the folded kernels hold, term by term against the FP64
oracle.  Bar: 1e-12 relative L2 (the stated FP64 tolerance).
"""
import math

import numpy as np
import pytest

import fmm_inputs as fi

pytestmark = pytest.mark.gpu

TOL64 = 1e-12


@pytest.fixture(scope="module")
def F():
    import torch
    from paper_2606_13793_amd import fmm
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return fmm


def rel(a, b):
    return float(np.linalg.norm(np.ravel(a) - np.ravel(b)) / np.linalg.norm(np.ravel(b)))


def oracle_expansions(orc, F, rho, p, which, level, nmax=None):
    """The oracle's in the kernels' scaled form and term order."""
    n, q = rho.shape[0], p if which == "L" or nmax is None else nmax
    X = orc.expansions(rho, p, which, level, nmax=nmax)
    order = [tuple(e) for e in orc.multi_index(q)]
    mi = [tuple(e) for e in F.multi_index(q)]
    X = X[:, [order.index(e) for e in mi]]
    deg = np.array([sum(e) for e in mi])
    dx, h = 1.0 / n, 2.0 ** -level
    if which == "L":
        return X * h ** (deg + 1) / dx ** 3
    fact = np.array([math.prod(math.factorial(k) for k in e) for e in mi], float)
    return X * ((-1.0) ** deg) / (fact * h ** deg * dx ** 3)


def harmonic(F, M, q):
    """Multipoles as Laplace's equation leaves them: a derivative with z exponent
    2 k + e is (-1)^k sum_l C(k, l) of the ones with x + 2 l, y + 2 (k - l), e."""
    mi = [tuple(e) for e in F.multi_index(q)]
    terms = [e for e in mi if e[2] < 2]
    out = np.zeros((M.shape[0], len(terms)))
    for t, (x, y, z) in enumerate(mi):
        k, e = divmod(z, 2)
        for l in range(k + 1):
            out[:, terms.index((x + 2 * l, y + 2 * (k - l), e))] += (-1) ** k * math.comb(k, l) * M[:, t]
    return out


# the upward pass in one kernel (up to 64^3) and by a kernel per level, one to
# three levels at once, truncation, both I/O types, FMM-2
@pytest.mark.parametrize("precision,n,p,nmax,delta_l", [
    ("fp64", 16, 3, None, 1), ("fp64", 64, 6, None, 1), ("fp64", 64, 8, 3, 1), ("fp64", 128, 5, None, 1),
    ("fp64", 128, 4, 2, 1), ("fp32", 128, 3, None, 1), ("fp64", 32, 7, None, 2), ("fp64", 128, 2, None, 2),
])
def test_stored_multipoles(F, orc, precision, n, p, nmax, delta_l):
    """What P2M and M2M left on the device, in harmonic terms; and that it is the
    device's: the backward pass leaves its cotangents in the same place."""
    import torch
    print(f"case stored multipoles {precision} n={n} p={p} nmax={nmax} delta_l={delta_l}", flush=True)
    dt = torch.float64 if precision == "fp64" else torch.float32
    rho = torch.as_tensor(fi.plummer_density(n, fi.multi_plummer_params(8, 600 + n + p))).to("cuda", dt)
    plan = F.Plan(n, p, precision, nmax=nmax, delta_l=delta_l)
    plan.solve(rho)
    torch.cuda.synchronize()
    q = p if nmax is None else nmax
    levels = range(2, n.bit_length() - 2)  # up to the cells of 4^3 unigrid cells
    first = {}
    for level in levels:
        want = oracle_expansions(orc, F, rho.double().cpu().numpy(), p, "M", level, nmax)
        got = first[level] = plan.expansions("M", level)
        e = rel(got, want), rel(harmonic(F, got, q), harmonic(F, want, q))
        assert e[0] <= TOL64 and e[1] <= TOL64, (level, e)
    plan.backward(torch.ones_like(rho))
    torch.cuda.synchronize()
    for level in levels:
        assert rel(harmonic(F, plan.expansions("M", level), q), harmonic(F, first[level], q)) > 1e-3, level
    plan.solve(rho)
    torch.cuda.synchronize()
    for level in levels:
        assert np.array_equal(plan.expansions("M", level), first[level]), level


# the finest level alone and with a parent, levels kept complete, FMM-2, the finest
# level in FP32 (bar: FP32 phi's 1e-5)
@pytest.mark.parametrize("precision,n,p,delta_l", [
    ("fp64", 16, 8, 1), ("fp64", 32, 1, 1), ("fp64", 64, 7, 1), ("fp64", 64, 4, 2), ("fp32", 64, 6, 1), ("fp32", 16, 3, 1),
])
def test_stored_locals(F, orc, precision, n, p, delta_l):
    import torch
    print(f"case stored locals {precision} n={n} p={p} delta_l={delta_l}", flush=True)
    dt = torch.float64 if precision == "fp64" else torch.float32
    rho = torch.as_tensor(fi.plummer_density(n, fi.multi_plummer_params(8, 650 + n + p))).to("cuda", dt)
    plan = F.Plan(n, p, precision, delta_l=delta_l, coarse_fp64_levels=2)
    plan.solve(rho)
    torch.cuda.synchronize()
    for level in range(3, plan.finest_level + 1):
        e = rel(plan.expansions("L", level), oracle_expansions(orc, F, rho.double().cpu().numpy(), p, "L", level))
        assert e <= (TOL64 if precision == "fp64" else 1e-5), (level, e)


def test_locals_cost_what_multipoles_cost(F):
    """Both exports of the finest level write the same number of values."""
    import time
    import torch
    plan = F.Plan(128, 6)
    plan.solve(torch.ones((128,) * 3, dtype=torch.float64, device="cuda"))
    torch.cuda.synchronize()

    def best(which):
        times = []
        for _ in range(3):
            t = time.perf_counter()
            plan.expansions(which, 6)
            times.append(time.perf_counter() - t)
        return min(times)

    m, l = best("M"), best("L")
    print(f"multipoles {m:.3f} s, locals {l:.3f} s", flush=True)
    assert l <= 8 * m, (l, m)


def test_refused_exports_say_why(F):
    """The finest level of an FP32 plan: no multipoles are formed there, at any
    size; its locals are exported from small grids."""
    plan = F.Plan(64, 3, "fp32")
    with pytest.raises(F.FmmError, match="forms no level-5 multipoles") as e:
        plan.expansions("M", 5)
    assert e.value.code == F.FMM_ERR_UNSUPPORTED
    for n, fine in ((64, True), (128, True), (256, False)):
        plan = F.Plan(n, 1, "fp32")
        if fine:
            plan.expansions("L", plan.finest_level)
            continue
        with pytest.raises(F.FmmError, match="kept in FP32 only") as e:
            plan.expansions("L", plan.finest_level)
        assert e.value.code == F.FMM_ERR_UNSUPPORTED
