"""The mirror-folded kernels at the edges of their tiles and dispatch, against
the FP64 oracle.  Bars: FP64 relative L2 <= 1e-12 (the stated FP64 tolerance);
FP32 phi <= 1e-5 and g <= 1e-4 of the float-rounded input.
"""
import sys

import numpy as np
import pytest

import fmm_inputs as fi

pytestmark = pytest.mark.gpu

BARS = {"fp64": (1e-12, 1e-12), "fp32": (1e-5, 1e-4)}


@pytest.fixture(scope="module")
def F():
    import torch
    from paper_2606_13793_amd import fmm
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return fmm


def rel(a, b):
    a, b = np.ravel(a), np.ravel(b)
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


# block tiles of 1 row (small grids), 2 rows (128^3 with the smaller tile) and
# 4 rows (128^3); orders whose term counts leave every remainder of the K steps
@pytest.mark.parametrize("precision,n,p,nmax,tile", [
    ("fp64", 8, 1, None, 0), ("fp64", 8, 8, 3, 16), ("fp64", 16, 7, 0, 8), ("fp64", 128, 2, None, 8),
    ("fp64", 128, 5, 2, 16), ("fp32", 16, 8, None, 0), ("fp32", 128, 3, None, 8), ("fp32", 128, 4, None, 0),
])
def test_finest_blocks(F, orc, precision, n, p, nmax, tile):
    import torch
    print(f"case blocks {precision} n={n} p={p} nmax={nmax} tile={tile}", flush=True)
    dt = torch.float64 if precision == "fp64" else torch.float32
    rho = torch.as_tensor(fi.plummer_density(n, fi.multi_plummer_params(12, 900 + n + p))).to("cuda", dt)
    plan = F.Plan(n, p, precision, nmax=nmax, bottom_tile=tile, coarse_fp64_levels=2)
    phi, g = plan.solve(rho)
    torch.cuda.synchronize()
    rho_h = rho.double().cpu().numpy()
    phi, g = phi.double().cpu().numpy(), g.double().cpu().numpy()
    if n <= 32:
        phi_o, g_o = orc.solve(rho_h, p, nmax=nmax)
    else:
        corners = [0, n - 1, n * n - 1, n ** 3 - 1]
        cells = np.unique(np.concatenate([corners, np.random.default_rng(p).choice(n ** 3, 48, replace=False)]))
        phi_o, g_o = orc.solve(rho_h, p, nmax=nmax, targets=cells)
        phi, g = phi.reshape(-1)[cells], g.reshape(3, -1)[:, cells]
    e = rel(phi, phi_o), rel(g, g_o)
    print(f"  phi {e[0]:.2e} g {e[1]:.2e}", flush=True)
    assert e[0] <= BARS[precision][0] and e[1] <= BARS[precision][1], e


# the shifts between levels: multipoles of one to three levels by one kernel (up
# to 64^3) or a kernel per level, locals of the coarsest level straight from the
# M2L, both types of a mixed plan in one M2L launch, block tiles of one column tile
# (up to 32^3); the smallest and largest orders and truncations
@pytest.mark.parametrize("precision,n,p,nmax,coarse", [
    ("fp64", 16, 6, None, 4), ("fp64", 32, 1, None, 4), ("fp64", 32, 8, 3, 4), ("fp64", 64, 6, None, 4),
    ("fp64", 64, 7, 2, 4), ("fp64", 128, 1, 0, 4), ("fp64", 128, 8, None, 4), ("fp32", 64, 5, None, 3),
    ("fp32", 64, 8, 4, 4), ("fp32", 128, 2, None, 4),
])
def test_level_shifts(F, orc, precision, n, p, nmax, coarse):
    import torch
    print(f"case shifts {precision} n={n} p={p} nmax={nmax} coarse={coarse}", flush=True)
    dt = torch.float64 if precision == "fp64" else torch.float32
    rho = torch.as_tensor(fi.plummer_density(n, fi.multi_plummer_params(9, 40 + n + p))).to("cuda", dt)
    plan = F.Plan(n, p, precision, nmax=nmax, coarse_fp64_levels=coarse)
    phi, g = plan.solve(rho)
    torch.cuda.synchronize()
    corners = [0, n - 1, n * n - 1, n ** 3 - 1]
    cells = np.unique(np.concatenate([corners, np.random.default_rng(n + p).choice(n ** 3, 48, replace=False)]))
    phi_o, g_o = orc.solve(rho.double().cpu().numpy(), p, nmax=nmax, targets=cells)
    e = rel(phi.double().cpu().numpy().reshape(-1)[cells], phi_o), rel(g.double().cpu().numpy().reshape(3, -1)[:, cells], g_o)
    print(f"  phi {e[0]:.2e} g {e[1]:.2e}", flush=True)
    assert e[0] <= BARS[precision][0] and e[1] <= BARS[precision][1], e


# the potential alone takes other products than phi and g: both against each other
# and the oracle, on block tiles of one column tile, one row and two rows
@pytest.mark.parametrize("n,p,nmax,delta_l", [
    (16, 4, None, 1), (64, 1, None, 1), (64, 7, 3, 1), (128, 3, None, 1), (128, 8, None, 1), (64, 5, None, 2), (128, 2, None, 2),
])
def test_potential_alone(F, orc, n, p, nmax, delta_l):
    import torch
    print(f"case phi alone n={n} p={p} nmax={nmax} delta_l={delta_l}", flush=True)
    rho = torch.as_tensor(fi.plummer_density(n, fi.multi_plummer_params(9, 70 + n + p))).cuda()
    plan = F.Plan(n, p, "fp64", nmax=nmax, delta_l=delta_l)
    both, _ = plan.solve(rho)
    alone = torch.full_like(rho, float("nan"))
    plan.solve_into(rho, alone, None)
    torch.cuda.synchronize()
    e = rel(alone.cpu().numpy(), both.cpu().numpy())
    cells = np.random.default_rng(n + p).choice(n ** 3, 48, replace=False)
    kw = {"delta_l": 2} if delta_l == 2 else {}
    phi_o, _ = orc.solve(rho.cpu().numpy(), p, nmax=nmax, targets=cells, **kw)
    eo = rel(alone.cpu().numpy().reshape(-1)[cells], phi_o)
    print(f"  against phi of both {e:.2e}, oracle {eo:.2e}", flush=True)
    assert e <= BARS["fp64"][0] and eo <= BARS["fp64"][0], (e, eo)


# the transposes: the coarsest grids (no M2L; one M2L level), one and several
# L2L levels, truncation, both types of a mixed plan, tiles of every height
@pytest.mark.parametrize("precision,n,p,nmax", [
    ("fp64", 8, 4, None), ("fp64", 16, 8, 3), ("fp64", 32, 7, None), ("fp64", 64, 3, 0),
    ("fp32", 16, 5, None), ("fp32", 64, 4, 2), ("fp64", 128, 2, None),
])
def test_folded_backward(F, orc, precision, n, p, nmax):
    import torch
    print(f"case backward {precision} n={n} p={p} nmax={nmax}", flush=True)
    dt = torch.float64 if precision == "fp64" else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(n + p)
    dphi = torch.randn((n, n, n), dtype=dt, device="cuda", generator=gen)
    dg = torch.randn((3, n, n, n), dtype=dt, device="cuda", generator=gen)
    plan = F.Plan(n, p, precision, nmax=nmax, coarse_fp64_levels=3)
    drho = plan.backward(dphi, dg)
    dphi_only = plan.backward(dphi)
    if n <= 32:
        want = orc.adjoint(dphi.double().cpu().numpy(), dg.double().cpu().numpy(), p, nmax=nmax)
        e = rel(drho.double().cpu().numpy(), want)
        print(f"  {e:.2e}", flush=True)
        assert e <= BARS[precision][1], e
    # <A rho, y> = <rho, A^T y> against the forward solve, with and without dg
    rho = torch.as_tensor(fi.plummer_density(n, fi.multi_plummer_params(12, 77 + n))).to("cuda", dt)
    phi, g = plan.solve(rho)
    torch.cuda.synchronize()
    for lhs, grad, scale in (((phi.double() * dphi).sum() + (g.double() * dg).sum(), drho,
                              phi.double().norm() * dphi.double().norm() + g.double().norm() * dg.double().norm()),
                             ((phi.double() * dphi).sum(), dphi_only, phi.double().norm() * dphi.double().norm())):
        d = float((lhs - (rho.double() * grad.double()).sum()).abs() / scale)
        print(f"  identity {d:.2e}", flush=True)
        assert d <= (1e-13 if precision == "fp64" else 1e-5), d


# FMM-2's folded M2P and its transpose: no M2L level, one, several; both types
@pytest.mark.parametrize("precision,n,p,nmax", [("fp64", 16, 5, None), ("fp64", 32, 8, 2), ("fp32", 64, 3, None)])
def test_folded_fmm2(F, orc, precision, n, p, nmax):
    import torch
    print(f"case fmm2 {precision} n={n} p={p} nmax={nmax}", flush=True)
    dt = torch.float64 if precision == "fp64" else torch.float32
    rho = torch.as_tensor(fi.plummer_density(n, fi.multi_plummer_params(12, 31 + n))).to("cuda", dt)
    gen = torch.Generator(device="cuda").manual_seed(n + p)
    dphi = torch.randn((n, n, n), dtype=dt, device="cuda", generator=gen)
    dg = torch.randn((3, n, n, n), dtype=dt, device="cuda", generator=gen)
    plan = F.Plan(n, p, precision, nmax=nmax, delta_l=2, coarse_fp64_levels=3)
    phi, g = plan.solve(rho)
    drho = plan.backward(dphi, dg)
    torch.cuda.synchronize()
    h = [t.double().cpu().numpy() for t in (rho, phi, g, dphi, dg, drho)]
    phi_o, g_o = orc.solve(h[0], p, nmax=nmax, delta_l=2)
    e = rel(h[1], phi_o), rel(h[2], g_o), rel(h[5], orc.adjoint(h[3], h[4], p, nmax=nmax, delta_l=2))
    print(f"  phi {e[0]:.2e} g {e[1]:.2e} drho {e[2]:.2e}", flush=True)
    bp, bg = BARS[precision]
    assert e[0] <= bp and e[1] <= bg and e[2] <= bg, e
