"""The folded kernels' tile shapes and their workspace."""
import numpy as np
import pytest

import fmm_inputs as fi

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F():
    import torch
    from paper_2606_13793_amd import fmm
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return fmm


def test_partial_sums_only_for_shared_groups(F):
    """A plan holds its expansions, tables (25 MB here) and the partial sums of the
    column groups whose K loops are shared, not of every group of such a launch."""
    n, p = 128, 6
    h, row, pairs = (p + 1) ** 2, 52, 16 * 25  # harmonic terms, padded row, folded row
    grids = sum(h * (2 ** k + 6) ** 3 for k in range(2, 6)) + sum(8 ** k * row for k in range(3, 6))
    grids += sum(8 ** (k - 1) * pairs for k in range(4, 7)) + n ** 3
    rest = F.Plan(n, p).workspace_bytes() - 8 * grids
    print(f"tables and partial sums {rest / 1e6:.1f} MB", flush=True)
    assert 0 < rest < 64 << 20, rest


# FMM-2 in FP32 at the size from which M2P, its transpose and the blocks take their
# large tiles; even and odd orders, truncation.  Bars: FP32 phi <= 1e-5, g <= 1e-4
# relative L2 against the FP64 oracle of the rounded input, the gradient <= 1e-4
# against an FP64 plan's, and <A rho, y> = <rho, A^T y> to 1e-5 of the norms.
@pytest.mark.parametrize("p,nmax", [(4, None), (5, None), (6, 3)])
def test_fmm2_fp32_large_tiles(F, orc, p, nmax):
    import torch
    n = 128
    print(f"case fmm2 fp32 n={n} p={p} nmax={nmax}", flush=True)
    rho = torch.as_tensor(fi.plummer_density(n, fi.multi_plummer_params(12, 310 + p))).to("cuda", torch.float32)
    gen = torch.Generator(device="cuda").manual_seed(p)
    dphi = torch.randn((n, n, n), device="cuda", generator=gen)
    dg = torch.randn((3, n, n, n), device="cuda", generator=gen)
    plan = F.Plan(n, p, "fp32", nmax=nmax, delta_l=2, coarse_fp64_levels=2)
    phi, g = plan.solve(rho)
    drho, dphi_only = plan.backward(dphi, dg), plan.backward(dphi)
    torch.cuda.synchronize()
    corners = [0, n - 1, n * n - 1, (n - 1) * n * n, n ** 3 - 1]
    cells = np.unique(np.concatenate([corners, np.random.default_rng(p).choice(n ** 3, 64, replace=False)]))
    want = F.Plan(n, p, "fp64", nmax=nmax, delta_l=2).backward(dphi.double(), dg.double())
    e = float((drho.double() - want).norm() / want.norm())
    print(f"  against the FP64 backward pass {e:.2e}", flush=True)
    assert e <= 1e-4, e
    phi_o, g_o = orc.solve(rho.double().cpu().numpy(), p, nmax=nmax, targets=cells, delta_l=2)
    for got, want, bar in ((phi.double().cpu().numpy().reshape(-1)[cells], phi_o, 1e-5),
                           (g.double().cpu().numpy().reshape(3, -1)[:, cells], g_o, 1e-4)):
        e = float(np.linalg.norm(got - want) / np.linalg.norm(want))
        print(f"  {e:.2e}", flush=True)
        assert e <= bar, e
    phi, g, rho = phi.double(), g.double(), rho.double()
    for lhs, grad, scale in (((phi * dphi).sum() + (g * dg).sum(), drho, phi.norm() * dphi.norm() + g.norm() * dg.norm()),
                             ((phi * dphi).sum(), dphi_only, phi.norm() * dphi.norm())):
        d = float((lhs - (rho * grad.double()).sum()).abs() / scale)
        print(f"  identity {d:.2e}", flush=True)
        assert d <= 1e-5, d
