"""The folded kernels' tile shapes and their workspace."""
import pytest

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
