"""Whole sweeps of small grids in one launch against the pass kernels (plans with
checkpoints keep to these): the parent windows of both sides on every pair of sides, with
the planes at either end, at both, between, and in a single slice; and more columns than
the chip has CUs.

Tolerance: either holds 1e-5 against the oracle."""
import pytest

from tests.test_gpu_sweep_starts import compare_windows

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ny,nx", [(64, 64), (64, 128), (128, 64), (128, 128)])
@pytest.mark.parametrize("nz,planes", [(3, [0]), (3, [2]), (5, [0, 2, 4]), (1, [0])])
def test_one_launch_matches_the_passes(ny, nx, nz, planes):
    print(f"[sweep {ny} x {nx}, {nz} slices, planes {planes}]", flush=True)
    compare_windows(ny, nx, nz, planes)
