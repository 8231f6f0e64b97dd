"""Batches that hold columns of both sides, which advance in shared row passes, against
the sides swept one after the other (plans with checkpoints): parent windows of both
sides with all columns in one batch, in batches that split either side, and with planes
that let the sides share every slice, some of them and none.

Tolerance: either holds 1e-5 against the oracle."""
import pytest

from tests.test_gpu_sweep_starts import compare_windows

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ny,nx", [(64, 256), (256, 64), (64, 512)])
@pytest.mark.parametrize("batch", [0, 13, 1])
@pytest.mark.parametrize("nz,planes", [(5, [0, 4]), (5, [3]), (5, [1, 2]), (4, [0]), (4, [3])])
def test_shared_batches_match_the_sides(ny, nx, batch, nz, planes, monkeypatch):
    monkeypatch.setenv("BIP_COLUMN_BATCH", str(batch))
    print(f"[both sides {ny} x {nx}, batches of {batch}, {nz} slices, planes {planes}]", flush=True)
    compare_windows(ny, nx, nz, planes)
