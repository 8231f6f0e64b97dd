"""Whole sweeps of small grids in one launch against the pass kernels (plans with
checkpoints keep to these): the parent windows of both sides on every pair of sides, with
the planes at either end, at both, between, and in a single slice; and against the oracle
with more columns than the chip has CUs.

Tolerance: either holds 1e-5 against the oracle."""
import numpy as np
import pytest

from tests._tiny import as_oracle_problem, tiny_cfg, tiny_problem
from tests.test_gpu_sweep_starts import compare_windows

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ny,nx", [(64, 64), (64, 128), (128, 64), (128, 128)])
@pytest.mark.parametrize("nz,planes", [(3, [0]), (3, [2]), (5, [0, 2, 4]), (1, [0])])
def test_one_launch_matches_the_passes(ny, nx, nz, planes):
    print(f"[sweep {ny} x {nx}, {nz} slices, planes {planes}]", flush=True)
    compare_windows(ny, nx, nz, planes)


@pytest.mark.parametrize("ny,nx,ly,lx", [(64, 64, 12.0, 12.0), (64, 128, 8.0, 16.0), (128, 64, 16.0, 8.0),
                                         (128, 128, 16.0, 16.0)])
def test_more_columns_than_cus_match_the_oracle(ny, nx, ly, lx):
    import torch
    from oracle import eels as E
    from oracle import multislice as ms
    from paper_2607_00756_amd import bip
    cfg = tiny_cfg(ny=ny, nx=nx, nz=3, ly=ly, lx=lx, alpha=15e-3, theta=24e-3, s=1, scan=(2, 2))
    tp = tiny_problem(cfg, n_atoms=1, n_ch=1, W=12, seed=nx, planes=[1])
    tp.win_origin[0] = (ny - 5, nx - 7)  # wraps both ways
    plan = bip.Plan.from_config(cfg, tp.tau, tp.win_size, tp.win_origin)
    assert plan.Bp1 + plan.Bp2 > torch.cuda.get_device_properties(0).multi_processor_count
    plan.build_smatrix(torch.from_numpy(tp.V).cuda())
    prob = as_oracle_problem(tp)
    y, x = prob.window(0)
    for side, n, which, columns, sign in ((1, plan.Bp1, bip.Q_PARENTS1, ms.s1_windows, -1),
                                          (2, plan.Bp2, bip.Q_PARENTS2, ms.s2_windows, +1)):
        out = torch.full((n, 12, 12), float("nan"), dtype=torch.complex64, device="cuda")
        plan.parent_windows(0, side, out)
        got, par = out.cpu().numpy(), plan.query(which)
        want = columns(cfg, par, prob.T, prob.P, [(1, y, x)])[0] * E.carrier(cfg, par, y, x, sign)
        print(f"[{ny} x {nx} side {side}] {n} columns", flush=True)
        assert np.linalg.norm(got - want) <= 1e-5 * np.linalg.norm(want)
    plan.close()
