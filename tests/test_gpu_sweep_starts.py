"""Sweeps that start in their first row pass and end with the windows' rows alone (plans
without checkpoints) against those that start from a stored state and store every slice
(plans with checkpoints): the parent windows of both sides, with the only plane at the
entrance, at the exit, at both and in a single slice, windows that wrap and that cover
the grid, on square and long grids.

Tolerance: either holds 1e-5 against the oracle."""
import dataclasses

import numpy as np
import pytest

from tests._tiny import tiny_cfg, tiny_problem

pytestmark = pytest.mark.gpu

GRIDS = [(64, 256), (256, 64), (256, 256), (512, 64)]


def compare_windows(ny, nx, nz, planes):
    import torch
    from paper_2607_00756_amd import bip
    cfg = tiny_cfg(ny=ny, nx=nx, nz=nz, ly=ny / 8.0, lx=nx / 8.0, alpha=9e-3, theta=14e-3, s=2, scan=(2, 2))
    tp = tiny_problem(cfg, n_atoms=2 * len(planes), n_ch=1, seed=ny + nz, vscale=25.0, planes=planes * 2,
                      win_sizes=[64] * len(planes) + [12] * len(planes))
    tp.win_origin[-1] = (ny - 5, nx - 7)  # wraps both ways
    V = torch.from_numpy(tp.V).cuda()
    got = []
    for stride in (0, 1):
        plan = bip.Plan.from_config(cfg, tp.tau, tp.win_size, tp.win_origin, ckpt_stride=stride)
        plan.build_smatrix(V)
        for a, W in enumerate(tp.win_size):
            for side, n in ((1, plan.Bp1), (2, plan.Bp2)):
                out = torch.full((n, W, W), float("nan"), dtype=torch.complex64, device="cuda")
                plan.parent_windows(a, side, out)
                got.append(out.cpu().numpy())
        plan.close()
    for a, b in zip(got[:len(got) // 2], got[len(got) // 2:]):
        assert np.linalg.norm(a - b) <= 2e-5 * np.linalg.norm(b)


@pytest.mark.parametrize("ny,nx", GRIDS)
@pytest.mark.parametrize("nz,planes", [(3, [0]), (3, [2]), (4, [0, 3]), (1, [0])])
def test_starts_and_ends_match_the_stored_sweep(ny, nx, nz, planes):
    print(f"[sweep {ny} x {nx}, {nz} slices, planes {planes}]", flush=True)
    compare_windows(ny, nx, nz, planes)
