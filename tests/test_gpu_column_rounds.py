"""Parent sweeps whose column pass runs several rounds of columns per workgroup (more
columns in a batch than a launch takes at once), on the grids where the block
mapping changes: blocks of x that 8 divides and that it does not, and fewer columns
in the last round.  Sampled S2 parent windows against the oracle's multislice of the
same columns; complex64 sweeps of 3 slices, bar 1e-5 as for the other windows."""
import dataclasses

import numpy as np
import pytest

from tests._tiny import as_oracle_problem, tiny_cfg, tiny_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ny,nx,ly,lx,theta", [(128, 128, 16.0, 16.0, 40e-3), (128, 256, 12.0, 24.0, 44e-3),
                                              (256, 64, 30.0, 7.5, 40e-3)])
def test_many_columns_match_the_oracle(ny, nx, ly, lx, theta, monkeypatch):
    import torch
    from oracle import eels as E
    from oracle import multislice as ms
    from paper_2607_00756_amd import bip
    monkeypatch.setenv("BIP_COLUMN_BATCH", "0")  # all columns in one batch
    cfg = dataclasses.replace(tiny_cfg(ny=ny, nx=nx, nz=3, ly=ly, lx=lx, alpha=15e-3, theta=theta, s=3, scan=(2, 2)),
                              s2_exact=True)
    tp = tiny_problem(cfg, n_atoms=1, n_ch=1, W=12, seed=11, planes=[0])
    plan = bip.Plan.from_config(cfg, tp.tau, tp.win_size, tp.win_origin)
    plan.build_smatrix(torch.from_numpy(tp.V).cuda())
    out = torch.empty((plan.Bp2, 12, 12), dtype=torch.complex64, device="cuda")
    plan.parent_windows(0, 2, out)
    got = out.cpu().numpy()
    par = plan.query(bip.Q_PARENTS2)
    pick = np.unique(np.linspace(0, len(par) - 1, 40).astype(int))
    prob = as_oracle_problem(tp)
    y, x = prob.window(0)
    want = ms.s2_windows(cfg, par[pick], prob.T, prob.P, [(0, y, x)])[0] * E.carrier(cfg, par[pick], y, x, +1)
    plan.close()
    assert np.linalg.norm(got[pick] - want) <= 1e-5 * np.linalg.norm(want)


@pytest.mark.parametrize("ny,nx,ly,lx,theta", [(128, 128, 16.0, 16.0, 40e-3), (128, 64, 16.0, 8.0, 60e-3)])
def test_many_columns_of_checkpointed_sweeps_match_the_oracle(ny, nx, ly, lx, theta, monkeypatch):
    """Grids of sides up to 128 run the column pass in plans with checkpoints only (without, as in
    the first case above, a sweep is one launch).  Four and two blocks of x; every column is checked."""
    import torch
    from oracle import eels as E
    from oracle import multislice as ms
    from paper_2607_00756_amd import bip
    monkeypatch.setenv("BIP_COLUMN_BATCH", "0")
    cfg = dataclasses.replace(tiny_cfg(ny=ny, nx=nx, nz=2, ly=ly, lx=lx, alpha=15e-3, theta=theta, s=3, scan=(2, 2)),
                              s2_exact=True)
    tp = tiny_problem(cfg, n_atoms=1, n_ch=1, W=8, seed=12, planes=[0])
    plan = bip.Plan.from_config(cfg, tp.tau, tp.win_size, tp.win_origin, ckpt_stride=1)
    at_once = 15 * torch.cuda.get_device_properties(0).multi_processor_count // (nx // 32)  # of a launch, 60 waves a CU
    assert plan.Bp2 > at_once and plan.Bp2 % at_once
    plan.build_smatrix(torch.from_numpy(tp.V).cuda())
    out = torch.full((plan.Bp2, 8, 8), float("nan"), dtype=torch.complex64, device="cuda")
    plan.parent_windows(0, 2, out)
    got, par = out.cpu().numpy(), plan.query(bip.Q_PARENTS2)
    plan.close()
    prob = as_oracle_problem(tp)
    y, x = prob.window(0)
    want = ms.s2_windows(cfg, par, prob.T, prob.P, [(0, y, x)])[0] * E.carrier(cfg, par, y, x, +1)
    print(f"[{ny} x {nx}] {len(par)} columns, {at_once} at once", flush=True)
    assert np.linalg.norm(got - want) <= 1e-5 * np.linalg.norm(want)
