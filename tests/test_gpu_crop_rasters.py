"""Interpolation factor f > 1 on rasters whose common divisor with f is 1, 2 and 4
(the residues that are summed), with crop masks from empty to more than 64 rows or
columns (the output blocks of the two DFTs) and more scans than one 128-row tile,
against the FP64 oracle.

Tolerance: the rel-L2 1e-4 of the other f > 1 outputs."""
import dataclasses

import numpy as np
import pytest

from tests._tiny import as_oracle_problem, tiny_cfg, tiny_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("f,scan,focal", [(4, (3, 5), False), (4, (6, 68), False), (4, (1, 64), False), (2, (130, 7), False),
                                          (2, (9, 132), False), (4, (16, 10), True), (2, (25, 33), False)])
@pytest.mark.parametrize("prec_name", ["PREC_FP32", "PREC_SPLIT_BF16"])
def test_crop_rasters_match_the_oracle(f, scan, focal, prec_name):
    import torch
    from oracle import eels as E
    from paper_2607_00756_amd import bip
    cfg = dataclasses.replace(tiny_cfg(ny=64, nx=64, nz=4, ly=16.0, lx=16.0, alpha=0.03, theta=0.035, s=2, scan=scan),
                              interp_f=f, focal=focal)
    tp = tiny_problem(cfg, n_atoms=3, n_ch=2, seed=scan[0], vscale=25.0, planes=[0, 3, 1], win_sizes=[4, 12, 16])
    plan = bip.Plan.from_config(cfg, tp.tau, tp.win_size, tp.win_origin)
    V, H = torch.from_numpy(tp.V).cuda(), torch.from_numpy(tp.H).cuda()
    plan.build_smatrix(V)
    want = E.BiP(as_oracle_problem(tp)).run(mode=E.OUT_BEAMS)
    masks = [E.crop_mask(cfg, tp.tau[a], f) for a in range(3)]
    print(f"[f {f} scan {scan} focal {focal}] scans per mask {[int(m.sum()) for m in masks]}", flush=True)
    P = scan[0] * scan[1]
    prec = getattr(bip, prec_name)
    for mode, ref in ((bip.OUT_MAP, want.sum(axis=1)), (bip.OUT_BEAMS, want)):
        out = torch.full((P,) if mode == bip.OUT_MAP else (P, plan.ndet), float("nan"), dtype=torch.float32, device="cuda")
        plan.eels_signal(2, H, tp.H_off, scan, mode, prec, out)
        got = out.cpu().numpy().astype(np.float64)
        assert np.linalg.norm(got - ref) <= 1e-4 * np.linalg.norm(ref)
        assert np.all(got.reshape(P, -1)[~np.logical_or.reduce(masks)] == 0.0)
    plan.close()


@pytest.mark.parametrize("prec_name", ["PREC_FP32", "PREC_SPLIT_BF16"])
def test_more_atoms_than_partial_rows_match_the_oracle(prec_name):
    """19 atoms whose masks take one row tile each, on a raster of one: the partial rows hold 16
    atoms at a time, so the quadratic form runs in two launches that reuse them, 16 atoms and 3."""
    import torch
    from oracle import eels as E
    from paper_2607_00756_amd import bip
    scan, n = (10, 12), 19
    cfg = dataclasses.replace(tiny_cfg(ny=64, nx=64, nz=4, ly=16.0, lx=16.0, alpha=0.03, theta=0.035, s=2, scan=scan),
                              interp_f=2)
    tp = tiny_problem(cfg, n_atoms=n, n_ch=2, seed=17, vscale=25.0, planes=[a % 4 for a in range(n)],
                      win_sizes=[(4, 12, 16, 8)[a % 4] for a in range(n)])
    assert min(int(E.crop_mask(cfg, tp.tau[a], 2).sum()) for a in range(n)) > 0
    plan = bip.Plan.from_config(cfg, tp.tau, tp.win_size, tp.win_origin)
    plan.build_smatrix(torch.from_numpy(tp.V).cuda())
    out = torch.full((scan[0] * scan[1],), float("nan"), dtype=torch.float32, device="cuda")
    plan.set_profiling(True)
    plan.stage_timings(reset=True)
    plan.eels_signal(2, torch.from_numpy(tp.H).cuda(), tp.H_off, scan, bip.OUT_MAP, getattr(bip, prec_name), out)
    launches = plan.stage_timings()["det_gemm"][1]
    got = out.cpu().numpy().astype(np.float64)
    plan.close()
    want = E.BiP(as_oracle_problem(tp)).run(mode=E.OUT_MAP)
    print(f"[{n} atoms {prec_name}] {launches} launches, {np.linalg.norm(got - want) / np.linalg.norm(want):.2e}", flush=True)
    assert launches == 2
    assert np.linalg.norm(got - want) <= 1e-4 * np.linalg.norm(want)
