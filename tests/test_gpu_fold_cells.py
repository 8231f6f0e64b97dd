"""The residue fold where its split over waves changes: rasters of one cell (every beam
in one), of more cells than beams (most of them empty), of one cell more than an LDS
chunk of 64 and of several chunks, and no more beams than waves; with and without rows
of more than six weights (hex parents).  Against the FP64 oracle, at the library's own
bar of 1e-4 rel-L2."""
import dataclasses

import numpy as np
import pytest

from tests._tiny import as_oracle_problem, tiny_cfg, tiny_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scan", [(1, 1), (2, 3), (3, 65), (41, 43), (2, 131), (64, 1)])
@pytest.mark.parametrize("alpha,parents", [(1.6e-3, "lattice"), (8e-3, "lattice"), (25e-3, "lattice"), (25e-3, "hex")])
def test_fold_matches_the_oracle(scan, alpha, parents):
    import torch
    from oracle import eels as E
    from paper_2607_00756_amd import bip
    cfg = dataclasses.replace(tiny_cfg(ny=64, nx=64, nz=3, ly=16.0, lx=16.0, alpha=alpha, theta=12e-3, s=2, scan=scan),
                              parents=parents, n_radial=3, n_angular=6)
    tp = tiny_problem(cfg, n_atoms=2, n_ch=2, seed=scan[1], vscale=25.0, planes=[2, 0], win_sizes=[4, 12])
    plan = bip.Plan.from_config(cfg, tp.tau, tp.win_size, tp.win_origin)
    out = torch.empty((scan[0] * scan[1],), dtype=torch.float32, device="cuda")
    plan.build_smatrix(torch.from_numpy(tp.V).cuda())
    plan.eels_signal(2, torch.from_numpy(tp.H).cuda(), tp.H_off, scan, bip.OUT_MAP, bip.PREC_FP32, out)
    got = out.cpu().numpy().astype(np.float64)
    want = E.BiP(as_oracle_problem(tp)).run(mode=E.OUT_MAP)
    print(f"[fold scan {scan} {plan.B} beams {parents}]", flush=True)
    plan.close()
    assert np.linalg.norm(got - want) <= 1e-4 * np.linalg.norm(want)
