"""Focal maps at the window sizes where the forward step's tiling changes (enlarged
windows of 8 to 128 pixels, sides off the 16-pixel blocks, several in one launch),
against the FP64 oracle.

Tolerance: the FP32 map holds 1e-5 without the focal step; the two window steps
are sums of at most 128 FP32 products each (4 products a rounding), which adds
less than 1e-6."""
import numpy as np
import pytest

from tests._tiny import as_oracle_problem, tiny_cfg, tiny_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("wins", [[4], [12], [20], [36], [64], [8, 28, 16]], ids=lambda w: "-".join(map(str, w)))
@pytest.mark.parametrize("out_name", ["map", "beams"])
def test_focal_windows_match_the_oracle(wins, out_name):
    import dataclasses

    import torch
    from oracle import eels as E
    from paper_2607_00756_amd import bip
    cfg = dataclasses.replace(tiny_cfg(ny=128, nx=128, nz=4, ly=16.0, lx=16.0, alpha=12e-3, theta=20e-3, s=2, scan=(5, 6)),
                              focal=True)
    tp = tiny_problem(cfg, n_atoms=len(wins), n_ch=2, seed=wins[0], planes=[3 - i for i in range(len(wins))],
                      win_sizes=wins)
    plan = bip.Plan.from_config(cfg, tp.tau, tp.win_size, tp.win_origin)
    mode, omode = (bip.OUT_MAP, E.OUT_MAP) if out_name == "map" else (bip.OUT_BEAMS, E.OUT_BEAMS)
    out = torch.empty((30,) if out_name == "map" else (30, plan.ndet), dtype=torch.float32, device="cuda")
    plan.build_smatrix(torch.from_numpy(tp.V).cuda())
    plan.eels_signal(2, torch.from_numpy(tp.H).cuda(), tp.H_off, cfg.scan, mode, bip.PREC_FP32, out)
    want = E.BiP(as_oracle_problem(tp)).run(mode=omode)
    got = out.cpu().numpy().astype(np.float64)
    plan.close()
    assert np.linalg.norm(got - want) <= 1.1e-5 * np.linalg.norm(want)
