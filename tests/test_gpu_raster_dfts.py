"""The raster DFTs by halves (outputs o and S - o from one set of products) at sides where
their rows and blocks change: 1 and 2, odd and even, one row off 32 and 64, several output
groups; the map's operand and the per-beam one.  Against the FP64 oracle at the library's
bar of 1e-4 rel-L2."""
import numpy as np
import pytest

from tests._tiny import as_oracle_problem, tiny_cfg, tiny_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scan", [(1, 2), (2, 1), (3, 4), (31, 32), (33, 16), (5, 63), (66, 2), (2, 129), (193, 3), (3, 256)])
def test_rasters_match_the_oracle(scan):
    import torch
    from oracle import eels as E
    from paper_2607_00756_amd import bip
    cfg = tiny_cfg(ny=64, nx=64, nz=3, ly=16.0, lx=16.0, alpha=20e-3, theta=12e-3, s=2, scan=scan)
    tp = tiny_problem(cfg, n_atoms=2, n_ch=2, seed=scan[0], vscale=25.0, planes=[2, 1], win_sizes=[4, 12])
    plan = bip.Plan.from_config(cfg, tp.tau, tp.win_size, tp.win_origin)
    V, H = torch.from_numpy(tp.V).cuda(), torch.from_numpy(tp.H).cuda()
    plan.build_smatrix(V)
    want = E.BiP(as_oracle_problem(tp)).run(mode=E.OUT_BEAMS)
    P = scan[0] * scan[1]
    print(f"[rasters {scan}]", flush=True)
    for mode, ref in ((bip.OUT_MAP, want.sum(axis=1)), (bip.OUT_BEAMS, want)):
        for prec in (bip.PREC_FP32, bip.PREC_SPLIT_BF16):
            out = torch.empty((P,) if mode == bip.OUT_MAP else (P, plan.ndet), dtype=torch.float32, device="cuda")
            plan.eels_signal(2, H, tp.H_off, scan, mode, prec, out)
            got = out.cpu().numpy().astype(np.float64)
            assert np.linalg.norm(got - ref) <= 1e-4 * np.linalg.norm(ref)
    plan.close()
