"""Contractions at the edges of their tiles and splits, against the FP64 oracle.

Window pixel counts on both sides of 64- and 128-row tile edges, one atom (the
Gram matrix and the quadratic form split over K segments) and several, narrow
outputs of the per-beam products (job groups with a slice each) and a plan with
checkpoints (contractions run whole).

Tolerances: FP32 operands carry 2^-24 and the parent sweeps about 1e-6, so maps
and beams are held to 1e-5; split operands carry 2^-17 per factor (hi + lo
bf16), four factors into an intensity, so 4 x 2^-17 = 3e-5 with the same
allowance for the sweeps."""
import numpy as np
import pytest

from tests._tiny import as_oracle_problem, tiny_cfg, tiny_problem

pytestmark = pytest.mark.gpu

TOL = {0: 1e-5, 1: 4e-5}
CASES = [
    # win sizes, channels, scan, planes
    ([8], 1, (3, 5), [1]),                 # 64 pixels: one 64-row tile exactly
    ([12], 3, (8, 16), [2]),               # 144: a 128-row tile and a remainder
    ([16, 20], 2, (9, 15), [0, 2]),        # 256 = two tiles; 400 = 6.25 of 64 rows
    ([4, 24, 8], 9, (12, 12), [1, 1, 2]),  # 16 .. 576 pixels in one launch, nine channels
    ([32], 2, (4, 4), [1]),                # 1024 pixels, 16 scans: far fewer tiles than compute units
]


def run(case, out_name, prec, ckpt=0):
    import torch
    from oracle import eels as E
    from paper_2607_00756_amd import bip
    wins, n_ch, scan, planes = case
    cfg = tiny_cfg(ny=64, nx=64, nz=3, ly=8.0, lx=8.0, s=2, scan=scan)
    tp = tiny_problem(cfg, n_atoms=len(wins), n_ch=n_ch, seed=len(wins) + wins[0], planes=planes, win_sizes=wins)
    mode = {"map": bip.OUT_MAP, "beams": bip.OUT_BEAMS, "direct": bip.OUT_MAP_DIRECT}[out_name]
    plan = bip.Plan.from_config(cfg, tp.tau, tp.win_size, tp.win_origin, ckpt_stride=ckpt)
    P = scan[0] * scan[1]
    out = torch.empty((P, plan.ndet) if out_name == "beams" else (P,), dtype=torch.float32, device="cuda")
    plan.build_smatrix(torch.from_numpy(tp.V).cuda())
    plan.eels_signal(n_ch, torch.from_numpy(tp.H).cuda(), tp.H_off, scan, mode, prec, out)
    want = E.BiP(as_oracle_problem(tp)).run(mode=E.OUT_BEAMS if out_name == "beams" else E.OUT_MAP)
    got = out.cpu().numpy().astype(np.float64)
    plan.close()
    return float(np.linalg.norm(got - want) / np.linalg.norm(want))


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("out_name", ["map", "direct", "beams"])
@pytest.mark.parametrize("case", CASES, ids=["w8", "w12", "w16-20", "w4-24-8", "w32"])
def test_splits_match_the_oracle(case, out_name, prec):
    assert run(case, out_name, prec) <= TOL[prec]


@pytest.mark.parametrize("prec", [0, 1])
def test_whole_contractions_match_the_oracle(prec):
    assert run(CASES[2], "map", prec, ckpt=1) <= TOL[prec]


@pytest.mark.parametrize("prec", [2, 3])
@pytest.mark.parametrize("out_name", ["direct", "beams"])
@pytest.mark.parametrize("case", CASES, ids=["w8", "w12", "w16-20", "w4-24-8", "w32"])
def test_single_16_bit_products_match_the_oracle(case, out_name, prec):
    """BF16 and FP16 operands carry 2^-9 and 2^-12, four factors into an intensity; held to the
    bounds of the tiny specimen's outputs in these precisions."""
    assert run(case, out_name, prec) <= {2: 3e-2, 3: 1e-3}[prec]


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("focal", [False, True])
@pytest.mark.parametrize("wins,n_ch,scan", [([8], 34, (5, 3)), ([4, 12], 7, (1, 2)), ([8], 2, (3, 64))])
def test_channel_groups_match_the_oracle(wins, n_ch, scan, focal, prec):
    """U_n written by several workgroups of channels: more groups than channels wanted, groups of
    unequal size, few groups; tolerances as above."""
    import dataclasses

    import torch
    from oracle import eels as E
    from paper_2607_00756_amd import bip
    cfg = dataclasses.replace(tiny_cfg(ny=64, nx=64, nz=3, ly=8.0, lx=8.0, s=2, scan=scan), focal=focal)
    tp = tiny_problem(cfg, n_atoms=len(wins), n_ch=n_ch, seed=n_ch, vscale=25.0, planes=[2, 1][:len(wins)], win_sizes=wins)
    plan = bip.Plan.from_config(cfg, tp.tau, tp.win_size, tp.win_origin)
    plan.build_smatrix(torch.from_numpy(tp.V).cuda())
    out = torch.full((scan[0] * scan[1], plan.ndet), float("nan"), dtype=torch.float32, device="cuda")
    plan.eels_signal(n_ch, torch.from_numpy(tp.H).cuda(), tp.H_off, scan, bip.OUT_BEAMS, prec, out)
    got = out.cpu().numpy().astype(np.float64)
    plan.close()
    want = E.BiP(as_oracle_problem(tp)).run(mode=E.OUT_BEAMS)
    assert np.linalg.norm(got - want) <= TOL[prec] * np.linalg.norm(want)
