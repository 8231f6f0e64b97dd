"""Launches that the profiled stages count for the parent sweeps, against the benchmark's own
account of them (its rates divide by what each stage moves): batches of one side, of both, planes
that let the sides share some slices and none, S2 streamed, and whole sweeps in one launch."""
import pytest

from tests._tiny import tiny_cfg, tiny_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ny,nx,batch,planes,window_gb", [
    (64, 256, 0, [0, 4], 0.0), (64, 256, 13, [1, 3], 0.0), (256, 64, 20, [2], 0.0), (64, 256, 9, [4], 0.0),
    (256, 64, 13, [0, 2, 4], 1e-5), (128, 128, 13, [0, 4], 0.0), (128, 64, 13, [0, 2, 4], 1e-5)])
def test_stage_launches(ny, nx, batch, planes, window_gb, monkeypatch):
    import bench
    import torch
    from paper_2607_00756_amd import bip
    monkeypatch.setenv("BIP_COLUMN_BATCH", str(batch))
    cfg = tiny_cfg(ny=ny, nx=nx, nz=5, ly=ny / 8.0, lx=nx / 8.0, alpha=12e-3, theta=18e-3, s=2, scan=(3, 4))
    tp = tiny_problem(cfg, n_atoms=len(planes), n_ch=1, seed=3, planes=planes, win_sizes=[12] * len(planes))
    plan = bip.Plan.from_config(cfg, tp.tau, tp.win_size, tp.win_origin, s2_window_gb=window_gb)
    plan.set_profiling(True)
    plan.build_smatrix(torch.from_numpy(tp.V).cuda())
    out = torch.empty(12, dtype=torch.float32, device="cuda")
    plan.eels_signal(1, torch.from_numpy(tp.H).cuda(), tp.H_off, cfg.scan, bip.OUT_MAP, bip.PREC_FP32, out)
    stages = plan.stage_timings()
    columns, segments = (int(v) for v in plan.query(bip.Q_SCALARS)[2:4])
    want = bench.sweep_passes(plan.Bp1, plan.Bp2, ny, nx, cfg.nz, max(planes), min(planes), columns, segments)
    print(f"[{ny} x {nx}] {plan.Bp1} + {plan.Bp2} columns, batches of {columns}, {segments} segments: {want}", flush=True)
    plan.close()
    assert (segments > 0) == (window_gb > 0)
    assert {st: n for st, (_, n) in stages.items() if st in want} == {st: n for st, (n, _) in want.items()}
