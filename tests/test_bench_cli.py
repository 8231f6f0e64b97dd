"""Host-side checks of bench.py: the one-GPU guard and the committed HBM
traffic record it reads."""
from __future__ import annotations

import json
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_more_than_one_gpu_is_refused():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"],
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 2
    msg = json.loads(r.stdout.strip().splitlines()[-1])
    assert msg["n_gpus"] == 2 and "one GPU" in msg["error"]


def test_traffic_record_is_consistent():
    """The counter record of the dominant pass: its bytes per launch lie
    within a few percent of the algorithmic 16 G bytes per column of the
    recorded batch (the state read once and written once), and the record
    names the sources it was taken with."""
    t = json.load(open(os.path.join(ROOT, "profiles", "hbm_traffic.json")))
    assert t["stage"] == "s2_row" and t["column_batch"] > 0
    G = 256 * 256
    n_cols = 2233 / -(-2233 // t["column_batch"])  # mean columns per launch of the S2 sweep
    alg = 16.0 * G * n_cols
    assert abs(t["bytes_per_launch"] / alg - 1.0) < 0.05
    for src in t["sources_sha256"]:
        assert os.path.exists(os.path.join(ROOT, src))


def _passes(**kw):
    sys.path.insert(0, ROOT)
    import bench
    plan = dict(bp1=61, bp2=177, ny=256, nx=256, nz=50, i_max=49, i_min=0, batch=448, segments=0)
    return bench.sweep_passes(**{**plan, **kw})


def test_sweep_stages_are_credited_with_their_own_columns():
    """Launches and columns of the sweeps' stages by hand: both sides in one batch, side by side for
    all slices but the last, which is each side's own; a batch of S1's last columns and S2's first; sides
    apart; streamed S2; one launch of whole sweeps.  Shared or not, a column passes as often."""
    assert _passes() == {"s1_row": [1, 61], "s1_col": [0, 0], "s2_row": [49 + 1, 49 * 238 + 177],
                         "s2_col": [49, 49 * 238]}
    # 100 + 70 columns, batches of 60: 57, 57, 56; the second holds 43 of S1 and 14 of S2
    got = _passes(bp1=100, bp2=70, nz=5, i_max=3, i_min=2, batch=60)
    both = 2  # min(i_max, nz - 1 - i_min)
    assert got == {"s1_row": [4 + 2, 4 * 57 + 2 * 43], "s1_col": [3 + 1, 3 * 57 + 43],
                   "s2_row": [both + 1 + 3, both * 57 + 14 + 3 * 56], "s2_col": [both + 2, both * 57 + 2 * 56]}
    for batch, segments in ((448, 0), (100, 0), (100, 3), (1, 0), (10 ** 9, 0), (10 ** 9, 2)):
        for i_max, i_min in ((49, 0), (20, 20), (0, 0), (49, 49), (7, 3)):
            n = _passes(bp1=447, bp2=1003, i_max=i_max, i_min=i_min, batch=batch, segments=segments)
            rows, cols = (n["s1_" + k][1] + n["s2_" + k][1] for k in ("row", "col"))
            assert rows == 447 * (i_max + 1) + 1003 * (50 - i_min)
            assert cols == 447 * i_max + 1003 * (49 - i_min)
            if segments or batch == 1:
                assert n["s1_row"][1] == 447 * (i_max + 1)
    assert _passes(ny=128, nx=64)["s2_row"] == [1, 0]
