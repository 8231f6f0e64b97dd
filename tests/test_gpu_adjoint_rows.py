"""Reverse sweeps on wide grids (each row length has its own kernel), with column
batches that give a workgroup one and several columns in turn (a launch has no more
workgroups a row than columns) and that leave a short one, against the FP64 oracle gradient.  Bar: rel-L2 1e-3, as for the other gradients."""
import numpy as np
import pytest

from oracle import adjoint as A
from oracle import eels as E
from tests._tiny import as_oracle_problem, tiny_cfg, tiny_problem
from tests.gpu_helpers import rel_l2
from tests.test_gpu_backward import _gpu_grad

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,batch", [(128, 1), (128, 33), (512, None), (512, 5), (1024, None)])
def test_wide_rows_match_the_oracle_gradient(nx, batch):
    cfg = tiny_cfg(ny=64, nx=nx, nz=3, ly=8.0, lx=nx / 8.0, alpha=9e-3, theta=14e-3, s=3, scan=(3, 5))
    tp = tiny_problem(cfg, n_atoms=2, n_ch=2, seed=nx, vscale=25.0, planes=[2, 0], win_sizes=[8, 12])
    prob = as_oracle_problem(tp)
    r = np.random.default_rng(3)
    I0 = E.BiP(prob).run(mode=E.OUT_MAP)
    It = I0 * (1.0 + 0.3 * r.normal(size=I0.shape))
    ref = A.MapGradient(prob).run(It)
    print(f"[adjoint rows nx {nx} batch {batch}]", flush=True)
    dV, gH, _ = _gpu_grad(cfg, tp, 2.0 * (ref["I"] - It), E.RECON_MAGNITUDE, batch=batch)
    gH_ref = np.concatenate([ref["gH"][a].ravel() for a in range(2)])
    assert rel_l2(dV, ref["dV"]) < 1e-3
    assert np.linalg.norm(gH - gH_ref) < 1e-3 * np.linalg.norm(gH_ref)


@pytest.mark.parametrize("nx,batch", [(128, 7), (1024, 45)])
def test_batches_of_a_few_columns_match_the_oracle_gradient(nx, batch):
    """15 and 31 columns in batches of 5 and of 7 with a short last one; more than the 32 groups
    of a launch in a batch of several, so that some workgroups have two columns and some one."""
    test_wide_rows_match_the_oracle_gradient(nx, batch)
