"""Backward with more aperture than detector beams, where the buffers of the
reconstruction adjoints hold fewer atoms than a chunk of products, windows of
different sizes in every launch, square-lattice and hex parents (the S2 operand by
its own kernel), against the FP64 oracle gradient.  Bar: rel-L2 1e-3, as for the
other gradients."""
import dataclasses

import numpy as np
import pytest

from oracle import adjoint as A
from oracle import eels as E
from tests._tiny import as_oracle_problem, tiny_cfg, tiny_problem
from tests.gpu_helpers import rel_l2
from tests.test_gpu_backward import _gpu_grad

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("alpha,theta,wins", [(0.03, 0.01, [8, 4, 8, 12, 8]), (0.01, 0.03, [4, 16, 8]),
                                              (0.02, 0.02, [12])])
@pytest.mark.parametrize("parents,prec", [("lattice", 0), ("lattice", 1), ("hex", 0)])
def test_atoms_of_a_launch_match_the_oracle_gradient(alpha, theta, wins, parents, prec):
    cfg = dataclasses.replace(tiny_cfg(ny=64, nx=64, nz=4, ly=16.0, lx=16.0, alpha=alpha, theta=theta, s=3, scan=(5, 7)),
                              parents=parents, n_radial=3, n_angular=6)
    tp = tiny_problem(cfg, n_atoms=len(wins), n_ch=2, seed=5, vscale=25.0, planes=[(3 * i + 1) % 4 for i in range(len(wins))],
                      win_sizes=wins)
    prob = as_oracle_problem(tp)
    r = np.random.default_rng(7)
    I0 = E.BiP(prob).run(mode=E.OUT_MAP)
    It = I0 * (1.0 + 0.3 * r.normal(size=I0.shape))
    dHx = r.normal(size=tp.H.shape) + 1j * r.normal(size=tp.H.shape)
    dHy = r.normal(size=tp.H.shape) + 1j * r.normal(size=tp.H.shape)
    cut = lambda d, a: d[tp.H_off[a]:tp.H_off[a + 1]].reshape(tp.n_ch, tp.win_size[a], tp.win_size[a])
    ref = A.MapGradient(prob).run(It, dH_dtau={a: (cut(dHx, a), cut(dHy, a)) for a in range(len(wins))})
    print(f"[backward atoms alpha {alpha} theta {theta} windows {wins} {parents} prec {prec}]", flush=True)
    dV, gH, tau = _gpu_grad(cfg, tp, 2.0 * (ref["I"] - It), E.RECON_MAGNITUDE, dHx, dHy, prec=prec)
    gH_ref = np.concatenate([ref["gH"][a].ravel() for a in range(len(wins))])
    assert rel_l2(dV, ref["dV"]) < 1e-3
    assert np.linalg.norm(gH - gH_ref) < 1e-3 * np.linalg.norm(gH_ref)
    assert rel_l2(tau, np.array([ref["dtau"][a] for a in range(len(wins))])) < 1e-3
