"""The FP32 Gram matrix of plans with checkpoints in small and in large tiles: few atoms
launch fewer 64 x 64 tiles than the chip has CUs and take 32 x 32, many take 64 x 64, and
an atom's cotangent dL/dH* (through G and Q) has the same bits in both; windows of one
tile, off the tile and block sizes, and of several blocks.  The small tiles against the
FP64 oracle gradient too, at the 1e-3 rel-L2 of the other gradients."""
import numpy as np
import pytest

from oracle import adjoint as A
from oracle import eels as E
from tests._tiny import as_oracle_problem, tiny_cfg, tiny_problem
from tests.test_gpu_backward import _gpu_grad

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W", [4, 8, 12, 20, 28])
def test_gram_tiles_give_the_same_bits(W):
    cfg = tiny_cfg(ny=64, nx=64, nz=3, ly=16.0, lx=16.0, alpha=0.012, theta=0.02, s=2, scan=(4, 5))
    wins = [W] + [32] * 12  # a window of 32: 144 tiles of 64 x 64
    tp = tiny_problem(cfg, n_atoms=13, n_ch=2, seed=W, vscale=25.0, planes=[i % 3 for i in range(13)], win_sizes=wins)
    r = np.random.default_rng(W)
    ibar = r.normal(size=20) * 1e-3
    print(f"[Gram tiles W {W}]", flush=True)
    many = _gpu_grad(cfg, tp, ibar, E.RECON_MAGNITUDE)[1][:tp.H_off[1]]
    one = tiny_problem(cfg, n_atoms=1, n_ch=2, seed=W, vscale=25.0, planes=[0], win_sizes=[W])
    one.V, one.tau, one.win_origin = tp.V, tp.tau[:1], tp.win_origin[:1]
    one.H = tp.H[:tp.H_off[1]]
    few = _gpu_grad(cfg, one, ibar, E.RECON_MAGNITUDE)[1]
    assert np.array_equal(few, many)
    prob = as_oracle_problem(one)
    I0 = E.BiP(prob).run(mode=E.OUT_MAP)
    ref = A.MapGradient(prob).run(I0 - ibar / 2.0)["gH"][0].ravel()
    assert np.linalg.norm(few - ref) < 1e-3 * np.linalg.norm(ref)


@pytest.mark.parametrize("W", [4, 8, 12, 20, 28])
def test_gram_tiles_give_q_the_same_bits(W):
    """dL/dV, whose S1 part comes through Q = G o conj(H) H^T of a complex H: the other atoms that
    make the launch one of 64 x 64 tiles have no transition potential and add zeros."""
    cfg = tiny_cfg(ny=64, nx=64, nz=3, ly=16.0, lx=16.0, alpha=0.012, theta=0.02, s=2, scan=(4, 5))
    tp = tiny_problem(cfg, n_atoms=13, n_ch=2, seed=W, vscale=25.0, planes=[1] + [2] * 12, win_sizes=[W] + [32] * 12)
    tp.H[tp.H_off[1]:] = 0
    one = tiny_problem(cfg, n_atoms=1, n_ch=2, seed=W, vscale=25.0, planes=[1], win_sizes=[W])
    one.V, one.tau, one.win_origin, one.H = tp.V, tp.tau[:1], tp.win_origin[:1], tp.H[:tp.H_off[1]]
    ibar = np.random.default_rng(W).normal(size=20) * 1e-3
    many, few = (_gpu_grad(cfg, p, ibar, E.RECON_MAGNITUDE)[0] for p in (tp, one))
    assert np.linalg.norm(few[0]) > 0 and np.array_equal(few, many)
