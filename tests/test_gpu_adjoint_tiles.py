"""The one-launch reverse step of small 2D grids at the edges of its 16 x 8
tiles: one cell short of, equal to and one past a tile along each axis, several
tiles, and grids narrower than the tile's halo, with walls and periodic axes
(the halo then wraps onto the tile's own cells, several times on the smallest
ones).

<w, J v> from the oracle's complex-step tangent against <J^T w, v>, FP64, for
every state field.  Both sides round at about 1e-16 of the sum of their terms'
magnitudes per operation; 1e-9 of that sum is the bar of the other dot-product
tests."""
import numpy as np
import pytest

from gpu_helpers import STATE, gpu_from, oracle_from
from inputs import busy_config, random_state

pytestmark = pytest.mark.gpu

GRIDS = [("binary2d", [15, 7], [0, 0, 1]), ("binary2d", [16, 8], [1, 1, 1]), ("ternary2d", [17, 9], [1, 0, 1]),
         ("ternary2d_nc2", [33, 8], [0, 1, 1]), ("ternary2d_nc2", [16, 25], [1, 1, 1]), ("binary2d", [2, 3], [1, 1, 1]),
         ("ternary2d", [3, 1], [0, 0, 1]), ("ternary2d_nc2", [1, 9], [1, 1, 1]), ("binary2d", [50, 2], [0, 1, 1]),
         # the last size with one launch in FP64 and the first with three
         ("binary2d", [384, 256], [1, 0, 1]), ("binary2d", [385, 256], [1, 0, 1])]


@pytest.mark.parametrize("kind,n,periodic", GRIDS)
@pytest.mark.parametrize("steps,K", [(5, 3), (3, 1)])
def test_dot_product_at_tile_edges(oracle, kind, n, periodic, steps, K):
    aniso = dict(delta=[[0, 0, 0.04], [0, 0, 0.03], [0.04, 0.03, 0]]) if "ternary" in kind else {}
    _dot_product(oracle, busy_config(kind, n, periodic=periodic, **aniso), steps, K)


def test_dot_product_two_phases_without_anisotropy(oracle):
    _dot_product(oracle, busy_config("binary2d", [33, 17], delta=[[0, 0], [0, 0]]), 5, 3)


@pytest.mark.parametrize("kind,n", [("ternary2d", [160, 160]), ("ternary2d_nc2", [161, 160])])
def test_dot_product_at_the_limit_of_three_phases(oracle, kind, n):
    """the last size with one launch in FP64 and the first with three"""
    _dot_product(oracle, busy_config(kind, n, delta=[[0, 0, 0.04], [0, 0, 0.03], [0.04, 0.03, 0]]), 5, 3)


def test_one_tape_bitwise():
    """a second tape that does not fit: the segments' ends are reversed by the
    same launches, so gradients and adjoint state keep their bits"""
    cfg = busy_config("binary2d", [48, 40])
    st = random_state(cfg, 5)
    steps, K, names = 14, 4, ["delta", "tau_pf", "D"]
    from paper_2608_26908_amd.gpf import Sim

    def sim(**kw):
        s = Sim(cfg, precision="fp64", **kw)
        for k in STATE:
            s.write(k, st[k])
        return s

    a = sim()
    a.record(K)
    a.step(steps)
    seed = np.cos(np.arange(2 * 48 * 40)).reshape(a.read("phi").shape)
    ga = a.adjoint(seed, names)
    la = {f: a.adjoint_state(f) for f in ("phi", "mu", "u", "f")}
    two = a.device_bytes
    tape = ((K - 1) * (2 + 1 + 2 + 1) + 2 * 9) * 48 * 40 * 8
    a.close()
    b = sim(memory_limit=two - tape // 2)
    b.record(K)
    b.step(steps)
    assert np.array_equal(ga, b.adjoint(seed, names))
    assert b.device_bytes <= two - tape + 4096
    for f in la:
        assert np.array_equal(la[f], b.adjoint_state(f)), f
    b.close()


def _dot_product(oracle, cfg, steps, K):
    st = random_state(cfg, 13)
    g = gpu_from(cfg, st, "fp64")
    g.record(K)
    g.step(steps)
    rng = np.random.default_rng(8)
    w = rng.standard_normal((cfg["N"],) + g.shape)
    g.adjoint(w, [])
    o = oracle_from(cfg, st)
    for field in ("phi", "mu", "u", "f"):
        lam = g.adjoint_state(field)
        v = rng.standard_normal(lam.shape)
        t = o.tangent_cs(steps, field, v, "phi")
        lhs, rhs = float((w * t).sum()), float((lam * v).sum())
        size = max(float(np.abs(w * t).sum()), float(np.abs(lam * v).sum()), 1e-30)
        assert abs(lhs - rhs) <= 1e-9 * size, (field, lhs, rhs)
