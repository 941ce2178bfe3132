"""The bulk history on 2D grids above the one-launch limit (3 MiB per
component), where a step is k_phi and k_mulbm: k_phi checks each 64 x 4 tile's
neighbours and skips the tile, or leaves its bulk cells unstored, and k_mulbm
takes phi^n from phi^{n+1} where a tile was left bulk.  Stepping with the
history gives bit for bit the state of stepping with the history voided after
every step (a write of the same state)."""
import numpy as np
import pytest

from gpu_helpers import STATE
from paper_2608_26908_amd.workloads import scaled

pytestmark = pytest.mark.gpu

ONE_LAUNCH_BYTES = 3 << 20


@pytest.mark.parametrize("name,n,precision,over", [
    # a moving front of lamellae, tiles filled
    ("eutectic2d", [1024, 512], "fp64", {}),
    # ragged along x (1030 = 16 tiles and 6 cells) and y (810), the seed across the periodic faces of both axes:
    # wrapped neighbour tiles in the skip decision
    ("dendrite2d", [1030, 810], "fp32", dict(periodic=[1, 1], init_center=[1.0, 808.5])),
    # four phases, walls along y, ragged along x only
    ("eutectic4", [1000, 900], "fp32", {})])
def test_bulk_history_skip_2d_is_bitwise(name, n, precision, over):
    from paper_2608_26908_amd.gpf import Sim
    assert n[0] * n[1] * (8 if precision == "fp64" else 4) > ONE_LAUNCH_BYTES
    cfg = scaled(name, n, **over)
    a, b = Sim(cfg, precision=precision), Sim(cfg, precision=precision)
    steps = 60
    a.step(steps)
    for _ in range(steps):
        b.step(1)
        b.write("phi", b.read("phi"))  # voids the history
    phi = a.read("phi")
    # bulk tiles and interface tiles are both there
    assert (phi.max(axis=0) == 1.0).mean() > 0.5 and (phi.max(axis=0) < 1.0).any()
    for k in STATE:
        assert np.array_equal(a.read(k), b.read(k)), k
    a.close()
    b.close()


def test_bulk_history_of_a_single_row_is_bitwise():
    """long single rows step in two launches below that limit too"""
    from paper_2608_26908_amd.gpf import Sim
    cfg = scaled("dendrite2d", [200001, 1], init_center=[100000.0, 0.0])
    a, b = Sim(cfg, precision="fp32"), Sim(cfg, precision="fp32")
    a.step(40)
    for _ in range(40):
        b.step(1)
        b.write("phi", b.read("phi"))  # voids the history
    for k in STATE:
        assert np.array_equal(a.read(k), b.read(k)), k
    a.close()
    b.close()
