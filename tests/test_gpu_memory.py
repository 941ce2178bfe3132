"""Device memory that runs out: a call that fails with GPF_ERR_NOMEM leaves a
context that can be used on, with nothing held that the call took in vain."""
import numpy as np
import pytest

from gpu_helpers import STATE
from inputs import busy_config, random_state

pytestmark = pytest.mark.gpu


class FailAt:
    """memory_limit of which allocation number `at` (1, 2, ... since it was last
    set; 0: none) does not fit"""

    def __init__(self):
        self.at = self.seen = 0

    def fail(self, at):
        self.at, self.seen = at, 0

    def __lt__(self, wanted):
        self.seen += 1
        return self.seen == self.at


def _sim(cfg, precision, limit=None):
    from paper_2608_26908_amd.gpf import Sim
    st = random_state(cfg, 5)
    s = Sim(cfg, precision=precision, memory_limit=limit)
    for k in STATE:
        s.write(k, st[k])
    return s


@pytest.mark.parametrize("kind,n", [("binary2d", [48, 10]), ("ternary3d_nc2", [16, 6, 5])])
def test_adjoint_after_a_failed_allocation(kind, n):
    """every allocation of a sweep fails once: the call reports it (or, where
    only the second tape did not fit, goes on with one), and the next call
    computes what a context with memory to spare computes"""
    from paper_2608_26908_amd.gpf import GPFError
    cfg, names = busy_config(kind, n), ["delta", "tau_pf", "D"]
    seed = np.cos(np.arange(cfg["N"] * int(np.prod(n)))).reshape([cfg["N"]] + n[::-1])

    def recorded(limit=None):
        s = _sim(cfg, "fp64", limit)
        s.record(3)
        s.step(5)
        return s

    a = recorded()
    want = a.adjoint(seed, names)
    lam = a.adjoint_state("f")
    a.close()
    failed, at = 0, 0
    while True:
        at += 1
        limit = FailAt()
        b = recorded(limit)
        limit.fail(at)
        try:
            got = b.adjoint(seed, names)
        except GPFError as e:
            assert e.code == -3
            failed += 1
            limit.fail(0)
            got = b.adjoint(seed, names)
        assert np.array_equal(got, want), at
        assert np.array_equal(b.adjoint_state("f"), lam), at
        b.close()
        if 0 < limit.at > limit.seen:  # no allocation of that number
            break
    assert failed >= 10


def test_failed_checkpoint():
    """a checkpoint that does not fit is not half kept, and a sweep that would
    start from it is refused"""
    from paper_2608_26908_amd.gpf import GPFError
    cfg, limit = busy_config("binary2d", [48, 10]), FailAt()
    s = _sim(cfg, "fp64", limit)
    start = s.device_bytes
    for at in range(1, 5):  # phi, mu, U, f
        limit.fail(at)
        with pytest.raises(GPFError) as e:
            s.record(3)
        assert e.value.code == -3 and s.device_bytes == start
    limit.fail(0)
    s.record(3)
    s.step(2)
    held = s.device_bytes
    for at in range(1, 5):
        limit.fail(at)
        with pytest.raises(GPFError) as e:
            s.step(1)
        assert e.value.code == -3 and s.device_bytes == held
        if at < 4:  # the same step once more
            s.step_index = s.step_index - 1
    limit.fail(0)
    s.step(1)
    with pytest.raises(GPFError) as e:
        s.adjoint(np.ones((2, 10, 48)), ["D"])
    assert e.value.code == -6
    s.close()


@pytest.mark.parametrize("kind,n,over", [
    ("ternary3d_nc2", [32, 24, 20], dict(delta=[[0] * 3] * 3)),  # three dimensions without anisotropy
    ("binary2d", [160, 64], {}),                                 # a 2D reverse step in one launch
])
def test_sweep_holds_what_it_uses(kind, n, over):
    """without anisotropy, and in the one-launch reverse step, no values per
    face are stored, so no memory is held for them"""
    cfg, K = busy_config(kind, n, **over), 3
    D, N, nc, Q = cfg["dim"], cfg["N"], cfg["nc"], 9 if cfg["dim"] == 2 else 19
    s = _sim(cfg, "fp32")
    s.record(K)
    s.step(2 * K - 1)
    before = s.device_bytes
    s.adjoint(np.ones([N] + n[::-1]), ["D"])
    # values per cell: two adjoint states, what the LBM reverse leaves (twice in one launch) and the seeds; two tapes
    # of K - 1 states and two sets of populations
    comps = 2 * (N + nc + D + Q) + (2 * (1 + nc) if D == 2 else 1 + nc + N) + 2 * ((K - 1) * (N + nc + D + 1) + 2 * Q)
    cells = int(np.prod(n))
    # bytes per cell: seed flags and the tapes' active sets; running sums of the gradients, 48 bytes per 256 cells and
    # kernel (D + 3 of them), or per 128, in 8 parts rounded up each, and 256 slices
    flags = (1 if D == 3 else 0) + 2 * (K - 1)
    sums = 48 * ((D + 3) * (cells / 256 + 8) + cells / 128 + 64 + 257) + 2 * n[1] * (n[2] if D == 3 else 1)
    assert s.device_bytes - before <= 4 * comps * cells + flags * cells + sums
    s.close()
