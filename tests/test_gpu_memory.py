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
