"""Exchange between workers in the split step kernels, in phases (few workers) and in one launch whose workgroups wait for each
other's messages (192 workers and more, exchange every fourth step or less often)."""
import numpy as np
import pytest

from tests.test_parity_gpu import B, make_data, to_dev  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


def context(B, X, k, W, b, E, **kw):
    g = B.ASGD(k, X.shape[1], W, b, 0.05, E=E, kernel=B.KERNEL_GENERIC, **kw)
    g.load_shards(to_dev(X))
    return g


@pytest.mark.parametrize("W,tune", [(6, 2), (200, 0)])
@pytest.mark.parametrize("parts", [1, 3])
def test_a_message_is_gone_once_it_was_looked_at(B, W, tune, parts):
    # ... whatever mode and interval the next run has; both may change between two runs
    k, d, b, E = 20, 13, 100, 4
    X = make_data(W * (3 * b + 5), d, k, seed=3)
    g = context(B, X, k, W, b, E, tune=tune, buffers=2, parts=parts)
    g.run_steps(10)                                     # rounds 0 and 1 were sent and merged
    assert g.stats().received == 2 * 2 * W
    g.set_option(B.OPT_MODE, B.MODE_FREE_RUNNING)
    values, rounds = g.get_exchange()
    assert np.all(rounds == -1) and np.all(values == 0)
    before = g.stats().received
    g.run_steps(1)
    g.set_option(B.OPT_EXCHANGE_EVERY, 11)             # step 11 is a merge point of this interval
    g.run_steps(1)
    assert g.stats().received == before
    h = context(B, X, k, W, b, E, tune=tune, buffers=2, parts=parts)
    h.run_steps(10)
    h.set_option(B.OPT_EXCHANGE_EVERY, 5)               # step 10 is merge point 2 and looks for messages of round 1
    h.run_steps(1)
    assert h.stats().received == 2 * 2 * W


FORMS = [  # kernel, k, d, W, b, E: shapes of the one launch, one workgroup per worker, and of two rounds of workers
    ("GENERIC", 20, 13, 200, 100, 4), ("GENERIC", 40, 150, 192, 96, 5), ("MFMA", 40, 20, 256, 512, 4), ("MFMA", 500, 24, 400, 64, 4),
]


@pytest.mark.parametrize("kernel,k,d,W,b,E", FORMS)
@pytest.mark.parametrize("refuse", [1])
def test_a_refused_launch_becomes_several(B, kernel, k, d, W, b, E, refuse):
    """Refused by the runtime: the run is done in phases, which need no workgroups resident together."""
    X = make_data(W * max(2 * b + 5, k), d, k, seed=3)
    res = []
    for value in (0, refuse):
        g = B.ASGD(k, d, W, b, 0.05, E=E, kernel=getattr(B, "KERNEL_" + kernel))
        g.set_option(B.OPT_REFUSE_ONE_LAUNCH, value)
        g.load_shards(to_dev(X))
        g.run_steps(2 * E + 2)
        g.run_steps(1)
        res.append((g.get_state(), g.worker_counters(), g.stats()))
    (wa, ca, sa), (wb, cb, sb) = res
    assert sa.launches == 1 and sb.launches > 1 and sb.steps == 2 * E + 3
    assert np.array_equal(ca[:, :2], cb[:, :2])
    # the same assignments; sums of several shares are rounded a few times more, the sums of Eq. 4 in another order
    assert np.abs(wa - wb).max() <= 1e-5 * np.abs(wa).max()
