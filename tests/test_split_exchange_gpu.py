"""Exchange between workers in the split step kernels, in phases (few workers) and in one launch whose workgroups wait for each
other's messages (192 workers and more, exchange every fourth step or less often)."""
import numpy as np
import pytest

from tests.parity_rules import check_counters, rel_fro
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
    ("GENERIC", 20, 13, 200, 100, 4), ("GENERIC", 40, 150, 192, 96, 5), ("MFMA", 64, 64, 192, 512, 4), ("MFMA", 500, 24, 400, 64, 4),
]


@pytest.mark.parametrize("kernel,k,d,W,b,E", FORMS)
@pytest.mark.parametrize("refuse", [1, 2])
def test_a_refused_launch_becomes_several(B, kernel, k, d, W, b, E, refuse):
    """Refused by the runtime, or one of its workgroups finds no place: one launch per round, which needs neither."""
    X = make_data(W * max(2 * b + 5, k), d, k, seed=3)
    res = []
    for value in (0, refuse):
        g = B.ASGD(k, d, W, b, 0.05, E=E, kernel=getattr(B, "KERNEL_" + kernel))
        g.set_option(B.OPT_REFUSE_ONE_LAUNCH, value)
        g.load_shards(to_dev(X))
        g.run_steps(2 * E + 2)
        launches = g.stats().launches
        g.run_steps(1)                                  # (less than two rounds: a plain launch)
        assert g.last_run_form() == B.FORM_SPLIT_LAUNCH and g.stats().launches == 1 and g.stats().steps == 2 * E + 3
        g.run_steps(2 * E + 1)
        res.append((g.get_state(), g.worker_counters(), launches, g.stats().launches))
    assert res[0][2:] == (1, 1) and res[1][2:] == (3, 3)
    assert np.array_equal(res[0][0], res[1][0]) and np.array_equal(res[0][1], res[1][1])


def test_a_slow_neighbour_is_waited_for(B):
    """One worker's samples and centroids coincide: all of its assignments are decided in fp64 against all centroids, tens of
    milliseconds per step, and nobody may give up on its messages."""
    k, d, W, b, E = 1000, 129, 192, 1024, 4
    rng = np.random.default_rng(1)
    X = rng.standard_normal((W, b, d), dtype=np.float32)
    X[5] = X[5, 0]
    X = X.reshape(W * b, d)
    res = []
    for tune in (0, 4):                                 # one launch, phases (no waits)
        g = context(B, X, k, W, b, E, tune=tune)
        g.run_steps(3 * E + 1)
        res.append((g.get_state(), g.worker_counters(), g.last_run_form()))
    assert res[0][2] == B.FORM_SPLIT_LAUNCH and res[1][2] == B.FORM_SPLIT_PHASES
    assert np.array_equal(res[0][1][:, :2], res[1][1][:, :2])
    assert np.abs(res[0][0] - res[1][0]).max() <= 1e-5


@pytest.mark.parametrize("kernel,k,d,W,b,E", FORMS)
def test_lost_messages_cuts_and_many_buffers_in_one_launch(B, oracle, kernel, k, d, W, b, E):
    # calls that end inside a round and at a merge point, messages that never come, two buffers; against the oracle and,
    # bit for bit, against the run in one call
    X = make_data(W * max(b + 3, k), d, k, seed=7)
    id = getattr(B, "KERNEL_" + kernel)
    steps = 3 * E + 2
    whole = B.ASGD(k, d, W, b, 0.05, E=E, kernel=id, buffers=2, drop_rate=0.3)
    whole.load_shards(to_dev(X))
    whole.run_steps(steps)
    assert whole.stats().launches == 1 and whole.last_run_form() == B.FORM_SPLIT_LAUNCH
    cut = B.ASGD(k, d, W, b, 0.05, E=E, kernel=id, buffers=2, drop_rate=0.3)
    cut.load_shards(to_dev(X))
    for n in (1, 1, E - 2, E - 1, 1, steps - 2 * E):
        cut.run_steps(n)
    assert np.array_equal(whole.get_state(), cut.get_state())
    assert np.array_equal(whole.worker_counters(), cut.worker_counters())
    o = oracle.OracleASGD(X, k=k, W=W, b=b, lr=0.05, E=E, buffers=2, drop_rate=0.3)
    o.run_steps(steps)
    assert rel_fro(whole.get_state(), o.w).max() <= 1e-4
    check_counters(whole.worker_counters(), o.counters, o.parzen_near)


@pytest.mark.parametrize("kernel,k,d,W,b,E", [("GENERIC", 3, 2, 192, 128, 4), ("MFMA", 500, 24, 400, 64, 4)])
def test_a_long_call_is_cut_into_launches(B, kernel, k, d, W, b, E):
    X = make_data(W * max(2 * b + 3, k), d, k, seed=47)
    steps = 2060 * E + 3                                # 1024 rounds a launch
    res = []
    for cuts in ((steps,), (1024 * E, 5, 1030 * E + 1, steps - 2054 * E - 6)):
        g = B.ASGD(k, d, W, b, 0.02, E=E, kernel=getattr(B, "KERNEL_" + kernel))
        g.load_shards(to_dev(X))
        for n in cuts:
            g.run_steps(n)
        res.append((g.get_state(), g.worker_counters(), g.stats().launches))
        assert g.last_run_form() == B.FORM_SPLIT_LAUNCH
    assert res[0][2] == 3
    assert np.array_equal(res[0][0], res[1][0]) and np.array_equal(res[0][1], res[1][1])


@pytest.mark.parametrize("kernel,k,d,W,b,E", FORMS[:3])
def test_an_expired_wait_is_reported_and_the_context_recovers(B, kernel, k, d, W, b, E):
    """As for the other kernels: messages get lost without the recipients being told, and the workgroups have four polls for
    all their waits; every kernel ends normally."""
    X = to_dev(make_data(W * max(b + 3, k), d, k, seed=43))
    g = B.ASGD(k, d, W, b, 0.05, E=E, drop_rate=1.0, kernel=getattr(B, "KERNEL_" + kernel))
    g.set_option(B.OPT_WAIT_POLLS, 4)
    g.set_option(B.OPT_DROP_UNANNOUNCED, 1)
    g.load_shards(X)
    w0 = g.get_state()
    with pytest.raises(B.AsgdError) as e:
        g.run_steps(2 * E + 1)
    assert e.value.code == B.ESYNC and g.stats().steps == 0 and g.stats().launches == 1
    assert g.last_run_form() == B.FORM_SPLIT_LAUNCH
    with pytest.raises(B.AsgdError) as e:
        g.run_steps(1)
    assert e.value.code == B.ESTATE
    g.set_option(B.OPT_DROP_UNANNOUNCED, 0)             # lost messages are skipped again: as in silent mode
    g.set_state(-2, w0)
    g.set_step(0)
    g.run_steps(2 * E + 1)
    s = B.ASGD(k, d, W, b, 0.05, E=0, kernel=getattr(B, "KERNEL_" + kernel))
    s.load_shards(X)
    s.run_steps(2 * E + 1)
    assert g.stats().steps == 2 * E + 1 and np.abs(g.get_state() - s.get_state()).max() <= 1e-5 * np.abs(w0).max()
