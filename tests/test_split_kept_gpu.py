"""Split step kernels, workers whose operands, sums and mini-batches stay in the LDS (one workgroup each, three quarters of the
compute units and more): against the oracle, and bit for bit however a run is cut."""
import numpy as np
import pytest

from tests.test_parity_gpu import B, make_data, run_both, to_dev      # noqa: F401 (B is a fixture)

pytestmark = pytest.mark.gpu
SPLIT = 2


# row lengths around the groups of 8 and chunks of 16 columns up to four chunks, aligned and not; centroids around the blocks
# of 32 rows, a unit of eight columns per thread (Eq. 4 and the update in one) and more; mini-batches around groups of 64 and
# sweeps of 512; a message every step, two and three buffers, silent
@pytest.mark.parametrize("k,d,W,b,E,buffers,mean", [
    (2, 1, 192, 1, 1, 1, 0), (3, 2, 193, 63, 2, 2, 0), (12, 7, 256, 130, 0, 1, 1), (31, 7, 192, 64, 1, 1, 0), (32, 8, 200, 65, 1, 3, 0),
    (33, 9, 192, 513, 3, 1, 0), (64, 32, 256, 129, 1, 2, 0), (65, 16, 192, 200, 0, 1, 1), (40, 31, 192, 96, 2, 1, 0), (100, 60, 192, 70, 1, 2, 0),
    (20, 64, 192, 80, 5, 1, 0), (513, 8, 192, 520, 2, 1, 0), (500, 5, 192, 500, 1, 1, 0), (12, 7, 192, 1025, 4, 1, 0),
    # two mini-batches end within 1 KB of the LDS of a compute unit
    (12, 7, 192, 2743, 1, 1, 0), (128, 7, 200, 2560, 2, 1, 0), (128, 12, 192, 1430, 0, 1, 1), (37, 15, 192, 1246, 1, 2, 0),
])
def test_kept_workers(B, oracle, k, d, W, b, E, buffers, mean):
    X = make_data(W * max(3 * b + 2, k) + 1, d, k, seed=300 + d)
    steps = 7
    g, _ = run_both(B, oracle, X, k, W, b, 0.05, E, steps, kernel=B.KERNEL_GENERIC, tune=SPLIT, buffers=buffers, lr_mode=mean)
    assert g.last_run_form() == B.FORM_SPLIT_LAUNCH and (E > 3 or g.stats().launches == 1)
    whole, cut = (B.ASGD(k, d, W, b, 0.05, E=E, kernel=B.KERNEL_GENERIC, tune=SPLIT, buffers=buffers, lr_mode=mean) for _ in range(2))
    for c in (whole, cut):
        c.load_shards(to_dev(X))
    whole.run_steps(steps)
    for n in (1, 4, 2):
        cut.run_steps(n)
    assert np.array_equal(whole.get_state(), cut.get_state()) and np.array_equal(g.get_state(), cut.get_state())


# lost messages, a runtime that refuses such launches, a workgroup without a place: the same bits
@pytest.mark.parametrize("k,d,b,E", [(12, 7, 100, 1), (64, 32, 200, 2), (100, 60, 70, 1)])
def test_kept_workers_with_lost_messages_and_refused_launches(B, oracle, k, d, b, E):
    W, steps = 192, 9
    X = make_data(W * max(2 * b + 2, k), d, k, seed=11)
    g, _ = run_both(B, oracle, X, k, W, b, 0.05, E, steps, kernel=B.KERNEL_GENERIC, tune=SPLIT, buffers=2, drop_rate=0.3)
    for refuse in (1, 2):
        h = B.ASGD(k, d, W, b, 0.05, E=E, kernel=B.KERNEL_GENERIC, tune=SPLIT, buffers=2, drop_rate=0.3)
        h.set_option(B.OPT_REFUSE_ONE_LAUNCH, refuse)
        h.load_shards(to_dev(X))
        h.run_steps(steps)
        assert np.array_equal(g.get_state(), h.get_state()) and h.stats().launches > 1
