"""Steps whose samples are screened with the high parts of their operands: a streamed state, sweeps of four and of two tiles, ragged ends, lists that
overflow and samples with dozens of nearest rows, against the oracle."""
import numpy as np
import pytest

from tests.parity_rules import rel_fro
from tests.test_parity_gpu import B, make_data, run_both, to_dev  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu
W = 192                                      # the fewest workers of one launch


# k up to the edges of a pair of row blocks, d around the chunks of 16 columns, mini-batches around a wave's 64 and 128 samples and the sweeps
# of eight waves (512 and 1024)
@pytest.mark.parametrize("k,d,b,E", [(1000, 20, 384, 4), (1025, 36, 520, 0), (700, 49, 513, 4), (640, 64, 1030, 4), (513, 81, 900, 8), (400, 128, 1024, 4), (577, 101, 1600, 4)])
def test_screened_steps(B, oracle, k, d, b, E):
    steps = E + 2 if E else 2
    H = max(2 * b + 11, k)
    X = make_data(W * H, d, k, seed=k + d)
    g, _ = run_both(B, oracle, X, k, W, b, 0.05, E, steps, kernel=B.KERNEL_GENERIC, check_qe=False)
    assert g.last_run_form() == B.FORM_SPLIT_LAUNCH


@pytest.mark.parametrize("k,d,b", [(600, 60, 1500), (512, 100, 2100)])
def test_many_undecided_samples(B, oracle, k, d, b):
    # every prototype twice or more: no score decides anything, lists overflow (more than 1024 samples), ties go to the lowest index
    H = max(b + 5, k)
    X = make_data(W * H, d, 8, seed=d)
    rng = np.random.default_rng(k)
    X[::3] = X[0]                            # one row a third of the data: dozens of equal prototypes, wherever workers start
    w0 = X[rng.integers(0, 64, k)]
    run_both(B, oracle, X, k, W, b, 0.05, 0, 1, kernel=B.KERNEL_GENERIC, check_qe=False, w0=w0)
