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


# ---- long rows whose operands fit the LDS ----
# one block of 32 rows to more than the waves can take at once, row lengths around the chunks that a wave keeps ahead, groups of 64 samples with ragged ends
@pytest.mark.parametrize("k,d,W,b,E,form", [(2, 129, 4, 64, 0, "SPLIT_PHASES"), (33, 200, 3, 65, 2, "SPLIT_PHASES"), (300, 385, 8, 200, 1, "SPLIT_PHASES"), (70, 500, 5, 130, 4, "SPLIT_PHASES"),
                                            (260, 256, 192, 130, 4, "SPLIT_LAUNCH"), (100, 150, 200, 257, 0, "SPLIT_LAUNCH"), (600, 300, 6, 70, 2, "SPLIT_PHASES")])
def test_long_rows(B, oracle, k, d, W, b, E, form):
    H = max(2 * b + 11, k)
    g, _ = run_both(B, oracle, make_data(W * H, d, k, seed=k + d), k, W, b, 0.05, E, max(2, E + 2), kernel=B.KERNEL_GENERIC, check_qe=False)
    assert g.last_run_form() == getattr(B, "FORM_" + form)


@pytest.mark.parametrize("k,d,W,b", [(150, 200, 4, 300), (150, 200, 192, 300), (40, 300, 6, 150)])
def test_many_equal_rows(B, oracle, k, d, W, b):
    # dozens of prototypes are the same: more samples than the list for the whole workgroup takes have to be tried against all of them
    X = make_data(W * max(b + 5, k), d, 8, seed=d)
    X[::2] = X[0]
    w0 = X[np.random.default_rng(k).integers(0, 16, k)]
    run_both(B, oracle, X, k, W, b, 0.05, 0, 1, kernel=B.KERNEL_GENERIC, check_qe=False, w0=w0)
