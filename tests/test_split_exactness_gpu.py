"""Data that lie awkwardly for scores from fp16-split operands: outlying prototypes, columns of very different size, groups
far apart, very small and very large numbers.  Whatever the scores are worth, the results have to be those of the
direct form."""
import numpy as np
import pytest

from tests.test_parity_gpu import B, make_data, run_both, to_dev  # noqa: F401  (fixtures)
from tests.test_split_kernel_gpu import SPLIT, quant_error

pytestmark = pytest.mark.gpu


# ---- Eq. 8 ----
def mixture(N, k, d, seed, sigma=0.5):
    """Samples of k Gaussians with centres in [0, 10]^d, and a state near the centres."""
    rng = np.random.default_rng(seed)
    centres = rng.uniform(0.0, 10.0, (k, d))
    X = centres[rng.integers(0, k, N)] + sigma * rng.standard_normal((N, d))
    return X.astype(np.float32), (centres + sigma * rng.standard_normal((k, d))).astype(np.float32)


def check_quant_error(B, oracle, X, w):
    # the direct form in fp32: one rounding per difference, one per fused multiply-add, all terms non-negative, and the
    # addition of the two half rows - (d + 3) 2^-24 of a distance, of the smallest one as of any other; the sum is fp64
    X, w = np.ascontiguousarray(X, dtype=np.float32), np.ascontiguousarray(w, dtype=np.float32)
    q, o = quant_error(B, X, w), oracle.quant_error(X, w.astype(np.float64))
    assert abs(q - o) <= (X.shape[1] + 3) * 2.0 ** -24 * o, (q, o, q / o - 1.0)


SHAPES = [(37, 75, 1500), (256, 384, 700), (12, 9, 101000), (31, 9, 3000), (300, 129, 700), (600, 40, 120000), (600, 101, 900)]


@pytest.mark.parametrize("k,d,N", SHAPES)
@pytest.mark.parametrize("row,size", [(3, 1.0e4), (3, 1.0e5), (3, 1.0e12), (11, -1.0e25), (-1, 1.0e5), (slice(1, 9), 1.0e5)])
def test_quant_error_with_an_outlying_prototype(B, oracle, k, d, N, row, size):
    X, w = mixture(N, k, d, seed=k + d)
    w[row] = np.float32(size)
    X[N // 2] = np.float32(size)                       # a sample on it: only the direct form sees that
    check_quant_error(B, oracle, X, w)


@pytest.mark.parametrize("k,d,N", SHAPES)
@pytest.mark.parametrize("levels", [1.0e4, 1.0e5])
def test_quant_error_with_one_wide_column(B, oracle, k, d, N, levels):
    X, w = mixture(N, k, d, seed=2 * k + d)
    rng = np.random.default_rng(k)
    at = d // 2
    w[:, at] = levels * rng.integers(0, 4, k)
    X[:, at] = levels * rng.integers(0, 4, N)
    check_quant_error(B, oracle, X, w)


@pytest.mark.parametrize("k,d,N", [(39, 13, 3000), (37, 75, 1500), (12, 9, 101000), (600, 40, 120000), (300, 129, 700)])
def test_quant_error_of_groups_far_apart(B, oracle, k, d, N):
    rng = np.random.default_rng(k + d)
    groups = rng.uniform(0.0, 1.0e4, (6, d))
    step = rng.standard_normal((k, d))
    w = groups[np.arange(k) % 6] + 3.0 * step / np.linalg.norm(step, axis=1, keepdims=True)
    X = w[rng.integers(0, k, N)] + rng.standard_normal((N, d))
    check_quant_error(B, oracle, X, w)


@pytest.mark.parametrize("k,d,N", SHAPES)
@pytest.mark.parametrize("scale", [1.0e-17, 1.0e15, 1.0e17])
def test_quant_error_of_small_and_large_numbers(B, oracle, k, d, N, scale):
    X, w = mixture(N, k, d, seed=k + 3 * d)
    check_quant_error(B, oracle, X * np.float32(scale), w * np.float32(scale))


@pytest.mark.parametrize("k,d,N", SHAPES)
def test_quant_error_of_coincident_and_of_distant_samples(B, oracle, k, d, N):
    X, w = mixture(N, k, d, seed=k + 5 * d)
    w[k // 3:2 * k // 3 + 1] = w[0]                  # candidates by the dozen
    X[::7] = w[1]                                       # distance zero
    X[5::11] = np.float32(3.0e5)                        # farther from the state than its own extent
    check_quant_error(B, oracle, X, w)


@pytest.mark.parametrize("k,d,N", SHAPES)
@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
def test_quant_error_with_a_prototype_that_is_not_finite(B, oracle, k, d, N, value):
    # no distance to such a prototype is below infinity: the others decide
    X, w = mixture(N, k, d, seed=k + 7 * d)
    rest = np.delete(w, 2, axis=0)
    w[2, d - 1] = value
    q, o = quant_error(B, X, w), oracle.quant_error(X, rest.astype(np.float64))
    assert abs(q - o) <= (d + 3) * 2.0 ** -24 * o
