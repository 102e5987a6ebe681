"""Data that lie awkwardly for scores from fp16-split operands: outlying prototypes, columns of very different size, groups
far apart, very small and very large numbers.  Whatever the scores are worth, the results have to be those of the
direct form."""
import numpy as np
import pytest

from tests.parity_rules import rel_fro
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


SHAPES = [(37, 75, 1500), (256, 384, 700), (12, 9, 101000), (31, 9, 3000), (300, 129, 700), (600, 40, 120000), (600, 101, 900),
          # rows of up to 16 columns, less than 300 of them, are screened beyond 120000 samples
          (12, 9, 121000), (40, 17, 130000), (70, 27, 121001)]


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


@pytest.mark.parametrize("k,d,N", [(39, 13, 3000), (37, 75, 1500), (12, 9, 101000), (600, 40, 120000), (300, 129, 700), (12, 9, 121000), (39, 13, 130000),
                                   (40, 31, 121001)])
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


# ---- steps ----
@pytest.mark.parametrize("kernel,k,d,b", [("GENERIC", 20, 13, 150), ("GENERIC", 40, 150, 150), ("MFMA", 64, 32, 600)])
@pytest.mark.parametrize("scale", [1.0e-36, 1.0e-30, 1.0e-22, 1.0e-20, 1.0e16, 1.0e25, 1.0e34])
def test_steps_on_small_and_large_numbers(B, oracle, kernel, k, d, b, scale):
    # squares that vanish or overflow in fp32; the same mixture decides nothing differently at any scale
    X = make_data(4 * (3 * b + 11), d, k, seed=9) * np.float32(scale)
    g, _ = run_both(B, oracle, X, k, 4, b, 0.05, 2, 6, kernel=getattr(B, "KERNEL_" + kernel), tune=SPLIT if kernel == "GENERIC" else 0,
                    check_qe=False)
    assert g.last_run_form() == B.FORM_SPLIT_PHASES and g.stats().exact_rechecks < 4 * 6 * b // 20             # (and without taking everything to fp64)


@pytest.mark.parametrize("k,d", [(20, 13), (40, 150)])
@pytest.mark.parametrize("size", [1.0e5, 1.0e10, 1.0e15, 1.0e20])
def test_steps_from_a_state_far_beyond_the_data(B, oracle, k, d, size):
    # offsets of the scores beyond that of the rows the state is padded with (k is no multiple of 32)
    rng = np.random.default_rng(k)
    X = make_data(4 * 500, d, k, seed=9) * np.float32(1.0e-12)
    w0 = (size * (1.0 + np.arange(k)[:, None] / k) * rng.choice([-1.0, 1.0], (k, d))).astype(np.float32)
    run_both(B, oracle, X, k, 4, 150, 0.05, 2, 4, kernel=B.KERNEL_GENERIC, tune=SPLIT, check_qe=False, w0=w0)


@pytest.mark.parametrize("kernel,tune,k,d,W,b", [("GENERIC", SPLIT, 20, 13, 4, 150), ("GENERIC", 0, 40, 150, 4, 150), ("GENERIC", 0, 12, 8, 200, 100),
                                                 ("MFMA", 0, 64, 32, 4, 600), ("MFMA", 0, 300, 32, 4, 600)])
@pytest.mark.parametrize("value", [1.0e9, 1.0e12, 1.0e20, -3.0e38])
def test_one_huge_element_does_not_touch_the_other_workers(B, oracle, kernel, tune, k, d, W, b, value):
    # sums in fixed point scaled by the largest element of a column would lose everything else in it
    H = max(3 * b + 11, k)
    X = make_data(W * H, d, k, seed=9)
    X[2 * H + b // 2, 1] = value
    g = B.ASGD(k, d, W, b, 0.05, E=0, kernel=getattr(B, "KERNEL_" + kernel), tune=tune)
    g.load_shards(to_dev(X))
    g.run_steps(6)
    o = oracle.OracleASGD(X, k=k, W=W, b=b, lr=0.05, E=0)
    o.run_steps(6)
    err = rel_fro(g.get_state(), o.w)
    if abs(value) > 1.0e10:
        assert g.last_run_form() == B.FORM_FP32
    # rounding of sums and updates (a few 2^-24 per step), and the odd near-tie of an fp32 state
    assert np.delete(err, 2).max() <= 1e-5


@pytest.mark.parametrize("what,form", [("lognormal", "SPLIT_PHASES"), ("sparse", "SPLIT_PHASES"), ("probabilities", "SPLIT_PHASES"),
                                        ("one in ten", "FP32"), ("half", "FP32"), ("tiny column", "FP32")])
def test_heavy_tails_stay_and_markers_go(B, oracle, what, form):
    """Columns whose elements spread over many magnitudes keep the split kernels; a marker of 1e30, in however many elements,
    takes the kernel with fp32 sums.  All against the oracle."""
    k, d, W, b = 20, 13, 4, 150
    rng = np.random.default_rng(3)
    X = make_data(W * (3 * b + 11), d, k, seed=9)
    if what == "lognormal":
        X = np.exp(2.5 * rng.standard_normal(X.shape))
    elif what == "sparse":
        X = X * (rng.random(X.shape) < 0.05)
    elif what == "probabilities":
        X = np.exp(1.2 * X - 1.2 * X.max(1, keepdims=True))
    elif what == "tiny column":
        X[:, 4] *= 1.0e-9
        X[77, 4] = 1.0e3
    else:
        X = np.where(rng.random(X.shape) < (0.1 if what == "one in ten" else 0.5), 1.0e30, X)
    X = np.ascontiguousarray(X, dtype=np.float32)
    g = B.ASGD(k, d, W, b, 0.05, E=0, kernel=B.KERNEL_GENERIC)
    g.load_shards(to_dev(X))
    g.run_steps(6)
    assert g.last_run_form() == getattr(B, "FORM_" + form)
    o = oracle.OracleASGD(X, k=k, W=W, b=b, lr=0.05, E=0)
    o.run_steps(6)
    if form == "SPLIT_PHASES":
        assert rel_fro(g.get_state(), o.w).max() <= 1e-5


@pytest.mark.parametrize("kernel,d,W,b", [("GENERIC", 75, 2, 20000), ("GENERIC", 13, 1, 8192), ("GENERIC", 5, 3, 6000), ("GENERIC", 300, 1, 40000),
                                          ("MFMA", 96, 2, 20000)])
def test_a_sum_over_many_shares_is_rounded_once(B, kernel, d, W, b):
    # One step of two centroids, all samples at the first, far from the origin, where c w - S cancels.  In units of the last
    # place of w: S is rounded by half a unit, its up to 64 shares by half a unit of THEIRS each (independently: an eighth of a
    # unit of S together), 0.75 of that reaches w, doubled where S and w lie differently in their binades; the update itself
    # rounds by half a unit and little more.
    rng = np.random.default_rng(d)
    X = (1.0e4 + rng.uniform(0.0, 6.0e3, (W * b, d))).astype(np.float32)
    w0 = np.stack([X[:b].mean(0, dtype=np.float64), np.full(d, 3.0e5)]).astype(np.float32)
    g = B.ASGD(2, d, W, b, 0.75, E=0, kernel=getattr(B, "KERNEL_" + kernel), tune=SPLIT if kernel == "GENERIC" else 0)
    g.load_shards(to_dev(X))
    g.set_state(-1, w0)
    g.run_steps(1)
    S = X.reshape(W, b, d).sum(1, dtype=np.float64)
    exact = w0[0].astype(np.float64) - 0.75 * (b * w0[0].astype(np.float64) - S) / b
    assert g.last_run_form() == B.FORM_SPLIT_PHASES
    off = np.abs(g.get_state()[:, 0] - exact) / np.spacing(exact.astype(np.float32))
    assert off.max() <= 1.6, off.max()
