"""The matrix-core form of the shape-agnostic kernel (fp32 operands as two fp16 parts, any row length): against the oracle
at the edges of its tiles, and against the form with one workgroup per worker where the data are awkward."""
import numpy as np
import pytest

from tests.test_parity_gpu import B, make_data, run_both, to_dev  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu

ONE_WORKGROUP, SPLIT = 1, 2      # ASGD_OPT_TUNE of the shape-agnostic kernel: which form, whatever the size


# row lengths around the groups of 8 and chunks of 16 columns, the last one with its operands in registers (128) and the
# long-row kernel (129 ...); centroids around the blocks of 32 rows; mini-batches around the groups of 64 samples
@pytest.mark.parametrize("k,d,W,b,E,buffers,parts", [
    (2, 1, 3, 1, 2, 1, 1), (3, 2, 3, 63, 2, 1, 1), (31, 7, 5, 64, 2, 1, 1), (32, 8, 4, 65, 1, 1, 1), (33, 9, 3, 130, 3, 2, 1),
    (64, 15, 3, 300, 2, 1, 1), (65, 16, 2, 257, 1, 1, 1), (20, 17, 6, 100, 2, 1, 4), (40, 31, 3, 200, 2, 2, 3),
    (37, 33, 4, 129, 2, 1, 1), (12, 65, 3, 500, 2, 1, 1), (70, 111, 2, 128, 1, 1, 1), (5, 127, 3, 200, 2, 1, 1),
    (96, 128, 2, 320, 1, 1, 1), (300, 61, 2, 640, 1, 1, 1), (9, 129, 3, 96, 2, 1, 1), (97, 135, 2, 260, 1, 1, 1),
    (34, 257, 3, 70, 2, 2, 1), (7680, 3, 2, 100, 1, 1, 1), (130, 40, 2, 1500, 1, 1, 1), (6, 520, 3, 64, 1, 1, 2), (700, 12, 2, 1400, 1, 1, 1),
])
def test_split_kernel_edges(B, oracle, k, d, W, b, E, buffers, parts):
    H = max(3 * b + 7, k)
    X = make_data(W * H + 1, d, k, seed=100 + d)
    g, _ = run_both(B, oracle, X, k, W, b, 0.05, E, 7, kernel=B.KERNEL_GENERIC, tune=SPLIT, buffers=buffers,
                    parts=parts)
    assert g.last_run_form() == B.FORM_SPLIT_PHASES
    again = B.ASGD(k, d, W, b, 0.05, E=E, kernel=B.KERNEL_GENERIC, tune=SPLIT, buffers=buffers, parts=parts)
    again.load_shards(to_dev(X))
    again.run_steps(3)
    again.run_steps(4)
    assert np.array_equal(g.get_state(), again.get_state())        # bit for bit, however the run is cut


# both sides of the rules that choose between the kernels and between the one launch and the phases: mini-batches of 512,
# k of 256, exchange at every step from 100 workers on, workers beyond one and two per compute unit
# (what runs: F the fp32 kernel, L one launch, P phases - of the matrix-core kernel, of the shape-agnostic one)
DISPATCH = {
    (64, 32, 8, 511, 4, 1): "FP", (64, 32, 8, 512, 4, 2): "PP", (256, 16, 4, 100, 4, 1): "FP", (257, 16, 4, 100, 4, 1): "PP",
    (12, 8, 99, 100, 1, 1): "FP", (12, 8, 100, 100, 1, 1): "PP", (32, 16, 191, 97, 4, 1): "FP", (32, 16, 192, 520, 4, 1): "FL",
    (40, 8, 256, 512, 4, 2): "FL", (32, 16, 192, 520, 0, 1): "LL", (64, 64, 192, 512, 4, 1): "LL", (500, 24, 4, 64, 4, 1): "FP",
    (500, 24, 64, 64, 4, 1): "PP", (32, 16, 257, 97, 4, 1): "FP", (500, 24, 300, 64, 4, 1): "PP", (32, 16, 384, 97, 3, 1): "PP",
    (24, 8, 600, 100, 0, 1): "FP",
}


@pytest.mark.parametrize("kernel", ["MFMA", "GENERIC"])
@pytest.mark.parametrize("k,d,W,b,E,buffers", [
    (64, 32, 8, 511, 4, 1), (64, 32, 8, 512, 4, 2), (256, 16, 4, 100, 4, 1), (257, 16, 4, 100, 4, 1),
    (12, 8, 99, 100, 1, 1), (12, 8, 100, 100, 1, 1), (32, 16, 191, 97, 4, 1), (32, 16, 192, 520, 4, 1), (40, 8, 256, 512, 4, 2),
    (32, 16, 257, 97, 4, 1), (500, 24, 300, 64, 4, 1), (32, 16, 384, 97, 3, 1), (24, 8, 600, 100, 0, 1),
    (32, 16, 192, 520, 0, 1), (64, 64, 192, 512, 4, 1), (500, 24, 4, 64, 4, 1), (500, 24, 64, 64, 4, 1),
])
def test_split_kernel_dispatch(B, oracle, k, d, W, b, E, buffers, kernel):
    X = make_data(W * max(2 * b + 5, k), d, k, seed=200 + W)
    g, _ = run_both(B, oracle, X, k, W, b, 0.05, E, 9, kernel=getattr(B, "KERNEL_" + kernel), buffers=buffers)
    form = {B.FORM_FP32: "F", B.FORM_SPLIT_LAUNCH: "L", B.FORM_SPLIT_PHASES: "P"}[g.last_run_form()]
    assert form == DISPATCH[(k, d, W, b, E, buffers)][0 if kernel == "MFMA" else 1]


# the shape-agnostic kernel takes one workgroup per worker where a step is tiny
@pytest.mark.parametrize("k,d,b,form", [(3, 2, 127, "FP32"), (3, 2, 128, "SPLIT_PHASES"), (10, 9, 66, "FP32"), (10, 9, 67, "SPLIT_PHASES")])
def test_split_kernel_dispatch_of_tiny_steps(B, oracle, k, d, b, form):
    X = make_data(4 * (2 * b + 3), d, k, seed=b)
    g, _ = run_both(B, oracle, X, k, 4, b, 0.05, 2, 5, kernel=B.KERNEL_GENERIC)
    assert g.last_run_form() == getattr(B, "FORM_" + form)


@pytest.mark.parametrize("k,d,b", [(7, 5, 200), (40, 77, 333), (12, 140, 90)])
def test_split_kernel_running_mean(B, oracle, k, d, b):
    X = make_data(4 * (5 * b + 3), d, k, seed=5)
    g, _ = run_both(B, oracle, X, k, 4, b, 0.1, 0, 9, lr_mode=1, kernel=B.KERNEL_GENERIC)
    assert g.last_run_form() == B.FORM_SPLIT_PHASES


def pair(B, X, k, W, b, steps, w0=None, **kw):
    """States of the matrix-core form and of the one-workgroup form, same run."""
    out = []
    for tune in (SPLIT, ONE_WORKGROUP):
        g = B.ASGD(k, X.shape[1], W, b, 0.1, E=2, kernel=B.KERNEL_GENERIC, tune=tune, **kw)
        g.load_shards(to_dev(X))
        if w0 is not None:
            g.set_state(-1, w0)
        g.run_steps(steps)
        out.append((g.get_state(), g.stats(), g.last_run_form()))
    return out


@pytest.mark.parametrize("k,d", [(20, 13), (40, 150)])
@pytest.mark.parametrize("what", ["far", "columns", "identical", "w0_far", "w0_zero"])
def test_split_kernel_awkward_data(B, k, d, what):
    """Both forms assign exactly, so they differ by the rounding of sums of b terms and of the update only: a few 2^-24
    of the column's size per step."""
    W, b, steps = 4, 150, 6
    X = make_data(W * (3 * b + 11), d, k, seed=9, sigma=0.5)
    w0 = None
    if what == "far":
        X = X + np.float32(1.0e4)
    elif what == "columns":
        X = X * (np.float32(10.0) ** np.linspace(-6, 6, d).astype(np.float32))
    elif what == "identical":
        X[:] = X[0]
    elif what == "w0_far":
        w0 = np.float32(3.0e5) * make_data(k, d, k, seed=3)
    elif what == "w0_zero":
        w0 = np.zeros((k, d), dtype=np.float32)
    (wa, sa, fa), (wb, sb, fb) = pair(B, np.ascontiguousarray(X, dtype=np.float32), k, W, b, steps, w0)
    scale = np.abs(wb).max(axis=(0, 1)) + np.float32(1e-30)
    # (identical samples: w - c G ties in Eq. 4 and equal distances are decided the same way in both forms)
    assert np.all(np.abs(wa - wb).max(axis=(0, 1)) <= 1e-6 * scale), what
    assert sa.sent == sb.sent and sa.received == sb.received
    assert fa == B.FORM_SPLIT_PHASES and fb == B.FORM_FP32


@pytest.mark.parametrize("value", [np.inf, np.nan])
def test_split_kernel_leaves_non_finite_samples_to_the_other_form(B, value):
    k, d, W, b = 20, 13, 4, 100
    X = make_data(W * 500, d, k, seed=9)
    X[777, 5] = value
    (wa, sa, fa), (wb, sb, fb) = pair(B, X, k, W, b, 6)
    assert fa == fb == B.FORM_FP32
    assert np.array_equal(wa, wb, equal_nan=True) and sa.launches == sb.launches


def quant_error(B, X, w):
    import torch
    Xd, wd = to_dev(X), to_dev(w)
    out = torch.zeros(1, dtype=torch.float64, device=Xd.device)
    B.asgd_quant_error_noalloc(Xd.data_ptr(), X.shape[0], w.shape[0], X.shape[1], wd.data_ptr(), out.data_ptr(),
                               torch.cuda.current_stream().cuda_stream)
    return float(out.cpu()[0])


# Eq. 8 at the edges of the tiles: groups of 64 and 512 samples, blocks of 32 rows, chunks of 16 columns, state resident in
# LDS or streamed, long rows; also far from the origin
@pytest.mark.parametrize("k,d,N", [
    (2, 8, 1), (13, 7, 63), (11, 8, 64), (33, 8, 65), (31, 9, 511), (64, 15, 513), (65, 17, 4096), (100, 101, 3000),
    (37, 75, 2000), (96, 127, 700), (512, 128, 66000), (2100, 41, 900), (300, 129, 800), (70, 384, 600), (12, 520, 300),
    # sizes past the lines of the rule that chooses the kernel
    (2, 136, 1), (40, 7, 63), (34, 8, 64), (35, 8, 65), (512, 128, 137000), (2, 16, 100001), (7, 7, 100003), (24, 7, 100001), (3, 17, 100065),
])
@pytest.mark.parametrize("offset", [0.0, 1.0e4])
def test_split_quant_error_edges(B, oracle, k, d, N, offset):
    X = make_data(N, d, k, seed=40 + d, sigma=0.5)
    rng = np.random.default_rng(k)
    w = (X[rng.integers(0, N, size=k)] + rng.standard_normal((k, d)) + offset).astype(np.float32)
    X = (X + np.float32(offset)).astype(np.float32)
    q, o = quant_error(B, X, w), oracle.quant_error(X, w.astype(np.float64))
    # every sample adds the smallest of its direct fp32 distances: (d + 3) 2^-24 of it at worst (test_split_exactness_gpu.py)
    assert abs(q - o) <= (d + 3) * 2.0 ** -24 * o


def test_split_quant_error_of_non_finite_samples(B):
    X = make_data(1000, 13, 20, seed=9)
    w = make_data(20, 13, 20, seed=10)
    for value in (np.inf, np.nan):
        Y = X.copy()
        Y[777, 5] = value
        assert quant_error(B, Y, w) == np.inf
