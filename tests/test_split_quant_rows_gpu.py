"""Eq. 8 with fp16-split operands: the direct distance of a sample to its nearest centroid over rows whose last chunks of columns
do not come in fours, against 64-bit distances."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


# (up to 16 columns samples are screened beyond 120000)
@pytest.mark.parametrize("d,N", [(d, 4001) for d in (17, 31, 33, 47, 49, 51, 63, 65, 75, 79, 81, 95, 97, 111, 113, 127)] + [(d, 121001) for d in (8, 9, 10, 11, 13, 15, 17, 18, 19, 22, 25, 31)])
def test_quant_error_row_lengths(d, N):
    import torch
    from paper_1505_04956_amd import binding as B
    k = 37
    rng = np.random.default_rng(d)
    w = rng.uniform(0.0, 10.0, (k, d)).astype(np.float32)
    X = (w[rng.integers(0, k, N)] + rng.standard_normal((N, d))).astype(np.float32)
    x, c = torch.from_numpy(X).to("cuda:0"), torch.from_numpy(w).to("cuda:0")
    out = torch.zeros(1, dtype=torch.float64, device="cuda:0")
    B.asgd_quant_error_noalloc(x.data_ptr(), N, k, d, c.data_ptr(), out.data_ptr(), torch.cuda.current_stream().cuda_stream)
    exact = 0.0
    for lo in range(0, N, 4000):
        exact += 0.5 * ((X[lo:lo + 4000, None].astype(np.float64) - w[None].astype(np.float64)) ** 2).sum(-1).min(1).sum()
    # d squares and additions of fp32 numbers, a difference each: (d + 3) roundings at most
    assert abs(float(out[0]) - exact) <= (d + 3) * 2.0 ** -24 * exact
