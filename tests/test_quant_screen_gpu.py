"""Eq. 8 with screened samples: whole sweeps of the device, the half sweep after them and its ragged end, both ways to form the distances, and
lists of undecided samples that overflow, against 64-bit distances."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def exact_error(x, w):
    import torch
    total, w = 0.0, w.double()
    for lo in range(0, x.shape[0], 8192):
        d2 = torch.full((x[lo:lo + 8192].shape[0],), float("inf"), dtype=torch.float64, device=x.device)
        for c in range(0, w.shape[0], 32):
            d2 = torch.minimum(d2, ((x[lo:lo + 8192].double()[:, None] - w[None, c:c + 32]) ** 2).sum(-1).min(1).values)
        total += 0.5 * float(d2.sum())
    return total


# Samples of a sweep: 2048 waves of 128 (k = 600; k = 12, d = 9), 64 (k = 37) and 32 (k = 16, d = 121) samples
@pytest.mark.parametrize("k,d,N", [(12, 9, 262144), (12, 9, 262144 + 131072 + 1), (37, 75, 131072 + 4001), (37, 75, 2 * 131072 - 1),
                                   (600, 20, 262144 + 65), (600, 65, 393216 + 77), (16, 121, 3 * 65536 + 31), (33, 128, 65537), (2, 8, 130), (200, 128, 262144 + 1)])
@pytest.mark.parametrize("ties", [False, True])
def test_sweeps_and_lists(k, d, N, ties):
    import torch
    from paper_1505_04956_amd import binding as B
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(k + d)
    w = 10.0 * torch.rand((k, d), generator=gen, device="cuda:0")
    if ties:                                     # every sample has two nearest rows or more: none is decided by its score
        w[k // 2:] = w[:k - k // 2].clone()
    x = w[torch.randint(0, k, (N,), generator=gen, device="cuda:0")] + torch.randn((N, d), generator=gen, device="cuda:0")
    x[N // 3] *= 1.0e4                           # beyond the common scale of the samples
    x[-1] += 3.0
    x, w = x.contiguous(), w.contiguous()
    out = torch.zeros(1, dtype=torch.float64, device="cuda:0")
    B.asgd_quant_error_noalloc(x.data_ptr(), N, k, d, w.data_ptr(), out.data_ptr(), torch.cuda.current_stream().cuda_stream)
    exact = exact_error(x, w)
    # listed samples: d squares and additions of fp32 numbers, a difference each: (d + 3) roundings at most
    assert abs(float(out[0]) - exact) <= (d + 3) * 2.0 ** -24 * exact
    assert np.isfinite(exact)


@pytest.mark.parametrize("k,d,N", [(37, 75, 300001), (1024, 128, 300001), (100, 100, 200001), (1000, 20, 300001), (12, 9, 300001), (500, 60, 200001)])
def test_every_decision_on_a_grid(k, d, N):
    # Multiples of 1/8 below 2^5: differences, squares and sums of up to 128 of them are exact in fp32, so a single sample at another
    # prototype than its nearest would show.
    import torch
    from paper_1505_04956_amd import binding as B
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(d)
    w = 10.0 * torch.rand((k, d), generator=gen, device="cuda:0")
    x = w[torch.randint(0, k, (N,), generator=gen, device="cuda:0")] + 2.0 * torch.randn((N, d), generator=gen, device="cuda:0")
    w += 0.7 * torch.randn((k, d), generator=gen, device="cuda:0")
    w[: k // 3] = w[k // 3: 2 * (k // 3)] + 0.3 * torch.randn((k // 3, d), generator=gen, device="cuda:0")       # pairs close together
    x, w = ((8.0 * v).round() / 8.0 for v in (x, w))
    out = torch.zeros(1, dtype=torch.float64, device="cuda:0")
    B.asgd_quant_error_noalloc(x.contiguous().data_ptr(), N, k, d, w.contiguous().data_ptr(), out.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert float(out[0]) == exact_error(x, w)
