"""Eq. 8 with screened samples: whole sweeps of the device, the half sweep after them and its ragged end, both ways to form the distances, lists of
undecided samples that overflow, and screening that is given up, against 64-bit distances."""
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


def quant_error(x, w):
    import torch
    from paper_1505_04956_amd import binding as B
    out = torch.zeros(1, dtype=torch.float64, device="cuda:0")
    B.asgd_quant_error_noalloc(x.data_ptr(), x.shape[0], w.shape[0], w.shape[1], w.data_ptr(), out.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    return float(out[0])


def with_copies(k, d, N, share, seed):
    """Even numbers from 0 to 14; the last quarter of the rows are copies of the first, and a share of the samples lies next to them, so that no score decides
    them.  Two samples lie far beyond the common scale of the others.  Differences are even and below 6001, their squares multiples of four below 2^26, and so
    are the sums of up to 128 of them: exact in fp32, whoever adds them."""
    import torch
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(seed)
    w = 2.0 * torch.randint(0, 8, (k, d), generator=gen, device="cuda:0").float()
    q = max(1, k // 4)
    w[k - q:] = w[:q]
    near = torch.rand(N, generator=gen, device="cuda:0") < share
    x = w[torch.where(near, torch.randint(0, q, (N,), generator=gen, device="cuda:0"), torch.randint(q, k - q, (N,), generator=gen, device="cuda:0"))]
    x += 2.0 * (0.75 * torch.randn((N, d), generator=gen, device="cuda:0")).round()
    x.clamp_(0.0, 14.0)
    x[[N // 3, N - 1][:N], [0, d - 1][:N]] = 6000.0
    return x.contiguous(), w


# Every instance, whole sweeps of the device, the half sweep after them and its ragged end; no row length is a multiple of four, which the fp32 matrix kernel would
# take.  Samples of a sweep: 2048 waves of 128, 64 or 32 (up to 32 columns, or many rows; up to 96; more).  Share 0.3 fills the lists past 64 entries,
# with a share of 1 screening is given up after the first sweep.
@pytest.mark.parametrize("k,d,N", [(12, 9, 3 * 262144), (12, 9, 262144 + 131072 + 1), (600, 21, 262144 + 65), (37, 45, 2 * 131072 - 1), (500, 45, 262144 + 77),
                                   (37, 61, 5 * 131072 + 4001), (400, 63, 2 * 262144 + 1), (37, 75, 131072 + 4001), (37, 75, 2 * 131072 - 1), (600, 77, 262144 + 131072 + 77),
                                   (20, 90, 131072 + 1), (500, 90, 262144 + 130), (90, 101, 3 * 65536 + 31), (300, 101, 262144 + 1), (16, 121, 9 * 65536 + 31),
                                   (33, 127, 65537), (200, 125, 3 * 262144 - 1), (37, 33, 1), (5, 37, 64), (37, 75, 130), (8, 125, 2000)])
@pytest.mark.parametrize("share", [0.0, 0.3, 1.0])
def test_sweeps_and_lists(k, d, N, share):
    x, w = with_copies(k, d, N, share, seed=k + d)
    assert quant_error(x, w) == exact_error(x, w)


# Rows longer than 16 bytes of a lane by one to three, the fewest columns, several equals of a row: with more than two candidates the distances to those alone are formed
@pytest.mark.parametrize("k,d,N", [(64, 8, 300000), (300, 11, 250000), (90, 29, 200000), (64, 64, 400000), (257, 70, 150000), (100, 112, 200000), (1024, 128, 150000)])
@pytest.mark.parametrize("copies", [2, 8, 1000])
def test_many_candidates(k, d, N, copies):
    import torch
    x, w = with_copies(k, d, N, 0.2, seed=k * d)
    w = w[torch.arange(k, device="cuda:0") % max(2, k // copies)]
    for rows in (w.contiguous(), w.flip(0).contiguous()):
        assert quant_error(x, rows) == exact_error(x, rows)


# Several candidates for most samples, because rows coincide or one column is a thousand times as wide as the others.  The limits are half of what such data cost while
# every sample with more than two candidates was compared with all k rows (times that of ordinary data: 17, 25, 66, 33), and twice what they cost now.  The last are
# few samples of short rows, in the kernel without screening 13 times (up to twice that of ordinary data is the measurement's own).
@pytest.mark.parametrize("k,d,N,kind,limit", [(100, 100, 1000000, "copies", 9.0), (300, 48, 1000000, "copies", 12.0), (1024, 128, 500000, "copies", 30.0), (1000, 32, 1000000, "wide", 16.0),
                                              (4000, 32, 20000, "wide", 5.0)])
def test_time_of_undecided_samples(k, d, N, kind, limit):
    import torch
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(k)
    c = 10.0 * torch.rand((k, d), generator=gen, device="cuda:0")
    x = c[torch.randint(0, k, (N,), generator=gen, device="cuda:0")]
    x += torch.randn((N, d), generator=gen, device="cuda:0")

    def time(x, w):
        ms = []
        for _ in range(6):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            quant_error(x, w)
            end.record()
            end.synchronize()
            ms.append(start.elapsed_time(end))
        return min(ms[1:])
    w = c + torch.randn((k, d), generator=gen, device="cuda:0")
    plain = time(x, w)
    if kind == "copies":
        w = w[torch.arange(k, device="cuda:0") % (k // 8)].contiguous()
    else:
        w[:, 0] *= 1000.0
        x[:, 0] *= 1000.0
    assert time(x, w) < limit * plain


@pytest.mark.parametrize("k,d,N", [(37, 75, 300001), (1024, 128, 300001), (100, 100, 200001), (1000, 20, 300001), (12, 9, 300001), (500, 60, 200001)])
def test_every_decision_on_a_grid(k, d, N):
    # Multiples of 1/8 below 2^5: differences, squares and sums of up to 128 of them are exact in fp32, so a single sample at another
    # prototype than its nearest would show.
    import torch
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(d)
    w = 10.0 * torch.rand((k, d), generator=gen, device="cuda:0")
    x = w[torch.randint(0, k, (N,), generator=gen, device="cuda:0")] + 2.0 * torch.randn((N, d), generator=gen, device="cuda:0")
    w += 0.7 * torch.randn((k, d), generator=gen, device="cuda:0")
    w[: k // 3] = w[k // 3: 2 * (k // 3)] + 0.3 * torch.randn((k // 3, d), generator=gen, device="cuda:0")       # pairs close together
    x, w = ((8.0 * v).round() / 8.0 for v in (x, w))
    assert quant_error(x.contiguous(), w.contiguous()) == exact_error(x, w)


# Differences of 1e19 have squares that fp32 numbers hold, of one sample alone the sum is larger than all of them: infinite, whoever adds it.  (Rows are 1e20 apart: every
# sample would be decided by screening.)
@pytest.mark.parametrize("k,d,N", [(12, 9, 130000), (37, 75, 3000), (100, 45, 3000), (600, 45, 3000), (200, 125, 9000)])
def test_distances_beyond_fp32(k, d, N):
    import torch
    c = torch.arange(k, device="cuda:0")
    w = torch.zeros((k, d), device="cuda:0")
    w[c, c % d] = 1.0e20 * (1.0 + c // d)
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(k)
    x = w[torch.randint(0, k, (N,), generator=gen, device="cuda:0")]
    x[:, 0] += 1.0e19
    exact = exact_error(x, w)
    assert abs(quant_error(x, w) - exact) <= (d + 3) * 2.0 ** -24 * exact
    x[N // 2, 1] += 1.8e19
    assert quant_error(x, w) == float("inf")


# Data far from the origin, in units of their spread: scores relative to the origin would say nothing.  The streaming and the fp32 matrix kernel (state resident, and
# streamed) decide by scores, whose error (20 roundings of |x - m||w - m| and the tags) is a thousandth of such data's distances; the others are exact.
@pytest.mark.parametrize("k,d,N,tol", [(10, 10, 30001, 1.0e-4), (4, 4, 5000, 1.0e-4), (8, 8, 3001, 1.0e-4), (8, 16, 3001, 1.0e-4), (16, 8, 3001, 1.0e-4), (16, 12, 3001, 1.0e-4),
                                       (32, 16, 60000, 1.0e-4), (40, 20, 3786, 1.0e-4), (37, 100, 2001, 1.0e-4), (64, 32, 1, 1.0e-4), (65, 64, 40000, 1.0e-4), (100, 100, 160, 1.0e-4),
                                       (128, 128, 5000, 1.0e-4), (243, 80, 33, 1.0e-4), (500, 128, 700, 1.0e-4), (8200, 16, 3000, 1.0e-4), (9000, 128, 300, 1.0e-4),
                                       (7, 5, 3001, 0.0), (12, 9, 3001, 0.0), (100, 3, 3001, 0.0), (37, 75, 3001, 0.0), (1000, 48, 10000, 0.0), (50, 200, 3001, 0.0)])
@pytest.mark.parametrize("mean", [300.0, 1.0e4])
def test_data_far_from_the_origin(k, d, N, tol, mean):
    import torch
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(k + d)
    w = mean + 10.0 * torch.rand((k, d), generator=gen, device="cuda:0")
    x = w[torch.randint(0, k, (N,), generator=gen, device="cuda:0")]
    x += torch.randn((N, d), generator=gen, device="cuda:0")
    w += torch.randn((k, d), generator=gen, device="cuda:0")
    exact = exact_error(x, w)
    assert abs(quant_error(x, w) - exact) <= max(tol, (d + 3) * 2.0 ** -24) * exact
