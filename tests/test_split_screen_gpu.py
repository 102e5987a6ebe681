"""Steps whose samples are screened with the high parts of their operands: a streamed state, sweeps of four and of two tiles, ragged ends, lists that
are emptied, screening that is given up and samples with dozens of nearest rows, against the oracle or the kernels that do not screen."""
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
    # every prototype twice or more: no score decides anything, screening is given up after the first sweep, ties go to the lowest index
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


# ---- data of which screening leaves a part open ----
def hard_data(k, d, b, share, seed, wide=0.0):
    """Samples of W workers and a common state whose last two eighths are copies of the first one.  share(n): how many of the samples n of a mini-batch
    lie next to one of the three copies.  wide: size of one column that says nothing about the others."""
    import torch
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(seed)
    q = k // 8
    w = 10.0 * torch.rand((k, d), generator=gen, device="cuda:0")
    w[k - q:] = w[:q]
    w[k - 2 * q:k - q] = w[:q]
    hard = torch.rand((W, b), generator=gen, device="cuda:0") < share(torch.arange(b, device="cuda:0"))
    at = torch.where(hard, torch.randint(0, q, (W, b), generator=gen, device="cuda:0"), torch.randint(q, k - 2 * q, (W, b), generator=gen, device="cuda:0"))
    x = w[at.reshape(-1)]
    x += torch.randn((W * b, d), generator=gen, device="cuda:0")
    if wide:
        x[:, 0] = wide * torch.rand(W * b, generator=gen, device="cuda:0")
        w[:, 0] = wide * torch.rand(k, generator=gen, device="cuda:0")
    return x.contiguous(), w.cpu().numpy()


def decisions(B, x, w, b, tune=0, steps=1):
    g = B.ASGD(w.shape[0], w.shape[1], W, b, 0.05, E=0, kernel=B.KERNEL_GENERIC, tune=tune)
    g.load_shards(x)
    g.set_state(-1, w)
    g.enable_assign_dump(steps)
    g.run_steps(steps)
    assert g.last_run_form() == (B.FORM_SPLIT_PHASES if tune else B.FORM_SPLIT_LAUNCH)
    out = g.assign_dump(steps), g.get_state(), g.last_run_ms()
    g.close()
    return out


# A state in one stage and in several; lists that are emptied in the middle of a mini-batch (1024 samples and more, with rows that have two
# equals), and a workgroup that gives screening up later than at the first sweep: before its list was emptied once (samples 6000 on) and after (11000 on)
@pytest.mark.parametrize("k,d", [(600, 60), (577, 101)])
@pytest.mark.parametrize("b,from_on", [(11300, None), (7777, 6000), (12800, 11000)])
def test_partly_undecided_samples(B, k, d, b, from_on):
    import torch
    at = b if from_on is None else from_on
    x, w = hard_data(k, d, b, lambda n: torch.where(n >= at, 1.0, 0.10), seed=k + b)
    idx, state, _ = decisions(B, x, w, b, steps=2)
    want, state_want, _ = decisions(B, x, w, b, tune=4, steps=2)             # (phases do not screen)
    assert np.array_equal(idx, want) and np.array_equal(state, state_want)


@pytest.mark.parametrize("k,d,b", [(600, 60, 1500), (400, 128, 2000)])
def test_undecided_samples_do_not_pay_for_screening(B, k, d, b):
    # (screened nevertheless: three to four times what phases take)
    x, w = hard_data(k, d, 4 * b, lambda n: 0.5 + 0.0 * n, seed=d, wide=1.0e4)
    ms = [min(decisions(B, x, w, b, tune=tune, steps=4)[2] for _ in range(3)) for tune in (0, 4)]
    assert ms[0] < 2.0 * ms[1], ms


# long rows where a mini-batch's shares do not divide the compute units: more than one round of workgroups, ragged last shares
@pytest.mark.parametrize("k,d,W,b", [(130, 140, 150, 300), (40, 150, 300, 130), (100, 200, 129, 515), (20, 150, 150, 250)])
def test_long_rows_in_rounds(B, oracle, k, d, W, b):
    g, _ = run_both(B, oracle, make_data(W * (2 * b + 3), d, k, seed=W + b), k, W, b, 0.05, 2, 3, kernel=B.KERNEL_GENERIC, check_qe=False)
    assert g.last_run_form() == B.FORM_SPLIT_PHASES
