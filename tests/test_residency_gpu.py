"""Streaming kernel, one launch for many rounds: its workgroups wait for each other's messages, so no more of them are started than
have a place at the same time; each takes several workers through a round in turn.  Worker counts that fill the device, with
states whose kernel uses fewer registers than it asks for."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


# two waves of a worker up to 1024 workers, one beyond; tune 4, 5, 6: private cells, ring depths 8, 4, 2
@pytest.mark.parametrize("k,d,W,b,tune", [(16, 8, 700, 128, 0), (16, 8, 1024, 200, 0), (16, 8, 1100, 64, 0), (16, 8, 2500, 64, 0), (4, 4, 1024, 256, 0),
                                          (4, 4, 2500, 64, 0), (4, 4, 4500, 64, 0), (8, 8, 2500, 64, 0), (8, 16, 1100, 64, 0), (16, 12, 1100, 64, 0),
                                          (10, 10, 1100, 512, 4), (10, 10, 1100, 512, 5), (10, 10, 1100, 512, 6), (10, 10, 2500, 64, 0)])
def test_long_calls_with_many_workers(k, d, W, b, tune):
    import torch
    from paper_1505_04956_amd import binding as B
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device; there is no CPU fallback")
    rng = np.random.default_rng(W + k)
    X = torch.from_numpy(rng.uniform(0.0, 10.0, (W * 2 * b, d)).astype(np.float32)).to("cuda:0")
    steps = 81
    one, short = (B.ASGD(k, d, W, b, 0.05, E=2, kernel=2, tune=tune) for _ in range(2))
    for g in (one, short):
        g.load_shards(X)
    one.run_steps(steps)
    assert one.stats().launches == 1
    for done in range(0, steps, 2):                # a round at a time: nothing to wait for
        short.run_steps(min(2, steps - done))
    assert np.array_equal(one.get_state(), short.get_state())
    assert np.array_equal(one.worker_counters(), short.worker_counters())
