"""The mean of the worker states is formed in worker order in fp64, 32 workers in flight: the same bits as the plain sum."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k,d,W", [(2, 1, 1), (3, 21, 31), (7, 9, 32), (5, 13, 33), (16, 4, 64), (11, 6, 95)])
def test_mean_state_in_worker_order(k, d, W):
    import torch
    from paper_1505_04956_amd import binding as B
    rng = np.random.default_rng(W)
    X = rng.uniform(-5.0, 5.0, (W * 40, d)).astype(np.float32)
    g = B.ASGD(k, d, W, 16, 0.1)
    g.load_shards(torch.from_numpy(X).to("cuda:0"))
    w = rng.standard_normal((W, k, d)).astype(np.float32) * np.float32(10.0) ** rng.integers(-6, 7, (W, k, d)).astype(np.float32)
    g.set_state(-2, w)
    s = np.zeros((k, d))
    for i in range(W):
        s = s + w[i].astype(np.float64)
    assert np.array_equal(g.get_mean_state(), (s / np.float64(W)).astype(np.float32).reshape(g.get_mean_state().shape))
