"""Performance cases of the ASGD K-Means path: the calls a user's program makes, over the sizes it makes them at.

Two kinds of pass.  `train` is a clustering job from data to result: the samples are handed to the workers
(`load_shards`), all of them start from their own first rows or from one common state (`common_start`, the paper's
"w0 is given to all workers"), `epochs` passes are run, and the states come back.  `eval` is the quantization error of
a state over a data set, enqueued on the caller's stream.  `exact` computes the same results in 64 bits with plain
torch operations, written from the definition of the method.
"""
import math

import numpy as np
import torch

from paper_1505_04956_amd import binding as B

ALL_STATES_BYTES = 4 << 20      # up to here a program takes every worker's state home, beyond it w^1 and the mean state


def _train(name, N, k, d, W, b, E, epochs, lr=0.05, sigma=1.0, skew=False, buffers=1, parts=1, running_mean=False,
           common_start=False, error=False):
    return {"name": name, "kind": "train", "N": N, "k": k, "d": d, "W": W, "b": b, "E": E, "epochs": epochs, "lr": lr,
            "sigma": sigma, "skew": skew, "buffers": buffers, "parts": parts, "running_mean": running_mean,
            "common_start": common_start, "error": error}


def _eval(name, N, k, d, sigma=1.0, skew=False):
    return {"name": name, "kind": "eval", "N": N, "k": k, "d": d, "sigma": sigma, "skew": skew}


def listed():
    return [
        # the repository's smallest configuration, whole: four workers, 250 steps of a few microseconds, with Eq. 8
        _train("tiny_four_workers", 100_000, 10, 10, 4, 500, 4, 5, common_start=True, error=True),
        # the benchmark's workload: one epoch over 4 GB of short rows
        _train("streaming", 100_000_000, 10, 10, 1024, 1000, 8, 1),
        # more workers than the device holds at once, 12 GB (the 100 GB configuration at the size that leaves room)
        _train("streaming_many_workers", 300_000_000, 10, 10, 4096, 1000, 16, 1, sigma=2.0),
        # the k = d = 100 configuration with unequal cluster sizes, both of its epochs
        _train("wider_skewed", 20_000_000, 100, 100, 512, 2000, 8, 2, lr=0.02, skew=True),
        # a codebook: 1024 prototypes of 128-dimensional descriptors (the configuration of that shape)
        _train("codebook", 5_000_000, 1024, 128, 256, 4096, 4, 2, lr=0.01),
        # tabular data with an odd number of columns, common start, a few epochs
        _train("table_odd_columns", 2_000_000, 37, 75, 256, 1000, 8, 2, skew=True, common_start=True),
        # long rows (embeddings), fewer workers than compute units
        _train("embeddings", 250_000, 256, 384, 64, 512, 4, 1, lr=0.1),
        # a short row with an odd length and few clusters: sensor data, silent mode with the 1/count step size
        _train("sensors_running_mean", 6_000_000, 12, 7, 256, 500, 0, 1, running_mean=True),
        # exchange after every step (Alg. 5 as printed) with two external buffers per worker (Eq. 3)
        _train("exchange_every_step", 4_000_000, 64, 32, 256, 500, 1, 1, buffers=2, common_start=True),
        # Eq. 8: monitoring the streaming workload, the codebook, and the odd table
        _eval("error_streaming", 100_000_000, 10, 10),
        _eval("error_codebook", 5_000_000, 1024, 128),
        _eval("error_odd_columns", 4_000_000, 37, 75, skew=True),
    ]


def _unnamed(case):
    del case["name"]
    return case


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """Any shape the listed ones stand for: k 2..1024, d 2..512, 4..2048 workers, mini-batches of 100..4096 (the paper:
    500 to 2000), exchange every 1..16 steps or never.  The work of a case is bounded in all, and per worker, by what
    the listed cases cost."""
    sigma, skew = rng.choice([0.5, 1.0, 2.0]), rng.random() < 0.5
    if rng.random() < 0.25:
        k, d = _log(rng, 2, 1024), _log(rng, 2, 512)
        N = min(_log(rng, 20_000, 50_000_000), int(5e10 / (k * d)), int(1e9 / d))
        return _unnamed(_eval("", max(N, 4 * k), k, d, sigma=sigma, skew=skew))
    while True:
        k, d = _log(rng, 2, 1024), _log(rng, 2, 512)
        W, b = _log(rng, 4, 2048), _log(rng, 100, 4096)
        steps = _log(rng, 2, 60)                                   # mini-batches per worker and epoch
        H = max(steps * b + rng.randrange(b), k)
        if W * H * d <= 1e9 and W * H * k * d <= 5e10 and H * k * d <= 2e8 and W * k * d <= 1 << 26:
            break
    mean = rng.random() < 0.15
    E = 0 if mean else rng.choice([0, 1, 2, 4, 8, 16])
    buffers = rng.choice([1, 1, 1, 2]) if E else 1
    parts = rng.choice([1, 1, 1, 2]) if E and k >= 4 and W * k * d <= 1 << 18 else 1
    return _unnamed(_train("", W * H + rng.randrange(W), k, d, W, b, E, rng.choice([1, 2]), lr=rng.choice([0.02, 0.05, 0.1]),
                  sigma=sigma, skew=skew, buffers=buffers, parts=parts, running_mean=mean,
                           common_start=rng.random() < 0.5, error=rng.random() < 0.3))


# ---- inputs ------------------------------------------------------------------------------------------------------
def _samples(case, seed):
    """N x d samples of a mixture of k Gaussians (centres uniform in [0, 10]^d) and a state near its centres."""
    dev, k, d, N = "cuda", case["k"], case["d"], case["N"]
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    centres = torch.rand((k, d), generator=gen, device=dev) * 10.0
    p = 1.0 / torch.arange(1, k + 1, device=dev, dtype=torch.float64) ** 1.1 if case["skew"] else \
        torch.ones(k, device=dev, dtype=torch.float64)
    edges = (torch.cumsum(p, 0) / p.sum())[:-1].float().contiguous()
    X = torch.empty((N, d), device=dev)
    rows = max(1, (1 << 27) // d)
    for lo in range(0, N, rows):
        out = X[lo:lo + rows]
        comp = torch.bucketize(torch.rand(out.shape[0], generator=gen, device=dev), edges)
        out.normal_(0.0, case["sigma"], generator=gen)
        out += centres[comp]
    w0 = centres + case["sigma"] * torch.randn((k, d), generator=gen, device=dev)
    return X, w0.contiguous()


def prepare(case, seed):
    X, w0 = _samples(case, seed)
    if case["kind"] == "eval":
        B.lib()
        return {"case": case, "X": X, "w": w0, "out": torch.zeros(1, dtype=torch.float64, device=X.device)}
    g = B.ASGD(case["k"], case["d"], case["W"], case["b"], case["lr"], E=case["E"], seed=1, buffers=case["buffers"],
               parts=case["parts"], lr_mode=B.LR_INV_COUNT if case["running_mean"] else B.LR_CONST)
    return {"case": case, "X": X, "w0": w0.cpu().numpy(), "g": g}


def run(state):
    case, X = state["case"], state["X"]
    if case["kind"] == "eval":
        B.asgd_quant_error_noalloc(X.data_ptr(), case["N"], case["k"], case["d"], state["w"].data_ptr(),
                                   state["out"].data_ptr(), torch.cuda.current_stream().cuda_stream)
        return state["out"]
    g = state["g"]
    g.load_shards(X)
    if case["common_start"]:
        g.set_state(-1, state["w0"])
    g.run_epochs(case["epochs"])
    if case["W"] * case["k"] * case["d"] * 4 <= ALL_STATES_BYTES:
        out = [g.get_state()]
    else:
        out = [g.get_state(0), g.get_mean_state()]
    if case["error"]:
        out.append(np.array([g.quant_error(0)]))
    return out


def work(case):
    k, d = case["k"], case["d"]
    if case["kind"] == "eval":
        return {"bytes": 4.0 * d * (case["N"] + k), "flops": case["N"] * (2.0 * k * d + k + 3 * d)}
    H = case["N"] // case["W"]
    n = case["epochs"] * (H // case["b"]) * case["b"] * case["W"]
    extra = case["N"] if case["error"] else 0
    return {"bytes": 4.0 * d * (n + extra) + 8.0 * case["W"] * k * d, "flops": (n + extra) * (2.0 * k * d + k + d)}


def tolerance(case):
    """Measured against `exact` over the listed and 16 drawn cases.  Eq. 8: at most 1e-9 off; the sum is 64-bit and a
    sample's distance is good to a few 2^-24.  States: 5e-8 to 2e-6 off, and up to 1e-5 (constant step) or 4e-5 (1/count
    step, whose first steps weigh a sample most) where the rounding of the state moves one sample of a near-tie to the
    other centroid."""
    if case["kind"] == "eval":
        return {"rel": 1e-7}
    return {"rel": 2e-4 if case["running_mean"] else 1e-4}


# ---- the same results in 64 bits ---------------------------------------------------------------------------------
_M64 = (1 << 64) - 1


def _mix(z):
    z = ((z ^ (z >> 30)) * 0xBF58476D1CE4E5B9) & _M64
    z = ((z ^ (z >> 27)) * 0x94D049BB133111EB) & _M64
    return z ^ (z >> 31)


def _shift(seed, r, W, n):
    """Cyclic shift of round r and copy n of the deterministic peer schedule (splitmix64 of the round number)."""
    h = _mix((seed + 0x9E3779B97F4A7C15 * (r + 1)) & _M64)
    return 1 + (h % (W - 1) + n) % (W - 1)


def _nearest(x, w):
    """Nearest row of w[i] for every row of x[i], and the squared distance to it (x: W x b x d, w: W x k x d)."""
    h = 0.5 * (w * w).sum(-1)
    arg = torch.empty(x.shape[:2], dtype=torch.int64, device=x.device)
    dist = torch.empty(x.shape[:2], dtype=x.dtype, device=x.device)
    step = max(1, int(2e8 / (x.shape[1] * w.shape[1])))
    for lo in range(0, x.shape[0], step):
        xs, ws = x[lo:lo + step], w[lo:lo + step]
        s = torch.baddbmm(h[lo:lo + step, None, :], xs, ws.transpose(1, 2).contiguous(), beta=1.0, alpha=-1.0)
        a = s.argmin(-1)
        arg[lo:lo + step] = a
        dist[lo:lo + step] = ((xs - ws.gather(1, a[..., None].expand(-1, -1, xs.shape[2]))) ** 2).sum(-1)
    return arg, dist


def _error(X, w):
    total, rows = 0.0, max(1, int(min(2e8 / w.shape[0], 1e8 / w.shape[1])))
    for lo in range(0, X.shape[0], rows):
        total += 0.5 * float(_nearest(X[None, lo:lo + rows].double(), w[None])[1].sum())
    return total


def exact(case, seed):
    X, w0 = _samples(case, seed)
    if case["kind"] == "eval":
        return torch.tensor([_error(X, w0.double())], dtype=torch.float64, device=X.device)
    k, d, W, b, E, nb, P = (case[q] for q in ("k", "d", "W", "b", "E", "buffers", "parts"))
    H = case["N"] // W
    S = H // b
    eps = float(np.float32(case["lr"]))
    shards = X[:W * H].view(W, H, d)
    w = w0.double().expand(W, k, d).clone() if case["common_start"] else shards[:, :k].double()
    seen = torch.zeros((W, k), dtype=torch.float64, device=X.device)
    rows, workers = torch.arange(k, device=X.device), torch.arange(W, device=X.device)
    sent = None
    for t in range(case["epochs"] * S):
        x = shards[:, (t % S) * b:(t % S) * b + b].double()
        arg, _ = _nearest(x, w)
        cells = (arg + workers[:, None] * k).reshape(-1)
        cnt = torch.bincount(cells, minlength=W * k).view(W, k, 1).double()
        sums = torch.zeros((W * k, d), dtype=torch.float64, device=X.device).index_add_(0, cells, x.reshape(-1, d)).view(W, k, d)
        if case["running_mean"]:
            seen += cnt[..., 0]
            w = torch.where(cnt > 0, w + (sums - cnt * w) / seen.clamp(min=1.0)[..., None], w)
            continue
        g = (cnt * w - sums) / b
        if E > 0 and W > 1 and t > 0 and t % E == 0:
            r = t // E - 1
            taken, total = torch.zeros((W, k, 1), dtype=torch.float64, device=X.device), w.clone()
            for n in range(nb):
                ext = sent[(workers - _shift(1, r, W, n)) % W]
                there = torch.ones((W, k), dtype=torch.bool, device=X.device)
                if P > 1:                                          # the rows that travel in this copy
                    there = (rows[None, :] % P) == ((r + workers + n) % P)[:, None]
                lhs, rhs, nrm = ((v * v).sum(-1) for v in (w - eps * g - ext, w - ext, ext))
                if P == 1:                                         # the whole state is gated at once
                    lhs, rhs, nrm = (v.sum(-1, keepdim=True) for v in (lhs, rhs, nrm))
                ok = (there & (lhs < rhs) & (nrm > 0))[..., None].double()
                taken += ok
                total += ok * ext
            g = torch.where(taken > 0, g + w - total / (taken + 1.0), g)
        w = w - eps * g
        if E > 0 and (t + 1) % E == 0:
            sent = w.clone()
    if W * k * d * 4 <= ALL_STATES_BYTES:
        out = [w]
    else:
        out = [w[0], w.mean(0)]
    if case["error"]:
        out.append(np.array([_error(X, w[0])]))
    return [v.cpu().numpy() if isinstance(v, torch.Tensor) else v for v in out]
