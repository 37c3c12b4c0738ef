"""The work that users of this framework have it do, as cases that can be timed and compared.

A case is one training problem (objective, layer widths, workers, minibatch, options) and the stretch of
iterations that one pass covers.  Every pass goes through the public calls of the package: Algorithm 1
(`drivers.run_algorithm1`), the epochs of Algorithms 2 and 3 (`drivers.run_algorithm2` / `_3`), and for
the small least-squares problem the read-out of the result.

A context keeps every worker's point in its replica buffer, which is what a pass returns.  Right after a
restart the library may hold the common point elsewhere, so a pass of Algorithm 1 is laid out to end one
local step after a restart: the iteration counter starts at 1 (a run resumed one step into an epoch) and
every pass takes whole intervals from there.  With interval 1 its last iteration is a bare local step.
"""
import math
import weakref

import numpy as np
import torch

from paper_1807_06629_amd import drivers, prsgd

ON_CHIP_BYTES = 256e6        # what the last-level cache holds: beyond it the parameters cross HBM every iteration


def _mlp(name, dims, n_workers, batch, interval, iterations, lr, dtype="bf16", activation="relu", rows=8192,
         momentum=0.0, alpha=0.0, algorithm=1):
    return {"name": name, "model": "mlp", "dims": "-".join(str(d) for d in dims), "n_workers": n_workers,
            "batch": batch, "rows": rows, "dtype": dtype, "activation": activation, "lr": lr,
            "momentum": momentum, "alpha": alpha, "algorithm": algorithm, "interval": interval,
            "iterations": iterations}


def listed():
    return [
        # a small convex problem solved from start to end, and its answer read: launches and latency
        {"name": "lsq_n4_d64", "model": "lsq", "dims": "64", "n_workers": 4, "batch": 16, "rows": 4096,
         "dtype": "f32", "activation": "none", "lr": 0.01, "momentum": 0.0, "alpha": 0.0, "algorithm": 1,
         "interval": 8, "iterations": 256},
        # many small replicas, averaged after every step (parallel mini-batch SGD) ...
        _mlp("small_fp32_n64_i1", (256, 128, 10), 64, 8, 1, 64, 0.02, "f32"),
        # ... and at a longer interval
        _mlp("small_fp32_n64_i8", (256, 128, 10), 64, 8, 8, 64, 0.02, "f32"),
        # a one-hidden-layer classifier on image-sized rows, all in fp32
        _mlp("fp32_784_256_10_i16", (784, 256, 10), 8, 32, 16, 64, 0.05, "f32", "tanh"),
        # fp32 with two hidden layers of ragged widths and a minibatch that fills no tile
        _mlp("fp32_784_300_100_10_i4", (784, 300, 100, 10), 8, 50, 4, 16, 0.02, "f32", "tanh"),
        # the mid-sized bf16 classifier on unlike shards, long interval
        _mlp("bf16_3072_1024_n16_i32", (3072, 1024, 1024, 10), 16, 64, 32, 32, 0.05, alpha=0.3),
        # the same net trained with momentum, the local step of the paper's experiment
        _mlp("bf16_3072_1024_n16_mom", (3072, 1024, 1024, 10), 16, 64, 16, 16, 0.002, momentum=0.9, alpha=0.3),
        # widths, minibatch and worker count that are multiples of nothing
        _mlp("bf16_1000_500_300_37_n6", (1000, 500, 300, 37), 6, 100, 4, 16, 0.01),
        # workers of unlike speed: Algorithm 3, epochs of one to four local steps
        _mlp("bf16_3072_1024_n16_alg3", (3072, 1024, 1024, 10), 16, 64, 4, 8, 0.002, alpha=0.3, algorithm=3),
        # large minibatches per worker: the matrix products weigh more than the parameters' traffic
        _mlp("bf16_3072_1024_n8_b512", (3072, 1024, 1024, 10), 8, 512, 8, 8, 0.005),
        # large replicas: every iteration streams all parameters of all workers through HBM
        _mlp("bf16_4096x3_1000_n8_i16", (4096, 4096, 4096, 4096, 1000), 8, 128, 16, 16, 0.01),
        # large replicas averaged after every step: one shared weight stream, products over all minibatches
        _mlp("bf16_4096x3_1000_n8_i1", (4096, 4096, 4096, 4096, 1000), 8, 128, 1, 16, 0.01),
    ]


def _log_int(rng, low, high):
    return int(round(math.exp(rng.uniform(math.log(low), math.log(high)))))


def _width(rng, low, high):
    """A layer width: as often a round one as one that is a multiple of nothing."""
    d = _log_int(rng, low, high)
    return max(low, d // 64 * 64) if rng.random() < 0.5 and d >= 128 else d


def draw(rng):
    """One more case of the listed ones' ranges."""
    kind = rng.choice(["lsq", "f32_one", "f32_one", "f32_deep", "bf16", "bf16", "bf16", "bf16_large"])
    if kind == "lsq":
        interval = _log_int(rng, 1, 32)
        d = _log_int(rng, 16, 512)
        return {"model": "lsq", "dims": str(d), "n_workers": _log_int(rng, 2, 64), "batch": _log_int(rng, 4, 64),
                "rows": 4096, "dtype": "f32", "activation": "none", "lr": 0.5 / max(d, 50), "momentum": 0.0,
                "alpha": 0.0, "algorithm": 1, "interval": interval, "iterations": interval * max(1, 128 // interval)}
    algorithm = rng.choice([1, 1, 1, 1, 2, 3])
    momentum = 0.9 if algorithm == 1 and rng.random() < 0.2 else 0.0
    alpha = rng.choice([0.0, 0.3])
    activation = rng.choice(["relu", "tanh"])
    interval = _log_int(rng, 1, 32)
    if kind == "f32_one":
        dims = (_width(rng, 64, 1024), _width(rng, 32, 256), rng.randint(4, 16))
        n, b, dtype, iterations = _log_int(rng, 2, 64), _log_int(rng, 4, 64), "f32", 48
    elif kind == "f32_deep":
        dims = (_width(rng, 128, 1024), _width(rng, 64, 512), _width(rng, 32, 256), rng.randint(5, 100))
        n, b, dtype, iterations = _log_int(rng, 2, 16), _log_int(rng, 8, 128), "f32", 16
    elif kind == "bf16":
        dims = (_width(rng, 512, 4096),) + tuple(_width(rng, 256, 1536) for _ in range(rng.randint(1, 3))) + \
            (_log_int(rng, 5, 500),)
        n, b, dtype, iterations = _log_int(rng, 2, 16), rng.choice([32, 64, 128, _log_int(rng, 16, 512)]), "bf16", 16
    else:
        dims = (_width(rng, 2048, 4096),) + tuple(_width(rng, 2048, 4096) for _ in range(rng.randint(2, 3))) + \
            (_log_int(rng, 100, 1000),)
        n, b, dtype, iterations = rng.randint(4, 8), rng.choice([32, 64, 128, rng.randint(24, 128)]), "bf16", 16
        interval, momentum, alpha = rng.choice([1, 4, 16]), 0.0, 0.0
    if algorithm == 3:
        interval = min(interval, 8)                      # the longest epoch of any worker
    iterations = interval * max(1, iterations // interval)
    lr = (0.002 if momentum else 0.01) * min(1.0, 1024.0 / dims[0])
    case = _mlp("", dims, n, b, interval, iterations, lr, dtype, activation, 4096, momentum, alpha, algorithm)
    del case["name"]
    return case


def _dims(case):
    return tuple(int(d) for d in case["dims"].split("-"))


class _State:
    """What a training program holds: the context with its tensors, and its schedule."""

    def __init__(self, handle, case):
        self.handle = handle
        self.case = case
        self.algorithm, self.interval, self.iterations = case["algorithm"], case["interval"], case["iterations"]
        n = case["n_workers"]
        # Algorithm 3: worker i takes between one step and the whole interval
        self.worker_steps = [1 + i % self.interval for i in range(n)]
        # Algorithm 2: epochs of growing length at falling rates
        self.lengths, self.rates = [], []
        left, k = self.iterations, 1
        while left > 0:
            step = min(k, left, self.interval)
            self.lengths.append(step)
            self.rates.append(case["lr"] / (1.0 + 0.1 * len(self.lengths)))
            left, k = left - step, k + 1
        weakref.finalize(self, prsgd.prsgd_destroy, handle)


def prepare(case, seed):
    dims, n, rows = _dims(case), case["n_workers"], case["rows"]
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    features = torch.empty((n, rows, dims[0]), dtype=torch.float32, device=dev)
    features.normal_(generator=g)
    if case["model"] == "lsq":
        truth = torch.randn(dims[0], generator=g, device=dev)
        targets = features @ truth + 0.1 * torch.randn((n, rows), generator=g, device=dev)
        x0 = np.zeros(dims[0], dtype=np.float32)
    else:
        classes = dims[-1]
        means = torch.randn((classes, dims[0]), generator=g, device=dev)
        targets = torch.empty((n, rows), dtype=torch.int32, device=dev)
        shares = np.random.default_rng(seed)
        for i in range(n):
            if case["alpha"] > 0.0:                      # every worker its own class proportions
                p = torch.from_numpy(shares.dirichlet(np.full(classes, case["alpha"]))).to(dev)
                label = torch.multinomial(p, rows, replacement=True, generator=g)
            else:
                label = torch.randint(classes, (rows,), generator=g, device=dev)
            targets[i] = label
            features[i] += means[label]
        scale = 2.0 if case["activation"] == "relu" else 1.0
        parts = []
        for d_in, d_out in zip(dims, dims[1:]):
            parts.append(torch.randn(d_in * d_out, generator=g, device=dev) * math.sqrt(scale / d_in))
            parts.append(torch.zeros(d_out, device=dev))
        x0 = torch.cat(parts).cpu().numpy()
    cfg = prsgd.make_config(n, case["model"], dims, case["batch"], rows, case["lr"], seed,
                            activation=case["activation"], gemm_dtype=case["dtype"], momentum=case["momentum"])
    handle = prsgd.prsgd_init(cfg, x0, features, targets)
    if case["algorithm"] == 1 and case["interval"] > 1:
        prsgd.prsgd_set_iteration(handle, 1)
    return _State(handle, case)


def run(state):
    h = state.handle
    if state.algorithm == 2:
        drivers.run_algorithm2(h, state.lengths, state.rates)
    elif state.algorithm == 3:
        drivers.run_algorithm3(h, state.worker_steps, state.iterations // state.interval)
    elif state.interval == 1:
        drivers.run_algorithm1(h, state.iterations - 1, 1)
        prsgd.prsgd_local_steps(h, 1)
    else:
        drivers.run_algorithm1(h, state.iterations, state.interval)
    if state.case["model"] == "lsq":
        return {"replicas": h.params, "average": prsgd.prsgd_read_params(h, -1)}
    return {"replicas": h.params}


def work(case):
    dims, n, b, iterations = _dims(case), case["n_workers"], case["batch"], case["iterations"]
    if case["model"] == "lsq":
        m = dims[0]
        return {"bytes": 4.0 * n * (iterations * b * (m + 1) + 2 * m), "flops": 4.0 * n * b * m * iterations}
    weights = [d_in * d_out for d_in, d_out in zip(dims, dims[1:])]
    m = sum(weights) + sum(dims[1:])
    steps = n * iterations                               # local steps of all workers
    if case["algorithm"] == 3:
        steps = sum(1 + i % case["interval"] for i in range(n)) * (iterations // case["interval"])
    # forward, weight gradient, and the delta of every layer but the first: 2 operations per weight and row each
    flops = steps * b * (6.0 * sum(weights) - 2.0 * weights[0])
    state_bytes = 4.0 * m * n * (2 if case["momentum"] else 1)
    rows_read = 4.0 * steps * b * (dims[0] + 1)
    if case["algorithm"] == 1 and case["interval"] == 1:
        # all workers stand at the same point: one read and one write of it per iteration, the replicas once
        once, passes = 8.0 * m, iterations if 4.0 * m > ON_CHIP_BYTES / 4 else 1
        return {"bytes": rows_read + once * passes + 4.0 * m * n, "flops": flops}
    # every local step rewrites its worker's point; a set that the chip can hold crosses HBM once
    passes = steps / n if state_bytes > ON_CHIP_BYTES else 1
    return {"bytes": rows_read + 2.0 * state_bytes * passes, "flops": flops}


def tolerance(case):
    """Four times the largest difference measured on these ranges over two passes: fp32 against the same run in
    64 bits (least squares 2.7e-7, nets 3.9e-7; single values 1e-5 between two orders of summation), bf16
    between the fused and the separate kernels (1.7e-4; single values 6e-3, where one operand's rounding or
    one unit's kink falls the other way)."""
    if case["model"] == "lsq":
        return {"rel": 1e-6, "max": 2e-5}
    if case["dtype"] == "f32":
        return {"rel": 2e-6, "max": 4e-5}
    return {"rel": 7e-4, "max": 2.5e-2}
