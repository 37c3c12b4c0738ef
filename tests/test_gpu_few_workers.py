"""Layers of whole tiles whose walk over the weights few workers do not repay: products of their own, around the lines of that rule.

Bounds: 1e-4 after one step (tests/test_gpu_products.py), 5e-3 and 2e-2 of the other short bf16 runs behind it.
"""
import numpy as np
import pytest
import torch

from helpers import inputs_for, oracle_run, rel_err, small_mlp

pytestmark = pytest.mark.gpu


# Backward launches of a step: one per walked layer; two of the three layers apart are two backward-data products and a launch of weight
# gradients beside the walk of the first, all three apart are three.
@pytest.mark.parametrize("dims,batch,n,launches", [
    ((128, 256, 896, 10), 32, 2, 4),              # 14 column tiles: the second layer apart (its bands: 8), and the last one with it
    ((128, 256, 832, 10), 32, 2, 4),              # 13: an odd number, no whole-tile walk
    ((128, 256, 768, 10), 32, 2, 3),              # 12: walked, and the last one by itself as well
    ((128, 768, 768, 10), 64, 6, 4),              # 72 bands of the second layer: apart
    ((128, 768, 768, 10), 64, 7, 3),              # 84: walked
    ((128, 256, 512, 10), 128, 2, 4),             # 8 column tiles
    ((128, 256, 448, 10), 128, 2, 4),             # 7: an odd number
    ((128, 256, 384, 10), 128, 2, 3),             # 6: walked
    ((640, 512, 10), 128, 3, 2),                  # a first layer apart: 30 bands of 8 column tiles
    ((640, 512, 512, 10), 128, 3, 3),             # ... and the layers behind it (four if it were walked)
])
def test_layers_apart_and_walked(dims, batch, n, launches):
    assert torch.cuda.is_available()
    from paper_1807_06629_amd import drivers as D, prsgd as P
    w = small_mlp(dims=dims, batch=batch, n_workers=n, gemm_dtype="bf16", activation="tanh", rows_per_worker=64, lr=0.01, interval=3,
                  iterations=7)
    inp = inputs_for(w)
    outs = []
    for first in (True, False):
        h = D.open_workload(w, inp)
        P.prsgd_set_first_layer_fusion(h, first)
        P.prsgd_profile_enable(h, True)
        P.prsgd_local_steps(h, 1)
        counts = {r["name"]: r["launches"] for r in P.prsgd_profile_read(h)}
        assert counts["gemm_bwd"] == launches and not counts.get("gemm_bwd_first")
        assert rel_err(D.read_all(h), oracle_run(w, inp, iterations=1)["x"]) <= 1e-4
        P.prsgd_destroy(h)
        h = D.open_workload(w, inp)
        P.prsgd_set_first_layer_fusion(h, first)
        P.prsgd_run(h, w.iterations, w.interval)
        outs.append((D.read_all(h), P.prsgd_read_loss(h)))
        P.prsgd_destroy(h)
    want = oracle_run(w, inp)
    for x, loss in outs:
        assert rel_err(x, want["x"]) <= 5e-3
        assert np.allclose(loss, want["losses"], rtol=2e-2, atol=2.0 ** -20)


# momentum in the weight gradients' launch: few and many bands, one layer and several of ragged widths, tiles of 64 and of 128, whole layers
# whose walk is too long, one row and 128, and (20 workers) layers walked with momentum.  Backward launches of a step where they tell layers
# apart from walked ones: six layers are seven launches, the head takes the delta below 30 classes, a fused first layer is counted elsewhere.
@pytest.mark.parametrize("dims,batch,n,launches", [
    ((130, 70), 40, 5, None), ((300, 200, 10), 33, 3, None), ((40, 66, 70, 80, 50, 30, 9), 33, 3, 7), ((65, 129, 64, 30), 1, 2, 2),
    ((1000, 1030, 20), 100, 8, None), ((1024, 1024, 1024, 10), 128, 2, 3), ((2000, 1300, 10), 24, 20, 1),
])
@pytest.mark.parametrize("restart", ["keep", "average", "reset"])
def test_momentum_of_layers_apart(dims, batch, n, launches, restart):
    momentum_against_oracle(dims, batch, n, launches, restart)


def test_momentum_of_streamed_layers_apart():
    """Velocities read and written non-temporally in 128 x 128 tiles: the second and third layer apart behind a fused first one."""
    momentum_against_oracle((3001, 3003, 3002, 10), 24, 3, 3, "keep", streamed=True)


def momentum_against_oracle(dims, batch, n, launches, restart, streamed=None):
    assert torch.cuda.is_available()
    from paper_1807_06629_amd import drivers as D, prsgd as P
    w = small_mlp(dims=dims, batch=batch, n_workers=n, gemm_dtype="bf16", activation="tanh", rows_per_worker=64, lr=0.002, interval=2,
                  iterations=5).scaled(momentum=0.9, momentum_restart=restart)
    inp = inputs_for(w)
    h = D.open_workload(w, inp)
    if streamed is not None:
        assert bool(P.prsgd_streamed_uses(h.cfg) & P.PRSGD_STREAM_STEPS) == streamed
    P.prsgd_profile_enable(h, True)
    P.prsgd_run(h, w.iterations, w.interval)
    counts = {r["name"]: r["launches"] for r in P.prsgd_profile_read(h)}
    assert counts["gemm_bwd"] == w.iterations * launches if launches else "gemm_bwd" in counts
    assert restart == "reset" or not counts.get("sgd_update")
    want = oracle_run(w, inp, momentum=0.9, momentum_restart=restart)
    assert rel_err(D.read_all(h), want["x"]) <= 5e-3
    v = np.stack([P.prsgd_read_velocity(h, i) for i in range(n)])
    assert rel_err(v, want["v"]) <= 2e-2                  # the bounds of the other momentum runs with bf16 operands
    P.prsgd_destroy(h)
