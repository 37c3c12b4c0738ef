"""The loss head that multiplies a narrow logits layer itself, at the edges of its tiles, against the CPU oracle.

The bounds are those of the grouped products: fp32 1e-5, the one-step gate; bf16 1e-4, since oracle and kernels round
the same operands and one step differs by its fp32 sums and by an operand whose rounding falls the other way.
"""
import numpy as np
import pytest
import torch

from helpers import inputs_for, oracle_run, rel_err, small_mlp

pytestmark = pytest.mark.gpu

# (dtype, width in front of the logits, classes, batch, workers, whether the head takes the product): class tiles of 16 and
# 64, whole and ragged; blocks of 16 rows; contractions of one element, around a piece (bf16 256 and 64, fp32 64 and 32
# elements per wavefront) and a round of four, and the largest whose weights are 128 KB and one beyond
SHAPES = [
    ("bf16", 1, 1, 1, 1, True),
    ("bf16", 255, 16, 15, 3, True),
    ("bf16", 257, 7, 16, 2, True),
    ("bf16", 1032, 10, 17, 2, True),
    ("bf16", 4097, 16, 33, 2, True),                 # any width up to 16 classes
    ("bf16", 63, 17, 16, 5, True),
    ("bf16", 65, 33, 31, 3, True),
    ("bf16", 263, 64, 129, 2, True),
    ("bf16", 1024, 64, 20, 2, True),
    ("bf16", 1025, 64, 20, 2, False),
    ("bf16", 72, 65, 20, 2, False),
    ("f32", 1, 1, 1, 1, True),
    ("f32", 63, 9, 15, 3, True),
    ("f32", 65, 16, 17, 2, True),
    ("f32", 259, 3, 130, 2, True),
    ("f32", 2048, 16, 16, 2, True),
    ("f32", 2049, 16, 16, 2, False),
    ("f32", 31, 17, 16, 5, True),
    ("f32", 33, 41, 33, 3, True),
    ("f32", 130, 64, 65, 2, True),
    ("f32", 512, 64, 20, 2, True),
    ("f32", 513, 64, 20, 2, False),
    ("f32", 512, 20, 20, 2, True),                   # tiles of 64 count, not the classes' own bytes
    ("f32", 1024, 17, 20, 2, False),
]


@pytest.mark.parametrize("dtype,width,classes,batch,n_workers,inside", SHAPES)
def test_logits_inside_the_head(dtype, width, classes, batch, n_workers, inside):
    assert torch.cuda.is_available()
    from paper_1807_06629_amd import drivers as D, prsgd as P
    w = small_mlp(dims=(24, 40, width, classes), batch=batch, n_workers=n_workers, gemm_dtype=dtype,
                  rows_per_worker=256, iterations=1)
    inp = inputs_for(w)
    h = D.open_workload(w, inp, device="cuda:0")
    P.prsgd_local_steps(h, 1)
    want = oracle_run(w, inp, iterations=1)
    assert rel_err(D.read_all(h), want["x"]) <= (1e-5 if dtype == "f32" else 1e-4)
    assert np.allclose(P.prsgd_read_loss(h), want["losses"], rtol=2e-5 if dtype == "f32" else 2e-3, atol=1e-6)
    P.prsgd_profile_enable(h, True)
    P.prsgd_local_steps(h, 1)
    launches = {r["name"]: r["launches"] for r in P.prsgd_profile_read(h)}
    assert launches["gemm_fwd"] == (2 if inside else 3), launches
    P.prsgd_destroy(h)


# (dtype, width in front of the logits, classes, batch, workers, whether the head takes the delta): tiles of 16 units, whole and
# ragged, one and more per wavefront and past a round of four each; rows in blocks of 16; contractions of one class, of 16,
# around 32 and of 64.  bf16 with more than 128 rows, whose products are apart.  Widths at the limits of the head, with few and with
# many workgroups of 16 rows, and far beyond them
BELOW = [
    ("f32", 1, 1, 1, 3, True), ("f32", 8, 16, 16, 3, True), ("f32", 17, 17, 15, 3, True), ("f32", 64, 10, 33, 3, True),
    ("f32", 65, 9, 17, 3, True), ("f32", 256, 64, 31, 3, True), ("f32", 263, 33, 16, 3, False), ("f32", 1030, 5, 20, 3, False),
    ("f32", 640, 16, 17, 3, True), ("f32", 641, 16, 17, 3, False), ("f32", 448, 10, 144, 15, True), ("f32", 449, 10, 144, 15, False),
    ("f32", 64, 64, 128, 8, True), ("f32", 64, 64, 80, 13, False), ("f32", 256, 40, 80, 13, True), ("f32", 2048, 10, 16, 2, False),
    ("bf16", 1, 1, 129, 3, True), ("bf16", 8, 16, 144, 3, True), ("bf16", 17, 17, 130, 3, True), ("bf16", 64, 10, 145, 3, True),
    ("bf16", 65, 24, 129, 3, True), ("bf16", 263, 32, 160, 3, True), ("bf16", 256, 64, 129, 3, True), ("bf16", 1030, 10, 131, 3, False),
    ("bf16", 768, 10, 131, 3, True), ("bf16", 511, 40, 129, 3, True), ("bf16", 513, 24, 129, 3, False), ("bf16", 769, 10, 131, 3, False),
    ("bf16", 448, 64, 129, 3, True), ("bf16", 449, 64, 129, 3, False), ("bf16", 448, 10, 160, 13, True), ("bf16", 449, 10, 160, 13, False),
    ("bf16", 40, 64, 256, 16, True), ("bf16", 40, 64, 256, 17, False), ("bf16", 4096, 10, 129, 2, False),
]


@pytest.mark.parametrize("activation", ["tanh", "relu"])
@pytest.mark.parametrize("dtype,width,classes,batch,n_workers,inside", BELOW)
def test_delta_below_the_head(dtype, width, classes, batch, n_workers, inside, activation):
    assert torch.cuda.is_available()
    from paper_1807_06629_amd import drivers as D, prsgd as P
    w = small_mlp(dims=(24, 40, width, classes), batch=batch, n_workers=n_workers, gemm_dtype=dtype, activation=activation,
                  rows_per_worker=256, iterations=1)
    inp = inputs_for(w)
    h = D.open_workload(w, inp, device="cuda:0")
    P.prsgd_local_steps(h, 1)
    want = oracle_run(w, inp, iterations=1)
    # relu in bf16: a pre-activation within the fp32 sums' error of the kink may fall on its other side and switch
    # gamma / B of a column, 0.05 / 129 of a gradient's size
    assert rel_err(D.read_all(h), want["x"]) <= (1e-5 if dtype == "f32" else 1e-4 if activation == "tanh" else 5e-4)
    assert np.allclose(P.prsgd_read_loss(h), want["losses"], rtol=2e-5 if dtype == "f32" else 2e-3, atol=1e-6)
    P.prsgd_profile_enable(h, True)
    P.prsgd_local_steps(h, 1)
    launches = {r["name"]: r["launches"] for r in P.prsgd_profile_read(h)}
    assert launches["gemm_dx"] == (1 if inside else 2), launches            # layer 2's, and the head's own
    P.prsgd_destroy(h)


# Ragged nets whose layers' products are apart with at most 128 rows: one launch for all weight gradients, one for each delta that
# the head does not take
@pytest.mark.parametrize("dims,batch,n_workers,launches", [
    ((40, 30, 20, 37), 100, 3, 2),
    ((300, 200, 24), 33, 8, 1),
    ((40, 70, 300, 64), 128, 3, 2),
    ((40, 70, 513, 17), 100, 3, 3),                      # beyond the head's units
    ((40, 30, 449, 64), 100, 3, 3),                      # ... and its weights
])
def test_delta_below_the_head_of_ragged_nets(dims, batch, n_workers, launches):
    assert torch.cuda.is_available()
    from paper_1807_06629_amd import drivers as D, prsgd as P
    w = small_mlp(dims=dims, batch=batch, n_workers=n_workers, gemm_dtype="bf16", activation="tanh", rows_per_worker=256,
                  iterations=1)
    inp = inputs_for(w)
    h = D.open_workload(w, inp, device="cuda:0")
    P.prsgd_local_steps(h, 1)
    want = oracle_run(w, inp, iterations=1)
    assert rel_err(D.read_all(h), want["x"]) <= 1e-4
    assert np.allclose(P.prsgd_read_loss(h), want["losses"], rtol=2e-3, atol=1e-6)
    P.prsgd_profile_enable(h, True)
    P.prsgd_local_steps(h, 1)
    counts = {r["name"]: r["launches"] for r in P.prsgd_profile_read(h)}
    assert counts["gemm_bwd"] == launches, counts
    P.prsgd_destroy(h)


# The pass that steps and restarts at once, whose head reads weights shared by all workers; the bounds are those of the other
# interval-one runs
@pytest.mark.parametrize("dims,batch,n_workers", [
    ((100, 72, 40, 37), 24, 4), ((64, 130, 256, 64), 128, 2), ((72, 96, 300, 24), 33, 5), ((80, 64, 640, 10), 64, 8),
])
@pytest.mark.parametrize("activation", ["relu", "tanh"])
def test_delta_below_the_head_at_interval_one(dims, batch, n_workers, activation):
    assert torch.cuda.is_available()
    from paper_1807_06629_amd import drivers as D, prsgd as P
    w = small_mlp(dims=dims, batch=batch, n_workers=n_workers, gemm_dtype="bf16", activation=activation, rows_per_worker=256,
                  interval=1, iterations=5)
    inp = inputs_for(w)
    h = D.open_workload(w, inp, device="cuda:0")
    P.prsgd_profile_enable(h, True)
    P.prsgd_run(h, w.iterations, 1)
    counts = {r["name"]: r["launches"] for r in P.prsgd_profile_read(h)}
    assert counts["gemm_dx"] == w.iterations, counts     # layer 2's only
    want = oracle_run(w, inp)
    assert np.all(np.abs(P.prsgd_read_loss(h) - want["losses"]) <= 2e-2 * np.abs(want["losses"]) + 2.0 ** -20)
    assert rel_err(D.read_all(h), want["x"]) <= 5e-3
    P.prsgd_destroy(h)


# Class counts whose contraction of D_{L-1} goes past the last column of W_L: that part of it is zero times zero
@pytest.mark.parametrize("dtype,classes,batch", [("f32", 5, 20), ("f32", 20, 20), ("bf16", 10, 144), ("bf16", 40, 144)])
def test_infinite_weight_below_the_head(dtype, classes, batch):
    assert torch.cuda.is_available()
    from paper_1807_06629_amd import drivers as D, prsgd as P
    dims, unit = (24, 40, 64, classes), 5
    w = small_mlp(dims=dims, batch=batch, n_workers=2, gemm_dtype=dtype, activation="relu", rows_per_worker=256,
                  iterations=1)
    inp = inputs_for(w)
    b2 = 24 * 40 + 40 + 40 * 64
    inp["targets"][:] = 0                                # every row's own class is the one that cannot be reached:
    inp["x0"][b2 + unit] = 50.0                          # the unit is active, its logit -inf, D = -1 / B there
    inp["x0"][b2 + 64 + unit * classes] = -np.inf
    h = D.open_workload(w, inp, device="cuda:0")
    P.prsgd_local_steps(h, 1)
    bias = D.read_all(h)[:, b2:b2 + 64]
    assert np.all(np.isneginf(bias[:, unit])), bias[:, unit]
    assert np.isfinite(np.delete(bias, unit, axis=1)).all()
    assert np.all(np.isposinf(P.prsgd_read_loss(h)))
    P.prsgd_destroy(h)
