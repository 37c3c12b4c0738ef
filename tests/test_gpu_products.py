"""The grouped matrix products at the edges of their tiles, against the CPU oracle.

One local step with the update kept apart (every product writes its result) and one with it fused.
Bounds: fp32 1e-5, the one-step gate.  bf16 1e-4: oracle and kernels round the same operands, so
one step differs by the fp32 sums (a relative sqrt(K) 2^-24, 5e-6 for the longest contraction here)
and by an operand whose rounding falls the other way: 2^-9 of one of the B terms of a gradient that
moves a weight by gamma = 0.05 times its size.  tanh: no kink that could switch a whole term.
"""
import numpy as np
import pytest
import torch

from helpers import inputs_for, oracle_run, rel_err, small_mlp

pytestmark = pytest.mark.gpu

# dims, batch, workers: contractions of one element, of a whole tile (64 bf16, 32 fp32 elements), one
# less and one more, of several tiles past the depth of the pipeline, and ragged last tiles; output
# tiles of 32, 64 and 128 rows and columns, whole and ragged; worker counts that do and do not fill
# the 8 chiplets evenly
SHAPES = [
    ("bf16", (1, 33, 3), 1, 1),
    ("bf16", (64, 65, 63, 10), 33, 3),
    ("bf16", (127, 128, 129, 37), 65, 6),
    ("bf16", (600, 40, 72, 9), 31, 5),
    ("bf16", (72, 600, 520, 12), 64, 20),            # 64 x 64 tiles
    ("bf16", (72, 520, 130, 12), 64, 32),            # several rounds of tiles
    ("bf16", (72, 1032, 1000, 12), 100, 12),         # 128 x 64 tiles, ragged rows
    ("bf16", (72, 1032, 1024, 12), 128, 12),         # 128 x 64 tiles, whole rows
    ("bf16", (72, 1032, 1000, 12), 160, 16),         # 128-row tiles, ragged contraction and rows
    ("bf16", (40, 66, 70, 80, 50, 30, 9), 33, 3),    # more weight gradients than one launch takes
    ("f32", (40, 66, 70, 80, 50, 30, 9), 33, 3),
    ("bf16", (130, 70), 40, 5),                      # a weight gradient alone in its launch, contraction of one tile
    ("bf16", (130, 70), 200, 3),                     # ... and of several
    ("f32", (130, 70), 40, 5),
    ("f32", (130, 70), 200, 3),
    ("f32", (1, 33, 3), 1, 1),
    ("f32", (31, 32, 33, 10), 33, 3),
    ("f32", (300, 65, 100, 37), 50, 6),
    ("f32", (40, 520, 72, 9), 130, 20),              # 64-row tiles
]


def test_every_tile_is_reached():
    # forward products have the columns of layers 1 and up, backward-data ones those of the hidden layers
    from paper_1807_06629_amd import prsgd as P
    for dtype, tiles in (("bf16", {(32, 64), (64, 64), (128, 64), (128, 128)}), ("f32", {(32, 32), (64, 64)})):
        seen = [{P.prsgd_product_tile(b, d, n, dtype)[:2] for t, dims, b, n in SHAPES if t == dtype for d in dims[1:last]}
                for last in (None, -1)]
        assert seen[0] == tiles and seen[1] == tiles, (dtype, seen)


@pytest.mark.parametrize("dtype,dims,batch,n_workers", SHAPES)
@pytest.mark.parametrize("fused", [True, False])
def test_products_at_tile_edges(dtype, dims, batch, n_workers, fused):
    assert torch.cuda.is_available()
    from paper_1807_06629_amd import drivers as D, prsgd as P
    w = small_mlp(dims=dims, batch=batch, n_workers=n_workers, gemm_dtype=dtype, activation="tanh",
                  rows_per_worker=256, iterations=1)
    inp = inputs_for(w)
    h = D.open_workload(w, inp, device="cuda:0", fused_update=fused)
    P.prsgd_local_steps(h, 1)
    want = oracle_run(w, inp, iterations=1)
    assert rel_err(D.read_all(h), want["x"]) <= (1e-5 if dtype == "f32" else 1e-4)
    assert np.allclose(P.prsgd_read_loss(h), want["losses"], rtol=2e-5 if dtype == "f32" else 2e-3, atol=1e-6)
    P.prsgd_destroy(h)


# 128 x 128 tiles, whose multiplying wavefronts swap fragment sets every tile: contractions of one to five tiles of 64, whole
# and ragged, rows and columns past the last whole tile
@pytest.mark.parametrize("hidden", [8, 64, 65, 128, 190, 192, 256, 300])
def test_contractions_of_the_largest_tiles(hidden):
    assert torch.cuda.is_available()
    from paper_1807_06629_amd import drivers as D, prsgd as P
    dims, batch, n_workers = (40, hidden, 1032, hidden, 12), 160, 16
    assert P.prsgd_product_tile(batch, 1032, n_workers, "bf16")[:2] == (128, 128)
    w = small_mlp(dims=dims, batch=batch, n_workers=n_workers, gemm_dtype="bf16", activation="tanh", rows_per_worker=256,
                  iterations=1)
    inp = inputs_for(w)
    h = D.open_workload(w, inp, device="cuda:0")
    P.prsgd_local_steps(h, 1)
    want = oracle_run(w, inp, iterations=1)
    assert rel_err(D.read_all(h), want["x"]) <= 1e-4
    assert np.allclose(P.prsgd_read_loss(h), want["losses"], rtol=2e-3, atol=1e-6)
    P.prsgd_destroy(h)


# launches of more than two small tiles per compute unit, whose workgroups have no requesting wavefronts: ragged rows, columns
# and contractions of one to four tiles
@pytest.mark.parametrize("dims,batch,n_workers", [
    ((40, 200, 193, 9), 31, 136),                    # 32 x 64 tiles
    ((70, 200, 256, 9), 32, 136),
    ((40, 520, 65, 9), 33, 64),                      # 64 x 64 tiles
    ((130, 513, 520, 9), 64, 64),
])
def test_many_small_tiles(dims, batch, n_workers):
    assert torch.cuda.is_available()
    from paper_1807_06629_amd import drivers as D, prsgd as P
    rows, cols, _ = P.prsgd_product_tile(batch, dims[1], n_workers, "bf16")
    assert rows == (32 if batch <= 32 else 64) and -(-dims[1] // cols) * n_workers > 512
    w = small_mlp(dims=dims, batch=batch, n_workers=n_workers, gemm_dtype="bf16", activation="tanh", rows_per_worker=64,
                  iterations=1)
    inp = inputs_for(w)
    h = D.open_workload(w, inp, device="cuda:0")
    P.prsgd_local_steps(h, 1)
    want = oracle_run(w, inp, iterations=1)
    assert rel_err(D.read_all(h), want["x"]) <= 1e-4
    assert np.allclose(P.prsgd_read_loss(h), want["losses"], rtol=2e-3, atol=1e-6)
    P.prsgd_destroy(h)


# 128 x 64 tiles with requesting wavefronts: contractions of one to five tiles of 64, whole and ragged, rows and columns past the last
# whole tile
@pytest.mark.parametrize("hidden", [8, 64, 65, 128, 190, 300])
def test_contractions_of_tall_narrow_tiles(hidden):
    assert torch.cuda.is_available()
    from paper_1807_06629_amd import drivers as D, prsgd as P
    dims, batch, n_workers = (40, hidden, 456, hidden, 12), 100, 20
    assert P.prsgd_product_tile(batch, 456, n_workers, "bf16")[:2] == (128, 64)
    w = small_mlp(dims=dims, batch=batch, n_workers=n_workers, gemm_dtype="bf16", activation="tanh", rows_per_worker=256,
                  iterations=1)
    inp = inputs_for(w)
    h = D.open_workload(w, inp, device="cuda:0")
    P.prsgd_local_steps(h, 1)
    want = oracle_run(w, inp, iterations=1)
    assert rel_err(D.read_all(h), want["x"]) <= 1e-4
    assert np.allclose(P.prsgd_read_loss(h), want["losses"], rtol=2e-3, atol=1e-6)
    P.prsgd_destroy(h)


# fp32 tiles of 32 x 32 with and without requesting wavefronts (up to two workgroups per compute unit, and more): contractions of one
# element to five tiles of 32, whole and ragged
@pytest.mark.parametrize("n_workers", [2, 68])
@pytest.mark.parametrize("hidden", [1, 32, 33, 63, 96, 131, 160])
def test_fp32_contractions_of_small_tiles(hidden, n_workers):
    assert torch.cuda.is_available()
    from paper_1807_06629_amd import drivers as D, prsgd as P
    dims, batch = (40, hidden, 250, hidden, 12), 31
    assert P.prsgd_product_tile(batch, 250, n_workers, "f32")[:2] == (32, 32) and (8 * n_workers > 512) == (n_workers == 68)
    w = small_mlp(dims=dims, batch=batch, n_workers=n_workers, gemm_dtype="f32", activation="tanh", rows_per_worker=64, iterations=1)
    inp = inputs_for(w)
    h = D.open_workload(w, inp, device="cuda:0")
    P.prsgd_local_steps(h, 1)
    want = oracle_run(w, inp, iterations=1)
    assert rel_err(D.read_all(h), want["x"]) <= 1e-5
    assert np.allclose(P.prsgd_read_loss(h), want["losses"], rtol=2e-5, atol=1e-6)
    P.prsgd_destroy(h)
