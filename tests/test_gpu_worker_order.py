"""Algorithm 3 layer by layer: launches hold the workers that take the step, by falling step counts.

Bounds against the oracle: fp32 1e-4, the gate of short multi-step runs; bf16 5e-3, that of the other heterogeneous runs.
"""
import numpy as np
import pytest
import torch

import oracle
from helpers import inputs_for, oracle_args, rel_err, small_mlp

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    assert torch.cuda.is_available(), "these tests need the GPU"
    from paper_1807_06629_amd import prsgd
    return prsgd


@pytest.fixture(scope="module")
def D():
    from paper_1807_06629_amd import drivers
    return drivers


# equal counts apart from each other, workers without a step, one worker that goes on alone, every worker alike, and more
# workers than integers travel in one launch; fp32 and bf16, whole tiles (whose first layer is fused while workers go on) and ragged
# ones, a narrow and a wide head, and the update as a launch of its own
@pytest.mark.parametrize("dtype,dims,batch,steps,fused", [
    ("bf16", (256, 128, 64, 10), 32, [2, 4, 1, 4, 2, 1, 3, 4, 1], True),
    ("bf16", (256, 128, 64, 10), 64, [1, 1, 5, 1, 0, 1, 1, 1, 2], True),
    ("bf16", (256, 64, 300), 32, [3, 1, 2, 3], True),
    ("bf16", (100, 72, 40, 10), 24, [0, 3, 1, 2, 3, 0, 1], True),
    ("bf16", (72, 136, 40, 10), 160, [2, 1, 3], True),
    ("bf16", (100, 72, 40, 10), 24, [1, 3, 2], False),
    ("f32", (60, 50, 40, 10), 20, [0, 3, 1, 2, 3, 0, 1], True),
    ("f32", (60, 50, 40, 300), 20, [2, 3, 1], True),
    ("f32", (60, 50, 40, 10), 20, [2, 1, 4, 1], False),
    ("f32", (12, 9, 8, 5), 4, [1 + (7 * i) % 4 for i in range(300)], True),
])
def test_workers_of_unlike_speed(P, D, dtype, dims, batch, steps, fused):
    n = len(steps)
    w = small_mlp(dims=dims, batch=batch, n_workers=n, gemm_dtype=dtype, activation="tanh", rows_per_worker=64, lr=0.02)
    inp = inputs_for(w)
    h = D.open_workload(w, inp, fused_update=fused)
    D.run_algorithm3(h, steps, 2)
    t = 2 * max(steps)
    want = oracle.run_heterogeneous(**oracle_args(w, inp), lr=w.lr, worker_steps=steps, n_epochs=2)
    assert P.prsgd_iteration(h) == t == want["t"]
    assert rel_err(D.read_all(h), want["x"]) <= (1e-4 if dtype == "f32" else 5e-3)
    # every worker's rows and loss are those of the last step that it took
    rows, loss = P.prsgd_read_indices(h), P.prsgd_read_loss(h)
    for i in range(n):
        if steps[i] > 0:
            last = t - max(steps) + steps[i]
            assert np.array_equal(rows[i], oracle.sample_rows(w.index_seed, i, last, batch, 64)), i
            assert np.allclose(loss[i], want["losses"][i], rtol=1e-3 if dtype == "f32" else 2e-2, atol=1e-6), i
    # a step of all workers goes on from there: no draw of the epoch is taken for its own
    P.prsgd_local_steps(h, 1)
    rows = P.prsgd_read_indices(h)
    for i in range(n):
        assert np.array_equal(rows[i], oracle.sample_rows(w.index_seed, i, t + 1, batch, 64)), i
    P.prsgd_destroy(h)


@pytest.mark.parametrize("steps_before", [0, 1, 2])
@pytest.mark.parametrize("steps", [[3, 1, 2, 3, 1], [4, 4, 0, 1, 4]])
def test_first_layer_of_the_workers_that_go_on(P, D, steps, steps_before):
    """The first layer fused with the next forward product for the workers that take another step, and apart for the others: same
    bits as with every product apart, also behind local steps that left the shadows of W_1 as they were."""
    w = small_mlp(dims=(256, 128, 10), batch=32, n_workers=5, gemm_dtype="bf16", activation="relu", rows_per_worker=64)
    inp = inputs_for(w)
    outs = []
    for on in (True, False):
        h = D.open_workload(w, inp)
        P.prsgd_set_first_layer_fusion(h, on)
        P.prsgd_local_steps(h, steps_before)
        P.prsgd_local_steps_hetero(h, steps)
        P.prsgd_local_steps_hetero(h, steps)              # from points that differ
        P.prsgd_average(h)
        P.prsgd_local_steps_hetero(h, steps)              # from the average
        P.prsgd_local_steps(h, 2)
        outs.append((D.read_all(h), P.prsgd_read_loss(h), P.prsgd_read_indices(h)))
        P.prsgd_destroy(h)
    for a, b in zip(*outs):
        assert np.array_equal(a, b)


def launches_of(P, h):
    return {r["name"]: r["launches"] for r in P.prsgd_profile_read(h)}


@pytest.mark.parametrize("steps_before", [0, 2])
def test_first_layer_fused_until_too_few_workers_go_on(P, D, steps_before):
    """24, 21, 8, 3 workers and the first layer fused for 20 and more: the second step multiplies activations that are there, and
    writes the shadows of its 21 workers alone, which the third step reads of eight of them.  Same bits as with every product apart."""
    steps = [4 if i % 8 == 3 else 3 if i % 8 in (1, 6) and i < 20 else 1 if i % 8 == 5 else 2 for i in range(24)]
    assert [sum(s > k for s in steps) for k in range(4)] == [24, 21, 8, 3]
    w = small_mlp(dims=(1024, 256, 10), batch=32, n_workers=24, gemm_dtype="bf16", activation="relu", rows_per_worker=64)
    inp = inputs_for(w)
    outs = []
    for on in (True, False):
        h = D.open_workload(w, inp)
        P.prsgd_set_first_layer_fusion(h, on)
        P.prsgd_local_steps(h, steps_before)
        P.prsgd_profile_enable(h, True)
        P.prsgd_local_steps_hetero(h, steps)
        assert launches_of(P, h).get("gemm_bwd_first", 0) == (1 if on else 0)
        P.prsgd_local_steps_hetero(h, steps)              # from points that differ
        P.prsgd_average(h)
        P.prsgd_local_steps_hetero(h, steps)              # from the average
        assert launches_of(P, h).get("gemm_bwd_first", 0) == (2 if on else 0)      # since then
        P.prsgd_local_steps(h, 2)
        outs.append((D.read_all(h), P.prsgd_read_loss(h), P.prsgd_read_indices(h)))
        P.prsgd_destroy(h)
    for a, b in zip(*outs):
        assert np.array_equal(a, b)


def test_ragged_first_layer_of_the_workers_that_go_on(P, D):
    """14, 12, 5 workers and a ragged first layer, fused for eleven and more: in each epoch once, for twelve of fourteen."""
    steps = [3, 2, 1, 2, 3, 2, 2, 3, 1, 2, 3, 2, 3, 2]
    assert [sum(s > k for s in steps) for k in range(3)] == [14, 12, 5]
    w = small_mlp(dims=(577, 513, 10), batch=32, n_workers=14, gemm_dtype="bf16", activation="tanh", rows_per_worker=64, lr=0.02)
    inp = inputs_for(w)
    want = oracle.run_heterogeneous(**oracle_args(w, inp), lr=w.lr, worker_steps=steps, n_epochs=2)
    for on in (True, False):
        h = D.open_workload(w, inp)
        P.prsgd_set_first_layer_fusion(h, on)
        P.prsgd_profile_enable(h, True)
        D.run_algorithm3(h, steps, 2)
        assert launches_of(P, h).get("gemm_bwd_first", 0) == (2 if on else 0)
        assert rel_err(D.read_all(h), want["x"]) <= 5e-3
        assert np.allclose(P.prsgd_read_loss(h), want["losses"], rtol=2e-2, atol=1e-6)
        P.prsgd_destroy(h)


def test_an_epoch_is_not_captured(P, D):
    """Refused before anything is launched; what the graph holds beside it still replays."""
    w = small_mlp(dims=(100, 72, 40, 10), batch=24, n_workers=3, gemm_dtype="bf16", activation="tanh", rows_per_worker=64, lr=0.02)
    inp = inputs_for(w)
    stream = torch.cuda.Stream()
    a, b = D.open_workload(w, inp, stream=stream), D.open_workload(w, inp, stream=stream)
    with torch.cuda.stream(stream):
        P.prsgd_local_steps(a, 1)
        P.prsgd_local_steps(b, 1)
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            with pytest.raises(RuntimeError, match="worker step counts"):
                P.prsgd_local_steps_hetero(a, [1, 2, 0])
            P.prsgd_local_steps(a, 1)
        assert P.prsgd_iteration(a) == 2
        for _ in range(3):
            graph.replay()
            P.prsgd_set_iteration(b, 1)
            P.prsgd_local_steps(b, 1)
            assert np.array_equal(D.read_all(a), D.read_all(b))
        P.prsgd_local_steps_hetero(a, [1, 2, 0])
        P.prsgd_set_iteration(b, 2)
        P.prsgd_local_steps_hetero(b, [1, 2, 0])
        assert np.array_equal(D.read_all(a), D.read_all(b))
    P.prsgd_destroy(a)
    P.prsgd_destroy(b)


# numbers of one byte, of two and of four, as many as travel with a launch and one more; step counts further apart than a byte
@pytest.mark.parametrize("n,last", [(256, 5), (257, 300), (1920, 255), (1921, 256)])
def test_many_workers_of_unlike_speed(P, D, n, last):
    steps = [(7 * i) % 5 for i in range(n - 1)] + [last]
    w = small_mlp(dims=(12, 9, 8, 5), batch=4, n_workers=n, gemm_dtype="f32", activation="tanh", rows_per_worker=8, lr=0.02)
    inp = inputs_for(w)
    h = D.open_workload(w, inp)
    D.run_algorithm3(h, steps, 1)
    want = oracle.run_heterogeneous(**oracle_args(w, inp), lr=w.lr, worker_steps=steps, n_epochs=1)
    assert rel_err(D.read_all(h), want["x"]) <= 1e-4
    rows = P.prsgd_read_indices(h)
    for i in range(n):
        if steps[i] > 0:
            assert np.array_equal(rows[i], oracle.sample_rows(w.index_seed, i, steps[i], 4, 8)), i
    P.prsgd_destroy(h)


@pytest.mark.parametrize("n,last", [(3840, 255), (3841, 3), (1921, 256), (961, 65536)])
def test_many_least_squares_workers_of_unlike_speed(P, D, n, last):
    """Where a launch takes the step counts themselves."""
    steps = [(7 * i) % 5 for i in range(n - 1)] + [last]
    w = small_mlp(model="lsq", dims=(8,), activation="none", batch=4, n_workers=n, n_classes=0, rows_per_worker=8, lr=0.02)
    inp = inputs_for(w)
    h = D.open_workload(w, inp)
    P.prsgd_local_steps_hetero(h, steps)
    got = D.read_all(h)
    few = steps[:-1] + [min(last, 300)]
    want = oracle.run_heterogeneous(**oracle_args(w, inp), lr=w.lr, worker_steps=few, n_epochs=1)["x"]
    assert rel_err(got[:-1], want[:-1]) <= 1e-4
    if last <= 300:
        assert rel_err(got[-1], want[-1]) <= 1e-4
    else:
        assert P.prsgd_iteration(h) == last
        assert np.array_equal(P.prsgd_read_indices(h)[-1], oracle.sample_rows(w.index_seed, n - 1, last, 4, 8))
    P.prsgd_destroy(h)
