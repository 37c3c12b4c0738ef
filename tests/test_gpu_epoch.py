"""One-hidden-layer fp32 nets in one launch: ragged widths, the forms of the exchange, restarts inside the launch.

The gates against the oracle are those of every fp32 net: 1e-5 after one step, 1e-4 after a short run.  Restarts inside the
launch add in the order of the restart kernels, so that a run in one launch has the bits of the same run
with a launch per epoch, which per-kernel timing asks for.
"""
import numpy as np
import pytest
import torch

import oracle
from helpers import inputs_for, oracle_args, oracle_run, rel_err, small_mlp
from workloads import get_workload, make_inputs

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


SHAPES = [
    dict(dims=(1, 1, 1), batch=1, n_workers=1),
    dict(dims=(5, 15, 3), batch=16, n_workers=2),                 # rows that are not 16-byte aligned
    dict(dims=(31, 17, 16), batch=17, n_workers=3),               # last hidden tile of one unit
    dict(dims=(32, 16, 17), batch=15, n_workers=9),               # one pair of row blocks; two class tiles
    dict(dims=(33, 33, 64), batch=33, n_workers=7),               # a block of one row; two hops (3 x 2112 floats)
    dict(dims=(255, 100, 10), batch=48, n_workers=4),             # three batch tiles
    dict(dims=(260, 40, 10), batch=49, n_workers=8),              # four; 9 pairs
    dict(dims=(500, 150, 12), batch=50, n_workers=3),             # partial pre-activations of two wavefronts in one place
    dict(dims=(512, 256, 10), batch=13, n_workers=8),             # two hops just reached (16 x 130 floats)
    dict(dims=(513, 255, 5), batch=32, n_workers=2),              # 33 row blocks
    dict(dims=(1023, 48, 10), batch=20, n_workers=2),             # 64 row blocks, single words
    dict(dims=(1024, 64, 10), batch=30, n_workers=20),            # quarters of the restart sum by groups of threads
    dict(dims=(96, 64, 10), batch=8, n_workers=33),
    # teams that fit the device but not with each on one XCD (4 or 5 teams of 7 to 12 on the first ones)
    dict(dims=(784, 192, 10), batch=32, n_workers=20),
    dict(dims=(784, 224, 10), batch=32, n_workers=33),
    dict(dims=(784, 160, 10), batch=32, n_workers=51),
    # teams of 44, 64, 125 and 256: the first hop in 8, 8, 16 and 32 groups of lanes
    dict(dims=(64, 700, 10), batch=8, n_workers=3),
    dict(dims=(784, 1024, 10), batch=32, n_workers=4),
    dict(dims=(100, 1999, 10), batch=16, n_workers=2),
    dict(dims=(256, 4096, 10), batch=16, n_workers=1),
    dict(dims=(33, 600, 3), batch=1, n_workers=5),                # 38 members, one hop
    # class rows of 64 with their chunks exchanged; sums of the second hop in batches (1300, 3072 and 4096 floats)
    dict(dims=(100, 48, 26), batch=50, n_workers=3),
    dict(dims=(256, 128, 48), batch=64, n_workers=2),
    dict(dims=(128, 50, 64), batch=64, n_workers=2),
]


@pytest.mark.parametrize("interval", [1, 4])
@pytest.mark.parametrize("shape", SHAPES)
def test_run_in_one_launch(P, D, shape, interval):
    activation = "relu" if interval == 1 else "tanh"
    w = small_mlp(activation=activation, rows_per_worker=128, interval=interval, iterations=11, lr=0.02, **shape)
    inp = inputs_for(w)
    h = D.open_workload(w, inp)
    P.prsgd_local_steps(h, 1)
    assert rel_err(D.read_all(h), oracle_run(w, inp, iterations=1, interval=100)["x"]) <= 1e-5
    P.prsgd_write_params(h, -1, inp["x0"])
    P.prsgd_set_iteration(h, 0)
    P.prsgd_run(h, w.iterations, interval)
    assert P.prsgd_waiting_launches(h)[0] == 1                    # the restarts were inside
    got, loss = D.read_all(h), P.prsgd_read_loss(h)
    last = w.n_workers - 1
    assert np.array_equal(P.prsgd_read_indices(h)[last],
                          oracle.sample_rows(w.index_seed, last, w.iterations, w.batch, w.rows_per_worker))
    P.prsgd_destroy(h)
    h = D.open_workload(w, inp)
    P.prsgd_profile_enable(h, True)                               # a launch per epoch, a launch per restart
    P.prsgd_run(h, w.iterations, interval)
    names = {r["name"] for r in P.prsgd_profile_read(h)}
    assert names == {"mlp2_epoch", "restart_mean"}, names
    assert np.array_equal(D.read_all(h), got) and np.array_equal(P.prsgd_read_loss(h), loss)
    P.prsgd_destroy(h)
    want = oracle_run(w, inp)
    assert rel_err(got, want["x"]) <= 1e-4
    assert np.allclose(loss, want["losses"], rtol=1e-3, atol=1e-6)


@pytest.mark.parametrize("shape", [
    dict(dims=(64, 32, 10), batch=8, n_workers=3),
    dict(dims=(100, 48, 33), batch=20, n_workers=8),              # class rows with their chunks exchanged
    dict(dims=(784, 256, 10), batch=32, n_workers=8),             # two hops
    dict(dims=(900, 64, 64), batch=20, n_workers=9),              # 57 row blocks, four class tiles
    dict(dims=(128, 64, 64), batch=64, n_workers=2),              # four batch and class tiles
    dict(dims=(36, 640, 10), batch=16, n_workers=2),              # teams of 40
])
def test_velocities_kept_over_restarts_in_one_launch(P, D, shape):
    w = small_mlp(activation="tanh", rows_per_worker=128, interval=3, iterations=10, lr=0.005, **shape).scaled(momentum=0.9)
    inp = inputs_for(w)
    out = []
    for apart in (False, True):
        h = D.open_workload(w, inp)
        P.prsgd_profile_enable(h, apart)                          # a launch per epoch, a launch per restart
        P.prsgd_run(h, w.iterations, w.interval)
        assert P.prsgd_waiting_launches(h)[0] == (0 if apart else 1)
        out.append((D.read_all(h), np.stack([P.prsgd_read_velocity(h, i) for i in range(w.n_workers)]), P.prsgd_read_loss(h)))
        P.prsgd_destroy(h)
    for a, b in zip(*out):
        assert np.array_equal(a, b)
    want = oracle_run(w, inp, momentum=0.9)
    assert rel_err(out[0][0], want["x"]) <= 1e-4 and rel_err(out[0][1], want["v"]) <= 1e-4


@pytest.mark.parametrize("shape", [
    dict(dims=(50, 21, 5), batch=7, n_workers=4),
    dict(dims=(301, 100, 20), batch=33, n_workers=3),
    dict(dims=(785, 530, 10), batch=20, n_workers=2),             # teams of 34, two hops
])
def test_epochs_of_unlike_lengths_on_ragged_widths(P, D, shape):
    w = small_mlp(rows_per_worker=128, lr=0.02, **shape)
    inp = inputs_for(w)
    steps = [5, 0, 3, 1][:w.n_workers]
    h = D.open_workload(w, inp)
    P.prsgd_profile_enable(h, True)
    D.run_algorithm3(h, steps, 3)
    names = {r["name"] for r in P.prsgd_profile_read(h)}
    assert "mlp2_epoch" in names and "gemm_fwd" not in names, names
    args = oracle_args(w, inp)
    args.pop("bf16")
    want = oracle.run_heterogeneous(**args, lr=w.lr, worker_steps=steps, n_epochs=3)
    assert P.prsgd_iteration(h) == want["t"]
    assert rel_err(D.read_all(h), want["x"]) <= 1e-4
    P.prsgd_destroy(h)


@pytest.mark.parametrize("model", ["lsq", "mlp"])
def test_run_in_a_captured_stream(P, D, model):
    """A run recorded in a graph has a launch per epoch.  Every replay, with eager work and synchronisations between
    them, takes the iterations of the recording from the points as they are."""
    if model == "lsq":
        w = get_workload("c1").scaled(dims=(64,), batch=16, rows_per_worker=128, n_workers=5, interval=4, iterations=8)
    else:
        w = small_mlp(dims=(784, 200, 10), batch=32, n_workers=5, rows_per_worker=128, interval=4, iterations=8, lr=0.02)
    inp = make_inputs(w)
    stream = torch.cuda.Stream()
    a, b = D.open_workload(w, inp, stream=stream), D.open_workload(w, inp, stream=stream)
    with torch.cuda.stream(stream):
        P.prsgd_local_steps(a, 1)
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            P.prsgd_run(a, 8, 4)                                  # from one step into an epoch: ends on a bare step
        assert P.prsgd_waiting_launches(a)[0] == 0
        P.prsgd_local_steps(b, 1)
        for _ in range(4):
            graph.replay()
            P.prsgd_set_iteration(b, 1)
            P.prsgd_run(b, 8, 4)
            assert np.array_equal(D.read_all(a), D.read_all(b))
            assert np.array_equal(P.prsgd_read_loss(a), P.prsgd_read_loss(b))
        assert P.prsgd_waiting_launches(b)[0] == 4
    P.prsgd_destroy(a)
    P.prsgd_destroy(b)


def test_contexts_of_three_streams_together(P, D):
    """Three grids of 128 workgroups on three streams: not all of them may wait as a whole at once."""
    w = small_mlp(dims=(784, 256, 10), batch=32, n_workers=8, rows_per_worker=128, interval=2, iterations=12)
    inp = inputs_for(w)
    h = D.open_workload(w, inp)
    P.prsgd_run(h, w.iterations, w.interval)
    want = D.read_all(h)
    P.prsgd_destroy(h)
    handles = [D.open_workload(w, inp, stream=torch.cuda.Stream()) for _ in range(3)]
    for _ in range(2):
        for h in handles:
            P.prsgd_run(h, w.iterations // 2, w.interval)
    for h in handles:
        assert np.array_equal(D.read_all(h), want)
        P.prsgd_destroy(h)


def test_small_contexts_of_several_streams_run_together(P, D):
    """Five contexts of two teams of 16 fit the device together once their teams are spread over the XCDs; the first of them
    has run alone (teams on XCDs 0 and 1) before the others come."""
    w = small_mlp(dims=(784, 256, 10), batch=32, n_workers=2, rows_per_worker=128, interval=2, iterations=12)
    inp = inputs_for(w)
    assert P.prsgd_waiting_regime([2] * 5, [16] * 5) == P.PRSGD_WAIT_TOGETHER
    handles = [D.open_workload(w, inp, stream=torch.cuda.Stream())]
    P.prsgd_run(handles[0], w.iterations, w.interval)
    want = D.read_all(handles[0])
    P.prsgd_write_params(handles[0], -1, inp["x0"])
    P.prsgd_set_iteration(handles[0], 0)
    handles += [D.open_workload(w, inp, stream=torch.cuda.Stream()) for _ in range(4)]
    before = [P.prsgd_waiting_launches(h)[0] for h in handles]
    for _ in range(2):
        for h in handles:
            P.prsgd_run(h, w.iterations // 2, w.interval)
    for h, n in zip(handles, before):
        assert P.prsgd_waiting_launches(h) == (n + 2, 0)
        assert np.array_equal(D.read_all(h), want)
        P.prsgd_destroy(h)


def test_contexts_that_do_not_fit_follow_each_other(P, D):
    """Three grids of 16 workgroups per XCD: two fit, so the launches of a third stream follow one of theirs."""
    w = small_mlp(dims=(784, 256, 10), batch=32, n_workers=8, rows_per_worker=128, interval=3, iterations=9)
    inp = inputs_for(w)
    assert P.prsgd_waiting_regime([8] * 3, [16] * 3) == P.PRSGD_WAIT_CROWDED
    handles = [D.open_workload(w, inp, stream=torch.cuda.Stream()) for _ in range(3)]
    for _ in range(3):
        for h in handles:
            P.prsgd_local_steps(h, 3)
            P.prsgd_average(h)
    got = [D.read_all(h) for h in handles]
    counts = [P.prsgd_waiting_launches(h) for h in handles]
    assert all(c[0] == 0 for c in counts) and sum(c[1] for c in counts) >= 7, counts
    for h in handles[1:]:
        P.prsgd_destroy(h)
    P.prsgd_write_params(handles[0], -1, inp["x0"])
    P.prsgd_set_iteration(handles[0], 0)
    P.prsgd_run(handles[0], w.iterations, w.interval)             # alone again: in one launch
    assert P.prsgd_waiting_launches(handles[0])[0] == 1
    want = D.read_all(handles[0])
    P.prsgd_destroy(handles[0])
    for g in got:
        assert np.array_equal(g, want)


def test_a_context_that_comes_during_a_pinned_launch_follows_it(P, D):
    """Alone, two teams of 32 take XCDs 0 and 1 whole: what is launched on another stream meanwhile goes behind them."""
    w = small_mlp(dims=(784, 512, 10), batch=32, n_workers=2, rows_per_worker=128, interval=4, iterations=600, lr=0.002)
    inp = inputs_for(w)
    a = D.open_workload(w, inp, stream=torch.cuda.Stream())
    P.prsgd_run(a, w.iterations, w.interval)
    b = D.open_workload(w, inp, stream=torch.cuda.Stream())
    P.prsgd_run(b, w.iterations, w.interval)
    assert P.prsgd_waiting_launches(a) == (1, 0) and P.prsgd_waiting_launches(b) == (1, 1)
    assert np.array_equal(D.read_all(a), D.read_all(b))
    P.prsgd_destroy(a)
    P.prsgd_destroy(b)


def test_every_context_that_comes_during_a_pinned_launch_follows_it(P, D):
    """The second one to come is ordered behind the pinned launch like the first, though the three fit together spread."""
    w = small_mlp(dims=(784, 512, 10), batch=32, n_workers=2, rows_per_worker=128, interval=4, iterations=600, lr=0.002)
    inp = inputs_for(w)
    assert P.prsgd_waiting_regime([2] * 3, [32] * 3) == P.PRSGD_WAIT_TOGETHER
    handles = []
    for _ in range(3):
        handles.append(D.open_workload(w, inp, stream=torch.cuda.Stream()))
        P.prsgd_run(handles[-1], w.iterations, w.interval)
    assert [P.prsgd_waiting_launches(h) for h in handles] == [(1, 0), (1, 1), (1, 1)]
    out = [D.read_all(h) for h in handles]
    for h, x in zip(handles, out):
        assert np.array_equal(x, out[0])
        P.prsgd_destroy(h)
