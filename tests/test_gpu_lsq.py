"""Least squares: the register-resident kernel at the edges of its tiles, and restarts inside a launch.

The gate against the oracle is the 1e-4 of every short multi-step run.  Restarts inside the launch add in the order
of the restart kernels, so a run in one launch has the bits of the same run with a launch per epoch.
"""
import numpy as np
import pytest
import torch

import oracle
from helpers import oracle_run, rel_err
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


def _problem(d, batch, n, interval, iterations=70, momentum=0.0):
    w = get_workload("c1").scaled(dims=(d,), batch=batch, rows_per_worker=128, n_workers=n, momentum=momentum,
                                  lr=(0.001 if momentum else 0.01) / max(1, d // 64), interval=interval,
                                  iterations=iterations)
    return w, make_inputs(w)


# widths around one, two, four and eight columns per lane; minibatches around one, two, four and eight rows per
# wavefront; worker counts around the quarters of the restart sum; 70 iterations cross the 64 drawn at a time
@pytest.mark.parametrize("momentum", [0.0, 0.9])
@pytest.mark.parametrize("d,batch,n,interval", [
    (1, 1, 2, 1), (63, 4, 3, 3), (64, 5, 7, 1), (65, 8, 8, 2), (100, 3, 4, 5), (128, 9, 9, 7), (129, 16, 13, 64),
    (256, 17, 5, 65), (257, 32, 6, 4), (300, 33, 17, 1), (511, 64, 4, 9), (512, 64, 64, 6), (512, 1, 2, 70), (4, 64, 33, 1),
    # more workers than compute units: the shorter rings, of one to eight iterations
    (3, 1, 257, 8), (64, 16, 300, 5), (100, 6, 257, 7), (130, 30, 260, 9), (512, 1, 257, 9), (511, 16, 258, 4), (512, 64, 257, 3),
])
def test_run_in_one_launch(P, D, d, batch, n, interval, momentum):
    w, inp = _problem(d, batch, n, interval, momentum=momentum)
    h = D.open_workload(w, inp)
    P.prsgd_run(h, w.iterations, interval)
    assert P.prsgd_waiting_launches(h)[0] == (1 if n <= 64 and interval < w.iterations else 0)
    got, loss = D.read_all(h), P.prsgd_read_loss(h)
    assert P.prsgd_iteration(h) == w.iterations
    assert np.array_equal(P.prsgd_read_indices(h)[n - 1],
                          oracle.sample_rows(w.index_seed, n - 1, w.iterations, batch, 128))
    P.prsgd_run(h, 3, interval)                                  # goes on from there
    later = D.read_all(h)
    P.prsgd_destroy(h)
    h = D.open_workload(w, inp)                                  # a launch per epoch, a launch per restart
    left = w.iterations
    while left > 0:
        k = min(left, interval - P.prsgd_iteration(h) % interval)
        P.prsgd_local_steps(h, k)
        left -= k
        if P.prsgd_iteration(h) % interval == 0:
            P.prsgd_average(h)
    assert np.array_equal(D.read_all(h), got) and np.array_equal(P.prsgd_read_loss(h), loss)
    for _ in range(3):
        P.prsgd_local_steps(h, 1)
        if P.prsgd_iteration(h) % interval == 0:
            P.prsgd_average(h)
    assert np.array_equal(D.read_all(h), later)
    P.prsgd_destroy(h)
    want = oracle_run(w, inp, momentum=momentum)
    assert rel_err(got, want["x"]) <= 1e-4


@pytest.mark.parametrize("d,batch,n", [(512, 1, 3), (100, 6, 4), (64, 33, 5), (512, 33, 4), (3, 1, 257), (512, 1, 257)])
def test_wavefronts_past_the_minibatch_meet_no_earlier_contents_of_lds(P, D, d, batch, n):
    """Workgroups on every compute unit leave NaN in the places of all rows; the run behind them reads its own rows only."""
    other, inp = _problem(d, batch, 256, 8, iterations=8)
    inp["features"] = np.full_like(inp["features"], np.nan)
    w, clean = _problem(d, batch, n, 8, iterations=24)
    h, dirty = D.open_workload(w, clean), D.open_workload(other, inp)
    for _ in range(3):
        P.prsgd_local_steps(dirty, 8)
        P.prsgd_local_steps(h, 8)
        P.prsgd_average(h)
    assert rel_err(D.read_all(h), oracle_run(w, clean)["x"]) <= 1e-4
    P.prsgd_destroy(dirty)
    P.prsgd_destroy(h)


def test_contexts_of_several_streams_together(P, D):
    """Five contexts of 64 workgroups on five streams could not all wait on the device at once: the runs are the
    same, whichever of them goes out in one launch."""
    w, inp = _problem(64, 16, 64, 2, iterations=40)
    h = D.open_workload(w, inp)
    P.prsgd_run(h, w.iterations, w.interval)
    want = D.read_all(h)
    P.prsgd_destroy(h)
    handles = [D.open_workload(w, inp, stream=torch.cuda.Stream()) for _ in range(5)]
    for _ in range(4):
        for h in handles:
            P.prsgd_run(h, w.iterations // 4, w.interval)
    for h in handles:
        assert np.array_equal(D.read_all(h), want)
        P.prsgd_destroy(h)


def test_give_up_is_reported_and_the_context_goes_on(P, D):
    """A wait limit of zero polls, set from the host: the first of 64 workgroups to look for the others' points
    gives up at once.  Every workgroup ends by itself."""
    w, inp = _problem(64, 16, 64, 2, iterations=12)
    h = D.open_workload(w, inp)
    P.prsgd_run(h, 4, 2)
    P.prsgd_status(h)
    good = P.prsgd_read_params(h, -1)
    P.prsgd_set_epoch_wait_limit(h, 0)
    P.prsgd_run(h, 7, 2)
    for call in (lambda: P.prsgd_read_params(h, -1), lambda: P.prsgd_run(h, 2, 2), lambda: P.prsgd_status(h)):
        with pytest.raises(P.PrsgdError) as err:
            call()
        assert err.value.code == P.PRSGD_ESTATE and "gave up" in str(err.value)
    P.prsgd_write_params(h, -1, good)
    P.prsgd_set_iteration(h, 4)
    P.prsgd_run(h, 8, 2)                                         # a launch per epoch from now on
    P.prsgd_status(h)
    want = oracle_run(w, inp)
    assert rel_err(D.read_all(h), want["x"]) <= 1e-4
    P.prsgd_destroy(h)
