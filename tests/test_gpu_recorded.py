"""Steps and restarts recorded in a graph: every replay takes the iterations of the recording from the points as they are, whatever
the recording found drawn, computed ahead or averaged when it was made, and whatever ran between the replays.

Against a context that is never recorded: same bits where its steps have the same form (the first layer apart, or with the bits of
that), otherwise the bound of two forms of a ragged first layer (tests/test_gpu_first_layer_ragged.py).  Rows are whole numbers and
have to agree; a loss on other rows than its own differs in the first digits.
"""
import numpy as np
import pytest
import torch

from helpers import inputs_for, rel_err, small_mlp

pytestmark = pytest.mark.gpu

NETS = {
    "whole": dict(dims=(256, 128, 10), batch=32, n_workers=3, gemm_dtype="bf16"),
    "whole_momentum": dict(dims=(256, 128, 64, 10), batch=64, n_workers=3, gemm_dtype="bf16", momentum=0.9),
    "odd_tiles": dict(dims=(640, 320, 10), batch=32, n_workers=20, gemm_dtype="bf16"),
    "ragged": dict(dims=(577, 513, 10), batch=31, n_workers=12, gemm_dtype="bf16"),
    "not_fused": dict(dims=(72, 136, 40, 10), batch=160, n_workers=2, gemm_dtype="bf16"),
    "f32_layers": dict(dims=(60, 50, 40, 10), batch=20, n_workers=3),
    "f32_epochs": dict(dims=(256, 128, 10), batch=8, n_workers=5),
}
SAME_BITS = {"whole", "whole_momentum", "not_fused", "f32_layers", "f32_epochs"}


@pytest.fixture(scope="module")
def P():
    assert torch.cuda.is_available(), "these tests need the GPU"
    from paper_1807_06629_amd import prsgd
    return prsgd


@pytest.fixture(scope="module")
def D():
    from paper_1807_06629_amd import drivers
    return drivers


def open_pair(D, net, stream):
    w = small_mlp(activation="tanh", rows_per_worker=64, lr=0.02, interval=50, **NETS[net])
    inp = inputs_for(w)
    return D.open_workload(w, inp, stream=stream), D.open_workload(w, inp, stream=stream)


def agree(P, D, net, a, b, what):
    x, y = D.read_all(a), D.read_all(b)
    assert np.array_equal(x, y) if net in SAME_BITS else rel_err(x, y) <= 1e-3, what
    assert np.array_equal(P.prsgd_read_indices(a), P.prsgd_read_indices(b)), what
    assert np.allclose(P.prsgd_read_loss(a), P.prsgd_read_loss(b), rtol=0.0 if net in SAME_BITS else 5e-3, atol=0.0), what


# one step (nothing ahead), two and three (the last minibatch in the buffer that held the first, or in the other one), behind an even and an
# odd number of steps
@pytest.mark.parametrize("net", list(NETS))
@pytest.mark.parametrize("before,k", [(2, 1), (1, 2), (2, 3)])
def test_replayed_steps(P, D, net, before, k):
    stream = torch.cuda.Stream()
    a, b = open_pair(D, net, stream)
    with torch.cuda.stream(stream):
        P.prsgd_local_steps(a, before)
        P.prsgd_local_steps(b, before)
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            P.prsgd_local_steps(a, k)
        for i in range(4):
            graph.replay()
            stream.synchronize()
            P.prsgd_set_iteration(b, before)
            P.prsgd_local_steps(b, k)
            agree(P, D, net, a, b, f"replay {i}")
            if i < 1:
                continue
            t = P.prsgd_iteration(a)                      # eager steps: of other rows, one or two of them
            P.prsgd_local_steps(a, i)
            P.prsgd_set_iteration(b, t)
            P.prsgd_local_steps(b, i)
            agree(P, D, net, a, b, f"eager steps behind replay {i}")
    P.prsgd_destroy(a)
    P.prsgd_destroy(b)


@pytest.mark.parametrize("net", list(NETS))
@pytest.mark.parametrize("how", ["run", "calls"])
def test_replayed_restarts(P, D, net, how):
    """Recorded from workers at points of their own: a restart at the end of the recording, and one between two replays."""
    stream = torch.cuda.Stream()
    a, b = open_pair(D, net, stream)

    def epoch(h):
        if how == "run":
            P.prsgd_run(h, 3, 4)                          # iterations 2, 3, 4 and the restart
        else:
            P.prsgd_local_steps(h, 1)
            P.prsgd_local_steps(h, 2)
            P.prsgd_average(h)

    with torch.cuda.stream(stream):
        P.prsgd_local_steps(a, 1)
        P.prsgd_local_steps(b, 1)
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            epoch(a)
        for i in range(4):
            graph.replay()
            stream.synchronize()
            P.prsgd_set_iteration(b, 1)
            epoch(b)
            agree(P, D, net, a, b, f"replay {i}")
            if i == 1:
                for h in (a, b):
                    P.prsgd_set_iteration(h, 20)
                    P.prsgd_local_steps(h, 2)
                    P.prsgd_average(h)
                agree(P, D, net, a, b, "eager epoch")
    P.prsgd_destroy(a)
    P.prsgd_destroy(b)


@pytest.mark.parametrize("net", ["ragged", "whole", "f32_layers"])
def test_replayed_restart_between_eager_steps(P, D, net):
    """A graph that holds a restart only moves the points under whatever eager steps left ahead."""
    stream = torch.cuda.Stream()
    a, b = open_pair(D, net, stream)
    with torch.cuda.stream(stream):
        for h in (a, b):
            P.prsgd_set_lazy_restart(h, False)
            P.prsgd_local_steps(h, 1)
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            P.prsgd_average(a)
        for i in range(3):
            graph.replay()
            stream.synchronize()
            P.prsgd_average(b)
            for h in (a, b):
                P.prsgd_local_steps(h, 2)
            agree(P, D, net, a, b, f"steps behind restart {i}")
    P.prsgd_destroy(a)
    P.prsgd_destroy(b)
