"""Host-side checks that need no GPU: the library loads, exports every symbol the header
declares, sizes its buffers as documented and rejects bad configurations."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def P():
    lib = os.path.join(ROOT, "paper_1807_06629_amd", "libprsgd.so")
    if not os.path.exists(lib):
        from paper_1807_06629_amd.build import build
        build()
    from paper_1807_06629_amd import prsgd
    return prsgd


def _declared_functions():
    names = set()
    inc = os.path.join(ROOT, "include")
    for header in sorted(os.listdir(inc)):
        if not header.endswith(".h"):
            continue
        text = open(os.path.join(inc, header)).read()
        text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
        names |= set(re.findall(r"\b(prsgd_[a-z0-9_]+)\s*\(", text))
    return sorted(names)


def test_library_exports_every_declared_symbol(P):
    names = _declared_functions()
    assert {"prsgd_init", "prsgd_local_steps", "prsgd_average", "prsgd_read_params"} <= set(names)
    lib = ctypes.CDLL(P.LIB_PATH)
    for name in names:
        assert hasattr(lib, name), name
    # and the binding mirrors each of them under the same name
    for name in names:
        assert hasattr(P, name), name


def test_parameter_counts_match_the_closed_form(P):
    c2 = P.make_config(8, "mlp", (784, 256, 10), 32, 8192, 0.05, 3, "tanh")
    assert P.prsgd_param_count(c2) == 784 * 256 + 256 + 256 * 10 + 10 == 203530
    c5 = P.make_config(8, "mlp", (4096, 4096, 4096, 4096, 1000), 128, 8192, 0.01, 3, "relu", "bf16")
    assert P.prsgd_param_count(c5) == 54440936
    c1 = P.make_config(4, "lsq", (64,), 16, 4096, 0.01, 3)
    assert P.prsgd_param_count(c1) == 64
    for c in (c1, c2, c5):
        stride = P.prsgd_param_stride(c)
        assert stride >= P.prsgd_param_count(c) and stride % 64 == 0
        assert P.prsgd_workspace_bytes(c) % 256 == 0 and P.prsgd_workspace_bytes(c) > 0


def test_workspace_grows_with_shadow_and_gradient_buffers(P):
    # two hidden layers: no epoch-kernel buffers, so the only differences are the ones named
    dims = (64, 32, 24, 10)
    f32 = P.make_config(2, "mlp", dims, 8, 64, 0.1, 1, "relu", "f32", True)
    bf = P.make_config(2, "mlp", dims, 8, 64, 0.1, 1, "relu", "bf16", True)
    unf = P.make_config(2, "mlp", dims, 8, 64, 0.1, 1, "relu", "f32", False)
    stride = P.prsgd_param_stride(f32)
    assert P.prsgd_workspace_bytes(unf) - P.prsgd_workspace_bytes(f32) >= 2 * stride * 4
    assert P.prsgd_workspace_bytes(bf) > 0


@pytest.mark.parametrize("kw", [
    dict(n_workers=0), dict(batch=0), dict(batch=5000), dict(rows_per_worker=100),
    dict(rows_per_worker=0), dict(dims=(5,)), dict(dims=(0, 4)), dict(lr=float("nan")),
    dict(momentum=1.0), dict(momentum=-0.1),
])
def test_invalid_configurations_are_rejected_without_touching_the_gpu(P, kw):
    base = dict(n_workers=2, model="mlp", dims=(8, 4), batch=4, rows_per_worker=16, lr=0.1, seed=1)
    base.update(kw)
    cfg = P.make_config(**base)
    assert P.prsgd_param_count(cfg) == 0
    assert P.prsgd_workspace_bytes(cfg) == 0
    ctx = ctypes.c_void_p()
    rc = P._lib.prsgd_init(ctypes.byref(cfg), None, None, None, None, None, None, ctypes.byref(ctx))
    assert rc == P.PRSGD_EINVAL and not ctx
    assert P.prsgd_last_error(None) != ""


@pytest.mark.parametrize("dims,n_workers,steps,step_mean", [
    ((3072, 1024, 1024, 10), 11, False, False),              # 177 MiB of replicas
    ((3072, 1024, 1024, 10), 16, True, False),               # 257 MiB, the average 16
    ((4096, 4096, 4096, 10), 8, True, False),                # 1026 MiB, the average 128
    ((4096, 4096, 4096, 4096, 1000), 1, True, True),         # 208 MiB
    ((4096, 4096, 4096, 4096, 1000), 8, True, True),
])
def test_streamed_launches_go_by_what_they_rewrite(P, dims, n_workers, steps, step_mean):
    # past the last-level cache: the replica set for local steps, the average for a step on the average
    uses = P.prsgd_streamed_uses(P.make_config(n_workers, "mlp", dims, 64, 1024, 0.1, 1, "relu", "bf16"))
    assert bool(uses & P.PRSGD_STREAM_STEPS) == steps
    assert bool(uses & P.PRSGD_STREAM_STEP_MEAN) == step_mean


@pytest.mark.parametrize("dims,n_workers,rows,streamed", [
    ((3072, 1024, 1024, 10), 16, 1024, False),               # replicas past the last-level cache, shards of 192 MiB
    ((3072, 1024, 1024, 10), 16, 2048, True),                # ... of 384
    ((4096, 4096, 4096, 10), 8, 2048, True),                 # ... of exactly 256
    ((3072, 1024, 1024, 10), 11, 4096, False),               # shards of 528 MiB, but replicas that the cache holds
    ((256, 128, 10), 64, 8192, False),
])
def test_drawn_rows_are_streamed_beside_streamed_steps(P, dims, n_workers, rows, streamed):
    uses = P.prsgd_streamed_uses(P.make_config(n_workers, "mlp", dims, 64, rows, 0.1, 1, "relu", "bf16"))
    assert bool(uses & P.PRSGD_STREAM_ROWS) == streamed


@pytest.mark.parametrize("dims,n_workers,mean,average", [
    ((3072, 1024, 1024, 10), 11, False, False),              # 177 MiB
    ((3072, 1024, 1024, 10), 16, True, False),               # 257 MiB
    ((4096, 4096, 4096, 10), 2, False, False),               # 257 MiB in two replicas
    ((2048, 2048, 2048, 10), 12, True, True),                # 386 MiB
    ((4096, 4096, 4096, 4096, 1000), 4, False, True),        # 832 MiB in four
    ((4096, 4096, 4096, 4096, 1000), 5, True, True),
])
def test_streamed_averages_go_by_what_is_read_again(P, dims, n_workers, mean, average):
    uses = P.prsgd_streamed_uses(P.make_config(n_workers, "mlp", dims, 64, 1024, 0.1, 1, "relu", "bf16"))
    assert bool(uses & P.PRSGD_STREAM_MEAN) == mean
    assert bool(uses & P.PRSGD_STREAM_AVERAGE) == average


@pytest.mark.parametrize("streams,regime", [
    ([(64, 16)], "ALONE"),                                   # whatever its own plan took
    ([(8, 16), (8, 16)], "TOGETHER"),                        # 16 + 16 of 32 places on every XCD
    ([(8, 16), (8, 16), (1, 1)], "CROWDED"),
    ([(2, 16)] * 5, "TOGETHER"),                             # spread: 4 each, where pinned teams would need 80 on XCD 0
    ([(1, 32), (1, 32)], "TOGETHER"),                        # 4 + 4, where pinned each would take all of XCD 0
    ([(1, 32)] * 8, "TOGETHER"),
    ([(1, 32)] * 9, "CROWDED"),
    ([(9, 16), (7, 16)], "TOGETHER"),                        # 18 + 14
    ([(9, 16), (7, 16), (1, 1)], "CROWDED"),
    ([(64, 1)] * 4, "TOGETHER"),                             # least squares: 8 each
    ([(64, 1)] * 5, "CROWDED"),
])
def test_launches_that_wait_are_counted_by_xcd(P, streams, regime):
    got = P.prsgd_waiting_regime([n for n, _ in streams], [t for _, t in streams], 256)
    assert got == getattr(P, "PRSGD_WAIT_" + regime)


@pytest.mark.parametrize("n_workers,dims,batch,momentum,scratch", [
    (8, (784, 256, 10), 32, 0.0, "RUNS"),
    # what the replicas' restarts pass through memory is as large as the replicas
    (64, (512, 128, 10), 8, 0.0, "EPOCHS"), (16, (784, 256, 10), 32, 0.0, "EPOCHS"), (100, (256, 128, 10), 8, 0.0, "EPOCHS"),
    (20, (784, 192, 10), 16, 0.0, "EPOCHS"), (12, (784, 512, 10), 16, 0.0, "EPOCHS"),
    # partial logits without padding, in one set
    (16, (100, 256, 64), 64, 0.0, "EPOCHS"),
    (196, (292, 32, 57), 16, 0.0, "LAYERS"),
])
def test_static_contexts_leave_out_scratch_before_they_are_refused(P, n_workers, dims, batch, momentum, scratch):
    cfg = P.make_config(n_workers, "mlp", dims, batch, 256, 0.1, 1, "relu", momentum=momentum)
    assert P.prsgd_static_scratch(cfg) == getattr(P, "PRSGD_SCRATCH_" + scratch)


def test_static_contexts_beyond_the_limit_are_refused(P):
    cfg = P.make_config(16, "mlp", (3072, 1024, 1024, 10), 64, 256, 0.1, 1, "relu", "bf16")
    with pytest.raises(P.PrsgdError) as err:
        P.prsgd_static_scratch(cfg)
    assert err.value.code == P.PRSGD_EINVAL


def test_null_context_calls_return_einval(P):
    assert P._lib.prsgd_local_steps(None, 1) == P.PRSGD_EINVAL
    assert P._lib.prsgd_average(None) == P.PRSGD_EINVAL
    assert P._lib.prsgd_run(None, 1, 1) == P.PRSGD_EINVAL
    assert P._lib.prsgd_read_params(None, 0, None, 0) == P.PRSGD_EINVAL
    assert P._lib.prsgd_iteration(None) == -1
    assert P._lib.prsgd_destroy(None) == P.PRSGD_EINVAL
    assert P._lib.prsgd_waiting_regime(None, None, 1, 256) == P.PRSGD_EINVAL
    assert P._lib.prsgd_waiting_launches(None, None) == P.PRSGD_EINVAL


def test_theorem2_schedule_of_the_library(P):
    ks, gs = P.prsgd_time_varying_schedule(27, 2)
    assert ks[0] == 1 and ks[7] == 1 and ks[26] == 2
    assert gs[0] == 2.0 and gs[7] == pytest.approx(0.5)
    assert P._lib.prsgd_time_varying_schedule(3, 0, None, None) == P.PRSGD_EINVAL
    assert P._lib.prsgd_time_varying_schedule(3, 1, None, None) == P.PRSGD_EINVAL
    assert len(P.prsgd_time_varying_schedule(0, 4)[0]) == 0


@pytest.mark.parametrize("n_workers", [1, 2, 8])
def test_theorem2_schedule_matches_the_oracle_and_the_integer_definition(P, n_workers):
    # K^s = ceil(s^(1/3) / N): the smallest integer k with (k N)^3 >= s, checked in exact integer
    # arithmetic, against the oracle's floating-point form and against the library
    import numpy as np
    import oracle
    S = 10000
    ks, gs = P.prsgd_time_varying_schedule(S, n_workers)
    oks, ogs = oracle.time_varying_schedule(S, n_workers)
    for s in range(1, S + 1):
        k = int(ks[s - 1])
        assert (k * n_workers) ** 3 >= s and (k == 1 or ((k - 1) * n_workers) ** 3 < s), s
        assert oks[s - 1] == k, s
    assert np.allclose(gs, np.asarray(ogs), rtol=2e-7, atol=0)
    # perfect cubes are where a rounded cube root would be off by one
    for r in (2, 3, 5, 10, 21):
        s = (r * n_workers) ** 3
        if s <= S:
            assert ks[s - 1] == r and (s == S or ks[s] == r + 1)
