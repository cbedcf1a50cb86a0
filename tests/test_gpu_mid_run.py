"""Runs of one system of 1537 to 16384 particles in launches of many block
steps (hermite_run with graphs) against the same steps one by one (without
graphs): the state bit for bit, the counters and the histogram, and the same
ends and errors.  Edges of the slices (1024 particles), blocks of one
to all particles, the largest such system and the first beyond it."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

TB = 20
KEYS = ("x", "v", "a", "j", "pot", "t", "dt")


@pytest.fixture(scope="module")
def H():
    from paper_1104_2700_amd import hermite
    return hermite


@pytest.fixture()
def ctx(H):
    c = H.Context(0)
    yield c
    c.close()


def _start(H, ctx, n, prec, k_min=3, k_max=20, eta=0.02):
    from paper_1104_2700_amd import inputs
    x, v, m = inputs.plummer(n, 90 + n)
    params = H.dt_params(eta, 0, k_min, k_max)
    s = H.State(x, v, m, TB)
    eps2 = (4.0 / n) ** 2
    ctx.initialize(s, eps2, params, prec)
    return s, eps2, params


def _launches(H, ctx):
    out = (ctypes.c_int64 * 3)()
    f = H.lib.hermite_small_run_launches
    f.argtypes = [ctypes.c_void_p, ctypes.c_void_p]
    assert f(ctx.h, out) == H.OK
    return tuple(out)


def _both(ctx, s0, eps2, params, prec, T_end, steps, sync_every=16):
    out = []
    for graph in (False, True):
        s = s0.clone()
        c0, h0 = ctx.counters(), np.array(ctx.block_histogram())
        res = ctx.run(s, eps2, params, T_end, prec, use_graph=graph, sync_every=sync_every,
                      max_steps=steps, with_done=True)
        c1, h1 = ctx.counters(), np.array(ctx.block_histogram())
        torch.cuda.synchronize()
        out.append((s, res, [c1[k] - c0[k] for k in ("steps", "interactions", "clamped")],
                    c1["T"], c1["n_act"], (h1 - h0).tolist()))
    return out


def _same(a, b):
    assert a[1:] == b[1:]
    for key in KEYS:
        assert torch.equal(getattr(a[0], key), getattr(b[0], key)), key


@pytest.mark.parametrize("n,prec,steps", [(1537, 0, 60), (2048, 1, 60), (2049, 0, 60),
                                          (3000, 2, 60), (5001, 0, 60), (8192, 1, 40),
                                          (9973, 0, 150), (16383, 2, 100), (16384, 0, 200),
                                          (16385, 0, 10)])
def test_mid_runs_match_single_steps(H, ctx, n, prec, steps):
    s0, eps2, params = _start(H, ctx, n, prec)
    _same(*_both(ctx, s0, eps2, params, prec, 1 << TB, steps))
    assert _launches(H, ctx) == (int(n <= 16384), 0, 0)


@pytest.mark.parametrize("n", [1800, 6000, 12000])
def test_mid_run_of_whole_blocks_to_the_end(H, ctx, n):
    """Blocks of many and of all particles, to the end, in calls of a few steps."""
    s0, eps2, params = _start(H, ctx, n, H.FP64, 6, 10, 0.08)
    T_end = 1 << (TB - 5)
    a, b = _both(ctx, s0, eps2, params, H.FP64, T_end, 0, sync_every=5)
    _same(a, b)
    assert a[1][2] and torch.all(b[0].t == T_end)
    s, total = s0.clone(), 0
    while True:
        steps, _, done = ctx.run(s, eps2, params, T_end, H.FP64, max_steps=7, with_done=True)
        total += steps
        if done:
            break
    torch.cuda.synchronize()
    assert total == a[1][0]
    for key in KEYS:
        assert torch.equal(getattr(s, key), getattr(a[0], key)), key
    assert ctx.run(s, eps2, params, T_end, H.FP64) == (0, 0)
    assert _launches(H, ctx)[1:] == (0, 0)


def test_mid_run_stops_on_a_non_finite_state(H, ctx):
    from paper_1104_2700_amd import inputs
    n = 2500
    x, v, m = inputs.plummer(n, 7)
    x[:, 5] = x[:, 2009]
    s0 = H.State(x, v, m, TB)
    params = H.dt_params(0.02, H.DT_PAPER, 3, 20)
    ctx.initialize(s0, 0.0, params, H.FP64)
    for graph in (True, False):
        s = s0.clone()
        with pytest.raises(H.HermiteError) as err:
            ctx.run(s, 0.0, params, 1 << TB, H.FP64, use_graph=graph, sync_every=8)
        assert err.value.code == H.ENONFINITE


def test_a_mid_launch_given_up_is_taken_step_by_step(H, ctx):
    s0, eps2, params = _start(H, ctx, 4000, H.FP64)
    a, b = _both(ctx, s0, eps2, params, H.FP64, 1 << TB, 30)
    _same(a, b)
    f = H.lib.hermite_small_run_patience
    f.argtypes = [ctypes.c_void_p, ctypes.c_int64]
    assert f(ctx.h, -1) == H.OK
    _, c = _both(ctx, s0, eps2, params, H.FP64, 1 << TB, 30)
    assert _launches(H, ctx) == (2, 1, 0)
    _same(a, c)
    assert f(ctx.h, 200000000) == H.OK
    _, d = _both(ctx, s0, eps2, params, H.FP64, 1 << TB, 30)
    _same(a, d)
