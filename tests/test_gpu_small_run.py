"""Runs of one small system in launches of many block steps (hermite_run with
graphs, up to 1536 particles) against the same steps one by one (without
graphs, and hermite_step): the state bit for bit, the counters and the
histogram, and the same ends and errors.  Tile edges (256 particles a wave),
the largest such system and the first beyond it, one particle, blocks of one
and of all particles."""
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


def _start(H, ctx, n, prec, seed=0, form=0):
    from paper_1104_2700_amd import inputs
    x, v, m = inputs.plummer(n, 70 + n + seed)
    params = H.dt_params(0.02, form, 3, 20)
    s = H.State(x, v, m, TB)
    eps2 = (4.0 / max(n, 64)) ** 2
    ctx.initialize(s, eps2, params, prec)
    return s, eps2, params


def _both(ctx, s0, eps2, params, prec, T_end, steps, sync_every=16):
    """The same run both ways; returns the states, results and counts."""
    out = []
    for graph in (True, False):
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
    for key in KEYS:
        assert torch.equal(getattr(a[0], key), getattr(b[0], key)), key
    assert a[1:] == b[1:]


@pytest.mark.parametrize("n,prec", [(1, 0), (2, 0), (63, 1), (255, 0), (256, 2), (257, 0),
                                    (512, 1), (1024, 0), (1025, 0), (1280, 1), (1536, 0),
                                    (1537, 0)])
def test_small_runs_match_single_steps(H, ctx, n, prec):
    s0, eps2, params = _start(H, ctx, n, prec)
    _same(*_both(ctx, s0, eps2, params, prec, 1 << TB, 70))
    # and hermite_step's
    s = s0.clone()
    ref = s0.clone()
    ctx.run(s, eps2, params, 1 << TB, prec, max_steps=9)
    for _ in range(9):
        ctx.step(ref, eps2, params, prec, T_end=1 << TB)
    torch.cuda.synchronize()
    for key in KEYS:
        assert torch.equal(getattr(s, key), getattr(ref, key)), key


def test_small_run_to_the_end_in_several_calls(H, ctx):
    """Whole blocks (all particles due at once) among the steps, the end, and
    calls that go on where the last one stopped."""
    n = 600
    s0, eps2, _ = _start(H, ctx, n, H.FP64)
    params = H.dt_params(0.08, H.DT_AARSETH, 6, 12)
    ctx.initialize(s0, eps2, params, H.FP64)
    T_end = 1 << (TB - 5)
    a, b = _both(ctx, s0, eps2, params, H.FP64, T_end, 0, sync_every=32)
    _same(a, b)
    assert a[1][2] and torch.all(a[0].t == T_end) and a[5][10] > 0
    s, total = s0.clone(), 0
    while True:
        steps, _, done = ctx.run(s, eps2, params, T_end, H.FP64, max_steps=11, with_done=True)
        total += steps
        if done:
            break
    torch.cuda.synchronize()
    assert total == a[1][0]
    for key in KEYS:
        assert torch.equal(getattr(s, key), getattr(a[0], key)), key
    assert ctx.run(s, eps2, params, T_end, H.FP64) == (0, 0)


@pytest.mark.parametrize("case", ["t_off_grid", "dt_not_pow2", "overdue"])
def test_small_run_of_an_odd_state(H, ctx, case):
    """States the block scheme would not leave behind."""
    n = 700
    s0, eps2, params = _start(H, ctx, n, H.FP64)
    if case == "t_off_grid":
        s0.t[17] = 1
    elif case == "dt_not_pow2":
        s0.dt[17] = 3 << 6
    else:
        s0.dt.fill_(1 << (TB - 8))
        s0.t[18] = 4 << (TB - 8)
    _same(*_both(ctx, s0, eps2, params, H.FP64, 1 << TB, 40))


def test_small_run_stops_on_a_non_finite_state(H, ctx):
    from paper_1104_2700_amd import inputs
    n = 300
    x, v, m = inputs.plummer(n, 7)
    x[:, 5] = x[:, 9]
    s0 = H.State(x, v, m, TB)
    params = H.dt_params(0.02, H.DT_PAPER, 3, 20)
    ctx.initialize(s0, 0.0, params, H.FP64)
    got = []
    for graph in (True, False):
        s = s0.clone()
        with pytest.raises(H.HermiteError) as err:
            ctx.run(s, 0.0, params, 1 << TB, H.FP64, use_graph=graph, sync_every=8)
        assert err.value.code == H.ENONFINITE
        torch.cuda.synchronize()
        got.append(s)
    assert torch.equal(got[0].t, got[1].t)


@pytest.mark.parametrize("n", [40, 1024])
def test_a_launch_given_up_is_taken_step_by_step(H, ctx, n):
    """With no patience every launch is given up at its first exchange: the
    run falls back to single steps and gives their result."""
    s0, eps2, params = _start(H, ctx, n, H.FP64)
    a, b = _both(ctx, s0, eps2, params, H.FP64, 1 << TB, 30)
    _same(a, b)
    f = H.lib.hermite_small_run_patience
    f.argtypes = [ctypes.c_void_p, ctypes.c_int64]
    assert f(ctx.h, -1) == H.OK
    c, _ = _both(ctx, s0, eps2, params, H.FP64, 1 << TB, 30)
    _same(a, c)
    assert f(ctx.h, 200000000) == H.OK
    d, _ = _both(ctx, s0, eps2, params, H.FP64, 1 << TB, 30)
    _same(a, d)
