"""Which runs go by launches of many block steps, by the context's own count
of them (launches, of these given up, of these ended before a block they
cannot take): so that the comparisons with single steps compare two things."""
import ctypes
import threading
import time

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


def _start(H, ctx, n):
    from paper_1104_2700_amd import inputs
    x, v, m = inputs.plummer(n, 70 + n)
    params = H.dt_params(0.02, H.DT_PAPER, 3, 20)
    s = H.State(x, v, m, TB)
    eps2 = (4.0 / max(n, 64)) ** 2
    ctx.initialize(s, eps2, params, H.FP64)
    return s, eps2, params


def _launches(H, ctx):
    out = (ctypes.c_int64 * 3)()
    f = H.lib.hermite_small_run_launches
    f.argtypes = [ctypes.c_void_p, ctypes.c_void_p]
    assert f(ctx.h, out) == H.OK
    return tuple(out)


def _run(H, ctx, s0, eps2, params, prec=0, graph=True, steps=40):
    s = s0.clone()
    ctx.run(s, eps2, params, 1 << TB, prec, use_graph=graph, max_steps=steps)
    torch.cuda.synchronize()
    return s


def _same(a, b):
    for key in KEYS:
        assert torch.equal(getattr(a, key), getattr(b, key)), key


@pytest.mark.parametrize("n,prec", [(1, 0), (300, 1), (1024, 0), (1536, 2)])
def test_small_runs_are_taken_in_one_launch(H, ctx, n, prec):
    args = _start(H, ctx, n)
    _run(H, ctx, *args, prec, graph=False)
    assert _launches(H, ctx) == (0, 0, 0)
    _run(H, ctx, *args, prec)
    assert _launches(H, ctx) == (1, 0, 0)


@pytest.mark.parametrize("n", [1024, 4000])
def test_a_launch_without_patience_is_given_up_and_counted(H, ctx, n):
    args = _start(H, ctx, n)
    f = H.lib.hermite_small_run_patience
    f.argtypes = [ctypes.c_void_p, ctypes.c_int64]
    assert f(ctx.h, -1) == H.OK
    a = _run(H, ctx, *args)
    assert _launches(H, ctx) == (1, 1, 0)
    _same(a, _run(H, ctx, *args, graph=False))


@pytest.mark.parametrize("n", [300, 1536, 4000, 16384])
def test_a_launch_given_up_by_some_ends_for_all(H, ctx, n):
    """Next to no time to start: a workgroup may give up while others, that
    saw all of them, go on to the next exchange, where they wait for seconds.
    They learn of it, and single steps give the run's result."""
    args = _start(H, ctx, n)
    ref = _run(H, ctx, *args, graph=False)
    f = H.lib.hermite_small_run_patience
    f.argtypes = [ctypes.c_void_p, ctypes.c_int64]
    begin = time.perf_counter()
    for ticks in (0, 30, 100, 300, 1000, 3000):
        assert f(ctx.h, ticks) == H.OK
        for _ in range(3):
            _same(_run(H, ctx, *args), ref)
    assert time.perf_counter() - begin < 1.5   # 18 runs of milliseconds; one long wait is 2 s
    assert _launches(H, ctx)[0] == 18 and _launches(H, ctx)[2] == 0


def test_systems_of_both_kinds_in_turn_on_one_context(H, ctx):
    """The launches of both kernels share the status and its numbering."""
    small, mid = _start(H, ctx, 700), _start(H, ctx, 5000)
    ref = [_run(H, ctx, *a, graph=False) for a in (small, mid)]
    for k in range(3):
        _same(_run(H, ctx, *mid), ref[1])
        _same(_run(H, ctx, *small), ref[0])
        assert _launches(H, ctx) == (2 * k + 2, 0, 0)


@pytest.mark.parametrize("n", [700, 5000])
@pytest.mark.parametrize("tuned_first", [False, True])
def test_only_the_default_tuning_goes_by_launches(H, ctx, n, tuned_first):
    """Also where the tuning changes between two runs of one context, in a
    field that the plan of a block does not depend on."""
    args = _start(H, ctx, n)
    default = ctx.get_tuning(H.FP64)
    tuned = H.CTuning(**dict(default.as_dict(), wg_per_cu=default.wg_per_cu + 1))
    count = 0
    for is_tuned in (tuned_first, not tuned_first, tuned_first):
        ctx.set_tuning(H.FP64, tuned if is_tuned else default)
        _run(H, ctx, *args)
        count += 0 if is_tuned else 1
        assert _launches(H, ctx) == (count, 0, 0)


def test_a_step_of_another_precision_does_not_decide(H, ctx):
    """A paper-faithful step of the same system has plans of its own."""
    s0, eps2, params = _start(H, ctx, 700)
    ctx.step(s0.clone(), eps2, params, H.MIXED_SP)
    _run(H, ctx, s0, eps2, params)
    assert _launches(H, ctx) == (1, 0, 0)


def test_runs_from_several_threads_use_the_chip(H):
    """Four small systems' launches fit the device side by side: every one of
    the runs is one launch and none is given up."""
    jobs = []
    for n in (900, 1500, 300, 700):
        c = H.Context(0)
        args = _start(H, c, n)
        jobs.append((c, args, _run(H, c, *args, graph=False)))
    errors = []

    def work(c, args, ref):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for _ in range(4):
                    s = args[0].clone()
                    c.run(s, args[1], args[2], 1 << TB, 0, max_steps=40)
                    torch.cuda.current_stream().synchronize()
                    _same(s, ref)
        except BaseException as e:   # noqa: BLE001 - reported by the test's own thread
            errors.append(e)

    threads = [threading.Thread(target=work, args=j) for j in jobs]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    counts = [_launches(H, j[0]) for j in jobs]
    for j in jobs:
        j[0].close()
    if errors:
        raise errors[0]
    assert counts == [(4, 0, 0)] * 4


@pytest.mark.parametrize("n,na", [(2048, 2048), (9000, 4500), (12000, 10753), (16384, 1025),
                                  (16384, 8193), (16384, 16384)])
def test_large_blocks_in_one_launch(H, ctx, n, na):
    """Blocks whose particles a row stages 64 or 512 at a time, with a
    remainder, against single steps."""
    s0, eps2, _ = _start(H, ctx, n)
    params = H.dt_params(1e-9, H.DT_PAPER, 6, 12)   # who is due stays at 2^-12
    g = torch.Generator().manual_seed(na)
    s0.dt.fill_(1 << 14)
    s0.dt[torch.randperm(n, generator=g)[:na].cuda()] = 1 << 8
    before = _launches(H, ctx)
    a = _run(H, ctx, s0, eps2, params, steps=12)
    assert _launches(H, ctx) == (before[0] + 1, 0, 0)
    assert ctx.counters()["n_act"] == na
    _same(a, _run(H, ctx, s0, eps2, params, graph=False, steps=12))


@pytest.mark.parametrize("n,na,launches", [(1536, 1536, 3), (1536, 652, 3), (1536, 651, 1),
                                           (1024, 1024, 3), (900, 900, 1)])
def test_small_systems_large_blocks_leave_the_chip(H, ctx, n, na, launches):
    """More than 1e6 interactions a block: a launch ends after eight of them,
    sync_every single steps follow, and another launch tries again; the state,
    the counts and the end are the single steps'."""
    s0, eps2, _ = _start(H, ctx, n)
    params = H.dt_params(1e-9, H.DT_PAPER, 6, 12)
    g = torch.Generator().manual_seed(na)
    s0.dt.fill_(1 << 14)
    s0.dt[torch.randperm(n, generator=g)[:na].cuda()] = 1 << 8
    out = []
    for graph in (True, False):
        s = s0.clone()
        c0 = ctx.counters()
        res = ctx.run(s, eps2, params, 1 << TB, H.FP64, use_graph=graph, sync_every=16,
                      max_steps=8 + 16 + 8 + 16 + 5, with_done=True)
        c1 = ctx.counters()
        out.append((s, res, [c1[k] - c0[k] for k in ("steps", "interactions", "clamped")], c1["T"]))
        if graph:
            assert _launches(H, ctx) == (launches, 0, 0)
    _same(out[0][0], out[1][0])
    assert out[0][1:] == out[1][1:] and out[0][1][0] == 53


def test_a_run_that_leaves_the_chip_reaches_its_end(H, ctx):
    n = 1536
    s0, eps2, _ = _start(H, ctx, n)
    params = H.dt_params(1e-9, H.DT_PAPER, 6, 12)
    s0.dt.fill_(1 << 8)
    for T_end in (1 << 14, 5 << 14):
        out = []
        for graph in (True, False):
            s = s0.clone()
            out.append((ctx.run(s, eps2, params, T_end, H.FP64, use_graph=graph, sync_every=5,
                                with_done=True), s))
        assert out[0][0] == out[1][0] and out[0][0][0] == T_end >> 8 and out[0][0][2]
        _same(out[0][1], out[1][1])
