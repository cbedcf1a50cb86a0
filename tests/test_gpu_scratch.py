"""Calls under capture, which cannot allocate: after one call on a system of a
size, another call on it is captured whatever its kind, and what was captured
stays valid when later calls make the sweep by pairs' scratch grow."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def H():
    from paper_1104_2700_amd import hermite
    return hermite


@pytest.fixture()
def ctx(H):
    c = H.Context(0)
    yield c
    c.close()


def _state(H, n):
    from paper_1104_2700_amd import inputs
    x, v, m = inputs.plummer(n, 11 + n)
    s = H.State(x, v, m)
    s.xp.copy_(s.x)
    s.vp.copy_(s.v)
    return s, (4.0 / n) ** 2


def _outputs(na):
    return [torch.full(k, 7.0, dtype=torch.float64, device="cuda") for k in ((3, na), (3, na), (na,))]


def _capture(ctx, s, idx, eps2, prec, out):
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        ctx.force_jerk(s, idx, eps2, prec, acc=out[0], jerk=out[1], pot=out[2])
    return g


def _replays(g, out, ref, other):
    """Several replays with eager work between them, each against ref."""
    for _ in range(3):
        for o in out:
            o.fill_(7.0)
        g.replay()
        torch.cuda.synchronize()
        for a, b in zip(out, ref):
            assert float((a - b).abs().max()) <= 2e-13 * float(b.abs().max())
        other()
        torch.cuda.synchronize()


@pytest.mark.parametrize("prec", [0, 3])
@pytest.mark.parametrize("warm", ["force", "energy", "initialize"])
@pytest.mark.parametrize("block", [True, False])
def test_a_call_is_captured_after_another_kind(H, ctx, warm, block, prec):
    n = 9000
    s, eps2 = _state(H, n)
    warm_up = {"force": lambda: ctx.force_jerk(s, None, eps2, H.FP64),
               "energy": lambda: ctx.energy(s, eps2),
               "initialize": lambda: ctx.initialize(
                   s, eps2, H.dt_params(0.02, H.DT_PAPER, 3, 20), H.FP64)}[warm]
    warm_up()
    idx = torch.arange(0, n, 2, dtype=torch.int32, device="cuda") if block else None
    out = _outputs(n // 2 if block else n)
    g = _capture(ctx, s, idx, eps2, prec, out)
    other = H.Context(0)
    try:
        ref = other.force_jerk(s, idx, eps2, prec)
        _replays(g, out, ref, warm_up)
    finally:
        other.close()


def test_a_captured_sweep_by_pairs_outlives_the_scratchs_growth(H, ctx):
    """The scratch of both kinds, made by a call with a list and by one
    without; then larger ones."""
    n = 8000
    s, eps2 = _state(H, n)
    ident = torch.arange(n, dtype=torch.int32, device="cuda")
    ctx.force_jerk(s, ident, eps2, H.FP64)
    ref = [o.clone() for o in ctx.force_jerk(s, None, eps2, H.FP64)]
    out = _outputs(n)
    g = _capture(ctx, s, None, eps2, H.FP64, out)
    held = []

    def grow(k=[12000, 17000, 24000]):
        if not k:
            return
        big, e2 = _state(H, k.pop(0))
        ctx.force_jerk(big, torch.arange(big.n, dtype=torch.int32, device="cuda"), e2, H.FP64)
        ctx.force_jerk(big, None, e2, H.FP64)
        held.append(torch.full((1 << 22,), float("nan"), device="cuda"))   # whoever gets freed memory

    _replays(g, out, ref, grow)
    for a, b in zip(out, ref):
        assert torch.equal(a, b)


def test_bits_do_not_depend_on_a_sweep_by_pairs_before(H):
    """A block's plan follows the scratch that calls of its kind asked for."""
    n, na = 9000, 4500
    s, eps2 = _state(H, n)
    idx = torch.arange(0, n, 2, dtype=torch.int32, device="cuda")
    res = []
    for first in (lambda c: c.force_jerk(s, None, eps2, H.FP64), lambda c: c.energy(s, eps2),
                  lambda c: c.force_jerk(s, torch.arange(n, dtype=torch.int32, device="cuda"),
                                         eps2, H.FP64)):
        c = H.Context(0)
        try:
            first(c)
            res.append([o.clone() for o in c.force_jerk(s, idx, eps2, H.FP64)])
        finally:
            c.close()
    for r in res[1:]:
        for a, b in zip(r, res[0]):
            assert torch.equal(a, b)
