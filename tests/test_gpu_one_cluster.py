"""Ensembles of one cluster: the same calls on one system, with the softening
that the cluster states (the scalar argument is then not used), through every
kernel that a call of one system may take: small blocks (up to 6400
particles), full sweeps one-sided and by pairs (from 6000 particles on,
potentials from 4500), block steps.

The two calls make the same sums, so they agree to the FP64 bar of 1e-13
(here: of the largest value), and block steps after a few steps to the same."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

EPS2 = 0.04          # far from the scalar's 0: another softening is another result


@pytest.fixture(scope="module")
def H():
    from paper_1104_2700_amd import hermite
    return hermite


@pytest.fixture(scope="module")
def ctx(H):
    c = H.Context(0)
    yield c
    c.close()


def _pair(H, n, seed=0):
    from paper_1104_2700_amd import inputs
    x, v, m = inputs.plummer(n, 40 + n + seed)
    s = H.State(x, v, m)
    s.xp.copy_(s.x)
    s.vp.copy_(s.v)
    return s, H.Clusters(np.array([0, n], dtype=np.int64), np.array([EPS2]))


def _close(got, ref):
    for a, b in zip(got, ref):
        assert float((a - b).abs().max()) <= 1e-13 * float(b.abs().max())


@pytest.mark.parametrize("n", [900, 4499, 4500, 5999, 6000, 6400, 6401, 20001])
def test_softening(H, ctx, n):
    from paper_1104_2700_amd import inputs
    s, cl = _pair(H, n)
    idx = torch.from_numpy(inputs.random_active(n, 77, 5)).cuda()
    for which in (None, idx):
        _close(ctx.force_jerk(s, which, 0.0, H.FP64, clusters=cl),
               [o.clone() for o in ctx.force_jerk(s, which, EPS2, H.FP64)])
        na = n if which is None else 77
        out = [torch.empty(k, dtype=torch.float64, device="cuda") for k in ((3, na), (3, na), (na,))]
        H.force_jerk_noalloc(s, which, 0.0, H.FP64, *out, clusters=cl)
        _close(out, ctx.force_jerk(s, which, EPS2, H.FP64))
    _close([ctx.energy(s, 0.0, clusters=cl).flatten()], [ctx.energy(s, EPS2).flatten()])
    params = H.dt_params(0.02, H.DT_PAPER, 3, 20)
    one = s.clone()
    ctx.initialize(s, EPS2, params, H.FP64)
    ctx.initialize(one, 0.0, params, H.FP64, clusters=cl)
    _close((one.a, one.j, one.pot), (s.a, s.j, s.pot))
    assert torch.equal(one.dt, s.dt)


@pytest.mark.parametrize("n,n_act", [(1200, 1200), (2500, 2000), (33000, 2000), (40000, 1300)])
@pytest.mark.parametrize("prec", [0, 1, 2, 3])
def test_plans(H, ctx, prec, n, n_act):
    """From 1e6 interactions on, where a default tuning's split is chosen by
    a model of the sweep's time: plans made on the host and on the device
    (a count in device memory), in every precision (mixed from 32768
    particles and 5e7 interactions on).  The same plans: the same bits."""
    from paper_1104_2700_amd import inputs
    s, cl = _pair(H, n, 1)
    idx = torch.from_numpy(inputs.random_active(n, n_act, 5)).cuda()
    count = torch.tensor([n_act], dtype=torch.int32, device="cuda")
    for dev in (None, count):
        ref = [o.clone() for o in ctx.force_jerk(s, idx, EPS2, prec, n_act_dev=dev)]
        got = ctx.force_jerk(s, idx, 0.0, prec, n_act_dev=dev, clusters=cl)
        for a, b in zip(got, ref):
            assert torch.equal(a, b)
            assert torch.isfinite(a).all()


@pytest.mark.parametrize("prec", [0, 1, 3])
@pytest.mark.parametrize("n", [1000, 2500, 17000, 33000])
def test_block_steps(H, ctx, prec, n):
    """A few steps, from a block of every particle on (the steps start equal)."""
    s, cl = _pair(H, n, 2)
    params = H.dt_params(0.02, H.DT_PAPER, 3, 20)
    ctx.initialize(s, EPS2, params, prec)
    s.dt.fill_(1 << 10)
    one = s.clone()
    for _ in range(3):
        ctx.step(s, EPS2, params, prec)
        ctx.step(one, 0.0, params, prec, clusters=cl)
    _close((one.x, one.v), (s.x, s.v))
    assert torch.equal(one.t, s.t)


@pytest.mark.parametrize("prec", [0, 1, 3])
@pytest.mark.parametrize("n", [1000, 2500, 17000, 33000])
def test_runs(H, ctx, prec, n):
    """A run selects its blocks from the step-size order, as one system's
    does, and integrates to the same state."""
    s, cl = _pair(H, n, 2)
    params = H.dt_params(0.02, H.DT_PAPER, 3, 20)
    ctx.initialize(s, EPS2, params, prec)
    for graph in (True, False):
        ref, one = s.clone(), s.clone()
        for _ in range(20):
            ctx.step(ref, EPS2, params, prec)
        steps, inter = ctx.run(one, 0.0, params, 1 << 20, prec, clusters=cl, use_graph=graph,
                               max_steps=20)
        assert steps == 20 and inter > 0
        _close((one.x, one.v), (ref.x, ref.v))
        assert torch.equal(one.t, ref.t)


def test_autotune_reports_its_plan(H, tmp_path):
    """The partial sums that the chosen shape writes and reads: a whole number
    of chunks of eight doubles a particle, twice."""
    n, n_act = 3000, 64
    s, cl = _pair(H, n, 3)
    c = H.Context(0)
    try:
        c.autotune(s, 0.0, H.FP64, n_act=n_act, cache_path=tmp_path / "t.json", clusters=cl)
    finally:
        c.close()
    text = (tmp_path / "t.json").read_text()
    chunks = float(text.split('"partial_bytes":')[1].split("}")[0]) / (2 * 64 * n_act)
    assert chunks == int(chunks) and 1 <= chunks <= 12   # tiles of 256 particles
