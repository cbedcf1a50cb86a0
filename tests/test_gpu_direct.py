"""Force calls on small blocks of one small system, which one kernel does
(a workgroup a particle): against the sweep and its reduction (the active
count in device memory) bit for bit and against the CPU oracle, at the edges
of tiles, of the reduction's two forms (16 chunks) and of the kernel's range."""
import numpy as np
import pytest

from tests.gpu_util import check_fp64

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def H():
    from paper_1104_2700_amd import hermite
    return hermite


@pytest.mark.parametrize("n,n_act", [(1, 1), (2, 2), (63, 5), (256, 256), (257, 31), (1000, 999),
                                     (2049, 100), (4096, 7), (4097, 240), (6400, 1), (6400, 150),
                                     (6401, 150)])
def test_small_blocks(H, n, n_act):
    from oracle import oracle as O
    from paper_1104_2700_amd import inputs
    x, v, m = inputs.plummer(n, 60 + n)
    s = H.State(x, v, m)
    s.xp.copy_(s.x)
    s.vp.copy_(s.v)
    eps2 = (4.0 / max(n, 64)) ** 2
    idx = inputs.random_active(n, n_act, n_act)
    ti = torch.from_numpy(idx).cuda()
    count = torch.tensor([n_act], dtype=torch.int32, device="cuda")
    ctx = H.Context(0)
    try:
        for prec in (H.FP64, H.MIXED):
            c0 = ctx.counters()["interactions"]
            one = [o.clone() for o in ctx.force_jerk(s, ti, eps2, prec)]
            c1 = ctx.counters()["interactions"]
            two = ctx.force_jerk(s, ti, eps2, prec, n_act_dev=count)
            assert c1 - c0 == n * n_act
            for a, b in zip(one, two):
                assert torch.equal(a, b)
        if n_act == n:
            for a, b in zip(one, ctx.force_jerk(s, None, eps2, H.FP64)):
                assert torch.equal(a, b)
        ref = O.force(x, v, m, idx, eps2, with_cond=True)
        for name, a, b, cond in zip(("acc", "jerk", "pot"), one, ref[:3], ref[3]):
            check_fp64(name, a.cpu().numpy(), np.atleast_2d(b), cond, n)
        acc, jerk = torch.full_like(one[0], 7.0), torch.full_like(one[0], 7.0)
        H._check(H.lib.hermite_force_jerk(ctx.h, H.ctypes.byref(s.c()), None, ti.data_ptr(), None,
                                          n_act, eps2, H.FP64, acc.data_ptr(), jerk.data_ptr(), None,
                                          None),
                 "hermite_force_jerk")
        torch.cuda.synchronize()
        assert torch.equal(acc, one[0]) and torch.equal(jerk, one[1])   # no potential asked for
    finally:
        ctx.close()


def test_coincident_particles_without_softening(H):
    """An infinite pair stays in its own particles; the self pair, and what
    lies past a ragged tile's end, add nothing."""
    n = 300
    from paper_1104_2700_amd import inputs
    x, v, m = inputs.plummer(n, 3)
    x[:, 5] = x[:, 9]
    s = H.State(x, v, m)
    s.xp.copy_(s.x)
    s.vp.copy_(s.v)
    ctx = H.Context(0)
    try:
        acc, jerk, pot = (o.cpu().numpy() for o in ctx.force_jerk(s, None, 0.0, H.FP64))
    finally:
        ctx.close()
    rest = np.setdiff1d(np.arange(n), (5, 9))
    for a in (acc, jerk, pot[None]):
        assert np.isfinite(a[:, rest]).all()
    assert not np.isfinite(pot[[5, 9]]).any()
