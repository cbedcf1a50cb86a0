"""How a sweep of one system is split over the chip: the plan made on the host
(the active count given to the call) against the one made on the device (the
count in device memory), and both against the CPU oracle, around the sizes
where the choice of the split changes."""
import numpy as np
import pytest

from tests.gpu_util import check_fp64

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def H():
    from paper_1104_2700_amd import hermite
    return hermite


# 1e6 interactions is where the split model takes over, 5e7 where the mixed
# precisions leave FP64; one active particle, a few, and all of them
SIZES = [(300, 300), (1000, 999), (1000, 1000), (1001, 1000), (4097, 244), (4097, 245),
         (20011, 1), (40000, 25), (40000, 26), (40000, 1249), (40000, 1251), (5000, 4999)]


@pytest.mark.parametrize("n,n_act", SIZES)
def test_host_plan_matches_device_plan(H, n, n_act):
    from oracle import oracle as O
    from paper_1104_2700_amd import inputs
    x, v, m = inputs.plummer(n, 40 + n)
    s = H.State(x, v, m)
    s.xp.copy_(s.x)
    s.vp.copy_(s.v)
    eps2 = (4.0 / n) ** 2
    idx = inputs.random_active(n, n_act, n_act)
    ti = torch.from_numpy(idx).cuda()
    count = torch.tensor([n_act], dtype=torch.int32, device="cuda")
    ctx = H.Context(0)
    try:
        for prec in (H.FP64, H.MIXED, H.MIXED_2F, H.MIXED_SP):
            before = ctx.counters()["interactions"]
            host = [o.clone() for o in ctx.force_jerk(s, ti, eps2, prec)]
            mid = ctx.counters()["interactions"]
            dev = ctx.force_jerk(s, ti, eps2, prec, n_act_dev=count)
            after = ctx.counters()["interactions"]
            assert mid - before == after - mid == n * n_act
            for a, b in zip(host, dev):
                assert torch.equal(a, b), prec
            if prec == H.FP64:
                pick = np.unique(np.linspace(0, n_act - 1, 40).astype(int))
                ra, rj, rp, cond = O.force(x, v, m, idx[pick], eps2, with_cond=True)
                acc, jerk, pot = (o.cpu().numpy() for o in host)
                check_fp64("acc", acc[:, pick], ra, cond[0], n)
                check_fp64("jerk", jerk[:, pick], rj, cond[1], n)
                check_fp64("pot", pot[None, pick], rp[None], cond[2], n)
    finally:
        ctx.close()
