"""The sums over a particle's lanes at the end of a sweep: every number of
lanes (64 to 1, set by the active count under a tuning that asks for no more
lanes than that), one and two particles per lane, full and ragged items, in
every precision, against the CPU oracle."""
import numpy as np
import pytest

from tests.gpu_util import check_fp64, check_mixed, fp32_policy

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

N = 700


@pytest.fixture(scope="module")
def H():
    from paper_1104_2700_amd import hermite
    return hermite


@pytest.mark.parametrize("variant", [0, 1])
@pytest.mark.parametrize("n_act", [1, 4, 5, 8, 16, 33, 64, 130, 257, 512])
def test_sums_over_lanes(H, n_act, variant):
    from oracle import oracle as O
    from paper_1104_2700_amd import inputs
    x, v, m = inputs.plummer(N, 5)
    s = H.State(x, v, m)
    s.xp.copy_(s.x)
    s.vp.copy_(s.v)
    eps2 = (4.0 / N) ** 2
    idx = inputs.random_active(N, n_act, n_act)
    ti = torch.from_numpy(idx).cuda()
    ref = O.force(x, v, m, idx, eps2, with_cond=True)
    ctx = H.Context(0)
    try:
        fp32_policy(H, ctx)
        for prec in (H.FP64, H.MIXED, H.MIXED_2F):
            ctx.set_tuning(prec, H.CTuning(256, 5, 1, variant))
            got = [o.cpu().numpy() for o in ctx.force_jerk(s, ti, eps2, prec)]
            for name, a, b, cond in zip(("acc", "jerk", "pot"), got, ref[:3], ref[3]):
                a, b = np.atleast_2d(a), np.atleast_2d(b)
                if prec == H.FP64:
                    check_fp64(name, a, b, cond, N)
                else:
                    check_mixed(name, a, b, cond)
    finally:
        ctx.close()
