"""Rounding of the full FP64 sweeps by pairs against that of the one-sided
sweep (an explicit list of every particle takes that one) on the same inputs,
both measured against the oracle's compensated sums.

A particle's error is taken relative to the sum of its terms' magnitudes: the
partial sums, whose roundings make it, are at most that, however far the sum
itself cancels.  In both sweeps a register adds a run of terms and the runs'
sums are added in further levels.  From 45000 particles on the runs of both are
of up to 256 terms and the root mean squares differ by their scatter (1500
particles: 1 / sqrt(2 * 1500) = 2 % for the potentials) and by the levels
above: 1.1.  Smaller systems' runs are within a factor of two in length (64 to
256 terms by pairs, 256 over the lanes of a particle one-sided), and a run's
rounding goes with the root of its length: sqrt(2) of that."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

ROWS = 1500


@pytest.fixture(scope="module")
def H():
    from paper_1104_2700_amd import hermite
    return hermite


@pytest.fixture(scope="module")
def ctx(H):
    c = H.Context(0)
    yield c
    c.close()


def _rms(got, ref, cond):
    e = np.linalg.norm(np.atleast_2d(got) - np.atleast_2d(ref), axis=0) / cond
    return float(np.sqrt(np.mean(e ** 2)))


@pytest.mark.parametrize("sizes,tol", [([6001], 1.1 * 2 ** 0.5), ([14001], 1.1 * 2 ** 0.5),
                                       ([44000], 1.1 * 2 ** 0.5), ([65536], 1.1), ([100000], 1.1),
                                       ([8192] * 8, 1.1 * 2 ** 0.5)])
def test_rounding_against_the_one_sided_sweep(H, ctx, sizes, tol):
    from oracle import oracle as O
    from paper_1104_2700_amd import inputs
    parts = [inputs.plummer(k, 21 + k + c) for c, k in enumerate(sizes)]
    x, v = (np.concatenate([p[q] for p in parts], axis=1) for q in (0, 1))
    m = np.concatenate([p[2] for p in parts])
    n, k = m.shape[0], sizes[0]
    eps2 = (4.0 / k) ** 2
    cl = None
    if len(sizes) > 1:
        off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
        cl = H.Clusters(off, np.full(len(sizes), eps2))
    s = H.State(x, v, m)
    s.xp.copy_(s.x)
    s.vp.copy_(s.v)
    ident = torch.arange(n, dtype=torch.int32, device="cuda")
    pairs = [o.cpu().numpy() for o in ctx.force_jerk(s, None, eps2, H.FP64, clusters=cl)]
    single = [o.cpu().numpy() for o in ctx.force_jerk(s, ident, eps2, H.FP64, clusters=cl)]
    rows = np.sort(np.random.default_rng(n).choice(k, ROWS, replace=False)).astype(np.int32)
    ref = O.force(x[:, :k], v[:, :k], m[:k], rows, eps2, with_cond=True)
    for name, a, b, r, c in zip(("acc", "jerk", "pot"), pairs, single, ref[:3], ref[3]):
        ea, eb = _rms(a[..., rows], r, c), _rms(b[..., rows], r, c)
        print("%s rms error: by pairs %.3e, one-sided %.3e" % (name, ea, eb))
        assert ea <= tol * eb, (name, ea, eb)
