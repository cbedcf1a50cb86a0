"""Full FP64 sweeps by pairs against the one-sided sweep (an explicit list of
every particle takes that one) and the CPU oracle, at the sizes where the
pair blocks, tiles and shapes end.

Tolerance: both paths are held to the FP64 bar of the other sweep tests
(1e-13 relative, or 4 sqrt(N) u sum_j |term_j|); against each other the bars
add."""
import numpy as np
import pytest

from tests.gpu_util import check_fp64

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def H():
    from paper_1104_2700_amd import hermite
    return hermite


@pytest.fixture(scope="module")
def ctx(H):
    c = H.Context(0)
    yield c
    c.close()


def _state(H, sizes, seed):
    from paper_1104_2700_amd import inputs
    rng = np.random.default_rng(seed)
    parts = [inputs.plummer(k, seed + 7 * c, masses=rng.uniform(0.1, 1.0, k))
             for c, k in enumerate(sizes)]
    x, v = (np.concatenate([p[q] for p in parts], axis=1) for q in (0, 1))
    m = np.concatenate([p[2] for p in parts])
    s = H.State(x, v, m)
    s.xp.copy_(s.x)
    s.vp.copy_(s.v)
    return s, x, v, m


def _check(ctx, H, s, x, v, m, off, eps2, cl):
    """Every particle against the one-sided sweep, some of every system
    against the oracle, and a second call bit for bit."""
    from oracle import oracle as O
    n = s.n
    out = [o.clone() for o in ctx.force_jerk(s, None, float(eps2[0]), H.FP64, clusters=cl)]
    again = ctx.force_jerk(s, None, float(eps2[0]), H.FP64, clusters=cl)
    ident = torch.arange(n, dtype=torch.int32, device="cuda")
    ref = ctx.force_jerk(s, ident, float(eps2[0]), H.FP64, clusters=cl)
    energy = ctx.energy(s, float(eps2[0]), clusters=cl).cpu().numpy()
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(out, again))
    out = [o.cpu().numpy() for o in out]
    ref = [o.cpu().numpy() for o in ref]
    rng = np.random.default_rng(n)
    for c in range(len(off) - 1):
        lo, hi = int(off[c]), int(off[c + 1])
        edges = [q for q in (lo, hi - 1, lo + 191, lo + 192, lo + 255, lo + 256, lo + 1023,
                             lo + 1024) if lo <= q < hi]
        idx = np.unique(np.concatenate([edges, rng.integers(lo, hi, 60)])).astype(np.int32)
        ra, rj, rp, cond = O.force(x, v, m, idx, float(eps2[c]), j_range=(lo, hi),
                                   with_cond=True)
        check_fp64("acc", out[0][:, idx], ra, cond[0], hi - lo)
        check_fp64("jerk", out[1][:, idx], rj, cond[1], hi - lo)
        check_fp64("pot", out[2][None, idx], rp[None], cond[2], hi - lo)
        w = 0.5 * np.sum(m[lo:hi] * out[2][lo:hi])
        k = 0.5 * np.sum(m[lo:hi] * np.sum(v[:, lo:hi] ** 2, axis=0))
        assert abs(energy[c, 1] - w) <= 1e-13 * abs(w) and abs(energy[c, 0] - k) <= 1e-13 * k
    # sum_j |term_j| of a particle is at most its potential's size over the
    # shortest distance's powers: here the jerk's condition is taken from the
    # oracle sample's worst, 1e4
    for q, tol in ((0, 2e-13), (1, 4 * np.sqrt(n) * 2.0 ** -53 * 1e4), (2, 2e-13)):
        a, b = np.atleast_2d(out[q]), np.atleast_2d(ref[q])
        err = np.linalg.norm(a - b, axis=0) / np.maximum(np.linalg.norm(b, axis=0), 1e-300)
        assert np.sqrt(np.mean(err ** 2)) <= tol, (q, err.max())


@pytest.mark.parametrize("n", [4500, 6000, 6144, 6145, 6335, 19999, 20000, 24577, 45000, 46081])
def test_one_system(H, ctx, n):
    """Even and odd numbers of blocks, a last block of one particle and a
    full one, and the first size of every shape."""
    s, x, v, m = _state(H, [n], 300 + n)
    _check(ctx, H, s, x, v, m, [0, n], [(4.0 / n) ** 2], None)


@pytest.mark.parametrize("sizes", [[192, 8192, 1, 5000], [8191, 193, 384, 6000, 2, 385],
                                   [700] * 150])
def test_ensembles(H, ctx, sizes):
    s, x, v, m = _state(H, sizes, 900 + len(sizes))
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    eps2 = (4.0 / np.maximum(np.array(sizes, float), 64)) ** 2
    _check(ctx, H, s, x, v, m, off, eps2, H.Clusters(off, eps2))


def test_coincident_particles_without_softening(H, ctx):
    """Two coincident particles at zero softening make each other's sums
    non-finite and nobody else's, as in the one-sided sweep."""
    n = 6200
    s, *_ = _state(H, [n], 77)
    s.xp[:, 5000] = s.xp[:, 17]
    ident = torch.arange(n, dtype=torch.int32, device="cuda")
    out = ctx.force_jerk(s, None, 0.0, H.FP64)
    ref = ctx.force_jerk(s, ident, 0.0, H.FP64)
    torch.cuda.synchronize()
    for a, b in zip(out, ref):
        bad = ~torch.isfinite(a.reshape(-1, n)).all(0)
        assert torch.equal(bad, ~torch.isfinite(b.reshape(-1, n)).all(0))
        assert bad.nonzero().flatten().tolist() == [17, 5000]
