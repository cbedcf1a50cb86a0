"""The step numbers that tag the words exchanged by runs of 1537 to 16384
particles: their start over at 2^32, and sizes in turn on one context, whose
words share one buffer.

A launch takes the numbers of its steps and two more; without max_steps these
are sync_every, whether or not it gets to do them.  A run up to time 0 does
none, so it moves the numbers on at no cost."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

TB = 20
STEPS = 40
KEYS = ("x", "v", "a", "j", "pot", "t", "dt")


class Runs:
    def __init__(self, H):
        self.H, self.ctx, self.at, self.known = H, H.Context(0), 1, {}
        self.params = H.dt_params(0.02, H.DT_PAPER, 3, 20)

    def _system(self, n):
        from paper_1104_2700_amd import inputs
        if n not in self.known:
            s = self.H.State(*inputs.plummer(n, 8 + n), TB)
            eps2 = (4.0 / n) ** 2
            self.ctx.initialize(s, eps2, self.params, self.H.FP64)
            ref = s.clone()
            self.ctx.run(ref, eps2, self.params, 1 << TB, self.H.FP64, use_graph=False,
                         max_steps=STEPS)
            self.known[n] = (s, eps2, ref)
        return self.known[n]

    def check(self, n):
        """A run against its single steps, bit for bit."""
        s0, eps2, ref = self._system(n)
        s = s0.clone()
        self.ctx.run(s, eps2, self.params, 1 << TB, self.H.FP64, max_steps=STEPS)
        torch.cuda.synchronize()
        for key in KEYS:
            assert torch.equal(getattr(s, key), getattr(ref, key)), (n, key)
        self.at += STEPS + 2

    def advance(self, to, n=1600):
        """Moves the number that the next launch starts from to `to` (at least
        4098 on: a launch is of 4096 steps or sync_every)."""
        s0, eps2, _ = self._system(n)
        while self.at < to:
            by = min(to - self.at, 1 << 31)
            rest = to - self.at - by
            if 0 < rest < 4098:
                by -= 4098
            assert self.ctx.run(s0.clone(), eps2, self.params, 0, self.H.FP64,
                                sync_every=by - 2) == (0, 0)
            self.at += by


@pytest.fixture()
def runs():
    from paper_1104_2700_amd import hermite as H
    r = Runs(H)
    yield r
    r.ctx.close()


@pytest.mark.parametrize("left", [1, 20, STEPS + 1, STEPS + 2, STEPS + 3])
def test_numbers_start_over(runs, left):
    """A launch that would pass 2^32, its last number just below, at and past
    it; then runs with the new numbers, over words of the old ones."""
    runs.check(3000)
    runs.advance((1 << 32) - left)
    for n in (3000, 9973, 3000, 1600):
        runs.check(n)


def test_plans_are_never_taken_for_words(runs):
    """A plan is a byte a block size (6: 64 lanes and one tile a chunk); four
    of them read as the number 0x06060606.  A larger system's run with that
    number after a smaller one's."""
    runs.check(16384)
    for n in (2048, 1600, 5000):
        runs.check(n)
    runs.advance(0x06060606 - STEPS // 2, n=2048)
    runs.check(16384)


def test_the_longest_interval_between_checks(runs):
    """sync_every = 2^31 - 1: one launch, checked at its end."""
    n = 1600
    s0, eps2, ref = runs._system(n)
    s = s0.clone()
    runs.ctx.run(s, eps2, runs.params, 1 << TB, runs.H.FP64, sync_every=(1 << 31) - 1,
                 max_steps=STEPS)
    torch.cuda.synchronize()
    for key in KEYS:
        assert torch.equal(getattr(s, key), getattr(ref, key)), key
