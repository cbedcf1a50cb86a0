"""Runs in launches of many block steps from several threads at once, each
with a context and a stream of its own: as many of up to 1536 particles as
fit share the device, one beyond has it alone, the others take single steps,
and every one gives the result it gives alone, bit for bit."""
import threading

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

TB = 20
KEYS = ("x", "v", "a", "j", "pot", "t", "dt")


def test_runs_from_several_threads():
    from paper_1104_2700_amd import hermite as H
    from paper_1104_2700_amd import inputs
    params = H.dt_params(0.02, 0, 3, 20)
    jobs = []
    for n in (900, 3000, 1500, 6000, 300, 700, 1100):
        ctx = H.Context(0)
        x, v, m = inputs.plummer(n, n)
        s0 = H.State(x, v, m, TB)
        eps2 = (4.0 / n) ** 2
        ctx.initialize(s0, eps2, params, H.FP64)
        alone = s0.clone()
        counts = ctx.run(alone, eps2, params, 1 << TB, H.FP64, max_steps=60)
        jobs.append((ctx, s0, eps2, alone, counts))
    torch.cuda.synchronize()
    errors = []

    def work(ctx, s0, eps2, alone, counts):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for _ in range(4):
                    s = s0.clone()
                    assert ctx.run(s, eps2, params, 1 << TB, H.FP64, max_steps=60) == counts
                    torch.cuda.current_stream().synchronize()
                    for key in KEYS:
                        assert torch.equal(getattr(s, key), getattr(alone, key)), key
        except BaseException as e:   # noqa: BLE001 - reported by the test's own thread
            errors.append(e)

    threads = [threading.Thread(target=work, args=j) for j in jobs]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for j in jobs:
        j[0].close()
    if errors:
        raise errors[0]
