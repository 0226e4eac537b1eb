"""FP64 launches of several steps against launches of one step (a plan that
measures at every step takes each of them in a launch of its own): the same
states, bit for bit."""
import numpy as np
import pytest

from paper_1211_7275_amd import workloads

pytestmark = pytest.mark.gpu

SEED = workloads.SEED_BASE + 170


def _states(qew, p, start=None, every_step=False, **options):
    steps = int(p["n_steps"])
    if every_step:
        p = dict(p, meas_steps=np.arange(steps))
    sim = qew.Simulation(p, precision=qew.QEW_FP64_PLAIN, path=qew.QEW_ONE_STEP, **options)
    try:
        if start is not None:
            for s, u in enumerate(start):
                sim.write_state(s, u, 0)
        sim.run(resume=start is not None)
        launches = sim.stats().step_launches
        assert launches == steps if every_step else launches < steps
        return [sim.read_state(s)[0] for s in range(len(p["L"]))]
    finally:
        sim.close()


def _same(qew, p, start=None):
    got, ref = _states(qew, p, start), _states(qew, p, start, every_step=True)
    for a, b in zip(got, ref):
        assert np.array_equal(a, b, equal_nan=True)


@pytest.mark.parametrize("kind", [0, 1, 2, 3])
@pytest.mark.parametrize("f", [20.0, -20.0, 7.0])
def test_bursts_on_wide_tiles(kind, f):
    """More cell changes in a wave and step than its request region holds, over a
    full launch and a part of one, on the widest tiles of every kind."""
    from paper_1211_7275_amd import qew
    L = 1_800_001
    print("[gpu-test] FP64 bursts on wide tiles, kind", kind, "f", f, flush=True)
    start = [np.cumsum(np.random.default_rng(kind).normal(0.0, 0.5, L))]
    _same(qew, workloads.custom(kind, [L], f, 90, [0], SEED, strength=0.7), start)
