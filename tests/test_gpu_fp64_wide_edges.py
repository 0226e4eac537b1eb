"""Wide FP64 tiles (1408 valid sites, 896 for random bond) whose last one is full,
short of one site, or a single site, at lengths where the plan takes them."""
import numpy as np
import pytest

from paper_1211_7275_amd import workloads

pytestmark = pytest.mark.gpu

SEED = workloads.SEED_BASE + 220
STEPS = 66  # a full launch and one of two steps


def _run(qew, p, start, step, k=0, valid=0):
    sim = qew.Simulation(p, precision=qew.QEW_FP64_PLAIN, path=qew.QEW_ONE_STEP, k=k)
    try:
        if valid:
            info = sim.info()
            assert info.fp64_tile - 2 * info.fp64_k == valid and info.n_tiles == -(-int(p["L"][0]) // valid)
        sim.write_state(0, start, step)
        out = sim.run(resume=True)
        return out, sim.read_state(0)[0]
    finally:
        sim.close()


@pytest.mark.parametrize("kind", [0, 1, 2, 3])
@pytest.mark.parametrize("over", [-1, 0, 1])
def test_wide_tile_edges(kind, over):
    """From rough lines (jumps of several cells, both directions), a period and strength
    0.8: one step per launch and, for random bond, the oracle; and the same line stopped
    inside a launch and resumed."""
    from paper_1211_7275_amd import qew
    valid = 896 if kind == 1 else 1408
    L = valid * (2800 if kind == 1 else 1700) + over
    print("[gpu-test] FP64 wide tile edges, kind", kind, "L", L, flush=True)
    start = np.cumsum(np.random.default_rng(L + kind).normal(0.0, 0.7, L)) - 3.0
    p = workloads.custom(kind, [L], 1.9, STEPS, [0, STEPS], SEED, strength=0.8, period=11)
    out, u = _run(qew, p, start, 0, valid=valid)
    ref, ur = _run(qew, p, start, 0, k=1)
    assert np.array_equal(u, ur)
    for key in ("v", "w2", "ubar"):
        assert np.array_equal(out[key], ref[key])
    half = workloads.custom(kind, [L], 1.9, 37, [0], SEED, strength=0.8, period=11)
    _, uh = _run(qew, half, start, 0, valid=valid)
    _, u2 = _run(qew, dict(p, meas_steps=np.array([STEPS])), uh, 37, valid=valid)
    assert np.array_equal(u2, u)
    if kind == 1 and over == 1:
        from oracle import oracle
        o = oracle.run_sample(kind, 0.8, SEED, 0, L, 1.0, 0.05, 1.9, STEPS, [], u0=start, period=11)
        assert np.max(np.abs(u - o["u"])) <= 1e-10
