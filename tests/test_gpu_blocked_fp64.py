"""Temporally blocked FP64 kernels against the oracle, in every launch geometry
of the path and at the edges of its launches."""
import numpy as np
import pytest

from paper_1211_7275_amd import workloads

pytestmark = pytest.mark.gpu

SEED = workloads.SEED_BASE + 130
# (L, samples, steps): narrow tiles at 112, 96 and 64 steps per launch, 512-site tiles, wide tiles.
SHAPES = [(5, 2, 260), (130, 1, 260), (1001, 4, 260), (9001, 1, 230), (40_007, 1, 140), (200_003, 2, 140),
          (1_000_003, 1, 70)]


def _run(qew, p, start=None, step=0):
    sim = qew.Simulation(p, precision=qew.QEW_FP64_PLAIN, path=qew.QEW_ONE_STEP)
    try:
        if start is not None:
            for s, u in enumerate(start):
                sim.write_state(s, u, step)
        out = sim.run(resume=start is not None)
        return out, [sim.read_state(s)[0] for s in range(len(p["L"]))]
    finally:
        sim.close()


@pytest.mark.parametrize("kind", [0, 1, 2, 3])
@pytest.mark.parametrize("L,samples,steps", SHAPES)
def test_blocked_fp64_matches_oracle(kind, L, samples, steps):
    """From rough lines (jumps of several cells, both directions, every kind, a
    period, strength 0.8), with stretches of 1, 2, 3 and more steps than a
    launch takes: per site within 1e-10, the bound of the FP64 path."""
    from oracle import oracle
    from paper_1211_7275_amd import qew
    rng = np.random.default_rng(L + kind)
    start = [np.cumsum(rng.normal(0.0, 0.7, L)) - 3.0 for _ in range(samples)]
    meas = [m for m in (0, 1, 3, 6, 70) if m < steps]
    p = workloads.custom(kind, [L] * samples, 2.1, steps, meas, SEED, strength=0.8, period=11)
    print("[gpu-test] blocked FP64 kind", kind, "L", L, "x", samples, flush=True)
    out, u = _run(qew, p, start)
    for s in range(samples):
        ref = oracle.run_sample(kind, 0.8, SEED, s, L, 1.0, 0.05, 2.1, steps, meas, u0=start[s], period=11)
        assert np.max(np.abs(u[s] - ref["u"])) <= 1e-10
        assert np.max(np.abs(out["v"][s] - ref["v"])) <= 1e-10
        assert np.max(np.abs(out["ubar"][s] - ref["ubar"])) <= 1e-10


@pytest.mark.parametrize("kind", [0, 1, 2, 3])
@pytest.mark.parametrize("L", [9856 * 86 - 1, 9856 * 86, 9856 * 86 + 1])
def test_wide_tile_edges(kind, L):
    """Wide tiles (1408 and 896 valid sites) whose last one is full, short of one
    site, or a single site; the second launch takes two steps."""
    from oracle import oracle
    from paper_1211_7275_amd import qew
    steps = 66
    start = [np.cumsum(np.random.default_rng(L + kind).normal(0.0, 0.7, L))]
    p = workloads.custom(kind, [L], 2.4, steps, [0], SEED + 2)
    print("[gpu-test] blocked FP64 tile edges, kind", kind, "L", L, flush=True)
    _, u = _run(qew, p, start)
    ref = oracle.run_sample(kind, 1.0, SEED + 2, 0, L, 1.0, 0.05, 2.4, steps, [], u0=start[0])
    assert np.max(np.abs(u[0] - ref["u"])) <= 1e-10


@pytest.mark.parametrize("L", [130, 1001, 40_007, 1_000_003])
def test_every_site_changes_cell_at_once(L):
    """A line that advances one cell in every step (more requests than a wave's
    region holds), and one stopped in the middle and resumed: the oracle's line
    and the uninterrupted run, bit for bit."""
    from oracle import oracle
    from paper_1211_7275_amd import qew
    steps = 90
    p = workloads.custom(0, [L], 20.0, steps, [0, steps], SEED + 1, strength=0.25)
    _, u = _run(qew, p)
    ref = oracle.run_sample(0, 0.25, SEED + 1, 0, L, 1.0, 0.05, 20.0, steps, [])
    assert np.max(np.abs(u[0] - ref["u"])) <= 1e-10
    half = workloads.custom(0, [L], 20.0, 37, [0], SEED + 1, strength=0.25)
    _, uh = _run(qew, half)
    _, ur = _run(qew, p, uh, 37)
    assert np.array_equal(ur[0], u[0])
