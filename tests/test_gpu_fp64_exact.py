"""FP64 launches of several steps against launches of one step (a plan that
measures at every step takes each of them in a launch of its own): the same
states, bit for bit."""
import numpy as np
import pytest

from paper_1211_7275_amd import workloads

pytestmark = pytest.mark.gpu

SEED = workloads.SEED_BASE + 170


def _states(qew, p, start=None, every_step=False, tile=0):
    steps = int(p["n_steps"])
    if every_step:
        p = dict(p, meas_steps=np.arange(steps))
    sim = qew.Simulation(p, precision=qew.QEW_FP64_PLAIN, path=qew.QEW_ONE_STEP)
    try:
        if start is not None:
            for s, u in enumerate(start):
                sim.write_state(s, u, 0)
        sim.run(resume=start is not None)
        launches = sim.stats().step_launches
        assert launches == steps if every_step else launches < steps
        if tile:
            assert sim.info().fp64_tile == tile
        return [sim.read_state(s)[0] for s in range(len(p["L"]))]
    finally:
        sim.close()


def _same(qew, p, start=None, tile=0):
    got, ref = _states(qew, p, start, tile=tile), _states(qew, p, start, every_step=True)
    for a, b in zip(got, ref):
        assert np.array_equal(a, b, equal_nan=True)


@pytest.mark.parametrize("kind", [0, 1, 2, 3])
@pytest.mark.parametrize("f,rough,strength", [(1.0, 4.0, 0.7), (-1.0, 8.0, 1.0), (2.0, 0.5, 1.0)])
def test_bursts_on_wide_tiles(kind, f, rough, strength):
    """More cell changes in a wave and step than its request region holds, jumps among
    them, over a full launch and a part of one, on the widest tiles of every kind."""
    from paper_1211_7275_amd import qew
    L = 2_500_001
    print("[gpu-test] FP64 bursts on wide tiles, kind", kind, "f", f, flush=True)
    start = [np.cumsum(np.random.default_rng(kind).normal(0.0, rough, L))]
    _same(qew, workloads.custom(kind, [L], f, 90, [0], SEED, strength=strength), start, tile=1024 if kind == 1 else 1536)


@pytest.mark.parametrize("kind", [0, 1, 2, 3])
@pytest.mark.parametrize("f", [20.0, -20.0, 18.9, 7.0])
@pytest.mark.parametrize("L", [203, 9001, 40_007])
def test_every_site_moves_on_narrow_tiles(kind, f, L):
    """A third of a cell to more than one per step, both directions."""
    from paper_1211_7275_amd import qew
    print("[gpu-test] FP64 fast lines, kind", kind, "f", f, "L", L, flush=True)
    start = [np.cumsum(np.random.default_rng(L + kind).normal(0.0, 0.5, L))]
    _same(qew, workloads.custom(kind, [L], f, 240, [0], SEED + 2, strength=0.7), start)


@pytest.mark.parametrize("kind", [0, 1, 2, 3])
@pytest.mark.parametrize("L", [203, 40_007])
@pytest.mark.parametrize("side", [1.0, -1.0])
def test_last_cells(kind, L, side):
    """Lines that reach the last 32-bit cells, whose windows go on past the largest
    integer, and pass beyond them (all sites then share the last cell)."""
    from paper_1211_7275_amd import qew
    stride, steps = 2.0**26, 24
    rng = np.random.default_rng(L + kind)
    start = [side * (2.0**31 + rng.uniform(-7.0, 5.0, L) - 20 * stride)]  # at the limit after 20 steps
    print("[gpu-test] last cells, FP64 kind", kind, "L", L, "side", side, flush=True)
    _same(qew, workloads.custom(kind, [L], side * 20.0 * stride, steps, [0], SEED), start)


@pytest.mark.parametrize("kind", [0, 1])
@pytest.mark.parametrize("L,k,tile", [(20_001, 0, 0), (200_003, 0, 0), (20_001, 24, 1024)])
def test_last_cells_split(kind, L, k, tile):
    """The same for the split state, whose cells count on past the limit: narrow
    tiles of both widths and wide ones against one step per launch."""
    from paper_1211_7275_amd import qew
    stride, at_limit = 65536, 17_520  # cells per step, the step after which the line stands at the limit
    steps = at_limit + 2
    # 4000 cells of spread: sites stand in each of the last cells
    start = 2.0**31 - at_limit * stride + 2000.0 * np.cos(2.0 * np.pi * np.arange(L) / L)
    p = workloads.custom(kind, [L], 20.0 * stride, steps, [steps], SEED + 1)
    print("[gpu-test] last cells, split kind", kind, "L", L, "k", k, flush=True)
    got = []
    for path, kk, tt in ((qew.QEW_FUSED, k, tile), (qew.QEW_ONE_STEP, 0, 0)):
        sim = qew.Simulation(p, precision=qew.QEW_FP32_SPLIT, path=path, k=kk, tile=tt)
        try:
            if not kk:
                sim.autotune()
            sim.write_state(0, start, 0)
            sim.run(resume=True)
            got.append(sim.read_state(0)[0])
        finally:
            sim.close()
    assert got[0].max() < 0.0  # past the last cell
    assert np.array_equal(got[0], got[1])


def test_one_step_per_launch_on_request():
    """k = 1: as many launches as steps, replayed as graphs, and the chosen path's bits."""
    from paper_1211_7275_amd import qew
    p = workloads.custom(0, [5000, 40_007], 1.2, 300, [0, 50], SEED + 3)
    runs = []
    for k in (0, 1):
        with qew.Simulation(p, precision=qew.QEW_FP64_PLAIN, path=qew.QEW_ONE_STEP, k=k) as sim:
            out = sim.run()
            st = sim.stats()
            assert st.step_launches == 300 if k else st.step_launches < 30
            assert st.graph_launches > 0 or not k
            runs.append([out["v"], out["w2"], out["ubar"]] + [sim.read_state(s)[0] for s in range(2)])
    for a, b in zip(*runs):
        assert np.array_equal(a, b)
