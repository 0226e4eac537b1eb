"""Narrow tiles of the fused path (small problems with the geometry left open)
against the one-step kernel of the split state, bit for bit."""
import numpy as np
import pytest

from paper_1211_7275_amd import workloads

pytestmark = pytest.mark.gpu

SEED = workloads.SEED_BASE + 140


def _run(qew, p, path, start=None, step=0, noalloc=False):
    import torch
    sim = qew.Simulation(p, precision=qew.QEW_FP32_SPLIT, path=path)
    try:
        sim.autotune()
        if start is not None:
            for s, u in enumerate(start):
                sim.write_state(s, u, step)
        if noalloc:
            out = {k: np.full((sim.S, sim.n_meas), np.nan) for k in ("v", "w2", "ubar")}
            qew.qew_run_noalloc(sim.plan, sim.ws, torch.cuda.current_stream(), start is not None, out["v"],
                                out["w2"], out["ubar"])
        else:
            out = sim.run(resume=start is not None)
        out["u"] = np.concatenate([sim.read_state(s)[0] for s in range(sim.S)])
        return out, sim.info()
    finally:
        sim.close()


def _same(a, b):
    for key in ("v", "w2", "ubar", "u"):
        assert np.array_equal(a[key], b[key], equal_nan=True), key


# (lengths, the tile the size rule takes; kinds 2 and 3 go from 256 to the timed tiles): one, a few
# and many workgroups per CU, and the timed tiles
SHAPES = [([3, 4, 5], 256), ([130, 1001, 255], 256), ([9001] * 3, 256), ([40_007] * 4, 512),
          ([100_003] * 3, 512), ([700_001], 0)]


@pytest.mark.parametrize("kind", [0, 1, 2, 3])
@pytest.mark.parametrize("L,tile", SHAPES)
def test_narrow_tiles_match_one_step(kind, L, tile):
    """From rough lines (jumps of several cells, both directions), a period and
    strength 0.8, with stretches of one to more steps than a launch takes."""
    from paper_1211_7275_amd import qew
    rng = np.random.default_rng(sum(L) + kind)
    start = [np.cumsum(rng.normal(0.0, 0.7, n)) - 3.0 for n in L]
    p = workloads.custom(kind, L, 2.1, 260, [0, 1, 5, 9, 100, 260], SEED, strength=0.8, period=11)
    print("[gpu-test] narrow tiles kind", kind, "L", L, flush=True)
    got, info = _run(qew, p, qew.QEW_FUSED, start)
    if tile == 512 and kind >= 2:
        tile = 0
    assert info.tile == tile if tile else info.tile >= 1024
    ref, _ = _run(qew, p, qew.QEW_ONE_STEP, start)
    _same(got, ref)
    if L[0] < 10_000:
        _same(_run(qew, p, qew.QEW_FUSED, start, noalloc=True)[0], ref)


@pytest.mark.parametrize("L", [[130, 60], [40_007] * 4])
def test_narrow_tiles_from_flat_and_with_every_site_moving(L):
    """The flat start under three drives: pinned, moving, and one cell in every
    step (the nodes made ahead run out at once); a graph of 16 launches is
    replayed with eager runs between."""
    from paper_1211_7275_amd import qew
    for f in (0.3, 1.5, 20.0):
        p = workloads.custom(1, L, f, 16 * 112 * 2 + 7, [7, 16 * 112 * 2 + 7], SEED + 1)
        ref, _ = _run(qew, p, qew.QEW_ONE_STEP)
        sim = qew.Simulation(p)
        try:
            for _ in range(2):
                out = sim.run()
                out["u"] = np.concatenate([sim.read_state(s)[0] for s in range(sim.S)])
                assert sim.info().tile in (256, 512) and sim.stats().graph_launches > 0
                _same(out, ref)
        finally:
            sim.close()
