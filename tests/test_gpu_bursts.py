"""Bursts of cell changes on the fused path: more requests in a wave and
sub-step than its region holds, on every tile width, both variants."""
import numpy as np
import pytest

from paper_1211_7275_amd import workloads

pytestmark = pytest.mark.gpu

SEED = workloads.SEED_BASE + 160


@pytest.mark.parametrize("tile", [1024, 1536, 2048, 3072, 4096])
@pytest.mark.parametrize("kind,f,strength", [(0, 20.0, 0.7), (1, 20.0, 0.7), (0, 7.0, 1.0), (1, 45.0, 1.0), (2, 12.0, 1.0),
                                             (3, -16.0, 1.0)])
def test_bursts_match_one_step(kind, f, strength, tile):
    """Lines that move a third of a cell to two cells per step, forwards and
    backwards, from a rough start: the one-step kernel's states, bit for bit."""
    from paper_1211_7275_amd import qew
    L = [7001, 1200]
    rng = np.random.default_rng(tile + kind)
    start = [np.cumsum(rng.normal(0.0, 0.5, n)) for n in L]
    p = workloads.custom(kind, L, f, 70, [0, 9, 70], SEED, strength=strength)
    print("[gpu-test] bursts kind", kind, "f", f, "tile", tile, flush=True)
    runs = []
    for path, k, t, flags in ((qew.QEW_ONE_STEP, 0, 0, 0), (qew.QEW_FUSED, 24, tile, qew.QEW_FLAG_FUSED_DENSE),
                              (qew.QEW_FUSED, 24, tile, qew.QEW_FLAG_FUSED_SPARSE)):
        sim = qew.Simulation(p, precision=qew.QEW_FP32_SPLIT, path=path, k=k, tile=t, flags=flags)
        try:
            for s, u in enumerate(start):
                sim.write_state(s, u, 0)
            out = sim.run(resume=True)
            runs.append((out, np.concatenate([sim.read_state(s)[0] for s in range(2)])))
        finally:
            sim.close()
    for out, u in runs[1:]:
        assert np.array_equal(u, runs[0][1])
        for key in ("v", "w2", "ubar"):
            assert np.array_equal(out[key], runs[0][0][key])
