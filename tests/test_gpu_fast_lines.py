"""Lines that move a cell or more in every step, on the fused path: the kernel whose
lanes make their own windows against the one-step kernel, bit for bit."""
import numpy as np
import pytest

from paper_1211_7275_amd import workloads

pytestmark = pytest.mark.gpu

SEED = workloads.SEED_BASE + 200


def _run(qew, p, start, path, k=0, tile=0):
    sim = qew.Simulation(p, precision=qew.QEW_FP32_SPLIT, path=path, k=k, tile=tile)
    try:
        for s, u in enumerate(start):
            sim.write_state(s, u, 0)
        out = sim.run(resume=True)
        return [out["v"], out["w2"], out["ubar"]] + [sim.read_state(s)[0] for s in range(len(start))]
    finally:
        sim.close()


@pytest.mark.parametrize("tile", [1024, 1536, 2048, 3072])
@pytest.mark.parametrize("kind", [0, 1, 2, 3])
@pytest.mark.parametrize("f,period", [(21.0, 0), (-45.0, 13), (18.9, 0)])
def test_fast_lines_match_one_step(kind, f, period, tile):
    """One and more cells per step, forwards and backwards (f dt on both sides of the
    line between the two kernels), rough chains longer and shorter than a tile."""
    from paper_1211_7275_amd import qew
    L = [7001, 900, 5]
    rng = np.random.default_rng(tile + kind)
    start = [np.cumsum(rng.normal(0.0, 0.5, n)) for n in L]
    p = workloads.custom(kind, L, f, 70, [0, 9, 70], SEED, strength=0.9, period=period)
    print("[gpu-test] fast lines kind", kind, "f", f, "tile", tile, flush=True)
    for a, b in zip(_run(qew, p, start, qew.QEW_FUSED, 24, tile), _run(qew, p, start, qew.QEW_ONE_STEP)):
        assert np.array_equal(a, b)
