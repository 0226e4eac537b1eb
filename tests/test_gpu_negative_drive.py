"""Lines under a negative drive, which move backwards: the geometry the fused path
takes for them by rule, and their states against the one-step kernel, bit for bit."""
import numpy as np
import pytest

from paper_1211_7275_amd import workloads

pytestmark = pytest.mark.gpu

SEED = workloads.SEED_BASE + 190


@pytest.mark.parametrize("kind", [0, 1])
@pytest.mark.parametrize("L,narrow", [(130, True), (1 << 13, True), (1 << 14, False), (1 << 16, False)])
def test_backward_lines(kind, L, narrow):
    """Narrow tiles keep no node behind a site, so they end where a few of them fill
    the chip; one negative drive in the batch is enough."""
    from paper_1211_7275_amd import qew
    drives = np.array([1.0, -1.0, 0.4, 1.7])
    p = workloads.custom(kind, [L] * 4, drives, 300, [0, 100, 300], SEED)
    print("[gpu-test] negative drive kind", kind, "L", L, flush=True)
    states = []
    for path in (qew.QEW_FUSED, qew.QEW_ONE_STEP):
        sim = qew.Simulation(p, precision=qew.QEW_FP32_SPLIT, path=path)
        try:
            out = sim.run()
            if path == qew.QEW_FUSED:
                assert (sim.info().tile < 1024) == narrow
            states.append([out["v"], out["w2"], out["ubar"]] + [sim.read_state(s)[0] for s in range(4)])
        finally:
            sim.close()
    for a, b in zip(*states):
        assert np.array_equal(a, b)
