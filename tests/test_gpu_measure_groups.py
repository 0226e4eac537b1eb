"""Measurements of chains of one or two measurement tiles (a workgroup takes a
whole sample) and of batches that hold a longer one (partials and a combine
launch): the same values, whichever way a batch goes."""
import numpy as np
import pytest

from paper_1211_7275_amd import workloads

pytestmark = pytest.mark.gpu

SEED = workloads.SEED_BASE + 170


@pytest.mark.parametrize("kind", [0, 1, 2, 3])
@pytest.mark.parametrize("fp64", [True, False])
@pytest.mark.parametrize("L", [[3, 4096, 100], [4097, 8192], [8193, 5, 12_288], [12_289, 16_384, 4096, 9000]])
def test_same_series_beside_a_longer_chain(kind, fp64, L):
    """Every sample's series, bit for bit, alone in its batch and beside a chain
    of five tiles; measured steps, the measurement kernels and a final one."""
    from paper_1211_7275_amd import qew
    rng = np.random.default_rng(len(L) + kind)
    start = [np.cumsum(rng.normal(0.0, 0.4, n)) for n in L + [16_385]]
    meas = [0, 1, 2, 12, 40]
    out = []
    for n in (len(L), len(L) + 1):
        p = workloads.custom(kind, (L + [16_385])[:n], 1.4, 40, meas, SEED)
        prec, path = (qew.QEW_FP64_PLAIN, qew.QEW_ONE_STEP) if fp64 else (qew.QEW_FP32_SPLIT, qew.QEW_FUSED)
        sim = qew.Simulation(p, precision=prec, path=path, k=0 if fp64 else 16, tile=0 if fp64 else 1024)
        try:
            for s in range(n):
                sim.write_state(s, start[s], 0)
            out.append(sim.run(resume=True))
        finally:
            sim.close()
    for key in ("v", "w2", "ubar"):
        assert np.all(np.isfinite(out[0][key]))
        assert np.array_equal(out[0][key], out[1][key][:len(L)]), key
