"""Structure factor in wide bins: every number of sample groups that the chunk
sums take, chunks of one mode more and less than a pass of theirs, against numpy."""
import numpy as np
import pytest

from paper_1211_7275_amd import workloads

pytestmark = pytest.mark.gpu

SEED = workloads.SEED_BASE + 180


@pytest.mark.parametrize("lgL", [13, 14])
@pytest.mark.parametrize("samples", [1, 2, 3, 4, 5])
def test_wide_bins_of_few_samples(lgL, samples):
    """Tolerance: that of the other rough lines (|U| good to 1e-13 of the largest,
    S to twice that times sqrt(S S_max), with room)."""
    from paper_1211_7275_amd import qew
    L = 1 << lgL
    widths = [9, 1023, 256, 255, 257, 1025] if lgL == 13 else [9, 4095, 256, 1281, 255]
    edges = np.cumsum([1] + widths)
    edges = np.append(edges, L // 2 + 1)
    p = workloads.custom(0, [L] * samples, 1.0, 0, [0], SEED, sq_edges=edges)
    print("[gpu-test] S_q chunks L = 2 ^", lgL, "x", samples, flush=True)
    rng = np.random.default_rng(lgL * 10 + samples)
    power = np.zeros(L // 2 + 1)
    worst = 0.0
    sim = qew.Simulation(p, precision=qew.QEW_FP64_PLAIN, path=qew.QEW_ONE_STEP)
    try:
        for s in range(samples):
            u = np.cumsum(rng.normal(0.0, 1.0, L)) * 0.3 + 5.0 * s
            sim.write_state(s, u, 0)
            S = (np.abs(np.fft.rfft(u - u[0])) / L) ** 2
            worst = max(worst, float(S[1:].max()))
            power += S / samples
        sim.run(resume=True)
        got = sim.structure_factor()[0]
    finally:
        sim.close()
    want = np.add.reduceat(power, edges[:-1]) / np.diff(edges)
    assert np.all(np.abs(got - want) <= 1e-12 * np.sqrt(want * worst) + 1e-24 * worst)
