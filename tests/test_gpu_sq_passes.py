"""Structure factor at the lengths where its plan of passes changes (one
workgroup per sample up to L = 2^13, then two, three and four passes of 32 to
128 points), sample groups and narrow, wide and mixed bins, against numpy."""
import numpy as np
import pytest

from paper_1211_7275_amd import workloads

pytestmark = pytest.mark.gpu

SEED = workloads.SEED_BASE + 150


def _edges(L, mode):
    if mode == "all":
        return workloads.sq_edges_full(L)
    if mode == "log":
        return workloads.sq_edges_log(L, 24)
    top = L // 2 + 1
    return np.unique(np.array([1, 2, 3, 4, min(9000, top - 1), top]))  # single modes beside one of several chunks


@pytest.mark.parametrize("fp64", [True, False])
@pytest.mark.parametrize("lgL,samples,mode", [(3, 2, "all"), (4, 1, "all"), (5, 3, "all"), (12, 5, "log"),
                                              (13, 70, "all"), (13, 3, "mix"), (14, 1, "all"), (14, 9, "mix"),
                                              (15, 3, "log"), (16, 6, "mix"), (18, 2, "all"), (19, 5, "log"),
                                              (23, 1, "mix")])
def test_modes_of_rough_lines(fp64, lgL, samples, mode):
    """Rough lines written and measured.  The chain holds the line to 2^-24 per
    offset in the split precision, so the reference takes the line read back.
    Error of the FFT: some 20 roundings per butterfly level of values up to the
    largest |U_n|, so |U| is good to 1e-13 of the largest (lgL 2^-53 20 = 5e-14)
    and S to twice that times sqrt(S S_max)."""
    from paper_1211_7275_amd import qew
    L = 1 << lgL
    rng = np.random.default_rng(lgL * 100 + samples)
    edges = _edges(L, mode)
    p = workloads.custom(0, [L] * samples, 1.0, 0, [0], SEED, sq_edges=edges)
    prec, path = (qew.QEW_FP64_PLAIN, qew.QEW_ONE_STEP) if fp64 else (qew.QEW_FP32_SPLIT, qew.QEW_ONE_STEP)
    print("[gpu-test] S_q L = 2 ^", lgL, "x", samples, mode, flush=True)
    sim = qew.Simulation(p, precision=prec, path=path)
    power = np.zeros(L // 2 + 1)
    try:
        for s in range(samples):
            sim.write_state(s, np.cumsum(rng.normal(0.0, 1.0, L)) * 0.3 + 5.0 * s, 0)
        sim.run(resume=True)
        got = sim.structure_factor()[0]
        worst = 0.0
        for s in range(samples):
            u = sim.read_state(s)[0]
            S = (np.abs(np.fft.rfft(u - u[0])) / L) ** 2
            worst = max(worst, float(S[1:].max()))
            power += S / samples
    finally:
        sim.close()
    want = np.add.reduceat(power[:edges[-1]], edges[:-1]) / np.diff(edges)
    assert np.all(np.abs(got - want) <= 1e-12 * np.sqrt(want * worst) + 1e-24 * worst)
