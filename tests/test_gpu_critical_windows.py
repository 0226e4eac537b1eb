"""Critical-force kernel at the edges of its forms: the node ring in LDS (up to
2048 sites; random bond in blocks of up to 512 and of up to 1024 threads) and
windows made on each visit (longer chains), even and odd lengths."""
import numpy as np
import pytest

from paper_1211_7275_amd import workloads

pytestmark = pytest.mark.gpu

SEED = workloads.SEED_BASE + 120


@pytest.mark.parametrize("kind", [0, 1])
@pytest.mark.parametrize("L", [3, 4, 5, 127, 130])
def test_short_chains_match_oracle(kind, L):
    """The same bracket as the oracle's bisection with Euler relaxations (trial
    drives this far apart are decided alike) and a pinned configuration: every
    force within the solver's 1e-10 plus FP64 rounding of the oracle's force at
    u of order M, below 1e-9."""
    from oracle import oracle
    from paper_1211_7275_amd import critical
    M, tol_f = 16, 1e-3
    print("[gpu-test] critical windows kind", kind, "L", L, flush=True)
    r = critical.critical_forces(kind, L, M, [5, 6], SEED, f_hi=4.0, tol_f=tol_f)
    for s, d in enumerate([5, 6]):
        ref = oracle.critical_force(kind, 1.0, SEED, d, L, M, f_hi=4.0, tol_f=tol_f)
        assert abs(r["f_lo"][s] - ref["f_lo"]) <= tol_f and r["f_hi"][s] - r["f_lo"][s] < tol_f
        F = oracle.forces(kind, 1.0, SEED, d, 1.0, r["f_lo"][s], r["u_c"][s], period=M)
        assert np.max(np.abs(F)) <= 1e-9


@pytest.mark.parametrize("kind", [0, 1])
@pytest.mark.parametrize("L", [1022, 1025, 1026, 2047, 2048, 2049, 4096])
def test_long_chains_from_a_rough_start(kind, L):
    """From a rough line (moves in both directions at the lower drive, across
    several cells) two samples close their bracket on a pinned configuration,
    which is the same whether they run alone or in a batch."""
    from oracle import oracle
    from paper_1211_7275_amd import critical
    M, tol_f = 8, 0.25
    print("[gpu-test] critical windows, rough start, kind", kind, "L", L, flush=True)
    u0 = np.random.default_rng(L + kind).normal(0.0, 3.0, (2, L))
    r = critical.critical_forces(kind, L, M, [7, 8], SEED + 1, f_hi=4.0, tol_f=tol_f, u0=u0)
    one = critical.critical_forces(kind, L, M, [8], SEED + 1, f_hi=4.0, tol_f=tol_f, u0=u0[1:])
    assert np.array_equal(one["u_c"][0], r["u_c"][1]) and one["sweeps"][0] == r["sweeps"][1]
    for s, d in enumerate([7, 8]):
        assert r["f_hi"][s] - r["f_lo"][s] < tol_f
        F = oracle.forces(kind, 1.0, SEED + 1, d, 1.0, r["f_lo"][s], r["u_c"][s], period=M)
        assert np.max(np.abs(F)) <= 1e-9
