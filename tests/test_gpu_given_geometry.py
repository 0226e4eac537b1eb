"""A geometry found by autotuning one plan, given to another of the same problem (also
through the call that allocates nothing): the same results, bit for bit."""
import numpy as np
import pytest

from paper_1211_7275_amd import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,L,tile", [(0, [130, 60], 256), (1, [9001] * 3, 256), (0, [40_007] * 4, 512),
                                         (3, [2001, 64], 256), (2, [300_007], 0)])
def test_autotuned_geometry_given_to_another_plan(kind, L, tile):
    import torch
    from paper_1211_7275_amd import qew
    p = workloads.custom(kind, L, 1.4, 500, [0, 5, 300, 500], workloads.SEED_BASE + 210)
    print("[gpu-test] given geometry kind", kind, "L", L, flush=True)
    with qew.Simulation(p) as sim:
        first = sim.run()
        u = [sim.read_state(s)[0] for s in range(sim.S)]
        info = sim.info()
    assert info.tile == tile if tile else info.tile >= 1024
    for noalloc in (False, True):
        with qew.Simulation(p, k=info.k, tile=info.tile) as sim:
            if noalloc:
                out = {q: np.full((sim.S, sim.n_meas), np.nan) for q in ("v", "w2", "ubar")}
                qew.qew_run_noalloc(sim.plan, sim.ws, torch.cuda.current_stream(), False, out["v"], out["w2"], out["ubar"])
            else:
                out = sim.run()
            assert sim.info().tile == info.tile and sim.info().k == info.k and not sim.info().autotuned
            for q in ("v", "w2", "ubar"):
                assert np.array_equal(out[q], first[q])
            for s in range(sim.S):
                assert np.array_equal(sim.read_state(s)[0], u[s])
