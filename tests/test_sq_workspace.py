"""CPU checks of the workspace of a plan with a structure factor."""
import numpy as np
import pytest

from paper_1211_7275_amd import workloads

qew = pytest.importorskip("paper_1211_7275_amd.qew", reason="libqew.so not built")


def _bytes(L, samples, edges):
    p = workloads.custom(0, [L] * samples, 1.0, 10, [0, 10], 1, sq_edges=edges)
    pr, keep = qew.make_problem(p, precision=qew.QEW_FP64_PLAIN, path=qew.QEW_ONE_STEP)
    plan = qew.qew_plan(pr)
    try:
        return qew.qew_workspace_bytes(plan)
    finally:
        qew.qew_plan_destroy(plan)


@pytest.mark.parametrize("L,samples", [(8, 1), (8, 5), (1 << 13, 64), (1 << 20, 1), (1 << 24, 5)])
def test_two_buffers_of_the_transform_and_no_more(L, samples):
    """Two complex buffers of L / 2 points per sample, the series and the chunk sums; the sums over
    samples fit the buffer that the last pass leaves free."""
    edges = workloads.sq_edges_log(L, 8) if L > 8 else np.array([1, 3, 5])
    extra = _bytes(L, samples, edges) - _bytes(L, samples, None)
    buffers = 2 * samples * (L // 2) * 16
    chunks = sum(-(-int(n) // 4096) for n in np.diff(edges))
    assert buffers <= extra <= buffers + 2 * (len(edges) - 1) * 8 + chunks * 16 + 8 * 256
    half = L // 2
    for groups in range(1, samples + 1):  # the rows, and the mean's where it is formed
        assert (groups + (groups > 4)) * (half + 1) * 8 <= samples * half * 16
