"""CPU checks of the launch geometry that a plan resolves to and reports."""
import numpy as np
import pytest

from paper_1211_7275_amd import workloads

qew = pytest.importorskip("paper_1211_7275_amd.qew", reason="libqew.so not built")


def _info(L, kind=0, f=1.0, fp64=True, strength=1.0, **options):
    p = workloads.custom(kind, L, f, 100, [0, 10, 100], 123, strength=strength)
    if fp64:
        options.update(precision=qew.QEW_FP64_PLAIN, path=qew.QEW_ONE_STEP)
    pr, keep = qew.make_problem(p, **options)
    plan = qew.qew_plan(pr)
    try:
        return qew.qew_plan_info_get(plan)
    finally:
        qew.qew_plan_destroy(plan)


@pytest.mark.parametrize("kind,L,k,tile", [(0, [1024] * 4, 112, 256), (0, [1 << 16] * 4, 64, 512),
                                           (0, [1 << 22] * 4, 64, 1536), (1, [1 << 22] * 4, 64, 1024),
                                           (2, [1 << 16] * 4, 64, 1536), (3, [40, 3, 500], 112, 256)])
def test_fp64_plan_reports_its_stepping_launch(kind, L, k, tile):
    info = _info(L, kind)
    assert (info.fp64_k, info.fp64_tile) == (k, tile)
    assert info.n_tiles == sum(-(-n // (tile - 2 * k)) for n in L)
    assert info.n_meas_tiles == sum(-(-n // 4096) for n in L)
    assert info.k == 1 and info.tile == 0  # of the fused path, which this is not


def test_plans_of_one_step_per_launch_report_none():
    for info in (_info([1 << 16] * 4, strength=0.0),
                 _info([1 << 16] * 4, fp64=False, path=qew.QEW_ONE_STEP),
                 _info([1 << 16] * 4, fp64=False, k=32, tile=2048)):
        assert info.fp64_k == 0 and info.fp64_tile == 0
    assert _info([1 << 16] * 4, strength=0.0).n_tiles == 64
