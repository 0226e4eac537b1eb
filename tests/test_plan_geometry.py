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
    one = _info([1 << 16] * 4, k=1)  # asked for
    assert one.fp64_k == 0 and one.fp64_tile == 0 and one.n_tiles == 64


@pytest.mark.parametrize("chains", [512, 4096, 32768])
@pytest.mark.parametrize("L", [64, 128, 256])
def test_fp64_batches_of_short_chains_take_no_wide_tiles(L, chains):
    """A chain costs whole tiles: 1024 or 1536 sites for one of 64 took up to four
    times what a step per launch takes."""
    for kind in (0, 1):
        info = _info([L] * chains, kind)
        assert info.fp64_tile in (256, 512) and info.n_tiles <= 2 * chains, (kind, info.fp64_tile)
    for kind in (2, 3):
        info = _info([L] * chains, kind)
        if chains >= 4096 and L < 256:  # a narrow tile costs more than a step per launch
            assert info.fp64_tile == 0, kind
        assert info.fp64_tile in (0, 256) or L == 256, (kind, info.fp64_tile)


@pytest.mark.parametrize("kind,expect", [(0, [(112, 256), (96, 256), (64, 256), (64, 256), (64, 512), (64, 1536), (64, 1536)]),
                                         (1, [(112, 256), (64, 256), (64, 256), (64, 256), (64, 512), (64, 512), (64, 1024)]),
                                         (2, [(112, 256), (96, 256), (64, 256), (64, 1536), (64, 1536), (64, 1536), (64, 1536)]),
                                         (3, [(112, 256), (64, 256), (64, 256), (64, 256), (64, 1536), (64, 1536), (64, 1536)])])
def test_fp64_geometry_of_four_chains(kind, expect):
    """From latency to throughput: four chains of 2^10, 2^12, 2^13, 2^14, 2^16, 2^18 and 2^22 sites."""
    got = [_info([1 << lg] * 4, kind) for lg in (10, 12, 13, 14, 16, 18, 22)]
    assert [(i.fp64_k, i.fp64_tile) for i in got] == expect


@pytest.mark.parametrize("kind", [0, 1])
def test_fp64_geometry_under_a_negative_drive(kind):
    """A line that moves backwards finds no node ready on narrow tiles, so they stop
    paying early; one such drive in a batch is enough."""
    for L in (1 << 16, 1 << 18):
        assert _info([L] * 4, kind).fp64_tile < 1024 or L > 1 << 16
        for f in (-1.0, np.array([1.0, 0.5, -0.2, 2.0])):
            assert _info([L] * 4, kind, f).fp64_tile == (1024 if kind == 1 else 1536)


def test_fp64_tiles_stay_within_one_launch():
    """A launch holds fewer than 2^32 threads, 256 to a tile: random-bond lines that
    fit the memory have more 896-site tiles than that, and run one step per launch."""
    assert _info([1 << 30] * 13, 1).fp64_tile == 1024
    info = _info([1 << 30] * 15, 1)
    assert info.fp64_tile == 0 and info.n_tiles == 15 * (1 << 30) // 4096


@pytest.mark.parametrize("kind", [0, 1, 2, 3])
def test_fp64_geometry_of_fast_lines(kind):
    """Lines that move a cell or more in every step remake every window in every step:
    large batches of them run one step per launch, as do short chains that would take
    wide tiles, while a few short lines stay on narrow ones."""
    wide = 1024 if kind == 1 else 1536
    for f in (20.0, -45.0):
        assert _info([1 << 22] * 4, kind, f).fp64_tile == 0
        assert _info([384] * 4096, kind, f).fp64_tile == 0
        assert _info([1 << 10] * 4, kind, f).fp64_tile == 256
    assert _info([1 << 22] * 4, kind, 3.0).fp64_tile == wide or kind == 0
    for f in (5.0, 10.0):
        assert _info([384] * 4096, kind, f).fp64_tile != wide


def test_narrow_geometries_can_be_given():
    """The (k, tile) pairs that small fused plans are autotuned to, and no others."""
    def status(kind=0, **options):
        try:
            return _info([1000, 64], kind, fp64=False, **options)
        except qew.QewError as e:
            assert e.status == qew.QEW_EINVAL
            return None
    for k, tile in ((112, 256), (96, 256), (64, 256), (64, 512)):
        for kind in range(4):
            info = status(kind, k=k, tile=tile)
            assert (info is None) == (tile == 512 and kind >= 2)
            if info:
                assert (info.k, info.tile, info.autotuned) == (k, tile, 0)
                assert info.n_tiles == -(-1000 // (tile - 2 * k)) + -(-64 // (tile - 2 * k))
        assert status(k=k, tile=tile, flags=qew.QEW_FLAG_FUSED_DENSE) is None
        assert status(k=k, tile=tile, flags=qew.QEW_FLAG_FUSED_SPARSE) is None
        assert status(k=k, tile=tile, path=qew.QEW_ONE_STEP) is None
    for k, tile in ((0, 256), (0, 512), (32, 256), (65, 256), (112, 512), (128, 256), (64, 768)):
        assert status(k=k, tile=tile) is None
