"""CPU check of the kernel launchers: a tile or variant that has no kernel is an error,
not a launch left out (nothing is launched, so no GPU is needed)."""
import ctypes
import subprocess

import pytest

qew = pytest.importorskip("paper_1211_7275_amd.qew", reason="libqew.so not built")


def _launcher(name):
    names = subprocess.run(["nm", "-D", "--defined-only", qew.LIB_PATH], capture_output=True, text=True,
                           check=True).stdout.split()
    symbol, = [n for n in names if name in n]
    f = getattr(qew.lib(), symbol)
    f.restype = ctypes.c_int
    return f


def _tables():
    return ctypes.create_string_buffer(512)  # n_ft = 0 and null pointers


@pytest.mark.parametrize("kind,tile", [(2, 512), (3, 512), (0, 768), (1, 1536), (2, 1024), (3, 3072)])
def test_fp64_tile_without_a_kernel(kind, tile):
    f = _launcher("launch_blocked_plain")
    t, ph = _tables(), _tables()
    st = f(t, None, None, ph, ctypes.c_int(kind), ctypes.c_int(tile), ctypes.c_int(64), ctypes.c_int(2), None)
    assert st == 1  # hipErrorInvalidValue


class _SplitBuf(ctypes.Structure):
    _fields_ = [("cell", ctypes.c_void_p), ("frac", ctypes.c_void_p), ("nodes", ctypes.c_void_p)]


@pytest.mark.parametrize("kind,tile,sparse", [(2, 512, 0), (3, 512, 0), (0, 256, 1), (1, 512, 1), (0, 768, 0),
                                              (2, 5000, 1)])
def test_fused_tile_without_a_kernel(kind, tile, sparse):
    f = _launcher("launch_step_fused")
    t, ph = _tables(), _tables()
    st = f(t, _SplitBuf(), _SplitBuf(), ph, ctypes.c_int(kind), ctypes.c_int(tile), ctypes.c_int(64), ctypes.c_int(2),
           ctypes.c_int(0), ctypes.c_bool(sparse), ctypes.c_bool(True), None)
    assert st == 1
