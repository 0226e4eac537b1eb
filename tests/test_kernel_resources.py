"""CPU check of the registers of the compiled kernels (the code object's own
metadata)."""
import os
import re
import struct
import subprocess

import pytest

qew = pytest.importorskip("paper_1211_7275_amd.qew", reason="libqew.so not built")

READELF = "/opt/rocm/llvm/bin/llvm-readelf"


def _gfx950_object():
    import bench
    data = open(qew.LIB_PATH, "rb").read()
    _, off, size, _ = bench._elf_sections(data)[".hip_fatbin"]
    blob = data[off:off + size]
    n, = struct.unpack_from("<Q", blob, 24)
    pos = 32
    for _ in range(n):
        eoff, esize, tlen = struct.unpack_from("<QQQ", blob, pos)
        if b"gfx950" in blob[pos + 24:pos + 24 + tlen]:
            return blob[eoff:eoff + esize]
        pos += 24 + tlen
    raise AssertionError("no gfx950 code object in the library")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{symbol: (vector registers, spilled ones)} of every kernel of the library."""
    path = tmp_path_factory.mktemp("code") / "gfx950.co"
    path.write_bytes(_gfx950_object())
    notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
    out = {}
    for entry in notes.split("- .agpr_count:")[1:]:
        field = {k: re.search(r"\.%s:\s+(\S+)" % k, entry)[1] for k in ("name", "vgpr_count", "vgpr_spill_count")}
        out[field["name"]] = (int(field["vgpr_count"]), int(field["vgpr_spill_count"]))
    return out


def _waves(vgprs):
    return min(8, 512 // (-(-vgprs // 8) * 8))


@pytest.mark.skipif(not os.path.exists(READELF), reason="no llvm-readelf")
@pytest.mark.parametrize("kind", [0, 1, 2, 3])
@pytest.mark.parametrize("per_thread", [4, 6, 8, 12, 16])
def test_sparse_kernel_runs_as_many_waves_as_the_dense_one(kernels, kind, per_thread):
    """The sparse variant exists to be faster on slow lines: it must not lose a wave
    per SIMD to registers, nor spill more than two of them more (which measured as
    nothing; eleven cost a seventh)."""
    rounds = per_thread <= 8  # the dense kernel of lines that are not fast
    dense, = [v for n, v in kernels.items() if f"k_step_fusedILi{kind}ELi{per_thread}ELb0ELb{int(rounds)}E" in n]
    sparse, = [v for n, v in kernels.items() if f"k_step_fusedILi{kind}ELi{per_thread}ELb1E" in n]
    assert _waves(sparse[0]) >= _waves(dense[0])
    assert sparse[1] <= dense[1] + 2
