"""The order of a score launch over sequences of unequal lengths (csrc/kvc_grid.h, compiled for the host): every
block of the grid once, in groups of 256 slices, and what blockIdx.x counts last is worked last."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2509_05165_amd", "csrc")


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("pairs")
    src, so = d / "pairs.cpp", d / "pairs.so"
    src.write_text('#include "kvc_grid.h"\n'
                   'extern "C" void block(uint32_t p, uint32_t gx, uint32_t hkv, uint32_t rcs, uint32_t gz, uint32_t* out) '
                   '{ auto b = kvc::pair_major_block(p, gx, hkv, rcs, gz); out[0] = b.bx; out[1] = b.by; out[2] = b.bz; }\n')
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, "-o", str(so), str(src)], check=True)
    lib = ctypes.CDLL(str(so))
    lib.block.restype, lib.block.argtypes = None, [ctypes.c_uint32] * 5 + [ctypes.c_void_p]
    return lib


@pytest.mark.parametrize("gx,hkv,row_chunks,gz", [
    (1, 1, 1, 1), (2, 8, 1, 32), (16, 4, 2, 28), (3, 5, 3, 7), (257, 1, 2, 2), (32, 8, 16, 5)])
def test_every_block_once_and_bx_slowest(lib, gx, hkv, row_chunks, gz):
    out = (ctypes.c_uint32 * 3)()
    got = []
    for p in range(gx * hkv * row_chunks * gz):
        lib.block(p, gx, hkv, row_chunks, gz, out)
        got.append(tuple(out))
    assert got[0] == (0, 0, 0)                       # the block that clears the list of the emit pass
    assert sorted(got) == [(x, y, z) for x in range(gx) for y in range(hkv * row_chunks) for z in range(gz)]
    group = 256 * row_chunks
    for at in range(0, len(got), group):
        part = got[at:at + group]
        assert [b[1] % row_chunks for b in part] == sorted(b[1] % row_chunks for b in part)
        for rc in range(row_chunks):
            bx = [b[0] for b in part if b[1] % row_chunks == rc]
            assert bx == sorted(bx)
        if at:
            assert min(b[0] for b in part) >= max(b[0] for b in got[at - group:at])


def test_nothing_wraps_at_the_largest_launch(lib):
    out = (ctypes.c_uint32 * 3)()
    lib.block(2 ** 31 - 1, 2 ** 21, 1, 8, 128, out)
    assert tuple(out) == (2 ** 21 - 1, 7, 127)
