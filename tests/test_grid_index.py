"""Flat thread indices of a launch (csrc/kvc_grid.h, compiled for the host) at the limits of a call:
layers * hkv <= 65535 pairs and 256 sequences give up to 2^24 workgroups of 1024 threads.  In 32
bits the index of the last ones is negative, and the step over a whole grid of 2^21 or 2^22
workgroups is -2^31 or 0: a loop over cleared words then leaves its buffer or never ends.  And the order of a score launch whose last row chunk is short: every block
of the grid once."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2509_05165_amd", "csrc")
THREADS = 1024


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("grid")
    src, so = d / "grid.cpp", d / "grid.so"
    src.write_text('#include "kvc_grid.h"\n'
                   'extern "C" int64_t first(uint32_t bx, uint32_t by, uint32_t gx, uint32_t n, uint32_t t) '
                   '{ return kvc::flat_thread(bx, by, gx, n, t); }\n'
                   'extern "C" int64_t step(uint32_t gx, uint32_t gy, uint32_t n) { return kvc::grid_threads(gx, gy, n); }\n'
                   'extern "C" void block(uint32_t p, uint32_t gx, uint32_t hkv, uint32_t rcs, uint32_t gz, uint32_t* out) '
                   '{ auto b = kvc::row_chunk_block(p, gx, hkv, rcs, gz); out[0] = b.bx; out[1] = b.by; out[2] = b.bz; }\n')
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, "-o", str(so), str(src)], check=True)
    lib = ctypes.CDLL(str(so))
    for f, n in ((lib.first, 5), (lib.step, 3)):
        f.restype, f.argtypes = ctypes.c_int64, [ctypes.c_uint32] * n
    return lib


@pytest.mark.parametrize("gx,gy", [(1, 1), (3, 2), (8192, 256), (16384, 256), (65535, 256), (65535, 1)])
def test_flat_index_is_exact_at_the_limits(lib, gx, gy):
    assert lib.step(gx, gy, THREADS) == gx * gy * THREADS
    for bx, by, t in ((0, 0, 0), (gx - 1, 0, 7), (gx // 2, gy // 2, 1), (gx - 1, gy - 1, THREADS - 1)):
        assert lib.first(bx, by, gx, THREADS, t) == (by * gx + bx) * THREADS + t
    assert lib.first(gx - 1, gy - 1, gx, THREADS, THREADS - 1) == lib.step(gx, gy, THREADS) - 1


def test_the_threads_of_a_grid_share_the_words_out(lib):
    gx, gy, words = 3, 2, 20000
    seen = []
    for by in range(gy):
        for bx in range(gx):
            for t in range(THREADS):
                seen += range(lib.first(bx, by, gx, THREADS, t), words, lib.step(gx, gy, THREADS))
    assert sorted(seen) == list(range(words))


@pytest.mark.parametrize("gx,hkv,row_chunks,gz", [
    (1, 1, 2, 1), (2, 8, 2, 32), (3, 5, 3, 7), (255, 1, 2, 1), (256, 1, 4, 1), (257, 1, 2, 2), (64, 4, 9, 3)])
def test_every_block_of_a_launch_with_a_short_row_chunk_comes_once(lib, gx, hkv, row_chunks, gz):
    out = (ctypes.c_uint32 * 3)()
    lib.block.restype = None
    got = []
    for p in range(gx * hkv * row_chunks * gz):
        lib.block(p, gx, hkv, row_chunks, gz, out)
        got.append(tuple(out))
    assert got[0] == (0, 0, 0)                                # the block that clears the list of the emit pass
    assert sorted(got) == [(x, y, z) for x in range(gx) for y in range(hkv * row_chunks) for z in range(gz)]
    # 256 slices at a time, their last row chunks behind all others
    head = min(256, gx * hkv * gz) * row_chunks
    last = [b[1] % row_chunks == row_chunks - 1 for b in got[:head]]
    assert last == sorted(last)
    # and nothing wraps at the largest launch
    lib.block(2 ** 31 - 1, 2 ** 21, 1, 8, 128, out)
    assert tuple(out) == (2 ** 21 - 1, 7, 127)
