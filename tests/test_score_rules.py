"""The rules by which kvc_score chooses its max-pooling emit pass and the order of a ragged batch (csrc/kvc_rules.h,
compiled for the host), at shapes where the two ways were measured at least 5 % apart, and that the first is total over
what a call accepts."""
import ctypes
import os
import subprocess

import pytest

import test_gpu_score_ragged as ragged

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2509_05165_amd", "csrc")


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    src, so = d / "rules.cpp", d / "rules.so"
    src.write_text('#include "kvc_rules.h"\n'
                   'extern "C" int by_keys(int rows, int hkv, int64_t k, int64_t wgs, int64_t n) '
                   '{ return kvc::emit_by_keys(rows, hkv, k, wgs, n); }\n'
                   'extern "C" int longest_first(int64_t wgs, int row_chunks, int whole, int last, int hi, int lo) '
                   '{ return kvc::longest_first(wgs, row_chunks, whole, last, hi, lo); }\n')
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, "-o", str(so), str(src)], check=True)
    lib = ctypes.CDLL(str(so))
    lib.by_keys.argtypes = [ctypes.c_int, ctypes.c_int] + [ctypes.c_int64] * 3
    lib.longest_first.argtypes = [ctypes.c_int64] + [ctypes.c_int] * 5
    return lib


@pytest.fixture(scope="module")
def by_keys(lib):
    def rule(hq, hkv, window, layers, *lens):
        wgs = sum((n + 255) // 256 for n in lens) * hkv * layers
        return bool(lib.by_keys(hq // hkv * window, hkv, layers * hkv * sum(lens) * 256, wgs, max(lens)))
    return rule


@pytest.mark.parametrize("hq,hkv,window,layers,lens,slower", [   # key- / query-stationary time
    (8, 1, 256, 1, [100], 2.02), (8, 1, 256, 28, [600], 1.44), (8, 1, 256, 1, [1500], 1.14), (28, 4, 256, 1, [100], 1.69),
    (28, 4, 256, 8, [300], 1.40), (32, 8, 512, 1, [600], 1.25), (64, 8, 128, 1, [300], 1.10), (8, 1, 64, 1, [100], 1.18),
    (28, 4, 64, 1, [100], 1.16), (32, 8, 256, 1, [100], 1.18), (28, 4, 256, 1, [50, 300, 120, 90], 1.51)])
def test_few_workgroups_of_many_rows_stay_query_stationary(by_keys, hq, hkv, window, layers, lens, slower):
    assert not by_keys(hq, hkv, window, layers, *lens)


@pytest.mark.parametrize("hq,hkv,window,layers,lens,faster", [
    (40, 8, 64, 1, [100], 0.88), (40, 8, 64, 28, [300], 0.95), (28, 4, 64, 1, [600], 0.89), (64, 8, 128, 1, [1500], 0.81),
    (32, 8, 512, 28, [100], 0.89), (32, 8, 1024, 80, [256], 0.83), (8, 1, 64, 1, [800], 0.90), (28, 4, 64, 28, [8192], 0.92),
    (40, 8, 128, 28, [8192], 0.90), (64, 8, 128, 80, [8192], 0.97), (128, 16, 256, 1, [1000], 0.80), (7, 1, 32, 1, [2500], 0.63)])
def test_enough_keys_or_workgroups_go_key_stationary(by_keys, hq, hkv, window, layers, lens, faster):
    assert by_keys(hq, hkv, window, layers, *lens)


def test_more_row_chunks_than_flags_never_go_key_stationary(by_keys):
    for n in (1, 300, 100000):
        assert by_keys(8, 1, 1024, 80, n, n, n, n, n, n, n)
        assert not by_keys(33, 1, 256, 80, n, n, n, n, n, n, n)


def _longest_first(lib, hq, hkv, window, layers, lens, chunk=2048):
    row_chunks = -(-(hq // hkv * window) // 256)
    whole, rest = sum(n // chunk for n in lens), [n % chunk for n in lens if n % chunk]
    wgs = (whole + len(rest)) * hkv * row_chunks * layers
    tiles = [chunk // 128] * (whole > 0) + [-(-n // 128) for n in rest]
    return bool(lib.longest_first(wgs, row_chunks, whole, len(rest), max(tiles), min(tiles)))


@pytest.mark.parametrize("hq,hkv,window,layers,lens,slower", [   # longest first / sequence by sequence
    (6, 2, 32, 1, [597, 130], 1.08), (16, 8, 32, 16, [42, 136], 1.07), (7, 1, 64, 16, [143, 79, 120], 1.07),
    (8, 8, 256, 16, [70, 59, 46], 1.11), (28, 4, 512, 28, [64, 66, 26], 1.07), (64, 8, 32, 16, [26, 107], 1.09),
    (40, 8, 1024, 1, [83, 29], 1.09), (64, 8, 128, 16, [11, 2], 1.08), (32, 8, 64, 32, [4096, 4096], 1.0)])
def test_few_or_equally_long_workgroups_stay_in_order(lib, hq, hkv, window, layers, lens, slower):
    assert not _longest_first(lib, hq, hkv, window, layers, lens)


@pytest.mark.parametrize("hq,hkv,window,layers,lens,faster", [
    (32, 8, 64, 32, [1000, 3000], 0.80), (28, 4, 64, 28, [150, 4000, 900, 2500], 0.90), (8, 1, 64, 64, [9] * 16, 0.93),
    (32, 8, 64, 32, [100, 900, 1500, 300], 0.81)])
def test_ragged_batches_go_longest_first(lib, hq, hkv, window, layers, lens, faster):
    assert _longest_first(lib, hq, hkv, window, layers, lens)


def test_launches_whose_workgroups_need_more_than_32_bits_stay_in_order(lib):
    assert lib.longest_first((1 << 31) - 1, 1, 5, 2, 16, 1)
    assert not lib.longest_first(1 << 31, 1, 5, 2, 16, 1)


@pytest.mark.parametrize("hq,hkv,window", ragged.SHAPES)
@pytest.mark.parametrize("chunk", [2048, 4096])
def test_the_gpu_tests_of_the_order_take_it(lib, hq, hkv, window, chunk):
    for lens in ragged.LENS:
        assert _longest_first(lib, hq, hkv, window, ragged.LAYERS, lens, chunk) or hq // hkv * window > 256 and chunk < max(lens)
    for lens in ragged.EXACT_LENS:
        assert _longest_first(lib, hq, hkv, window, ragged.LAYERS, lens, chunk)
    assert _longest_first(lib, hq, hkv, window, 40, ragged.LENS[0]) and not _longest_first(lib, hq, hkv, window, 1, ragged.LENS[0])
