"""The rule by which kvc_score chooses its max-pooling emit pass (csrc/kvc_rules.h, compiled for the host), at
shapes where the two passes were measured at least 5 % apart, and that it is total over what a call accepts."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2509_05165_amd", "csrc")


@pytest.fixture(scope="module")
def by_keys(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    src, so = d / "rules.cpp", d / "rules.so"
    src.write_text('#include "kvc_rules.h"\n'
                   'extern "C" int by_keys(int rows, int hkv, int64_t k, int64_t wgs, int64_t n) '
                   '{ return kvc::emit_by_keys(rows, hkv, k, wgs, n); }\n')
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, "-o", str(so), str(src)], check=True)
    lib = ctypes.CDLL(str(so))
    lib.by_keys.argtypes = [ctypes.c_int, ctypes.c_int] + [ctypes.c_int64] * 3

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
