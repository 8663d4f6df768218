"""kvc_score where the tiles of query rows of the key-stationary kernels wrap: one to ten tiles of 64
rows (the emit pass has three in LDS, the statistics pass two and joins the statistics of four at a
time), the last of them full or not, heads padded to 8 rows or not, rows whose pieces do not fill their slots.

The oracle is float64; the bound is that of tests/test_gpu_score_shapes.py."""
import numpy as np
import pytest

import paper_2509_05165_amd as kv
from kvc_testlib import DeviceWorkload
from test_gpu_score_shapes import _check, _scores, _workload

pytestmark = pytest.mark.gpu

CASES = [("bf16", 64, 2, 1, w, [70]) for w in (32, 33, 64, 95, 128, 129, 160, 250, 289, 320)]
CASES += [("bf16", d, 3, 1, w, [257, 5]) for d in (80, 96, 136, 192) for w in (21, 64, 107)]
CASES += [("f32", d, 2, 1, w, [200]) for d in (36, 64, 132) for w in (31, 96, 161)]


@pytest.mark.parametrize("dtype,d,hq,hkv,window,lens", CASES)
@pytest.mark.parametrize("agg", [kv.KVC_AGG_MAX, kv.KVC_AGG_MEAN])
def test_tiles(dtype, d, hq, hkv, window, lens, agg):
    print(f"[case] {dtype} d={d} hq={hq} M={window} {lens} agg={agg}", flush=True)
    w = _workload(dtype, d, hq, hkv, window, lens, layers=1)
    dw = DeviceWorkload(w)
    _check(w, _scores(w, dw, dw.ptrs(dw.q), dw.ptrs(dw.k), agg_task=agg), agg_task=agg)


@pytest.mark.parametrize("agg", [kv.KVC_AGG_MAX, kv.KVC_AGG_MEAN])
@pytest.mark.parametrize("dtype,d", [("bf16", 72), ("bf16", 136), ("bf16", 192), ("bf16", 128), ("f32", 20), ("f32", 48), ("f32", 64)])
def test_keys_of_minus_infinity(dtype, d, agg):
    """Logits of minus infinity: such a key's score is 0 and the others' are what they were without it, also
    where a row does not fill its k-steps."""
    print(f"[case] minus infinity {dtype} d={d} agg={agg}", flush=True)
    w = _workload(dtype, d, 4, 2, 9, [130, 3], layers=1)
    bits = dtype == "bf16"
    q = np.where(w.q[0] & 0x7fff, w.q[0] & 0x7fff, 1) if bits else np.abs(w.q[0]) + 1e-3
    w.q[0] = q.astype(w.q[0].dtype)                              # positive, so that no logit is plus infinity
    for at, (b, n) in enumerate([(0, 130), (1, 3)]):
        for key in (0, n - 1):
            w.k[0][:, int(w.cu[b]) + key, d - 1 - at] = 0xff80 if bits else -np.inf
        lo, hi = int(w.cu[b]), int(w.cu[b + 1])
        w.seq[b][0] = (w.q[0][b], np.ascontiguousarray(w.k[0][:, lo:hi]), w.seq[b][0][2])
    dw = DeviceWorkload(w)
    got = _scores(w, dw, dw.ptrs(dw.q), dw.ptrs(dw.k), agg_task=agg)
    assert (got[0][:, [0, 129, 130, 132]] == 0).all()
    _check(w, got, agg_task=agg)
