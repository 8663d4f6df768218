"""kvc_score at the shapes of the key-stationary matrix-core kernels: head sizes and types
whose rows need padding to whole k-steps, windows around the padding of a query head to 8
rows and of a tile to 64, sequences around a workgroup's 256 (128) keys, the masks, the other
aggregators, more layers than one launch takes, and rows at addresses its loads cannot take.

The oracle is float64.  A logit is a float32 sum of d products: its rounding error is about
sqrt(d) 2^-24 |q| |k| scale <= 16 * 6e-8 * 60 = 6e-5 at d = 256 with these inputs' sinks, and a
score is relative to exp(logit): hence 1e-4."""
import numpy as np
import pytest
import torch

import paper_2509_05165_amd as kv
import workloads as wl
from oracle import kvc_oracle as orc
from kvc_testlib import DeviceWorkload, Workload, stream

pytestmark = pytest.mark.gpu

MEAN = dict(agg_task=kv.KVC_AGG_MEAN)
GMAX = dict(agg_group=kv.KVC_AGG_MAX)
CAUSAL = dict(causal_tail=1)
CASES = [
    # dtype, d, hq, hkv, window, lens, options
    ("bf16", 64, 8, 2, 64, [1, 255, 256, 257], {}),
    ("bf16", 80, 4, 4, 8, [300, 31], {}),
    ("bf16", 96, 7, 1, 9, [513, 33], {}),
    ("bf16", 128, 8, 2, 200, [700, 64], {}),
    ("bf16", 256, 6, 2, 63, [259], {}),
    ("bf16", 72, 4, 2, 17, [300], {}),
    ("bf16", 8, 2, 2, 5, [40], {}),
    ("bf16", 192, 2, 1, 65, [257], {}),
    ("bf16", 64, 24, 12, 7, [300], {}),
    ("bf16", 128, 4, 1, 1, [2000], {}),
    ("bf16", 64, 3, 3, 300, [100, 600], {}),
    ("f32", 20, 4, 2, 33, [300], {}),
    ("f32", 32, 8, 2, 12, [255, 1, 400], {}),
    ("f32", 64, 8, 2, 32, [513], {}),
    ("f32", 128, 4, 2, 71, [257], {}),
    ("f32", 256, 6, 2, 40, [127, 128, 129], {}),
    ("bf16", 64, 8, 2, 100, [100, 356, 613], CAUSAL),
    ("bf16", 128, 6, 2, 24, [281, 24], CAUSAL),
    ("f32", 64, 8, 4, 257, [300, 600], CAUSAL),
    ("f32", 256, 4, 2, 30, [150], dict(CAUSAL, **MEAN)),
    ("bf16", 64, 8, 2, 30, [290], dict(CAUSAL, **MEAN)),
    ("bf16", 80, 8, 2, 13, [300], MEAN),
    ("f32", 64, 8, 2, 64, [300], dict(MEAN, **GMAX)),
    ("bf16", 96, 8, 2, 21, [300], dict(GMAX, add_head_mean=0)),
    ("bf16", 64, 4, 2, 30, [290], dict(keep_first=3, keep_last=5)),
]


def _scores(w, dw, q, k, **pkw):
    c = w.cfg
    S = torch.full((c.layers, c.hkv, w.total), -1.0, dtype=torch.float32, device="cuda")
    kv.kvc_score(w.params(**pkw), q, k, w.cu, S.data_ptr(), dw.ws.data_ptr(), dw.ws_bytes, stream())
    torch.cuda.synchronize()
    return S.cpu().numpy()


def _check(w, got, **pkw):
    okw = {x: pkw[x] for x in ("agg_task", "agg_group") if x in pkw}
    okw["add_head_mean"] = bool(pkw.get("add_head_mean", 1))
    okw["causal_tail"] = bool(pkw.get("causal_tail", 0))
    for b in range(w.cfg.batch):
        for l in range(w.cfg.layers):
            ref = orc.score_layer(orc.widen(w.seq[b][l][0]), orc.widen(w.seq[b][l][1]), **okw)
            ref = orc.force_keep(ref, pkw.get("keep_first", 0), pkw.get("keep_last", 0))
            np.testing.assert_allclose(got[l][:, int(w.cu[b]):int(w.cu[b + 1])], ref, rtol=1e-4,
                                       err_msg=f"sequence {b} layer {l}")


def _workload(dtype, d, hq, hkv, window, lens, layers=2):
    cfg = wl.get_config(1, layers=layers, batch=len(lens), n=max(lens), dtype=dtype, head_dim=d,
                        hq=hq, hkv=hkv, window=window)
    return Workload(cfg, seed=3, lens=lens)


@pytest.mark.parametrize("dtype,d,hq,hkv,window,lens,pkw", CASES)
def test_scores_of_any_shape(dtype, d, hq, hkv, window, lens, pkw):
    print(f"[case] {dtype} d={d} hq={hq} hkv={hkv} M={window} {lens} {pkw}", flush=True)
    w = _workload(dtype, d, hq, hkv, window, lens)
    dw = DeviceWorkload(w)
    _check(w, _scores(w, dw, dw.ptrs(dw.q), dw.ptrs(dw.k), **pkw), **pkw)


def test_more_layers_than_one_launch_takes():
    # 32 * 16 * 100 rows x (16 chunks x 8 + 4) bytes = 6.8 MB of statistics a layer: nine
    # layers reach the 64 MB that are held at once
    w = _workload("bf16", 16, 16, 2, 100, [4096] + [40] * 31, layers=11)
    dw = DeviceWorkload(w)
    _check(w, _scores(w, dw, dw.ptrs(dw.q), dw.ptrs(dw.k)))


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_rows_off_16_byte_addresses(dtype):
    w = _workload(dtype, 64, 8, 2, 20, [300, 45])
    dw = DeviceWorkload(w)

    def shifted(t):
        buf = torch.empty(t.numel() + 1, dtype=t.dtype, device="cuda")
        buf[1:] = t.reshape(-1)
        return buf

    q, k = [shifted(t) for t in dw.q], [shifted(t) for t in dw.k]
    esz = q[0].element_size()
    got = _scores(w, dw, [t.data_ptr() + esz for t in q], [t.data_ptr() + esz for t in k])
    _check(w, got)
