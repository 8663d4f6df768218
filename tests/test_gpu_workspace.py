"""A workspace below kvc_workspace_size is accepted as long as the stages fit one by one, and gives
the same results: the selection's scratch then takes a launch of its own to clear, and the scores
of shapes outside the query-stationary kernels take fewer layers at a time, or, where not even one
fits, the plain kernels.  `small` is the size that the library asked for before it reserved space
for those routes.  Nothing may be written behind the bytes that were given."""
import numpy as np
import pytest
import torch

import paper_2509_05165_amd as kv
import workloads as wl
from kvc_testlib import DeviceWorkload, Workload, stream

pytestmark = pytest.mark.gpu

GUARD = 1 << 16
CASES = [
    # layers, hq, hkv, d, window, dtype, lens, small, plain, options
    (3, 8, 2, 128, 64, "bf16", [2000], 360704, False, {}),
    (2, 8, 8, 128, 32, "bf16", [400, 12289], 5787392, False, dict(order=kv.KVC_ORDER_POSITION)),
    (8, 16, 2, 64, 100, "bf16", [700], 336384, False, {}),
    (3, 24, 12, 80, 40, "bf16", [300, 500], 816384, False, dict(value_norm=1)),
    (2, 8, 1, 256, 512, "f32", [700], 137472, True, {}),
    (2, 4, 2, 64, 33, "f32", [600], 72704, False, dict(unstructured=1, order=kv.KVC_ORDER_POSITION)),
    (40, 8, 8, 128, 32, "bf16", [400, 13000, 300], 124944384, False, dict(unstructured=1)),
]


@pytest.mark.parametrize("layers,hq,hkv,d,window,dtype,lens,small,plain,pkw", CASES)
def test_a_small_workspace_gives_the_same_results(layers, hq, hkv, d, window, dtype, lens, small, plain, pkw):
    print(f"[case] {dtype} d={d} {hq}/{hkv} M={window} {lens} in {small} bytes {pkw}", flush=True)
    cfg = wl.get_config(1, layers=layers, batch=len(lens), n=max(lens), dtype=dtype, head_dim=d, hq=hq, hkv=hkv,
                        window=window)
    w = Workload(cfg, seed=9, lens=lens, budgets=[0] * len(lens))
    dw = DeviceWorkload(w)
    p = w.params(**pkw)
    full = kv.kvc_workspace_size(p, w.total, max(lens))
    rows = layers * (hkv if pkw.get("unstructured") else 1)
    heads = 1 if pkw.get("unstructured") else hkv
    budget = [kv.kvc_budget(30, rows, n) for n in lens]
    got = []
    for size in (full, small):
        ws = torch.full((size + GUARD,), 0xAB, dtype=torch.uint8, device="cuda")
        S = torch.full((layers, hkv, w.total), -1.0, device="cuda")
        out = {"k": torch.zeros(sum(budget) * heads * d, dtype=dw.k[0].dtype, device="cuda")}
        out["v"] = torch.zeros_like(out["k"])
        out["lengths"] = torch.full((len(lens) * rows,), -1, dtype=torch.int32, device="cuda")
        out["offsets"] = torch.full((len(lens) * rows + 1,), -1, dtype=torch.int64, device="cuda")
        kv.kvc_score(p, dw.ptrs(dw.q), dw.ptrs(dw.k), w.cu, S.data_ptr(), ws.data_ptr(), size, stream(),
                     v=dw.ptrs(dw.v))
        kv.kvc_compress(p, dw.ptrs(dw.q), dw.ptrs(dw.k), dw.ptrs(dw.v), w.cu, budget, out["k"].data_ptr(),
                        out["v"].data_ptr(), out["lengths"].data_ptr(), out["offsets"].data_ptr(), ws.data_ptr(),
                        size, stream())
        torch.cuda.synchronize()
        assert bool((ws[size:] == 0xAB).all())
        assert int(out["lengths"].sum()) == sum(budget)
        got.append((S, out))
    (S0, out0), (S1, out1) = got
    if plain:   # other sums of the same float32 products: see test_gpu_score_shapes.py
        np.testing.assert_allclose(S1.cpu().numpy(), S0.cpu().numpy(), rtol=1e-4)
        return
    assert torch.equal(S0, S1)
    for name in out0:
        assert torch.equal(out0[name].view(torch.uint8), out1[name].view(torch.uint8)), name
