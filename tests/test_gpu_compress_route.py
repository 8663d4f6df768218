"""kvc_compress takes the composite, the selection and their scratch through a route of its own
(aggregation and first histogram in one launch, counts of the sorted rows by searching them).
It must give what the stage calls give on the same scores, bit for bit: composite, threshold,
lengths and offsets, over the borders of that route (4 and 8 heads with and without 16-byte
aligned sequences, other head counts around their batches of four, pools of up to 256 rows and more,
floors, ties, forced
tokens, empty sequences, budgets of nothing and of everything)."""
import numpy as np
import pytest
import torch

import paper_2509_05165_amd as kv
import workloads as wl
from kvc_testlib import DeviceWorkload, Workload, stream

pytestmark = pytest.mark.gpu

CASES = [
    # layers, hq, hkv, lens, keep percent, options
    (3, 16, 8, [400, 36], 30, {}),
    (3, 16, 8, [401, 35, 1], 30, dict(min_per_layer=7)),
    (5, 8, 4, [4100, 64], 50, {}),
    (2, 8, 4, [4099], 10, dict(agg_head=kv.KVC_AGG_MAX)),
    (2, 6, 3, [300, 0, 77], 40, dict(min_per_layer=100)),
    (2, 9, 9, [2047, 1], 30, {}),                                # heads in batches of four behind the first: 4 + 4
    (2, 12, 12, [2049, 300], 30, dict(min_per_layer=7)),         # 4 + 4 + 3
    (2, 6, 6, [4100], 30, dict(agg_head=kv.KVC_AGG_MAX)),        # 4 + 1
    (3, 2, 1, [2100], 30, {}),                                   # none
    (1, 8, 8, [40], 100, {}),
    (4, 8, 8, [257], 0, {}),
    (70, 2, 2, [130], 25, {}),                                   # more rows than lanes of a wave
    (32, 8, 8, [300, 20], 35, dict(unstructured=1)),             # 256 rows: searched
    (33, 8, 8, [300, 20], 35, dict(unstructured=1, min_per_layer=3)),   # 264 rows: swept
    (3, 16, 8, [2500], 20, dict(keep_first=4, keep_last=64)),    # +inf scores at the top of every row
]


@pytest.mark.parametrize("ties", [False, True])
@pytest.mark.parametrize("layers,hq,hkv,lens,keep,pkw", CASES)
def test_compress_selects_what_the_stages_select(layers, hq, hkv, lens, keep, pkw, ties):
    print(f"[case] layers={layers} hkv={hkv} {lens} keep={keep} {pkw} ties={ties}", flush=True)
    cfg = wl.get_config(1, layers=layers, batch=len(lens), n=max(lens), hq=hq, hkv=hkv, window=32, head_dim=128)
    w = Workload(cfg, seed=5, lens=lens, budgets=[0] * len(lens))
    rows = layers * (hkv if pkw.get("unstructured") else 1)
    floor = pkw.get("min_per_layer", 0)
    budget = [max(kv.kvc_budget(keep, rows, n), rows * min(floor, n)) for n in lens]
    dw = DeviceWorkload(w)
    if ties:                                                     # equal keys: equal scores in long runs
        for k in dw.k:
            k[:, 1::2] = k[:, 0:1]
    p = w.params(**pkw)
    total, nblk = w.total, len(lens) * rows
    ws_bytes = kv.kvc_workspace_size(p, total, max(lens))
    ws = torch.empty(ws_bytes, dtype=torch.uint8, device="cuda")
    heads = 1 if pkw.get("unstructured") else hkv
    out = [torch.zeros(max(sum(budget) * heads, 1) * 128, dtype=torch.bfloat16, device="cuda") for _ in range(2)]

    def results():
        return dict(composite=torch.full((layers, total), -1.0, device="cuda"),
                    tau=torch.full((len(lens),), -1.0, device="cuda"),
                    lengths=torch.full((nblk,), -1, dtype=torch.int32, device="cuda"),
                    offsets=torch.full((nblk + 1,), -1, dtype=torch.int64, device="cuda"))

    S = torch.empty((layers, hkv, total), device="cuda")
    idx = torch.empty((layers, hkv, total), dtype=torch.int32, device="cuda")
    ss = torch.empty_like(S)
    for _ in range(2):                                           # the second pass meets a used workspace
        got = results()
        kv.kvc_compress(p, dw.ptrs(dw.q), dw.ptrs(dw.k), dw.ptrs(dw.v), w.cu, budget, out[0].data_ptr(),
                        out[1].data_ptr(), got["lengths"].data_ptr(), got["offsets"].data_ptr(),
                        ws.data_ptr(), ws_bytes, stream(), scores=S.data_ptr(), idx=idx.data_ptr(),
                        s_sorted=ss.data_ptr(), composite=got["composite"].data_ptr(), tau=got["tau"].data_ptr())
    want = results()
    if pkw.get("unstructured"):
        want["composite"] = got["composite"]                     # not computed
        pool = ss
    else:
        kv.kvc_composite(p, ss.data_ptr(), w.cu, want["composite"].data_ptr(), stream())
        pool = want["composite"]
    kv.kvc_global_select(p, pool.data_ptr(), w.cu, budget, want["tau"].data_ptr(), want["lengths"].data_ptr(),
                         want["offsets"].data_ptr(), ws.data_ptr(), ws_bytes, stream())
    torch.cuda.synchronize()
    for name in want:
        np.testing.assert_array_equal(got[name].cpu().numpy(), want[name].cpu().numpy(), err_msg=name)
    assert int(got["lengths"].sum()) == sum(budget)
