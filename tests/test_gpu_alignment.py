"""Caches, queries and pools at addresses that suit their elements but no wider load: the scores (also of
the shapes that the query-stationary kernels take when they can), the value norms, the gather and the
whole pass must be what they are at aligned addresses.  Scores come from other kernels then, with
other float32 sums: see test_gpu_score_shapes.py for the tolerance.  Copies are bit for bit."""
import numpy as np
import pytest
import torch

import paper_2509_05165_amd as kv
import workloads as wl
from kvc_testlib import DeviceWorkload, Workload, check_end_to_end, run_compress, stream

pytestmark = pytest.mark.gpu


class Shifted(DeviceWorkload):
    """The same workload with every q, k and v moved one element off its allocation."""

    def __init__(self, w):
        super().__init__(w)
        self.q, self.k, self.v = ([self.shift(t) for t in ts] for ts in (self.q, self.k, self.v))

    @staticmethod
    def shift(t):
        out = torch.empty(t.numel() + 1, dtype=t.dtype, device="cuda")[1:]
        out.copy_(t.reshape(-1))
        assert out.data_ptr() % 16 != 0
        return out


def _workload(layers, hq, hkv, d, window, dtype, lens):
    cfg = wl.get_config(1, layers=layers, batch=len(lens), n=max(lens), dtype=dtype, head_dim=d, hq=hq, hkv=hkv,
                        window=window)
    return Workload(cfg, seed=12, lens=lens)


@pytest.mark.parametrize("layers,hq,hkv,d,window,dtype,lens,pkw", [
    (2, 8, 2, 128, 64, "bf16", [300, 45], {}),
    (2, 4, 1, 128, 32, "bf16", [5000], {}),                       # chunks of 1024 keys: shorter ones do not fit
    (1, 4, 2, 128, 256, "bf16", [2100], dict(value_norm=1)),
    (2, 10, 2, 128, 64, "bf16", [700], dict(agg_task=kv.KVC_AGG_MEAN)),
    (2, 12, 12, 128, 32, "bf16", [700, 300], dict(value_norm=1, causal_tail=1)),
    (2, 4, 2, 64, 20, "f32", [300], dict(value_norm=1)),
])
def test_scores(layers, hq, hkv, d, window, dtype, lens, pkw):
    print(f"[case] {dtype} d={d} {hq}/{hkv} M={window} {lens} {pkw}", flush=True)
    w = _workload(layers, hq, hkv, d, window, dtype, lens)
    size = kv.kvc_workspace_size(w.params(**pkw), w.total, max(lens))
    got = []
    for dw in (DeviceWorkload(w), Shifted(w)):
        ws = torch.empty(size, dtype=torch.uint8, device="cuda")
        S = torch.full((layers, hkv, w.total), -1.0, device="cuda")
        kv.kvc_score(w.params(**pkw), dw.ptrs(dw.q), dw.ptrs(dw.k), w.cu, S.data_ptr(), ws.data_ptr(), size, stream(),
                     v=dw.ptrs(dw.v))
        torch.cuda.synchronize()
        got.append(S.cpu().numpy())
    np.testing.assert_allclose(got[1], got[0], rtol=1e-4)


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 8), ("f32", 64)])
def test_gather(dtype, d):
    print(f"[case] gather {dtype} d={d}", flush=True)
    layers, hkv, n, keep = 3, 5, 1000, 333
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    k, v = (torch.randn((layers, hkv, n, d), generator=gen, device="cuda").to(tdt) for _ in range(2))
    idx = torch.stack([torch.randperm(n, generator=gen, device="cuda") for _ in range(layers * hkv)]).int()
    lengths = torch.full((layers,), keep, dtype=torch.int32, device="cuda")
    offsets = torch.arange(layers + 1, device="cuda", dtype=torch.int64) * keep
    p = kv.KvcParams(1, layers, hkv, hkv, d, 64, kv.KVC_BF16 if dtype == "bf16" else kv.KVC_F32)
    kl, vl = ([Shifted.shift(t) for t in x] for x in (k, v))
    rows = layers * keep * hkv
    out = [torch.full((rows * d + 2,), 7.0, dtype=tdt, device="cuda") for _ in range(2)]
    esz = out[0].element_size()
    kv.kvc_gather(p, [t.data_ptr() for t in kl], [t.data_ptr() for t in vl], idx.data_ptr(), lengths.data_ptr(),
                  offsets.data_ptr(), [0, n], layers * keep, out[0].data_ptr() + esz, out[1].data_ptr() + esz, stream())
    torch.cuda.synchronize()
    at = idx.view(layers, hkv, n)[:, :, :keep].long()
    for o, src in zip(out, (k, v)):
        want = torch.gather(src, 2, at[..., None].expand(-1, -1, -1, d)).reshape(-1)
        assert torch.equal(o[1:-1], want)
        assert float(o[0]) == 7.0 and float(o[-1]) == 7.0


def test_whole_pass():
    w = _workload(2, 8, 2, 128, 64, "bf16", [900, 120])
    check_end_to_end(w, run_compress(Shifted(w)), w.oracle())
