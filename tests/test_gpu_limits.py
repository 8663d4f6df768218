"""A call at the limits of its grids: 128 layers and 256 sequences of one token with 64 and 128 heads
are 2^21 and 2^22 workgroups of the rank kernel, whose flat thread index needs 64 bits."""
import numpy as np
import pytest
import torch

import paper_2509_05165_amd as kv
from kvc_testlib import stream

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hkv", [64, 128])
def test_compress_of_millions_of_segments(hkv):
    print(f"[case] 128 layers, {hkv} heads, 256 sequences of one token", flush=True)
    layers, batch, d = 128, 256, 8
    cu = list(range(batch + 1))
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1)

    def cache():
        return [torch.randn((hkv, batch, d), generator=gen, device="cuda").to(torch.bfloat16) for _ in range(layers)]

    q = torch.randn((batch, hkv, 1, d), generator=gen, device="cuda").to(torch.bfloat16)
    k, v = cache(), cache()
    p = kv.KvcParams(batch, layers, hkv, hkv, d, 1, kv.KVC_BF16)
    keep = [b % (layers + 1) for b in range(batch)]
    rows = sum(keep) * hkv
    ws_bytes = kv.kvc_workspace_size(p, batch, 1)
    ws = torch.empty(ws_bytes, dtype=torch.uint8, device="cuda")
    k_out = torch.zeros((rows, d), dtype=torch.bfloat16, device="cuda")
    v_out = torch.zeros_like(k_out)
    lengths = torch.full((batch * layers,), -1, dtype=torch.int32, device="cuda")
    offsets = torch.full((batch * layers + 1,), -1, dtype=torch.int64, device="cuda")
    kv.kvc_compress(p, [q.data_ptr()] * layers, [t.data_ptr() for t in k], [t.data_ptr() for t in v], cu, keep,
                    k_out.data_ptr(), v_out.data_ptr(), lengths.data_ptr(), offsets.data_ptr(), ws.data_ptr(),
                    ws_bytes, stream())
    torch.cuda.synchronize()
    # one token takes the whole softmax: all scores are equal, and ties go to the first layers
    want = np.array([[l < keep[b] for l in range(layers)] for b in range(batch)], dtype=np.int32)
    np.testing.assert_array_equal(lengths.cpu().numpy().reshape(batch, layers), want)
    np.testing.assert_array_equal(offsets.cpu().numpy(), np.concatenate([[0], np.cumsum(want.reshape(-1))]))
    for out, src in ((k_out, k), (v_out, v)):
        ref = torch.cat([torch.stack(src[:keep[b]])[:, :, b].reshape(-1, d) for b in range(batch) if keep[b]])
        assert torch.equal(out.view(torch.int16), ref.view(torch.int16))
