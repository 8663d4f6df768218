"""kvc_gather over pools of many blocks (one, two and three steps of the 64-way block search, blocks
of no rows among them, waves whose rows lie in several blocks), on both sides of the pool size
from which a wave takes 64 rows instead of 32 or 16, and position-ordered lists around the
stretches of 1024 words of the bit map.  Copies are bit for bit."""
import numpy as np
import pytest
import torch

import paper_2509_05165_amd as kv
from kvc_testlib import stream, to_dev, to_host_bits
from oracle import kvc_oracle as orc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order", [kv.KVC_ORDER_RANK, kv.KVC_ORDER_POSITION])
@pytest.mark.parametrize("lyr,hkv,lens,most", [
    (8, 8, [40], 40),                     # 64 blocks
    (13, 5, [40, 0, 3], 40),              # 195 blocks, an empty sequence
    (75, 8, [20] * 8, 3),                 # 4800 blocks of at most three rows
    (60, 8, [70, 700], 700),              # 262144 rows and more: 64 a wave
    (2, 3, [32767, 1], 32767),
    (1, 2, [32769, 31, 33], 32769),       # two stretches of words
    (3, 2, [16384, 16385, 16383], 16385), # a list is marked in steps of 16384 entries
    (1, 1, [491520], 491520),             # the longest list that is ordered in LDS
    (1, 1, [491521, 40], 491521),         # and the shortest that is not
])
def test_gather_of_many_blocks(order, lyr, hkv, lens, most):
    print(f"[case] gather pools order={order} lyr={lyr} hkv={hkv} {lens}", flush=True)
    r, d, nb = np.random.default_rng(4), 8, len(lens)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    total = int(cu[-1])
    ks = [r.integers(0, 2 ** 16, size=(hkv, total, d)).astype(np.uint16) for _ in range(lyr)]
    idx = np.zeros((lyr, hkv, total), dtype=np.int32)
    lengths = np.zeros((nb, lyr, hkv), dtype=np.int32)
    for b in range(nb):
        for l in range(lyr):
            for h in range(hkv):
                idx[l, h, cu[b]:cu[b + 1]] = r.permutation(lens[b])
                full = r.random() < 0.8 and most > 100
                lengths[b, l, h] = lens[b] if full else r.integers(0, min(most, lens[b]) + 1)
    offsets = np.concatenate([[0], np.cumsum(lengths.reshape(-1))]).astype(np.int64)
    rows = int(offsets[-1])
    p = kv.KvcParams(nb, lyr, hkv, hkv, d, 64, kv.KVC_BF16, unstructured=1, order=order)
    ws_bytes = kv.kvc_workspace_size(p, total, max(lens))
    ws = torch.empty(ws_bytes, dtype=torch.uint8, device="cuda")
    dk = [to_dev(x) for x in ks]
    out = torch.zeros((2, rows * d), dtype=torch.bfloat16, device="cuda")
    d_idx, d_len, d_off = to_dev(idx), to_dev(lengths.reshape(-1)), to_dev(offsets)
    ptrs = [t.data_ptr() for t in dk]
    kv.kvc_gather(p, ptrs, ptrs, d_idx.data_ptr(), d_len.data_ptr(), d_off.data_ptr(), cu, rows,
                  out[0].data_ptr(), out[1].data_ptr(), stream(), workspace=ws.data_ptr(), workspace_bytes=ws_bytes)
    torch.cuda.synchronize()
    got = to_host_bits(out).reshape(2, rows, d)
    want = np.empty((rows, d), dtype=np.uint16)
    for b in range(nb):
        lo, hi = int(cu[b]), int(cu[b + 1])
        for l in range(lyr):
            parts = orc.gather_heads(ks[l][:, lo:hi], idx[l, :, lo:hi], lengths[b, l], order == kv.KVC_ORDER_POSITION)
            for h in range(hkv):
                at = int(offsets[(b * lyr + l) * hkv + h])
                want[at:at + int(lengths[b, l, h])] = parts[h]
    np.testing.assert_array_equal(got[0], want)
    np.testing.assert_array_equal(got[1], want)
