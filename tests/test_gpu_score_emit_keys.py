"""The key-stationary emit pass of heads of more than 256 rows: blocks of 32 rows in odd and even number,
query heads of 1 to 16 blocks, sequences around a workgroup's 256 keys and a wave's 64, ten KV heads (the
partials are finished out of place), the group maximum, the causal mask, forced tokens, and one row
chunk of several in the exact form.

The oracle is float64; the bound is that of tests/test_gpu_score_routes.py."""
import numpy as np
import pytest

import paper_2509_05165_amd as kv
import workloads as wl
from oracle import kvc_oracle as orc
from test_gpu_score_routes import _check, _scores, _workload

pytestmark = pytest.mark.gpu

LENS = [1, 63, 64, 65, 255, 256, 257, 700]
SHAPES = [   # hq, hkv, window: rows of a KV head
    (9, 1, 32),      # 288: an odd block at the end
    (10, 2, 32),     # 160: the query-stationary pass, for comparison
    (16, 1, 32),     # 512: two full row chunks
    (7, 1, 64),      # 448
    (8, 2, 128),     # 512
    (6, 2, 128),     # 384
    (8, 2, 256),     # 1024
    (2, 2, 512),     # 512: a query head of two row chunks
    (6, 2, 512),     # 1536
]


@pytest.mark.parametrize("causal", [0, 1])
@pytest.mark.parametrize("hq,hkv,window", SHAPES)
def test_lengths(hq, hkv, window, causal):
    print(f"[case] {hq}/{hkv} M={window} causal={causal}", flush=True)
    w = _workload(hq, hkv, window, [n + window for n in LENS] if causal else LENS)
    _check(w, _scores(w, causal_tail=causal), causal_tail=causal)


@pytest.mark.parametrize("hq,hkv,window", SHAPES)
def test_group_maximum_and_forced_tokens(hq, hkv, window):
    print(f"[case] {hq}/{hkv} M={window} group maximum", flush=True)
    w = _workload(hq, hkv, window, [300, 70])
    got = _scores(w, agg_group=kv.KVC_AGG_MAX, keep_first=3, keep_last=5)
    for b in range(2):
        ref = orc.score_layer(orc.widen(w.seq[b][0][0]), orc.widen(w.seq[b][0][1]), agg_group=kv.KVC_AGG_MAX)
        ref = orc.force_keep(ref, 3, 5)
        np.testing.assert_allclose(got[0][:, int(w.cu[b]):int(w.cu[b + 1])], ref, rtol=1e-4)


@pytest.mark.parametrize("lens", [[200, 3, 256], [400], [3000], [9000]])   # the last: more than four chunks
@pytest.mark.parametrize("hq,hkv,window", [(1, 1, 32), (5, 1, 32), (7, 1, 32), (2, 1, 64), (3, 1, 64), (2, 1, 128), (1, 1, 256)])
def test_heads_of_one_row_chunk(hq, hkv, window, lens):
    print(f"[case] {hq}/{hkv} M={window} {lens}", flush=True)
    w = _workload(hq, hkv, window, lens)
    _check(w, _scores(w))


def test_one_row_chunk_in_the_exact_form_merging_for_itself():
    w = _workload(7, 1, 32, [300, 40])
    for b in range(2):
        q, k, v = w.seq[b][0]
        qf = (q.astype(np.uint32) << 16).view(np.float32).copy()
        qf[:, 1::2] *= 20
        q = wl.f32_to_bf16_bits(qf)
        w.seq[b][0] = (q, k, v)
        w.q[0][b] = q
    _check(w, _scores(w), dust=1e-30)


def test_ten_heads():
    w = _workload(50, 10, 64, [300, 65], layers=2)
    _check(w, _scores(w))


@pytest.mark.parametrize("far", [0, 1, 2])
def test_one_row_chunk_in_the_exact_form(far):
    """Every second query of one row chunk is 20 times sharper than the others."""
    w = _workload(12, 1, 64, [700])               # 768 rows: three row chunks of four query heads
    q, k, v = w.seq[0][0]
    qf = (q.astype(np.uint32) << 16).view(np.float32).copy()
    qf[4 * far:4 * far + 4, 1::2] *= 20
    q = wl.f32_to_bf16_bits(qf)
    w.seq[0][0] = (q, k, v)
    w.q[0][0] = q
    _check(w, _scores(w), dust=1e-30)
