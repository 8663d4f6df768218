"""The key-stationary emit pass: heads of 32 to 8192 rows, blocks of 32 rows in odd and even number,
query heads of 1 to 32 blocks, sequences around a workgroup's 256 keys and a wave's 64, ten KV heads (the
partials are finished out of place), the group maximum, the causal mask, forced tokens, one row
chunk of several in the exact form, and the same bits on both sides of the rule that chooses the pass.

The oracle is float64; the bound is that of tests/test_gpu_score_routes.py."""
import numpy as np
import pytest
import torch

import paper_2509_05165_amd as kv
from oracle import kvc_oracle as orc
from test_gpu_score_routes import EMIT, EMIT_KEYS, _check, _many_layers, _scores, _sharpen, _workload

pytestmark = pytest.mark.gpu

LENS = [1, 63, 64, 65, 255, 256, 257, 700]
SHAPES = [   # hq, hkv, window: rows of a KV head
    (9, 1, 32),      # 288: an odd block at the end
    (10, 2, 32),     # 160: one row chunk of five blocks
    (16, 1, 32),     # 512: two full row chunks
    (7, 1, 64),      # 448
    (8, 2, 128),     # 512
    (6, 2, 128),     # 384
    (8, 2, 256),     # 1024
    (2, 2, 512),     # 512: a query head of two row chunks
    (6, 2, 512),     # 1536
]


def _scores_by_keys(w, **pkw):
    """Of layer 0, from a launch with workgroups enough for the key-stationary pass at any number of rows."""
    ran = set()
    S = _many_layers(w, 64, ran, **pkw)
    assert EMIT_KEYS in ran and EMIT not in ran
    assert torch.equal(S[:1].expand_as(S), S)
    return S[:1].cpu().numpy()


@pytest.mark.parametrize("causal", [0, 1])
@pytest.mark.parametrize("hq,hkv,window", SHAPES)
def test_lengths(hq, hkv, window, causal):
    print(f"[case] {hq}/{hkv} M={window} causal={causal}", flush=True)
    w = _workload(hq, hkv, window, [n + window for n in LENS] if causal else LENS)
    _check(w, _scores_by_keys(w, causal_tail=causal), causal_tail=causal)


@pytest.mark.parametrize("hq,hkv,window", SHAPES)
def test_group_maximum_and_forced_tokens(hq, hkv, window):
    print(f"[case] {hq}/{hkv} M={window} group maximum", flush=True)
    w = _workload(hq, hkv, window, [300, 70, 9, 33, 256, 257])
    got = _scores_by_keys(w, agg_group=kv.KVC_AGG_MAX, keep_first=3, keep_last=5)
    for b in range(w.cfg.batch):
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
    w, ran = _workload(7, 1, 32, [300, 40]), set()
    _sharpen(w)
    got = _scores(w, ran)
    assert EMIT_KEYS in ran
    _check(w, got, dust=1e-30)


def test_ten_heads():
    w = _workload(50, 10, 64, [300, 65], layers=2)
    _check(w, _scores(w))


@pytest.mark.parametrize("far", [0, 1, 2])
def test_one_row_chunk_in_the_exact_form(far):
    """Every second query of one row chunk is 20 times sharper than the others."""
    w, ran = _workload(12, 1, 64, [780]), set()   # 768 rows: three row chunks of four query heads
    _sharpen(w, slice(4 * far, 4 * far + 4))
    got = _scores(w, ran)
    assert EMIT_KEYS in ran
    _check(w, got, dust=1e-30)


BORDERS = [   # hq, hkv, window, lens, layers of the two launches: query-stationary, key-stationary
    (32, 8, 64, [512], 128, 1),              # one row chunk: at most 1536 workgroups of two chunks of keys
    (32, 8, 64, [300, 5, 512], 128, 1),
    (16, 8, 32, [400], 128, 1),
    (7, 1, 64, [300], 1, 128),               # 448 rows, few keys: from 192 workgroups on
    (9, 1, 32, [140], 1, 128),               # 288: a short last row chunk of one block
    (6, 1, 64, [150], 1, 128),               # 384: of four
    (3, 1, 128, [120, 90], 1, 100),          # of four, two sequences
    (8, 1, 256, [600], 8, 80),               # 2048
    (6, 1, 512, [300, 41, 256, 257], 1, 100),   # 3072, heads of 16 blocks: from 512 workgroups on below
    (4, 1, 1024, [2000], 1, 64),             # 4096: query heads of 32 blocks
    (8, 1, 1024, [2000], 1, 64),             # 8192: 32 row chunks, as many as there are flags
]


@pytest.mark.parametrize("far", [None, 0, -1])
@pytest.mark.parametrize("hq,hkv,window,lens,by_queries,by_keys", BORDERS)
def test_both_passes_give_the_same_bits(hq, hkv, window, lens, by_queries, by_keys, far):
    """far: the first or the last row chunk of each head in the exact form."""
    print(f"[case] both passes {hq}/{hkv} M={window} {lens} far={far}", flush=True)
    w = _workload(hq, hkv, window, lens)
    if far is not None:
        group, rows = hq // hkv, hq // hkv * window
        first = 0 if far == 0 else (rows - 1) // 256 * 256
        for h in range(hkv):
            for g in range(group):
                lo, hi = max(first - g * window, 0), min(first + 256 - g * window, window)
                if lo < hi:
                    _sharpen(w, slice(h * group + g, h * group + g + 1), slice(lo + 1, hi, 2))
    ran = set()
    a = _many_layers(w, by_queries, ran)
    assert EMIT in ran and EMIT_KEYS not in ran
    ran = set()
    b = _many_layers(w, by_keys, ran)
    assert EMIT_KEYS in ran and EMIT not in ran
    assert torch.equal(a[:1].expand_as(a), a) and torch.equal(a[:1].expand_as(b), b)
    _check(w, a[:1].cpu().numpy(), dust=0.0 if far is None else 1e-30)
