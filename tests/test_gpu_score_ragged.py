"""kvc_score over sequences of unequal lengths, whose workgroups go out longest first: whole chunks and
shorter last ones, lengths that repeat, sequences without keys, one row chunk, several, a short last one,
and workgroups of such a batch that hand themselves to the exact form.

The oracle is float64; the bound is that of tests/test_gpu_score_routes.py."""
import numpy as np
import pytest
import torch

import paper_2509_05165_amd as kv
from oracle import kvc_oracle as orc
from test_gpu_score_routes import EMIT, EMIT_KEYS, _check, _many_layers, _scores, _sharpen, _spread, _workload

pytestmark = pytest.mark.gpu

LAYERS = 128        # (all with the same queries and keys) enough workgroups for the order to be taken
SHAPES = [(4, 2, 32), (4, 1, 64), (5, 1, 64), (7, 1, 64), (8, 1, 128)]
LENS = [
    [40, 2048, 7, 2049, 300, 300, 1],        # two whole chunks of 2048
    [500, 131, 130, 500, 2],                 # none
    [7, 9, 2, 128, 30, 64, 1, 90, 90, 5, 33, 100],      # of a tile each, twelve sequences
    [2100, 1, 4096, 0, 6200, 0, 33],         # six, and sequences without keys
]
EXACT_LENS = [[40, 2048, 7, 2049, 700], [131, 600, 130, 2, 55, 40]]


@pytest.mark.parametrize("agg", [kv.KVC_AGG_MAX, kv.KVC_AGG_MEAN])
@pytest.mark.parametrize("hq,hkv,window", SHAPES)
@pytest.mark.parametrize("lens", LENS)
def test_ragged(lens, hq, hkv, window, agg):
    print(f"[case] {lens} {hq}/{hkv} M={window} agg={agg}", flush=True)
    w = _workload(hq, hkv, window, lens)
    S = _many_layers(w, LAYERS, set(), agg_task=agg)
    assert torch.equal(S[:1].expand_as(S), S)
    got = S[:1].cpu().numpy()
    for b, n in enumerate(lens):
        if n:
            ref = orc.score_layer(orc.widen(w.seq[b][0][0]), orc.widen(w.seq[b][0][1]), agg_task=agg)
            np.testing.assert_allclose(got[0][:, int(w.cu[b]):int(w.cu[b + 1])], ref, rtol=1e-4, err_msg=f"sequence {b}")


@pytest.mark.parametrize("hq,hkv,window", SHAPES[:2])
@pytest.mark.parametrize("lens", EXACT_LENS)
def test_listed_workgroups_of_a_reordered_batch(lens, hq, hkv, window):
    """The exact kernel finds the keys of a listed workgroup by the same order."""
    print(f"[case] exact form {lens} {hq}/{hkv} M={window}", flush=True)
    w, ran = _workload(hq, hkv, window, lens), set()
    _sharpen(w)
    assert np.all(_spread(w, 1).max(axis=1) > 64)
    S = _many_layers(w, LAYERS, ran)
    assert EMIT in ran and EMIT_KEYS not in ran
    assert torch.equal(S[:1].expand_as(S), S)
    _check(w, S[:1].cpu().numpy(), dust=1e-30)


@pytest.mark.parametrize("hq,hkv,window", SHAPES)
def test_the_order_changes_no_bits(hq, hkv, window):
    """One layer has too few workgroups for it."""
    w = _workload(hq, hkv, window, LENS[0])
    S = _many_layers(w, 40, set())                # (chunks of 2048 keys, as in the other launch)
    assert torch.equal(torch.from_numpy(_scores(w)).expand_as(S), S.cpu())
