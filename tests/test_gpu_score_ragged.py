"""kvc_score over sequences of unequal lengths, whose workgroups go out longest first: whole chunks and
shorter last ones, lengths that repeat, sequences without keys, one row chunk, several, a short last one.

The oracle is float64; the bound is that of tests/test_gpu_score_routes.py."""
import numpy as np
import pytest

import paper_2509_05165_amd as kv
from oracle import kvc_oracle as orc
from test_gpu_score_routes import _scores, _workload

pytestmark = pytest.mark.gpu

LENS = [
    [40, 2048, 7, 2049, 300, 300, 1],        # two whole chunks of 2048
    [500, 131, 130, 500, 2],                 # none
    [2100, 1, 4096, 0, 6200, 0, 33],         # six, and sequences without keys
]


@pytest.mark.parametrize("agg", [kv.KVC_AGG_MAX, kv.KVC_AGG_MEAN])
@pytest.mark.parametrize("hq,hkv,window", [(4, 2, 32), (4, 1, 64), (5, 1, 64), (7, 1, 64), (8, 1, 128)])
@pytest.mark.parametrize("lens", LENS)
def test_ragged(lens, hq, hkv, window, agg):
    print(f"[case] {lens} {hq}/{hkv} M={window} agg={agg}", flush=True)
    w = _workload(hq, hkv, window, lens)
    got = _scores(w, agg_task=agg)
    for b, n in enumerate(lens):
        if n:
            ref = orc.score_layer(orc.widen(w.seq[b][0][0]), orc.widen(w.seq[b][0][1]), agg_task=agg)
            np.testing.assert_allclose(got[0][:, int(w.cu[b]):int(w.cu[b + 1])], ref, rtol=1e-4, err_msg=f"sequence {b}")
