"""kvc_score at the shapes of the query-stationary kernels: one, two and four waves along the rows, a
short last row chunk worked by one or two of them (1 to 4 blocks of 32 rows left over 256), up to
four chunks of keys (the emit pass merges the statistics itself) and more (a launch of its own), the two
aggregators, the causal mask, and workgroups that hand themselves to the exact form.  The max-pooling emit
pass of most heads of more than 256 rows is the key-stationary one: EMIT_SHAPES lists heads whose emit pass
is query-stationary, and the tests over it look at the kernels that ran.

The oracle is float64.  A logit is a float32 sum of 128 products: about sqrt(128) 2^-24 |q| |k| scale
<= 11 * 6e-8 * 60 = 4e-5 with these inputs' sinks, and a score is relative to exp(logit): 1e-4."""
import numpy as np
import pytest
import torch

import paper_2509_05165_amd as kv
import workloads as wl
from oracle import kvc_oracle as orc
from kvc_testlib import DeviceWorkload, Workload, stream

pytestmark = pytest.mark.gpu

EMIT, EMIT_KEYS = "score_mfma<emit>", "score_emit_keys"
MEAN = dict(agg_task=kv.KVC_AGG_MEAN)
CAUSAL = dict(causal_tail=1)
SHAPES = [   # hq, hkv, window: rows of a KV head
    (2, 2, 64),      # 64: one wave along the rows
    (4, 2, 64),      # 128: two
    (4, 1, 64),      # 256: four
    (7, 1, 64),      # 256 + 192: a last chunk too long for the short form
    (9, 1, 32),      # 256 + 32
    (10, 2, 64),     # 256 + 64
    (11, 1, 32),     # 256 + 96
    (6, 2, 128),     # 256 + 128
    (7, 1, 128),     # 3 x 256 + 128
]
# few keys for the rows of a head, or few workgroups of very many rows: the emit pass of max pooling is the
# query-stationary one.  hq, hkv, window, tokens
EMIT_SHAPES = [
    (2, 2, 64, 700), (4, 2, 64, 700), (4, 1, 64, 700),
    (7, 1, 64, 130),                                    # 256 + 192
    (9, 1, 32, 130), (10, 2, 64, 140), (33, 1, 64, 300),      # a short form of one wave along the rows
    (11, 1, 32, 200), (6, 2, 128, 200), (7, 1, 128, 700), (67, 1, 32, 300),   # of two
    (33, 1, 64, 8300), (67, 1, 32, 8300),               # the same and a merge of more than four chunks
]


def _workload(hq, hkv, window, lens, layers=1, **over):
    cfg = wl.get_config(1, layers=layers, batch=len(lens), n=max(lens), hq=hq, hkv=hkv, window=window, **over)
    return Workload(cfg, seed=6, lens=lens)


def _scores(w, ran=None, **pkw):
    """ran: a set that the names of the kernels are added to."""
    dw = DeviceWorkload(w)
    S = torch.full((w.cfg.layers, w.cfg.hkv, w.total), -1.0, device="cuda")
    if ran is not None:
        kv.kvc_profile_collect()
        kv.kvc_profile_enable(True)
    try:
        kv.kvc_score(w.params(**pkw), dw.ptrs(dw.q), dw.ptrs(dw.k), w.cu, S.data_ptr(), dw.ws.data_ptr(), dw.ws_bytes,
                     stream())
    finally:
        if ran is not None:
            kv.kvc_profile_enable(False)
            ran.update(kv.kvc_profile_collect())
    torch.cuda.synchronize()
    return S.cpu().numpy()


def _many_layers(w, layers, ran, **pkw):
    """Scores of a launch of `layers` layers that all have the queries and keys of layer 0.  ran: as in _scores."""
    dw, c = DeviceWorkload(w), w.cfg
    p = kv.KvcParams(c.batch, layers, c.hq, c.hkv, c.head_dim, c.window, w.dtype, **pkw)
    size = kv.kvc_workspace_size(p, w.total, int(w.lens.max()))
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    S = torch.full((layers, c.hkv, w.total), -1.0, device="cuda")
    kv.kvc_profile_collect()
    kv.kvc_profile_enable(True)
    try:
        kv.kvc_score(p, dw.ptrs(dw.q) * layers, dw.ptrs(dw.k) * layers, w.cu, S.data_ptr(), ws.data_ptr(), size, stream())
    finally:
        kv.kvc_profile_enable(False)
        ran.update(kv.kvc_profile_collect())
    torch.cuda.synchronize()
    return S


def _sharpen(w, heads=slice(None), rows=slice(1, None, 2)):
    """Layer 0: queries of these heads and rows 20 times sharper.  The log-sum-exps of a block of 32 rows then lie
    more than 64 log2 units apart, which the cheap form of the max-pooling emit pass does not take."""
    for b in range(w.cfg.batch):
        q, k, v = w.seq[b][0]
        qf = (q.astype(np.uint32) << 16).view(np.float32).copy()
        qf[heads, rows] *= 20
        q = wl.f32_to_bf16_bits(qf)
        w.seq[b][0] = (q, k, v)
        w.q[0][b] = q


def _spread(w, b=0):
    """Distance of the log-sum-exps from the first of their block of 32 rows, [blocks, 32]."""
    q, k, _ = w.seq[b][0]
    logits = np.einsum("hmd,hnd->hmn", orc.widen(q), np.repeat(orc.widen(k), w.cfg.hq // w.cfg.hkv, axis=0)) / np.sqrt(128.0)
    top = logits.max(axis=2, keepdims=True)
    lse2 = ((np.log(np.exp(logits - top).sum(axis=2, keepdims=True)) + top)[..., 0] / np.log(2.0)).reshape(-1, 32)
    return np.abs(lse2 - lse2[:, :1])


def _check(w, got, dust=0.0, **pkw):
    for b in range(w.cfg.batch):
        for l in range(w.cfg.layers):
            ref = orc.score_layer(orc.widen(w.seq[b][l][0]), orc.widen(w.seq[b][l][1]),
                                  agg_task=pkw.get("agg_task", kv.KVC_AGG_MAX),
                                  agg_group=pkw.get("agg_group", kv.KVC_AGG_MEAN),
                                  causal_tail=bool(pkw.get("causal_tail", 0)))
            mine = got[l][:, int(w.cu[b]):int(w.cu[b + 1])]
            big = ref > dust
            np.testing.assert_allclose(mine[big], ref[big], rtol=1e-4, err_msg=f"sequence {b} layer {l}")
            assert np.all(mine[~big] <= 10 * dust)


@pytest.mark.parametrize("pkw", [{}, MEAN, CAUSAL, dict(CAUSAL, **MEAN)])
@pytest.mark.parametrize("n", [700, 8300])          # one chunk of 2048 keys, five
@pytest.mark.parametrize("hq,hkv,window", SHAPES)
def test_forms(hq, hkv, window, n, pkw):
    print(f"[case] {hq}/{hkv} M={window} n={n} {pkw}", flush=True)
    w = _workload(hq, hkv, window, [n])
    _check(w, _scores(w, **pkw), **pkw)


@pytest.mark.parametrize("pkw", [{}, MEAN])
def test_short_row_chunk_in_a_ragged_batch(pkw):
    # 5 + 1 + 1 + 2 stretches of K, 2 heads, 16 layers: 288 slices, more than a group of 256
    print(f"[case] ragged, short row chunk, {pkw}", flush=True)
    w = _workload(10, 2, 64, [8300, 33, 2048, 2049], layers=16)
    _check(w, _scores(w, **pkw), **pkw)


@pytest.mark.parametrize("n", [700, 8300])
@pytest.mark.parametrize("hq,hkv,window", SHAPES)
def test_rows_too_far_apart_for_the_cheap_form(hq, hkv, window, n):
    """In the query-stationary emit pass the exact kernel redoes all workgroups, in the key-stationary one
    every row chunk takes the exact form."""
    print(f"[case] exact form {hq}/{hkv} M={window} n={n}", flush=True)
    w = _workload(hq, hkv, window, [n])
    _sharpen(w)
    assert np.all(_spread(w).max(axis=1) > 64)
    _check(w, _scores(w), dust=1e-30)


@pytest.mark.parametrize("pkw", [{}, CAUSAL, dict(agg_group=kv.KVC_AGG_MAX)])
@pytest.mark.parametrize("hq,hkv,window,n", EMIT_SHAPES)
def test_forms_of_the_emit_pass(hq, hkv, window, n, pkw):
    print(f"[case] emit {hq}/{hkv} M={window} n={n} {pkw}", flush=True)
    w, ran = _workload(hq, hkv, window, [n]), set()
    got = _scores(w, ran, **pkw)
    assert EMIT in ran and EMIT_KEYS not in ran
    _check(w, got, **pkw)


@pytest.mark.parametrize("hq,hkv,window,n", EMIT_SHAPES)
def test_the_exact_form_of_the_emit_pass(hq, hkv, window, n):
    """In the long row chunks and in the short one, all of whose workgroups are on the list."""
    print(f"[case] emit, exact form {hq}/{hkv} M={window} n={n}", flush=True)
    w, ran = _workload(hq, hkv, window, [n]), set()
    _sharpen(w)
    assert np.all(_spread(w).max(axis=1) > 64)
    got = _scores(w, ran)
    assert EMIT in ran and EMIT_KEYS not in ran
    _check(w, got, dust=1e-30)


@pytest.mark.parametrize("lens", [[900, 300], [2000, 1300]])      # up to four chunks, and more
@pytest.mark.parametrize("d", [32, 64, 128, 256])
def test_float32_keeps_what_rounding_takes_from_the_log_sum_exps(d, lens):
    """Queries and keys of small integers: every product and sum of a logit is exact, so what is left is
    the rounding of the log-sum-exps, of the exponent and of the sum.  For probabilities above 1/16 the
    exponent is below 4 in size: half an ulp of it, 1.2e-7, of log2 of a sum below 16, 2.4e-7, and of c2
    times the distance of 4 from the reference, 2.4e-7, times ln 2, and two roundings of 6e-8 in exp2 and
    the sum: 6e-7, hence 1e-6.  A log-sum-exp of 50 nats rounded to float32 alone is up to 2.6e-6 off."""
    print(f"[case] float32 log-sum-exps d={d} {lens}", flush=True)
    layers, heads, window = 3, 16, 4
    rng = np.random.default_rng([d, len(lens), sum(lens)])
    cfg = wl.get_config(1, layers=layers, batch=len(lens), n=max(lens), dtype="f32", head_dim=d, hq=heads, hkv=heads,
                        window=window)
    w = Workload(cfg, seed=1, lens=lens)
    for l in range(layers):
        w.q[l] = rng.integers(-4, 5, size=w.q[l].shape).astype(np.float32)
        w.k[l] = rng.integers(-4, 5, size=w.k[l].shape).astype(np.float32)
    scale = float(np.float32(2.0 / np.sqrt(d)))                  # 4 sigma of a logit: 4 * 6.67 * sqrt(d) * scale = 53 nats
    got = _scores(w, softmax_scale=scale, add_head_mean=0)
    worst = planted = 0.0
    for b in range(len(lens)):
        lo, hi = int(w.cu[b]), int(w.cu[b + 1])
        for l in range(layers):
            t = np.matmul(w.q[l][b].astype(np.float64), w.k[l][:, lo:hi].astype(np.float64).transpose(0, 2, 1)) * scale
            top = t.max(axis=2, keepdims=True)
            lse = np.log(np.exp(t - top).sum(axis=2, keepdims=True)) + top
            ref = np.exp(t - lse).max(axis=1)
            rounded = np.float32(lse / np.log(2.0)).astype(np.float64) * np.log(2.0)
            big = ref > 1.0 / 16
            worst = max(worst, float((np.abs(got[l][:, lo:hi] - ref) / ref)[big].max()))
            planted = max(planted, float((np.abs(np.exp(t - rounded).max(axis=1) - ref) / ref)[big].max()))
    print(f"worst {worst:.2e}, with rounded log-sum-exps {planted:.2e}", flush=True)
    assert planted > 1.5e-6                                      # the test can tell
    assert worst <= 1e-6
