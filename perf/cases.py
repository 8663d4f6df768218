"""The work that users of the compression pass have it do, as cases to be measured.

Two of the public entry points are called here:

* ``kvc_compress``, the whole pass, as a serving engine calls it after a prefill: a bf16
  cache, a window of the last 32..1024 (task) tokens, a retained share of the cache.  Its
  outputs are bit copies of cache rows and whole numbers, so they are compared exactly.
* ``kvc_score``, the stage that dominates it, for everything outside that regime: task
  prompts (whose token count is whatever the task text has), other head sizes, float32
  caches, and engines that reduce scores over GPUs between the stages.  Scores are numbers
  and are compared as numbers: ranks of nearly equal scores, hence the rows the later stages
  copy, are not comparable between two correct implementations.

Head layouts are those of ``workloads/gen.py``; so is the structure of the inputs (attention
sinks, needles, log-normal key norms, a per-layer ramp of the query scale).
"""
import random

import torch

import paper_2509_05165_amd as kv

# (layers, query heads, KV heads) of the repository's workloads
LAYOUTS = ((32, 32, 8), (28, 28, 4), (40, 40, 8), (80, 64, 8))
WINDOWS = (32, 64, 128, 256, 512, 1024)
SINKS, NEEDLES = 4, 64


def _case(entry, layout, batch, n_lo, n_hi, window, **more):
    case = dict(entry=entry, layers=layout[0], hq=layout[1], hkv=layout[2], batch=batch, n_lo=n_lo,
                n_hi=n_hi, lens_seed=1, window=window, head_dim=128, dtype="bf16", keep=20,
                key_sigma=0.0, q_ramp=False, causal_tail=False, by_position=False,
                unstructured=False, value_norm=False, keep_first=0, keep_last=0, min_per_layer=0)
    case.update(more)
    return case


def listed():
    llama, qwen7, qwen14, deep = LAYOUTS
    return [
        # the smallest call: one short prompt, where latency and launches count
        _case("compress", llama, 1, 777, 777, 32, keep=50, name="prompt-777"),
        # one request of the 4096-token regime
        _case("compress", llama, 1, 4096, 4096, 64, keep=50, name="one-4k"),
        # a serving batch of short requests of any length, the 28/4-head layout
        _case("compress", qwen7, 16, 150, 4096, 64, keep=50, name="ragged-16x4k"),
        # a full batch of 4096-token requests, the 40/8-head layout
        _case("compress", qwen14, 32, 4096, 4096, 64, keep=50, name="batch-32x4k"),
        # a mixed batch of medium to long requests with heavy-tailed key norms
        _case("compress", llama, 8, 4096, 32768, 64, keep=20, key_sigma=0.5, name="mixed-8x32k"),
        # one very long context: the headline workload
        _case("compress", llama, 1, 131072, 131072, 64, keep=10, name="one-128k"),
        # a deep model at 64k whose layers attend with different sharpness: the largest case
        _case("compress", deep, 1, 65536, 65536, 128, keep=15, q_ramp=True, name="deep-64k"),
        # task-agnostic window at the end of the context; sinks and recent tokens forced, rows
        # kept in token order for an engine that relies on positions; an odd length
        _case("compress", llama, 1, 30011, 30011, 64, keep=20, causal_tail=True, by_position=True,
              keep_first=4, keep_last=64, min_per_layer=128, name="in-order-30k"),
        # every head keeps its own tokens, scores weighted by the value norms; a large window
        _case("compress", llama, 2, 16384, 16384, 256, keep=25, unstructured=True, value_norm=True,
              name="per-head-2x16k"),
        # a task prompt: its token count is whatever the task's text has
        _case("score", llama, 1, 8192, 8192, 200, name="task-200x8k"),
        # a small model's heads of 64 in a ragged batch
        _case("score", (16, 32, 8), 4, 1000, 6000, 64, head_dim=64, name="d64-4x6k"),
        # a float32 cache (validation runs)
        _case("score", (4, 16, 4), 1, 4096, 4096, 32, head_dim=64, dtype="f32", name="f32-4k"),
    ]


def _log_int(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    if rng.random() < 0.65:
        layout = rng.choice(LAYOUTS)
        window = rng.choice(WINDOWS)
        n_hi = _log_int(rng, 256, 131072)
        batch = _log_int(rng, 1, 32)
        # no more work than the largest listed case: K + V below 21 GB, 1.1e13 flops
        per_token = max(4 * layout[0] * layout[2] * 128 / 21e9,
                        2 * layout[0] * layout[1] * window * 128 / 1.1e13)
        n_hi = max(64, min(n_hi, int(1 / per_token)))
        batch = max(1, min(batch, int(1 / per_token / n_hi)))
        n_lo = n_hi if rng.random() < 0.4 else max(1, int(n_hi * rng.uniform(0.05, 0.9)))
        keep = rng.randint(5, 75)
        return _case("compress", layout, batch, n_lo, n_hi, window, lens_seed=rng.randrange(1 << 20),
                     keep=keep, key_sigma=rng.choice((0.0, 0.0, 0.5)), q_ramp=rng.random() < 0.3,
                     causal_tail=n_lo >= window and rng.random() < 0.3,
                     by_position=rng.random() < 0.3, unstructured=rng.random() < 0.2,
                     value_norm=rng.random() < 0.2, keep_first=rng.choice((0, 0, 0, 4)),
                     keep_last=rng.choice((0, 0, 0, 32)), min_per_layer=rng.choice((0, 0, 0, 16)))
    f32 = rng.random() < 0.3
    layers, hq, hkv = rng.choice(((16, 32, 8), (4, 16, 4), (32, 32, 8), (28, 28, 4), (8, 6, 2)))
    head_dim = rng.choice((32, 64, 128) if f32 else (64, 80, 96, 128, 256))
    window = _log_int(rng, 8, 300)
    n_hi = _log_int(rng, 256, 16384)
    # no more than the listed task prompt asks for (a sixteenth of it in float32)
    most = 2 * 32 * 32 * 200 * 128 * 8192 / (16 if f32 else 1)
    n_hi = max(64, min(n_hi, int(most / (2 * layers * hq * window * head_dim))))
    batch = max(1, min(_log_int(rng, 1, 8), int(most / (2 * layers * hq * window * head_dim * n_hi))))
    n_lo = n_hi if rng.random() < 0.4 else max(1, int(n_hi * rng.uniform(0.05, 0.9)))
    return _case("score", (layers, hq, hkv), batch, n_lo, n_hi, window, lens_seed=rng.randrange(1 << 20),
                 head_dim=head_dim, dtype="f32" if f32 else "bf16",
                 causal_tail=n_lo >= window and rng.random() < 0.2)


def _lens(case):
    rng = random.Random(case["lens_seed"])
    return [rng.randint(case["n_lo"], case["n_hi"]) for _ in range(case["batch"])]


def _rows(case):
    return case["layers"] * (case["hkv"] if case["unstructured"] else 1)


def _budgets(case, lens):
    rows = _rows(case)
    return [max(kv.kvc_budget(case["keep"], rows, n), rows * min(case["min_per_layer"], n)) for n in lens]


def _layer(case, layer, lens, cu, gen, dtype):
    """Queries, keys and values of one layer: normal draws with sinks and needles."""
    d, hq, hkv, window, batch = case["head_dim"], case["hq"], case["hkv"], case["window"], case["batch"]
    group, total = hq // hkv, sum(lens)
    q = torch.randn((batch, hq, window, d), generator=gen, device="cuda")
    if case["q_ramp"]:
        q *= 0.5 + 1.5 * layer / max(case["layers"] - 1, 1)
    k = torch.randn((hkv, total, d), generator=gen, device="cuda", dtype=dtype)
    if case["key_sigma"]:
        k *= torch.exp(case["key_sigma"] * torch.randn((hkv, total, 1), generator=gen, device="cuda")).to(dtype)
    rows = q.view(batch, hkv, group * window, d)
    # sinks: the first tokens lie along the mean direction of the window queries
    mean = rows.mean(dim=2)
    mean = (4.0 * d ** 0.5) * mean / mean.norm(dim=-1, keepdim=True)
    at, seq = [], []
    for b, n in enumerate(lens):
        at += range(cu[b], cu[b] + min(SINKS, n))
        seq += [b] * min(SINKS, n)
    k[:, at] += mean[seq].transpose(0, 1).to(dtype)
    # needles: one key in each of up to 64 stretches is pushed along one of the queries
    at, seq = [], []
    for b, n in enumerate(lens):
        count = max(0, min(NEEDLES, n - SINKS))
        at += [cu[b] + SINKS + j * (n - SINKS) // count for j in range(count)]
        seq += [b] * count
    if at:
        one = torch.randint(group * window, (len(at), hkv), generator=gen, device="cuda")
        needle = rows[torch.tensor(seq, device="cuda")[:, None], torch.arange(hkv, device="cuda"), one]
        needle = 8.0 * needle / needle.norm(dim=-1, keepdim=True)
        k[:, at] += needle.transpose(0, 1).to(dtype)
    v = None
    if case["entry"] == "compress":
        v = torch.randn((hkv, total, d), generator=gen, device="cuda", dtype=dtype)
    return q.to(dtype), k, v


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    dtype = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    lens = _lens(case)
    cu = [0]
    for n in lens:
        cu.append(cu[-1] + n)
    layers = [_layer(case, l, lens, cu, gen, dtype) for l in range(case["layers"])]
    s = {"case": case, "cu": cu, "layers": layers, "q": [x[0].data_ptr() for x in layers],
         "k": [x[1].data_ptr() for x in layers]}
    s["params"] = kv.KvcParams(
        case["batch"], case["layers"], case["hq"], case["hkv"], case["head_dim"], case["window"],
        kv.KVC_BF16 if case["dtype"] == "bf16" else kv.KVC_F32, value_norm=int(case["value_norm"]),
        order=kv.KVC_ORDER_POSITION if case["by_position"] else kv.KVC_ORDER_RANK,
        min_per_layer=case["min_per_layer"], unstructured=int(case["unstructured"]),
        causal_tail=int(case["causal_tail"]), keep_first=case["keep_first"], keep_last=case["keep_last"])
    s["ws_bytes"] = kv.kvc_workspace_size(s["params"], cu[-1], max(lens))
    s["ws"] = torch.empty(s["ws_bytes"], dtype=torch.uint8, device="cuda")
    if case["entry"] == "score":
        s["scores"] = torch.empty((case["layers"], case["hkv"], cu[-1]), dtype=torch.float32, device="cuda")
        return s
    s["v"] = [x[2].data_ptr() for x in layers]
    s["budget"] = _budgets(case, lens)
    heads = 1 if case["unstructured"] else case["hkv"]
    shape = (sum(s["budget"]) * heads, case["head_dim"])
    s["k_out"] = torch.empty(shape, dtype=dtype, device="cuda")
    s["v_out"] = torch.empty(shape, dtype=dtype, device="cuda")
    blocks = case["batch"] * _rows(case)
    s["lengths"] = torch.empty(blocks, dtype=torch.int32, device="cuda")
    s["offsets"] = torch.empty(blocks + 1, dtype=torch.int64, device="cuda")
    return s


def run(s):
    stream = torch.cuda.current_stream().cuda_stream
    if s["case"]["entry"] == "score":
        kv.kvc_score(s["params"], s["q"], s["k"], s["cu"], s["scores"].data_ptr(), s["ws"].data_ptr(),
                     s["ws_bytes"], stream)
        return {"scores": s["scores"]}
    kv.kvc_compress(s["params"], s["q"], s["k"], s["v"], s["cu"], s["budget"], s["k_out"].data_ptr(),
                    s["v_out"].data_ptr(), s["lengths"].data_ptr(), s["offsets"].data_ptr(),
                    s["ws"].data_ptr(), s["ws_bytes"], stream)
    return {"k": s["k_out"], "v": s["v_out"], "lengths": s["lengths"], "offsets": s["offsets"]}


def work(case):
    """One read of Q, of K and of what is needed of V, one write of the outputs; one Q.K^T."""
    lens = _lens(case)
    total, esz = sum(lens), 2 if case["dtype"] == "bf16" else 4
    row = case["head_dim"] * esz
    cache = case["layers"] * case["hkv"] * total * row
    queries = case["layers"] * case["batch"] * case["hq"] * case["window"] * row
    flops = 2 * case["layers"] * case["hq"] * case["window"] * case["head_dim"] * total
    if case["entry"] == "score":
        return {"bytes": cache + queries + 4 * case["layers"] * case["hkv"] * total, "flops": flops}
    retained = sum(_budgets(case, lens)) * (1 if case["unstructured"] else case["hkv"]) * row
    values = cache if case["value_norm"] else retained
    return {"bytes": cache + queries + values + 2 * retained, "flops": flops}


def tolerance(case):
    if case["entry"] == "compress":
        return "exact"
    # fp32 accumulation, then exp(logit - lse) in fp32: 4.2e-7 and 3e-6 off float64 at worst
    # over head sizes 32..256, windows 12..200, both types
    return {"rel": 2e-6, "max": 1.5e-5}


def exact(case, seed):
    """The scores in float64: softmax over the keys of a sequence, the largest probability over
    the task tokens, its mean over the query heads of a group, plus the mean over KV heads.
    What the whole pass returns are copies of cache rows and whole numbers."""
    if case["entry"] == "compress":
        return None
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    dtype = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    lens, window, hkv, d = _lens(case), case["window"], case["hkv"], case["head_dim"]
    cu = [0]
    for n in lens:
        cu.append(cu[-1] + n)
    scores = torch.empty((case["layers"], hkv, cu[-1]), dtype=torch.float64, device="cuda")
    for l in range(case["layers"]):
        q, k, _ = _layer(case, l, lens, cu, gen, dtype)
        for b, n in enumerate(lens):
            if n == 0:
                continue
            for h in range(hkv):
                keys = k[h, cu[b]:cu[b + 1]].double()
                rows = q[b].view(hkv, -1, window, d)[h].double()
                logits = (rows.reshape(-1, d) @ keys.T).view(-1, window, n) / d ** 0.5
                if case["causal_tail"]:
                    seen = torch.arange(n, device="cuda") <= torch.arange(n - window, n, device="cuda")[:, None]
                    logits = logits.masked_fill(~seen, float("-inf"))
                scores[l, h, cu[b]:cu[b + 1]] = torch.softmax(logits, dim=-1).amax(dim=1).mean(dim=0)
        scores[l] += scores[l].mean(dim=0, keepdim=True)
    return {"scores": scores}
