"""The work that programs have this library do, as cases that can be timed and compared.

A serving loop calls two things per micro-batch: the layers of a pipeline stage (`Stage.forward`, in the first stage
behind `gllm_op_embedding`) and, in the last stage, the next token of the rows that receive one (`Head.logits`, then
`gllm_op_sample`).  Shapes are the stage shapes of `synth.SHAPES` (fewer layers of the large ones: a layer is the unit
that repeats) and the two vocabularies of the tests; batches are the ones of the benchmarks, and sizes between and
beside them.

A case of kind "stage":
  shape, layers, bias      stage shape, number of layers, QKV bias (Qwen-shaped models carry one)
  embed                    first stage of a pipeline: token ids go through the embedding table first
  f32                      last stage of a pipeline: the fp32 residual stream is returned too (the head reads it)
  prefill, chunks, prefix  new prompt tokens, in `chunks` near-equal chunks; chunk i continues a prompt of which
                           prefix*i/(chunks-1) tokens are cached already (one chunk: prefix)
  decodes, lo, hi, log     decode rows, their cached lengths spread over [lo, hi] (log: evenly in the logarithm)
A case of kind "head":
  hidden, vocab, rows      final norm + projection of `rows` rows, then one sampled token each
  sampling                 greedy | top_k (50, with nucleus 0.95) | nucleus (0.95, no top-k) | mixed (of all three)
"""
import dataclasses
import math
import random

import torch

from paper_2504_14775_amd import binding, head, synth

DEV = "cuda:0"
VOCABS = (128256, 152064)      # of the Llama-3- and Qwen2.5-shaped models
EMBED_VOCAB = VOCABS[0]


def _stage(name, shape, layers, prefill, chunks, prefix, decodes, lo, hi, log=False, bias=False, embed=False, f32=False):
    return dict(name=name, kind="stage", shape=shape, layers=layers, bias=bias, embed=embed, f32=f32, prefill=prefill,
                chunks=chunks, prefix=prefix, decodes=decodes, lo=lo, hi=hi, log=log)


def _head(name, hidden, vocab, rows, sampling):
    return dict(name=name, kind="head", hidden=hidden, vocab=vocab, rows=rows, sampling=sampling)


def listed():
    return [
        # the smallest call: the one-layer test configuration (head size 64, intermediate size not a tile multiple),
        # two chunks and four decode rows; all launches and host work
        _stage("tiny_hybrid_52", "tiny", 1, 48, 2, 48, 4, 17, 64, f32=True),
        # one user at the keyboard: a single decode row through the 8B-shaped stage, a stream of its weights
        _stage("8b_decode_1", "llama3_8b_pp4", 8, 0, 0, 0, 1, 2500, 2500),
        # a new, short prompt alone (time to first token): no cache, an odd number of rows
        _stage("8b_prompt_197", "llama3_8b_pp4", 8, 197, 1, 0, 0, 0, 0, embed=True),
        # the decode-only micro-batch that throttling leaves when few requests are decoding
        _stage("8b_decode_64", "llama3_8b_pp4", 8, 0, 0, 0, 64, 1500, 3500),
        # the mean micro-batch of closed-loop chat serving: 251 decode rows at chat lengths, ends of two prompts
        _stage("8b_serving_322", "llama3_8b_pp4", 8, 71, 2, 300, 251, 64, 1100, log=True, f32=True),
        # the benchmark's batch: the full token budget, one long chunk over a cached prefix plus 256 decode rows
        _stage("8b_hybrid_2048", "llama3_8b_pp4", 8, 1792, 1, 1013, 256, 512, 4096, embed=True),
        # many long-running conversations: decode only, 14B shape, QKV bias
        _stage("14b_decode_512", "qwen25_14b_pp4", 3, 0, 0, 0, 512, 1024, 8192, log=True, bias=True),
        # prompts arriving together: four chunks over cached prefixes, a few decode rows beside them
        _stage("32b_prefill_4160", "qwen25_32b_pp4", 2, 4096, 4, 6144, 64, 256, 4096, bias=True),
        # the smallest batch of the 70B-shaped series: decode rows with a short chunk
        _stage("70b_hybrid_773", "llama3_70b_pp4", 2, 318, 1, 145, 455, 512, 8192),
        # last stage of the benchmark's batch: 256 decode rows and the row that ends the chunk
        _head("head_8b_257_top_k", 4096, VOCABS[0], 257, "top_k"),
        # last stage of a decode-only micro-batch, nucleus sampling without top-k
        _head("head_14b_64_nucleus", 5120, VOCABS[1], 64, "nucleus"),
        # one user at the keyboard, greedy
        _head("head_8b_1_greedy", 4096, VOCABS[0], 1, "greedy"),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _cost(case):
    w = work(case)
    return w["bytes"] / 5e12 + w["flops"] / 1e15


def draw(rng):
    """One more case of the same ranges, no costlier than the costliest listed one."""
    most = max(_cost(c) for c in listed())
    while True:
        if rng.random() < 0.25:
            c = _head("", rng.choice((4096, 5120, 8192)), rng.choice(VOCABS), _log_int(rng, 1, 512),
                      rng.choice(("greedy", "top_k", "nucleus", "mixed")))
        else:
            shape = rng.choice(("tiny", "llama3_8b_pp4", "llama3_8b_pp4", "llama3_8b_pp4", "qwen25_14b_pp4", "qwen25_32b_pp4",
                                "llama3_70b_pp4"))
            layers = rng.randint(1, {"tiny": 4, "llama3_8b_pp4": 8}.get(shape, 3))
            work_kind = rng.choice(("prefill", "decode", "both", "both"))
            prefill = _log_int(rng, 8, 4096) if work_kind != "decode" else 0
            chunks = rng.randint(1, min(4, prefill // 4)) if prefill else 0
            decodes = _log_int(rng, 1, 512) if work_kind != "prefill" else 0
            hi = _log_int(rng, 64, 8192) if decodes else 0
            c = _stage("", shape, layers, prefill, chunks, rng.choice((0, rng.randint(0, 6144))) if prefill else 0, decodes,
                       max(1, int(hi * rng.uniform(0.1, 1.0))) if decodes else 0, hi, log=rng.random() < 0.5,
                       bias=shape.startswith("qwen") and rng.random() < 0.7, embed=rng.random() < 0.25, f32=rng.random() < 0.25)
        del c["name"]
        if _cost(c) <= most:
            return c


def _shape(case):
    return dataclasses.replace(synth.SHAPES[case["shape"]], num_layers=case["layers"], has_qkv_bias=case["bias"])


def _sequences(case):
    """[(new tokens, cached tokens)] of a stage case: chunks first, then the decode rows, in no particular order of length."""
    n, c = case["prefill"], case["chunks"]
    seqs = [(n // c + (i < n % c), case["prefix"] if c == 1 else case["prefix"] * i // (c - 1)) for i in range(c)]
    d, lo, hi = case["decodes"], case["lo"], case["hi"]
    at = [(i + 0.5) / d for i in range(d)]
    lens = [int(lo * (hi / lo) ** f) if case["log"] else int(lo + (hi - lo) * f) for f in at]
    random.Random(d * 8209 + hi).shuffle(lens)
    return seqs + [(1, k) for k in lens]


def _layer(shape, gen):
    w = {}
    for name, size in synth.weight_shapes(shape).items():
        mean, std = (1.0, 0.1) if name.startswith("norm") else (0.0, 0.02)
        w[name] = torch.empty(size, dtype=torch.bfloat16, device=DEV).normal_(mean, std, generator=gen)
    return w


def _prepare_stage(case, seed):
    shape, seqs = _shape(case), _sequences(case)
    gen = torch.Generator(device=DEV).manual_seed(seed)
    batch = synth.build_batch(seqs, seed, spare_blocks=64)
    # the pages that receive new tokens were handed out from one end of the pool, so that run() can return them as a
    # view (in an order of their own: batches name pages in any order)
    tables, first_new = batch.block_tables, batch.cached_len // synth.PAGE
    last_new = (batch.cached_len + batch.new_tokens - 1) // synth.PAGE
    written = [int(p) for s in range(batch.num_seqs) for p in tables[s, first_new[s]:last_new[s] + 1]]
    low, high = sorted(set(range(len(written))) - set(written)), [p for p in written if p >= len(written)]
    swap = dict(zip(low + high, high + low))
    for s in range(batch.num_seqs):
        row = tables[s]
        for i in range(int(last_new[s]) + 1):
            row[i] = swap.get(int(row[i]), row[i])
    stage = binding.stage_for_batches(shape, [batch], device=DEV)
    for l in range(shape.num_layers):
        stage.load_layer(l, _layer(shape, gen))
    per_page = shape.n_kv_heads * synth.PAGE * shape.head_dim
    k_pool, v_pool = (torch.empty(shape.num_layers, batch.num_blocks, per_page, dtype=torch.bfloat16, device=DEV)
                      .normal_(0.0, synth.kv_sigma(shape), generator=gen) for _ in range(2))
    stage.bind_kv_pool(k_pool, v_pool, batch.num_blocks)
    T, H = batch.num_tokens, shape.hidden
    st = dict(kind="stage", stage=stage, batch=batch, k=k_pool[:, :len(written)], v=v_pool[:, :len(written)], ids=None,
              x=torch.empty(T, H, dtype=torch.bfloat16, device=DEV).normal_(generator=gen),
              out=torch.empty(T, H, dtype=torch.bfloat16, device=DEV),
              out32=torch.empty(T, H, dtype=torch.float32, device=DEV) if case["f32"] else None)
    if case["embed"]:
        st["table"] = torch.empty(EMBED_VOCAB, H, dtype=torch.bfloat16, device=DEV).normal_(generator=gen)
        st["ids"] = torch.randint(0, EMBED_VOCAB, (T,), dtype=torch.int32, device=DEV, generator=gen)
    return st


def _prepare_head(case, seed):
    gen = torch.Generator(device=DEV).manual_seed(seed)
    H, V, M = case["hidden"], case["vocab"], case["rows"]
    # a final norm's gain of about 3 gives logits with a standard deviation of 4 to 5: a few to a few thousand tokens
    # share nearly all of the probability, as for a trained model
    gain = torch.empty(H, dtype=torch.bfloat16, device=DEV).normal_(3.0, 0.3, generator=gen)
    w = torch.empty(V, H, dtype=torch.bfloat16, device=DEV).normal_(0.0, 0.02, generator=gen)
    h = head.Head(H, V, M, 1e-6, device=DEV)
    h.load(gain, w)
    T = 2 * M                                                     # every other row of the batch receives a token
    x = torch.empty(T, H, device=DEV).normal_(0.0, 4.0, generator=gen)
    r = random.Random(seed)
    kinds = [case["sampling"] if case["sampling"] != "mixed" else r.choice(("greedy", "top_k", "nucleus")) for _ in range(M)]
    temp = [0.0 if k == "greedy" else r.choice((0.7, 0.8, 1.0)) for k in kinds]
    return dict(kind="head", head=h, vocab=V, x=x, rows=torch.arange(1, T, 2, dtype=torch.int32, device=DEV),
                logits=torch.empty(M, h.padded_vocab, device=DEV), ids=torch.empty(M, dtype=torch.int32, device=DEV),
                temp=torch.tensor(temp, device=DEV), top_k=torch.tensor([50 if k == "top_k" else 0 for k in kinds], dtype=torch.int32, device=DEV),
                top_p=torch.tensor([1.0 if k == "greedy" else 0.95 for k in kinds], device=DEV),
                u=torch.rand(M, device=DEV, generator=gen))


def prepare(case, seed):
    return (_prepare_stage if case["kind"] == "stage" else _prepare_head)(case, seed)


def run(s):
    if s["kind"] == "head":
        s["head"].logits(s["x"], s["rows"], s["logits"])
        head.gllm_op_sample(s["logits"], s["vocab"], s["temp"], s["top_k"], s["top_p"], s["u"], s["ids"])
        return [s["logits"], s["ids"]]
    if s["ids"] is not None:
        head.gllm_op_embedding(s["ids"], s["table"], s["x"])
    b = s["batch"]
    s["stage"].forward(b.new_tokens, b.cached_len, b.block_tables, s["x"], s["out"], s["out32"])
    return [s["out"], s["out32"], s["k"], s["v"]]


def work(case):
    if case["kind"] == "head":
        H, V, M = case["hidden"], case["vocab"], case["rows"]
        return {"bytes": 2 * V * H + 4 * M * H + 4 * M * V, "flops": 2 * M * V * H}
    shape, seqs = _shape(case), _sequences(case)
    T = sum(n for n, _ in seqs)
    H, L = shape.hidden, shape.num_layers
    keys = sum(n + c for n, c in seqs)                                 # each read or written once per layer
    pairs = sum(n * c + n * (n + 1) // 2 for n, c in seqs)
    moved = T * H * (2 + 2 + (4 if case["f32"] else 0) + (2 if case["embed"] else 0))
    return {"bytes": moved + L * (2 * shape.weight_elems_per_layer + keys * shape.kv_bytes_per_token_layer),
            "flops": L * (T * shape.gemm_flop_per_token_layer + 4 * shape.q_dim * pairs)}


def tolerance(case):
    """About four times what the same path differs by from itself with its sums in another order (other partitions of the
    keys, other rows beside a row and so other tiles and k-shares): bf16 roundings fall the other way."""
    if case["kind"] == "head":
        # measured 1.2e-5 and 7e-4 (normalised rows one ulp of the reciprocal root apart); no token moved, but a draw within
        # rounding of the boundary between two tokens may go to either
        return {"rel": 1e-4, "max": 4e-3, "differ": 0.005}
    # measured 4.9e-3 (2 layers), 5.8e-3 (3), 8.9e-3 (8); largest single difference 0.045
    return {"rel": min(0.03, 0.014 * math.sqrt(case["layers"])), "max": 0.2}
