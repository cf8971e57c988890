"""Performance cases of the layer stack: what a serving program has the library do, through the public binding.

A pass is one step as the serving loop makes it (`serve.TraceRunner.step`): the batches are resident, the call runs
them through the layers of the stack on the current CU layout, and the loop waits for the step because the
scheduler decides the next batch from its completion.  A state is a context with its packed weights, its KV pools and
one pair of batches; passes on a state repeat the same step (the K/V it appends land in the same slots).

Shapes, lengths and splits are those of `synth.SHAPES` / `synth.config` and of the trace-driven configuration: Llama-3-8B,
Qwen2.5-14B (with its QKV bias) and Llama-3-70B-shaped layers and the tiny test shape.  Stacks are cut to a few layers:
every layer is the same work, and a few exceed the caches.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2507_06608_amd import binding, synth

DEVICE = "cuda:0"

# A case: shape and number of layers; `chunk_*`: prefill requests, their tokens in all, and the longest cached prefix
# (chunk lengths and prefixes are drawn ragged from the seed unless `even`); `decode_*`: decode requests and the range of their
# contexts; `prefill_cus`: CUs of the prefill share of a partitioned step (0: the step runs on all CUs);
# `handover`: layer from which the prefill phase takes all CUs (0: the split is held).
_NONE = {"chunk_reqs": 0, "chunk_tokens": 0, "prefix_max": 0, "even": False, "decode_reqs": 0, "ctx_min": 0, "ctx_max": 0,
         "prefill_cus": 0, "handover": 0}


def _case(name, shape, layers, **kw):
    return dict({"name": name, "shape": shape, "layers": layers}, **dict(_NONE, **kw))


def listed():
    return [
        # the smallest step: a short chunk next to a handful of decodes of a small model, where launches are the time
        _case("tiny_mixed", "tiny", 1, chunk_reqs=1, chunk_tokens=128, even=True, decode_reqs=8, ctx_min=64, ctx_max=256, prefill_cus=128),
        # one user waiting for one token: every weight read for a single row
        _case("decode_1_8b", "llama3_8b", 8, decode_reqs=1, ctx_min=700, ctx_max=900),
        # a part-filled pool of odd size with the lengths of a chat mix
        _case("decode_23_14b", "qwen25_14b", 4, decode_reqs=23, ctx_min=60, ctx_max=2500),
        # the ordinary decode batch
        _case("decode_64_8b", "llama3_8b", 4, decode_reqs=64, ctx_min=512, ctx_max=4096),
        # a full pool of the trace-driven configuration
        _case("decode_128_14b", "qwen25_14b", 4, decode_reqs=128, ctx_min=200, ctx_max=6000),
        # the heaviest decode batch: long contexts, mostly KV traffic
        _case("decode_256_8b", "llama3_8b", 2, decode_reqs=256, ctx_min=1024, ctx_max=8192),
        # a short prompt (or the tail of a long one): fewer rows than a tile
        _case("prefill_45_8b", "llama3_8b", 4, chunk_reqs=1, chunk_tokens=45, prefix_max=0),
        # the ordinary chunk in the middle of a prompt
        _case("prefill_512_8b", "llama3_8b", 4, chunk_reqs=1, chunk_tokens=512, prefix_max=1536, even=True),
        # a token budget filled by several prompts at once, ragged chunks over ragged prefixes
        _case("prefill_5x_14b", "qwen25_14b", 4, chunk_reqs=5, chunk_tokens=1021, prefix_max=4000),
        # the heaviest prefill batch
        _case("prefill_8192_8b", "llama3_8b", 2, chunk_reqs=4, chunk_tokens=8192, prefix_max=6144),
        # both phases of the ordinary batch side by side on disjoint CU shares
        _case("mixed_8b", "llama3_8b", 4, chunk_reqs=1, chunk_tokens=512, prefix_max=1536, even=True, decode_reqs=64, ctx_min=512, ctx_max=4096, prefill_cus=192),
        # the large model: a chunk and a decode batch on their shares, the decode share handed over once decoding is done
        _case("mixed_70b", "llama3_70b", 4, chunk_reqs=1, chunk_tokens=2048, prefix_max=2048, even=True, decode_reqs=64, ctx_min=1024, ctx_max=4096,
              prefill_cus=160, handover=1),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """Any of the three kinds of step on any of the shapes: 1 to 256 decode requests with contexts up to 8192, chunks of 1 to 8192 tokens
    from 1 to 8 requests over prefixes up to 6144, every split in steps of 32 CUs."""
    limit = [max(work(c)[k] for c in listed()) for k in ("flops", "bytes")]
    while True:
        c = {"shape": rng.choice(["tiny", "llama3_8b", "llama3_8b", "qwen25_14b", "llama3_70b"]), "layers": rng.randint(1, 4), **_NONE}
        kind = rng.choice(["decode", "prefill", "mixed"])
        if kind != "decode":
            c["chunk_reqs"] = rng.choice([1, 1, 2, 3, 4, 5, 8])
            c["chunk_tokens"] = c["chunk_reqs"] * 2 + _log_int(rng, 4, 8192 - 16)
            c["prefix_max"] = rng.choice([0, _log_int(rng, 16, 6144)])
        if kind != "prefill":
            c["decode_reqs"] = _log_int(rng, 1, 256)
            c["ctx_min"] = _log_int(rng, 16, 2048)
            c["ctx_max"] = _log_int(rng, c["ctx_min"] + 1, 8192)
        if kind == "mixed":
            c["prefill_cus"] = 32 * rng.randint(1, 7)
            c["handover"] = rng.randint(0, c["layers"] - 1)
        w, slower = work(c), 256 / min(c["prefill_cus"], 256 - c["prefill_cus"]) if c["prefill_cus"] else 1  # a small share takes longer
        if slower * w["flops"] <= limit[0] and slower * w["bytes"] <= limit[1]:
            return c


def _lengths(case, seed):
    """(chunk lengths, prefix lengths, decode contexts) of a case."""
    rng = np.random.default_rng([seed, 31])
    n, total = case["chunk_reqs"], case["chunk_tokens"]
    if case["even"]:
        chunks, prefixes = [total // n] * n, [case["prefix_max"]] * n
        chunks[-1] += total - sum(chunks)
    elif n:
        share = rng.uniform(0.3, 1.7, n)
        chunks = [max(1, int(total * s / share.sum())) for s in share]
        chunks[int(np.argmax(chunks))] += total - sum(chunks)
        prefixes = rng.integers(0, case["prefix_max"] + 1, n).tolist()
    else:
        chunks, prefixes = [], []
    ctx = rng.integers(case["ctx_min"], case["ctx_max"] + 1, case["decode_reqs"]).tolist()
    return chunks, prefixes, ctx


def _pages(tokens):
    return -(-tokens // synth.PAGE_SIZE)


def _pool_pages(case):
    """Pages of the pool: enough for the longest lengths of the case, whatever the seed draws (a server's pool has a fixed size)."""
    n = case["chunk_reqs"]
    return n * (_pages(case["prefix_max"]) + 1) + _pages(case["chunk_tokens"]) + n + case["decode_reqs"] * _pages(case["ctx_max"] + 1)


def _layer_weights(shape, seed, layer):
    """One layer's bf16 weights (the values of `synth.make_weights`: N(0, std), gains around 1), drawn on the GPU."""
    g = torch.Generator(device=DEVICE)
    g.manual_seed(seed * 1009 + layer)
    std = synth.weight_std(shape)

    def mat(r, c):
        return torch.randn((r, c), generator=g, device=DEVICE, dtype=torch.bfloat16).mul_(std)

    def gain():
        return (1.0 + torch.randn(shape.hidden, generator=g, device=DEVICE) * 0.02).to(torch.bfloat16)

    w = {"attn_norm_g": gain(), "w_qkv": mat(shape.n_qkv, shape.hidden), "w_o": mat(shape.hidden, shape.q_dim), "ffn_norm_g": gain(),
         "w_gate_up": mat(2 * shape.ffn, shape.hidden), "w_down": mat(shape.hidden, shape.ffn)}
    if shape.name == "qwen25_14b":
        w["b_qkv"] = (torch.randn(shape.n_qkv, generator=g, device=DEVICE) * 0.5).to(torch.bfloat16)
    return w


def _workload(case, seed):
    chunks, prefixes, ctx = _lengths(case, seed)
    used = sum(_pages(p + n) for n, p in zip(chunks, prefixes)) + sum(_pages(c + 1) for c in ctx)
    return synth.make_workload("case", synth.SHAPES[case["shape"]], seed, chunk_lens=chunks, prefix_lens=prefixes, decode_ctx=ctx,
                               kv_device=DEVICE, page_slack=_pool_pages(case) - used)


def prepare(case, seed):
    shape, layers = synth.SHAPES[case["shape"]], case["layers"]
    wl = _workload(case, seed)
    nx = binding.context_for(wl, n_layers=layers)
    for layer in range(layers):
        nx.load_layer(layer, _layer_weights(shape, seed, layer))
    state = {"nx": nx, "kv": nx.make_kv(wl.k_pool, wl.v_pool, layers=layers), "layers": (0, layers), "handover": case["handover"],
             "prefill": binding.DevPrefill(wl.prefill, nx.device) if wl.prefill else None,
             "decode": binding.DevDecode(wl.decode, nx.device) if wl.decode else None}
    if case["prefill_cus"]:
        nx.set_cu_split(case["prefill_cus"], nx.cu_count - case["prefill_cus"])
    return state


def run(state):
    nx, kv, layers, pb, db = state["nx"], state["kv"], state["layers"], state["prefill"], state["decode"]
    if pb is not None and db is not None:
        if state["handover"]:
            nx.mixed_step_handover(pb, db, kv, state["handover"], layers=layers)
        else:
            nx.mixed_step(pb, db, kv, layers=layers)
    elif pb is not None:
        nx.prefill_chunk(pb, kv, layers=layers)
    else:
        nx.decode_step(db, kv, layers=layers)
    nx.sync()  # the loop waits for every step: its completion decides the next batch
    return {"prefill": pb.y if pb is not None else None, "decode": db.y if db is not None else None, "k": kv.pools[0], "v": kv.pools[1]}


def work(case):
    """Per phase: the weights once, the batch's input and output rows, the cached K/V of its requests once and the appended K/V;
    flops of the projections and of attention over the visible (query, key) pairs."""
    s, layers = synth.SHAPES[case["shape"]], case["layers"]
    mean_share = 1.0 if case["even"] else 0.5
    kv_row = 2.0 * 2 * s.kv_dim
    flops = moved = 0.0
    if case["chunk_reqs"]:
        n, t = case["chunk_reqs"], case["chunk_tokens"]
        prefix = mean_share * case["prefix_max"]
        pairs = t * (prefix + (t / n + 1) / 2)
        flops += layers * (2.0 * t * s.params_per_layer + 4.0 * s.q_dim * pairs)
        moved += layers * (2.0 * s.params_per_layer + kv_row * (n * prefix + t)) + 2.0 * 2 * t * s.hidden
    if case["decode_reqs"]:
        b = case["decode_reqs"]
        keys = b * (0.5 * (case["ctx_min"] + case["ctx_max"]) + 1)
        flops += layers * (2.0 * b * s.params_per_layer + 4.0 * s.q_dim * keys)
        moved += layers * (2.0 * s.params_per_layer + kv_row * keys) + 2.0 * 2 * b * s.hidden
    return {"bytes": moved, "flops": flops}


def tolerance(case):
    # Against the same stack in fp64 (nothing rounded but weights, inputs and cached K/V) the outputs are off by 1.7e-3 after one tiny layer,
    # which is the bf16 rounding of the output itself, and by 4.3e-3 to 6.9e-3 after 4 to 8 wide layers (bf16 K/V, queries and layer outputs,
    # carried on by every layer behind them); the worst element by 0.032 of the result's rms.  With the attention's sums in another order,
    # everything else the same, the outputs move by 2.2e-3 (2 layers) to 8.2e-3 (8 layers, one row).
    return {"rel": 1e-2 if case["layers"] <= 2 else 2e-2, "max": 0.12}
