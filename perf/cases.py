"""Timed work of the generation library: what an RLHF step asks of one GPU, at the sizes this repository is configured for.

A case is one pass of a user's program over a model of a known width and reduced depth (the widths set the kernels' shapes, the
depth only repeats them):

  mode "generate"   a generation phase: optionally the weight copies are re-laid (the weights were just trained), the prompts are
                    prefilled, then every decode step feeds one token per sequence.  The tokens that are fed are given (the loop of
                    reference-token scoring): free-running feedback would turn one near-tie between two logits into a different
                    text, while the work of a step does not depend on the values it is fed.
  mode "logprobs"   the Actor / Reference inference call: the log-probability of every following token
  mode "values"     the Critic / Reward inference call: a scalar per position

The program keeps its generator (weights, arenas, copies) and its buffers from pass to pass, as a training loop does.
"""
from __future__ import annotations

import math
from dataclasses import dataclass

import torch

from paper_2406_14088_amd import Generator, kv_block_scaled, precision_level


@dataclass(frozen=True)
class Shape:
    n_layers: int
    hidden: int
    n_heads: int
    n_kv_heads: int
    head_dim: int
    ffn: int
    vocab: int
    rope_base: float = 10000.0
    rms_eps: float = 1e-5
    rope_style: int = 1


# widths of the configured workloads (layers come from the case)
MODELS = {
    "tiny": (256, 4, 4, 64, 688, 1024),
    "llama7b": (4096, 32, 32, 128, 11008, 32000),
    "llama13b": (5120, 40, 40, 128, 13824, 32000),
    "llama70b": (8192, 64, 8, 128, 28672, 32000),
    "llama3_7b": (4096, 32, 8, 128, 14336, 128256),
    "llama3_34b": (8192, 64, 8, 128, 22016, 128256),
}
LAYER_TENSORS = ("attn_norm", "wq", "wk", "wv", "wo", "ffn_norm", "w_gate", "w_up", "w_down")


def shape_of(case):
    return Shape(case["layers"], *MODELS[case["model"]])


def _case(name, model, layers, batch, prompt, gen, mode="generate", repack=False, packed=True, page=0, ragged=False, fp32=False):
    c = dict(model=model, layers=layers, batch=batch, prompt=prompt, gen=gen, mode=mode, repack=repack, packed=packed, page=page,
             ragged=ragged, fp32=fp32)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest configuration as a whole generation phase, fp32 master weights: launches and host time are what counts
        _case("tiny_phase", "tiny", 2, 4, 16, 16, repack=True, fp32=True),
        # one sequence through a full-depth 7B model: latency of a prompt and of single tokens (an evaluation or chat use)
        _case("single_7b", "llama7b", 32, 1, 128, 32),
        # the headline workload of this repository, batch 128, prompt 128, 256 tokens, with the re-layout that opens a phase
        _case("phase_7b", "llama7b", 4, 128, 128, 256, repack=True),
        # its prefill alone (first token of 128 prompts)
        _case("prefill_7b", "llama7b", 8, 128, 128, 1),
        # long contexts: prompts of 2048 tokens, cached rows from 2048 on
        _case("long_7b", "llama7b", 2, 32, 2048, 64),
        # the widest batch: 256 sequences of the 13B width (every projection takes two activation terms)
        _case("batch_13b", "llama13b", 2, 256, 256, 32),
        # grouped-query attention, 64/8 heads, the widest model
        _case("gqa_70b", "llama70b", 2, 64, 128, 128),
        # grouped-query attention, 32/8 heads, vocabulary 128256, prompt 1024
        _case("gqa_llama3", "llama3_7b", 2, 64, 1024, 32),
        # prompts of different lengths on a paged cache, a batch that fills no tile
        _case("ragged_paged", "llama7b", 4, 37, 205, 96, page=16, ragged=True),
        # no memory left for weight copies: every projection from the row-major weights, a small batch
        _case("rowmajor_7b", "llama7b", 4, 16, 64, 32, packed=False),
        # scoring finished sequences of the headline workload (prompt + response) with the Actor or the Reference model
        _case("logprobs_7b", "llama7b", 4, 32, 384, 0, mode="logprobs"),
        # scoring with the Critic or the Reward model, odd sizes
        _case("values_13b", "llama13b", 2, 24, 333, 0, mode="values"),
    ]


def _rough_seconds(case):
    w = work(case)
    return w["flops"] / 6e14 + w["bytes"] / 4e12 + case["gen"] * case["layers"] * 5e-5


def draw(rng):
    """One more case: sizes over their logarithms, options as often as they are used."""
    most = max(_rough_seconds(c) for c in listed())

    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    while True:
        model = rng.choice(["tiny", "llama7b", "llama7b", "llama7b", "llama13b", "llama70b", "llama3_7b", "llama3_34b"])
        mode = rng.choice(["generate"] * 6 + ["logprobs", "values"])
        batch, prompt = log_int(1, 256), log_int(2, 2048)
        layers = rng.randint(1, 8 if model == "llama7b" else 2)
        packed = rng.random() < 0.85
        if mode == "generate":
            ragged = rng.random() < 0.25
            page = rng.choice([16, 64, 128]) if rng.random() < 0.25 else 0
            case = _case(None, model, layers, batch, prompt, log_int(1, 256), repack=packed and rng.random() < 0.3, packed=packed,
                         page=page, ragged=ragged, fp32=model == "tiny")
        else:
            case = _case(None, model, layers, batch, prompt, 0, mode=mode, packed=packed, fp32=model == "tiny")
        if batch * prompt <= 131072 and 1e-3 < _rough_seconds(case) <= most:
            return case


def _weights(shape, g, dtype, dev):
    d, qd, kvd = shape.hidden, shape.n_heads * shape.head_dim, shape.n_kv_heads * shape.head_dim
    sizes = {"wq": (qd, d), "wk": (kvd, d), "wv": (kvd, d), "wo": (d, qd), "w_gate": (shape.ffn, d), "w_up": (shape.ffn, d),
             "w_down": (d, shape.ffn)}

    def matrix(size):
        return (torch.randn(size, generator=g, device=dev) * 0.02).to(torch.bfloat16).to(dtype)

    out = {"tok_emb": matrix((shape.vocab, d)), "lm_head": matrix((shape.vocab, d)), "final_norm": torch.ones(d, dtype=dtype, device=dev)}
    for name in LAYER_TENSORS:
        out[name] = [matrix(sizes[name]) if name in sizes else torch.ones(d, dtype=dtype, device=dev) for _ in range(shape.n_layers)]
    return out


def prepare(case, seed):
    """The generator over weights drawn from the seed, the prompts, the tokens to feed and the program's own buffers."""
    dev = "cuda:0"
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    shape = shape_of(case)
    B, P, G = case["batch"], case["prompt"], case["gen"]
    max_seq = P + max(G, 1)
    weights = _weights(shape, g, torch.float32 if case["fp32"] else torch.bfloat16, dev)
    pages = -(-max_seq // case["page"]) if case["page"] else 0
    gen = Generator(shape, weights, B, max_seq, packed=case["packed"], page_size=case["page"], n_pages=B * pages)
    if case["page"]:
        # pages handed out in a scattered order, as a pool looks after sequences came and went
        order = torch.randperm(B * pages, generator=torch.Generator().manual_seed(seed)).tolist()
        gen.set_block_table([order[b * pages:(b + 1) * pages] for b in range(B)], [max_seq] * B)
    tokens = torch.randint(0, shape.vocab, (B, P), generator=g, device=dev, dtype=torch.int32)
    state = {"case": case, "gen": gen, "tokens": tokens}
    if case["mode"] == "values":
        state["head"] = (torch.randn(shape.hidden, generator=g, device=dev) * 0.02).to(torch.float32 if case["fp32"] else torch.bfloat16)
    if case["mode"] == "generate":
        if case["ragged"]:
            state["lens"] = torch.randint((P + 1) // 2, P + 1, (B,), generator=g, device=dev, dtype=torch.int32)
        state["feed"] = torch.randint(0, shape.vocab, (B, max(G - 1, 1)), generator=g, device=dev, dtype=torch.int32)
        state["cur"] = torch.empty(B, dtype=torch.int32, device=dev)
        state["next"] = torch.empty(B, dtype=torch.int32, device=dev)
        state["logits"] = torch.empty((B, shape.vocab), dtype=torch.float32, device=dev)
    return state


def run(state):
    case, gen, tokens = state["case"], state["gen"], state["tokens"]
    if case["mode"] == "logprobs":
        return gen.logprobs(tokens)
    if case["mode"] == "values":
        return gen.values(tokens, state["head"])
    B, G = case["batch"], case["gen"]
    if case["repack"]:
        gen.pack_weights()
    few = B * G < 512
    out = torch.empty((B, G), dtype=torch.int32, device=tokens.device)
    every = torch.empty((B, G, gen.shape.vocab), dtype=torch.float32, device=tokens.device) if few else None
    if case["ragged"]:
        first, nxt = gen.prefill_ragged(tokens, state["lens"])
    else:
        first, nxt = gen.prefill(tokens)
    out[:, 0].copy_(nxt)
    if few:
        every[:, 0].copy_(first)
    cur, nxt, feed = state["cur"], state["next"], state["feed"]
    for i in range(G - 1):
        cur.copy_(feed[:, i])
        want = few or i == G - 2
        gen.decode_step(cur, logits=state["logits"] if want else None, next_tokens=nxt, want_logits=want)
        out[:, i + 1].copy_(nxt)
        if few:
            every[:, i + 1].copy_(state["logits"])
    # many tokens: all of them, and the logits of both ends; few: the logits of every position (one near-tie is already a large
    # share of few tokens)
    if few:
        return {"logits": every}
    return {"tokens": out, "prefill_logits": first, "last_logits": state["logits"]} if G > 1 else {"tokens": out, "prefill_logits": first}


def work(case):
    """Weights once per prefill and once per decode step, cache rows as stored, one multiply-add per weight and row."""
    s = shape_of(case)
    B, P, G = case["batch"], case["prompt"], case["gen"]
    qd, kvd, d = s.n_heads * s.head_dim, s.n_kv_heads * s.head_dim, s.hidden
    layer = (qd + 2 * kvd) * d + qd * d + 3 * d * s.ffn
    row = 2 * s.n_layers * s.n_kv_heads * (2 * s.head_dim + (4 if kv_block_scaled(s) else 0))
    head_rows = {"generate": B, "logprobs": B * P, "values": 0}[case["mode"]]
    weights = 2 * (s.n_layers * layer + (s.vocab * d if head_rows else 0))
    attention = 4 * s.n_layers * s.n_heads * s.head_dim
    flops = 2 * B * P * s.n_layers * layer + 2 * head_rows * s.vocab * d + attention * B * P * (P + 1) // 2
    nbytes = weights + B * P * (row + 4 + 2 * d) + (B * s.vocab * 4 if case["mode"] == "generate" else B * P * 4)
    if case["repack"]:
        nbytes += 2 * weights
    for i in range(G - 1):
        cached = P + i + 1
        nbytes += weights + B * (cached + 1) * row + B * 2 * d
        flops += 2 * B * (s.n_layers * layer + s.vocab * d) + attention * B * cached
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Four times what the two weight layouts (the same products, summed in another order) differ by on one MI355X.  Rounding flips of
    half values grow with the root of the depth where activations are one half term (levels 1 and 2: 7B width, 4 layers 7.1e-4,
    32 layers 2.3e-3 of the logits; largest difference 5 times that), and are absent where every activation has two terms (level 3:
    2.1e-5 at 2 layers).  Log-probabilities are near -ln(vocab), ten times the deviation of a logit."""
    per_layer = 6e-5 if precision_level(shape_of(case)) >= 3 else 1.6e-3
    rel = per_layer * math.sqrt(max(case["layers"], 1)) * (0.1 if case["mode"] == "logprobs" else 1.0)
    return {"rel": rel, "max": 6 * rel, "differ": 0.008}
