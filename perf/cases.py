"""The work whose time is tracked: whole requests through the public entry points, from a batch of prompts to its tokens.

One pass is `prefill` on a batch of prompts followed by the decode steps (`generate`, then one `step` that also returns the
logits and hidden states) or by rounds of standard speculative decoding (`sd_generate`).  The model shapes, batches,
prompt lengths and verifier sizes are those of `workloads.config` / `workloads.mini_config`.

The weights stand for a trained triple.  Random-init models sample nearly uniformly, so that a rounding difference anywhere
changes tokens and with them everything later; trained models are confident, and so are these: a LLaMA-shaped model
continues token v with `nxt[v]`, a GPT-shaped one continues position p with `word[p]`, both by a margin of many nats over the
rest of the vocabulary (the layers add their contribution to the residual stream on top).  The target agrees with the draft on
four tokens of five.  Every `1 / reject`-th token (or position) carries a direction that the verifier reads, so the rejected
share is the case's and no score lies near the threshold.  The arithmetic and the memory traffic are those of any weights.
"""
import math

import numpy as np
import torch

import workloads as W
from paper_2502_04557_amd import binding

AGREE = 0.8          # share of the tokens on which the target continues as the draft does
PEAK = 64.0          # logit of the continuation when nothing else is in the residual stream
MARK = 10.0          # length of the verifier's direction in a marked embedding, against 1 per other direction


def _case(name, pair, batch, prompt_min, prompt_max, n_gen, reject, full_prefix=False, correction=False, gamma=0):
    return dict(name=name, pair=pair, batch=batch, prompt_min=prompt_min, prompt_max=prompt_max, n_gen=n_gen, reject=reject,
                full_prefix=full_prefix, correction=correction, gamma=gamma)


def listed():
    return [
        # the float32 mode: one row of the smallest pair (a chain of very short kernels), and a ragged batch of it
        _case("f32_single", "c1", 1, 16, 16, 64, 0.25),
        _case("f32_batch24", "c1", 24, 5, 60, 32, 0.25),
        # bf16 on a small grouped-query pair with an odd vocabulary and a batch that fills no tile
        _case("mini_ragged19", "mini-llama", 19, 3, 21, 20, 0.4),
        # one interactive request to the GPT pair, and the batch of 16 that its workload names
        _case("gpt_single", "c2", 1, 44, 44, 24, 0.09),
        _case("gpt_batch16", "c2", 16, 97, 128, 64, 0.25),
        # the same batch with the target conditioned on the whole prefix and the p/q rule on rejections
        _case("gpt_full_prefix", "c2", 16, 97, 128, 32, 0.25, full_prefix=True, correction=True),
        # standard speculative decoding on the same pair: n_gen counts rounds here
        _case("gpt_speculative", "c2", 16, 97, 128, 8, 0.0, gamma=4),
        # the 7B pair at the reject rate of the paper's tables, and the compaction stress with ragged prompts
        _case("llama_batch32", "c3", 32, 256, 256, 64, 0.09),
        _case("llama_ragged128", "c4", 128, 64, 512, 32, 0.25),
        # the 8B grouped-query pair: the large batch, one interactive request, a few long documents
        _case("gqa_batch64", "c5", 64, 512, 512, 64, 0.25),
        _case("gqa_single", "c5", 1, 200, 200, 32, 0.09),
        _case("gqa_long4", "c5", 4, 1500, 2000, 16, 0.5),
    ]


# pair -> (largest batch, longest prompt, most prompt tokens of a pass, most generated positions per row, most steps)
_RANGE = {"c1": (32, 60, 1500, 64), "mini-gpt": (40, 64, 1500, 30), "mini-llama": (40, 96, 2000, 30),
          "c2": (40, 512, 4096, 64), "c3": (64, 700, 12000, 48), "c4": (128, 512, 30000, 32), "c5": (64, 1900, 28000, 48)}


def _log_uniform(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.49)))))))


def draw(rng):
    pair = rng.choice(("c1", "mini-gpt", "mini-llama", "c2", "c2", "c3", "c4", "c5", "c5"))
    max_b, max_p, max_tok, max_gen = _RANGE[pair]
    batch = _log_uniform(rng, 1, max_b)
    hi = _log_uniform(rng, 4, max(4, min(max_p, max_tok // batch)))
    lo = hi if rng.random() < 0.4 else rng.randint(2, hi)
    reject = rng.choice((0.0, 0.05, 0.09, 0.25, 0.4, 0.6, 1.0))
    kind = rng.random()
    if kind < 0.15:
        gamma = rng.randint(1, 4)
        return _case("drawn", pair, batch, lo, hi, rng.randint(2, max(2, min(10, max_gen // (gamma + 1)))), 0.0, gamma=gamma)
    full, corr = kind < 0.30, 0.22 < kind < 0.37
    return _case("drawn", pair, batch, lo, hi, _log_uniform(rng, 4, max_gen), reject, full, corr)


def _config(case):
    kind = case["pair"]
    base = W.config(kind) if kind.startswith("c") else W.mini_config(kind.split("-")[1])
    per = case["gamma"] + 1 if case["gamma"] else 1
    need = case["prompt_max"] + case["n_gen"] * per
    max_pos = min(base.draft.max_pos, base.target.max_pos)
    return W.configs.replace(base, max_batch=case["batch"], max_seq=min(max_pos, -(-need // 32) * 32),
                             target_ctx_mode=W.CTX_FULL_PREFIX if case["full_prefix"] else W.CTX_OWN_HISTORY,
                             reject_mode=W.REJECT_SD if case["correction"] else W.REJECT_REPLACE, sd_gamma=case["gamma"])


def _marked(n, share):
    """n flags, a fraction `share` of them set, evenly spread."""
    i = torch.arange(n, dtype=torch.float64, device="cuda")
    return torch.floor((i + 1) * share) > torch.floor(i * share)


def _disagree(order, g):
    """`order` with a fraction 1 - AGREE of its entries moved among themselves."""
    out = order.clone()
    at = torch.nonzero(torch.rand(order.numel(), generator=g, device="cuda") > AGREE).flatten()
    out[at] = order[torch.roll(at, 1)]
    return out


def _model(m, dtype, g, path, marks, mark_dir):
    """Weights of one decoder on the GPU.  path: LLaMA: the token after each token [V]; GPT: the token after each position.
    marks: which tokens / positions carry mark_dir (None for the target, which the verifier does not read)."""
    d, gpt = m.d_model, m.arch == W.ARCH_GPT
    shapes, w = W.synth.model_weight_shapes(m), {}
    for name, shape in shapes.items():
        if name in ("tok_emb", "pos_emb", "lm_head", "normf.g"):
            continue
        t = torch.empty(shape, dtype=dtype if len(shape) == 2 else torch.float32, device="cuda")
        # matrices that write to the residual stream are scaled down with the depth, as such models are initialised
        std = 0.02 / math.sqrt(2 * m.n_layer) if name.endswith((".wo", ".w2")) else 0.02
        w[name] = t.normal_(1.0 if name.endswith(".g") else 0.0, std, generator=g)
    e = torch.empty((m.vocab, d), dtype=torch.float32, device="cuda").normal_(generator=g)
    sign = None if marks is None else (marks.to(torch.float32) * 2 - 1)[:, None] * mark_dir * MARK
    if gpt:
        w["tok_emb"] = e.to(dtype)
        w["pos_emb"] = (2.0 * e[path] + (0 if sign is None else 2.0 * sign)).to(dtype)
        gain = PEAK / d
    else:
        head = torch.empty_like(e)
        head[path] = e * (PEAK / d)
        w["lm_head"] = head.to(dtype)
        w["tok_emb"] = (e if sign is None else e + sign).to(dtype)
        gain = 1.0
    w["normf.g"] = torch.full((d,), gain, dtype=torch.float32, device="cuda")
    return {n: w[n] for n in shapes}


def _verifier(cfg, g, mark_dir):
    d, h, gpt = cfg.draft.d_model, cfg.ver_d_hidden, cfg.draft.arch == W.ARCH_GPT
    side = torch.where(torch.arange(h, device="cuda") % 2 == 0, 1.0, -1.0)
    w1 = torch.empty((h, d), device="cuda").normal_(0, 0.02, generator=g) + 0.5 * side[:, None] * mark_dir
    return {"v.w1": w1 * (d / PEAK if gpt else 1.0), "v.b1": torch.empty(h, device="cuda").normal_(0, 0.02, generator=g),
            "v.w2": -2.0 / h * side, "v.b2": torch.zeros(1, device="cuda")}


def _prompts(case, vocab, seed):
    r = np.random.default_rng(seed)
    lens = r.integers(case["prompt_min"], case["prompt_max"] + 1, size=case["batch"]).astype(np.int32)
    lens[-1] = case["prompt_max"]
    ranks = r.choice(vocab, size=(case["batch"], case["prompt_max"]), p=W.zipf_probs(vocab))
    toks = r.permutation(vocab)[ranks].astype(np.int32)
    toks[np.arange(case["prompt_max"])[None, :] >= lens[:, None]] = 0
    return toks, lens


def prepare(case, seed):
    """A context with its weights loaded, and the prompts of the batch in host memory."""
    cfg = _config(case)
    dtype = torch.float32 if cfg.dtype == W.DT_F32 else torch.bfloat16
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    vocab = cfg.draft.vocab
    mark_dir = torch.empty(cfg.draft.d_model, device="cuda").normal_(generator=g)
    mark_dir /= mark_dir.norm()
    order = torch.randperm(vocab, generator=g, device="cuda")
    if cfg.draft.arch == W.ARCH_GPT:
        path = order[torch.arange(cfg.draft.max_pos, device="cuda") % vocab]
        marks = _marked(cfg.draft.max_pos, case["reject"])
    else:                                   # one cycle through the whole vocabulary, marked along the cycle
        path = torch.empty_like(order)
        path[order] = torch.roll(order, -1)
        marks = torch.empty(vocab, dtype=torch.bool, device="cuda")
        marks[order] = _marked(vocab, case["reject"])
    s = binding.Sprinter(cfg, "cuda:0")
    s.load_weights(binding.DRAFT, _model(cfg.draft, dtype, g, path, marks, mark_dir))
    s.load_weights(binding.TARGET, _model(cfg.target, dtype, g, _disagree(path, g), None, None))
    s.load_weights(binding.VERIFIER, _verifier(cfg, g, mark_dir))
    prompts, lens = _prompts(case, vocab, seed)
    return dict(sprinter=s, prompts=prompts, lens=lens, n_gen=case["n_gen"], gamma=case["gamma"], logits=not case["full_prefix"])


def run(state):
    s = state["sprinter"]
    s.prefill(state["prompts"], state["lens"])
    if state["gamma"]:
        return s.sd_generate(state["gamma"], state["n_gen"])
    out = s.generate(state["n_gen"] - 1)
    # the library gives no logits when the target reads the whole prefix
    return {"generated": out, "last": s.step(debug=state["logits"])}


def _params(m):
    """(elements of the block matrices, elements of the LM head) of one decoder."""
    s = W.synth.model_weight_shapes(m)
    blocks = sum(a[0] * a[1] for n, a in s.items() if len(a) == 2 and n not in ("tok_emb", "pos_emb", "lm_head"))
    return blocks, m.vocab * m.d_model


def work(case):
    """Prefill: both models' blocks read once, one product with each per cached token.  A decode step: the draft once, the
    target once if any row is rejected, the rows' own cache entries; speculative rounds: gamma draft passes and one target pass."""
    cfg = _config(case)
    size = 4 if cfg.dtype == W.DT_F32 else 2
    B, mean = case["batch"], (case["prompt_min"] + case["prompt_max"]) / 2
    per = 1 + case["gamma"] * AGREE if case["gamma"] else 1
    any_rejected = 1.0 - (1.0 - case["reject"]) ** B
    nbytes = flops = 0.0
    for m, draft in ((cfg.draft, True), (cfg.target, False)):
        blocks, head = _params(m)
        kv = 2 * m.n_layer * m.n_kv_head * m.d_head             # cache elements per position
        attn = 4 * m.n_layer * m.n_head * m.d_head              # attention operations per (query, key)
        ctx = mean + case["n_gen"] * per / 2
        nbytes += blocks * size + B * mean * kv * size
        flops += B * mean * (2 * blocks + attn * mean / 2)
        if case["gamma"]:
            passes, rows = (case["gamma"], B) if draft else (1, B * (case["gamma"] + 1))
        else:
            passes, rows = (1, B) if draft else (any_rejected, B if case["full_prefix"] else B * case["reject"])
        caches = passes * B if draft or case["gamma"] else B * case["reject"]      # whole caches read
        nbytes += case["n_gen"] * (passes * (blocks + head) * size + caches * ctx * kv * size)
        flops += case["n_gen"] * (passes if draft else 1) * rows * (2 * (blocks + head) + attn * ctx)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """About four times what the bf16 mode and the float32 mode differ by on the same bf16 weights (relative: 2e-4 on the
    GPT-shaped and the small pairs, 1.2e-3 on the deep LLaMA-shaped targets); float32: rounding of sums in another order."""
    if case["pair"] == "c1":
        return {"rel": 2e-5, "max": 2e-4}
    if case["pair"] in ("c2", "mini-gpt", "mini-llama"):
        return {"rel": 1e-3, "max": 8e-3}
    return {"rel": 5e-3, "max": 6e-2}
