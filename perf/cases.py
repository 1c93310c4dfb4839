"""Performance cases: whole requests and single decoder layers through the public
entry points (prefill, decode_step, decode_batch, reset_kv), over the range a
program that uses the library meets.

A case is one client's request or one batch of clients, on one model:

* shape, layers, vocab: the layer shape of a configuration in configs.py with that
  many layers and output rows.  A few layers with a small vocabulary measure the
  layers themselves; two cases run whole models.
* weights / kv: storage of the matrices ("bf16", "q8", "f32") and the KV cache.
* clients: sequences that share one copy of the weights (1: the single-client calls).
* prompt, steps: prompt rows prefilled and decode steps after them.  Clients of a
  batch have prompts of several lengths up to `prompt`.
* chunk, page: prefill rows per pass and positions per KV page.

Decode steps are fed given tokens (scoring a known continuation), so that the
outputs are functions of the inputs alone and a near tie in one step's logits
cannot change the next step's input.

One pass forgets the sequence, prefills it and decodes; its outputs are the last
step's logits, the logit of the token the call picked, and the whole KV cache.
"""

from __future__ import annotations

import math

import numpy as np
import torch

from paper_2608_24204_amd import configs
from paper_2608_24204_amd.binding import WiciModel

LAYER_VOCAB = 4096   # output rows of the layer cases (the smallest configuration's)
INIT_STD = 0.02      # the repository's seeded weights: N(0, 0.02^2)
GAIN_STD = 0.1       # norm gains 1 + N(0, 0.1^2)


def _case(name, shape, layers, prompt, steps=0, *, vocab=LAYER_VOCAB, weights="bf16", kv="bf16",
          clients=1, chunk=2048, page=64):
    c = dict(shape=shape, layers=layers, vocab=vocab, weights=weights, kv=kv, clients=clients,
             prompt=prompt, steps=steps, chunk=chunk, page=page)
    return dict(name=name, **c) if name else c


def listed():
    return [
        # the smallest model, fp32 throughout: launches and latency are all there is
        _case("tiny_f32_request", "tiny", 2, 32, 16, weights="f32", kv="f32"),
        # a whole small model answering a prompt: prefill, then the per-token call
        _case("1b_request", "1b", 16, 512, 32, vocab=128256),
        # the whole flagship model (prompt 1024), fewer tokens than its benchmark
        _case("8b_request", "8b", 32, 1024, 24, vocab=128256),
        # its layers: the prompt of the flagship workload, one chunk
        _case("8b_prefill_1024", "8b", 4, 1024),
        # a prompt of middling, odd length
        _case("8b_prefill_333", "8b", 4, 333),
        # a short question: fewer rows than one output tile
        _case("8b_prefill_45", "8b", 4, 45),
        # long context: four chunks, then decode over 8K positions
        _case("8b_long_8192", "8b", 2, 8192, 16),
        # the widest layers, one full chunk
        _case("32b_prefill_2048", "32b", 2, 2048),
        # 8-bit weights: a prompt and its answer
        _case("8b_q8_request", "8b", 2, 600, 24, weights="q8"),
        # several clients on one copy of the weights, one token per call for all:
        # a moderate and a large group, and a group on 8-bit weights
        _case("8b_batch16", "8b", 4, 96, 32, clients=16, chunk=256),
        _case("8b_batch48", "8b", 2, 64, 48, clients=48, chunk=256),
        _case("8b_q8_batch8", "8b", 2, 96, 32, weights="q8", clients=8, chunk=256),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges: the four layer shapes, both weight
    formats, prompts of 1 to 4096 rows, 0 to 32 decode steps, 1 to 60 clients."""
    kind = rng.choice(["prefill", "prefill", "request", "batch", "batch"])
    shape = rng.choice(["tiny", "1b", "8b", "8b", "32b"])
    weights = "f32" if shape == "tiny" else rng.choice(["bf16", "bf16", "q8"])
    kv = "f32" if shape == "tiny" else "bf16"
    layers = 2 if shape == "tiny" or weights == "q8" or shape == "32b" else rng.randint(2, 4)
    page = rng.choice([16, 32, 64, 64, 128])
    if kind == "batch":
        return _case(None, shape, layers, _log_int(rng, 8, 200), rng.randint(16, 32), weights=weights,
                     kv=kv, clients=_log_int(rng, 2, 60), chunk=256, page=page)
    prompt = _log_int(rng, 1, 512 if shape == "tiny" else 4096)
    steps = 0 if kind == "prefill" else rng.randint(4, 32)
    return _case(None, shape, layers, prompt, steps, weights=weights, kv=kv,
                 chunk=rng.choice([512, 2048, 2048]), page=page)


# ---------------------------------------------------------------- inputs
def _config(case):
    base = configs.CONFIGS[case["shape"]]
    return configs.reduced(base, case["layers"], vocab=case["vocab"], weight_dtype=case["weights"],
                           kv_dtype=case["kv"])


def _lengths(case):
    """Prompt length of each client: up to `prompt`, spread over its upper half."""
    P = case["prompt"]
    return [P - (37 * b) % (P // 2 + 1) for b in range(case["clients"])]


def _capacity(case):
    return max(_lengths(case)) + max(case["steps"], 1)


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _tensors(case, gen):
    """Yields lists of (name, tensor): the embedding, each layer's, the rest, drawn
    on the GPU in this order."""
    c = _config(case)
    d, F, V = c.d_model, c.ffn_dim, c.vocab
    qd, kvd = c.n_heads * c.head_dim, c.n_kv_heads * c.head_dim
    dt = torch.float32 if case["weights"] == "f32" else torch.bfloat16

    def mat(n, k):
        w = torch.empty(n, k, dtype=dt, device="cuda")
        return w.normal_(0.0, INIT_STD, generator=gen)

    def gain():
        return 1.0 + GAIN_STD * torch.randn(d, device="cuda", generator=gen)

    yield [("tok_embeddings", mat(V, d))]
    for l in range(c.n_layers):
        p = f"layers.{l}."
        yield [(p + "attn_norm", gain()), (p + "wq", mat(qd, d)), (p + "wk", mat(kvd, d)),
               (p + "wv", mat(kvd, d)), (p + "wo", mat(d, qd)), (p + "ffn_norm", gain()),
               (p + "w_gate", mat(F, d)), (p + "w_up", mat(F, d)), (p + "w_down", mat(d, F))]
    yield [("norm", gain())] + ([] if c.tied_embeddings else [("lm_head", mat(V, d))])


def _tokens(case, seed):
    """(prompt of each client, tokens fed to each decode step [steps, clients])."""
    rng = np.random.default_rng([seed, 1])
    prompts = [rng.integers(0, case["vocab"], n).astype(np.int32) for n in _lengths(case)]
    return prompts, rng.integers(0, case["vocab"], (case["steps"], case["clients"])).astype(np.int32)


def prepare(case, seed):
    """Models loaded with weights, one per client, and the token ids."""
    cfg = _config(case)
    kw = dict(max_seq=_capacity(case), prefill_chunk=case["chunk"], kv_page=case["page"])
    lead = WiciModel(cfg, **kw)
    gen = _gen(seed)
    for group in _tensors(case, gen):
        # drawn on torch's stream, read on the model's: drawn first
        torch.cuda.current_stream().synchronize()
        lead.load_weights(dict(group))
    models = [lead] + [WiciModel(cfg, share_weights_of=lead, **kw)
                       for _ in range(case["clients"] - 1)]
    kvs = []
    for m in models:
        m._kv.zero_()   # the outputs hold every slot, also those no pass writes
        kvs.append(m._kv.view(torch.float32 if case["kv"] == "f32" else torch.bfloat16))
    torch.cuda.current_stream().synchronize()
    prompts, fed = _tokens(case, seed)
    return dict(models=models, kvs=kvs, prompts=prompts, fed=fed)


# ---------------------------------------------------------------- one pass
def run(state):
    models, fed = state["models"], state["fed"]
    steps = len(fed)
    for m, p in zip(models, state["prompts"]):
        m.reset_kv()
        tok, logits = m.prefill(p, want_logits=steps == 0 and len(models) == 1)
    if len(models) == 1:
        for i in range(steps):
            tok, logits = models[0].decode_step(int(fed[i, 0]), want_logits=i == steps - 1)
        toks, logits = [tok], logits[None]
    else:
        for i in range(steps):
            if i < steps - 1:
                WiciModel.decode_batch(models, fed[i])
            else:
                toks, logits = WiciModel.decode_batch(models, fed[i], want_logits=True)
    picked = np.array([logits[b, t] for b, t in enumerate(toks)], np.float32)
    return dict(logits=logits, picked=picked, kv=list(state["kvs"]))


# ---------------------------------------------------------------- what it takes
def work(case):
    """Weights once per prefill call and once per decode call, the cached keys and
    values read by each step and written once; matrix products and causal
    attention of every row."""
    c = _config(case)
    wb = {"bf16": 2.0, "f32": 4.0, "q8": 34 / 32}[case["weights"]]
    layer = c.n_layers * c.layer_matrix_params()
    head = c.vocab * c.d_model
    kv_pos = c.n_layers * 2 * c.n_kv_heads * c.head_dim * c.kvbytes  # bytes per position
    att = c.n_layers * 4 * c.n_heads * c.head_dim                    # flops per (query, key)
    nbytes = flops = 0.0
    for n in _lengths(case):
        nbytes += (layer + head) * wb + n * kv_pos + n * c.d_model * wb
        flops += 2 * (layer * n + head) + att * n * (n + 1) / 2
        for i in range(case["steps"]):
            nbytes += (n + i + 2) * kv_pos
            flops += 2 * (layer + head) + att * (n + i + 1)
    nbytes += case["steps"] * (layer + head) * wb
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Four times the distances from 64 bits that were measured (two-norms): fp32
    throughout 5e-7; bf16 caches 5e-4 with two layers, 1e-3 with four to sixteen
    and 1.7e-3 with 32 (a key or value next to a rounding boundary may round the
    other way, one bf16 step, at most 2^-7 of it, and what follows it sees that)."""
    if case["kv"] == "f32":
        return {"rel": 4e-6, "max": 4e-4}
    rel = 2e-3 if case["layers"] <= 2 else 4e-3 if case["layers"] <= 16 else 7e-3
    return {"rel": rel, "max": 0.03}


# ---------------------------------------------------------------- 64 bits
def _stored(w, fmt):
    """The values of a matrix as stored, in float64."""
    if fmt != "q8":
        return w.double()
    b = w.float().view(w.shape[0], -1, 32)
    d = (b.abs().amax(-1, keepdim=True) / 127.0).half().float()
    q = torch.where(d > 0, torch.round(b / d).clamp(-127, 127), torch.zeros_like(b))
    return (q.double() * d.double()).view(w.shape)


def exact(case, seed):
    """The same sequences through a plain float64 decoder; keys and values rounded
    to the cache type as they are cached."""
    c = _config(case)
    Hq, Hkv, hd, eps = c.n_heads, c.n_kv_heads, c.head_dim, c.rms_eps
    half, fmt = hd // 2, case["weights"]
    prompts, fed = _tokens(case, seed)
    seqs = [np.concatenate([p, fed[:, b]]) for b, p in enumerate(prompts)]
    n = [len(s) for s in seqs]
    ids = torch.from_numpy(np.concatenate(seqs)).long().cuda()
    pos = torch.cat([torch.arange(k, device="cuda") for k in n]).double()
    inv = c.rope_base ** (-2.0 * torch.arange(half, device="cuda", dtype=torch.float64) / hd)
    cos, sin = torch.cos(pos[:, None] * inv)[:, None], torch.sin(pos[:, None] * inv)[:, None]

    def rot(z):
        a, b = z[..., :half], z[..., half:]
        return torch.cat([a * cos - b * sin, a * sin + b * cos], -1)

    def norm(x, g):
        return x / torch.sqrt((x * x).mean(-1, keepdim=True) + eps) * g.double()

    def cached(z):
        return z.float().double() if case["kv"] == "f32" else z.bfloat16().double()

    page, n_pages = case["page"], -(-_capacity(case) // case["page"])
    kvs = [torch.zeros(c.n_layers, n_pages, 2, Hkv, page, hd, dtype=torch.float64, device="cuda")
           for _ in n]
    groups = _tensors(case, _gen(seed))
    emb = dict(next(groups))["tok_embeddings"]
    x = _stored(emb, fmt)[ids] if fmt == "q8" else emb[ids].double()
    for l in range(c.n_layers):
        t = {k.split(".")[-1]: v for k, v in next(groups)}
        a = norm(x, t["attn_norm"])
        q = rot((a @ _stored(t["wq"], fmt).T).view(-1, Hq, hd)) / math.sqrt(hd)
        k = cached(rot((a @ _stored(t["wk"], fmt).T).view(-1, Hkv, hd)))
        v = cached((a @ _stored(t["wv"], fmt).T).view(-1, Hkv, hd))
        out = torch.empty_like(q)
        at = 0
        for b, T in enumerate(n):
            for h in range(Hq):
                g = h // (Hq // Hkv)
                kk, vv = k[at:at + T, g], v[at:at + T, g]
                for r in range(0, T, 2048):
                    e = min(T, r + 2048)
                    s = q[at + r:at + e, h] @ kk[:e].T
                    keep = (torch.arange(e, device="cuda")[None]
                            <= torch.arange(r, e, device="cuda")[:, None])
                    out[at + r:at + e, h] = torch.softmax(s.masked_fill(~keep, -math.inf), -1) @ vv[:e]
            # position p: slot p % page of physical page n_pages - 1 - p // page
            for w, z in enumerate((k, v)):
                pad = torch.zeros(n_pages * page, Hkv, hd, dtype=torch.float64, device="cuda")
                pad[:T] = z[at:at + T]
                kvs[b][l, :, w] = pad.view(n_pages, page, Hkv, hd).flip(0).transpose(1, 2)
            at += T
        x = x + out.reshape(len(ids), -1) @ _stored(t["wo"], fmt).T
        a = norm(x, t["ffn_norm"])
        gate = a @ _stored(t["w_gate"], fmt).T
        h = gate / (1.0 + torch.exp(-gate)) * (a @ _stored(t["w_up"], fmt).T)
        x = x + h @ _stored(t["w_down"], fmt).T
    t = dict(next(groups))
    last = torch.tensor(np.cumsum(n) - 1, device="cuda")
    logits = norm(x[last], t["norm"]) @ _stored(t.get("lm_head", emb), fmt).T
    return dict(logits=logits, picked=logits.amax(-1), kv=[z.view(-1) for z in kvs])
