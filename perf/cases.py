"""Timed cases of the decoder library: what a program that serves Qwen3-shaped models has it do.

Three kinds of pass, all through the public calls of `paper_2512_21571_amd.binding.Model`:

* ``layer``    one fp32 decoder layer without embedding and head: a prompt of hidden-state rows, then one
               row at a time against the cache;
* ``prompt``   reset a slot and run one prompt (or two turns of one), logits of the last position out;
* ``generate`` reset, one prompt per slot, read the first tokens back, a greedy run of all slots with the
               tokens fed back on the device, and a closing step (the turn's end token) whose logits are
               returned: they depend on every cache row the run wrote.

Shapes are those of the repository's own configurations (0.6B, 1.7B, 4B, 8B).  Where `layers` is less than
the model's depth, the vocabulary is cut by the same factor, so that the head keeps its share of a pass.

Embedding rows have unit variance and an untied head is the embedding moved by one row, so that the
arg-max of every greedy step is decided by a margin like a trained model's (the current token where
the head is tied, the next id where it is not) and a greedy run does not hang on the last bits.
"""
import math
import types

import numpy as np
import torch

from paper_2512_21571_amd import binding

# hidden, query heads, kv heads, ffn, depth, tied head
MODELS = {
    "0.6b": (1024, 16, 8, 3072, 28, True),
    "1.7b": (2048, 16, 8, 6144, 28, True),
    "4b": (2560, 32, 8, 9728, 36, True),
    "8b": (4096, 32, 8, 12288, 36, False),
}
VOCAB, HEAD_DIM, EPS, THETA, STD = 151936, 128, 1e-6, 1e6, 0.02
DTYPES = {"f32": binding.F32, "bf16": binding.BF16, "f16": binding.F16, "w8": binding.W8}
TORCH = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}


def listed():
    return [
        # the smallest configuration: one fp32 layer, 16 rows then 16 single rows (launches and latency count)
        dict(name="layer-f32-p16-d16", kind="layer", model="0.6b", dtype="f32", layers=1, batch=1, prompt=16, spread=0, more=0, steps=16),
        # a short chat prompt on the smallest model, whole depth: time to first token
        dict(name="prompt-0.6b-p128", kind="prompt", model="0.6b", dtype="bf16", layers=28, batch=1, prompt=128, spread=0, more=0, steps=0),
        # an ordinary prompt, up to which every activation carries two pieces
        dict(name="prompt-1.7b-p512", kind="prompt", model="1.7b", dtype="bf16", layers=7, batch=1, prompt=512, spread=0, more=0, steps=0),
        # a document, and then an odd-sized second turn on top of it
        dict(name="prompt-4b-p2048-p333", kind="prompt", model="4b", dtype="bf16", layers=4, batch=1, prompt=2048, spread=0, more=333, steps=0),
        # a full context in one call, matrix-core bound
        dict(name="prompt-8b-p4096", kind="prompt", model="8b", dtype="bf16", layers=4, batch=1, prompt=4096, spread=0, more=0, steps=0),
        # one user, smallest model, whole depth: the paper's own setting
        dict(name="gen-0.6b-b1-p128-d128", kind="generate", model="0.6b", dtype="bf16", layers=28, batch=1, prompt=128, spread=0, more=0, steps=128),
        # one user in the paper's 16-bit format
        dict(name="gen-1.7b-f16-b1-p512-d256", kind="generate", model="1.7b", dtype="f16", layers=7, batch=1, prompt=512, spread=0, more=0, steps=256),
        # one user on a long context
        dict(name="gen-4b-b1-p2048-d128", kind="generate", model="4b", dtype="bf16", layers=4, batch=1, prompt=2048, spread=0, more=0, steps=128),
        # a few users of a small model, prompts of different lengths
        dict(name="gen-0.6b-b4-p128-d128", kind="generate", model="0.6b", dtype="bf16", layers=7, batch=4, prompt=128, spread=27, more=0, steps=128),
        # a batch of eight on the 4B shape
        dict(name="gen-4b-b8-p2048-d128", kind="generate", model="4b", dtype="bf16", layers=4, batch=8, prompt=2048, spread=0, more=0, steps=128),
        # weight-only 8-bit layers, a server's batch with contexts of different lengths
        dict(name="gen-8b-w8-b16-p512-d128", kind="generate", model="8b", dtype="w8", layers=4, batch=16, prompt=512, spread=200, more=0, steps=128),
        # the largest configuration: 16 full contexts
        dict(name="gen-8b-b16-p4096-d128", kind="generate", model="8b", dtype="bf16", layers=4, batch=16, prompt=4096, spread=0, more=0, steps=128),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _cost(case):
    w = work(case)
    return w["bytes"] / 6e12 + w["flops"] / 1e15


def draw(rng):
    most = max(_cost(c) for c in listed())
    while True:
        kind = rng.choice(["prompt", "prompt", "generate", "generate", "generate", "layer"])
        model = rng.choice(list(MODELS))
        if kind == "layer":
            c = dict(kind=kind, model=rng.choice(["0.6b", "1.7b"]), dtype="f32", layers=rng.randint(1, 2), batch=1,
                     prompt=_log_uniform(rng, 1, 96), spread=0, more=0, steps=rng.randint(1, 24))
        elif kind == "prompt":
            n, more = _log_uniform(rng, 9, 4096), rng.choice([0, 0, _log_uniform(rng, 9, 512)])
            if more:  # a first turn that a server has cached in whole pages
                n = max(64, n // 64 * 64)
            c = dict(kind=kind, model=model, dtype=rng.choice(["bf16", "bf16", "f16", "w8"]), layers=rng.randint(2, 6), batch=1,
                     prompt=n, spread=0, more=more, steps=0)
        else:
            n = _log_uniform(rng, 16, 4096)
            c = dict(kind=kind, model=model, dtype=rng.choice(["bf16", "bf16", "f16", "w8"]), layers=rng.randint(2, 6),
                     batch=rng.choice([1, 1, 2, 3, 4, 5, 8, 11, 16]), prompt=n, spread=rng.choice([0, n // 3]), more=0,
                     steps=_log_uniform(rng, 16, 256))
        if _cost(c) <= most:
            return c


# ---- inputs ---------------------------------------------------------------------------------


def _shape(case):
    H, nq, nkv, F, depth, tied = MODELS[case["model"]]
    layer = case["kind"] == "layer"
    vocab = 0 if layer else max(16, int(round(VOCAB * min(1.0, case["layers"] / depth) / 16)) * 16)
    return types.SimpleNamespace(hidden=H, n_layers=case["layers"], n_q_heads=nq, n_kv_heads=nkv, head_dim=HEAD_DIM, ffn=F, vocab=vocab,
                                 rms_eps=EPS, rope_theta=THETA, has_embed_and_head=not layer, tied_lm_head=tied and not layer,
                                 dtype=DTYPES[case["dtype"]])


def _entries(s):
    """The canonical blob's tensors in order: (name, rows, columns; rows 0 for a gain vector)."""
    dq, dkv = s.n_q_heads * HEAD_DIM, s.n_kv_heads * HEAD_DIM
    out = [("embed", s.vocab, s.hidden)] if s.has_embed_and_head else []
    for i in range(s.n_layers):
        out += [("%d.%s" % (i, n), r, c) for n, r, c in (
            ("g_in", 0, s.hidden), ("wq", dq, s.hidden), ("wk", dkv, s.hidden), ("wv", dkv, s.hidden), ("g_q", 0, HEAD_DIM), ("g_k", 0, HEAD_DIM),
            ("wo", s.hidden, dq), ("g_post", 0, s.hidden), ("wgate", s.ffn, s.hidden), ("wup", s.ffn, s.hidden), ("wdown", s.hidden, s.ffn))]
    if s.has_embed_and_head:
        out += [("g_final", 0, s.hidden)] + ([] if s.tied_lm_head else [("lm_head", s.vocab, s.hidden)])
    return out


def _weights(case, seed):
    """The blob's bytes on the GPU, and name -> the tensor (or bytes and row scales) inside it."""
    s, w8 = _shape(case), case["dtype"] == "w8"
    half = TORCH["bf16" if w8 else case["dtype"]]
    size = torch.empty(0, dtype=half).element_size()
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    sizes = [4 * c if r == 0 else r * c + 4 * r if w8 and n[0].isdigit() else size * r * c for n, r, c in _entries(s)]
    blob, at, named = torch.empty(sum(sizes), dtype=torch.uint8, device="cuda"), 0, {}
    for (name, r, c), n in zip(_entries(s), sizes):
        part = blob[at:at + n]
        at += n
        if r == 0:
            named[name] = part.view(torch.float32)
            named[name].normal_(1.0, 0.1, generator=g)
            continue
        if name == "lm_head":
            named[name] = part.view(half).view(r, c)
            named[name].copy_(torch.roll(named["embed"], 1, 0))
            continue
        v = torch.empty((r, c), dtype=torch.float32, device="cuda").normal_(0.0, 1.0 if name == "embed" else STD, generator=g)
        if w8 and name[0].isdigit():
            scale = part[r * c:].view(torch.float32)
            scale.copy_((v.abs().amax(1) / 127).to(torch.bfloat16).to(torch.float32) * (1 + 2.0 ** -7))
            q = part[:r * c].view(torch.int8).view(r, c)
            q.copy_((v / scale[:, None]).round().clamp(-127, 127))
            named[name] = (q, scale)
        else:
            named[name] = part.view(half).view(r, c)
            named[name].copy_(v)
    return blob, named


def _lengths(case):
    return [case["prompt"] - (case["spread"] * i) // max(1, case["batch"] - 1) for i in range(case["batch"])]


def _prompts(case, seed):
    r, vocab = np.random.RandomState(seed % (1 << 31)), _shape(case).vocab
    first = [r.randint(0, vocab, n).astype(np.int32) for n in _lengths(case)]
    return first, r.randint(0, vocab, case["more"]).astype(np.int32), r.randint(0, vocab, case["batch"]).astype(np.int32)


def _rows(case, seed):
    g = torch.Generator(device="cuda").manual_seed(int(seed) + 1)
    return torch.empty((case["prompt"] + case["steps"], MODELS[case["model"]][0]), device="cuda").normal_(generator=g)


def prepare(case, seed):
    blob, _ = _weights(case, seed)
    host = blob.cpu().numpy()
    del blob
    room = (case["prompt"] + case["more"] + case["steps"] + 1 + 127) // 128 * 128
    state = {"case": case, "model": binding.Model(_shape(case), host, case["batch"], room)}
    if case["kind"] == "layer":
        x = _rows(case, seed)
        state.update(prompt=x[:case["prompt"]].clone(), rows=[r.clone() for r in x[case["prompt"]:].split(1)])
    else:
        first, more, closing = _prompts(case, seed)
        state.update(first=first, more=more, closing=closing, slots=list(range(case["batch"])))
    return state


def run(state):
    case, model = state["case"], state["model"]
    model.kv_reset()
    if case["kind"] == "layer":
        return [model.prefill_hidden(0, state["prompt"])] + [model.decode_step_hidden([0], r) for r in state["rows"]]
    if case["kind"] == "prompt":
        out = [model.prefill(0, state["first"][0])[0]]
        if case["more"]:
            out.append(model.prefill(0, state["more"])[0])
        return out
    starts = [model.prefill(i, p) for i, p in enumerate(state["first"])]
    tokens, _ = model.decode_greedy(state["slots"], [int(t.item()) for _, t in starts], case["steps"])
    last, _ = model.decode_step(state["slots"], state["closing"])
    return {"prompt": [logits for logits, _ in starts], "tokens": tokens, "last": last}


# ---- what a pass cannot do without ------------------------------------------------------------


def work(case):
    s = _shape(case)
    size = {"f32": 4, "w8": 1}.get(case["dtype"], 2)
    row = 4 if case["dtype"] == "f32" else 2
    dq, dkv = s.n_q_heads * HEAD_DIM, s.n_kv_heads * HEAD_DIM
    layer = (dq + 2 * dkv) * s.hidden + s.hidden * dq + 3 * s.ffn * s.hidden
    scales = 4 * (dq + 2 * dkv + 2 * s.hidden + 2 * s.ffn) if case["dtype"] == "w8" else 0
    weights = s.n_layers * (size * layer + scales)
    head = row * s.vocab * s.hidden
    moved = flops = 0.0

    def step(batch, rows, new, heads):
        """One call: `rows` = cached rows read, `new` = tokens in, `heads` = logit rows out."""
        nonlocal moved, flops
        moved += weights + (head if heads else 0) + s.n_layers * 2 * dkv * row * (rows + new) + new * s.hidden * row + 4.0 * heads * s.vocab

    def products(new, pairs, heads):
        nonlocal flops
        flops += 2.0 * new * s.n_layers * layer + 4.0 * s.n_layers * dq * pairs + 2.0 * heads * s.vocab * s.hidden

    heads = 1 if s.has_embed_and_head else 0
    for n in _lengths(case):
        step(1, 0, n, heads)
        products(n, n * (n + 1) / 2, heads)
    if case["more"]:
        n, m = case["prompt"], case["more"]
        step(1, n, m, heads)
        products(m, m * n + m * (m + 1) / 2, heads)
    b, total = case["batch"], sum(_lengths(case))
    for i in range(case["steps"] + (1 if case["kind"] == "generate" else 0)):
        step(b, total + b * i, b, b * heads)
        products(b, total + b * (i + 1), b * heads)
    return {"bytes": moved, "flops": flops}


def tolerance(case):
    """About four times the distance to exact() over these ranges: 2e-7 with fp32 weights and cache, 5e-4 in binary16,
    3e-3 in bf16 (the cache rows' own rounding, through all layers)."""
    return {"rel": {"f32": 1e-6, "f16": 2e-3}.get(case["dtype"], 1e-2)}


# ---- the same in 64 bits ------------------------------------------------------------------------


def _wide(w):
    return w[0].double() * w[1].double()[:, None] if isinstance(w, tuple) else w.double()


def _norm(x, gain):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + EPS) * gain.double()


def _layers(s, named, seqs):
    """Hidden-state sequences [T, hidden] through every layer, causal."""
    G, D = s.n_q_heads // s.n_kv_heads, HEAD_DIM
    inv = THETA ** (-torch.arange(0, D, 2, dtype=torch.float64, device="cuda") / D)

    def turn(v):  # [T, heads, D]
        a = torch.arange(v.shape[0], dtype=torch.float64, device="cuda")[:, None, None] * inv
        lo, hi = v[..., :D // 2], v[..., D // 2:]
        return torch.cat([lo * a.cos() - hi * a.sin(), hi * a.cos() + lo * a.sin()], -1)

    for i in range(s.n_layers):
        w = {n: _wide(named["%d.%s" % (i, n)]) for n in ("wq", "wk", "wv", "wo", "wgate", "wup", "wdown")}
        gain = {n: named["%d.%s" % (i, n)] for n in ("g_in", "g_q", "g_k", "g_post")}
        for j, x in enumerate(seqs):
            T = x.shape[0]
            h = _norm(x, gain["g_in"])
            q = turn(_norm((h @ w["wq"].T).view(T, -1, D), gain["g_q"])).view(T, s.n_kv_heads, G, D)
            k = turn(_norm((h @ w["wk"].T).view(T, -1, D), gain["g_k"]))
            v = (h @ w["wv"].T).view(T, -1, D)
            out = torch.empty((T, s.n_kv_heads, G, D), dtype=torch.float64, device="cuda")
            mask = torch.ones((T, T), dtype=torch.bool, device="cuda").triu(1)
            for a in range(s.n_kv_heads):
                for b in range(G):
                    p = (q[:, a, b] @ k[:, a].T) / math.sqrt(D)
                    out[:, a, b] = torch.softmax(p.masked_fill_(mask, -math.inf), -1) @ v[:, a]
            x = x + out.view(T, -1) @ w["wo"].T
            h = _norm(x, gain["g_post"])
            seqs[j] = x + (torch.nn.functional.silu(h @ w["wgate"].T) * (h @ w["wup"].T)) @ w["wdown"].T
    return seqs


def exact(case, seed):
    """The whole sequence of every slot as one causal pass; the tokens of a greedy run are known beforehand
    (see the top of this file)."""
    s = _shape(case)
    _, named = _weights(case, seed)
    n, d = case["prompt"], case["steps"]
    if case["kind"] == "layer":
        y = _layers(s, named, [_rows(case, seed).double()])[0]
        return [y[:n]] + list(y[n:].split(1))
    head = _wide(named["embed" if s.tied_lm_head else "lm_head"])

    def logits(x):
        return _norm(x, named["g_final"]) @ head.T

    first, more, closing = _prompts(case, seed)
    seqs = []
    for i, p in enumerate(first):
        run_ = [p.astype(np.int64)]
        if case["kind"] == "generate":
            run_ += [(int(p[-1]) + (0 if s.tied_lm_head else 1 + np.arange(d))) % s.vocab + np.zeros(d, np.int64), closing[i:i + 1].astype(np.int64)]
        elif case["more"]:
            run_.append(more.astype(np.int64))
        seqs.append(named["embed"][torch.from_numpy(np.concatenate(run_)).cuda()].double())
    seqs = _layers(s, named, seqs)
    if case["kind"] == "prompt":
        return [logits(seqs[0][n - 1])] + ([logits(seqs[0][-1])] if case["more"] else [])
    return {"prompt": [logits(x[len(p) - 1]) for x, p in zip(seqs, first)], "tokens": None, "last": logits(torch.stack([x[-1] for x in seqs]))}
