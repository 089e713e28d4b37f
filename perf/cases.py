"""Performance cases of the verification path: what a program that decodes with this library asks of it.

Every case goes through ``paper_2404_08698_amd.binding`` as such a program would: the model, the caches and the
packed weights are made once (``prepare``), and ``run`` is one step, one prompt or one matrix product on them.

The widths are those of the repository's workloads (the tiny fp32 decoder, the LLaMA-7B, LLaMA-13B and
ChatGLM3-6B shapes).  One listed case is the whole 32-layer 7B model; the others hold a stack of a few layers and
the LM head at the same widths, so that a change of rounding in one layer stays visible as what it is.
Cached contents are N(0, 1), as projected keys and values of normalised rows are; token ids are random with copied
spans, like the prompts the drafter is made for.
"""
import math

import numpy as np
import torch

from paper_2404_08698_amd import binding as B
from paper_2404_08698_amd import synth

#: width -> (d_model, heads, head_dim, ffn, vocab, key / value heads, storage type)
WIDTHS = {
    "tiny_f32": (256, 4, 64, 688, 1024, 4, "f32"),
    "tiny_bf16": (256, 4, 64, 688, 1024, 4, "bf16"),
    "7b": (4096, 32, 128, 11008, 32000, 32, "bf16"),
    "13b": (5120, 40, 128, 13824, 32000, 40, "bf16"),
    "glm6b": (4096, 32, 128, 13696, 65024, 2, "bf16"),
}
EPS, ROPE_BASE = 1e-5, 10000.0
#: passes of a step before the cache is put back to its starting length (a decoding loop does not roll back its
#: own steps); each pass commits the window's first row and whatever drafts happen to be right
SLACK = 96


def listed():
    return [
        # the smallest use: the tiny fp32 decoder, a window of k = 4 drafts after a 128-token prompt; its launches
        # and the host path are all there is
        {"name": "tiny_f32_step", "kind": "step", "width": "tiny_f32", "layers": 2, "rows": 5, "length": 128, "scattered": False},
        # the same model reading its prompt
        {"name": "tiny_f32_prompt", "kind": "prompt", "width": "tiny_f32", "layers": 2, "rows": 128, "length": 0, "export": False},
        # the headline: the whole 7B model, k = 5 drafts, 512 cached tokens
        {"name": "7b_step_6rows", "kind": "step", "width": "7b", "layers": 32, "rows": 6, "length": 512, "scattered": False},
        # plain decoding far into a long context, pages handed out in no order (a cache that has been in use)
        {"name": "7b_decode_long", "kind": "step", "width": "7b", "layers": 8, "rows": 1, "length": 4096, "scattered": True},
        # the widest single draft of the long-context workload: k = 16
        {"name": "7b_step_17rows", "kind": "step", "width": "7b", "layers": 8, "rows": 17, "length": 2048, "scattered": False},
        # the 13B workload's window: k = 8 drafts, about 1100 cached tokens
        {"name": "13b_step_9rows", "kind": "step", "width": "13b", "layers": 8, "rows": 9, "length": 1101, "scattered": False},
        # several candidate drafts in one forward: 4 candidates of 5 tokens
        {"name": "7b_tree_21rows", "kind": "tree", "width": "7b", "layers": 8, "candidates": 4, "depth": 5, "length": 633},
        # a full serving batch in plain decoding: 32 sequences of 300 to 700 tokens
        {"name": "7b_batch_32x1", "kind": "batch", "width": "7b", "layers": 8, "sequences": 32, "rows": 1, "length": 512},
        # the 7B workload's prompt
        {"name": "7b_prompt_512", "kind": "prompt", "width": "7b", "layers": 4, "rows": 512, "length": 0, "export": False},
        # the long-context workload's prompt
        {"name": "7b_prompt_3584", "kind": "prompt", "width": "7b", "layers": 4, "rows": 3584, "length": 0, "export": False},
        # a ragged piece of a prompt behind what is cached already, grouped key / value heads, and the piece's keys
        # and values read back (a program that stores or ships its caches)
        {"name": "glm6b_piece_205", "kind": "prompt", "width": "glm6b", "layers": 4, "rows": 205, "length": 777, "export": True},
        # one matrix product on its own, gate / up of the 7B shape
        {"name": "linear_22016x4096_17", "kind": "linear", "rows": 17, "n": 22016, "k": 4096},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("step", "step", "step", "batch", "batch", "tree", "prompt", "prompt", "linear"))
    if kind == "linear":
        return {"kind": kind, "rows": rng.randint(1, 32), "n": 16 * _log(rng, 16, 2750), "k": 8 * _log(rng, 32, 1728)}
    width = rng.choice(("7b", "7b", "13b", "glm6b", "tiny_bf16") + (("tiny_f32",) if kind != "batch" else ()))
    tiny = width.startswith("tiny")
    if kind == "prompt":
        return {"kind": kind, "width": width, "layers": 2 if tiny else 4, "rows": _log(rng, 16, 400 if tiny else 1800),
                "length": rng.choice((0, 0, _log(rng, 16, 1500))), "export": rng.random() < 0.3}
    case = {"kind": kind, "width": width, "layers": 2 if tiny else 8}
    if kind == "step":
        return {**case, "rows": _log(rng, 1, 32), "length": _log(rng, 32, 4096), "scattered": rng.random() < 0.5}
    if kind == "tree":
        candidates = rng.randint(2, 6)
        return {**case, "candidates": candidates, "depth": rng.randint(1, 31 // candidates), "length": _log(rng, 32, 2048)}
    sequences = _log(rng, 2, 32)
    return {**case, "sequences": sequences, "rows": rng.randint(1, min(8, 32 // sequences)), "length": _log(rng, 32, 1024)}


# ------------------------------------------------------------------------------------------------------ inputs

def _shape(case):
    d, heads, dh, ffn, vocab, kv_heads, dtype = WIDTHS[case["width"]]
    return synth.ModelShape(case["layers"], d, heads, dh, ffn, vocab, dtype, EPS, ROPE_BASE, 0 if kv_heads == heads else kv_heads)


def _weights(case, gen):
    d, heads, dh, ffn, vocab, kv_heads, dtype = WIDTHS[case["width"]]
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    kvd = kv_heads * dh

    def mat(*shape):
        return torch.empty(shape, dtype=dt, device="cuda").normal_(0.0, 0.02, generator=gen)

    def gain():
        return torch.empty(d, dtype=dt, device="cuda").normal_(1.0, 0.02, generator=gen)

    w = {"embed": mat(vocab, d), "final_norm": gain(), "lm_head": mat(vocab, d)}
    per = {"attn_norm": gain, "wq": lambda: mat(d, d), "wk": lambda: mat(kvd, d), "wv": lambda: mat(kvd, d),
           "wo": lambda: mat(d, d), "ffn_norm": gain, "w_gate": lambda: mat(ffn, d), "w_up": lambda: mat(ffn, d),
           "w_down": lambda: mat(d, ffn)}
    for name, make in per.items():
        w[name] = [make() for _ in range(case["layers"])]
    return w


def _tokens(rng, vocab, n):
    """Random ids of which about 40 % are copied spans of 4 to 16 earlier ones."""
    out = list(rng.randint(0, vocab, 16))
    while len(out) < n:
        if rng.rand() < 0.06:
            span = rng.randint(4, 17)
            at = rng.randint(0, max(1, len(out) - span))
            out.extend(out[at:at + span])
        else:
            out.append(rng.randint(0, vocab))
    return [int(t) for t in out[:n]]


def _cached(case, gen, length):
    """[(k, v)] per layer: float32 values that the storage type holds exactly."""
    d, heads, dh, ffn, vocab, kv_heads, dtype = WIDTHS[case["width"]]
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    return [tuple(torch.empty(length, kv_heads * dh, dtype=torch.float32, device="cuda").normal_(0.0, 1.0, generator=gen).to(dt).float()
                  for _ in range(2)) for _ in range(case["layers"])]


def _lengths(case, rng):
    """Cached tokens of every sequence."""
    if case["kind"] == "batch":
        return [max(8, int(case["length"] * f)) for f in rng.uniform(0.6, 1.4, case["sequences"])]
    return [case["length"]]


def _tree(case):
    parents = [-1]
    for _ in range(case["candidates"]):
        for j in range(case["depth"]):
            parents.append(0 if j == 0 else len(parents) - 1)
    return parents


def _inputs(case, seed):
    """(weights, [(length, cached)], [tokens]) of a model case, from the seed alone."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    rng = np.random.RandomState(seed % (1 << 32))
    weights = _weights(case, gen)
    lengths = _lengths(case, rng)
    caches = [(n, _cached(case, gen, n)) for n in lengths]
    rows = len(_tree(case)) if case["kind"] == "tree" else case["rows"]
    tokens = [_tokens(rng, WIDTHS[case["width"]][4], rows) for _ in lengths]
    return weights, caches, tokens


def _linear_inputs(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.empty(case["rows"], case["k"], dtype=torch.float32, device="cuda").normal_(0.0, 1.0, generator=gen)
    w = torch.empty(case["n"], case["k"], dtype=torch.bfloat16, device="cuda").normal_(0.0, 0.02, generator=gen)
    return x, w


# ----------------------------------------------------------------------------------------------- prepare and run

def prepare(case, seed):
    if case["kind"] == "linear":
        x, w = _linear_inputs(case, seed)
        ws = torch.empty(B.lib().anpd_linear_workspace_bytes(case["rows"], case["k"]), dtype=torch.uint8, device="cuda")
        return {"case": case, "x": x, "w": w, "packed": B.pack_weights(w), "ws": ws,
                "y": torch.empty(case["rows"], case["n"], dtype=torch.float32, device="cuda")}
    weights, caches, tokens = _inputs(case, seed)
    shape = _shape(case)
    prompt = case["kind"] == "prompt"
    rows = max(len(t) for t in tokens)
    capacity = max(n for n, _ in caches) + rows + (0 if prompt else SLACK)
    model = B.Model(shape, weights, max_window=32, max_positions=capacity)
    kvs = []
    for length, layers in caches:
        kv = B.KVCache(model, capacity)
        if case.get("scattered"):
            kv.set_page_order(np.random.RandomState(seed % (1 << 32)).permutation(kv.num_pages).tolist())
        if length:
            for layer, (k, v) in enumerate(layers):
                kv.write(layer, 0, k, v)
        kv.truncate(length)
        kvs.append(kv)
    state = {"case": case, "model": model, "kvs": kvs, "tokens": tokens, "lengths": [n for n, _ in caches], "capacity": capacity}
    n_logits = 1 if prompt else sum(len(t) for t in tokens)
    state["logits"] = torch.empty(n_logits, shape.vocab, dtype=torch.float32, device="cuda")
    if prompt:
        state["ws"] = torch.empty(max(256, B.prefill_workspace_bytes(model, rows)), dtype=torch.uint8, device="cuda")
    if case["kind"] == "tree":
        state["parents"] = _tree(case)
    return state


def run(state):
    case = state["case"]
    if case["kind"] == "linear":
        return B.linear(state["x"], state["w"], B.GEMM_MFMA, packed=state["packed"], Y=state["y"], workspace=state["ws"])
    model, kvs, tokens, logits = state["model"], state["kvs"], state["tokens"], state["logits"]
    if case["kind"] == "prompt":
        kv, at = kvs[0], state["lengths"][0]
        if kv.length != at:
            kv.truncate(at)
        B.prefill(model, kv, tokens[0], out_logits=logits, workspace=state["ws"])
        out = {"logits": logits}
        if case["export"]:
            out["kv"] = [kv.read(layer, at, case["rows"]) for layer in range(case["layers"])]
        return out
    for kv, at, window in zip(kvs, state["lengths"], tokens):
        if kv.length + len(window) > at + SLACK:
            kv.truncate(at)
    if case["kind"] == "batch":
        done = B.verify_batch(model, kvs, tokens, out_logits=logits)
        return {"logits": logits, "accepted": np.array([a for a, _ in done])}
    if case["kind"] == "tree":
        accepted, _, _ = B.verify_tree(model, kvs[0], tokens[0], state["parents"], out_logits=logits)
    else:
        accepted, _ = B.verify(model, kvs[0], tokens[0], out_logits=logits)
    return {"logits": logits, "accepted": accepted}


# ------------------------------------------------------------------------------------------ work and tolerance

def work(case):
    if case["kind"] == "linear":
        m, n, k = case["rows"], case["n"], case["k"]
        return {"bytes": 2 * n * k + 4 * m * (n + k), "flops": 2 * m * n * k}
    d, heads, dh, ffn, vocab, kv_heads, dtype = WIDTHS[case["width"]]
    el = 2 if dtype == "bf16" else 4
    kvd = kv_heads * dh
    matrices = case["layers"] * (2 * d * d + 2 * d * kvd + 3 * d * ffn)
    per_seq = len(_tree(case)) if case["kind"] == "tree" else case["rows"]
    n_seq = case.get("sequences", 1)
    rows, out_rows = per_seq * n_seq, (1 if case["kind"] == "prompt" else per_seq * n_seq)
    cached = n_seq * case["length"]
    nbytes = el * (matrices + vocab * d + rows * d)                       # weights once, embedding rows
    nbytes += case["layers"] * 2 * kvd * el * (cached + rows)             # cache read, new rows written
    nbytes += 4 * out_rows * vocab                                        # logits
    if case.get("export"):
        nbytes += case["layers"] * 2 * kvd * (el + 4) * rows
    seen = rows * case["length"] + n_seq * per_seq * (per_seq + 1) / 2    # (row, key) pairs
    flops = 2 * rows * matrices + 2 * out_rows * vocab * d + case["layers"] * 4 * heads * dh * seen
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # about four times the largest relative error against the 64-bit result that was seen
    if case["kind"] == "linear":
        return {"rel": 1e-5}    # 2.5e-6: activations as a sum of two bf16 terms, fp32 accumulation
    if WIDTHS[case["width"]][6] == "f32":
        return {"rel": 4e-6}    # 2.3e-7 to the 64-bit result; longer chains of fp32 sums in another order
    # a new key or value next to a bf16 rounding boundary falls on either side of it: prompts, whose keys are all
    # new, are 5e-4 off (keys and values of the fourth layer 9e-4), steps 2e-5 to 1e-4, more the shorter their cache
    return {"rel": 4e-3} if case["kind"] == "prompt" else {"rel": 2e-3}


# ------------------------------------------------------------------------------------------------------- exact

def _norm(x, g):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + EPS) * g.double()


def _rope(x, pos, heads, dh):
    half = dh // 2
    theta = ROPE_BASE ** (-2.0 * torch.arange(half, dtype=torch.float64, device=x.device) / dh)
    ang = pos.double()[:, None] * theta[None, :]
    c, s = torch.cos(ang)[:, None, :], torch.sin(ang)[:, None, :]
    x = x.reshape(-1, heads, dh)
    a, b = x[..., :half], x[..., half:]
    return torch.cat([a * c - b * s, b * c + a * s], -1).reshape(x.shape[0], heads * dh)


def _forward(case, w, cached, length, tokens, parents=None):
    """64-bit hidden rows before the LM head, and the new (k, v) of every layer as the cache stores them."""
    d, heads, dh, ffn, vocab, kv_heads, dtype = WIDTHS[case["width"]]
    store = (lambda t: t.to(torch.bfloat16).double()) if dtype == "bf16" else (lambda t: t.float().double())
    n, group = len(tokens), heads // kv_heads
    own = torch.ones(n, n, dtype=torch.bool, device="cuda").tril()
    depth = list(range(n))
    if parents is not None:
        sees = np.zeros((n, n), dtype=bool)
        for r, p in enumerate(parents):
            depth[r] = 0 if p < 0 else depth[p] + 1
            if p >= 0:
                sees[r] = sees[p]
            sees[r, r] = True
        own = torch.from_numpy(sees).cuda()
    mask = torch.cat([torch.ones(n, length, dtype=torch.bool, device="cuda"), own], 1)
    pos = torch.tensor(depth, device="cuda") + length
    x = w["embed"][torch.tensor(tokens, device="cuda")].double()
    new = []
    for l in range(case["layers"]):
        h = _norm(x, w["attn_norm"][l])
        q = _rope(h @ w["wq"][l].double().t(), pos, heads, dh)
        k = store(_rope(h @ w["wk"][l].double().t(), pos, kv_heads, dh))
        v = store(h @ w["wv"][l].double().t())
        new.append((k, v))
        ks = torch.cat([cached[l][0].double(), k]) if length else k
        vs = torch.cat([cached[l][1].double(), v]) if length else v
        att = torch.empty_like(q)
        for i in range(heads):
            j = i // group
            s = q[:, i * dh:(i + 1) * dh] @ ks[:, j * dh:(j + 1) * dh].t().contiguous() / math.sqrt(dh)
            s = torch.softmax(s.masked_fill(~mask, -math.inf), -1)
            att[:, i * dh:(i + 1) * dh] = s @ vs[:, j * dh:(j + 1) * dh].contiguous()
        x = x + att @ w["wo"][l].double().t()
        h = _norm(x, w["ffn_norm"][l])
        g = h @ w["w_gate"][l].double().t()
        x = x + (g * torch.sigmoid(g) * (h @ w["w_up"][l].double().t())) @ w["w_down"][l].double().t()
    return _norm(x, w["final_norm"]), new


def exact(case, seed):
    if case["kind"] == "linear":
        x, w = _linear_inputs(case, seed)
        return x.double() @ w.double().t()
    w, caches, tokens = _inputs(case, seed)
    parents = _tree(case) if case["kind"] == "tree" else None
    head, rows, new = w["lm_head"].double().t(), [], None
    for (length, cached), ids in zip(caches, tokens):
        h, new = _forward(case, w, cached, length, ids, parents)
        rows.append(h[-1:] if case["kind"] == "prompt" else h)
    out = {"logits": torch.cat(rows) @ head}
    if case["kind"] == "prompt":
        if case["export"]:
            out["kv"] = new
    else:
        out["accepted"] = None
    return out
