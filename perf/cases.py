"""Workloads whose time is measured: what a user of the library calls, over the range of sizes it is called with.

A case is a dict of plain values; `kind` says which calls one pass makes:

  forward   one forward pass over `segments` segments (batch 1), diagonal, sequential or automatic order,
            from the empty memory or from a carried-in state
  batched   the same for `batch` independent sequences
  prompt    token ids -> embeddings -> forward -> logits of the last `rows` positions
  train     forward with tape + backward: gradients of all weights, memory-token embeddings and token embeddings
  head      final norm + head on `rows` rows, and its backward from an upstream gradient of the logits

`model` names one of the repository's shapes (armt_synth.CONFIGS); `seg_len` and `n_mem` replace its segmentation."""
from __future__ import annotations

import math

import torch
import torch.utils.checkpoint

import armt_synth as S
import paper_2506_05229_amd as P

# models of the repository's shape table: their widths and depth; segmentation and length come from the case
MODELS = {"tiny": "tiny", "160m": "160m_128k", "1b": "1b_128k", "3b": "3b_128k"}


def listed():
    return [
        # the fp32 correctness configuration of the repository: the smallest calls, where launches and latency count
        dict(name="tiny_f32", kind="forward", model="tiny", seg_len=64, n_mem=8, segments=8, order="diagonal", carry=False),
        dict(name="tiny_f32_train", kind="train", model="tiny", seg_len=64, n_mem=8, segments=8, batch=1),
        # a stream that arrives segment by segment: one more segment on top of the state so far, one cell at a time
        dict(name="1b_stream_1k", kind="forward", model="1b", seg_len=1024, n_mem=16, segments=1, order="auto", carry=True),
        # a short prompt up to the logits of the next token: the groups at both ends of the schedule weigh most
        dict(name="1b_prompt_8k", kind="prompt", model="1b", seg_len=1024, n_mem=16, segments=8, rows=1),
        # several requests at once, segment length not a multiple of any tile
        dict(name="1b_batch3_ragged", kind="batched", model="1b", seg_len=1000, n_mem=16, segments=4, batch=3, order="diagonal"),
        # short segments: more, smaller cells
        dict(name="1b_32k_s512", kind="forward", model="1b", seg_len=512, n_mem=16, segments=64, order="diagonal", carry=False),
        # the timing-table segmentation of the paper: long segments, many memory tokens
        dict(name="1b_16k_s4096_m128", kind="forward", model="1b", seg_len=4096, n_mem=128, segments=4, order="diagonal", carry=False),
        # small and large model
        dict(name="160m_32k", kind="forward", model="160m", seg_len=1024, n_mem=16, segments=32, order="diagonal", carry=False),
        dict(name="3b_16k", kind="forward", model="3b", seg_len=1024, n_mem=16, segments=16, order="diagonal", carry=False),
        # the benchmark's long input
        dict(name="1b_128k", kind="forward", model="1b", seg_len=1024, n_mem=16, segments=128, order="diagonal", carry=False),
        # training: forward with tape and backward; head and its backward on one step's worth of rows
        dict(name="1b_train_8k", kind="train", model="1b", seg_len=1024, n_mem=16, segments=8, batch=1),
        dict(name="head_train_4k", kind="head", model="1b", seg_len=1024, n_mem=16, rows=4096, vocab=S.LLAMA3_VOCAB),
    ]


def _log_int(rng, lo, hi):
    """An integer spread evenly over the logarithm of [lo, hi]."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case of the same ranges; costs at most what the longest listed one does."""
    kind = rng.choice(["forward"] * 5 + ["batched", "prompt", "train", "train", "head"])
    if kind == "head":
        return dict(kind="head", model=rng.choice(["160m", "1b", "3b"]), seg_len=1024, n_mem=16, rows=_log_int(rng, 64, 6000),
                    vocab=_log_int(rng, 8000, S.LLAMA3_VOCAB))
    model = rng.choice(["tiny", "160m", "1b", "1b", "1b", "3b"])
    if model == "tiny":
        seg_len, n_mem, most = _log_int(rng, 24, 300), rng.choice([4, 8, 16]), 64
    else:
        seg_len = rng.choice([512, 1024, 2048, _log_int(rng, 200, 3000)])
        n_mem = rng.choice([16, 16, 16, 32, 128])
        # forward-equivalents of the longest listed case: 131072 tokens of the 1B model
        cost = {"160m": 0.25, "1b": 1.0, "3b": 3.0}[model]
        most = max(2, int(100000 / (cost * (seg_len + n_mem))))
    if kind == "train":
        # the gradients' workspace grows with the rows of a cell: cells of at most about 1100 rows, two sequences
        if model != "tiny":
            seg_len, n_mem = min(seg_len, _log_int(rng, 256, 1040)), rng.choice([16, 32])
            most = max(2, int(16000 / (cost * (seg_len + n_mem))))
        batch = 1 if model == "3b" else rng.choice([1, 1, 2])
        return dict(kind="train", model=model, seg_len=seg_len, n_mem=n_mem, segments=_log_int(rng, 2, min(32, max(2, most // batch))),
                    batch=batch)
    if kind == "batched":
        batch = rng.randint(2, 6)
        return dict(kind="batched", model=model, seg_len=seg_len, n_mem=n_mem, segments=_log_int(rng, 1, max(2, min(32, most // batch))),
                    batch=batch, order=rng.choice(["diagonal", "diagonal", "sequential"]))
    if kind == "prompt":
        model = "1b" if model in ("tiny", "3b") else model
        seg_len, n_mem = max(200, seg_len), max(16, n_mem)
        return dict(kind="prompt", model=model, seg_len=seg_len, n_mem=n_mem, segments=_log_int(rng, 1, 16), rows=_log_int(rng, 1, 128))
    order = rng.choice(["diagonal", "diagonal", "diagonal", "auto", "sequential"])
    most = min(most, 128)
    if order == "sequential":       # one cell per launch: slower per token than the diagonal order
        most = max(1, most // 6)
    return dict(kind="forward", model=model, seg_len=seg_len, n_mem=n_mem, segments=_log_int(rng, 1, most), order=order,
                carry=rng.random() < 0.4)


def _shape(case):
    base = S.get_shape(MODELS[case["model"]])
    kw = dict(name=case["kind"] + "_" + case["model"], seg_len=case["seg_len"], n_mem=case["n_mem"],
              n_tokens=case["seg_len"] * case.get("segments", 1))
    if case["model"] != "tiny":
        # keys written together are positively correlated and make the recurrence of the memory diverge when |phi(k)|^2
        # exceeds assoc_eps a few times: two powers of two below the scale found for 16 memory tokens, more for more tokens
        kw["mem_k_scale"] = base.mem_k_scale / 4 * min(1.0, 16 / case["n_mem"])
    return base.replace(**kw)


def _dims(s):
    d, H, Hkv, dh, F, dm = s.d_model, s.n_heads, s.n_kv_heads, s.head_dim, s.d_ff, s.d_mem
    return {"rms1": (d,), "wq": (H * dh, d), "wk": (Hkv * dh, d), "wv": (Hkv * dh, d), "wo": (d, H * dh), "rms2": (d,),
            "wgate": (F, d), "wup": (F, d), "wdown": (d, F), "wm_q": (dm, d), "wm_k": (dm, d), "wm_v": (d, d), "wm_b": (1, d)}


def _drawer(seed, dt):
    gen = torch.Generator(device="cuda").manual_seed(int(seed))

    def normal(dims, std=1.0, mean=0.0, dtype=dt):
        return torch.randn(dims, generator=gen, device="cuda", dtype=torch.float32).mul_(std).add_(mean).to(dtype)

    return gen, normal


def _ends(case, shape, normal):
    """Embedding table (prompts only), final gain and head weight."""
    vocab = case.get("vocab", S.LLAMA3_VOCAB)
    table = normal((vocab, shape.d_model)) if case["kind"] == "prompt" else None
    return table, normal((shape.d_model,), 0.1, 1.0), normal((vocab, shape.d_model), 0.02)


def _head_inputs(case, shape, normal):
    """Hidden states and the gradient of a mean loss over the rows."""
    return normal((case["rows"], shape.d_model), 3.0), normal((case["rows"], case["vocab"]), 1.0 / case["rows"], dtype=torch.float32)


def _weights(shape, normal):
    layers = []
    for _ in range(shape.n_layers):
        lw = {}
        for f, dims in _dims(shape).items():
            scale = {"wm_k": shape.mem_k_scale, "wm_v": shape.mem_v_scale}.get(f, 1.0)
            lw[f] = normal(dims, 0.1, 1.0) if f.startswith("rms") else normal(dims, 0.02 * scale)
        layers.append(lw)
    return layers, normal((shape.n_mem, shape.d_model), 0.02)


def _sequences(case, shape, normal):
    """Token embeddings; for a carried-in state also the three segments in front of them."""
    B = case.get("batch", 1)
    lead = (B,) if case["kind"] == "batched" or B > 1 else ()
    x = normal(lead + (shape.n_tokens, shape.d_model))
    first = normal((3 * shape.seg_len, shape.d_model)) if case.get("carry") else None
    return x, first, normal(lead + (shape.n_tokens, shape.d_model)) if case["kind"] == "train" else None


def _act_type(shape):
    return torch.bfloat16 if shape.dtype == "bf16" else torch.float32


def prepare(case, seed):
    """Inputs and the model a user's program holds: weights ~ N(0, 0.02^2), gains ~ N(1, 0.1^2), embeddings ~ N(0, 1)."""
    shape = _shape(case)
    gen, normal = _drawer(seed, _act_type(shape))
    st = {"kind": case["kind"], "case": dict(case), "shape": shape}
    if case["kind"] in ("prompt", "head"):
        table, gain, w_lm = _ends(case, shape, normal)
        if table is None:
            table = torch.zeros((1, shape.d_model), dtype=_act_type(shape), device="cuda")
        st["ends"] = P.TokenEnds(shape, table, gain, w_lm)
        if case["kind"] == "head":
            st["hidden"], st["d_logits"] = _head_inputs(case, shape, normal)
            st["grads"] = (torch.zeros(shape.d_model, device="cuda"), torch.zeros((case["vocab"], shape.d_model), device="cuda"))
            return st
        st["ids"] = torch.randint(0, S.LLAMA3_VOCAB, (shape.n_tokens,), generator=gen, device="cuda", dtype=torch.int32)
    layers, mem_emb = _weights(shape, normal)
    st["model"] = P.Armt(shape, layers, mem_emb)
    if case["kind"] == "prompt":
        return st
    st["x"], first, d_hidden = _sequences(case, shape, normal)
    if first is not None:
        # a state as earlier segments leave it: the state after three other segments (one pass of the library itself)
        _, st["A"], st["z"] = st["model"].forward(first, diagonal=True)
    if case["kind"] == "train":
        st["d_hidden"] = d_hidden
        # one buffer per kind of weight over the layers, as an optimizer that works on flat parameters keeps them
        st["flat"] = {f: torch.zeros((shape.n_layers,) + dims, device="cuda") for f, dims in _dims(shape).items()}
        st["d_mem_emb"] = torch.zeros((shape.n_mem, shape.d_model), device="cuda")
    return st


def run(st):
    """One pass through the public entry points."""
    kind, case = st["kind"], st["case"]
    if kind == "forward":
        order = {"diagonal": True, "sequential": False, "auto": "auto"}[case["order"]]
        return st["model"].forward(st["x"], diagonal=order, A_in=st.get("A"), z_in=st.get("z"))
    if kind == "batched":
        return st["model"].forward_batched(st["x"], diagonal=case["order"] == "diagonal")
    if kind == "prompt":
        x = st["ends"].embed(st["ids"])
        hidden, A, z = st["model"].forward(x, diagonal="auto")
        return hidden, A, z, st["ends"].logits(hidden[-case["rows"]:])
    if kind == "head":
        ends, (d_gain, d_w) = st["ends"], st["grads"]
        logits = ends.logits(st["hidden"])
        d_gain.zero_()
        d_w.zero_()
        return logits, ends.logits_backward(st["hidden"], st["d_logits"], grads=(d_gain, d_w))
    model, shape = st["model"], st["shape"]
    for t in st["flat"].values():
        t.zero_()
    st["d_mem_emb"].zero_()
    hidden, A, z, tape = model.forward_train(st["x"])
    grads = {"layers": [{f: t[l] for f, t in st["flat"].items()} for l in range(shape.n_layers)], "mem_emb": st["d_mem_emb"]}
    out = model.backward(tape, shape.n_tokens, st["d_hidden"], grads=grads)
    return hidden, A, z, st["flat"], out["mem_emb"], out["x"]


# ---- the same passes from the definition, in 64 bits

def _norm64(x, gain, eps):
    return x * torch.rsqrt((x * x).mean(-1, keepdim=True) + eps) * gain


def _dpfp64(k, nu):
    r = torch.cat([k.clamp_min(0), (-k).clamp_min(0)], -1)
    return torch.cat([r * r.roll(j, -1) for j in range(1, nu + 1)], -1)


def _attention64(q, k, v):
    """Causal, grouped heads; q [T, H, dh], a block of query rows at a time."""
    T, H, dh = q.shape
    k, v = (t.repeat_interleave(H // t.shape[1], 1).transpose(0, 1).contiguous() for t in (k, v))
    rows = max(64, int(2 ** 27 / (H * T)))
    out = []
    for i in range(0, T, rows):
        e = min(T, i + rows)
        score = torch.matmul(q[i:e].transpose(0, 1), k[:, :e].transpose(1, 2).contiguous()) / math.sqrt(dh)
        ahead = torch.arange(e, device=q.device)[None, :] > torch.arange(i, e, device=q.device)[:, None]
        out.append(torch.matmul(score.masked_fill_(ahead, float("-inf")).softmax(-1), v[:, :e]).transpose(0, 1))
    return torch.cat(out).reshape(T, H * dh)


def _cell64(s, w, x, A, z, empty):
    """One (layer, segment) cell: read, decoder block, delta-rule update.  Returns (output rows, A, z)."""
    T, H, G, dh = x.shape[0], s.n_heads, s.n_kv_heads, s.head_dim
    w = {f: t.double() for f, t in w.items()}
    if not empty:
        f = _dpfp64(x @ w["wm_q"].T, s.dpfp_nu)
        x = x + (f @ A.T) / (f @ z + s.assoc_eps)[:, None]
    n = _norm64(x, w["rms1"], s.rms_eps)
    at = torch.arange(T, device=x.device, dtype=torch.float64)[:, None]
    angle = at * float(s.rope_theta) ** (-2.0 * torch.arange(dh // 2, device=x.device, dtype=torch.float64) / dh)
    cos, sin = angle.cos()[:, None], angle.sin()[:, None]

    def rotated(t):
        a, b = t[..., :dh // 2], t[..., dh // 2:]
        return torch.cat([a * cos - b * sin, b * cos + a * sin], -1)

    q, k, v = ((n @ w[f].T).reshape(T, heads, dh) for f, heads in (("wq", H), ("wk", G), ("wv", G)))
    x = x + _attention64(rotated(q), rotated(k), v) @ w["wo"].T
    n = _norm64(x, w["rms2"], s.rms_eps)
    x = x + (torch.nn.functional.silu(n @ w["wgate"].T) * (n @ w["wup"].T)) @ w["wdown"].T
    y = x[s.seg_len:]
    f, v = _dpfp64(y @ w["wm_k"].T, s.dpfp_nu), y @ w["wm_v"].T
    zf = f @ z
    old = 0.0 if empty else (f @ A.T) / (zf + s.assoc_eps)[:, None]
    beta = torch.sigmoid(y @ w["wm_b"][0])[:, None]
    return x, A + (beta * (v - old)).T @ f, z + (1.0 - zf / ((f * f).sum(-1) + s.assoc_eps)) @ f


def _forward64(s, layers, mem_emb, x, state=None, recompute=False):
    """(hidden, A [layers], z [layers]); recompute keeps only the cells' inputs for the gradients."""
    dev, empty = x.device, state is None
    A, z = state or ([torch.zeros(s.d_model, s.phi, dtype=torch.float64, device=dev)] * s.n_layers,
                     [torch.zeros(s.phi, dtype=torch.float64, device=dev)] * s.n_layers)
    A, z, hidden = list(A), list(z), []
    for i in range(0, x.shape[0], s.seg_len):
        rows = torch.cat([x[i:i + s.seg_len].double(), mem_emb.double()])
        for l, w in enumerate(layers):
            args = (s, w, rows, A[l], z[l], empty and i == 0)
            rows, A[l], z[l] = torch.utils.checkpoint.checkpoint(_cell64, *args, use_reentrant=False) if recompute else _cell64(*args)
        hidden.append(rows[:s.seg_len])
    return torch.cat(hidden), torch.stack(A), torch.stack(z)


def exact(case, seed):
    """What run() returns, in 64 bits; None where that would take long."""
    s = _shape(case)
    if case["kind"] != "head" and work(case)["flops"] * (4 / 3 if case["kind"] == "train" else 1) > 1.5e14:
        return None
    gen, normal = _drawer(seed, _act_type(s))
    if case["kind"] in ("prompt", "head"):
        table, gain, w_lm = _ends(case, s, normal)
    if case["kind"] == "head":
        hidden, d_logits = _head_inputs(case, s, normal)
        h, g, w = (t.double().requires_grad_() for t in (hidden, gain, w_lm))
        logits = _norm64(h, g, s.rms_eps) @ w.T
        return logits.detach(), torch.autograd.grad(logits, (h, g, w), d_logits.double())
    if case["kind"] == "prompt":
        ids = torch.randint(0, S.LLAMA3_VOCAB, (s.n_tokens,), generator=gen, device="cuda", dtype=torch.int32)
        layers, mem_emb = _weights(s, normal)
        hidden, A, z = _forward64(s, layers, mem_emb, table[ids.long()])
        return hidden, A, z, _norm64(hidden[-case["rows"]:], gain.double(), s.rms_eps) @ w_lm.double().T
    layers, mem_emb = _weights(s, normal)
    x, first, d_hidden = _sequences(case, s, normal)
    if case["kind"] == "forward":
        state = None if first is None else _forward64(s, layers, mem_emb, first)[1:]
        return _forward64(s, layers, mem_emb, x, state)
    if case["kind"] == "batched":
        return tuple(torch.stack(t) for t in zip(*(_forward64(s, layers, mem_emb, xb) for xb in x)))
    layers = [{f: t.double().requires_grad_() for f, t in w.items()} for w in layers]
    mem_emb = mem_emb.double().requires_grad_()
    out, d_x = [], []
    leaves = [mem_emb] + [t for w in layers for t in w.values()]
    sums = [torch.zeros_like(t) for t in leaves]
    for xb, db in zip(x, d_hidden) if x.dim() == 3 else [(x, d_hidden)]:
        xb = xb.double().requires_grad_()
        res = _forward64(s, layers, mem_emb, xb, recompute=True)
        grads = torch.autograd.grad(res[0], leaves + [xb], db.double(), allow_unused=True)
        for total, g in zip(sums, grads):
            if g is not None:
                total += g
        out.append([t.detach() for t in res])
        d_x.append(grads[-1])
    hidden, A, z = (torch.stack(t) if x.dim() == 3 else t[0] for t in zip(*out))
    flat = {f: torch.stack([sums[1 + l * len(w) + i] for l, w in enumerate(layers)]) for i, f in enumerate(layers[0])}
    if s.dtype == "bf16":
        flat["wm_k"] = None     # its denominators are as small as assoc_eps: bf16 operands leave this gradient one digit (0.14 off)
    return hidden, A, z, flat, sums[0], torch.stack(d_x) if x.dim() == 3 else d_x[0]


def work(case):
    """Bytes: weights, inputs, states and results once.  Flops: the products of the definition (causal attention counts the
    lower triangle), times three for a training step."""
    s = _shape(case)
    e = 2 if s.dtype == "bf16" else 4
    if case["kind"] == "head":
        r, v, d = case["rows"], case["vocab"], s.d_model
        return {"bytes": r * d * e + v * d * e + 2 * r * v * 4 + r * d * 4 + v * d * 4, "flops": 3 * 2.0 * r * v * d}
    B = case.get("batch", 1)
    params = s.n_layers * sum(math.prod(dims) for dims in _dims(s).values())
    state = s.n_layers * (s.d_model * s.phi + s.phi) * 4 * B
    tokens = B * s.n_tokens * s.d_model * e
    flops = B * s.flops_total(carry_in=bool(case.get("carry")))
    nbytes = params * e + 2 * tokens + state * (2 if case.get("carry") else 1)
    if case["kind"] == "train":
        return {"bytes": nbytes + params * 4 + tokens + B * s.n_tokens * s.d_model * 4, "flops": 3 * flops}
    if case["kind"] == "prompt":
        flops += 2.0 * case["rows"] * S.LLAMA3_VOCAB * s.d_model
        nbytes += S.LLAMA3_VOCAB * s.d_model * e + case["rows"] * S.LLAMA3_VOCAB * 4
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    if case["model"] == "tiny":
        # fp32 against float64: forward 4e-7 (A), largest element 7e-6; gradients 1.8e-5 (W_Q of the memory), 1e-4
        return {"rel": 7e-5, "max": 4e-4} if case["kind"] == "train" else {"rel": 5e-6, "max": 5e-5}
    if case["kind"] == "head":
        # plain fp32-FMA kernels on the same bf16 operands against the matrix-core path: 6e-6, largest element 4e-5
        return {"rel": 3e-5, "max": 2e-4}
    # the same comparison for a whole model: hidden states 1.2e-2 (1B) and 2.2e-2 (3B), A 5e-2, largest element 0.7; a
    # difference of one bf16 rounding in an early layer reaches all later ones.  Against 64 bits: hidden states 0.8e-2 (1B)
    # and 1.5e-2 (3B), A 3.5e-2 and 6e-2; gradients 1.5e-2 to 7e-2, that of wm_k 0.14.
    return {"rel": 0.25, "max": 0.95} if case["kind"] == "train" else {"rel": 0.1, "max": 0.9}
