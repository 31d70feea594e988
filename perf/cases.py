"""The work this library is used for, as cases that can be timed and compared: zeroth-order steps, blocks and passes
through the public binding, over the range of model shapes, batch sizes, storage types and schedules it serves.

listed() names the cases, draw() makes more of the same ranges, prepare() builds what a program has in hand before the
call, run() is one pass, work() what the pass cannot do without, tolerance() how far another correct implementation may
be off, exact() the same outputs in 64 bits from plain torch.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2409_15520_amd as M
import workloads as W

# Decoder shapes: (norm / position / activation family, d_model, heads, key-value heads, d_ffn, vocabulary).  The first
# five are this repository's workloads; the last two are widths between them.
SHAPES = {
    "tiny": ("opt-gelu", 128, 4, 4, 512, 512),
    "125m": ("opt", 768, 12, 12, 3072, 50272),
    "1b3": ("opt", 2048, 32, 32, 8192, 50272),
    "1b1": ("llama", 2048, 32, 4, 5632, 32000),
    "7b": ("llama", 4096, 32, 32, 11008, 32000),
    "w1024": ("llama", 1024, 16, 8, 2816, 32000),
    "w2560": ("opt", 2560, 20, 20, 6912, 32000),
}


def _case(name, kind, shape, layers, q, E, S, dtype="bf16", quant="none", rank=16, targets="qv",
          loss="last_pos_label_subset", eps=1e-3):
    c = dict(kind=kind, shape=shape, layers=layers, q=q, E=E, S=S, dtype=dtype, quant=quant, rank=rank, targets=targets,
             loss=loss, eps=eps)
    return dict(name=name, **c) if name else c


def listed():
    return [
        # a whole step of the smallest model: fp32 weights, exact arithmetic, a call whose time is launches and latency
        _case("step_tiny_f32", "step", "tiny", 2, 2, 2, 32, dtype="f32", rank=4),
        # a whole step of the 125M-shaped model with its two-way label loss: every kernel lasts tens of microseconds
        _case("step_125m", "step", "125m", 12, 4, 8, 128, rank=8, eps=1e-2),
        # a whole step of the 1.1B-shaped model, 65536 stacked tokens, adapters on all four projections, next-token
        # loss over the whole vocabulary: the largest call
        _case("step_1b1", "step", "1b1", 22, 16, 4, 512, targets="qkvo", loss="next_token_all_pos", eps=1e-2),
        # embedding and one decoder block of the 7B-shaped model at its step's 8192 stacked tokens
        _case("block_7b", "block", "7b", 1, 4, 2, 512),
        # one block, final norm, 50272-wide head and next-token loss of the 1.3B-shaped model
        _case("block_head_1b3", "block_head", "1b3", 1, 8, 8, 256, rank=8, loss="next_token_all_pos"),
        # one query on one short sequence through two 7B-shaped blocks: bound by reading the weights
        _case("fewtok_7b", "block", "7b", 2, 1, 1, 64),
        # the same regime with 4-bit weights
        _case("fewtok_7b_nf4", "block", "7b", 2, 1, 1, 96, quant="nf4"),
        # int8 weights at an ordinary batch: 1024 stacked tokens
        _case("block_7b_int8", "block", "7b", 1, 2, 1, 256, quant="int8"),
        # sequences whose length is no multiple of anything, right as a user's data comes
        _case("block_1b1_odd", "block", "1b1", 1, 4, 3, 77, targets="qkvo"),
        # unequal sequences packed back to back, two 1.1B-shaped blocks and the next-token loss
        _case("packed_1b1", "packed", "1b1", 2, 8, 8, 384, targets="qkvo", loss="next_token_all_pos", eps=1e-2),
        # one forward pass per perturbed copy (the sequential schedule the batched pass is compared with), 125M shape
        _case("sequential_125m", "sequential", "125m", 12, 2, 4, 128, rank=8, loss="next_token_all_pos", eps=1e-2),
        # an fp32 block at the 125M widths
        _case("block_125m_f32", "block", "125m", 1, 2, 2, 96, dtype="f32", rank=8),
    ]


def _loguniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        kind = rng.choice(["block", "block", "block", "block", "block_head", "step", "packed", "sequential", "block_f32"])
        S = _loguniform(rng, 16, 512)
        if rng.random() < 0.6:                            # most batches are padded to a multiple of 32 or 64
            S = max(32, S // 32 * 32)
        q, E = _loguniform(rng, 1, 16), _loguniform(rng, 1, 8)
        if kind == "block_f32":
            c = _case(None, "block", rng.choice(["tiny", "125m"]), 1, min(q, 4), min(E, 2), min(S, 128), dtype="f32",
                      rank=rng.choice([4, 8]))
        else:
            shape = rng.choice(["125m", "1b3", "1b1", "7b", "w1024", "w2560"])
            if kind != "block":
                shape = rng.choice(["125m", "1b1", "w1024"])
            layers = {"block": 1, "block_head": 1, "step": 4, "packed": 2, "sequential": 4}[kind]
            quant = rng.choice(["none", "none", "int8", "nf4"]) if kind == "block" else "none"
            if quant == "int8":
                S = max(32, S // 32 * 32)                 # int8 weights take whole 32-row tiles per copy
            if kind == "packed":
                S = max(64, S)
            c = _case(None, kind, shape, layers, q, E, S, quant=quant, rank=rng.choice([8, 16]),
                      targets=rng.choice(["qv", "qkvo"]),
                      loss="last_pos_label_subset" if kind == "block" else "next_token_all_pos",
                      eps=1e-2 if kind in ("step", "packed", "sequential") else 1e-3)
        ragged = (c["E"] * c["S"]) % 32 != 0
        if 32 <= 2 * c["q"] * c["E"] * c["S"] and work(c)["flops"] <= (1e12 if ragged else 4e12):
            return c


def _workload(c):
    family, d, heads, kv, ffn, vocab = SHAPES[c["shape"]]
    llama = family == "llama"
    return W.Workload(
        name=c["kind"], n_layers=c["layers"], d_model=d, n_heads=heads, n_kv_heads=kv, d_ffn=ffn, vocab=vocab,
        max_seq=max(64, c["S"]), act="swiglu" if llama else "gelu" if family == "opt-gelu" else "relu",
        norm="rmsnorm" if llama else "layernorm", pos="rope" if llama else "learned", has_bias=not llama,
        tie_embeddings=not llama, dtype=c["dtype"], lora_rank=c["rank"], lora_targets=tuple(c["targets"]),
        loss_mode=c["loss"], q=c["q"], E=c["E"], S=c["S"], steps=1, eps=c["eps"], lr=1e-3,
        label_tokens=(vocab // 7, vocab // 3), weight_quant=c["quant"])


def _inputs(c, seed):
    """Everything made from the seed: weights on the device, adapters half-way through training (B drawn as A is),
    tokens, labels, and for packed batches the sequence lengths."""
    w = _workload(c)
    frozen = M.device_random_weights(w, 1000 + seed)
    masters = W.make_lora_masters(w, 2000 + seed, b_std=0.02)
    tokens = torch.from_numpy(W.make_tokens(w, 3000 + seed)).cuda()
    labels = torch.from_numpy(W.make_labels(w, 3000 + seed)).cuda()
    lengths = W.make_lengths(w, 3000 + seed) if c["kind"] == "packed" else None
    return w, frozen, masters, tokens, labels, lengths


def prepare(case, seed):
    w, frozen, masters, tokens, labels, lengths = _inputs(case, seed)
    model = M.ZoModel(w, frozen, masters)
    state = dict(kind=case["kind"], model=model, tokens=tokens, labels=labels, E=case["E"], S=case["S"],
                 layers=case["layers"], seed=4000 + seed, step=0)
    if case["kind"] == "packed":
        state["batch"] = model.pack_batch(tokens, torch.from_numpy(lengths).cuda())
    if case["kind"] != "step":
        model.regen_noise(state["seed"], 0)               # a step draws its noise itself
    return state


def run(state):
    m, kind = state["model"], state["kind"]
    if kind == "step":                                     # noise, batched pass, update
        m.zo_step(state["tokens"], state["labels"], state["seed"], state["step"])
        state["step"] += 1
        return {"losses": m.losses[:2 * m.q], "masters": m.masters}
    if kind == "packed":
        return {"losses": m.forward_packed(state["batch"], state["labels"])}
    if kind == "sequential":
        return {"losses": m.forward_sequential(state["tokens"], state["labels"])}
    h = m.run_layers(m.embed(state["tokens"]), 0, state["layers"], state["E"], state["S"])
    if kind == "block":
        return {"h": h}
    return {"h": h, "losses": m.head_loss(h, state["tokens"], state["labels"])}


def _tokens_per_copy(c):
    if c["kind"] != "packed":
        return c["E"] * c["S"]
    return int(c["E"] * c["S"] * 0.7)                       # the mean of make_lengths


def work(case):
    family, d, heads, kv, ffn, vocab = SHAPES[case["shape"]]
    llama, n, L = family == "llama", 2 * case["q"], case["layers"]
    dkv, wb = kv * (d // heads), 4.0 if case["dtype"] == "f32" else 2.0
    lin_b = {"none": wb, "int8": 1.0, "nf4": 0.5 + 4.0 / 64}[case["quant"]]
    per_layer = d * (d + 2 * dkv) + d * d + (2 if llama else 1) * d * ffn + ffn * d
    tpc, T = _tokens_per_copy(case), n * _tokens_per_copy(case)
    S = case["S"]
    lora = sum(case["rank"] * (d + (dkv if t in "kv" else d)) for t in case["targets"])
    flops = 2.0 * T * L * (per_layer + lora) + 2.0 * T * (S + 1) * d * L
    copies_read = n if case["kind"] == "sequential" else 1
    nbytes = L * per_layer * lin_b * copies_read + 4.0 * L * lora + 4.0 * tpc + wb * min(tpc, vocab) * d
    if case["kind"] in ("block", "block_head"):
        nbytes += 4.0 * T * d                              # the residual rows that come back
    if case["loss"] == "next_token_all_pos" and case["kind"] != "block":
        flops += 2.0 * T * d * vocab
        nbytes += wb * vocab * d * copies_read
    if case["kind"] == "step":
        nbytes += 4.0 * L * lora                           # the masters are written back
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # four times what was seen against exact() over several seeds, and between the one-block and the split-K sums
    if case["dtype"] == "f32":                             # fp32 storage, 64-bit sums: rounding of stored values alone
        if case["kind"] == "step":                         # two-point differences of rounded losses: masters 8e-7
            return {"rel": 4e-6, "max": 1e-4}
        return {"rel": 5e-7, "max": 2e-5}
    if case["kind"] == "step" and case["loss"] == "last_pos_label_subset":
        return {"rel": 5e-3, "max": 5e-2}                  # losses 3e-4 to 8e-4, masters 3e-4 to 1.4e-3
    if case["kind"] in ("step", "packed", "sequential"):
        return {"rel": 1e-3, "max": 1e-2}                  # losses 5e-6 to 3e-5, masters 7e-5 to 2.8e-4
    return {"rel": 1.6e-2, "max": 0.15}                    # bf16 roundings of one or two blocks: 4e-3, largest 2.2e-2


# ---- the same outputs in 64 bits ---------------------------------------------------------------------------------
def _philox(j, tensor_id, step, k, seed):
    """Philox4x32-10 words of counters (j, tensor_id, step, k), key = the two halves of the seed (int64 arithmetic)."""
    mask = 0xFFFFFFFF
    c = [j.clone(), torch.full_like(j, tensor_id), torch.full_like(j, step), torch.full_like(j, k)]
    k0, k1 = seed & mask, (seed >> 32) & mask
    for _ in range(10):
        p0, p1 = c[0] * 0xD2511F53, c[2] * 0xCD9E8D57
        c = [((p1 >> 32) & mask) ^ c[1] ^ k0, p1 & mask, ((p0 >> 32) & mask) ^ c[3] ^ k1, p0 & mask]
        k0, k1 = (k0 + 0x9E3779B9) & mask, (k1 + 0xBB67AE85) & mask
    return c


def _normals(numel, tensor_id, step, k, seed):
    x = _philox(torch.arange(numel // 4, device="cuda"), tensor_id, step, k, seed)
    u = [((v >> 9).double() + 0.5) * 2.0 ** -23 for v in x]
    z = []
    for a, b in ((u[0], u[1]), (u[2], u[3])):
        rho = torch.sqrt(-2.0 * torch.log(a))
        z += [rho * torch.cos(2 * math.pi * b), rho * torch.sin(2 * math.pi * b)]
    return torch.stack(z, 1).reshape(-1)


_NF4 = (-1.0, -0.6961928009986877, -0.5250730514526367, -0.39491748809814453, -0.28444138169288635, -0.18477343022823334,
        -0.09105003625154495, 0.0, 0.07958029955625534, 0.16093020141124725, 0.24611230194568634, 0.33791524171829224,
        0.44070982933044434, 0.5626170039176941, 0.7229568362236023, 1.0)


def _dense(w, scale, quant):
    if quant == "none":
        return w.double()
    if quant == "int8":
        return w.double() * scale.double()[:, None]
    levels = torch.tensor(_NF4, dtype=torch.float32, device=w.device)
    codes = torch.stack([w & 15, w >> 4], -1).reshape(w.shape[0], -1).long()
    block = levels[codes].reshape(w.shape[0], -1, 64) * scale[:, :, None]
    return block.to(torch.bfloat16).double().reshape(w.shape[0], -1)       # the format's weight is its bf16 value


def _norm(x, g, b, w):
    if w.norm == "layernorm":
        x = x - x.mean(-1, keepdim=True)
    y = x / torch.sqrt((x * x).mean(-1, keepdim=True) + float(np.float32(w.norm_eps))) * g.double()
    return y if b is None else y + b.double()


def _attention(q, k, v, scale):
    """[E, H, S, dh] causal."""
    S = q.shape[2]
    s = torch.matmul(q, k.transpose(2, 3).contiguous()) * scale
    s = s.masked_fill(torch.ones(S, S, dtype=torch.bool, device=q.device).triu(1), -math.inf)
    return torch.matmul(torch.softmax(s, -1), v)


def _copies(c, w, masters, seed, step):
    lay = W.lora_layout(w)
    theta = torch.from_numpy(masters).cuda().double()
    eps = float(np.float32(w.eps))
    zs = [torch.cat([_normals(t.rows * t.cols, t.tensor_id, step, k, seed) for t in lay]) for k in range(w.q)]
    return lay, theta, zs, eps


def exact(case, seed):
    if case["kind"] == "step" and case["loss"] == "last_pos_label_subset" and case["dtype"] == "bf16":
        # two logits at one position per sequence: the error of such a loss is one draw of the rounding noise (3e-4 to
        # 8e-4 over four seeds with the same code) and says nothing about the precision of the arithmetic
        return None
    w, frozen, masters, tokens, labels, lengths = _inputs(case, seed)
    nseed, step = 4000 + seed, 0
    lay, theta, zs, eps = _copies(case, w, masters, nseed, step)
    n, E, S, d, dkv, H, dh = 2 * w.q, w.E, w.S, w.d_model, w.d_kv, w.n_heads, w.d_head
    tok = tokens.long()
    h0 = frozen["emb"].double()[tok.reshape(-1)].reshape(E, S, d)
    if w.pos == "learned":
        h0 = h0 + frozen["pos_emb"].double()[:S]
    else:
        half = dh // 2
        ang = torch.arange(S, device="cuda").double()[:, None] * \
            torch.pow(torch.tensor(float(np.float32(w.rope_theta)), dtype=torch.float64, device="cuda"),
                      -2.0 * torch.arange(half, device="cuda").double() / dh)
        cos, sin = torch.cos(ang)[None, :, None, :], torch.sin(ang)[None, :, None, :]

    def rotate(x):                                         # [E, S, heads, dh]
        lo, hi = x[..., :dh // 2], x[..., dh // 2:]
        return torch.cat([lo * cos - hi * sin, hi * cos + lo * sin], -1)

    h = [h0.clone() for _ in range(n)]
    for l in range(w.n_layers):
        lw = frozen["layers"][l]
        dense = {k: _dense(lw["w_" + k], lw.get("s_" + k), w.weight_quant) for k in ("qkv", "o", "up", "down")}
        bias = {k: None if lw["b_" + k] is None else lw["b_" + k].double() for k in dense}
        factors = [t for t in lay if t.layer == l]

        def lin(x, k):
            y = torch.matmul(x.reshape(E * S, -1), dense[k].t()).reshape(E, S, -1)
            return y if bias[k] is None else y + bias[k]

        for c in range(n):
            th = theta + (eps if c % 2 == 0 else -eps) * zs[c // 2]
            ab = {(t.target, t.factor): th[t.offset:t.offset + t.rows * t.cols].reshape(t.rows, t.cols) for t in factors}

            def low_rank(x, target):
                if (target, 0) not in ab:
                    return 0.0
                return torch.matmul(torch.matmul(x, ab[target, 0]), ab[target, 1]) * float(np.float32(w.lora_scale))

            x = _norm(h[c], lw["ln1_g"], lw["ln1_b"], w)
            y = lin(x, "qkv")
            q = (y[..., :d] + low_rank(x, 0)).reshape(E, S, H, dh)
            k = (y[..., d:d + dkv] + low_rank(x, 1)).reshape(E, S, w.n_kv_heads, dh)
            v = (y[..., d + dkv:] + low_rank(x, 2)).reshape(E, S, w.n_kv_heads, dh)
            if w.pos == "rope":
                q, k = rotate(q), rotate(k)
            rep = H // w.n_kv_heads
            k, v = (t.repeat_interleave(rep, 2).transpose(1, 2).contiguous() for t in (k, v))
            a = _attention(q.transpose(1, 2).contiguous(), k, v, 1.0 / math.sqrt(dh)).transpose(1, 2).reshape(E, S, d)
            h[c] = h[c] + lin(a, "o") + low_rank(a, 3)
            x = _norm(h[c], lw["ln2_g"], lw["ln2_b"], w)
            y = lin(x, "up")
            if w.act == "swiglu":
                f = w.d_ffn
                u = torch.nn.functional.silu(y[..., :f]) * y[..., f:]
            elif w.act == "gelu":
                u = 0.5 * y * (1.0 + torch.erf(y / math.sqrt(2.0)))
            else:
                u = torch.relu(y)
            h[c] = h[c] + lin(u, "down")
    out_h = torch.cat([x.reshape(E * S, d) for x in h])
    if case["kind"] == "block":
        return {"h": out_h}
    lens = np.full(E, S) if lengths is None else lengths
    head = frozen["lm_head"].double()
    losses = []
    for c in range(n):
        x = _norm(h[c], frozen["lnf_g"], frozen["lnf_b"], w)
        ce = []
        for e in range(E):
            if w.loss_mode == "next_token_all_pos":
                lg = torch.matmul(x[e, :int(lens[e]) - 1], head.t())
                tg = tok[e, 1:int(lens[e])]
            else:
                lg = torch.matmul(x[e, int(lens[e]) - 1:int(lens[e])], head[list(w.label_tokens)].t())
                tg = labels[e:e + 1].long()
            ce.append(torch.logsumexp(lg, -1) - lg.gather(1, tg[:, None])[:, 0])
        losses.append(torch.cat(ce).mean())
    losses = torch.stack(losses)
    if case["kind"] == "block_head":
        return {"h": out_h, "losses": losses}
    if case["kind"] != "step":
        return {"losses": losses}
    g = (losses[0::2] - losses[1::2]) / (2 * eps)
    update = sum(float(np.float32(w.lr)) * g[k] / w.q * zs[k] for k in range(w.q))
    return {"losses": losses, "masters": theta - update}
