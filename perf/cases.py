"""The work that a user of this library has it do, as cases that can be timed and compared.

A case is one call (or one worker's short sequence of calls) through the Python binding of the C ABI: a rollout, a
continuous rollout, a teacher-forced scoring pass, a snapshot install, the learner-side tensors of a batch of records.
Model shapes are the repository's own (config 1's tiny model, the 4B / 8B / 32B decoder widths); all but one are cut to a
few layers, because every layer does the same work and a pass of the whole depth would say nothing more.

Rollouts are teacher-forced (`forced=`): the token that is fed back is given, the sampled token and its log-probability
are returned at every step as in a free-running rollout, by the same kernels.  Free-running sequences differ in everything
that follows the first near-tie which rounding resolves the other way, so two correct runs could not be compared.
"""
import math

import numpy as np
import torch

from paper_2602_02192_amd import echo, synth

_TINY = dict(layers=2, hidden=256, q_heads=4, kv_heads=2, head_dim=64, ffn=704, vocab=1024, dtype="fp32", qk_norm=False, tied=False)
_4B = dict(hidden=2560, q_heads=32, kv_heads=8, head_dim=128, ffn=9728, vocab=151936, dtype="bf16", qk_norm=False, tied=False)
_8B = dict(hidden=4096, q_heads=32, kv_heads=8, head_dim=128, ffn=12288, vocab=151936, dtype="bf16", qk_norm=False, tied=False)
_32B = dict(hidden=5120, q_heads=64, kv_heads=8, head_dim=128, ffn=25600, vocab=151936, dtype="bf16", qk_norm=False, tied=False)


def _rollout(name, model, layers, prompts, group, plen, new, stop_lo=0, top_p=1.0, slots=0, ragged=False, logits=False, temperature=1.0):
    """`group` samples of each of `prompts` prompts of (up to) `plen` tokens, `new` tokens each; stop_lo > 0: per-sequence stop
    lengths between stop_lo and new; slots > 0: the continuous entry point over that many cache slots; logits: the raw
    logits of every step come back as well."""
    c = dict(kind="rollout", prompts=prompts, group=group, plen=plen, new=new, stop_lo=stop_lo, top_p=top_p, slots=slots, ragged=ragged,
             logits=logits, temperature=temperature, **dict(model, layers=layers))
    return dict(c, name=name) if name else c


def _score(name, model, layers, seqs, length, ragged=False, temperature=1.0):
    c = dict(kind="score", seqs=seqs, length=length, ragged=ragged, temperature=temperature, **dict(model, layers=layers))
    return dict(c, name=name) if name else c


def _install(name, model, layers, form, length):
    c = dict(kind="install", form=form, length=length, **dict(model, layers=layers))
    return dict(c, name=name) if name else c


def _grpo(name, records, stride, group, per_token=True):
    c = dict(kind="grpo", records=records, stride=stride, group=group, per_token=per_token)
    return dict(c, name=name) if name else c


def listed():
    return [
        # config 1: the all-fp32 model that every other path is checked against; tens of microseconds of work per step
        _rollout("tiny-fp32-8x16+32", _TINY, 2, 4, 2, 16, 32),
        # one prompt, one answer: an interactive look at a policy; nothing but latency
        _rollout("4b-1x97+48", _4B, 4, 1, 1, 97, 48),
        # the benchmark's workload at its whole depth, fewer generated tokens: the ordinary GRPO rollout
        _rollout("4b-full-64x512+24", _4B, 36, 8, 8, 512, 24),
        # a wide batch that drains: ragged prompts, ragged stop lengths, rows moved together as sequences end
        _rollout("4b-256x512+32-ragged", _4B, 4, 32, 8, 512, 32, stop_lo=6, ragged=True),
        # the paper's sampling setting: 16 samples per prompt, top-p 0.95
        _rollout("8b-128x1024+20-top_p", _8B, 3, 8, 16, 1024, 20, top_p=0.95),
        # the largest policy's width: weights dominate the decode step
        _rollout("32b-64x1000+20", _32B, 2, 8, 8, 1000, 20),
        # more prompts than cache slots: groups are admitted as others end
        _rollout("4b-continuous-64x300+40", _4B, 4, 24, 8, 300, 40, stop_lo=10, slots=64),
        # long contexts in a small batch, with the raw logits, as a user does who compares a policy with another framework's
        _rollout("8b-6x4001+8-logits", _8B, 2, 2, 3, 4001, 8, logits=True),
        # scoring a batch of finished answers of all lengths (the learner's importance ratio)
        _score("4b-score-24x700-ragged", _4B, 4, 24, 700, ragged=True),
        # scoring long strings at the largest width: the matrix cores' case
        _score("32b-score-3x4096", _32B, 2, 3, 4096),
        # a worker takes a new snapshot and scores a short string under it
        _install("4b-install-bf16", dict(_4B, vocab=32000), 4, "bf16", 65),
        # the learner-side tensors of a batch of long records
        _grpo("grpo-512x9216", 512, 9216, 16),
    ]


def _cost(c):
    """A rough time in seconds, to keep a drawn case below the largest listed one."""
    w = work(c)
    t = w["bytes"] / 4e12 + w["flops"] / 6e14
    if c["kind"] == "rollout":
        t += _decode_steps(c) * (c["layers"] * 40e-6 + 60e-6)
    if c["kind"] == "install":
        t += w["bytes"] / 2.5e10
    if c["kind"] == "grpo":
        t += w["bytes"] / 1e10
    return t


def draw(rng):
    def span(lo, hi):   # log-uniform whole number, odd ones among them
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    def model(max_layers):
        if rng.random() < 0.5:
            m = dict(rng.choice([_4B, _8B, _32B]))
            m["vocab"] = rng.choice([151936, 151936, 32000, span(2000, 150000)])
        else:
            hd, kv, grp = rng.choice([64, 128]), rng.choice([1, 2, 4, 8]), rng.choice([1, 2, 4, 8])
            h = 16 * span(32, 256)
            m = dict(hidden=h, q_heads=kv * grp, kv_heads=kv, head_dim=hd, ffn=16 * max(16, int(h * rng.uniform(2, 5) / 16)), vocab=span(1000, 150000), dtype="bf16")
        return dict(m, qk_norm=rng.random() < 0.3, tied=rng.random() < 0.3), rng.randint(1, max_layers)

    most = max(_cost(c) for c in listed())
    while True:
        kind = rng.choice(["rollout", "rollout", "rollout", "continuous", "score", "score", "install", "grpo"])
        if kind == "grpo":
            c = _grpo(None, 16 * span(1, 32), span(33, 9300), rng.choice([2, 4, 8, 16]), rng.random() < 0.7)
        elif kind == "install":
            m, layers = model(3)
            m["vocab"] = min(m["vocab"], 40000)
            c = _install(None, m, layers, rng.choice(["bf16", "q8"]), span(9, 200))
        elif kind == "score":
            m, layers = model(3)
            c = _score(None, m, layers, span(1, 24), span(17, 3000), rng.random() < 0.6, rng.choice([1.0, 0.8]))
        else:
            m, layers = model(4)
            G = rng.choice([1, 2, 3, 4, 8, 16])
            P, plen, new = span(1, max(1, 256 // G)), span(3, 2500), span(6, 48)
            ragged, top_p, temp = rng.random() < 0.5, rng.choice([1.0, 1.0, 0.95]), rng.choice([1.0, 1.0, 0.8])
            stop = rng.choice([0, max(1, new // 4)])
            if kind == "continuous":
                slots = G * max(1, min(P - 1, span(1, 256 // G)))
                if P * G <= slots:
                    continue
                c = _rollout(None, m, layers, P, G, plen, new, max(1, stop), top_p, slots, ragged, False, temp)
            else:
                logits = P * G * new * m["vocab"] < 2e7 and rng.random() < 0.4
                c = _rollout(None, m, layers, P, G, plen, new, 0 if logits else stop, top_p, 0, ragged, logits, temp)
        if "hidden" in c and (_params(c)[0] * c["layers"] + _params(c)[1] * 2 > 2.6e9 or 16 * c["kv_heads"] * c["head_dim"] > 16 * 8192):
            continue
        if _cost(c) <= most:
            return c


# ---- inputs ------------------------------------------------------------------------------------------------------------

def _shape(c):
    return synth.ModelShape(c["layers"], c["hidden"], c["q_heads"], c["kv_heads"], c["head_dim"], c["ffn"], c["vocab"], dtype=c["dtype"],
                            qk_norm=c["qk_norm"], tie_embeddings=c["tied"])


def _tensors(c):
    """(name, rows, columns) of a policy blob in its order; rows 0: a norm gain."""
    H, hd, Q, KV, F, V = c["hidden"], c["head_dim"], c["q_heads"] * c["head_dim"], c["kv_heads"] * c["head_dim"], c["ffn"], c["vocab"]
    yield "embed", V, H
    for l in range(c["layers"]):
        yield f"{l}.attn_norm", 0, H
        yield f"{l}.q", Q, H
        yield f"{l}.k", KV, H
        yield f"{l}.v", KV, H
        if c["qk_norm"]:
            yield f"{l}.q_norm", 0, hd
            yield f"{l}.k_norm", 0, hd
        yield f"{l}.o", H, Q
        yield f"{l}.ffn_norm", 0, H
        yield f"{l}.gate", F, H
        yield f"{l}.up", F, H
        yield f"{l}.down", H, F
    yield "final_norm", 0, H
    if not c["tied"]:
        yield "lm_head", V, H


def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _weights(c, seed):
    """(name, tensor on the GPU) in blob order: matrices N(0, 0.02^2), gains 1 + N(0, 0.1^2), in the model's type."""
    dev = _device()
    g = torch.Generator(device=dev).manual_seed(seed)
    dt = torch.float32 if c["dtype"] == "fp32" else torch.bfloat16
    for name, rows, cols in _tensors(c):
        if rows == 0:
            yield name, (1.0 + 0.1 * torch.randn(cols, generator=g, device=dev)).to(dt)
        else:
            w = torch.empty(rows, cols, dtype=dt, device=dev)
            step = max(1, (1 << 27) // cols)
            for a in range(0, rows, step):
                w[a:a + step] = (torch.randn(min(step, rows - a), cols, generator=g, device=dev) * 0.02).to(dt)
            yield name, w


def _weights_q8(c, seed):
    """(name, gain) or (name, (scales, codes)) in blob order."""
    dev = _device()
    g = torch.Generator(device=dev).manual_seed(seed)
    for name, rows, cols in _tensors(c):
        if rows == 0:
            yield name, (1.0 + 0.1 * torch.randn(cols, generator=g, device=dev)).to(torch.bfloat16)
        else:
            scales = (0.5 + torch.rand(rows, generator=g, device=dev)) * (0.02 / 42.0)
            codes = (torch.randn(rows, cols, generator=g, device=dev) * 42.0).round().clamp(-127, 127).to(torch.int8)
            yield name, (scales, codes)


def _bytes_of(t):
    return t.contiguous().view(-1).view(torch.uint8)


_CHUNK = 64 << 20


def _load(ctx, version, c, seed):
    """The snapshot goes in as it would arrive: piece by piece through a pinned host buffer."""
    host = torch.empty(_CHUNK, dtype=torch.uint8, pin_memory=True)
    ctx.load_policy_begin(version, echo.blob_bytes(ctx.desc))
    for _, w in _weights(c, seed):
        b = _bytes_of(w)
        for a in range(0, b.numel(), _CHUNK):
            n = min(_CHUNK, b.numel() - a)
            host[:n].copy_(b[a:a + n])
            ctx.load_policy_chunk(host[:n].numpy())
    ctx.load_policy_commit()


def _pinned_blob(pieces, nbytes):
    host = torch.empty(nbytes, dtype=torch.uint8, pin_memory=True)
    at = 0
    for p in pieces:
        for t in (p if isinstance(p, tuple) else (p,)):
            b = _bytes_of(t)
            host[at:at + b.numel()].copy_(b)
            at += b.numel()
    assert at == nbytes
    return host.numpy()


def _rollout_inputs(c, seed):
    r = np.random.default_rng(seed)
    P, N = c["prompts"], c["prompts"] * c["group"]
    prompts = r.integers(0, c["vocab"], (P, c["plen"])).astype(np.int32)
    lens = r.integers(max(1, c["plen"] // 4), c["plen"] + 1, P).astype(np.int32) if c["ragged"] else np.full(P, c["plen"], np.int32)
    lens[r.integers(0, P)] = c["plen"]
    stop = r.integers(c["stop_lo"], c["new"] + 1, N).astype(np.int32) if c["stop_lo"] else None
    if stop is not None:
        stop[r.integers(0, N)] = c["new"]
    return prompts, lens, stop, r.integers(0, c["vocab"], (N, c["new"])).astype(np.int32)


def _strings(c, seed):
    """Strings to score: whole, or of lengths between a sixteenth and all of `length`."""
    r = np.random.default_rng(seed)
    n = c.get("seqs", 1)
    lens = r.integers(max(2, c["length"] // 16), c["length"] + 1, n).astype(np.int32) if c.get("ragged") else np.full(n, c["length"], np.int32)
    lens[r.integers(0, n)] = c["length"]
    return r.integers(0, c["vocab"], (n, c["length"])).astype(np.int32), lens


def _records(c, seed):
    """Multi-turn records: a turn-start token now and then, outcome rewards, whole groups alike among them."""
    r = np.random.default_rng(seed)
    n, t = c["records"], c["stride"]
    turn = 11
    tokens = r.integers(0, 150000, (n, t), dtype=np.int32)
    tokens[:, 0] = turn
    tokens[np.arange(n)[:, None], r.integers(0, t, (n, 8))] = turn
    lens = r.integers(0, t + 1, n).astype(np.int32)
    rewards = (r.random(n) < 0.4).astype(np.float32)
    rewards[:c["group"]] = 1.0
    return tokens, lens, turn, rewards


def prepare(case, seed):
    c = case
    if c["kind"] == "grpo":
        ctx = echo.Context(echo.desc_from_shape(synth.DENSE_4B.replace(n_layers=1), 64, 64))   # needs no snapshot
        return dict(case=c, ctx=ctx, args=_records(c, seed))
    if c["kind"] == "rollout":
        prompts, lens, stop, forced = _rollout_inputs(c, seed)
        slots = c["slots"] or c["prompts"] * c["group"]
        ctx = echo.Context(echo.desc_from_shape(_shape(c), slots, c["plen"] + c["new"]))
        _load(ctx, 1, c, seed)
        return dict(case=c, ctx=ctx, prompts=prompts, lens=lens, stop=stop, forced=forced, seed=seed)
    tokens, lens = _strings(c, seed)
    ctx = echo.Context(echo.desc_from_shape(_shape(c), len(lens), c["length"]))
    if c["kind"] == "score":
        _load(ctx, 1, c, seed)
        return dict(case=c, ctx=ctx, tokens=tokens, lens=lens)
    q8 = c["form"] == "q8"
    pieces = (p for _, p in (_weights_q8 if q8 else _weights)(c, seed))
    blob = _pinned_blob(pieces, (echo.q8_blob_bytes if q8 else echo.blob_bytes)(ctx.desc))
    return dict(case=c, ctx=ctx, tokens=tokens, lens=lens, blob=blob, version=0)


def run(state):
    c, ctx = state["case"], state["ctx"]
    if c["kind"] == "rollout":
        out = ctx.rollout(state["prompts"], state["lens"], c["group"], c["new"], c["temperature"], state["seed"], stop_lens=state["stop"],
                          top_p=c["top_p"], forced=state["forced"], want_logits=c["logits"], continuous=c["slots"] > 0)
        keys = ("tokens", "logprobs", "lens") + (("logits",) if c["logits"] else ())
        return {k: out[k] for k in keys}
    if c["kind"] == "grpo":
        tokens, lens, turn, rewards = state["args"]
        mask, adv, adv_tok = ctx.grpo_tensors(tokens, lens, c["group"], turn, rewards, per_token=c["per_token"])
        return {"mask": mask, "adv": adv, "adv_tok": adv_tok}
    if c["kind"] == "install":
        state["version"] += 1
        (ctx.load_policy_q8 if c["form"] == "q8" else ctx.load_policy)(state["version"], state["blob"])
        return {"logprobs": ctx.logprobs(state["tokens"], state["lens"])}
    return {"logprobs": ctx.logprobs(state["tokens"], state["lens"], c["temperature"])}


# ---- what a pass cannot do without -----------------------------------------------------------------------------------------

def _params(c):
    """Weights of one layer, of the lm_head."""
    H, hd = c["hidden"], c["head_dim"]
    return H * (2 * c["q_heads"] + 2 * c["kv_heads"]) * hd + 3 * H * c["ffn"], c["vocab"] * H


def _mean_len(c):
    return (c["stop_lo"] + c["new"]) / 2 if c["stop_lo"] else c["new"]


def _decode_steps(c):
    """Decode passes of a rollout: the first token comes out of the prompt pass."""
    if c["slots"]:
        return max(c["new"], math.ceil(c["prompts"] * c["group"] * _mean_len(c) / c["slots"]))
    return c["new"] - 1


def work(case):
    c = case
    if c["kind"] == "grpo":
        cells = c["records"] * c["stride"]
        return {"bytes": cells * (9 if c["per_token"] else 5) + 12 * c["records"], "flops": 0}
    e = 4 if c["dtype"] == "fp32" else 2
    layer, head = _params(c)
    L, kv = c["layers"], 2 * c["layers"] * c["kv_heads"] * c["head_dim"] * e       # kv: cache bytes of a token
    att = 4 * L * c["q_heads"] * c["head_dim"]                                       # flops per (token, key)
    if c["kind"] in ("score", "install"):
        n, T = c.get("seqs", 1), c["length"]
        mean = T * 17 / 32 if c.get("ragged") else T
        rows = n * (mean - 1)
        w = {"bytes": (L * layer + head) * e + 2 * rows * kv + 8 * n * T, "flops": rows * 2 * (L * layer + head) + att * rows * mean / 2}
        if c["kind"] == "install":   # the snapshot is read, and written in the layout that the passes want
            params = L * layer + head * (1 if c["tied"] else 2)
            w["bytes"] += params * ((1 if c["form"] == "q8" else 2) + 2)
        return w
    P, G = c["prompts"], c["group"]
    N, plen, gen = P * G, c["plen"] * (5 / 8 if c["ragged"] else 1.0), _mean_len(c)
    steps = _decode_steps(c)
    rows = P * plen                                                                    # prompt pass
    flops = rows * 2 * L * layer + att * rows * plen / 2 + N * 2 * head
    nbytes = (L * layer + head) * e + rows * kv
    toks = N * max(0.0, gen - 1)                                                       # decode passes
    flops += toks * 2 * (L * layer + head) + att * toks * (plen + gen / 2)
    share = min(1.0, (c["slots"] or N) / N)
    nbytes += steps * ((L * layer + head) * e + share * P * plen * kv * min(1.0, gen / max(1, c["new"]))) + toks * (gen / 2 + 1) * kv
    nbytes += N * c["new"] * 16 + (N * c["new"] * c["vocab"] * 4 if c["logits"] else 0)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """About four times what other launch forms of the same kernels (other split counts, the plain attention kernel, another
    batch composition) were seen to differ by: scored log-probabilities 9e-5 in norm and 4e-4 at most, logits 8e-4 and 5e-3,
    log-probabilities of a rollout 2e-4 where every draw agrees.  One draw in a few thousand falls the other way, and
    then that token's log-probability is another one (by up to a fifth; 3e-3 in the norm of all)."""
    c = case
    if c["kind"] == "grpo":
        return {"rel": 1e-6, "differ": 0.0}
    if c["kind"] in ("score", "install"):
        return {"rel": 4e-4, "max": 2e-3}
    if c["dtype"] == "fp32":
        return {"rel": 1e-5, "max": 1e-4, "differ": 0.005}
    if c["logits"]:
        return {"rel": 4e-3, "max": 3e-2, "differ": 0.01}
    return {"rel": 1e-2, "max": 0.6, "differ": 0.005}


# ---- the same in 64 bits -------------------------------------------------------------------------------------------------------

def _forward64(c, weights, strings, wanted):
    """Final normed hidden states (float64) of every string at its wanted positions (a slice), and the lm_head.
    `weights`: (name, tensor) in blob order.  Plain decoder: pre-norm, grouped-query causal attention, half-split rotary
    embedding, SwiGLU."""
    dev, eps = _device(), 1e-6
    hd, Hq, Hkv = c["head_dim"], c["q_heads"], c["kv_heads"]

    def norm(x, gain):
        return x * torch.rsqrt((x * x).mean(-1, keepdim=True) + eps) * gain

    def rope(x, cos, sin):   # [T, heads, hd]
        a, b = x[..., :hd // 2], x[..., hd // 2:]
        return torch.cat([a * cos - b * sin, a * sin + b * cos], -1)

    theta = 1e4 ** (-2.0 * torch.arange(hd // 2, dtype=torch.float64, device=dev) / hd)
    it = iter(weights)

    def take():
        return next(it)[1].to(torch.float64)

    embed = next(it)[1]
    hs = [embed[torch.from_numpy(s.astype(np.int64)).to(dev)].to(torch.float64) for s in strings]
    head = embed if c["tied"] else None
    del embed
    for _ in range(c["layers"]):
        an, wq, wk, wv = take(), take(), take(), take()
        qn, kn = (take(), take()) if c["qk_norm"] else (None, None)
        wo, fn, wg, wu, wd = take(), take(), take(), take(), take()
        for i, h in enumerate(hs):
            T = h.shape[0]
            ang = torch.arange(T, dtype=torch.float64, device=dev)[:, None] * theta
            cos, sin = torch.cos(ang)[:, None], torch.sin(ang)[:, None]
            x = norm(h, an)
            q, k, v = (x @ wq.T).view(T, Hq, hd), (x @ wk.T).view(T, Hkv, hd), (x @ wv.T).view(T, Hkv, hd)
            if c["qk_norm"]:
                q, k = norm(q, qn), norm(k, kn)
            q, k = rope(q, cos, sin), rope(k, cos, sin)
            causal = torch.ones(T, T, dtype=torch.bool, device=dev).triu(1)
            o = torch.empty(T, Hq, hd, dtype=torch.float64, device=dev)
            for j in range(Hq):
                s = (q[:, j] @ k[:, j // (Hq // Hkv)].T.contiguous()) / math.sqrt(hd)
                o[:, j] = torch.softmax(s.masked_fill_(causal, -math.inf), -1) @ v[:, j // (Hq // Hkv)]
            h = h + o.reshape(T, Hq * hd) @ wo.T
            x = norm(h, fn)
            g = x @ wg.T
            hs[i] = h + ((g * torch.sigmoid(g)) * (x @ wu.T)) @ wd.T
        del wq, wk, wv, wo, wg, wu, wd
    fin = take()
    if head is None:
        head = next(it)[1]
    return [norm(h[w], fin) for h, w in zip(hs, wanted)], head


def _logits64(x, head):
    out = torch.empty(x.shape[0], head.shape[0], dtype=torch.float64, device=x.device)
    for a in range(0, head.shape[0], 32768):
        out[:, a:a + 32768] = x @ head[a:a + 32768].to(torch.float64).T
    return out


def _scores64(c, weights, tokens, lens, temperature):
    strings = [tokens[n, :lens[n] - 1] for n in range(len(lens))]
    hs, head = _forward64(c, weights, strings, [slice(None)] * len(strings))
    out = np.zeros(tokens.shape, np.float64)
    for n, x in enumerate(hs):
        tgt = torch.from_numpy(tokens[n, 1:lens[n]].astype(np.int64)).to(x.device)
        for a in range(0, x.shape[0], 1024):
            z = _logits64(x[a:a + 1024], head) / temperature
            t = tgt[a:a + 1024, None]
            out[n, 1 + a:1 + a + z.shape[0]] = (z.gather(1, t)[:, 0] - torch.logsumexp(z, 1)).cpu().numpy()
    return out


def exact(case, seed):
    """Scored log-probabilities, raw logits and advantages in 64 bits.  The token that a rollout samples, and with it that token's
    log-probability, is a draw: near-ties resolve either way, so it has no such value; the kernels behind it are compared
    through the logits and the scores."""
    c = case
    if c["kind"] == "grpo":
        tokens, lens, turn, rewards = _records(c, seed)
        inside = np.arange(c["stride"])[None] < lens[:, None]
        count = np.cumsum((tokens == turn) & inside, axis=1)
        mask = inside & (count > 1) & (count % 2 == 1)
        r = rewards.astype(np.float64).reshape(-1, c["group"])
        adv = ((r - r.mean(1, keepdims=True)) / (r.std(1, ddof=1, keepdims=True) + 1e-6)).reshape(-1)
        return {"mask": None, "adv": adv, "adv_tok": adv[:, None] * mask if c["per_token"] else None}
    if c["kind"] == "install":
        tokens, lens = _strings(c, seed)

        def dequantised():
            for name, p in _weights_q8(c, seed):
                yield name, (p[1].float() * p[0][:, None]).to(torch.bfloat16) if isinstance(p, tuple) else p
        return {"logprobs": _scores64(c, dequantised() if c["form"] == "q8" else _weights(c, seed), tokens, lens, 1.0)}
    if work(c)["flops"] > 1e14:
        return None
    if c["kind"] == "score":
        tokens, lens = _strings(c, seed)
        return {"logprobs": _scores64(c, _weights(c, seed), tokens, lens, c["temperature"])}
    if not c["logits"]:
        return None
    prompts, lens, _, forced = _rollout_inputs(c, seed)
    strings = [np.concatenate([prompts[n // c["group"], :lens[n // c["group"]]], f[:-1]]) for n, f in enumerate(forced)]
    hs, head = _forward64(c, _weights(c, seed), strings, [slice(-c["new"], None)] * len(strings))
    logits = np.stack([_logits64(x, head).cpu().numpy() for x in hs])
    return {"tokens": None, "logprobs": None, "lens": None, "logits": logits}
