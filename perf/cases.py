"""What a user of this library has it do, as cases that can be timed and checked.

A self-play actor prefills game histories, appends new turns to them, and decodes one token per live game and step,
with or without the fused sampler; an evaluation run decodes a few games with truncated sampling; the learner scores
the finished games.  Every case goes through the entry points of `paper_2506_24119_amd.binding` as such a program
does, with the model, the page pool, the workspace and the histories already in place (`prepare`).

Geometries are the repository's own (`inputs.GEOMETRIES`); "layers" below the geometry's depth and a smaller "vocab"
make a block of such a model that keeps every projection and attention shape and whose outputs can be compared
closely (in a whole model one layer's rounding travels through all that follow).

Kinds:
  decode    `steps` decode steps with given input tokens (the second step reads what the first appended) -> logits
  sampled   `steps` fused decode + sample steps with given input tokens, then one step that returns logits
  prefill   appends runs of tokens to histories (lengths may start at 0) -> next-token logits
  score     per-token log-probabilities of appended runs and the two objective sums
  sample    categorical (temperature > 0) or greedy (0) draw from logits
  truncated top-k / top-p draw from logits with a workspace -> tokens and the cut's threshold
"""
import math

import numpy as np
import torch

from paper_2506_24119_amd import binding as sb
from paper_2506_24119_amd import inputs as si

DEV = "cuda:0"
GROUP = 16384                     # prompt tokens per prefill call when the histories are laid down


def listed():
    return [
        # the fp32 model of the smallest configuration: four games, greedy; latency of a call
        {"name": "decode fp32 tiny B4", "kind": "decode", "model": "tiny", "layers": 2, "vocab": 1024, "batch": 4,
         "ctx_lo": 64, "ctx_hi": 96, "steps": 2},
        # the tail of a batch of games, or an evaluation of a few: a whole small model, full vocabulary
        {"name": "decode 0.6B B3", "kind": "decode", "model": "qwen3-0.6b", "layers": 28, "vocab": 151936, "batch": 3,
         "ctx_lo": 200, "ctx_hi": 1500, "steps": 2},
        # an odd number of live games on the 7B shape (QKV bias, seven query heads per kv head)
        {"name": "decode 7B block B27", "kind": "decode", "model": "qwen2.5-7b", "layers": 3, "vocab": 8192, "batch": 27,
         "ctx_lo": 512, "ctx_hi": 2560, "steps": 2},
        # the full batch of the training run on the 4B shape, contexts of its first half
        {"name": "decode 4B block B128", "kind": "decode", "model": "qwen3-4b", "layers": 4, "vocab": 8192, "batch": 128,
         "ctx_lo": 256, "ctx_hi": 1280, "steps": 2},
        # the same batch on long multi-turn histories
        {"name": "decode 4B block long", "kind": "decode", "model": "qwen3-4b", "layers": 2, "vocab": 8192, "batch": 128,
         "ctx_lo": 1024, "ctx_hi": 5120, "steps": 2},
        # the benchmark's step: the whole 4B shape, 128 games, the actor's sampler inside the step
        {"name": "sampled 4B B128", "kind": "sampled", "model": "qwen3-4b", "layers": 36, "vocab": 151936, "batch": 128,
         "ctx_lo": 512, "ctx_hi": 1280, "steps": 3},
        # new turns appended to the histories of a few games
        {"name": "prefill turns 4B block", "kind": "prefill", "model": "qwen3-4b", "layers": 4, "vocab": 8192, "batch": 9,
         "ctx_lo": 400, "ctx_hi": 2000, "new_lo": 30, "new_hi": 250},
        # first prompts, one group of a ragged batch
        {"name": "prefill prompts 4B block", "kind": "prefill", "model": "qwen3-4b", "layers": 2, "vocab": 8192, "batch": 24,
         "ctx_lo": 0, "ctx_hi": 0, "new_lo": 256, "new_hi": 1024},
        # a few long histories at once
        {"name": "prefill long 0.6B block", "kind": "prefill", "model": "qwen3-0.6b", "layers": 4, "vocab": 8192, "batch": 4,
         "ctx_lo": 0, "ctx_hi": 0, "new_lo": 2048, "new_hi": 4096},
        # the learner: log-probabilities of finished games under the full vocabulary, then the objective
        {"name": "score 4B block", "kind": "score", "model": "qwen3-4b", "layers": 1, "vocab": 151936, "batch": 8,
         "ctx_lo": 0, "ctx_hi": 0, "new_lo": 400, "new_hi": 1400},
        # the actor's sampler on stored logits
        {"name": "sample B128", "kind": "sample", "batch": 128, "vocab": 151936, "temperature": 1.0, "spread": 1.0},
        # the evaluation setting (temperature 0.6, top-p 0.95) on a small batch
        {"name": "truncated B16", "kind": "truncated", "batch": 16, "vocab": 151936, "temperature": 0.6, "top_k": 0,
         "top_p": 0.95, "spread": 3.0},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["decode", "decode", "decode", "sampled", "prefill", "prefill", "prefill", "score", "sample", "truncated"])
    if kind in ("sample", "truncated"):
        c = {"kind": kind, "batch": _log_int(rng, 1, 200), "vocab": rng.choice([151936, 152064, _log_int(rng, 1000, 150000)]),
             "temperature": rng.choice([0.6, 1.0]), "spread": round(rng.uniform(1.0, 4.0), 2)}
        if kind == "truncated":
            c["top_k"], c["top_p"] = rng.choice([(0, 0.95), (0, 0.9), (50, 1.0), (20, 0.9)])
        else:
            c["temperature"] = rng.choice([0.0, 0.6, 1.0])
        return c
    if kind == "decode" and rng.random() < 0.12:
        lo = rng.randint(1, 200)
        return {"kind": "decode", "model": "tiny", "layers": 2, "vocab": 1024, "batch": _log_int(rng, 1, 32), "ctx_lo": lo,
                "ctx_hi": lo + rng.randint(0, 200), "steps": 2}
    c = {"kind": kind, "model": rng.choice(["qwen3-0.6b", "qwen3-4b", "qwen2.5-7b"]), "layers": rng.randint(2, 4), "vocab": 8192}
    if kind in ("decode", "sampled"):
        c["batch"] = _log_int(rng, 1, 160)
        c["ctx_lo"] = _log_int(rng, 16, 1500)
        c["ctx_hi"] = c["ctx_lo"] + _log_int(rng, 16, 2500)
        c["steps"] = rng.randint(1, 3)
        if kind == "sampled":
            c["vocab"] = si.GEOMETRIES[c["model"]].vocab
        return c
    if kind == "score":
        c["layers"], c["vocab"] = 1, si.GEOMETRIES[c["model"]].vocab
    c["batch"] = _log_int(rng, 1, 24)
    c["ctx_lo"] = rng.choice([0, _log_int(rng, 16, 1500)])
    c["ctx_hi"] = c["ctx_lo"] + (_log_int(rng, 16, 1500) if c["ctx_lo"] else 0)
    total = _log_int(rng, 24 if kind == "prefill" else 256, 8192)            # about this many new tokens in all
    c["new_lo"] = max(1, total // (2 * c["batch"]))
    c["new_hi"] = max(c["new_lo"], (3 * total) // (2 * c["batch"]))
    return c


# ---------------------------------------------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------------------------------------------
def _geometry(case):
    return si.scaled_geometry(case["model"], n_layers=case["layers"], vocab=case["vocab"])


def _weights(g, seed):
    """Random-init weights on the GPU: matrices and biases N(0, 0.02), norm gains around 1."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    wdt = torch.bfloat16 if g.weight_dtype == si.WEIGHT_BF16 else torch.float32

    def matrix(shape):
        return torch.empty(shape, dtype=wdt, device=DEV).normal_(0.0, 0.02, generator=gen)

    def gain(shape):
        return torch.empty(shape, dtype=torch.float32, device=DEV).normal_(1.0, 0.1, generator=gen)

    w = {"embed": matrix((g.vocab, g.d_model)), "final_norm": gain((g.d_model,))}
    w["layers"] = [{k: gain(s) if k.endswith("norm") else matrix(s) for k, s in si.layer_tensor_shapes(g).items()}
                   for _ in range(g.n_layers)]
    w["lm_head"] = w["embed"] if g.tie_lm_head else matrix((g.vocab, g.d_model))
    return w


def _lengths(case):
    """History lengths and appended lengths of the sequences: ragged, and fixed by the case."""
    B = case["batch"]
    rng = np.random.Generator(np.random.PCG64(1000003 * B + 1009 * case["ctx_hi"] + case["ctx_lo"] + case.get("new_hi", 0)))
    hist = rng.integers(case["ctx_lo"], case["ctx_hi"] + 1, B)
    if case["kind"] in ("prefill", "score"):
        return hist, rng.integers(case["new_lo"], case["new_hi"] + 1, B)
    return hist, np.full(B, case["steps"] + (1 if case["kind"] == "sampled" else 0))


def _games(case, seed):
    """History tokens, and the tokens the pass consumes, of every sequence (host arrays)."""
    rng = np.random.Generator(np.random.PCG64(seed))
    B, V = case["batch"], case["vocab"]
    hl, nl = _lengths(case)
    hist = [rng.integers(0, V, int(n)).astype(np.int32) for n in hl]
    if case["kind"] in ("prefill", "score"):
        new = [rng.integers(0, V, int(n)).astype(np.int32) for n in nl]
    else:
        n = case["steps"] + (1 if case["kind"] == "sampled" else 0)
        forced = rng.integers(0, V, (n, B)).astype(np.int32)
        new = [forced[:, b].copy() for b in range(B)]
    return hist, new


def _learner(rows, seed):
    """Old log-probabilities' offsets, advantages and mask of the packed rows (the mask drops the players' prompts)."""
    rng = np.random.Generator(np.random.PCG64(seed + 77))
    return (rng.normal(0.0, 0.1, rows).astype(np.float32), rng.uniform(-1.0, 1.0, rows).astype(np.float32),
            (rng.random(rows) < 0.7).astype(np.int32))


def _logits(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    return torch.empty((case["batch"], case["vocab"]), dtype=torch.float32, device=DEV).normal_(0.0, case["spread"], generator=gen)


def prepare(case, seed):
    if case["kind"] in ("sample", "truncated"):
        B = case["batch"]
        st = {"case": case, "seed": seed, "logits": _logits(case, seed), "ids": np.arange(B, dtype=np.int32),
              "steps": (np.arange(B, dtype=np.int32) * 7 + seed % 97).astype(np.int32),
              "tokens": torch.empty(B, dtype=torch.int32, device=DEV)}
        if case["kind"] == "truncated":
            st["threshold"] = torch.empty(B, dtype=torch.float32, device=DEV)
            st["need"] = sb.spiral_sample_truncated_workspace_bytes(B, case["vocab"])
            st["work"] = torch.empty(st["need"], dtype=torch.uint8, device=DEV)
        return st

    g, B = _geometry(case), case["batch"]
    hist, new = _games(case, seed)
    hl, nl = np.array([len(h) for h in hist]), np.array([len(n) for n in new])
    blocks = (hl + nl + 1 + 15) // 16
    n_pages = int(blocks.sum()) + 4
    packed = case["kind"] in ("prefill", "score")
    max_rows = max(B, min(int(hl.sum()), GROUP + int(hl.max())), int(nl.sum()) if packed else 1)
    sess = sb.Session(g, _weights(g, seed), n_pages, B, int(blocks.max()), max_rows, int((hl + nl).max()) + 1,
                      page_order=si.make_page_order(n_pages, seed % (1 << 31)), device=DEV)
    ids = np.arange(B, dtype=np.int32)
    st = {"case": case, "seed": seed, "sess": sess, "ids": ids, "lens": hl.astype(np.int32)}
    if hl.max() > 0:
        i = 0
        while i < B:                                     # the histories, in groups of about GROUP tokens
            j, tok = i, 0
            while j < B and (j == i or tok + hl[j] <= GROUP):
                tok += int(hl[j])
                j += 1
            sess.prefill(ids[i:j], hist[i:j])
            i = j
    if packed:
        st["new"] = nl.astype(np.int32)
        st["packed"] = torch.from_numpy(np.concatenate(new)).to(DEV)
    else:
        st["forced"] = [torch.from_numpy(np.array([n[k] for n in new], dtype=np.int32)).to(DEV) for k in range(int(nl[0]))]
    rows = int(nl.sum())
    if case["kind"] == "prefill":
        st["logits"] = sess.new_logits(B)
    elif case["kind"] == "decode":
        st["logits"] = [sess.new_logits(B) for _ in range(case["steps"])]
    elif case["kind"] == "sampled":
        st["logits"] = sess.new_logits(B)
        st["tokens"] = [torch.empty(B, dtype=torch.int32, device=DEV) for _ in range(case["steps"])]
        st["at"] = [np.full(B, 1 + k, dtype=np.int32) for k in range(case["steps"])]
    else:
        targets = np.concatenate([np.concatenate([n[1:], [-1]]) for n in new]).astype(np.int32)
        off, adv, mask = _learner(rows, seed)
        st["targets"] = torch.from_numpy(targets).to(DEV)
        st["old"] = torch.from_numpy(-math.log(case["vocab"]) + off).to(DEV)
        st["adv"], st["mask"] = torch.from_numpy(adv).to(DEV), torch.from_numpy(mask).to(DEV)
        st["logp"] = torch.empty(rows, dtype=torch.float32, device=DEV)
        st["sums"] = torch.empty(2, dtype=torch.float64, device=DEV)
    return st


# ---------------------------------------------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------------------------------------------
def run(st):
    case, kind = st["case"], st["case"]["kind"]
    if kind == "sample":
        sb.spiral_sample(st["logits"], case["batch"], case["vocab"], case["temperature"], st["seed"], st["ids"], st["steps"],
                         None, st["tokens"])
        return st["tokens"]
    if kind == "truncated":
        sb.spiral_sample_truncated_ws(st["logits"], case["batch"], case["vocab"], case["temperature"], case["top_k"],
                                      case["top_p"], st["seed"], st["ids"], st["steps"], None, st["tokens"], st["threshold"],
                                      st["work"], st["need"])
        return {"tokens": st["tokens"], "threshold": st["threshold"]}

    sess, ids = st["sess"], st["ids"]
    sb.spiral_seq_truncate(sess.pool, ids, st["lens"])             # back to the histories
    if kind == "decode":
        for k in range(case["steps"]):
            sess.decode_step(ids, st["forced"][k], st["logits"][k])
        return st["logits"]
    if kind == "sampled":
        for k in range(case["steps"]):
            sess.decode_sample_step(ids, st["forced"][k], 1.0, st["seed"], st["at"][k], st["tokens"][k])
        sess.decode_step(ids, st["forced"][case["steps"]], st["logits"])
        return {"tokens": st["tokens"], "logits": st["logits"]}
    if kind == "prefill":
        sb.spiral_prefill(sess.model, sess.pool, ids, st["new"], st["packed"], sess.ws, st["logits"])
        return st["logits"]
    sb.spiral_score(sess.model, sess.pool, ids, st["new"], st["packed"], st["targets"], sess.ws, st["logp"])
    sb.spiral_policy_objective(st["logp"], st["old"], st["adv"], st["mask"], st["logp"].numel(), 0.2, st["sums"])
    return {"logp": st["logp"], "sums": st["sums"]}


# ---------------------------------------------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------------------------------------------
def work(case):
    if case["kind"] in ("sample", "truncated"):
        n = case["batch"] * case["vocab"]
        return {"bytes": 4.0 * n + 4 * case["batch"], "flops": 2.0 * n}
    g, B = _geometry(case), case["batch"]
    wb = 2 if g.weight_dtype == si.WEIGHT_BF16 else 4
    kv = 2 * g.n_kv_heads * g.head_dim * 2                         # K + V bytes of a token in a layer
    layer_w, head_w = g.n_layers * g.params_per_layer(), g.vocab * g.d_model
    attn = 4.0 * g.head_dim * g.n_q_heads * g.n_layers             # flops per (token, visible token)
    hist, new = (x.astype(np.float64) for x in _lengths(case))
    if case["kind"] in ("decode", "sampled"):
        n = int(new[0])
        stored = n if case["kind"] == "decode" else 1              # steps whose logits are an output
        seen = float(sum((hist + k + 1).sum() for k in range(n)))  # tokens that all steps' attention reads
        return {"bytes": n * (wb * (layer_w + head_w) + B * kv * g.n_layers) + kv * g.n_layers * seen + stored * 4.0 * B * g.vocab,
                "flops": n * B * 2.0 * (layer_w + head_w) + attn * seen}
    rows, scored = float(new.sum()), float(new.sum()) if case["kind"] == "score" else B
    seen = float((new * hist + new * (new + 1) / 2).sum())
    outputs = 4.0 * rows if case["kind"] == "score" else 4.0 * B * g.vocab
    return {"bytes": wb * (layer_w + head_w) + kv * g.n_layers * float((hist + new).sum()) + 4.0 * rows + outputs,
            "flops": 2.0 * layer_w * rows + attn * seen + 2.0 * head_w * scored}


def tolerance(case):
    # samplers: the draw is defined to the bit (stated noise generator, fp32 score, lowest index on ties)
    if case["kind"] in ("sample", "truncated"):
        return "exact"
    # floating results: about four times the distance from 64 bits that the half-precision activations, q, k, v and
    # softmax weights cost (2-norm, measured: 1.5e-4 with fp32 weights, 0.9 to 1.6e-3 for a block's logits)
    if case["model"] == "tiny":
        return {"rel": 6e-4, "max": 5e-3}
    if case["kind"] == "score":
        return {"rel": 4e-4, "max": 4e-3}       # 1e-4 measured: log-probabilities around -12, a logit's error is small against them
    # through a whole model's depth one layer's rounding travels through all that follow
    t = {"rel": 2e-2, "max": 1.2e-1} if case["layers"] > 4 else {"rel": 6e-3, "max": 4e-2}
    if case["kind"] == "sampled":
        t["differ"] = 0.05                      # draws whose two best scores lie within the logits' rounding
    return t


# ---------------------------------------------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------------------------------------------
def _rms(x, gain, eps):
    return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + eps) * gain


def _rotate(x, cos, sin):
    half = x.shape[-1] // 2
    lo, hi = x[..., :half], x[..., half:]
    return torch.cat([lo * cos - hi * sin, hi * cos + lo * sin], -1)


def _forward(g, w, games, last):
    """Final-normed hidden states of the last `last[b]` positions of every sequence, in float64."""
    f64 = torch.float64
    Hq, Hkv, hd, eps = g.n_q_heads, g.n_kv_heads, g.head_dim, g.rms_eps
    inv = float(g.rope_theta) ** (-2.0 * torch.arange(hd // 2, dtype=f64, device=DEV) / hd)
    xs = [w["embed"][torch.from_numpy(t).to(DEV).long()].to(f64) for t in games]
    for l, lw in enumerate(w["layers"]):
        m = {k: v.to(f64) for k, v in lw.items()}
        for b, x in enumerate(xs):
            n = x.shape[0]
            first = n - last[b] if l == g.n_layers - 1 else 0        # rows still needed after this layer's K and V
            ang = torch.arange(n, dtype=f64, device=DEV)[:, None] * inv
            cos, sin = ang.cos()[:, None, :], ang.sin()[:, None, :]
            h = _rms(x, m["attn_norm"], eps)
            q, k, v = h[first:] @ m["wq"].t(), h @ m["wk"].t(), h @ m["wv"].t()
            if g.qkv_bias:
                q, k, v = q + m["bq"], k + m["bk"], v + m["bv"]
            q, k, v = q.view(n - first, Hq, hd), k.view(n, Hkv, hd), v.view(n, Hkv, hd)
            if g.qk_norm:
                q, k = _rms(q, m["q_norm"], eps), _rms(k, m["k_norm"], eps)
            q, k = _rotate(q, cos[first:], sin[first:]), _rotate(k, cos, sin)
            o = torch.empty((n - first, Hq, hd), dtype=f64, device=DEV)
            hidden = torch.arange(n, device=DEV)[None, :] > torch.arange(first, n, device=DEV)[:, None]
            for h_ in range(Hq):
                kv = h_ // (Hq // Hkv)
                s = (q[:, h_].contiguous() @ k[:, kv].t().contiguous()) / math.sqrt(hd)
                o[:, h_] = torch.softmax(s.masked_fill_(hidden, -math.inf), -1) @ v[:, kv].contiguous()
            x = x[first:] + o.reshape(n - first, Hq * hd) @ m["wo"].t()
            h = _rms(x, m["mlp_norm"], eps)
            xs[b] = x + (torch.nn.functional.silu(h @ m["w_gate"].t()) * (h @ m["w_up"].t())) @ m["w_down"].t()
    return [_rms(x[-last[b]:], w["final_norm"].to(f64), eps) for b, x in enumerate(xs)]


def exact(case, seed):
    if case["kind"] == "sample":
        return None                              # whole numbers only
    if case["kind"] == "truncated":
        return {"tokens": None, "threshold": _exact_threshold(case, seed)}
    g = _geometry(case)
    if 2.0 * g.n_layers * g.params_per_layer() * case["batch"] * (case["ctx_lo"] + case["ctx_hi"]) / 2.0 > 3e14:
        return None                              # the whole 4B shape over 100,000 tokens of history: minutes in 64 bits
    w = _weights(g, seed)
    hist, new = _games(case, seed)
    games = [np.concatenate([h, n]) for h, n in zip(hist, new)]
    head = w["lm_head"].to(torch.float64)
    last = [1] * len(games) if case["kind"] in ("prefill", "sampled") else [len(n) for n in new]
    hidden = _forward(g, w, games, last)
    if case["kind"] in ("prefill", "sampled"):
        logits = torch.cat(hidden) @ head.t()
        return logits if case["kind"] == "prefill" else {"tokens": None, "logits": logits}
    if case["kind"] == "decode":
        return [torch.stack([h[k] for h in hidden]) @ head.t() for k in range(case["steps"])]
    logp = []
    for h, n in zip(hidden, new):
        tgt = torch.from_numpy(n[1:]).to(DEV).long()
        for i in range(0, len(n) - 1, 512):
            z = h[i:min(i + 512, len(n) - 1)] @ head.t()
            logp.append(z.gather(1, tgt[i:i + z.shape[0], None])[:, 0] - torch.logsumexp(z, 1))
        logp.append(torch.zeros(1, dtype=torch.float64, device=DEV))
    logp = torch.cat(logp)
    off, adv, mask = _learner(logp.numel(), seed)
    adv, mask = torch.from_numpy(adv).to(DEV).double(), torch.from_numpy(mask).to(DEV).double()
    old = torch.from_numpy(-math.log(case["vocab"]) + off).to(DEV).double()
    r = torch.exp(logp - old)
    clip = float(np.float32(0.2))
    surrogate = torch.minimum(r * adv, r.clamp(1.0 - clip, 1.0 + clip) * adv)
    return {"logp": logp, "sums": torch.stack([(mask * surrogate).sum(), (mask * adv * logp).sum()])}


def _exact_threshold(case, seed):
    z = (_logits(case, seed) / case["temperature"]).double().sort(dim=1, descending=True).values
    V = case["vocab"]
    k = case["top_k"] if 0 < case["top_k"] < V else V
    tau = z[:, k - 1].clone() if k < V else torch.full((z.shape[0],), -math.inf, dtype=torch.float64, device=z.device)
    if case["top_p"] < 1.0:
        kept = z >= z[:, k - 1:k]                # equal scores are kept together
        mass = torch.where(kept, torch.exp(z - z[:, :1]), torch.zeros_like(z)).cumsum(1)
        at = (mass >= float(np.float32(case["top_p"])) * mass[:, -1:]).int().argmax(1)
        tau = torch.maximum(tau, z.gather(1, at[:, None])[:, 0])
    return tau
