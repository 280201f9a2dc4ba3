"""The calls that programs make on this library, as cases that can be timed and compared.

A labelling job prefills a batch of corpus sequences, rolls anchors out from them and reads
labels; each case is one of those calls through ``binding.Engine`` (or one whole small job).
Models are this package's own workload shapes.  The 7B/8B ones are cut to two decoder layers
(and, for rollouts, to a sixteenth of the vocabulary, which keeps the layers' and the output
head's shares of a step), so that a case is a block of the model with a tolerance of its own;
the output heads are zero-layer models at the full vocabulary; the fp32 and 1B-like models are
whole.

bf16 rollouts feed forced tokens (a public option): with greedy feedback one rounding difference
at a near tie changes every later token of that anchor, and outputs could no longer be compared.
The work is the same.  They return log-probs and features; the tokens are those rows' argmax.
"""
import dataclasses
import math
import random

import numpy as np
import torch

from paper_2609_38795_amd import binding, workloads

_TINY = workloads.WORKLOADS["tiny_fp32"].shape
_1B = workloads.WORKLOADS["small_bf16"].shape
_8B = workloads.WORKLOADS["llama8b_like"].shape
_7B = workloads.WORKLOADS["vl_prefix_7b"].shape

# model name -> (shape, leading image rows per sequence)
MODELS = {
    "tiny": (_TINY, 0),
    "1b": (_1B, 0),
    # two layers; the second one's output is the feature row
    "8b": (dataclasses.replace(_8B, n_layers=2, vocab=8064, feat_layers=(1,)), 0),
    # the same for the vision-language shapes, 24 x 24 image rows on M-RoPE grid positions
    "7b": (dataclasses.replace(_7B, n_layers=2, vocab=9536, feat_layers=(1,),
                               mrope_sections=(16, 24, 24)), 576),
    "8b_head": (dataclasses.replace(_8B, n_layers=0, feat_layers=()), 0),
    "7b_head": (dataclasses.replace(_7B, n_layers=0, feat_layers=()), 0),
}


def listed():
    return [
        # secondary blocks and slot weights of 1024 rolled-out anchors: one call each, no model work
        dict(name="ira_labels", kind="ira", anchors=1024, secondaries=1024, block=16),
        # the 2-layer fp32 job: prefill, then greedy top-8 labels, log-probs and features
        dict(name="job_tiny_f32", kind="job", model="tiny", n_seq=1, seq_len=128, ragged=0,
             anchors=8, block=4),
        # 1B-like model, one short sequence with a handful of anchors: latency and launches
        dict(name="rollout_1b_few", kind="rollout", model="1b", n_seq=1, seq_len=701, ragged=0,
             anchors=7, block=16),
        # 1B-like model at its workload's size, both directions, all eight layers
        dict(name="prefill_1b", kind="prefill", model="1b", n_seq=4, seq_len=2048, ragged=0),
        dict(name="rollout_1b", kind="rollout", model="1b", n_seq=4, seq_len=2048, ragged=0,
             anchors=256, block=16),
        # the headline workload's prefill: 8 x 4096 tokens
        dict(name="prefill_8b", kind="prefill", model="8b", n_seq=8, seq_len=4096, ragged=0),
        # vision-language prefixes of uneven lengths, image rows given as embeddings, M-RoPE
        dict(name="prefill_7b_image", kind="prefill", model="7b", n_seq=8, seq_len=1600, ragged=5),
        # one corpus sample's anchors, as the paper batches them
        dict(name="rollout_8b_sample", kind="rollout", model="8b", n_seq=1, seq_len=4096, ragged=0,
             anchors=128, block=16),
        # the headline workload's rollout: 1024 anchors of 8 sequences
        dict(name="rollout_8b", kind="rollout", model="8b", n_seq=8, seq_len=4096, ragged=0,
             anchors=1024, block=16),
        # long contexts, many branches
        dict(name="rollout_long", kind="rollout", model="8b", n_seq=4, seq_len=8192, ragged=0,
             anchors=2048, block=16),
        # one step's output head of the headline workload: full log-softmax rows
        dict(name="head_8b", kind="head", model="8b_head", n_seq=8, seq_len=128, ragged=0,
             anchors=1024, block=1),
        # corpus labels (top 8 + tail, gates) of two samples at the largest vocabulary
        dict(name="corpus_labels_7b", kind="corpus", model="7b_head", n_seq=2, seq_len=1024,
             ragged=3, anchors=192, block=16),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    k = rng.randrange(10)
    rag = rng.randrange(1, 1000)
    if k == 0:
        return dict(kind="ira", anchors=_log(rng, 32, 4096), secondaries=_log(rng, 32, 4096),
                    block=rng.randint(3, 16))
    if k == 1:
        n = rng.randint(1, 2)
        return dict(kind="job", model="tiny", n_seq=n, seq_len=_log(rng, 40, 300), ragged=rag,
                    anchors=n * _log(rng, 1, 12), block=rng.randint(2, 6))
    if k == 2:
        return dict(kind="prefill", model="1b", n_seq=rng.randint(1, 4),
                    seq_len=_log(rng, 100, 2048), ragged=rag)
    if k == 3:
        n = rng.randint(1, 4)
        return dict(kind="rollout", model="1b", n_seq=n, seq_len=_log(rng, 300, 2048), ragged=rag,
                    anchors=n * _log(rng, 1, 64), block=rng.randint(4, 16))
    if k == 4:
        return dict(kind="prefill", model="8b", n_seq=rng.randint(1, 8),
                    seq_len=_log(rng, 128, 4096), ragged=rag)
    if k == 5:
        return dict(kind="prefill", model="7b", n_seq=rng.randint(1, 8),
                    seq_len=_log(rng, 800, 1600), ragged=rag)
    if k == 6:
        n = rng.randint(1, 8)
        return dict(kind="rollout", model="8b", n_seq=n, seq_len=_log(rng, 512, 4096), ragged=rag,
                    anchors=n * _log(rng, 2, 128), block=rng.randint(4, 16))
    if k == 7:
        n = rng.randint(1, 4)
        return dict(kind="rollout", model="7b", n_seq=n, seq_len=_log(rng, 1000, 1600), ragged=rag,
                    anchors=n * _log(rng, 4, 96), block=rng.randint(4, 16))
    if k == 8:
        n = rng.randint(1, 8)
        return dict(kind="head", model="8b_head", n_seq=n, seq_len=128, ragged=0,
                    anchors=n * _log(rng, 1, 128), block=1)
    n = rng.randint(1, 2)
    return dict(kind="corpus", model="7b_head", n_seq=n, seq_len=_log(rng, 256, 1024), ragged=rag,
                anchors=n * _log(rng, 4, 96), block=rng.randint(2, 16))


# ------------------------------------------------------------------ inputs


def _lens(case):
    """Sequence lengths: all seq_len, or (ragged) down to 60% of it (with images, to the image
    and 124 tokens)."""
    n, full = case["n_seq"], case["seq_len"]
    if not case["ragged"]:
        return [full] * n
    r = random.Random(case["ragged"])
    image = MODELS[case["model"]][1]
    least = max((6 * full + 9) // 10, image + 124 if image else 1)
    return [full] + [r.randint(least, full) for _ in range(n - 1)]


def _lo(case, length):
    """First anchor position: past the image and prompt, or the first quarter of the sequence."""
    image = MODELS[case["model"]][1]
    return min(image + 64, length - 1) if image else length // 4


def _per_seq(case):
    return case["anchors"] // case["n_seq"]


def _anchors(case, seed):
    rng = np.random.RandomState(seed % (1 << 31))
    seqs, pos = [], []
    for i, length in enumerate(_lens(case)):
        lo, n = _lo(case, length), _per_seq(case)
        span = length - lo
        pos.append(lo + (rng.choice(span, n, replace=False) if n <= span
                         else rng.randint(0, span, n)))
        seqs.append(np.full(n, i))
    return np.concatenate(seqs).astype(np.int32), np.concatenate(pos).astype(np.int32)


def _weights(shape, gen):
    """N(0, 0.02) matrices and gains near 1, on the GPU, in the storage type."""
    dt = torch.bfloat16 if shape.dtype == "bf16" else torch.float32

    def mat(name):
        return (torch.randn(workloads.weight_shape(shape, name), generator=gen, device="cuda")
                * 0.02).to(dt)

    def gain():
        return (1 + 0.1 * torch.randn(shape.d_model, generator=gen, device="cuda")).to(dt)

    layers = []
    for _ in range(shape.n_layers):
        ld = {n: mat(n) for n in ("wq", "wk", "wv", "wo", "w_gate", "w_up", "w_down")}
        ld["attn_norm"], ld["ffn_norm"] = gain(), gain()
        layers.append(ld)
    return {"tok_embed": mat("tok_embed"), "lm_head": mat("lm_head"), "final_norm": gain(),
            "layers": layers}


def _tokens(gen, n, vocab):
    """Zipf(1.1) token ids by inverse CDF, int32 on the GPU."""
    cdf = torch.arange(1, vocab + 1, dtype=torch.float64, device="cuda").pow(-1.1).cumsum(0)
    u = torch.rand(n, generator=gen, device="cuda", dtype=torch.float64) * cdf[-1]
    return torch.searchsorted(cdf, u).clamp_(max=vocab - 1).to(torch.int32)


def _inputs(case, seed):
    """Everything a case is fed, as tensors on the GPU (and host arrays for the anchors)."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    shape, image = MODELS[case["model"]]
    lens = _lens(case)
    total = sum(lens)
    s = {"shape": shape, "lens": lens, "weights": _weights(shape, gen),
         "tokens": _tokens(gen, total, shape.vocab), "embeds": None, "mask": None,
         "positions": None}
    if image or case["kind"] == "head":
        # image rows at the head of every sequence; the output head reads given rows throughout
        off = np.concatenate([[0], np.cumsum(lens)])
        mask = torch.zeros(total, dtype=torch.uint8, device="cuda")
        for i, length in enumerate(lens):
            mask[off[i]:off[i] + (image or length)] = 1
        rows = torch.randn((total, shape.d_model), generator=gen, device="cuda")
        s["embeds"] = (rows * mask[:, None]).to(torch.bfloat16)
        s["mask"] = mask
    if any(shape.mrope_sections):
        side = int(round(math.sqrt(image)))
        s["positions"] = np.concatenate([workloads.grid_positions(n, side) for n in lens])
    if "anchors" in case:
        s["anchor_seq"], s["anchor_pos"] = _anchors(case, seed)
        if case["kind"] == "rollout":
            s["forced"] = _tokens(gen, len(s["anchor_seq"]) * case["block"],
                                  shape.vocab).view(-1, case["block"])
    return s


def _host(t):
    return t.view(torch.int16).cpu().numpy().view(np.uint16) if t.dtype == torch.bfloat16 \
        else t.cpu().numpy()


def _engine(case, s):
    w = s["weights"]
    host = {k: _host(w[k]) for k in ("tok_embed", "lm_head", "final_norm")}
    host["layers"] = [{k: _host(v) for k, v in ld.items()} for ld in w["layers"]]
    block = case.get("block", 1)
    lim = binding.make_limits(sum(s["lens"]), len(s["lens"]), max(1, case.get("anchors", 1)), block)
    return binding.Engine(s["shape"], host, max(s["lens"]) + block, lim)


def _prefill(s, feats_out=None):
    s["engine"].prefill(s["tokens"], s["lens"], s["embeds"], s["mask"], feats_out, s["positions"])


def _ira_inputs(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    n, b, q = case["anchors"], case["block"], case["secondaries"]
    dev = dict(generator=gen, device="cuda")
    logp = torch.log_softmax(torch.randn((n, b, 64), **dev) * 3, -1).topk(8, -1).values
    rng = np.random.RandomState(seed % (1 << 31))
    return {"tokens": torch.randint(0, 2000, (n, b), dtype=torch.int32, **dev),
            "top_ids": torch.randint(0, 2000, (n, b, 8), dtype=torch.int32, **dev),
            "top_logp": logp.contiguous(), "tail": 1 - logp.exp().sum(-1),
            "primary": rng.randint(0, n, q).astype(np.int32),
            "offset": rng.randint(1, b, q).astype(np.int32)}


def prepare(case, seed):
    if case["kind"] == "ira":
        s = _ira_inputs(case, seed)
        # a context of any model assembles labels: the tiny one's
        big = max(case["anchors"], case["secondaries"])
        s["engine"] = binding.Engine(
            _TINY, workloads.random_weights(_TINY, 1), 64 + case["block"],
            binding.make_limits(64, 1, big, case["block"]))
    else:
        s = _inputs(case, seed)
        s["engine"] = _engine(case, s)
        del s["weights"]
        if case["kind"] == "prefill":
            shape = s["shape"]
            s["feats"] = torch.empty((sum(s["lens"]), shape.n_feat, shape.d_model), device="cuda")
        elif case["kind"] != "job":
            _prefill(s)  # the rollout and label calls follow a prefill
    s["case"] = case
    return s


# ------------------------------------------------------------------ the calls


def run(s):
    case, eng = s["case"], s["engine"]
    kind = case["kind"]
    if kind == "ira":
        return {"secondary": eng.ira_assemble(s["tokens"], s["top_ids"], s["top_logp"], s["tail"],
                                              s["primary"], s["offset"], eos_id=7),
                "weights": eng.slot_weights(s["tokens"], eos_id=7)}
    if kind == "prefill":
        _prefill(s, s["feats"])
        return s["feats"]
    if kind == "job":
        _prefill(s)
        tok, ids, top, tail, lp, ft = eng.rollout_topk(s["anchor_seq"], s["anchor_pos"],
                                                       case["block"], want_logprobs=True)
        return dict(tokens=tok, top_ids=ids, top_logp=top, tail=tail, logprobs=lp, feats=ft)
    if kind == "rollout":
        _, lp, ft = eng.rollout(s["anchor_seq"], s["anchor_pos"], case["block"], forced=s["forced"])
        return dict(logprobs=lp, feats=ft)
    if kind == "head":
        tok, lp, _ = eng.rollout(s["anchor_seq"], s["anchor_pos"], case["block"])
        return dict(tokens=tok, logprobs=lp)
    return {k: v for k, v in eng.corpus_labels(s["anchor_seq"], s["anchor_pos"],
                                               case["block"]).items() if v is not None}


# ------------------------------------------------------------------ what a call cannot do without


def work(case):
    if case["kind"] == "ira":
        n, q, b = case["anchors"], case["secondaries"], case["block"]
        return {"bytes": n * b * 8 + q * b * 2 * 68 + q * b * 4, "flops": 0}
    shape = MODELS[case["model"]][0]
    lens, d, V = _lens(case), shape.d_model, shape.vocab
    es = 2 if shape.dtype == "bf16" else 4
    L, hd, H = shape.n_layers, shape.head_dim, shape.n_heads
    layer = d * (shape.q_dim + 2 * shape.kv_dim) + shape.q_dim * d + 3 * d * shape.d_ffn
    T = sum(lens)
    total = {"bytes": 0.0, "flops": 0.0}

    def add(bytes_, flops):
        total["bytes"] += bytes_
        total["flops"] += flops

    if case["kind"] in ("prefill", "job"):
        seen = sum(n * (n + 1) / 2 for n in lens)
        add(L * (layer * es + T * 2 * shape.kv_dim * es) + T * d * es + T * shape.n_feat * d * 4,
            L * (2.0 * T * layer + 4.0 * hd * H * seen))
    if case["kind"] == "prefill":
        return total
    n, B = case["anchors"], case["block"]
    if case["kind"] == "corpus":
        add(V * d * es + T * d * es + n * B * 68, 2.0 * n * B * V * d)
        return total
    # a step needs the tokens of the one before it, so each reads the weights and the shared
    # keys and values; an anchor sits on average midway between its range's ends
    keys = sum((_lo(case, m) + m) / 2 for m in lens) / len(lens)
    out = n * B * (V + shape.n_feat * d) * 4
    step = L * (layer * es + T * 2 * shape.kv_dim * es) + V * d * es
    add(out + V * d * es + (B - 1) * step,
        2.0 * n * B * V * d + (B - 1) * n * L * (2.0 * layer + 4.0 * hd * H * keys))
    return total


def tolerance(case):
    if case["kind"] == "ira":
        return {"rel": 1e-6, "max": 1e-5}
    if case["kind"] == "job":
        # fp32 sums in another order
        return {"rel": 1e-5, "max": 4e-4, "differ": 0.01}
    if case["kind"] in ("head", "corpus"):
        # the same bf16 rows, fp32 sums in another order; near ties may swap ranks
        return {"rel": 1e-4, "max": 2e-3, "differ": 0.01}
    # bf16 operands: another order of sums moves single roundings of each layer's operands
    return {"rel": 2e-2, "max": 0.3}


# ------------------------------------------------------------------ 64-bit evaluation


def _norm(x, g, eps):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + eps) * g


def _rope(x, pos, shape):
    """Rotate-half RoPE of x[rows, heads, hd] at pos[rows, 3]."""
    half = shape.head_dim // 2
    sec = shape.mrope_sections if any(shape.mrope_sections) else (half, 0, 0)
    axis = torch.repeat_interleave(torch.arange(3), torch.tensor(sec)).cuda()
    inv = shape.rope_base ** (-2.0 * torch.arange(half, dtype=torch.float64, device="cuda")
                              / shape.head_dim)
    ang = pos.double()[:, axis] * inv
    c, s = torch.cos(ang)[:, None], torch.sin(ang)[:, None]
    a, b = x[..., :half], x[..., half:]
    return torch.cat([a * c - b * s, b * c + a * s], -1)


def _qkv(x, w, pos, shape):
    n1 = _norm(x, w["attn_norm"], shape.rms_eps)
    hd, rows = shape.head_dim, x.shape[0]
    return (_rope((n1 @ w["wq"].T).view(rows, -1, hd), pos, shape),
            _rope((n1 @ w["wk"].T).view(rows, -1, hd), pos, shape),
            (n1 @ w["wv"].T).view(rows, -1, hd))


def _rest(x, att, w, shape):
    x = x + att @ w["wo"].T
    n2 = _norm(x, w["ffn_norm"], shape.rms_eps)
    return x + (torch.nn.functional.silu(n2 @ w["w_gate"].T) * (n2 @ w["w_up"].T)) @ w["w_down"].T


def _prefix64(x, pos, W, shape):
    """One sequence: (every layer's output, keys, values)."""
    n, hd = x.shape[0], shape.head_dim
    rep = shape.n_heads // shape.n_kv_heads
    hidden = torch.ones(n, n, dtype=torch.bool, device="cuda").triu_(1)
    outs, keys, vals = [], [], []
    for w in W["layers"]:
        q, k, v = _qkv(x, w, pos, shape)
        att = torch.empty(n, shape.n_heads, hd, dtype=torch.float64, device="cuda")
        for h in range(shape.n_heads):
            sc = (q[:, h] @ k[:, h // rep].T / math.sqrt(hd)).masked_fill_(hidden, -math.inf)
            att[:, h] = torch.softmax(sc, -1) @ v[:, h // rep]
        x = _rest(x, att.view(n, -1), w, shape)
        outs.append(x)
        keys.append(k)
        vals.append(v)
    return outs, keys, vals


def _block64(fed, apos, pos, keys, vals, W, shape):
    """Layer outputs of the tokens fed[anchors, m] that follow each anchor of one sequence."""
    n, m = fed.shape
    hd, G = shape.head_dim, shape.n_kv_heads
    rep = shape.n_heads // G
    length = keys[0].shape[0]
    a = torch.as_tensor(apos, device="cuda").long()
    x = W["tok_embed"][fed.long()].view(n * m, -1)
    p = (pos[a][:, None] + torch.arange(1, m + 1, device="cuda")[None, :, None]).view(n * m, 3)
    past = (torch.arange(length, device="cuda")[None] > a[:, None])[:, None, None]
    later = torch.ones(m, m, dtype=torch.bool, device="cuda").triu_(1)[None, :, None]
    outs = []
    for w, kc, vc in zip(W["layers"], keys, vals):
        q, k, v = _qkv(x, w, p, shape)
        att = torch.empty(n, m, G, rep, hd, dtype=torch.float64, device="cuda")
        q = q.view(n, m, G, rep, hd) / math.sqrt(hd)
        k, v = k.view(n, m, G, hd), v.view(n, m, G, hd)
        for g in range(G):
            qg = q[:, :, g].reshape(-1, hd)
            shared = (qg @ kc[:, g].T).view(n, m, rep, length).masked_fill_(past, -math.inf)
            own = (qg.view(n, m * rep, hd) @ k[:, :, g].transpose(1, 2).contiguous())
            own = own.view(n, m, rep, m).masked_fill_(later, -math.inf)
            pr = torch.softmax(torch.cat([shared, own], -1), -1)
            att[:, :, g] = (pr[..., :length].reshape(-1, length) @ vc[:, g]).view(n, m, rep, hd)
            att[:, :, g] += (pr[..., length:].reshape(n, m * rep, m)
                             @ v[:, :, g].contiguous()).view(n, m, rep, hd)
        x = _rest(x, att.view(n * m, -1), w, shape)
        outs.append(x)
    return outs


def _wide(W):
    out = {k: W[k].double() for k in ("tok_embed", "lm_head", "final_norm")}
    out["layers"] = [{k: v.double() for k, v in ld.items()} for ld in W["layers"]]
    return out


def _ira64(case, seed):
    s = _ira_inputs(case, seed)
    n, b, gamma = case["anchors"], case["block"], 2.0
    env = torch.exp(-torch.arange(b, dtype=torch.float64, device="cuda") / gamma)
    ended = torch.cumsum((s["tokens"] == 7).long(), 1) - (s["tokens"] == 7).long() > 0
    sec = torch.as_tensor(s["primary"], device="cuda").long()
    src = torch.as_tensor(s["offset"], device="cuda").long()[:, None] \
        + torch.arange(b, device="cuda")
    inside = src <= b - 1
    at = src.clamp(max=b - 1)
    top = s["top_logp"].double()[sec[:, None], at]
    top = torch.where(inside[..., None], top, torch.full_like(top, -math.inf))
    tail = s["tail"].double()[sec[:, None], at] * inside
    weight = env * ((src + 1 <= b - 1) & ~ended[sec[:, None], at])
    return {"secondary": (None, None, top, tail, weight), "weights": env * ~ended}


def exact(case, seed):
    if case["kind"] == "ira":
        return _ira64(case, seed)
    s = _inputs(case, seed)
    shape, W, lens = s["shape"], _wide(s["weights"]), s["lens"]
    off = np.concatenate([[0], np.cumsum(lens)])
    x0 = W["tok_embed"][s["tokens"].long()]
    if s["embeds"] is not None:
        x0 = torch.where(s["mask"][:, None].bool(), s["embeds"].double(), x0)
    feats = list(shape.feat_layers)

    def pos_of(i):
        if s["positions"] is None:
            return torch.arange(lens[i], device="cuda")[:, None].expand(-1, 3)
        return torch.as_tensor(s["positions"][off[i]:off[i + 1]], device="cuda").long()

    def head(x):
        return torch.log_softmax(_norm(x, W["final_norm"], shape.rms_eps) @ W["lm_head"].T, -1)

    if case["kind"] == "prefill":
        rows = []
        for i in range(len(lens)):
            outs, _, _ = _prefix64(x0[off[i]:off[i + 1]], pos_of(i), W, shape)
            rows.append(torch.stack([outs[f] for f in feats], 1))
        return torch.cat(rows)
    B, n = case["block"], len(s["anchor_seq"])
    if case["kind"] == "corpus":
        return _corpus64(case, s, x0, off, head)
    lp = torch.empty(n, B, shape.vocab, dtype=torch.float64, device="cuda")
    ft = torch.empty(n, B, len(feats), shape.d_model, dtype=torch.float64, device="cuda")
    for i in range(len(lens)):
        mine = np.nonzero(s["anchor_seq"] == i)[0]
        apos, pos = s["anchor_pos"][mine], pos_of(i)
        idx = torch.as_tensor(mine, device="cuda")
        x = x0[off[i]:off[i + 1]]
        outs, keys, vals = _prefix64(x, pos, W, shape)
        at = torch.as_tensor(apos, device="cuda").long()
        last = (outs[-1] if outs else x)[at]
        lp[idx, 0] = head(last)
        if feats:
            ft[idx, 0] = torch.stack([outs[f][at] for f in feats], 1)
        if B == 1:
            continue

        def block(fed):
            o = _block64(fed, apos, pos, keys, vals, W, shape)
            m = fed.shape[1]
            lp[idx, 1:m + 1] = head(o[-1]).view(len(mine), m, -1)
            ft[idx, 1:m + 1] = torch.stack([o[f] for f in feats], 1).view(
                len(mine), m, len(feats), -1)

        if case["kind"] == "job":  # greedy: one more fed token at a time
            for m in range(1, B):
                block(lp[idx, :m].argmax(-1))
        else:
            block(s["forced"][idx, :B - 1])
    if case["kind"] == "job":
        top = lp.topk(8, -1).values
        return dict(tokens=None, top_ids=None, top_logp=top, tail=_tail(lp, top), logprobs=lp,
                    feats=ft)
    if case["kind"] == "head":
        return dict(tokens=None, logprobs=lp)
    return dict(logprobs=lp, feats=ft)


def _tail(lp, top):
    kth = top[..., -1:]
    return torch.where(lp < kth, lp.exp(), torch.zeros_like(lp)).sum(-1)


def _corpus64(case, s, x0, off, head):
    B, n = case["block"], len(s["anchor_seq"])
    dev = dict(dtype=torch.float64, device="cuda")
    out = dict(argmax=None, top_ids=None, top_logp=torch.full((n, B, 8), -math.inf, **dev),
               tail=torch.zeros(n, B, **dev), corpus_logp=torch.full((n, B), math.nan, **dev),
               gate_soft=torch.zeros(n, B, **dev), gate_hard=torch.zeros(n, B, **dev))
    seq = torch.as_tensor(s["anchor_seq"], device="cuda").long()
    first = torch.as_tensor(off, device="cuda")[seq]
    end = torch.as_tensor(off, device="cuda")[seq + 1] - 1
    a = first + torch.as_tensor(s["anchor_pos"], device="cuda").long()
    total, hard = torch.zeros(n, **dev), torch.ones(n, **dev)
    alive = torch.ones(n, dtype=torch.bool, device="cuda")
    for t in range(B):
        ok, more = a + t <= end, a + t + 1 <= end
        lp = head(x0[torch.minimum(a + t, end)])
        top = lp.topk(8, -1).values
        nxt = s["tokens"].long()[torch.minimum(a + t + 1, end)]
        clp = lp.gather(1, nxt[:, None])[:, 0]
        out["top_logp"][:, t] = torch.where(ok[:, None], top, out["top_logp"][:, t])
        out["tail"][:, t] = _tail(lp, top) * ok
        out["corpus_logp"][:, t] = torch.where(more, clp, out["corpus_logp"][:, t])
        out["gate_soft"][:, t] = total.exp() * (ok & alive)
        out["gate_hard"][:, t] = hard * (ok & alive)
        alive = alive & more
        total = total + clp
        hard = hard * (lp.argmax(-1) == nxt)
    return out
