"""Performance cases of the SSD hot path: what a decoding program asks of the library, call by call.

A case is one call (or the two calls that belong together) on a context that the program keeps:

  draft     one-node forward per sequence: the self-draft of a block start, and every step of stepwise decoding
  verify    the batched verification forward of the greedy chain, N + 1 nodes per sequence
  prefill   a prompt into the KV cache and the first block's self-draft behind it: the time to the first token
  refresh   the dual cache's forward over a whole sequence
  generate  ssd_generate from the prompt to the last token, host loop included

on the model shapes of synth.py (the fp32 parity model, the 8B class and the 7B class with grouped-query heads)
and on the small bf16 model with head size 64 of the tests.  Depths, vocabularies and widths are the full ones.

Weights.  Every projection is the random initialisation of synth.gen_weights.  A random bf16 model decides among
near-ties: a confidence's order against the next one changes with the rounding of a sum, and no two correct
implementations would return the same tokens.  A trained model is sure of most of its predictions, so the bf16
models get what makes a random model sure: token embeddings of unit size and an LM head tied to them (row t
belongs to the embedding of token t + shift), wide enough that the predicted token leads by tens of logits and
the confidences saturate; ties then go to the lowest position, as documented.  The maximum logits still depend
on every layer.  The fp32 model is the plain random one.
"""
from __future__ import annotations

import math
import random

import torch

from paper_2510_04147_amd import binding, synth

SMALL_HEADS = dict(dtype="bf16", n_layers=3, d_model=512, n_q_heads=8, n_kv_heads=2, head_dim=64, d_ffn=1536, vocab=2080)


def model(name: str) -> dict:
    return synth.model_config("tiny", **SMALL_HEADS) if name == "small_heads" else synth.model_config(name)


def case(kind, mdl, batch, block, draft, prefix, gen=0, accept=0, name=None):
    """prefix: cached positions per sequence (verify, draft), prompt length (prefill, generate) or positions in front
    of the block (refresh); gen: tokens to generate (refresh: positions from the block on); accept: how many of
    the drafts the model agrees with."""
    c = dict(kind=kind, model=mdl, batch=batch, block=block, draft=draft, prefix=prefix, gen=gen, accept=accept)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the fp32 parity model: a forward is a few dozen tiny kernels, launches and host work are what counts
        case("draft", "tiny", 1, 32, 4, 64, name="tiny_draft"),
        # the same model end to end: prompt 64, 64 tokens, block 32, draft depth 4
        case("generate", "tiny", 1, 32, 4, 64, gen=64, name="tiny_generate"),
        # head size 64, grouped-query heads, blocks that fill a tile only partly, two sequences, an odd prefix
        case("verify", "small_heads", 2, 24, 3, 45, accept=3, name="small_heads_verify"),
        # stepwise decoding of the 8B class, and every block start: 32 rows, the weight stream
        case("draft", "8b", 1, 32, 4, 384, name="8b_draft"),
        # the paper's decoding shape: block 8, draft length 4, 40 rows; an odd prefix
        case("verify", "8b", 1, 8, 4, 381, accept=2, name="8b_verify_b8_n4"),
        # the headline workload: block 32, draft depth 4, 160 rows
        case("verify", "8b", 1, 32, 4, 384, accept=4, name="8b_verify_b32_n4"),
        # block 64, draft depth 8: 576 rows
        case("verify", "8b", 1, 64, 8, 768, accept=3, name="8b_verify_b64_n8"),
        # four sequences with long prompts: 640 rows
        case("verify", "8b", 4, 32, 4, 1152, accept=4, name="8b_verify_batch4"),
        # eight sequences, depth 8, grouped-query heads: 2304 rows, the largest forward
        case("verify", "7b_gqa", 8, 32, 8, 640, accept=5, name="7b_verify_batch8_n8"),
        # time to the first token of a 1000-token prompt (no multiple of any tile)
        case("prefill", "8b", 1, 32, 4, 1000, name="8b_prefill"),
        # the dual cache renews all 512 positions every 8 decoded tokens
        case("refresh", "8b", 1, 8, 4, 392, gen=120, name="8b_refresh"),
        # one request of the paper's shape end to end
        case("generate", "8b", 1, 8, 4, 256, gen=32, name="8b_generate"),
    ]


def _log_int(rng, lo, hi):
    """An integer spread evenly over the logarithm of [lo, hi]."""
    return max(lo, min(hi, round(math.exp(rng.uniform(math.log(lo), math.log(hi))))))


def draw(rng: random.Random):
    mdl = rng.choice(["8b", "8b", "8b", "7b_gqa", "7b_gqa", "small_heads", "tiny"])
    kind = rng.choice(["draft", "verify", "verify", "verify", "prefill", "refresh", "generate"])
    small = mdl in ("tiny", "small_heads")
    block = rng.choice([8, 8, 16, 24, 32, 32, 64, 64])
    draft = rng.randint(3, 8)
    batch = 1
    if kind in ("draft", "verify"):
        nodes = 1 if kind == "draft" else draft + 1
        batch = max(1, min(8, _log_int(rng, 1, 16), (640 if small else 1984) // (nodes * block)))
    if kind in ("draft", "verify"):
        prefix, gen = _log_int(rng, 16, 200 if small else 1152), 0
    elif kind == "prefill":
        prefix, gen = _log_int(rng, 32, 200 if small else 1100), 0
    elif kind == "refresh":
        prefix, gen = _log_int(rng, 32, 120 if small else 700), block + _log_int(rng, 8, 100 if small else 256)
    else:
        block, draft = (rng.choice([8, 16, 32]), rng.randint(3, 5)) if small else (8, rng.randint(3, 5))
        prefix, gen = _log_int(rng, 16, 120 if small else 300), rng.randint(16, 64) if small else 8
    accept = rng.randint(0, draft) if mdl != "tiny" and kind == "verify" else 0
    return case(kind, mdl, batch, block, draft, prefix, gen, accept)


_STREAM = None


def _stream():
    """The program's decoding stream, one for all its contexts."""
    global _STREAM
    if _STREAM is None:
        _STREAM = torch.cuda.Stream()
    return _STREAM


def _inputs(case, seed):
    """Weights, prompts, block states and drafts of a case, from the seed alone."""
    cfg = model(case["model"])
    n, B, N, P, G = case["batch"], case["block"], case["draft"], case["prefix"], case["gen"]
    rng = random.Random(seed)
    w = synth.gen_weights(cfg, rng.randrange(1 << 30), device="cuda")
    V, mask = cfg["vocab"], cfg["mask_id"]
    shift = rng.randrange(1, V // 2)
    sure = (mask - shift) % V                     # the token a bf16 model predicts for a masked position
    if cfg["dtype"] == "bf16":
        w["embed"] *= 100.0                       # 0.02 -> 2: the embedding stays visible behind every layer
        w["lm_head"] = torch.roll(w["embed"], -shift, 0) * 0.125
    s = dict(cfg=cfg, w=w, prompts=[synth.gen_prompt(cfg, rng.randrange(1 << 30), P) for _ in range(n)])
    # the block: a quarter decoded already, the rest masked; drafts in the order of the masked positions,
    # `accept` of them what the model predicts
    toks, masks, drafts = [], [], []
    for i in range(n):
        open_ = sorted(rng.sample(range(B), max(min(B, N + 1), B - B // 4)))
        row = [rng.randrange(V - 1) for _ in range(B)]
        for p in open_:
            row[p] = mask
        toks.append(row)
        masks.append(sum(1 << p for p in open_))
        drafts.append([(p, sure if j < case["accept"] else (sure + 1 + rng.randrange(V - 2)) % (V - 1))
                       for j, p in enumerate(open_[:min(N, len(open_) - 1)])])
    s.update(toks=toks, masks=masks, drafts=drafts)
    if case["kind"] == "prefill":
        s["toks"], s["masks"] = [[mask] * B], [(1 << B) - 1]
    if case["kind"] == "refresh":
        s["sequence"] = list(s["prompts"][0]) + toks[0] + [mask] * (G - B)
    return s


def prepare(case, seed):
    n, B, N, P, G = case["batch"], case["block"], case["draft"], case["prefix"], case["gen"]
    s = _inputs(case, seed)
    torch.cuda.synchronize()                      # the library reads the weights on the decoding stream
    total = P + max(G, B)
    rows = max(P, total if case["kind"] == "refresh" else 0, n * (N + 1) * B)
    with torch.cuda.stream(_stream()):
        eng = binding.SSD(s.pop("cfg"), s.pop("w"), max_seqs=n, max_seq_len=total, block=B, max_draft=N, max_rows=rows)
        out = eng.new_out(n)
        s.update(case=case, eng=eng, out=out, seqs=list(range(n)), pos0=[P] * n)
        if case["kind"] in ("draft", "verify"):
            for i in range(n):
                eng.prefill_kv(i, s["prompts"][i], 0)
        _stream().synchronize()
    return s


def run(s):
    c, eng, out = s["case"], s["eng"], s["out"]
    if c["kind"] == "generate":
        toks, stats = eng.generate(s["prompts"], c["gen"], c["block"], c["draft"])
        return {"tokens": toks, "forwards": stats["forwards"], "accepted": stats["tokens"]}
    if c["kind"] == "refresh":
        eng.refresh_kv(0, s["sequence"], c["prefix"], c["block"], c["draft"], out)
    elif c["kind"] == "verify":
        eng.verify_tree(s["seqs"], s["toks"], s["masks"], s["pos0"], s["drafts"], c["draft"], out)
    else:
        if c["kind"] == "prefill":
            eng.prefill_kv(0, s["prompts"][0], 0)
        eng.draft(s["seqs"], s["toks"], s["masks"], s["pos0"], c["draft"], out)
    return {k: getattr(out, k) for k in ("n_accept", "acc_pos", "acc_tok", "n_next", "next_pos", "next_tok",
                                         "row_maxlogit", "row_argmax", "row_conf")}


def _forward(cfg, rows, logit_rows, keys, prefix_rows):
    """Bytes and operations of one forward: every weight it needs once, the cached keys and values it reads,
    2 operations per weight and row, 4 per key, row and query channel."""
    e = 4 if cfg["dtype"] == "fp32" else 2
    d, F, nq, nkv = cfg["d_model"], cfg["d_ffn"], cfg["n_q_heads"] * cfg["head_dim"], cfg["n_kv_heads"] * cfg["head_dim"]
    L, qkv, rest = cfg["n_layers"], (nq + 2 * nkv) * d, d * nq + 3 * F * d
    if logit_rows:
        weights = L * (qkv + rest) + cfg["vocab"] * d
        flops = 2 * rows * L * (qkv + rest) + 2 * logit_rows * cfg["vocab"] * d + 4 * rows * keys * nq * L
    else:                                          # a pure KV pass ends with the last layer's keys and values
        weights = L * qkv + (L - 1) * rest
        flops = 2 * rows * weights + 4 * rows * keys * nq * (L - 1)
    return dict(bytes=weights * e + prefix_rows * synth.kv_bytes_per_token(cfg) + rows * d * e, flops=flops)


def work(case):
    cfg = model(case["model"])
    n, B, N, P, G, kind = (case[k] for k in ("batch", "block", "draft", "prefix", "gen", "kind"))
    fw = []
    if kind == "draft":
        fw = [_forward(cfg, n * B, n * B, P + B, n * P)]
    elif kind == "verify":
        fw = [_forward(cfg, n * (N + 1) * B, n * (N + 1) * B, P + B, n * P)]
    elif kind == "prefill":
        fw = [_forward(cfg, P, 0, P, 0), _forward(cfg, B, B, P + B, P)]
    elif kind == "refresh":
        fw = [_forward(cfg, P + G, B, P + G, 0)]
    else:
        # the prompt, and per block the self-draft and at least ceil((B - 1) / (N + 1)) verification rounds
        fw = [_forward(cfg, P, 0, P, 0)]
        for b in range(0, G, B):
            bl = min(B, G - b)
            fw.append(_forward(cfg, bl, bl, P + b + bl, P + b))
            left = bl - 1
            while left > 0:
                nodes = min(N + 1, left)
                fw.append(_forward(cfg, nodes * bl, nodes * bl, P + b + bl, P + b))
                left -= N + 1
    return dict(bytes=sum(f["bytes"] for f in fw), flops=sum(f["flops"] for f in fw))


def tolerance(case):
    if case["kind"] == "generate":
        return "exact"                             # tokens and counts
    if case["model"] == "tiny":
        return {"rel": 2e-5, "max": 2e-4}
    return {"rel": 0.008, "max": 0.05}      # four times what the plain kernels differ from the matrix-core ones by


def _rows64(cfg, w, tokens, pos, kv, keep, heads=8):
    """The layers in 64 bits for sets of rows: tokens / pos [sets, rows], kv: per layer the cached (keys, values)
    [positions, heads, channels] the rows see besides their own set's.  Returns the hidden rows and, with keep,
    every layer's keys and values of the one set."""
    dh, Hq, Hkv, F = cfg["head_dim"], cfg["n_q_heads"], cfg["n_kv_heads"], cfg["d_ffn"]
    n, B = tokens.shape
    f64 = torch.float64
    norm = lambda x, g: x / torch.sqrt((x * x).mean(-1, keepdim=True) + cfg["rms_eps"]) * g.to(f64)
    ang = pos.to(f64)[..., None] * cfg["rope_theta"] ** (torch.arange(dh // 2, device=pos.device, dtype=f64) * (-2.0 / dh))
    cos, sin = torch.cos(ang)[:, :, None], torch.sin(ang)[:, :, None]
    turn = lambda x: torch.cat([x[..., :dh // 2] * cos - x[..., dh // 2:] * sin, x[..., dh // 2:] * cos + x[..., :dh // 2] * sin], -1)
    h, kept = w["embed"][tokens].to(f64), []
    for l, lw in enumerate(w["layers"]):
        x = norm(h, lw["norm1"]) @ lw["wqkv"].to(f64).T
        q, k, v = (t.reshape(n, B, -1, dh) for t in x.split([Hq * dh, Hkv * dh, Hkv * dh], -1))
        q, k = turn(q), turn(k)
        if keep:
            kept.append((k[0], v[0]))
        if kv is not None:
            k = torch.cat([kv[l][0].expand(n, -1, -1, -1), k], 1)
            v = torch.cat([kv[l][1].expand(n, -1, -1, -1), v], 1)
        a = torch.empty_like(q)
        for i in range(n):
            for h0 in range(0, Hq, heads):
                hs = torch.arange(h0, min(Hq, h0 + heads), device=pos.device)
                kk, vv = (t[i].transpose(0, 1)[hs // (Hq // Hkv)].contiguous() for t in (k, v))
                p = torch.softmax(q[i][:, hs].transpose(0, 1).contiguous() @ kk.transpose(1, 2).contiguous() / math.sqrt(dh), -1)
                a[i][:, hs] = (p @ vv).transpose(0, 1)
        h = h + a.reshape(n, B, Hq * dh) @ lw["wo"].to(f64).T
        x = norm(h, lw["norm2"]) @ lw["wgu"].to(f64).T
        h = h + (torch.nn.functional.silu(x[..., :F]) * x[..., F:]) @ lw["wdown"].to(f64).T
    return norm(h, w["final_norm"]), kept


def _head64(cfg, w, x):
    """Largest logit of every row and its softmax probability, the mask token left out."""
    top, total = torch.full(x.shape[:-1], -math.inf, device=x.device, dtype=x.dtype), torch.zeros(x.shape[:-1], device=x.device, dtype=x.dtype)
    for v0 in range(0, cfg["vocab"], 16384):
        lg = x @ w["lm_head"][v0:v0 + 16384].to(x.dtype).T
        if v0 <= cfg["mask_id"] < v0 + 16384:
            lg[..., cfg["mask_id"] - v0] = -math.inf
        new = torch.maximum(top, lg.amax(-1))
        total = total * torch.exp(top - new) + torch.exp(lg - new[..., None]).sum(-1)
        top = new
    return top, 1.0 / total


def exact(case, seed):
    """The maximum logits and confidences in 64 bits (whole numbers have no such value, nor have tokens)."""
    if case["kind"] == "generate":
        return None
    s = _inputs(case, seed)
    cfg, w = s["cfg"], s["w"]
    n, B, N, P, G = case["batch"], case["block"], case["draft"], case["prefix"], case["gen"]
    dev = w["embed"].device
    top = torch.zeros(n, N + 1, B, device=dev, dtype=torch.float64)
    conf = torch.zeros_like(top)
    span = lambda a, b: torch.arange(a, b, device=dev)
    for i in range(n):
        if case["kind"] == "refresh":
            t = torch.tensor([[int(v) for v in s["sequence"]]], device=dev)
            x = _rows64(cfg, w, t, span(0, P + G)[None], None, False)[0][:, P:P + B]
        else:
            prompt = torch.tensor([[int(v) for v in s["prompts"][i]]], device=dev)
            kv = _rows64(cfg, w, prompt, span(0, P)[None], None, True)[1]
            nodes = []
            for j in range((len(s["drafts"][i]) if case["kind"] == "verify" else 0) + 1):
                row = list(s["toks"][i])
                for p, tok in s["drafts"][i][:j]:
                    row[p] = tok
                nodes.append(row)
            t = torch.tensor(nodes, device=dev)
            x = _rows64(cfg, w, t, span(P, P + B).expand(len(nodes), B), kv, False)[0]
        top[i, :x.shape[0]], conf[i, :x.shape[0]] = _head64(cfg, w, x)
    return dict(n_accept=None, acc_pos=None, acc_tok=None, n_next=None, next_pos=None, next_tok=None,
                row_maxlogit=top, row_argmax=None, row_conf=conf)
