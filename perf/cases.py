"""What the performance of the verify step is measured on: the work a user has
this framework do, through its public entry points.

A case names a decoder shape of workloads/configs.py, optionally cut to its first
layers, and one of four uses of it:

* ``verify``   verify + commit of one step over a batch of sequences
               (chain drafts from a drafter or from the suffix cache; k = 0 is
               a plain greedy step);
* ``tree``     verify + commit of one token-tree draft per sequence;
* ``prefill``  a new prompt, up to its first logits (time to first token);
* ``loop``     the device-resident verify loop: open, a number of steps with
               the copy drafter, close, and one greedy step after it.

The weights are random but for one thing: embedding row t points along LM-head
row (t + SHIFT) mod vocab, strongly enough that this token is the model's
clear choice after t, as a trained model's usually is.  So drafts with a chosen
number of accepted tokens can be drawn from the seed alone, no top-2 near tie
lies on any accepted path, and accepted lengths and tokens compare exactly.
One process holds one copy of each model's weights, as a serving program does;
prompts, drafts and acceptance come from the seed.
"""

import math

import numpy as np
import torch

from workloads import tokens as wt
from workloads import trees
from workloads.configs import config_by_name

SHIFT = 7919          # the clear next token after t is (t + SHIFT) % vocab
EMBED_STD = 0.35      # x sqrt(layers): the embedding's share of the residual stream
MAX_ROWS = 848        # rows of the largest listed verify batch
MAX_CTX = {"8b": 20000}  # cached positions of a drawn batch (65536 for the cut shapes)
MAX_PROMPT = {"8b": 3500, "32b-L4": 12000, "tiny": 3500}  # longest drawn prompt (16384 else)


# ------------------------------------------------------------------- the cases

def _case(kind, model, batch=1, ctx=(2048, 2048), k=(8, 8), drafts="each", shape=1, pair=False, steps=0):
    return {"kind": kind, "model": model, "batch": batch, "ctx_lo": ctx[0], "ctx_hi": ctx[1], "k_lo": k[0],
            "k_hi": k[1], "drafts": drafts, "shape": shape, "pair": pair, "steps": steps}


def listed():
    return [
        # the smallest decoder: a step of a few launches, where latency counts
        {"name": "tiny chain k=8", **_case("verify", "tiny", ctx=(511, 511))},
        # one user, one token: the greedy step between drafts
        {"name": "8b greedy", **_case("verify", "8b", k=(0, 0))},
        # the headline: one user, a drafter's chain (9 rows, one row tile)
        {"name": "8b chain k=8", **_case("verify", "8b")},
        # one user, a longer chain at a ragged context (17 rows, two row tiles)
        {"name": "8b chain k=16", **_case("verify", "8b", ctx=(3001, 3001), k=(16, 16))},
        # a model drafter's token tree (33 rows)
        {"name": "8b tree 32", **_case("tree", "8b", k=(32, 32), shape=2)},
        # a suffix-cache draft over an agentic session's long context (65 rows)
        {"name": "8b cache k=64 ctx 16k", **_case("verify", "8b", ctx=(16384, 16384), k=(64, 64))},
        # a small serving batch with a drafter's chains (72 rows)
        {"name": "8b batch 8", **_case("verify", "8b", batch=8, ctx=(700, 4000))},
        # a serving batch of short chains and long cache drafts (several hundred rows), 8 layers
        {"name": "8b-L8 mixed batch 32", **_case("verify", "8b-L8", batch=32, ctx=(1024, 8192), k=(8, 64), drafts="mixed")},
        # the 32B widths, cache drafts at context 8192 (about 270 rows), 4 layers; both
        # MLP GEMMs on the hi + lo pair, as the full 64 layers run
        {"name": "32b-L4 batch 8", **_case("verify", "32b-L4", batch=8, ctx=(8192, 8192), k=(4, 64), drafts="uniform", pair=True)},
        # a chat prompt up to its first logits
        {"name": "8b prefill 2k", **_case("prefill", "8b", ctx=(2047, 2047), k=(0, 0))},
        # a long prompt, 8 layers
        {"name": "8b-L8 prefill 16k", **_case("prefill", "8b-L8", ctx=(16000, 16000), k=(0, 0))},
        # the loop that stays on the device: 16 steps of k = 8 with the copy drafter
        {"name": "8b device loop", **_case("loop", "8b", steps=16)},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("verify", "verify", "verify", "verify", "tree", "prefill", "prefill", "loop"))
    model = rng.choice(("8b", "8b", "8b-L8", "8b-L8", "32b-L4", "tiny"))
    top = 3500 if model == "tiny" else 16384  # the tiny shape's rotary table ends at 4096
    shape = rng.randrange(1 << 20)
    pair = rng.random() < 0.2  # the exact-numerics setting of the MLP
    if kind == "prefill":
        n = _log_int(rng, 48, MAX_PROMPT.get(model, 16384))
        return _case(kind, model, ctx=(n, n), k=(0, 0), shape=shape, pair=pair)
    if kind == "loop":
        n = _log_int(rng, 64, top // 2)
        k = rng.choice((0, 2, 4, 5, 8, 12, 16))
        return _case(kind, model, ctx=(n, n), k=(k, k), shape=shape, steps=rng.randrange(4, 17))
    batch = 1 if rng.random() < 0.5 else _log_int(rng, 2, 32)
    hi = min(top, MAX_CTX.get(model, 65536) // batch)
    lo = _log_int(rng, 64, hi)
    ctx = (lo, lo) if rng.random() < 0.5 else (lo, _log_int(rng, lo, hi))
    most = min(64, MAX_ROWS // batch - 1)
    if kind == "tree":
        n = rng.randrange(4, min(63, most) + 1)
        return _case(kind, model, batch=batch, ctx=ctx, k=(n, n), shape=shape, pair=pair)
    k = min(most, _log_int(rng, 1, 65) - 1)
    drafts = rng.choice(("each", "uniform", "mixed"))
    return _case(kind, model, batch=batch, ctx=ctx, k=(k if drafts == "each" else min(k, 8), k), drafts=drafts, shape=shape, pair=pair)


def _shapes(case):
    """(context lengths, draft lengths) of the batch; the context is the
    number of cached positions before the step."""
    B = case["batch"]
    r = np.random.default_rng([case["shape"], B])
    ctx = r.integers(case["ctx_lo"], case["ctx_hi"] + 1, size=B)
    lo, hi = case["k_lo"], case["k_hi"]
    if case["drafts"] == "each":
        k = np.full(B, hi)
    else:
        k = r.integers(lo if case["drafts"] == "uniform" else min(16, hi), hi + 1, size=B)
        if case["drafts"] == "mixed":  # the first half short chains
            k[: B // 2] = lo
    return [int(c) for c in ctx], [int(x) for x in k]


# --------------------------------------------------------------------- weights

_host, _models = {}, {}


def _weights(name):
    """The canonical tensors as host uint16 bf16 bits (one set per shape)."""
    if name not in _host:
        c = config_by_name(name)
        gen = torch.Generator("cuda").manual_seed(20 + c.n_layers)
        rnd = lambda *s, std=0.02: torch.randn(*s, generator=gen, device="cuda", dtype=torch.float32).mul_(std)
        bits = lambda t: t.to(torch.bfloat16).view(torch.int16).cpu().numpy().view(np.uint16)
        D, F, V = c.d_model, c.ffn_dim, c.vocab
        w = {}
        lm = rnd(V, D)
        w["embed"] = bits(torch.roll(lm, -SHIFT % V, 0).mul_(EMBED_STD * math.sqrt(c.n_layers) / 0.02))
        for l in range(c.n_layers):
            p = f"layers.{l}."
            for n, s in (("wq", (c.q_dim, D)), ("wk", (c.kv_dim, D)), ("wv", (c.kv_dim, D)), ("wo", (D, c.q_dim)),
                         ("wg", (F, D)), ("wu", (F, D)), ("wd", (D, F))):
                w[p + n] = bits(rnd(*s))
            for n in ("attn_norm", "mlp_norm"):
                w[p + n] = bits(rnd(D, std=0.1).add_(1.0))
        w["final_norm"] = bits(rnd(D, std=0.1).add_(1.0))
        w["lm_head"] = bits(lm)
        _host[name] = w
    return _host[name]


def _model(name):
    if name not in _models:
        import paper_2606_01019_amd as hvd
        _models[name] = hvd.Model(config_by_name(name), _weights(name))
    return _models[name]


# ---------------------------------------------------------------------- inputs

def _greedy(token, n, vocab):
    """The model's n next tokens after `token`."""
    return (int(token) + SHIFT * np.arange(1, n + 1, dtype=np.int64)) % vocab


def _inputs(case, seed):
    """Prompts (the last token becomes the pending one), drafts or trees, and
    for a loop the copy drafter's stream, of every sequence."""
    c = config_by_name(case["model"])
    ctx, ks = _shapes(case)
    out = {"ctx": ctx, "prompts": [], "drafts": [], "trees": [], "ref": None}
    for b, (n, k) in enumerate(zip(ctx, ks)):
        r = np.random.default_rng([seed, b])
        # natural-language-like ranks; long sessions repeat their own segments
        make = wt.segment_context if n > 8192 else wt.zipf_context
        prompt = make(r, n + 1, c.vocab)
        out["prompts"].append(prompt)
        greedy = _greedy(prompt[-1], max(k, 1) + 1, c.vocab)
        if case["kind"] == "tree":
            parents = trees.eagle_tree(np.random.default_rng([case["shape"], b, 7]), n_nodes=k)
            depth = max(len(trees.path_to(parents, j)) for j in range(len(parents)))
            a = int(r.integers(0, min(depth, 4) + 1))
            out["trees"].append((trees.plant_path(r, parents, _greedy(prompt[-1], depth + 1, c.vocab), a, c.vocab), parents))
        else:
            a = wt.uniform_accept(r, k) if k > 16 else wt.geometric_accept(r, 0.3, k)
            out["drafts"].append(wt.plant_cache_draft(r, prompt, greedy, a, k, c.vocab) if k > 16
                                 else wt.plant_chain(r, greedy, a, k, c.vocab))
        if case["kind"] == "loop":
            n_ref = (case["steps"] + 1) * (k + 1)
            out["ref"] = wt.corrupt_stream(r, _greedy(prompt[-1], n_ref, c.vocab), 0.3, c.vocab)
    return out


def prepare(case, seed):
    import paper_2606_01019_amd as hvd
    m = _model(case["model"])
    x = _inputs(case, seed)
    ctx, B = x["ctx"], case["batch"]
    room = case["steps"] * (case["k_hi"] + 1) + 72
    kv = hvd.KVCache(m, max_seqs=B, n_pages=sum((n + room) // 16 + 2 for n in ctx))
    if case["pair"]:
        kv.set_mlp_single(False)
    rows = {"prefill": 1, "loop": 1, "tree": sum(len(t) + 1 for t, _ in x["trees"]),
            "verify": sum(len(d) + 1 for d in x["drafts"])}[case["kind"]]
    st = {"case": case, "kv": kv, "ids": list(range(B)), "ctx": ctx, "drafts": x["drafts"], "trees": x["trees"],
          "prompts": x["prompts"], "pending": [int(p[-1]) for p in x["prompts"]], "live": False,
          "logits": torch.zeros(rows, m.cfg.vocab, dtype=torch.float32, device="cuda")}
    if case["kind"] == "loop":
        st["ref"] = torch.from_numpy(x["ref"]).to("cuda").reshape(1, -1)
    if case["kind"] != "prefill":
        for b in range(B):
            kv.prefill(b, x["prompts"][b])
    return st


_NONE = np.zeros(0, np.int32)


def run(st):
    case, kv, ids = st["case"], st["kv"], st["ids"]
    if case["kind"] == "prefill":
        if st["live"]:
            kv.seq_free(0)  # the previous request has ended
        kv.prefill(0, st["prompts"][0])
        st["live"] = True
        acc, nxt = kv.verify(ids, st["ctx"], [_NONE], logits=st["logits"])
        kv.commit(ids)
        return {"logits": st["logits"], "accepted": acc, "next": nxt}
    if st["live"]:  # the same step again: back to the prompt
        for b in ids:
            kv.truncate(b, st["ctx"][b], st["pending"][b])
    st["live"] = True
    if case["kind"] == "loop":
        loop = kv.async_loop(ids, st["ctx"], [case["k_hi"]], case["steps"], ref=st["ref"], ref_start=[st["ctx"][0] + 1])
        loop.step(case["steps"])
        loop.end()
        ctx, _, _ = kv.seq_info(0)
        acc, nxt = kv.verify(ids, [ctx], [_NONE], logits=st["logits"])
        kv.commit(ids)
        return {"logits": st["logits"], "next": nxt, "history": loop.history, "state": loop.state}
    if case["kind"] == "tree":
        acc, nxt, paths = kv.verify_tree(ids, st["ctx"], st["trees"], logits=st["logits"])
        kv.commit(ids)
        path = np.array([p + [-1] * (63 - len(p)) for p in paths])
        return {"logits": st["logits"], "accepted": acc, "next": nxt, "paths": path}
    acc, nxt = kv.verify(ids, st["ctx"], st["drafts"], logits=st["logits"])
    kv.commit(ids)
    return {"logits": st["logits"], "accepted": acc, "next": nxt}


# ------------------------------------------------------------- work, tolerance

def _layer_params(c):
    return c.d_model * (2 * c.q_dim + 2 * c.kv_dim + 3 * c.ffn_dim)


def _forward_work(c, seqs, lm_rows):
    """(bytes, flops) of one forward over seqs = [(cached, rows)]: weights and
    cached K/V read once, the rows' K/V and the logits written once."""
    M = sum(r for _, r in seqs)
    by = 2.0 * c.n_layers * _layer_params(c) + 2.0 * c.d_model * M
    by += sum(4.0 * c.kv_dim * c.n_layers * (n + r) for n, r in seqs)
    fl = 2.0 * M * c.n_layers * _layer_params(c)
    fl += sum(4.0 * c.q_dim * c.n_layers * r * (n + (r + 1) / 2.0) for n, r in seqs)
    if lm_rows:
        by += 2.0 * c.vocab * c.d_model + 4.0 * lm_rows * c.vocab
        fl += 2.0 * lm_rows * c.vocab * c.d_model
    return by, fl


def work(case):
    c = config_by_name(case["model"])
    ctx, ks = _shapes(case)
    if case["kind"] == "prefill":
        parts = [_forward_work(c, [(0, ctx[0] + 1)], 1)]
    elif case["kind"] == "loop":  # the drafts are accepted about twice a step
        k = ks[0]
        parts = [_forward_work(c, [(ctx[0] + min(k + 1, 3) * s, k + 1)], 0) for s in range(case["steps"])]
        parts = [(b + 2.0 * c.vocab * c.d_model, f + 2.0 * (k + 1) * c.vocab * c.d_model) for b, f in parts]
        parts.append(_forward_work(c, [(ctx[0] + min(k + 1, 3) * case["steps"], 1)], 1))
    else:
        if case["kind"] == "tree":
            ks = [len(trees.eagle_tree(np.random.default_rng([case["shape"], b, 7]), n_nodes=k)) for b, k in enumerate(ks)]
        seqs = [(n, k + 1) for n, k in zip(ctx, ks)]
        parts = [_forward_work(c, seqs, sum(r for _, r in seqs))]
    return {"bytes": sum(p[0] for p in parts), "flops": sum(p[1] for p in parts)}


def tolerance(case):
    # fp16 K/V, queries and probabilities and the fp16 gate/up activation, over
    # up to 32 layers: measured against exact(), the logits are off by 0.02%
    # (tiny), 0.06-0.11% (4 to 8 layers) and 0.13-0.18% (32 layers)
    return {"rel": 2e-3, "max": 2e-2} if case["model"] == "tiny" else {"rel": 6e-3, "max": 5e-2}


# ------------------------------------------------------------- 64-bit outcome

def _committed(case, x, c):
    """Tokens a loop commits after the pending one: the model's own choices."""
    k, ref, pos = case["k_hi"], x["ref"], 0
    for _ in range(case["steps"]):
        want = _greedy(x["prompts"][0][-1], pos + k + 1, c.vocab)[pos:]
        a = 0
        while a < k and int(ref[pos + a]) == int(want[a]):
            a += 1
        pos += a + 1
    return _greedy(x["prompts"][0][-1], pos, c.vocab)


def exact(case, seed):
    c = config_by_name(case["model"])
    if sum(_shapes(case)[0]) * c.n_layers * _layer_params(c) > 3.2e14:
        return None  # over about 20 seconds
    x = _inputs(case, seed)
    w = _weights(case["model"])
    f64 = lambda n: torch.from_numpy(w[n].view(np.int16)).to("cuda").view(torch.bfloat16).to(torch.float64)
    D, H, Hk, dh = c.d_model, c.n_q_heads, c.n_kv_heads, c.head_dim
    # each sequence: all its tokens, their positions, how many are rows of the
    # step, and which rows of the step each row sees (None: those before it)
    seqs = []
    for b in range(case["batch"]):
        p = x["prompts"][b]
        toks, see, tail = [int(t) for t in p], None, []
        if case["kind"] == "verify":
            tail = [int(t) for t in x["drafts"][b]]
            pos = list(range(len(toks) + len(tail)))
        elif case["kind"] == "tree":
            t, parents = x["trees"][b]
            tail = [int(v) for v in t]
            paths = [trees.path_to(parents, j) for j in range(len(parents))]
            pos = list(range(len(toks))) + [len(toks) - 1 + len(q) for q in paths]
            see = torch.zeros(len(tail) + 1, len(tail) + 1, dtype=torch.bool)
            see[:, 0] = True
            for j, q in enumerate(paths):
                see[j + 1, [i + 1 for i in q]] = True
        else:
            if case["kind"] == "loop":
                toks += [int(t) for t in _committed(case, x, c)]
            pos = list(range(len(toks)))
        seqs.append((toks + tail, pos, len(tail) + 1, see))
    n_tok = [len(s[0]) for s in seqs]
    start = np.cumsum([0] + n_tok)
    toks = torch.tensor(sum((s[0] for s in seqs), []), device="cuda")
    pos = torch.tensor(sum((s[1] for s in seqs), []), device="cuda", dtype=torch.float64)
    ang = pos[:, None] * c.rope_theta ** (-2.0 * torch.arange(dh // 2, device="cuda", dtype=torch.float64) / dh)
    cos, sin = torch.cos(ang)[:, None], torch.sin(ang)[:, None]
    emb = torch.from_numpy(w["embed"].view(np.int16))[toks.cpu()].to("cuda").view(torch.bfloat16).to(torch.float64)
    h, STEP = emb, 8192

    def rms(v, gain):
        return v / torch.sqrt((v * v).mean(-1, keepdim=True) + c.rms_eps) * gain

    def rot(v):
        u, z = v[..., : dh // 2], v[..., dh // 2:]
        return torch.cat((u * cos - z * sin, z * cos + u * sin), -1)

    def attend(q, kt, v, rows, n, see):
        """q [H, r, dh] of rows `rows`.. of a sequence of n tokens."""
        r = q.shape[1]
        top = rows + r
        s = torch.bmm(q, kt[:, :, :top].contiguous()).mul_(dh ** -0.5)
        i = torch.arange(rows, top, device="cuda")[:, None]
        j = torch.arange(top, device="cuda")[None]
        hide = j > i
        if see is not None:  # tree rows: the context, then their own path
            first = n - see.shape[0]
            if top > first:
                lo = max(0, first - rows)
                hide[lo:, first:] = ~see[rows + lo - first: top - first, : top - first].to("cuda")
        s.masked_fill_(hide, -math.inf)
        return torch.bmm(torch.softmax(s, -1), v[:, :top].contiguous())

    for l in range(c.n_layers):
        p = f"layers.{l}."
        y = rms(h, f64(p + "attn_norm"))
        q = rot((y @ f64(p + "wq").T).view(-1, H, dh))
        kk = rot((y @ f64(p + "wk").T).view(-1, Hk, dh))
        v = (y @ f64(p + "wv").T).view(-1, Hk, dh)
        o = torch.empty_like(q)
        for b, (_, _, R, see) in enumerate(seqs):
            a, e, n, G = start[b], start[b + 1], n_tok[b], H // Hk
            # the last layer only has to serve the step's own rows
            first = n - R if l == c.n_layers - 1 else 0
            block = max(64, (1 << 28) // (G * n))
            for g in range(Hk):  # one kv head at a time bounds the score matrix
                kt, vg = kk[a:e, g].T.contiguous()[None].expand(G, -1, -1), v[a:e, g][None].expand(G, -1, -1)
                for r0 in range(first, n, block):
                    r1 = min(n, r0 + block)
                    qb = q[a + r0: a + r1, g * G:(g + 1) * G].transpose(0, 1).contiguous()
                    o[a + r0: a + r1, g * G:(g + 1) * G] = attend(qb, kt, vg, r0, n, see).transpose(0, 1)
        if l == c.n_layers - 1:
            keep = torch.cat([torch.arange(start[b + 1] - s[2], start[b + 1]) for b, s in enumerate(seqs)]).to("cuda")
            h, o = h[keep], o[keep]
        h = h + o.reshape(len(o), -1) @ f64(p + "wo").T
        wg, wu, wd = f64(p + "wg").T, f64(p + "wu").T, f64(p + "wd").T
        gain = f64(p + "mlp_norm")
        for r0 in range(0, len(h), STEP):
            y = rms(h[r0: r0 + STEP], gain)
            h[r0: r0 + STEP] += (torch.nn.functional.silu(y @ wg) * (y @ wu)) @ wd
        del wg, wu, wd
    out = {"logits": rms(h, f64("final_norm")) @ f64("lm_head").T}
    none = {"verify": ("accepted", "next"), "prefill": ("accepted", "next"), "tree": ("accepted", "next", "paths"),
            "loop": ("next", "history", "state")}[case["kind"]]
    return {**out, **{n: None for n in none}}
