"""Performance cases of the verification step, through the library's public Python entry points.

A case is one model (a width the repository's configurations name, cut in depth so that it loads in about a
second), one cache with a prefix, and a short run of steps on it.  Depth is cut and the vocabulary with it, so that
the head keeps about the share of a step that it has in the whole model (a 32-layer model with 128256 tokens becomes 4 layers
with 16384); one case keeps a whole 128256-token head.

Every verify pass is `steps` blocks on the same prefix whose first draft token is not the pending one: the block is
computed, nothing is accepted, the cache stays as it is, and the pass can be repeated.  What a step costs does
not depend on how many tokens it accepts.  A prefill pass rolls the cache back to nothing, puts the prompt in and verifies one
block on top of it.  Outputs: the last block's logits, what the steps returned, and the whole K/V pool (the torch
tensor the cache object owns), in the page layout the library documents.
"""
import math
import random

import numpy as np
import torch

import paper_2505_01572_amd as pv
from pv_inputs import CONFIGS, ModelShape

SIGMA = 0.02                                # every matrix is N(0, 0.02^2), norm gains 1 + N(0, 0.02^2)
PIECE = 16 << 20                            # weights go in in pieces of at most this many elements ...
POOL = PIECE + (1 << 20)                    # ... each a window of one pool of draws at an offset of its own

# Widths: the repository's benchmark configurations, and two ragged shapes of its tests (65 K-tiles and 129 of them).
WIDTHS = {name: CONFIGS[name] for name in ("tiny", "1b", "7b", "8b", "70b", "8b_q4", "70b_q4")}
WIDTHS["ragged_2080"] = ModelShape("ragged_2080", 2, 2080, 8, 2, 128, 4096, 8192, rope_base=500000.0)
WIDTHS["ragged_4128"] = ModelShape("ragged_4128", 2, 1024, 8, 2, 128, 4128, 2000, rope_base=500000.0)

MATRICES = ("wq", "wk", "wv", "wo", "wg", "wu", "wd")
PER_LAYER = ("attn_norm", "wq", "wk", "wv", "wo", "ffn_norm", "wg", "wu", "wd")
Q4_KINDS = MATRICES + ("lm_head",)


def listed():
    return [
        # the smallest call: the two-layer fp32 configuration (vector path), where launches and the host count
        {"name": "tiny_f32_g4", "do": "verify", "width": "tiny", "layers": 2, "vocab": 1024, "prefix": 100, "rows": 4, "steps": 8},
        # the drafter of the three-stage pipeline: one token at a time, whole 128256-token head
        {"name": "draft_1b_g1", "do": "verify", "width": "1b", "layers": 8, "vocab": 128256, "prefix": 1024, "rows": 1, "steps": 16},
        # multi-head attention (no GQA), an odd window
        {"name": "verify_7b_g5", "do": "verify", "width": "7b", "layers": 4, "vocab": 4000, "prefix": 517, "rows": 5, "steps": 8},
        # the headline: 8B-shaped verifier, window 8, prefix 2048
        {"name": "verify_8b_g8", "do": "verify", "width": "8b", "layers": 4, "vocab": 16384, "prefix": 2048, "rows": 8, "steps": 8},
        # the final stage of the pipeline in 16 bit
        {"name": "verify_70b_g8", "do": "verify", "width": "70b", "layers": 2, "vocab": 800, "prefix": 1024, "rows": 8, "steps": 4},
        # the final stage as the paper runs it, in 4 bit
        {"name": "verify_70b_q4_g8", "do": "verify", "width": "70b_q4", "layers": 4, "vocab": 1600, "prefix": 1024, "rows": 8, "steps": 4},
        # a window over 8 rows, in 4 bit, with an odd size
        {"name": "verify_8b_q4_g13", "do": "verify", "width": "8b_q4", "layers": 4, "vocab": 16384, "prefix": 777, "rows": 13, "steps": 8},
        # a long context: 16384 cached tokens, short window, shuffled pages
        {"name": "verify_8b_16k_g4", "do": "verify", "width": "8b", "layers": 2, "vocab": 8192, "prefix": 16384, "rows": 4, "steps": 8, "shuffled": True},
        # four sequences of different lengths in one pass over the weights
        {"name": "batch_8b_4x8", "do": "batch", "width": "8b", "layers": 4, "vocab": 16384, "prefix": 2048, "rows": 8, "seqs": 4, "steps": 8, "shuffled": True},
        # a draft tree of 48 nodes
        {"name": "tree_8b_48", "do": "tree", "width": "8b", "layers": 4, "vocab": 16384, "prefix": 1024, "rows": 48, "steps": 8},
        # a prompt, 16 bit: the largest
        {"name": "prefill_8b_2048", "do": "prefill", "width": "8b", "layers": 4, "vocab": 16384, "prefix": 2048, "rows": 8, "steps": 1},
        # a ragged prompt, 4 bit
        {"name": "prefill_70b_q4_1000", "do": "prefill", "width": "70b_q4", "layers": 2, "vocab": 800, "prefix": 1000, "rows": 8, "steps": 1},
    ]


def draw(rng):
    """One more case: any width, any kind of call, windows of 1 to 64 rows, prefixes of 1 to 12000 tokens."""
    log = lambda lo, hi: int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))  # noqa: E731
    do = rng.choice(["verify"] * 4 + ["batch", "tree"] + ["prefill"] * 3)
    width = rng.choice([w for w in sorted(WIDTHS) if not (do in ("batch", "tree") and WIDTHS[w].dtype == "f32")])
    big = width.startswith("70b")
    case = {"do": do, "width": width, "layers": 1 if big else rng.randint(1, 3), "vocab": 16 * rng.randint(50, 1024), "steps": rng.randint(2, 8)}
    if do == "prefill":
        room = 3.5e12 / (2 * params(dict(case, rows=1)))
        case.update(prefix=log(17, max(18, min(6000, int(room)))), rows=log(1, 16), steps=1)
    else:
        case.update(prefix=log(1, 4000 if big else 12000), rows=log(2 if do == "tree" else 1, 64))
    if do == "batch":
        case["seqs"] = rng.randint(2, 8)
        case["rows"] = max(1, min(case["rows"], 64 // case["seqs"]))
        case["prefix"] = min(case["prefix"], 3000)
    if WIDTHS[width].dtype == "f32":
        case["prefix"] = min(case["prefix"], 600)
    if rng.random() < 0.4:
        case["shuffled"] = True
    return case


# ---- the model of a case ----

def shape_of(case):
    w = WIDTHS[case["width"]]
    return w.replace(n_layers=case["layers"], vocab=case["vocab"], name=w.name + "_cut")


def dims(s, kind):
    qd, kvd = s.n_q_heads * s.head_dim, s.n_kv_heads * s.head_dim
    return {"embed": (s.vocab, s.d_model), "wq": (qd, s.d_model), "wk": (kvd, s.d_model), "wv": (kvd, s.d_model), "wo": (s.d_model, qd),
            "wg": (s.ffn_dim, s.d_model), "wu": (s.ffn_dim, s.d_model), "wd": (s.d_model, s.ffn_dim), "lm_head": (s.vocab, s.d_model)}.get(kind, (1, s.d_model))


def params(case):
    """Weights that a step multiplies with."""
    s = shape_of(case)
    return s.n_layers * sum(math.prod(dims(s, k)) for k in MATRICES) + math.prod(dims(s, "lm_head"))


def is_q4(s, kind):
    return s.weight_bits == 4 and kind in Q4_KINDS


def pieces(s, seed):
    """(kind, layer, first row, rows, columns, offset into the pool) of every piece of every tensor."""
    r = random.Random(seed)
    for kind, layer in [("embed", 0)] + [(k, l) for l in range(s.n_layers) for k in PER_LAYER] + [("final_norm", 0), ("lm_head", 0)]:
        rows, cols = dims(s, kind)
        step = max(16, PIECE // cols // 16 * 16)
        for r0 in range(0, rows, step):
            yield kind, layer, r0, min(step, rows - r0), cols, 32 * r.randrange((POOL - PIECE) // 32)


def pool_of(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.randn(POOL, generator=g, device="cuda", dtype=torch.float32) * SIGMA


def quantised(pool):
    """The pool as 4-bit codes and bf16 scales per 32 values (weight = (code - 8) * scale)."""
    v = pool.to(torch.bfloat16).float().view(-1, 32)
    scale = (v.abs().amax(1, keepdim=True) / 7).to(torch.bfloat16)
    return (torch.round(v / scale.float()) + 8).clamp_(0, 15).to(torch.uint8).view(-1), scale.view(-1)


def inputs_of(case, seed):
    """Token ids of a case: prompts, one block per step and (trees) parents, pending tokens that no block starts with."""
    s, r = shape_of(case), np.random.default_rng(seed)
    n = case.get("seqs", 1)
    lens = [max(1, case["prefix"] * (n - i) // n - 3 * i) for i in range(n)]           # ragged from the whole prefix down
    prompts = [r.integers(0, s.vocab, m, dtype=np.int32) for m in lens]
    blocks = [[r.integers(0, s.vocab, case["rows"], dtype=np.int32) for _ in range(n)] for _ in range(case["steps"])]
    pending = [int(r.integers(0, s.vocab)) for _ in range(n)]
    for step in blocks:
        for p, b in zip(pending, step):
            b[b == p] = (p + 1) % s.vocab
    # a tree's nodes hang under one of the few nodes before them or under the prefix, as a beam of drafts does
    parents = [np.array([-1 if i == 0 else int(r.integers(max(-1, i - 6), i)) for i in range(case["rows"])], dtype=np.int32) for _ in range(case["steps"])]
    room = max(lens) + case["rows"] + 16
    pages = -(-room // s.page_tokens)
    tables = [r.permutation(pages).astype(np.int32) if case.get("shuffled") else np.arange(pages, dtype=np.int32) for _ in range(n)]
    return prompts, blocks, pending, parents, tables, room


# ---- what a user's program has in hand, and the pass ----

def prepare(case, seed):
    s = shape_of(case)
    rows = case["rows"] * case.get("seqs", 1)
    model = pv.Model(s, max_gamma=16 if rows <= 16 else 64)
    pool = pool_of(seed)
    if s.weight_bits == 4:
        c, sc = quantised(pool)
        codes, scales = (c[0::2] | (c[1::2] << 4)).cpu().numpy(), sc.view(torch.uint16).cpu().numpy()
    plain = (pool.to(torch.bfloat16).view(torch.uint16) if s.dtype == "bf16" else pool).cpu().numpy()
    gains = ((1 + pool[:PIECE // 16]).to(torch.bfloat16).view(torch.uint16) if s.dtype == "bf16" else 1 + pool[:PIECE // 16]).cpu().numpy()
    for kind, layer, r0, n, cols, o in pieces(s, seed):
        if is_q4(s, kind):
            model.load_weights_q4(kind, layer, r0, codes[o // 2:(o + n * cols) // 2].reshape(n, -1), scales[o // 32:(o + n * cols) // 32].reshape(n, -1))
        else:
            src = gains if kind.endswith("norm") else plain
            o = o % 32768 if kind.endswith("norm") else o
            model.load_weights(kind, layer, r0, src[o:o + n * cols].reshape(n, cols))
    prompts, blocks, pending, parents, tables, room = inputs_of(case, seed)
    caches = [pv.Cache(model, room) for _ in prompts]
    for c, p, t, first in zip(caches, prompts, tables, pending):
        if case.get("shuffled"):
            c.set_page_table(t)
        if case["do"] != "prefill":
            c.prefill(p)
            c.set_pending(first)
    kv = [c.pool.view(torch.bfloat16 if s.dtype == "bf16" else torch.float32) for c in caches]
    return {"do": case["do"], "caches": caches, "prompt": prompts[0], "blocks": blocks, "pending": pending, "parents": parents, "lens": [len(p) for p in prompts], "kv": kv}


def run(state):
    caches, lens, got = state["caches"], state["lens"], []
    one = caches[0]
    if state["do"] == "prefill":
        one.rollback(0)
        one.prefill(state["prompt"])
        one.set_pending(state["pending"][0])
    for block, parents in zip(state["blocks"], state["parents"]):
        if state["do"] == "batch":
            got.append(pv.verify_batch(caches, block))
        elif state["do"] == "tree":
            got.append(one.verify_tree(lens[0], block[0], parents)[:2])
        else:
            got.append(one.verify(lens[0], block[0]))
    return {"logits": one.debug_logits(), "kv": state["kv"], "steps": np.array(got, dtype=np.int32)}


# ---- what a pass cannot do without ----

def work(case):
    s = shape_of(case)
    _, blocks, _, _, _, _ = inputs_of(case, 0)
    lens = [max(1, case["prefix"] * (case.get("seqs", 1) - i) // case.get("seqs", 1) - 3 * i) for i in range(case.get("seqs", 1))]
    p, rows = params(case), case["rows"] * case.get("seqs", 1)
    elt = 2 if s.dtype == "bf16" else 4
    wbytes = p * (9 / 16 if s.weight_bits == 4 else elt)
    kv = s.n_layers * 2 * s.n_kv_heads * s.head_dim * elt                      # bytes of one token's keys and values
    attn = s.n_layers * 4 * s.n_q_heads * s.head_dim                           # operations of one query with one key
    nbytes = case["steps"] * (wbytes + kv * sum(m + 2 * case["rows"] for m in lens)) + rows * s.vocab * 4
    flops = case["steps"] * (2.0 * p * rows + attn * sum(case["rows"] * (m + case["rows"] / 2) for m in lens))
    if case["do"] == "prefill":
        body = p - math.prod(dims(s, "lm_head"))
        nbytes += wbytes + 2 * kv * case["prefix"]
        flops += 2.0 * body * case["prefix"] + attn * case["prefix"] ** 2 / 2
    return {"bytes": float(nbytes), "flops": float(flops)}


def tolerance(case):
    # fp32: sums in another order.  bf16: activations and the softmax carry 16 mantissa bits or more, but keys and values are
    # rounded to bf16 when they are stored, and one that lies on a rounding boundary comes out a whole bf16 step
    # (1/256 of it) apart; what each layer adds to that travels into the logits.
    if WIDTHS[case["width"]].dtype == "f32":
        return {"rel": 1e-5, "max": 1e-3}
    return {"rel": 4e-3, "max": 0.06}


# ---- the same in 64 bits ----

def weights64(case, seed):
    """{(kind, layer): [pieces]}, each piece a function that gives its rows in 64 bits."""
    s, pool = shape_of(case), pool_of(seed)
    store = (lambda t: t.to(torch.bfloat16).double()) if s.dtype == "bf16" else (lambda t: t.double())
    if s.weight_bits == 4:
        codes, scales = quantised(pool)
    found = {}
    for kind, layer, r0, n, cols, o in pieces(s, seed):
        if is_q4(s, kind):
            get = lambda o=o, n=n, cols=cols: ((codes[o:o + n * cols].double() - 8).view(-1, 32) * scales[o // 32:(o + n * cols) // 32].double()[:, None]).view(n, cols)  # noqa: E731
        elif kind.endswith("norm"):
            get = lambda o=o % 32768, cols=cols: store(1 + pool[o:o + cols])  # noqa: E731
        else:
            get = lambda o=o, n=n, cols=cols: store(pool[o:o + n * cols]).view(n, cols)  # noqa: E731
        found.setdefault((kind, layer), []).append(get)
    return found


def linear(x, get):
    return torch.cat([x @ g().t() for g in get], 1)


def norm(x, gain, eps):
    return x * torch.rsqrt((x * x).mean(1, keepdim=True) + eps) * gain


def rotated(x, pos, base):
    """x [rows, heads, hd]: the pair (i, i + hd / 2) turned by pos * base^(-2 i / hd)."""
    half = x.shape[2] // 2
    ang = pos[:, None].double() * base ** (-2.0 * torch.arange(half, device=x.device, dtype=torch.float64) / x.shape[2])
    c, sn = ang.cos()[:, None], ang.sin()[:, None]
    a, b = x[:, :, :half], x[:, :, half:]
    return torch.cat([a * c - b * sn, b * c + a * sn], 2)


def attention(s, q, k, v, see):
    """q [rows, heads, hd] over k, v [keys, kv heads, hd]; see [rows, keys]: what each row may attend to."""
    out, group = torch.empty_like(q), s.n_q_heads // s.n_kv_heads
    for h in range(s.n_q_heads):
        for r0 in range(0, q.shape[0], 4096):
            sc = (q[r0:r0 + 4096, h] @ k[:, h // group].t()) / math.sqrt(s.head_dim)
            sc.masked_fill_(~see(r0, min(q.shape[0], r0 + 4096)), -math.inf)
            out[r0:r0 + 4096, h] = torch.softmax(sc, 1) @ v[:, h // group]
    return out.reshape(q.shape[0], -1)


def paged(s, ks, vs, table):
    """Keys and values of every layer ([tokens, kv heads, hd] each) as the pages hold them."""
    pt, hd, hk, np_ = s.page_tokens, s.head_dim, s.n_kv_heads, len(table)
    out = torch.zeros(s.n_layers, np_, hk, 2, pt * hd, dtype=torch.float64, device="cuda")
    at = torch.from_numpy(table.astype(np.int64)).cuda()
    for l, (k, v) in enumerate(zip(ks, vs)):
        k, v = (torch.cat([t, t.new_zeros(np_ * pt - t.shape[0], hk, hd)]).view(np_, pt // 16 if s.dtype == "bf16" else 1, -1, hk, hd) for t in (k, v))
        if s.dtype == "bf16":                                # 16 tokens at a time: K as [hd / 32][8-feature group][token][8], V as [hd][token]
            k = k.view(np_, pt // 16, 16, hk, hd // 32, 4, 8).permute(0, 3, 1, 4, 5, 2, 6)
        else:                                                # K as [token][hd], V as [hd][token]
            k = k.permute(0, 3, 1, 2, 4)
        v = v.permute(0, 3, 1, 4, 2)
        out[l, at, :, 0] = k.reshape(np_, hk, -1)
        out[l, at, :, 1] = v.reshape(np_, hk, -1)
    return out.view(-1)


def exact(case, seed):
    s, w = shape_of(case), weights64(case, seed)
    prompts, blocks, pending, parents, tables, _ = inputs_of(case, seed)
    if sum(len(p) for p in prompts) * params(case) * 2 > 3e14:
        return None
    keep = (lambda t: t.to(torch.bfloat16).double()) if s.dtype == "bf16" else (lambda t: t.float().double())
    last, n, hd = blocks[-1], case["rows"], s.head_dim
    par = parents[-1] if case["do"] == "tree" else np.arange(-1, n - 1)
    depth, anc = np.zeros(n, dtype=np.int64), np.eye(n, dtype=bool)
    for i in range(n):
        if par[i] >= 0:
            depth[i] = depth[par[i]] + 1
            anc[i] |= anc[par[i]]
    anc = torch.from_numpy(anc).cuda()
    xs, ks, vs = [], [[] for _ in prompts], [[] for _ in prompts]
    embed = torch.cat([g() for g in w["embed", 0]])
    for p, b in zip(prompts, last):
        xs.append(embed[torch.from_numpy(np.concatenate([p, b]).astype(np.int64)).cuda()])
    del embed
    for l in range(s.n_layers):
        x = torch.cat(xs)
        a = norm(x, w["attn_norm", l][0](), s.rms_eps)
        q, k, v = (linear(a, w[kind, l]).view(len(x), -1, hd) for kind in ("wq", "wk", "wv"))
        att, at = [], 0
        for i, p in enumerate(prompts):
            m = len(p)
            pos = torch.cat([torch.arange(m), m + torch.from_numpy(depth)]).cuda()
            part = slice(at, at + m + n)
            at += m + n
            ki, vi = keep(rotated(k[part], pos, s.rope_base)), keep(v[part])
            ks[i].append(ki)
            vs[i].append(vi)
            keys = torch.arange(m + n, device="cuda")

            def see(r0, r1, m=m, keys=keys):
                ok = keys[None] <= keys[r0:r1, None]
                if r1 > m:
                    lo = max(r0, m)
                    ok[lo - r0:, m:] = anc[lo - m:r1 - m]
                return ok
            att.append(attention(s, rotated(q[part], pos, s.rope_base), ki, vi, see))
        x = x + linear(torch.cat(att), w["wo", l])
        del q, k, v, att
        a = norm(x, w["ffn_norm", l][0](), s.rms_eps)
        g = linear(a, w["wg", l])
        x = x + linear(g * torch.sigmoid(g) * linear(a, w["wu", l]), w["wd", l])
        xs = list(torch.split(x, [len(p) + n for p in prompts]))
    rows = torch.cat([x[-n:] for x in xs])
    logits = linear(norm(rows, w["final_norm", 0][0](), s.rms_eps), w["lm_head", 0])
    return {"logits": logits, "kv": [paged(s, k, v, t) for k, v, t in zip(ks, vs, tables)], "steps": None}
