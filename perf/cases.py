"""Performance cases: what a program built on this library has it do, through the public Python entry points.

A case is a dict of plain values; `kind` says which call or calls one pass makes:

  attn    one verify_attn call (ragged metadata + one attention layer)
  accept  one accept call
  draft   one draft_sample call (one draft step of the batch)
  step    one verification step of a model with `layers` layers: the metadata once, per layer kv_append and
          verify_attn, then accept and commit
  tree    one step over draft TREES: kv_append, verify_attn(parents), accept_tree, kv_compact_path, commit

Raggedness: a case fixes the multiset of context lengths and of draft lengths (evenly spaced quantiles of its
distribution); the seed says which request gets which. So every seed has the same total work.
"""
import math
import random
from statistics import NormalDist

import torch

import paper_2503_05096_amd as pkg

PAGE = 16
_TORCH = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
_SIZE = {"f32": 4, "f16": 2, "bf16": 2}


# --------------------------------------------------------------------------------------------------
# the cases
# --------------------------------------------------------------------------------------------------
def _attn(name, dtype, batch, ctx_lo, ctx_hi, spec_lo, spec_hi, hq, hkv, d, lognormal=False, **kw):
    return dict(name=name, kind=kw.pop("kind", "attn"), dtype=dtype, batch=batch, ctx_lo=ctx_lo, ctx_hi=ctx_hi,
                lognormal=lognormal, spec_lo=spec_lo, spec_hi=spec_hi, hq=hq, hkv=hkv, d=d, **kw)


def _accept(name, dtype, probs, batch, spec_lo, spec_hi, vocab, temp):
    return dict(name=name, kind="accept", logits=dtype, probs=probs, batch=batch, spec_lo=spec_lo, spec_hi=spec_hi,
                vocab=vocab, temp=temp)


def listed():
    return [
        # the smallest call: a unit-sized fp32 batch as in development and in accuracy checks (benchmark config 1)
        _attn("attn-f32-tiny", "f32", 4, 128, 512, 1, 4, 8, 8, 64),
        # one interactive user: nothing in the batch to hide latency behind; four layers stand for the many of a model
        _attn("step-one-request", "bf16", 1, 1500, 1500, 5, 5, 32, 8, 128, kind="step", layers=4, logits="bf16",
              probs="bf16", vocab=128256, temp="0.8"),
        # a 7B multi-head model without GQA in fp16 (benchmark config 2)
        _attn("attn-mha-f16", "f16", 32, 256, 2048, 0, 8, 32, 32, 128),
        # an 8B GQA model at a serving batch with skewed contexts (benchmark config 3, the headline)
        _attn("attn-gqa", "bf16", 128, 128, 4096, 0, 6, 32, 8, 128, lognormal=True),
        # a 70B GQA model on long contexts: many query rows per kv head (benchmark config 4)
        _attn("attn-gqa-long", "bf16", 64, 2048, 8192, 0, 5, 64, 8, 128),
        # a 1B-sized model with 64-wide heads, the usual draft model and a small target in its own right
        _attn("attn-d64", "bf16", 64, 256, 4096, 0, 6, 32, 8, 64),
        # acceptance of the headline batch: sampled requests, bf16 logits as the model leaves them (config 3)
        _accept("accept-sampled", "bf16", "bf16", 128, 0, 6, 128256, "0.8"),
        # acceptance where the program holds logits and draft probabilities in fp32 (processed logits)
        _accept("accept-f32", "f32", "f32", 64, 0, 6, 128256, "1.0"),
        # acceptance over a 256K vocabulary, greedy and sampled requests side by side as in config 5
        _accept("accept-vocab-256k", "bf16", "bf16", 64, 0, 4, 262144, "mixed"),
        # one draft step of the headline batch: probabilities, tokens, confidences
        dict(name="draft-sample", kind="draft", logits="bf16", probs="bf16", rows=128, vocab=128256, temp="0.8"),
        # a step over draft trees of width 3 at a medium batch
        _attn("tree-step", "bf16", 64, 128, 4096, 1, 6, 32, 8, 128, lognormal=True, kind="tree", layers=1, width=3,
              logits="bf16", probs="bf16", vocab=128256, temp="0.8"),
        # a loaded server whose draft lengths have shrunk, mixed temperatures (config 5), four layers of a pass
        _attn("step-mixed", "bf16", 64, 1024, 2048, 0, 1, 32, 8, 128, kind="step", layers=4, logits="bf16",
              probs="bf16", vocab=128256, temp="mixed"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# (query heads, kv heads, head dim): the configurations' head layouts and those between them
_HEADS = ((32, 32, 128), (32, 8, 128), (64, 8, 128), (28, 4, 128), (16, 2, 128), (8, 8, 64), (32, 8, 64), (14, 2, 64))
_MOST_KV_BYTES = 1.3e9        # cached K and V of one pass: below the largest listed case
_MOST_ROW_BYTES = 1.2e8       # logits of one pass


def _draw_attention(rng, dtype, layers=1):
    hq, hkv, d = rng.choice(_HEADS)
    per_token = 2.0 * hkv * d * _SIZE[dtype] * layers
    most = _MOST_KV_BYTES if dtype != "f32" else 3e7
    spec_hi = rng.randint(0, 8)
    spec_lo = rng.randint(0, spec_hi)
    ctx_hi = _log(rng, 24, 8192 if dtype != "f32" else 1024)
    ctx_lo = max(spec_hi + 1, int(ctx_hi * rng.uniform(0.05, 1.0)))
    ctx_hi = max(ctx_hi, ctx_lo)
    batch = _log(rng, 1, max(1, min(256 if dtype != "f32" else 16, int(most / per_token / ctx_hi))))
    return dict(dtype=dtype, batch=batch, ctx_lo=ctx_lo, ctx_hi=ctx_hi, lognormal=rng.random() < 0.3, spec_lo=spec_lo,
                spec_hi=spec_hi, hq=hq, hkv=hkv, d=d)


def _draw_vocab(rng):
    # vocabularies are multiples of 8 in practice; the odd thousands are as common as the round ones
    return rng.choice((1024, 32000, 50272, 128256, 152064, 262144)) if rng.random() < 0.5 else 8 * _log(rng, 125, 32768)


def draw(rng):
    """One more case of the same ranges."""
    kind = rng.choice(("attn", "attn", "attn", "accept", "accept", "draft", "step", "tree"))
    temp = rng.choice(("0.8", "1.0", "0.0", "mixed"))
    logits = rng.choice(("bf16", "bf16", "f16", "f32"))
    if kind == "attn":
        return dict(kind=kind, **_draw_attention(rng, rng.choice(("bf16", "bf16", "f16", "f32"))))
    vocab = _draw_vocab(rng)
    if kind == "accept":
        spec_hi = rng.randint(0, 8)
        spec_lo = rng.randint(0, spec_hi)
        batch = _log(rng, 1, max(1, min(300, int(_MOST_ROW_BYTES / (vocab * _SIZE[logits] * (spec_hi + 1))))))
        probs = logits if rng.random() < 0.8 else rng.choice(("f32", "bf16"))
        return dict(kind=kind, logits=logits, probs=probs, batch=batch, spec_lo=spec_lo, spec_hi=spec_hi, vocab=vocab,
                    temp=temp)
    if kind == "draft":
        rows = _log(rng, 1, max(1, min(300, int(_MOST_ROW_BYTES / (vocab * _SIZE[logits])))))
        return dict(kind=kind, logits=logits, probs=logits if rng.random() < 0.8 else "bf16", rows=rows, vocab=vocab, temp=temp)
    layers = 1 if kind == "tree" else rng.randint(1, 4)
    logits = rng.choice(("bf16", "f16"))
    c = dict(kind=kind, layers=layers, logits=logits, probs=logits, vocab=vocab, temp=temp,
             **_draw_attention(rng, rng.choice(("bf16", "f16")), layers))
    c["batch"] = max(1, min(c["batch"], int(_MOST_ROW_BYTES / (vocab * 2.0 * (c["spec_hi"] + 1)))))
    if kind == "tree":
        c["width"] = rng.randint(1, 4)
    return c


# --------------------------------------------------------------------------------------------------
# ragged lengths
# --------------------------------------------------------------------------------------------------
def _spec_lens(c):
    B, lo, hi = c["batch"], c["spec_lo"], c["spec_hi"]
    return [lo + min(hi - lo, int((hi - lo + 1) * (i + 0.5) / B)) for i in range(B)]


def _ctx_lens(c):
    B, lo, hi = c["batch"], c["ctx_lo"], c["ctx_hi"]
    at = [(i + 0.5) / B for i in range(B)]
    if c["lognormal"]:      # median 1.4 x the middle of the logarithmic range, sigma 0.7, clipped (config 3)
        mid = 1.4 * math.sqrt(lo * hi)
        return [min(hi, max(lo, int(mid * math.exp(0.7 * NormalDist().inv_cdf(u))))) for u in at]
    return [lo + int((hi - lo) * u) for u in at]


# --------------------------------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------------------------------
class _State:
    pass


def _randn(shape, gen, dtype, sigma=1.0):
    # drawn in the storage type: normal values of the model's activations, keys and values
    x = torch.empty(shape, dtype=_TORCH[dtype], device="cuda")
    x.normal_(0.0, sigma, generator=gen)
    return x


def _ints(v):
    return torch.tensor(v, dtype=torch.int32, device="cuda")


def _attention_inputs(s, c, r, gen):
    ctx = _ctx_lens(c)
    r.shuffle(ctx)
    s.ctx_list = ctx
    pages = [-(-L // PAGE) for L in ctx]
    need = sum(pages)
    num_pages = max(1, math.ceil(1.25 * need))       # a pool with room, handed out in random order
    ids = list(range(num_pages))
    r.shuffle(ids)
    table, at = [], 0
    for p in pages:
        table.append(ids[at:at + p] + [-1] * (max(pages) - p))
        at += p
    s.block_table, s.ctx_lens = _ints(table), _ints(ctx)
    layers = c.get("layers", 1)
    kv = (layers, num_pages, c["hkv"], PAGE, c["d"])
    s.k_pages, s.v_pages = _randn(kv, gen, c["dtype"]), _randn(kv, gen, c["dtype"])
    s.q = _randn((layers, s.TQ, c["hq"], c["d"]), gen, c["dtype"])
    if c["kind"] != "attn":
        s.k_new = _randn((layers, s.TQ, c["hkv"], c["d"]), gen, c["dtype"])
        s.v_new = _randn((layers, s.TQ, c["hkv"], c["d"]), gen, c["dtype"])


def _temperatures(c, B, r):
    if c["temp"] != "mixed":
        return [float(c["temp"])] * B
    t = [(0.0, 0.7, 1.0)[i % 3] for i in range(B)]
    r.shuffle(t)
    return t


def _acceptance_inputs(s, c, r, gen):
    """Logits of a target, a draft distribution that follows it with noise, tokens drawn from that distribution."""
    B, V = c["batch"], c["vocab"]
    temps = _temperatures(c, B, r)
    s.temperature = torch.tensor(temps, dtype=torch.float32, device="cuda")
    s.uniforms = torch.rand((s.TQ, 2), generator=gen, device="cuda")
    s.target_logits = _randn((s.TQ, V), gen, c["logits"], 3.0)
    s.draft_probs = torch.empty((s.TD, V), dtype=_TORCH[c["probs"]], device="cuda")
    tokens = torch.zeros((s.TD,), dtype=torch.int32, device="cuda")
    for i in range(B):
        k, d0, r0 = s.spec_list[i], s.cu[i] - i, s.cu[i]
        if k == 0:
            continue
        noisy = s.target_logits[r0:r0 + k].float() + _randn((k, V), gen, "f32", 1.5)
        q = torch.softmax(noisy / 1.2, dim=1).to(s.draft_probs.dtype)
        s.draft_probs[d0:d0 + k] = q
        # the token of draft j comes from the row of its parent (a chain: the row before it, which is row j)
        rows = q.float()
        if c["kind"] == "tree":
            rows = rows[_longs([p for p in s.parent_lists[i][1:]])]
        if temps[i] > 0.0:
            rows = rows / torch.empty_like(rows).exponential_(generator=gen).clamp_(min=1e-20)
        tokens[d0:d0 + k] = rows.argmax(dim=1).to(torch.int32)
    s.draft_tokens = tokens


def _longs(v):
    return torch.tensor(v, dtype=torch.int64, device="cuda")


def _trees(s, c, r):
    """parent of every node: among the earlier nodes with room, half of the time the most recent one."""
    s.parent_lists = []
    for k in s.spec_list:
        par, n_child = [-1], [0] * (k + 1)
        for j in range(1, k + 1):
            room = [u for u in range(j) if n_child[u] < c["width"]]
            p = room[-1] if r.random() < 0.5 else r.choice(room)
            n_child[p] += 1
            par.append(p)
        s.parent_lists.append(par)
    s.parents = _ints([p for par in s.parent_lists for p in par])


def prepare(case, seed):
    c, s = case, _State()
    r = random.Random("inputs %d" % seed)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    s.case = c
    if c["kind"] == "draft":
        s.draft_logits = _randn((c["rows"], c["vocab"]), gen, c["logits"], 3.0)
        s.temperature = torch.tensor(_temperatures(c, c["rows"], r), dtype=torch.float32, device="cuda")
        s.uniforms = torch.rand((c["rows"],), generator=gen, device="cuda")
        return s
    spec = _spec_lens(c)
    r.shuffle(spec)
    s.spec_list, s.spec_lens = spec, _ints(spec)
    s.TD = sum(spec)
    s.TQ = s.TD + len(spec)
    s.cu = [0]
    for k in spec:
        s.cu.append(s.cu[-1] + k + 1)
    if c["kind"] == "tree":
        _trees(s, c, r)
    if c["kind"] != "accept":
        _attention_inputs(s, c, r, gen)
    if c["kind"] != "attn":
        _acceptance_inputs(s, c, r, gen)
    if c["kind"] == "step":
        # a pass of several layers keeps its metadata in a workspace of its own
        dims = pkg.attn_dims(s.q[0], s.k_pages[0], s.block_table, max_spec_len=c["spec_hi"])
        nbytes = pkg.lib().adaspec_verify_attn_workspace_bytes(dims)
        s.workspace = torch.empty(max(nbytes, 256), dtype=torch.uint8, device="cuda")
    return s


# --------------------------------------------------------------------------------------------------
# one pass
# --------------------------------------------------------------------------------------------------
def run(s):
    c = s.case
    kind = c["kind"]
    if kind == "draft":
        probs, tokens, conf = pkg.draft_sample(s.draft_logits, s.temperature, s.uniforms, probs_dtype=_TORCH[c["probs"]])
        return {"probs": probs, "tokens": tokens, "confidence": conf}
    most = c["spec_hi"]
    if kind == "attn":
        return {"out": pkg.verify_attn(s.q[0], s.k_pages[0], s.v_pages[0], s.block_table, s.ctx_lens, s.spec_lens,
                                       max_spec_len=most)}
    if kind == "accept":
        tokens, lens = pkg.accept(s.target_logits, s.draft_probs, s.draft_tokens, s.uniforms, s.spec_lens, s.temperature,
                                  max_spec_len=most)
        return {"tokens": tokens, "lens": lens}
    if kind == "tree":
        k, v = s.k_pages[0], s.v_pages[0]
        pkg.kv_append(s.k_new[0], s.v_new[0], k, v, s.block_table, s.ctx_lens, s.spec_lens, max_spec_len=most)
        out = pkg.verify_attn(s.q[0], k, v, s.block_table, s.ctx_lens, s.spec_lens, max_spec_len=most, parents=s.parents)
        tokens, lens, path = pkg.accept_tree(s.target_logits, s.draft_probs, s.draft_tokens, s.parents, s.uniforms,
                                             s.spec_lens, s.temperature, max_spec_len=most)
        pkg.kv_compact_path(k, v, s.block_table, s.ctx_lens, s.spec_lens, path, lens, max_spec_len=most)
        kept, _, last = pkg.commit(tokens, lens, s.spec_lens, s.ctx_lens, max_spec_len=most)
        return {"out": out, "tokens": tokens, "lens": lens, "path": path, "kept": kept, "last": last,
                "k_pages": s.k_pages, "v_pages": s.v_pages}
    pkg.verify_attn(s.q[0], s.k_pages[0], s.v_pages[0], s.block_table, s.ctx_lens, s.spec_lens, max_spec_len=most,
                    plan="build", workspace=s.workspace)
    outs = []
    for n in range(c["layers"]):
        k, v = s.k_pages[n], s.v_pages[n]
        pkg.kv_append(s.k_new[n], s.v_new[n], k, v, s.block_table, s.ctx_lens, s.spec_lens, max_spec_len=most)
        outs.append(pkg.verify_attn(s.q[n], k, v, s.block_table, s.ctx_lens, s.spec_lens, max_spec_len=most,
                                    plan="reuse", workspace=s.workspace))
    tokens, lens = pkg.accept(s.target_logits, s.draft_probs, s.draft_tokens, s.uniforms, s.spec_lens, s.temperature,
                              max_spec_len=most)
    kept, _, last = pkg.commit(tokens, lens, s.spec_lens, s.ctx_lens, max_spec_len=most)
    return {"out": outs, "tokens": tokens, "lens": lens, "kept": kept, "last": last,
            "k_pages": s.k_pages, "v_pages": s.v_pages}


# --------------------------------------------------------------------------------------------------
# what a pass cannot do without
# --------------------------------------------------------------------------------------------------
def work(case):
    c = case
    if c["kind"] == "draft":
        n = c["rows"] * c["vocab"]
        return {"bytes": n * (_SIZE[c["logits"]] + _SIZE[c["probs"]]), "flops": 5.0 * n}
    spec = _spec_lens(c)
    B, TD = len(spec), sum(spec)
    TQ = TD + B
    nbytes = flops = 0.0
    if c["kind"] != "accept":
        ctx, size, layers = sum(_ctx_lens(c)), _SIZE[c["dtype"]], c.get("layers", 1)
        nbytes += layers * (2.0 * ctx * c["hkv"] * c["d"] * size + 2.0 * TQ * c["hq"] * c["d"] * size + 4.0 * ctx / PAGE)
        # two products over the cached tokens, for every query row; context and draft length are dealt independently
        flops += layers * 4.0 * ctx * (TQ / B) * c["hq"] * c["d"]
        if c["kind"] != "attn":
            nbytes += layers * 4.0 * TQ * c["hkv"] * c["d"] * size          # the new K/V rows, in and out
    if c["kind"] != "attn":
        # every draft row's logits for its test; per request one more row to draw the last token from
        # (the draft probabilities of the rejected row, or the logits after the last draft)
        nbytes += c["vocab"] * (TD * _SIZE[c["logits"]] + B * min(_SIZE[c["logits"]], _SIZE[c["probs"]]))
        flops += 5.0 * c["vocab"] * TQ
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # About four times what the calls are off from exact(): 1.7e-3 in bf16 and 2.9e-4 in f16 (one rounding to the storage
    # type, softmax weights in f16 as well), 4e-7 to 1e-6 in f32. Tokens and lengths agreed in all cases tried; where a
    # uniform falls on the border of two tokens' intervals, sums in another order can give the neighbour.
    kind = case["kind"]
    store = case["probs"] if kind == "draft" else case["dtype"] if kind != "accept" else None
    rel = {"f32": 4e-6, "f16": 1.2e-3, "bf16": 7e-3, None: 0.0}[store]
    return {"rel": rel, "differ": 0.01}


# --------------------------------------------------------------------------------------------------
# the same in 64 bits
# --------------------------------------------------------------------------------------------------
def _exact_attention(s, c, layer):
    """Request by request over the gathered cache; a step's new rows are put at the cache's end first."""
    Hkv, G, d = c["hkv"], c["hq"] // c["hkv"], c["d"]
    out = torch.empty((s.TQ, c["hq"], d), dtype=torch.float64, device="cuda")
    for i, L in enumerate(s.ctx_list):
        n, r0 = s.spec_list[i] + 1, s.cu[i]
        ids = s.block_table[i, :-(-L // PAGE)].long()
        k, v = (p[layer][ids].permute(1, 0, 2, 3).reshape(Hkv, -1, d)[:, :L].double() for p in (s.k_pages, s.v_pages))
        if c["kind"] != "attn":
            k[:, L - n:] = s.k_new[layer, r0:r0 + n].double().transpose(0, 1)
            v[:, L - n:] = s.v_new[layer, r0:r0 + n].double().transpose(0, 1)
        q = s.q[layer, r0:r0 + n].double().reshape(n, Hkv, G, d).permute(1, 0, 2, 3).reshape(Hkv, n * G, d).contiguous()
        seen = torch.ones((n, L), dtype=torch.bool)
        for j in range(n):
            seen[j, L - n + j + 1:] = False
            if c["kind"] == "tree":
                seen[j, L - n:] = False
                u = j
                while u >= 0:
                    seen[j, L - n + u] = True
                    u = s.parent_lists[i][u]
        score = torch.bmm(q, k.transpose(1, 2).contiguous()).reshape(Hkv, n, G, L) / math.sqrt(d)
        score = score.masked_fill(~seen.cuda()[None, :, None, :], -math.inf)
        p = torch.softmax(score, dim=3).reshape(Hkv, n * G, L)
        out[r0:r0 + n] = torch.bmm(p, v.contiguous()).reshape(Hkv, n, G, d).permute(1, 0, 2, 3).reshape(n, c["hq"], d)
    return out


def _exact_draw(mass, u):
    total = torch.cumsum(mass, 0)
    t = int(torch.searchsorted(total, u * total[-1], right=True))
    return min(t, int(mass.nonzero()[-1]))


def _exact_acceptance(s, c):
    B = c["batch"]
    tokens = torch.full((B, c["spec_hi"] + 1), -1, dtype=torch.int32)
    lens = torch.zeros((B,), dtype=torch.int32)
    drafts, uni, temps = s.draft_tokens.tolist(), s.uniforms.double().tolist(), s.temperature.tolist()
    for i in range(B):
        k, r0 = s.spec_list[i], s.cu[i]
        z = s.target_logits[r0:r0 + k + 1].double()
        q = s.draft_probs[r0 - i:r0 - i + k].double()
        T = temps[i]
        best = z.argmax(dim=1).tolist()
        p = torch.softmax(z / T, dim=1) if T > 0.0 else None
        a, last = 0, None
        while a < k:
            x, u0 = drafts[r0 - i + a], uni[r0 + a][0]
            if T == 0.0:
                fine = x == best[a]
            else:
                px, qx = float(p[a, x]), float(q[a, x])
                fine = qx == 0.0 or u0 < px / qx
            if not fine:
                break
            tokens[i, a] = x
            a += 1
        if T == 0.0:
            last = best[a]
        else:
            mass = p[a]
            if a < k:
                res = (p[a] - q[a]).clamp_(min=0.0)
                mass = res if float(res.sum()) > 0.0 else mass
            last = _exact_draw(mass, uni[r0 + a][1])
        tokens[i, a], lens[i] = last, a
    return tokens.cuda(), lens.cuda()


def exact(case, seed):
    c, s = case, prepare(case, seed)
    kind = c["kind"]
    if kind == "draft":
        t = s.temperature.double()[:, None]
        probs = torch.softmax(s.draft_logits.double() / torch.where(t > 0.0, t, torch.ones_like(t)), dim=1)
        return {"probs": probs, "tokens": None, "confidence": None}     # both follow from the stored, rounded row
    if kind == "attn":
        return {"out": _exact_attention(s, c, 0)}
    if kind == "accept":
        tokens, lens = _exact_acceptance(s, c)
        return {"tokens": tokens, "lens": lens}
    none = {"kept": None, "last": None, "k_pages": None, "v_pages": None}
    if kind == "tree":
        return {"out": _exact_attention(s, c, 0), "tokens": None, "lens": None, "path": None, **none}
    tokens, lens = _exact_acceptance(s, c)
    return {"out": [_exact_attention(s, c, n) for n in range(c["layers"])], "tokens": tokens, "lens": lens, **none}
