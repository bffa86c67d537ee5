"""The work whose speed is measured: calls of this package as a serving engine makes
them, over the range of shapes, types and options that it makes them with.

Kinds of case
  prefill     pic_kv_write of the fresh rows, then pic_attn_prefill of every query span.
              A request holds cached documents (shared between requests where the pool
              has fewer than they ask for), fresh documents computed in the call, and a
              query tail that sees all of them.  With "prerotated" the conventional path
              instead: q and the fresh keys rotated in place by pic_rope_rotate, the
              rotated keys stored, attention without rotation.
  decode      pic_kv_write of one new row per request, then pic_attn_decode (or its
              no-allocation form) of one query per request.
  offload     pic_blocks_gather of cache blocks into pinned host memory (or a device
              buffer) and pic_blocks_scatter of them under new block ids.
  span_cache  host only: block hashes of a prompt, lookup, the span list from the hits,
              insertion of the missed blocks, and their eviction.
"""
import math
import random

import numpy as np
import torch

from paper_2606_13126_amd import _binding as B

SSEP, PDEP, QUERY = B.PIC_SSEP, B.PIC_PDEP, B.PIC_QUERY
BLOCK = 16
DTYPES = {"bf16": (torch.bfloat16, B.PIC_BF16), "f32": (torch.float32, B.PIC_F32)}


def prefill(reqs=1, docs=0, pool=0, doc_len=512, fresh=0, fresh_len=512, tail=128, hq=32, hkv=8, d=128, dtype="bf16",
            style="neox", table=True, rotary=0, ragged=False, mixed=False, prerotated=False, theta=5e5, layout=1):
    return dict(kind="prefill", reqs=reqs, docs=docs, pool=pool, doc_len=doc_len, fresh=fresh, fresh_len=fresh_len,
                tail=tail, hq=hq, hkv=hkv, d=d, dtype=dtype, style=style, table=table, rotary=rotary, ragged=ragged,
                mixed=mixed, prerotated=prerotated, theta=theta, layout=layout)


def decode(reqs=1, ctx=1024, shared=0, ragged=False, hq=32, hkv=8, d=128, dtype="bf16", style="neox", table=True,
           rotary=0, noalloc=False, theta=5e5, layout=1):
    return dict(kind="decode", reqs=reqs, ctx=ctx, shared=shared, ragged=ragged, hq=hq, hkv=hkv, d=d, dtype=dtype,
                style=style, table=table, rotary=rotary, noalloc=noalloc, theta=theta, layout=layout)


def offload(blocks=1024, hkv=8, d=128, dtype="bf16", to="host"):
    return dict(kind="offload", blocks=blocks, hkv=hkv, d=d, dtype=dtype, to=to)


def span_cache(tokens=8192, doc_len=512, cached=0.75, layout=1):
    return dict(kind="span_cache", tokens=tokens, doc_len=doc_len, cached=cached, layout=layout)


def listed():
    cases = {
        # one long prompt of a 70B-shaped model: half of its documents are in the cache,
        # half are computed in the call, then the question over all 33K tokens (bench.py's
        # headline step, and the largest call)
        "prefill_long": prefill(docs=32, pool=32, fresh=32, mixed=True, tail=512, hq=64),
        # retrieval-augmented question of an 8B-shaped model: ten cached documents, only
        # the question is computed
        "prefill_rag": prefill(docs=10, pool=10, tail=256),
        # sixteen such users at once over a common set of documents
        "prefill_reuse": prefill(reqs=16, docs=8, pool=32, tail=128),
        # a short prompt of a small model, spans of odd lengths, cos/sin not tabulated,
        # interleaved pairing: the latency of one small call
        "prefill_short": prefill(fresh=3, fresh_len=201, tail=11, hq=8, hkv=2, d=64, style="gptj", table=False,
                                 ragged=True, theta=1e4),
        # full precision, as a model is validated with
        "prefill_f32": prefill(docs=3, pool=3, doc_len=256, fresh=2, fresh_len=333, tail=77, hq=8, hkv=2, dtype="f32",
                               ragged=True, theta=1e4),
        # the conventional path (keys rotated when they are stored), four new documents
        # and a question
        "prefill_prerotated": prefill(fresh=4, tail=128, prerotated=True),
        # a decode step of 64 users with contexts of their own: nothing shared, HBM-bound
        "decode_own": decode(reqs=64, ctx=8193),
        # the same with the contexts built from 16 common documents in 64 orders
        "decode_shared": decode(reqs=64, ctx=8193, shared=16),
        # one user: the latency of a decode step, from a loop that allocates nothing
        "decode_single": decode(reqs=1, ctx=1537, noalloc=True),
        # many users with contexts of very different lengths, a model with few KV heads
        "decode_ragged": decode(reqs=200, ctx=4000, ragged=True, hq=28, hkv=4),
        # idle documents leave for host memory and come back under other block ids
        "offload_host": offload(blocks=1024),
        # the prompt of a RAG call: three quarters of its documents are known
        "span_cache": span_cache(),
    }
    return [dict(c, name=n) for n, c in cases.items()]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """Another case of the listed ones' ranges."""
    kind = rng.choice(["prefill", "prefill", "prefill", "prefill", "decode", "decode", "decode", "offload", "span_cache"])
    layout = rng.randrange(1, 1 << 20)
    style, table = rng.choice(["neox", "neox", "gptj"]), rng.random() < 0.75
    if kind in ("prefill", "decode"):
        f32 = rng.random() < 0.15
        hq, hkv, d = rng.choice([(32, 8, 128), (64, 8, 128), (32, 8, 64), (28, 4, 128), (8, 2, 64), (12, 12, 64)])
        theta = rng.choice([1e4, 5e5])
        rotary = d // 2 if rng.random() < 0.1 else 0
        common = dict(d=d, style=style, table=table, rotary=rotary, theta=theta, layout=layout)
        if f32:
            common["dtype"] = "f32"
            hq, hkv = 8, rng.choice([2, 8])
    if kind == "prefill":
        reqs = 1 if f32 else _logint(rng, 1, 24)
        doc_len = 16 * _logint(rng, 4, 32)
        most = 1200 if f32 else max(doc_len, 32768 // reqs)
        docs = min(rng.randrange(0, 24), most // doc_len)
        fresh_len = _logint(rng, 17, 700)
        fresh = 0 if docs and rng.random() < 0.4 else min(rng.randrange(1, 12), max(1, (600 if f32 else 16384 // reqs) // fresh_len))
        fresh_len = min(fresh_len, 600) if f32 else fresh_len
        tail = _logint(rng, 5, 90 if f32 else 512)
        return prefill(reqs=reqs, docs=docs, pool=max(docs, rng.randrange(docs, 2 * docs + 1)), doc_len=doc_len, fresh=fresh,
                       fresh_len=fresh_len, tail=tail, hq=hq, hkv=hkv, ragged=rng.random() < 0.7,
                       prerotated=rng.random() < 0.15, **common)
    if kind == "decode":
        reqs = _logint(rng, 1, 16 if f32 else 256)
        ctx = _logint(rng, 33, min(32768, (16384 if f32 else 524288) // reqs))
        return decode(reqs=reqs, ctx=ctx, shared=rng.choice([0, 0, max(1, ctx // 512)]), ragged=rng.random() < 0.6, hq=hq,
                      hkv=hkv, noalloc=reqs <= 8 and rng.random() < 0.5, **common)
    if kind == "offload":
        hkv, d, dtype = rng.choice([2, 8]), rng.choice([64, 128]), rng.choice(["bf16", "bf16", "f32"])
        most = 1024 * 8 * 128 // (hkv * d * (2 if dtype == "f32" else 1))
        return offload(blocks=_logint(rng, 9, most), hkv=hkv, d=d, dtype=dtype, to=rng.choice(["host", "device"]))
    return span_cache(tokens=_logint(rng, 200, 32768), doc_len=16 * _logint(rng, 4, 64), cached=rng.random(), layout=layout)


# ------------------------------------------------------------------------------------
# layout: spans, lengths and which document a request holds (from the case alone)
# ------------------------------------------------------------------------------------

def requests_of(case):
    """Per request its spans as (length, flags, shared document or None, fresh)."""
    rng = random.Random(case["layout"])
    out = []
    if case["kind"] == "decode":
        for _ in range(case["reqs"]):
            n = case["ctx"] - 1
            if case["ragged"]:
                n = max(1, min(n, _logint(rng, max(2, case["ctx"] // 24), case["ctx"])))
            spans = []
            if case["shared"]:
                each = max(BLOCK, n // case["shared"] // BLOCK * BLOCK)
                full = case["ctx"] // case["shared"] // BLOCK * BLOCK or BLOCK
                order = rng.sample(range(case["shared"]), case["shared"])
                for i in order:
                    if sum(s[0] for s in spans) + each <= n:
                        spans.append((each, SSEP, (i, full), False))
            rest = n - sum(s[0] for s in spans)
            if rest:
                spans.append((rest, SSEP, None, False))
            out.append(spans + [(1, PDEP, None, True)])
        return out
    for _ in range(case["reqs"]):
        spans = [(case["doc_len"], SSEP, (i, case["doc_len"]), False) for i in rng.sample(range(case["pool"]), case["docs"])]
        new = []
        for _ in range(case["fresh"]):
            n = case["fresh_len"] - (rng.randrange(0, max(1, case["fresh_len"] // 2)) if case["ragged"] else 0)
            new.append((n, SSEP | QUERY, None, True))
        if case["mixed"]:
            spans = spans + new
            rng.shuffle(spans)
        else:
            spans = spans + new
        tail = case["tail"] - (rng.randrange(0, max(1, case["tail"] // 4)) if case["ragged"] else 0)
        out.append(spans + [(tail, PDEP | QUERY, None, True)])
    return out


def describe(case):
    """Host arrays of the batch: span descriptor, window of every query span, and which
    blocks are whose (block ids count from 0 in order of first use)."""
    reqs = requests_of(case)
    seq, cu, start, flags, tables, queries = [], [0], [], [], [], []
    docs, used = {}, 0
    for r, spans in enumerate(reqs):
        n, blocks = 0, []
        for length, fl, doc, fresh in spans:
            start.append(n)
            flags.append(fl)
            if doc is not None:
                i, whole = doc
                if i not in docs:
                    docs[i] = list(range(used, used + whole // BLOCK))
                    used += whole // BLOCK
                blocks += docs[i][: length // BLOCK]
            else:
                need = -(-(n + length) // BLOCK) - len(blocks)
                blocks += range(used, used + need)
                used += need
            if fl & QUERY:
                queries.append((r, n, n + length, n if fl & SSEP else 0))
            n += length
        if case["kind"] == "decode":
            queries.append((r, n - 1, n, 0))
        seq.append(n)
        cu.append(len(start))
        tables.append(blocks)
    width = max(len(b) for b in tables)
    bt = np.zeros((len(reqs), width), np.int32)
    for r, b in enumerate(tables):
        bt[r, : len(b)] = b
    fresh = [(r, a, a + s[0]) for r, spans in enumerate(reqs)
             for a, s in zip(np.cumsum([0] + [s[0] for s in spans]).tolist(), spans) if s[3]]
    return dict(seq=np.array(seq, np.int32), cu=np.array(cu, np.int32), start=np.array(start, np.int32),
                flags=np.array(flags, np.int32), tables=bt, blocks=used, queries=queries, fresh=fresh)


# ------------------------------------------------------------------------------------
# inputs (from the seed alone), without any of the package's arithmetic
# ------------------------------------------------------------------------------------

def inputs(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    rng = np.random.default_rng(seed)

    def normal(shape, dtype):
        return torch.randn(shape, generator=gen, device="cuda", dtype=dtype)

    if case["kind"] == "offload":
        dt = DTYPES[case["dtype"]][0]
        n = case["blocks"]
        page = (case["hkv"], BLOCK, case["d"])
        ids = torch.from_numpy(rng.permutation(2 * n + 64)[: 2 * n].astype(np.int32)).cuda()
        return dict(k_pool=normal((2 * n + 64,) + page, dt), v_pool=normal((2 * n + 64,) + page, dt), old=ids[:n].contiguous(),
                    new=ids[n:].contiguous())
    if case["kind"] == "span_cache":
        tokens = rng.integers(5, 128000, case["tokens"], dtype=np.int32)
        tokens[:: case["doc_len"]] = 1            # a separator starts every document
        tail = (case["tokens"] - 1) // BLOCK * BLOCK   # the question depends on all of them
        tokens[tail] = 2
        known = np.random.default_rng(case["layout"]).random(-(-case["tokens"] // case["doc_len"])) < case["cached"]
        return dict(tokens=tokens, seed=rng.bytes(32), known=known)

    dt = DTYPES[case["dtype"]][0]
    x = describe(case)
    hq, hkv, d = case["hq"], case["hkv"], case["d"]
    nb = x["blocks"] + 8
    tables = rng.permutation(nb).astype(np.int32)[x["tables"]]
    tok = np.concatenate([np.arange(a, b, dtype=np.int64) for _, a, b in x["fresh"]])
    req = np.concatenate([np.full(b - a, r, np.int64) for r, a, b in x["fresh"]])
    slots = (tables[req, tok // BLOCK].astype(np.int64) * BLOCK + tok % BLOCK).astype(np.int32)
    rows = sum(b - a for _, a, b, _ in x["queries"])
    positions = np.concatenate([np.arange(n, dtype=np.int32) for n in x["seq"]])
    key_pos = np.concatenate([np.arange(a, b, dtype=np.int32) for _, a, b in x["fresh"]])
    q_pos = np.concatenate([np.arange(a, b, dtype=np.int32) for _, a, b, _ in x["queries"]])
    x.update(q=normal((rows, hq, d), dt), k_pool=normal((nb, hkv, BLOCK, d), dt), v_pool=normal((nb, hkv, BLOCK, d), dt),
             k_new=normal((len(tok), hkv, d), dt), v_new=normal((len(tok), hkv, d), dt),
             slots=torch.from_numpy(slots).cuda(), bt=torch.from_numpy(tables).cuda(),
             positions=torch.from_numpy(positions).cuda(), key_pos=torch.from_numpy(key_pos).cuda(),
             q_pos=torch.from_numpy(q_pos).cuda())
    return x


def prepare(case, seed):
    x = inputs(case, seed)
    if case["kind"] == "offload":
        cfg = B.make_config(case["hkv"], case["hkv"], case["d"], dtype=DTYPES[case["dtype"]][1])
        shape = (case["blocks"],) + tuple(x["k_pool"].shape[1:])
        where = dict(device="cuda") if case["to"] == "device" else dict(pin_memory=True)
        x.update(kind="offload", cfg=cfg, k_buf=torch.empty(shape, dtype=x["k_pool"].dtype, **where),
                 v_buf=torch.empty(shape, dtype=x["k_pool"].dtype, **where))
        return x
    if case["kind"] == "span_cache":
        x["kind"] = "span_cache"
        x["cache"] = Cache()
        hashes = B.pic_block_hashes(x["tokens"], 1, 2, x["seed"])
        doc = np.arange(len(hashes)) * BLOCK // case["doc_len"]
        ids = np.where(x["known"][doc] & (x["tokens"][: len(hashes) * BLOCK : BLOCK] != 2), np.arange(len(hashes)), -1)
        B.pic_block_cache_insert(x["cache"].handle, hashes, ids.astype(np.int32))
        return x
    cfg = B.make_config(case["hq"], case["hkv"], case["d"], dtype=DTYPES[case["dtype"]][1], rope_theta=case["theta"],
                        rope_style=B.PIC_ROPE_NEOX if case["style"] == "neox" else B.PIC_ROPE_GPTJ,
                        k_prerotated=int(case.get("prerotated", False)), rotary_dim=case["rotary"])
    host = B.HostBatch(x["seq"], x["cu"], x["start"], x["flags"])
    is_decode = case["kind"] == "decode"
    size = B.pic_workspace_size(cfg, host, is_decode)
    table = None
    if case["table"]:
        n, half = int(x["seq"].max()), case["d"] // 2
        table = torch.empty((n, half, 2) if case["dtype"] == "f32" else (n, half), dtype=torch.float32, device="cuda")
        B.pic_rope_table_build(cfg, table)
    x.update(kind=case["kind"], cfg=cfg, host=host, table=table, o=torch.empty_like(x["q"]),
             workspace=torch.empty(max(size, 1), dtype=torch.uint8, device="cuda"),
             prerotated=case.get("prerotated", False), noalloc=case.get("noalloc", False))
    return x


class Cache:
    """A span cache handle that goes with its owner."""

    def __init__(self):
        self.handle = B.pic_block_cache_create()

    def __del__(self):
        B.pic_block_cache_destroy(self.handle)


# ------------------------------------------------------------------------------------
# one pass
# ------------------------------------------------------------------------------------

def run(s):
    if s["kind"] == "offload":
        B.pic_blocks_gather(s["cfg"], s["k_pool"], s["v_pool"], s["old"], s["k_buf"], s["v_buf"])
        B.pic_blocks_scatter(s["cfg"], s["k_pool"], s["v_pool"], s["new"], s["k_buf"], s["v_buf"])
        return {k: s[k] for k in ("k_buf", "v_buf", "k_pool", "v_pool")}
    if s["kind"] == "span_cache":
        c = s["cache"].handle
        hashes = B.pic_block_hashes(s["tokens"], 1, 2, s["seed"])
        ids, hits = B.pic_block_cache_lookup(c, hashes)
        start, flags = B.pic_spans_from_blocks(s["tokens"], 1, 2, ids >= 0)
        missed = hashes[ids < 0]
        B.pic_block_cache_insert(c, missed, np.arange(len(missed), dtype=np.int32))
        size = B.pic_block_cache_size(c)
        B.pic_block_cache_erase(c, missed)
        return {"hashes": hashes, "ids": ids, "hits": hits, "start": start, "flags": flags, "size": size}
    if s["prerotated"]:
        B.pic_rope_rotate(s["cfg"], s["k_new"], s["key_pos"], table=s["table"])
        B.pic_rope_rotate(s["cfg"], s["q"], s["q_pos"], table=s["table"])
    B.pic_kv_write(s["cfg"], s["k_pool"], s["v_pool"], s["k_new"], s["v_new"], s["slots"])
    if s["kind"] == "decode" and s["noalloc"]:
        B.pic_attn_decode_noalloc(s["cfg"], s["host"], s["bt"], s["positions"], s["q"], s["o"], s["k_pool"], s["v_pool"],
                                  table=s["table"])
    else:
        attend = B.pic_attn_decode if s["kind"] == "decode" else B.pic_attn_prefill
        attend(s["cfg"], s["host"], s["bt"], s["positions"], s["q"], s["o"], s["k_pool"], s["v_pool"],
               workspace=s["workspace"], table=s["table"])
    out = {"o": s["o"], "k_pool": s["k_pool"], "v_pool": s["v_pool"]}
    if s["prerotated"]:
        out["q"] = s["q"]
    return out


# ------------------------------------------------------------------------------------
# what a pass cannot do without, and what it computes
# ------------------------------------------------------------------------------------

def work(case):
    if case["kind"] == "offload":
        e = 4 if case["dtype"] == "f32" else 2
        # two copies (out and back) of K and V, each read once and written once
        return {"bytes": 8.0 * case["blocks"] * case["hkv"] * BLOCK * case["d"] * e, "flops": 0}
    if case["kind"] == "span_cache":
        # the tokens once, and 32 bytes per block's hash (the last block's covers all tokens)
        return {"bytes": 4.0 * case["tokens"] * 2 + 32.0 * (case["tokens"] // BLOCK), "flops": 0}
    x = describe(case)
    e = 4 if case["dtype"] == "f32" else 2
    pairs = sum(sum(range(a - w + 1, b - w + 1)) for _, a, b, w in x["queries"])
    rows = sum(b - a for _, a, b, _ in x["queries"])
    new = sum(b - a for _, a, b in x["fresh"])
    seen = set()
    for r, a, b, w in x["queries"]:
        seen.update(x["tables"][r, w // BLOCK : -(-b // BLOCK)].tolist())
    row = case["d"] * e
    # q and o; the distinct cache blocks that some query sees; the new rows in and out
    total = 2.0 * rows * case["hq"] * row + 2.0 * len(seen) * BLOCK * case["hkv"] * row + 4.0 * new * case["hkv"] * row
    if case.get("prerotated"):
        total += 2.0 * (rows * case["hq"] + new * case["hkv"]) * row   # rotated in place: read and written
    return {"bytes": total, "flops": 4.0 * case["d"] * case["hq"] * pairs}


def tolerance(case):
    if case["kind"] in ("offload", "span_cache"):
        return "exact"   # copies and hashes
    if case["dtype"] == "f32":
        return {"rel": 2e-6, "max": 1e-4}
    # bf16 rotated keys, probabilities and outputs, 32-bit sums
    return {"rel": 1e-2, "max": 0.2}


def rotate(t, pos, case):
    """The rotary embedding of rows t [n][heads][d] at positions pos, in 64 bits."""
    r = case["rotary"] or case["d"]
    t = t.double()
    freq = case["theta"] ** (-torch.arange(0, r, 2, device=t.device, dtype=torch.float64) / r)
    ang = (pos.double()[:, None] * freq)[:, None, :]
    c, s = ang.cos(), ang.sin()
    out = t.clone()
    a, b = (t[..., : r // 2], t[..., r // 2 : r]) if case["style"] == "neox" else (t[..., 0:r:2], t[..., 1:r:2])
    ra, rb = a * c - b * s, b * c + a * s
    if case["style"] == "neox":
        out[..., : r // 2], out[..., r // 2 : r] = ra, rb
    else:
        out[..., 0:r:2], out[..., 1:r:2] = ra, rb
    return out


def exact(case, seed):
    if case["kind"] == "span_cache":
        return None   # bytes: the same or wrong
    x = inputs(case, seed)
    if case["kind"] == "offload":
        k, v = x["k_pool"], x["v_pool"]
        out = {"k_buf": k[x["old"].long()], "v_buf": v[x["old"].long()]}
        k[x["new"].long()], v[x["new"].long()] = out["k_buf"], out["v_buf"]
        return dict(out, k_pool=k, v_pool=v)
    hq, hkv, d = case["hq"], case["hkv"], case["d"]
    group = hq // hkv
    pre = case.get("prerotated", False)
    k_new = rotate(x["k_new"], x["key_pos"], case) if pre else x["k_new"]
    q = rotate(x["q"], x["q_pos"], case) if pre else x["q"]
    kp, vp = (x["k_pool"].double(), x["v_pool"].double()) if pre else (x["k_pool"], x["v_pool"])
    at = x["slots"].long()
    kp[at // BLOCK, :, at % BLOCK] = k_new
    vp[at // BLOCK, :, at % BLOCK] = x["v_new"].to(vp.dtype)
    o = torch.empty((x["q"].shape[0], hq, d), dtype=torch.float64, device="cuda")
    row, held = 0, None
    for r, a, b, w in x["queries"]:
        if held is None or held[0] != r:
            n = torch.arange(int(x["seq"][r]), device="cuda")
            blk = x["bt"][r].long()[n // BLOCK]
            k = kp[blk, :, n % BLOCK]
            held = (r, k.double() if pre else rotate(k, n, case), vp[blk, :, n % BLOCK].double())
        k, v = held[1][w:b], held[2][w:b]
        n = b - a
        qr = q[row : row + n] if pre else rotate(q[row : row + n], torch.arange(a, b, device="cuda"), case)
        hide = torch.arange(w, b, device="cuda")[None, :] > torch.arange(a, b, device="cuda")[:, None]
        for h in range(hkv):
            kt, vh = k[:, h].t().contiguous(), v[:, h].contiguous()
            for t in range(0, n, 256):
                m = min(256, n - t)
                z = qr[t : t + m, h * group : (h + 1) * group].reshape(m * group, d) @ kt
                z = (z / math.sqrt(d)).view(m, group, -1).masked_fill_(hide[t : t + m, None, :], -math.inf)
                p = torch.softmax(z, dim=-1).view(m * group, -1)
                o[row + t : row + t + m, h * group : (h + 1) * group] = (p @ vh).view(m, group, d)
        row += n
    out = {"o": o, "k_pool": kp, "v_pool": vp}
    if pre:
        out["q"] = q
    return out
