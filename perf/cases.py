"""Performance cases of libsegattn: the calls a program that runs segmented attention makes, over the
sizes it makes them at.

    prompt        seg_attn_fwd_seq: a whole prompt of one layer in one call
    packed        seg_attn_fwd_varlen: prompts of different lengths packed into one call
    train         seg_attn_fwd_seq + seg_attn_bwd_seq: one layer of a training step on windows of
                  consecutive segments (truncated backpropagation); returns the gradients
    train_packed  the same on a packed ragged batch
    turn          seg_attn_fwd + seg_kv_commit on a filled cache: a chunk of new tokens (a user's turn
                  of a conversation, a chunk of a prompt prefilled piece by piece)
    decode        seg_attn_decode: tokens generated one by one on filled caches
    retrieval     seg_kv_retrieve_seq + seg_attn_fwd_seq_retrieved: a whole prompt in retrieval mode
    stream        seg_kv_retrieve + seg_kv_past_select + seg_attn_fwd + seg_kv_commit: the next segment
                  of a stream in retrieval mode
    rope          seg_rope_apply: queries and keys of a layer turned by their positions, in place

A cached case first declares the lengths of its sequences (seg_kv_set_lengths), as a server does
that gives a context's slots to the sequences it runs next; so a pass can be repeated.

`policy` has a digit per KV head: 0 own segment only, 1 carried tail, 2 past, 3 tail and past.  Values
are N(0, 1) rounded to bf16, as in every workload of this repository.
"""
import math

import torch

import paper_2605_11744_amd as sa

BF16, F32, F64 = torch.bfloat16, torch.float32, torch.float64

# Appendix F's operating point of the retrieval operator (R = 512, 32 queries); the sizes that the
# paper leaves open as everywhere in this repository.
RETRIEVAL = dict(n_queries=32, pool_window=8, tail_avg=4, n_anchors=16, win_before=8, win_after=23)


def listed():
    return [
        # A short prompt of a small multi-head layer: the smallest call, one launch of a few microseconds.
        {"name": "prompt_2k_mha", "kind": "prompt", "batch": 1, "n": 2048, "hq": 4, "hkv": 4, "d": 64,
         "seg": 512, "tail": 128, "policy": "1133", "f32": False},
        # A Llama-3-8B-shaped layer on a 32K prompt, half of the KV groups long-range.
        {"name": "prompt_32k", "kind": "prompt", "batch": 1, "n": 32768, "hq": 32, "hkv": 8, "d": 128,
         "seg": 4096, "tail": 1024, "policy": "33331111", "f32": False},
        # The long prompt: 128K tokens, a quarter of the KV groups long-range.  The largest call.
        {"name": "prompt_128k", "kind": "prompt", "batch": 1, "n": 131072, "hq": 32, "hkv": 8, "d": 128,
         "seg": 4096, "tail": 1024, "policy": "33111111", "f32": False},
        # A server's batch of prompts of very different lengths, without padding.
        {"name": "packed_prompts", "kind": "packed", "lengths": "9001,6000,4096,2500,1211,720,333,65", "hq": 32,
         "hkv": 8, "d": 128, "seg": 2048, "tail": 512, "policy": "33111111", "f32": False},
        # Training, truncation depth 1: a window of two segments of 4096 tokens, the paper's tail of 512
        # and half of the heads long-range (Appendix F), one sequence per GPU.
        {"name": "train_8k", "kind": "train", "batch": 1, "n": 8192, "hq": 32, "hkv": 8, "d": 128,
         "seg": 4096, "tail": 512, "policy": "33331111", "f32": False},
        # Training on short documents packed together, a smaller model (head width 64), fp32 results.
        {"name": "train_packed_d64", "kind": "train_packed", "lengths": "2100,1500,1027,900,512,301,130,77", "hq": 16,
         "hkv": 4, "d": 64, "seg": 512, "tail": 128, "policy": "3311", "f32": True},
        # A user's turn of a conversation: 173 new tokens behind a history of 37K.
        {"name": "turn_173", "kind": "turn", "batch": 1, "m": 173, "closed": 9, "fill": 611, "hq": 32, "hkv": 8,
         "d": 128, "seg": 4096, "tail": 1024, "policy": "33111111"},
        # A server's generation step: 64 sequences with contexts of 4K to 64K.
        {"name": "decode_b64", "kind": "decode", "batch": 64, "tokens": 2, "context": 65536, "hq": 32, "hkv": 8,
         "d": 128, "seg": 4096, "tail": 1024, "policy": "33111111"},
        # One user's generation: a single sequence.
        {"name": "decode_b1", "kind": "decode", "batch": 1, "tokens": 8, "context": 24576, "hq": 32, "hkv": 8,
         "d": 128, "seg": 4096, "tail": 1024, "policy": "33331111"},
        # The paper's own long-range channel on a whole prompt: tail 512, R = 512, half of the heads.
        {"name": "retrieval_64k", "kind": "retrieval", "batch": 1, "n": 65536, "hq": 32, "hkv": 8, "d": 128,
         "seg": 4096, "tail": 512, "policy": "22221111", "rows": 512, "theta": 0.0},
        # The same channel segment by segment: retrieve, gather (re-rotated), attend, hand over.
        {"name": "stream_segment", "kind": "stream", "batch": 1, "m": 4096, "closed": 15, "hq": 32, "hkv": 8, "d": 128,
         "seg": 4096, "tail": 512, "policy": "22221111", "rows": 512, "theta": 500000.0},
        # Positions of a 32K prompt's queries and keys.
        {"name": "rope_32k", "kind": "rope", "batch": 1, "n": 32768, "hq": 32, "hkv": 8, "d": 128, "theta": 500000.0},
    ]


# --------------------------------------------------------------------------------------------------
# more cases of the same ranges
# --------------------------------------------------------------------------------------------------
def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


HEADS = [(32, 8, 128), (32, 8, 128), (16, 4, 128), (8, 8, 128), (16, 2, 128), (4, 4, 64), (16, 4, 64), (32, 8, 64)]


def _policy(rng, hkv, past):
    n = rng.choice([max(1, hkv // 4), max(1, hkv // 2)])
    return past * n + "1" * (hkv - n)


def _lengths(rng, total, least):
    got = []
    while total >= least and len(got) < 16:
        n = min(total, _log_int(rng, least, max(least + 1, total)))
        got.append(n)
        total -= n
    return ",".join(str(x) for x in got)


def draw(rng):
    kind = rng.choice(["prompt", "prompt", "packed", "train", "train_packed", "turn", "turn", "decode", "decode",
                       "retrieval", "stream", "rope"])
    hq, hkv, d = rng.choice(HEADS)
    c = {"kind": kind, "hq": hq, "hkv": hkv, "d": d}
    if kind == "prompt":
        n = _log_int(rng, 300, 70000)
        seg = rng.choice([512, 1000, 2048, 4096])
        c.update(batch=1 if n > 8000 else rng.choice([1, 1, 2, 5]), n=n, seg=seg, tail=rng.choice([0, seg // 8, seg // 4]),
                 policy=_policy(rng, hkv, rng.choice("23")), f32=rng.random() < 0.25)
    elif kind in ("packed", "train_packed"):
        seg = rng.choice([512, 1024, 2048] if kind == "train_packed" else [1000, 2048, 4096])
        c.update(lengths=_lengths(rng, _log_int(rng, 1500, 12000 if kind == "train_packed" else 40000), 33), seg=seg,
                 tail=seg // rng.choice([4, 8]), policy=_policy(rng, hkv, "3"), f32=rng.random() < 0.5)
    elif kind == "train":
        seg = rng.choice([512, 1024, 2048, 4096])
        c.update(batch=rng.choice([1, 1, 2, 4]), n=rng.randint(seg, 2 * seg), seg=seg, tail=seg // rng.choice([4, 8]),
                 policy=_policy(rng, hkv, "3"), f32=rng.random() < 0.5)
    elif kind == "turn":
        seg = rng.choice([2048, 4096])
        m = _log_int(rng, 2, seg)
        c.update(batch=rng.choice([1, 1, 1, 3]), m=m, closed=rng.randint(1, 16), fill=rng.randint(0, seg - m), seg=seg,
                 tail=seg // rng.choice([4, 8]), policy=_policy(rng, hkv, "3"))
    elif kind == "decode":
        seg = rng.choice([2048, 4096])
        c.update(batch=_log_int(rng, 1, 64), tokens=rng.randint(1, 4), context=seg * rng.randint(2, 16), seg=seg,
                 tail=seg // rng.choice([4, 8]), policy=_policy(rng, hkv, rng.choice("23")))
    elif kind == "retrieval":
        seg = rng.choice([1024, 2048, 4096])
        c.update(batch=1, n=_log_int(rng, 2 * seg, 90000), seg=seg, tail=seg // 8, policy=_policy(rng, hkv, "2"),
                 rows=rng.choice([256, 512]), theta=rng.choice([0.0, 10000.0]))
    elif kind == "stream":
        seg = rng.choice([1024, 2048, 4096])
        c.update(batch=rng.choice([1, 1, 2, 6]), m=rng.choice([seg, seg, rng.randint(64, seg)]), closed=rng.randint(2, 16),
                 seg=seg, tail=seg // 8, policy=_policy(rng, hkv, "2"), rows=rng.choice([256, 512]),
                 theta=rng.choice([0.0, 500000.0]))
    else:
        c.update(batch=rng.choice([1, 2, 3]), n=_log_int(rng, 64, 40000), theta=rng.choice([10000.0, 500000.0]))
    return c


# --------------------------------------------------------------------------------------------------
# inputs, from the seed alone
# --------------------------------------------------------------------------------------------------
def _randn(g, *shape):
    """N(0, 1) in bf16, drawn a part at a time so that the fp32 draws stay small."""
    out = torch.empty(shape, dtype=BF16, device="cuda")
    flat = out.view(-1)
    for i in range(0, flat.numel(), 1 << 27):
        part = flat[i:i + (1 << 27)]
        part.copy_(torch.randn(part.numel(), generator=g, device="cuda", dtype=F32))
    return out


def _lens(c):
    return [int(x) for x in c["lengths"].split(",")]


def _contexts(c, seed):
    """Closed segments and open rows of every sequence of a decode batch: one sequence has the whole
    context, a batch a uniform mix of everything up to it.  No segment fills up within the tokens
    of the case."""
    most, seg, room = c["context"] // c["seg"] - 1, c["seg"], c["seg"] - c["tokens"] - 1
    if c["batch"] == 1:
        return [max(most, 1)], [seg // 2 + 5]
    g = torch.Generator().manual_seed(1000 * c["batch"] + c["context"])  # sizes belong to the case, not to the seed
    k = torch.randint(1, max(most, 1) + 1, (c["batch"],), generator=g)
    f = torch.randint(0, room, (c["batch"],), generator=g)
    return k.tolist(), f.tolist()


def _inputs(c, seed):
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    kind, hq, hkv, d = c["kind"], c["hq"], c["hkv"], c["d"]
    s = {}
    if kind in ("prompt", "train", "retrieval", "rope"):
        b, n = c["batch"], c["n"]
        s["q"], s["k"] = _randn(g, b, n, hq, d), _randn(g, b, n, hkv, d)
        if kind != "rope":
            s["v"] = _randn(g, b, n, hkv, d)
        if kind == "train":
            s["go"] = _randn(g, b, n, hq, d)
    elif kind in ("packed", "train_packed"):
        n = sum(_lens(c))
        s["q"], s["k"], s["v"] = _randn(g, n, hq, d), _randn(g, n, hkv, d), _randn(g, n, hkv, d)
        if kind == "train_packed":
            s["go"] = _randn(g, n, hq, d)
    else:
        b, seg, tail = c["batch"], c["seg"], c["tail"]
        if kind == "decode":
            closed, fill = _contexts(c, seed)
            s["q"], s["k"], s["v"] = (_randn(g, c["tokens"], b, h, d) for h in (hq, hkv, hkv))
        else:
            closed, fill = [c["closed"]] * b, [c.get("fill", 0)] * b
            s["q"], s["k"], s["v"] = (_randn(g, b, c["m"], h, d) for h in (hq, hkv, hkv))
            if kind == "stream":
                s["q_prev"] = _randn(g, b, seg, hq, d)
        # rows that the cache holds before the call, per (sequence, KV head), oldest first
        held = [[(closed[i] * seg if int(p) & 2 else min(tail, closed[i] * seg)) + fill[i] for p in c["policy"]]
                for i in range(b)]
        flat_k, flat_v = (_randn(g, sum(map(sum, held)), d) for _ in range(2))
        at, s["hist"] = 0, []
        for row in held:
            s["hist"].append([])
            for n in row:
                s["hist"][-1].append((flat_k[at:at + n], flat_v[at:at + n]))
                at += n
        s["closed"], s["fill"] = [x * seg for x in closed], fill
    return s


class _Context:
    """A libsegattn context over an arena that torch owns."""

    def __init__(self, cfg):
        self.bytes = sa.segattn_cache_bytes(cfg)
        self.arena = torch.empty(self.bytes, dtype=torch.uint8, device="cuda")
        self.handle = sa.segattn_create(cfg, self.arena, self.bytes)

    def rows(self, b, h, d):
        ko, vo, cap = sa.segattn_cache_span(self.handle, b, h)
        return tuple(self.arena[o:o + cap * d * 2].view(BF16).view(cap, d) for o in (ko, vo))

    def __del__(self):
        if getattr(self, "handle", None):
            sa.segattn_destroy(self.handle)


def prepare(case, seed):
    c = case
    kind, hq, hkv, d = c["kind"], c["hq"], c["hkv"], c["d"]
    s = _inputs(c, seed)
    s["case"], s["stream"] = c, torch.cuda.current_stream().cuda_stream
    policy = [int(p) for p in c.get("policy", "1" * hkv)]
    base = dict(n_q_heads=hq, n_kv_heads=hkv, head_dim=d, kv_policy=policy)
    odt = F32 if c.get("f32") else BF16
    if kind == "rope":
        s["cfg"] = sa.make_config(batch=c["batch"], seg_len=4096, tail_len=0, rope_theta=c["theta"], **base)
    elif kind in ("packed", "train_packed"):
        lens = _lens(c)
        n = sum(lens)
        s["total"], s["longest"] = n, max(lens)
        s["cu"] = torch.tensor([0] + [sum(lens[:i + 1]) for i in range(len(lens))], dtype=torch.int32, device="cuda")
        s["cfg"] = sa.make_config(batch=len(lens), seg_len=c["seg"], tail_len=c["tail"], out_fp32=bool(c["f32"]), **base)
        s["out"] = torch.empty((n, hq, d), dtype=odt, device="cuda")
        s["lse"] = torch.empty((hq, n), dtype=F32, device="cuda")
        if kind == "train_packed":
            s["ws"] = torch.empty(sa.seg_attn_bwd_varlen_workspace_bytes(s["cfg"], n), dtype=torch.uint8, device="cuda")
    elif kind in ("prompt", "train", "retrieval"):
        b, n = c["batch"], c["n"]
        s["cfg"] = sa.make_config(batch=b, seg_len=c["seg"], tail_len=c["tail"], out_fp32=bool(c.get("f32")),
                                  rope_theta=c.get("theta", 0.0), **base)
        s["out"] = torch.empty((b, n, hq, d), dtype=odt, device="cuda")
        s["lse"] = torch.empty((b, hq, n), dtype=F32, device="cuda")
        if kind == "train":
            s["ws"] = torch.empty(sa.seg_attn_bwd_workspace_bytes(s["cfg"], n), dtype=torch.uint8, device="cuda")
        if kind == "retrieval":
            s["r"] = sa.make_retrieval(**RETRIEVAL)
            segs = -(-n // c["seg"])
            s["ws"] = torch.empty(sa.seg_kv_retrieve_seq_workspace_bytes(s["cfg"], s["r"], n), dtype=torch.uint8, device="cuda")
            s["ws2"] = torch.empty(sa.seg_attn_fwd_seq_retrieved_workspace_bytes(s["cfg"], n, c["rows"]), dtype=torch.uint8, device="cuda")
            s["idx"] = torch.zeros((b, segs, sum(p >> 1 for p in policy), c["rows"]), dtype=torch.int32, device="cuda")
    else:
        b, seg, tail = c["batch"], c["seg"], c["tail"]
        new = c["tokens"] if kind == "decode" else c["m"]
        room = (max(s["closed"]) // seg + 2) * seg
        s["cfg"] = sa.make_config(batch=b, seg_len=seg, tail_len=tail, past_capacity=room,
                                  retrieved_capacity=c["rows"] if kind == "stream" else 0,
                                  rope_theta=c.get("theta", 0.0), **base)
        s["ctx"] = _Context(s["cfg"])
        s["tails"] = [min(tail, x) for x in s["closed"]]
        for i in range(b):
            for h, p in enumerate(policy):
                first = 0 if p & 2 else tail - s["tails"][i]
                for to, rows in zip(s["ctx"].rows(i, h, d), s["hist"][i][h]):
                    to[first:first + rows.shape[0]] = rows
        if kind == "decode":
            s["out"] = torch.empty((new, b, hq, d), dtype=BF16, device="cuda")
            s["lse"] = torch.empty((new, b, hq), dtype=F32, device="cuda")
            # the rows that the steps append to the last sequence's first head
            s["kept"] = s["ctx"].rows(b - 1, 0, d)[1][s["closed"][-1] + s["fill"][-1]:][:new]
        else:
            s["out"] = torch.empty((b, new, hq, d), dtype=BF16, device="cuda")
            s["lse"] = torch.empty((b, hq, new), dtype=F32, device="cuda")
            # the rows that the commit leaves in the cache, of the first head that keeps them all
            # and of the last head
            k0 = s["ctx"].rows(0, 0, d)[0]
            s["kept"] = k0[s["closed"][0] + s["fill"][0]:][:new]
            closes = s["fill"][0] + new == seg
            kl = s["ctx"].rows(0, hkv - 1, d)[1]
            s["kept_last"] = kl[:tail] if closes else kl[tail + s["fill"][0]:][:new]
        if kind == "stream":
            s["r"] = sa.make_retrieval(**RETRIEVAL)
            s["ws"] = torch.empty(sa.seg_kv_retrieve_workspace_bytes(s["ctx"].handle, s["r"]), dtype=torch.uint8, device="cuda")
            s["idx"] = torch.zeros((b, sum(p >> 1 for p in policy), c["rows"]), dtype=torch.int32, device="cuda")
        del s["hist"]
    if kind in ("train", "train_packed"):
        for x, like in (("dq", "q"), ("dk", "k"), ("dv", "v")):
            s[x] = torch.empty_like(s[like], dtype=odt)
    return s


# --------------------------------------------------------------------------------------------------
# one pass
# --------------------------------------------------------------------------------------------------
def run(s):
    c, st = s["case"], s["stream"]
    kind = c["kind"]
    if kind == "prompt":
        sa.seg_attn_fwd_seq(s["cfg"], s["q"], s["k"], s["v"], c["n"], s["out"], s["lse"], st)
        return [s["out"], s["lse"]]
    if kind == "packed":
        sa.seg_attn_fwd_varlen(s["cfg"], s["q"], s["k"], s["v"], s["cu"], s["total"], s["longest"], s["out"], s["lse"], st)
        return [s["out"], s["lse"]]
    if kind == "train":
        sa.seg_attn_fwd_seq(s["cfg"], s["q"], s["k"], s["v"], c["n"], s["out"], s["lse"], st)
        sa.seg_attn_bwd_seq(s["cfg"], s["q"], s["k"], s["v"], s["out"], s["lse"], s["go"], c["n"], s["dq"], s["dk"], s["dv"],
                            s["ws"], s["ws"].numel(), st)
        return [s["out"], s["lse"], s["dq"], s["dk"], s["dv"]]
    if kind == "train_packed":
        sa.seg_attn_fwd_varlen(s["cfg"], s["q"], s["k"], s["v"], s["cu"], s["total"], s["longest"], s["out"], s["lse"], st)
        sa.seg_attn_bwd_varlen(s["cfg"], s["q"], s["k"], s["v"], s["out"], s["lse"], s["go"], s["cu"], s["total"], s["longest"],
                               s["dq"], s["dk"], s["dv"], s["ws"], s["ws"].numel(), st)
        return [s["out"], s["lse"], s["dq"], s["dk"], s["dv"]]
    if kind == "retrieval":
        sa.seg_kv_retrieve_seq(s["cfg"], s["r"], s["q"], s["k"], c["n"], c["rows"], s["idx"], s["ws"], s["ws"].numel(), st)
        sa.seg_attn_fwd_seq_retrieved(s["cfg"], s["q"], s["k"], s["v"], c["n"], s["idx"], c["rows"], s["ws2"], s["ws2"].numel(),
                                      s["out"], s["lse"], st)
        return [s["idx"][:, 1:], s["out"], s["lse"]]
    if kind == "rope":
        sa.seg_rope_apply(s["cfg"], s["q"], s["k"], c["n"], None, st)
        return [s["q"], s["k"]]
    ctx = s["ctx"].handle
    sa.seg_kv_set_lengths(ctx, s["closed"], s["tails"], s["fill"], st)
    if kind == "decode":
        for t in range(c["tokens"]):
            sa.seg_attn_decode(ctx, s["q"][t], s["k"][t], s["v"][t], s["out"][t], s["lse"][t], st)
        return [s["out"], s["lse"], s["kept"]]
    if kind == "stream":
        sa.seg_kv_retrieve(ctx, s["r"], s["q_prev"], c["seg"], c["rows"], s["idx"], s["ws"], s["ws"].numel(), st)
        sa.seg_kv_past_select(ctx, s["idx"], c["rows"], st)
    sa.seg_attn_fwd(ctx, s["q"], s["k"], s["v"], c["m"], s["out"], s["lse"], st)
    sa.seg_kv_commit(ctx, s["k"], s["v"], c["m"], st)
    done = [s["out"], s["lse"], s["kept"], s["kept_last"]]
    return done + [s["idx"]] if kind == "stream" else done


# --------------------------------------------------------------------------------------------------
# what a pass cannot do without
# --------------------------------------------------------------------------------------------------
def _pairs(n, seg, tail, pol, rows=None):
    """(visible, differentiable) (query, key) pairs of one query head of a sequence of n rows; `rows`:
    a past head sees that many retrieved rows instead of its whole history."""
    vis = diff = 0
    for s in range(0, n, seg):
        m = min(seg, n - s)
        own = m * (m + 1) // 2
        t = m * min(tail, s) if pol & 1 else 0
        past = m * (s if rows is None else min(rows, s)) if pol & 2 else 0
        vis += own + max(t, past)
        diff += own + t
    return vis, diff


def work(case):
    c = case
    kind, hq, hkv, d = c["kind"], c["hq"], c["hkv"], c["d"]
    g, e = hq // hkv, 4 if c.get("f32") else 2
    if kind == "rope":
        return {"bytes": 2 * 2 * c["batch"] * c["n"] * (hq + hkv) * d, "flops": 3 * c["batch"] * c["n"] * (hq + hkv) * d}
    pols = [int(p) for p in c["policy"]]
    if kind in ("prompt", "packed", "train", "train_packed", "retrieval"):
        lens = _lens(c) if "lengths" in c else [c["n"]] * c["batch"]
        n, vis, diff = sum(lens), 0, 0
        for x in lens:
            for p in pols:
                a, b = _pairs(x, c["seg"], c["tail"], p, c.get("rows"))
                vis, diff = vis + g * a, diff + g * b
        nbytes = n * (hq * d * 2 + 2 * hkv * d * 2 + hq * d * e + hq * 4)
        flops = 4 * d * vis
        if kind.startswith("train"):
            nbytes += n * (hq * d * 2 + hq * d * e + 2 * hkv * d * e)
            flops += 6 * d * vis + 4 * d * diff
        if kind == "retrieval":  # every key before a segment is scored against the segment's summaries
            past = sum(p >> 1 for p in pols)
            segs = -(-n // c["seg"])
            flops += 2 * d * g * 5 * past * c["seg"] * segs * (segs - 1) // 2
            nbytes += 4 * past * segs * c["rows"]
        return {"bytes": nbytes, "flops": flops}
    b, seg, tail = c["batch"], c["seg"], c["tail"]
    nbytes = flops = 0
    if kind == "decode":
        closed, fill = _contexts(c, 0)
        for t in range(c["tokens"]):
            for i in range(b):
                for p in pols:
                    rows = fill[i] + t + 1 + (closed[i] * seg if p & 2 else min(tail, closed[i] * seg) if p & 1 else 0)
                    nbytes += rows * 2 * d * 2
                    flops += 4 * d * g * rows
            nbytes += b * (hq * d * 2 * 2 + hq * 4)
        return {"bytes": nbytes, "flops": flops}
    m, history = c["m"], c["closed"] * seg
    for p in pols:
        before = c.get("fill", 0)
        if p & 2:
            before += c["rows"] if kind == "stream" else history
        elif p & 1:
            before += min(tail, history)
        flops += b * 4 * d * g * (m * before + m * (m + 1) // 2)
        nbytes += b * 2 * d * 2 * (before + 2 * m)  # held rows and new rows read, new rows written
        if kind == "stream" and p & 2:  # the scan of the pool's keys
            nbytes += b * history * d * 2
            flops += 2 * d * g * 5 * b * history
    nbytes += b * m * hq * (2 * d * 2 + 4)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """bf16 operands: the weights of the second product (and dS in the backward pass) are rounded to bf16,
    about 1e-3 in the 2-norm, and so are bf16 results (1.7e-3).  Measured against exact(): outputs
    2.0e-3 to 2.3e-3 off in bf16 and 1.2e-3 in fp32, gradients up to 2.5e-3; four times that."""
    if case["kind"] == "rope":  # 32-bit arithmetic, bf16 results: a value next to a tie may round the other way
        return {"rel": 2e-3, "max": 1.6e-2}
    if case["kind"] in ("stream", "retrieval"):  # an index may differ where two scores are a rounding apart
        return {"rel": 1e-2, "differ": 5e-3}
    return {"rel": 1e-2}


# --------------------------------------------------------------------------------------------------
# the same in 64 bits, from the definition
# --------------------------------------------------------------------------------------------------
def _attend(q, k, v, n0, own, scale, go=None):
    """Rows q [m, g, d] of one KV group against k, v [n0 + own rows, d]: row t sees the first n0 rows and the next
    t + 1 + own - m.  Returns out [m, g, d], lse [g, m], and with go [m, g, d] also dq, dk, dv (all keys)."""
    m, g, d = q.shape
    out = torch.empty((m, g, d), dtype=F64, device="cuda")
    lse = torch.empty((g, m), dtype=F64, device="cuda")
    k, v = k.to(F64), v.to(F64)
    grads = None if go is None else [torch.zeros((m, g, d), dtype=F64, device="cuda"), torch.zeros_like(k), torch.zeros_like(v)]
    step = max(1, min(m, (1 << 28) // (g * (n0 + own))))
    for t0 in range(0, m, step):
        t1 = min(m, t0 + step)
        n = n0 + own - m + t1  # keys that the last row of the part sees
        x = q[t0:t1].to(F64).reshape(-1, d)
        z = (x @ k[:n].t()) * scale
        sees = n0 + own - m + 1 + torch.arange(t0, t1, device="cuda").repeat_interleave(g)
        z.masked_fill_(torch.arange(n, device="cuda")[None, :] >= sees[:, None], -math.inf)
        top = z.amax(1, keepdim=True)
        z.sub_(top).exp_()
        total = z.sum(1, keepdim=True)
        z.div_(total)
        o = z @ v[:n]
        out[t0:t1] = o.view(-1, g, d)
        lse[:, t0:t1] = (top + total.log()).view(-1, g).t()
        if go is not None:
            dy = go[t0:t1].to(F64).reshape(-1, d)
            grads[2][:n] += z.t() @ dy
            ds = dy @ v[:n].t()
            ds.sub_((dy * o).sum(1, keepdim=True)).mul_(z).mul_(scale)
            grads[0][t0:t1] = (ds @ k[:n]).view(-1, g, d)
            grads[1][:n] += ds.t() @ x
    return (out, lse) if go is None else (out, lse, *grads)


def _sequence(c, q, k, v, go=None, prefix=None):
    """One sequence, q [n, hq, d]; k, v [n, hkv, d]; prefix(kv head, segment start) -> retrieved K and V rows."""
    (n, hq, d), hkv = q.shape, k.shape[1]
    g = hq // hkv
    out = torch.empty((n, hq, d), dtype=F64, device="cuda")
    lse = torch.empty((hq, n), dtype=F64, device="cuda")
    dq, dk, dv = (None,) * 3 if go is None else (torch.zeros(x.shape, dtype=F64, device="cuda") for x in (q, k, v))
    for h in range(hkv):
        p, hs = int(c["policy"][h]), slice(h * g, (h + 1) * g)
        for s in range(0, n, c["seg"]):
            e = min(n, s + c["seg"])
            lo = 0 if p & 2 else max(0, s - c["tail"]) if p & 1 else s
            if prefix is not None and p & 2:
                pk, pv = prefix(h, s)
                kk, vv = torch.cat([pk, k[s:e, h]]), torch.cat([pv, v[s:e, h]])
            else:
                kk, vv = k[lo:e, h].contiguous(), v[lo:e, h].contiguous()
            n0 = kk.shape[0] - (e - s)
            got = _attend(q[s:e, hs], kk, vv, n0, e - s, d ** -0.5, None if go is None else go[s:e, hs])
            out[s:e, hs], lse[hs, s:e] = got[0], got[1]
            if go is not None:
                dq[s:e, hs] = got[2]
                first = max(0, s - c["tail"]) if p & 1 else s  # rows reached only as past get no gradient
                dk[first:e, h] += got[3][first - lo:]
                dv[first:e, h] += got[4][first - lo:]
    return (out, lse) if go is None else (out, lse, dq, dk, dv)


def _retrieve(q, k, rows):
    """The retrieval operator on the query rows q [L, g, d] of a group and the pool k [n, d]."""
    r = RETRIEVAL
    q = q[-r["n_queries"]:].to(F64)
    parts = list(q.split(r["pool_window"])) + [q[-r["tail_avg"]:]]
    sums = torch.stack([x.mean(0) for x in parts]).reshape(-1, q.shape[-1]).to(BF16).to(F64)
    score = torch.cat([(part.to(F64) @ sums.t()).amax(1) for part in k.split(1 << 15)])
    n, chosen, count = k.shape[0], torch.zeros(k.shape[0], dtype=torch.bool), 0
    for a in torch.sort(score, descending=True, stable=True).indices[:r["n_anchors"]].tolist():
        for x in range(max(0, a - r["win_before"]), min(n, a + r["win_after"] + 1)):
            if count < rows and not chosen[x]:
                chosen[x], count = True, count + 1
    left = (~chosen).nonzero().view(-1)[:rows - count]
    chosen[left] = True
    return chosen.nonzero().view(-1).cuda()


def _turn_by(x, positions, theta):
    """x [rows, ..., d] turned by positions [rows], channel i with channel i + d / 2, in 64 bits."""
    d = x.shape[-1]
    f = theta ** (-2.0 * torch.arange(d // 2, dtype=F64, device="cuda") / d)
    a = positions.to(F64)[:, None] * f
    a = a.view(a.shape[0], *[1] * (x.dim() - 2), d // 2)
    lo, hi = x[..., :d // 2].to(F64), x[..., d // 2:].to(F64)
    return torch.cat([lo * a.cos() - hi * a.sin(), lo * a.sin() + hi * a.cos()], -1)


def _gathered(k, v, at, idx, theta):
    """Rows idx of a pool that ends at position `at`, as the retrieved prefix."""
    pk, pv = k[idx], v[idx]
    if theta:
        where = at - idx.numel() + torch.arange(idx.numel(), device="cuda")
        pk = _turn_by(pk, where - idx, theta).to(BF16)  # the gathered keys are bf16 rows again
    return pk, pv


def exact(case, seed):
    c = case
    kind, hq, hkv, d = c["kind"], c["hq"], c["hkv"], c["d"]
    s = _inputs(c, seed)
    q, k, g = s["q"], s["k"], hq // hkv
    if kind == "rope":
        at = torch.arange(c["n"], device="cuda")
        return [torch.stack([_turn_by(x[b], at, c["theta"]) for b in range(c["batch"])]) for x in (q, k)]
    v = s["v"]
    if kind in ("packed", "train_packed"):
        got, at = [], 0
        for n in _lens(c):
            r = slice(at, at + n)
            got.append(_sequence(c, q[r], k[r], v[r], s["go"][r] if "go" in s else None))
            at += n
        return [torch.cat(x, 1 if i == 1 else 0) for i, x in enumerate(zip(*got))]
    if kind in ("prompt", "train"):
        got = [_sequence(c, q[b], k[b], v[b], s["go"][b] if "go" in s else None) for b in range(c["batch"])]
        return [torch.stack(x) for x in zip(*got)]
    if kind == "retrieval":
        idx, got, seg = [], [], c["seg"]
        for b in range(c["batch"]):
            lists = {}
            for s0 in range(seg, c["n"], seg):
                for h, p in enumerate(c["policy"]):
                    if int(p) & 2:
                        lists[h, s0] = _retrieve(q[b, s0 - seg:s0, h * g:(h + 1) * g], k[b, :s0, h], c["rows"])
            idx.append(torch.stack([torch.stack([lists[h, s0] for h, p in enumerate(c["policy"]) if int(p) & 2])
                                    for s0 in range(seg, c["n"], seg)]))

            def prefix(h, s0):
                i = lists.get((h, s0), torch.zeros(0, dtype=torch.int64, device="cuda"))
                return _gathered(k[b, :, h], v[b, :, h], s0, i, c["theta"] if s0 else 0.0)
            got.append(_sequence(c, q[b], k[b], v[b], prefix=prefix))
        return [torch.stack(idx)] + [torch.stack(x) for x in zip(*got)]
    b = c["batch"]
    if kind == "decode":
        out = torch.empty((c["tokens"], b, hq, d), dtype=F64, device="cuda")
        lse = torch.empty((c["tokens"], b, hq), dtype=F64, device="cuda")
        for i in range(b):
            for h in range(hkv):
                hs = slice(h * g, (h + 1) * g)
                kk = torch.cat([s["hist"][i][h][0], k[:, i, h]])
                vv = torch.cat([s["hist"][i][h][1], v[:, i, h]])
                o, l = _attend(q[:, i, hs], kk, vv, s["hist"][i][h][0].shape[0], c["tokens"], d ** -0.5)
                out[:, i, hs], lse[:, i, hs] = o, l.t()
        return [out, lse, v[:, b - 1, 0].to(F64)]
    m = c["m"]
    out = torch.empty((b, m, hq, d), dtype=F64, device="cuda")
    lse = torch.empty((b, hq, m), dtype=F64, device="cuda")
    idx = []
    for i in range(b):
        for h, p in enumerate(c["policy"]):
            hs, (hk, hv) = slice(h * g, (h + 1) * g), s["hist"][i][h]
            if kind == "stream" and int(p) & 2:
                idx.append(_retrieve(s["q_prev"][i, :, hs], hk, c["rows"]))
                hk, hv = _gathered(hk, hv, s["closed"][i], idx[-1], c["theta"])
            kk, vv = torch.cat([hk, k[i, :, h]]), torch.cat([hv, v[i, :, h]])
            out[i, :, hs], lse[i, hs] = _attend(q[i, :, hs], kk, vv, hk.shape[0], m, d ** -0.5)
    last = v[0, :, hkv - 1].to(F64)
    if s["fill"][0] + m == c["seg"]:  # the segment closes: the last head keeps its tail
        hv = s["hist"][0][hkv - 1][1]
        last = torch.cat([hv[hv.shape[0] - s["fill"][0]:].to(F64), last])[-c["tail"]:]
    done = [out, lse, k[0, :, 0].to(F64), last]
    return done + [torch.stack(idx).view(b, -1, c["rows"])] if kind == "stream" else done
