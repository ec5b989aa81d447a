"""The work that a program has this library do, as cases that can be timed.

A case is a dict of plain values: what is called (``path``), how many
dialogues, their lengths, the head shape, and how the KV cache is kept. The
dialogue layout is drawn from the case's own ``layout`` number, so that a
case is always the same amount of work; the tensors are drawn from the seed.

Paths (each through ``paper_2408_00539_amd.ops``):

* ``fwd``: the forward over packed multi-turn dialogues (``ops.fwd``);
* ``train``: forward and backward of one attention layer (``ops.fwd``,
  ``ops.bwd``);
* ``prefill``: a new segment per dialogue against its KV cache
  (``ops.prefill_cached``, ``ops.prefill_cached_segment``,
  ``ops.prefill_cached_rope2d``, ``ops.prefill_paged``);
* ``decode``: one answer token per dialogue (``ops.decode``,
  ``ops.decode_paged``).

``cached`` and ``tokens`` are the longest dialogue's; with ``ragged`` the
others are shorter, down to ``ragged`` times that (1 = all the same length).
"""

from __future__ import annotations

import math

import numpy as np
import torch

from paper_2408_00539_amd import ops
from paper_2408_00539_amd import workloads as W

# --------------------------------------------------------------------------
# Cases
# --------------------------------------------------------------------------


def _packed(path, dialogues, tokens, ragged, turns, hq, hkv, d, layout):
    return {"path": path, "dialogues": dialogues, "tokens": tokens, "ragged": ragged,
            "turns": turns, "hq": hq, "hkv": hkv, "d": d, "layout": layout}


def _cached(path, dialogues, cached, ragged, new, new_ragged, hq, hkv, d, layout, page=0,
            answer=False, rope=False):
    return {"path": path, "dialogues": dialogues, "cached": cached, "ragged": ragged,
            "new": new, "new_ragged": new_ragged, "hq": hq, "hkv": hkv, "d": d,
            "layout": layout, "page": page, "answer": answer, "rope": rope}


def listed():
    def named(name, case):
        return dict(case, name=name)

    return [
        # one short dialogue of a small model, forward only: latency and
        # launches (scoring a single sample, a unit of an interactive tool)
        named("fwd_1x320_h16_d64", _packed("fwd", 1, 320, 1.0, 4, 16, 16, 64, 1)),
        # a long-context forward with grouped KV heads (evaluation of long
        # dialogues)
        named("fwd_2x16384_h32kv8_d128", _packed("fwd", 2, 16384, 1.0, 24, 32, 8, 128, 2)),
        # a small fine-tuning step: a few short dialogues of unequal length
        named("train_6x900_h16kv4_d64", _packed("train", 6, 900, 0.15, 4, 16, 4, 64, 3)),
        # an ordinary fine-tuning micro-batch: packed dialogues of unequal
        # length, grouped KV heads
        named("train_12x3001_h32kv8_d128", _packed("train", 12, 3001, 0.2, 6, 32, 8, 128, 4)),
        # the benchmark's training step
        named("train_4x8192_h32_d128", _packed("train", 4, 8192, 1.0, 16, 32, 32, 128, 5)),
        # a new user turn over a long reused cache, all dialogues in a batch
        named("prefill_32x8192_new64to512_h32_d128",
              _cached("prefill", 32, 8192, 1.0, 512, 0.125, 32, 32, 128, 6)),
        # the short turns of the multi-turn latency test: 40 dialogues, 40
        # new query tokens, the middle of a 4000-token conversation
        named("prefill_40x2000_new40_h32kv8_d128",
              _cached("prefill", 40, 2000, 1.0, 40, 1.0, 32, 8, 128, 7)),
        # turns of a model with 2-D rotary positions, unequal histories
        named("prefill_rope_8x3000_new200_h32kv2_d128",
              _cached("prefill", 8, 3000, 0.2, 200, 0.1, 32, 2, 128, 8, rope=True)),
        # speculative decoding: one chunk of 8 drafted answer tokens per
        # dialogue, over a paged cache
        named("verify_24x6000_new8_paged256_h32kv8_d128",
              _cached("prefill", 24, 6000, 0.25, 8, 1.0, 32, 8, 128, 9, page=256, answer=True)),
        # one decode step of a large batch with long caches
        named("decode_32x8192_h32_d128",
              _cached("decode", 32, 8192, 1.0, 1, 1.0, 32, 32, 128, 10)),
        # a decode step of a serving batch: grouped heads, paged cache,
        # dialogues of every length
        named("decode_40x4000_paged64_h32kv8_d128",
              _cached("decode", 40, 4000, 0.05, 1, 1.0, 32, 8, 128, 11, page=64)),
        # a decode step of a single conversation: latency
        named("decode_1x2500_h32kv8_d128",
              _cached("decode", 1, 2500, 1.0, 1, 1.0, 32, 8, 128, 12)),
    ]


# (query heads, KV heads): ungrouped, grouped by 2 to 8 and 16, and a group
# size that is no power of two
_HEADS = ((8, 8), (16, 16), (32, 32), (16, 8), (16, 4), (32, 8), (64, 8), (32, 2), (24, 8))


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case of the same ranges: short to long dialogues, one to many
    of them, equal and ragged, every path and head shape."""
    most = {k: max(work(c)[k] for c in listed()) for k in ("bytes", "flops")}
    while True:
        hq, hkv = rng.choice(_HEADS)
        d = rng.choice((64, 128, 128))
        path = rng.choice(("fwd", "train", "prefill", "prefill", "decode"))
        layout = rng.randrange(1 << 20)
        ragged = rng.choice((1.0, 0.5, 0.1))
        if path in ("fwd", "train"):
            tokens = _log_int(rng, 100, 16384 if path == "fwd" else 8192)
            c = _packed(path, _log_int(rng, 1, 16), tokens, ragged,
                        rng.randint(1, max(1, min(24, tokens // 64))), hq, hkv, d, layout)
        else:
            page = rng.choice((0, 64, 128, 256))
            answer = path == "prefill" and rng.random() < 0.4
            new = 1 if path == "decode" else _log_int(rng, 4, 64 if answer else 512)
            rope = path == "prefill" and page == 0 and rng.random() < 0.4
            c = _cached(path, _log_int(rng, 1, 48), _log_int(rng, 128, 12288), ragged, new,
                        rng.choice((1.0, 0.2)), hq, hkv, d, layout, page, answer, rope)
        w = work(c)
        if w["bytes"] <= most["bytes"] and w["flops"] <= most["flops"]:
            return c


# --------------------------------------------------------------------------
# Layouts (from the case alone)
# --------------------------------------------------------------------------

def _lengths(rng, n, longest, ragged):
    if ragged >= 1.0:
        return np.full(n, longest, dtype=np.int64)
    x = rng.integers(max(1, int(longest * ragged)), longest + 1, size=n)
    x[rng.integers(n)] = longest
    return x


def _dialogues(case):
    """Packed dialogue structure: alternating query and answer segments with
    lognormal lengths (queries shorter than answers)."""
    rng = np.random.default_rng(case["layout"])
    out = []
    for n in _lengths(rng, case["dialogues"], case["tokens"], case["ragged"]):
        turns = max(1, min(case["turns"], int(n) // 4))
        x = np.empty(2 * turns)
        x[0::2] = rng.lognormal(math.log(96.0), 0.8, size=turns)
        x[1::2] = rng.lognormal(math.log(320.0), 0.7, size=turns)
        out.append(W.alternating(W.rescale_lengths(x, int(n))))
    return W.segments_from_lengths(out)


def _cache_lengths(case):
    """(cached tokens, new tokens) of each dialogue."""
    rng = np.random.default_rng(case["layout"])
    n = case["dialogues"]
    return (_lengths(rng, n, case["cached"], case["ragged"]),
            _lengths(rng, n, case["new"], case["new_ragged"]))


def _lim(segs):
    """Last key each token of a packed batch sees."""
    lim = np.empty(segs.total, dtype=np.int64)
    for g, q in enumerate(segs.seg_is_query):
        a, c = int(segs.cu_segs[g]), int(segs.cu_segs[g + 1])
        lim[a:c] = c - 1 if q else np.arange(a, c)
    return lim


def work(case):
    """Bytes of the inputs and outputs, and the products of the visible
    (row, key) pairs: 4 d per pair and query head forward, 10 d backward."""
    hq, hkv, d = case["hq"], case["hkv"], case["d"]
    if case["path"] in ("fwd", "train"):
        segs = _dialogues(case)
        T = segs.total
        start = np.repeat(segs.cu_seqlens[:-1].astype(np.int64), np.diff(segs.cu_seqlens))
        pairs = int((_lim(segs) - start + 1).sum())
        nbytes = T * (4 * hq * d + 4 * hkv * d + 4 * hq)  # q, o, k, v, lse
        flops = 4 * d * hq * pairs
        if case["path"] == "train":  # again those, dO, and fp32 dQ, dK, dV
            nbytes += T * (4 * hq * d + 4 * hkv * d + 4 * hq)
            nbytes += T * (2 * hq * d + 4 * hq * d + 8 * hkv * d)
            flops += 10 * d * hq * pairs
        return {"bytes": nbytes, "flops": flops}
    cached, new = _cache_lengths(case)
    Tn = int(new.sum())
    if case["answer"]:
        pairs = int((cached * new + new * (new + 1) // 2).sum())
    else:
        pairs = int((new * (cached + new)).sum())
    # the cached K and V; the new rows of q, o, lse; new K and V read and appended
    nbytes = int(cached.sum()) * 4 * hkv * d + Tn * (4 * hq * d + 4 * hq + 8 * hkv * d)
    return {"bytes": nbytes, "flops": 4 * d * hq * pairs}


# --------------------------------------------------------------------------
# State and one pass
# --------------------------------------------------------------------------

def _normal(gen, *shape):
    """N(0, 1) in bf16 (projected, normalised activations have unit scale)."""
    return torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32).bfloat16()


def _int32(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.int32)).cuda()


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    hq, hkv, d = case["hq"], case["hkv"], case["d"]
    st = {"case": dict(case)}
    if case["path"] in ("fwd", "train"):
        h = _dialogues(case)
        st["segs"] = ops.Segments.from_host(h.cu_seqlens, h.cu_segs, h.seg_is_query)
        T = h.total
        st["q"], st["k"], st["v"] = (_normal(gen, T, n, d) for n in (hq, hkv, hkv))
        if case["path"] == "train":
            st["dout"] = _normal(gen, T, hq, d)
        return st
    cached, new = _cache_lengths(case)
    B, Tn = case["dialogues"], int(new.sum())
    # capacity as a serving program would set it: room for the new segment
    # and some answer tokens, in whole pages
    need = int((cached + new).max()) + 64
    page = case["page"]
    st["lens"], st["cu"] = _int32(cached), _int32(np.concatenate([[0], np.cumsum(new)]))
    st["max_new"], st["max_len"] = int(new.max()), int((cached + new).max())
    if page:
        mp = -(-need // page)
        pages = B * mp + 8
        # the dialogues' pages lie scattered over the pool
        order = np.random.default_rng([case["layout"], int(seed)]).permutation(pages)
        st["table"] = _int32(order[:B * mp].reshape(B, mp))
        shape = (pages, hkv, page, d)
    else:
        shape = (B, hkv, -(-need // 256) * 256, d)
    st["k_cache"] = torch.empty(shape, device="cuda", dtype=torch.bfloat16)
    st["v_cache"] = torch.empty(shape, device="cuda", dtype=torch.bfloat16)
    for t in (st["k_cache"], st["v_cache"]):
        for i in range(0, shape[0], 64):
            t[i:i + 64] = _normal(gen, *t[i:i + 64].shape)
    rows = (B,) if case["path"] == "decode" else (Tn,)
    st["q"], st["k"], st["v"] = (_normal(gen, *rows, n, d) for n in (hq, hkv, hkv))
    if case["rope"]:
        # the new segment's index in its dialogue, and the offset inside it
        turns = np.random.default_rng(case["layout"]).integers(1, 40, size=B)
        st["pos1"] = _int32(np.repeat(turns, new))
        st["pos2"] = _int32(np.concatenate([np.arange(n) for n in new]))
    return st


def run(state):
    s, c = state, state["case"]
    if c["path"] == "fwd":
        return ops.fwd(s["q"], s["k"], s["v"], s["segs"])
    if c["path"] == "train":
        o, lse = ops.fwd(s["q"], s["k"], s["v"], s["segs"])
        dq, dk, dv = ops.bwd(s["q"], s["k"], s["v"], o, lse, s["dout"], s["segs"])
        return o, lse, dq, dk, dv
    qkv = s["q"], s["k"], s["v"], s["k_cache"], s["v_cache"]
    if c["path"] == "decode":
        if c["page"]:
            o, lse = ops.decode_paged(*qkv, s["table"], s["lens"], max_seqlen=s["max_len"])
        else:
            o, lse = ops.decode(*qkv, s["lens"], max_seqlen=s["max_len"])
    elif c["page"]:
        o, lse = ops.prefill_paged(*qkv, s["table"], s["lens"], s["cu"], s["max_new"],
                                   seg_is_query=not c["answer"])
    elif c["rope"]:
        o, lse = ops.prefill_cached_rope2d(*qkv, s["lens"], s["cu"], s["max_new"], s["pos1"],
                                           s["pos2"], seg_is_query=not c["answer"])
    elif c["answer"]:
        o, lse = ops.prefill_cached_segment(*qkv, s["lens"], s["cu"], s["max_new"], False)
    else:
        o, lse = ops.prefill_cached(*qkv, s["lens"], s["cu"], s["max_new"])
    return o, lse, s["k_cache"], s["v_cache"]


def tolerance(case):
    # bf16 operands and results with fp32 sums: the probabilities and the
    # score gradients are rounded to bf16 before their products (2^-9 each),
    # o is rounded to bf16, and the backward takes that o. Against exact(),
    # over the listed cases and 30 drawn ones: rel up to 2.4e-3 (o; gradients
    # 1.8e-3), max up to 0.1 (dQ, dV of rows that see few keys, whose values
    # are many times the tensor's root mean square). About four times that:
    return {"rel": 1e-2, "max": 0.4}


# --------------------------------------------------------------------------
# The same in 64 bits, in plain torch
# --------------------------------------------------------------------------

def _attend(q, k, v, last):
    """q [n, d], k and v [m, d] in float64; row r sees keys 0 .. last[r].
    Returns (o, lse, p)."""
    s = (q @ k.t().contiguous()) * (1.0 / math.sqrt(q.shape[1]))
    s.masked_fill_(torch.arange(k.shape[0], device=q.device)[None, :] > last[:, None], -math.inf)
    lse = torch.logsumexp(s, 1)
    p = s.sub_(lse[:, None]).exp_()
    return p @ v, lse, p


def _exact_packed(case, st):
    h = _dialogues(case)
    lim = torch.from_numpy(_lim(h)).cuda()
    hq, hkv, d = case["hq"], case["hkv"], case["d"]
    T, train = h.total, case["path"] == "train"
    new = lambda *s: torch.zeros(s, dtype=torch.float64, device="cuda")  # noqa: E731
    o, lse = new(T, hq, d), new(hq, T)
    dq, dk, dv = (new(T, n, d) for n in (hq, hkv, hkv)) if train else (None,) * 3
    sc = 1.0 / math.sqrt(d)
    for b in range(h.batch):
        a, e = int(h.cu_seqlens[b]), int(h.cu_seqlens[b + 1])
        last = lim[a:e] - a
        for i in range(hq):
            g = i // (hq // hkv)
            q, k, v = (st[n][a:e, j].double().contiguous() for n, j in
                       (("q", i), ("k", g), ("v", g)))
            oo, ll, p = _attend(q, k, v, last)
            o[a:e, i], lse[i, a:e] = oo, ll
            if train:
                do = st["dout"][a:e, i].double().contiguous()
                dp = do @ v.t().contiguous()
                ds = dp.sub_((do * oo).sum(1)[:, None]).mul_(p)
                dv[a:e, g] += p.t().contiguous() @ do
                dq[a:e, i] = (ds @ k) * sc
                dk[a:e, g] += (ds.t().contiguous() @ q) * sc
    return (o, lse, dq, dk, dv) if train else (o, lse)


def _rotate(x, pos1, pos2):
    """2-D rotary positions of x [n, heads, d] in float64: the first half of
    the head by pos1, the second by pos2, pairs (j, j + d/4) of a half at
    angle pos * 10000^(-4 j / d)."""
    n, _, d = x.shape
    j = torch.arange(d // 4, device=x.device, dtype=torch.float64)
    freq = 10000.0 ** (-4.0 * j / d)
    out = []
    for half, pos in ((x[..., :d // 2], pos1), (x[..., d // 2:], pos2)):
        ang = pos.double()[:, None, None] * freq
        a, b = half[..., :d // 4], half[..., d // 4:]
        out += [a * ang.cos() - b * ang.sin(), a * ang.sin() + b * ang.cos()]
    return torch.cat(out, -1)


def exact(case, seed):
    st = prepare(case, seed)
    if case["path"] in ("fwd", "train"):
        return _exact_packed(case, st)
    hq, hkv, d, page = case["hq"], case["hkv"], case["d"], case["page"]
    cached, new = _cache_lengths(case)
    q, k, v = (st[n].double() for n in ("q", "k", "v"))
    if case["rope"]:
        q, k = (_rotate(x, st["pos1"], st["pos2"]) for x in (q, k))
        # the cache holds the rotated keys in bf16, and attention reads them
        # from there; rotated queries are bf16 as well
        q, k = q.bfloat16().double(), k.bfloat16().double()
    Tn = q.shape[0]
    o = torch.zeros((Tn, hq, d), dtype=torch.float64, device="cuda")
    lse = torch.zeros((hq, Tn), dtype=torch.float64, device="cuda")
    r0 = 0
    for b in range(case["dialogues"]):
        C, L = int(cached[b]), int(new[b])
        rows = slice(r0, r0 + L)
        r0 += L
        for src, name in ((k, "k_cache"), (v, "v_cache")):  # append the new rows
            x = src[rows].bfloat16()
            for t in range(L):
                if page:
                    st[name][int(st["table"][b, (C + t) // page]), :, (C + t) % page] = x[t]
                else:
                    st[name][b, :, C + t] = x[t]
        kk, vv = (st[n][st["table"][b].long()].transpose(0, 1).reshape(hkv, -1, d) if page
                  else st[n][b] for n in ("k_cache", "v_cache"))
        last = torch.full((L,), C + L - 1, device="cuda")
        if case["answer"]:
            last = C + torch.arange(L, device="cuda")
        for i in range(hkv):
            kd, vd = (x[i, :C + L].double().contiguous() for x in (kk, vv))
            for j in range(i * (hq // hkv), (i + 1) * (hq // hkv)):
                oo, ll, _ = _attend(q[rows, j].contiguous(), kd, vd, last)
                o[rows, j], lse[j, rows] = oo, ll
    # a rotated key lies on a rounding boundary now and then: no exact value
    k_cache = None if case["rope"] else st["k_cache"]
    return o, lse, k_cache, st["v_cache"]
