"""Workloads over which the speed of the WnW library is watched, each through its public entry points.

A case is a dict of plain values.  `kind` says which call a pass makes:

* "step"      one wnw_decode_step in the middle of a generation (the context has its history, the
              queries move on by one generated token per pass);
* "open"      a whole request: wnw_init_cache, wnw_set_roles_device, the first generated tokens
              (wnw_append_kv + wnw_decode_step each), wnw_destroy;
* "prefill"   prefill scores of a prompt (wnw_prefill_scores, or its allocation-free variant);
* "hits"      calibration: voice-score hits of a sample's answer tokens (wnw_voice_hits);
* "sens"      calibration: key sensitivity of one answer token's gradients (wnw_key_sensitivity).

Shapes are those of the backbones in synth/configs.py (30 layers, 32 query / 8 KV heads; 36 layers,
16 / 2; one layer, 24 / 8) and of the configurations the tests run (overlapping chunks, per-head
retention, ragged lengths).  Everything is drawn on the device from the seed alone.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2608_22704_amd import wnw as W

D = 128
WARM = 4      # steps a "step" context has run before the first pass (eviction lag + one)
RING = 32     # queries of a "step" context; the passes walk them in a circle
FIRST = 3     # tokens an "open" pass generates
TOPIC = 64    # audio positions that share a topic direction

VOXTRAL = dict(layers=30, q_heads=32, kv_heads=8)
QWEN = dict(layers=36, q_heads=16, kv_heads=2)


def _step(name, shape, audio, text, chunk, budget_bp, **kw):
    c = dict(kind="step", batch=1, audio=audio, text=text, chunk=chunk, budget_bp=budget_bp, next_step=True,
             copy_engines=False, overlap=False, per_head=False, bf16_out=False, fast_drift=False)
    c.update(shape, **kw)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest cache (one layer, 40 s of audio), library defaults: launches and latency
        _step("step_tiny", dict(layers=1, q_heads=24, kv_heads=8), 1000, 64, 32, 2000, next_step=False),
        # ten minutes at 12.5 tokens/s on the 2-KV-head backbone, the paper's timing, default recall
        _step("step_qwen", QWEN, 7500, 256, 32, 2000),
        # ten minutes at 25 tokens/s, the paper's timing, copy-engine recall; attention that moves
        # slowly over the audio, so that little is recalled per token (the paper: 0.05 to 1.04 MB)
        _step("step_voxtral", VOXTRAL, 15000, 512, 64, 2000, copy_engines=True),
        # the same cache with queries that jump along the clip (the benchmark's recipe): a recall
        # of tens of MB per token, bound by the host link
        _step("step_voxtral_jumps", VOXTRAL, 15000, 512, 64, 2000, copy_engines=True, fast_drift=True),
        # the same cache with the library's defaults (selection serves its own step), bf16 output
        _step("step_voxtral_same", VOXTRAL, 15000, 512, 64, 2000, next_step=False, bf16_out=True),
        # a small batch, odd lengths, overlapping chunks, per-head retention (Eq. 1)
        _step("step_ragged_b3", VOXTRAL, 9377, 211, 100, 2000, batch=3, copy_engines=True, overlap=True, per_head=True),
        # an hour of audio at 25 tokens/s, 10 % budget: the longest context
        _step("step_hour", VOXTRAL, 90000, 1024, 128, 1000, copy_engines=True),
        # a request from its prefilled cache to its third token
        _step("open_voxtral", VOXTRAL, 15000, 512, 64, 2000, kind="open", copy_engines=True),
        # prefill scores of a ten-minute prompt with a long instruction
        dict(name="prefill_voxtral", kind="prefill", batch=1, audio=15000, text=512, static=False, **VOXTRAL),
        # a five-minute prompt with a short question, odd lengths, allocation-free entry point
        dict(name="prefill_qwen_ragged", kind="prefill", batch=1, audio=3607, text=147, static=True, **QWEN),
        # calibration on a ten-minute sample with a sentence of answer tokens
        dict(name="hits_voxtral", kind="hits", audio=15000, text=512, tokens=64, top_k=4, **VOXTRAL),
        # calibration: the gradients of one answer token (one backward pass)
        dict(name="sens_qwen", kind="sens", audio=7500, tokens=1, **QWEN),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ranges (lengths on a logarithmic scale, odd ones among them)."""
    kind = rng.choice(["step", "step", "step", "step", "open", "prefill", "prefill", "hits", "sens"])
    shape = dict(rng.choice([VOXTRAL, QWEN, dict(layers=rng.randint(1, 8), q_heads=24, kv_heads=8)]))
    heads = shape["layers"] * shape["kv_heads"]
    rows_max = 240 * 90000 // heads
    if kind in ("step", "open"):
        batch = rng.choice([1, 1, 2, 3, 4]) if kind == "step" else 1
        top = min(90000, rows_max // batch) if kind == "step" else min(15000, rows_max)
        audio = _log_int(rng, 600, max(601, top))
        chunk = rng.choice([32, 50, 64, 100, 128])
        next_step = rng.random() < 0.75
        overlap = rng.random() < 0.3
        budget = rng.choice([1000, 2000, 2500])
        # the default recall reads small segment blocks, the copy engines large ones
        block = (chunk // 2 if overlap else chunk) * 0.8 * 0.5 * heads * 2 * D * 2
        return _step("", shape, audio, rng.randint(16, 1024 if kind == "step" else 512), chunk, budget, kind=kind, batch=batch,
                     next_step=next_step, copy_engines=next_step and block >= 1 << 20, overlap=overlap,
                     per_head=rng.random() < 0.3, bf16_out=rng.random() < 0.3,
                     fast_drift=kind == "step" and rng.random() < 0.2)
    audio = _log_int(rng, 600, 15000)
    if kind == "prefill":
        return dict(kind=kind, batch=1, audio=audio, text=rng.randint(16, 512), static=rng.random() < 0.5, **shape)
    if kind == "hits":
        return dict(kind=kind, audio=audio, text=rng.randint(16, 512), tokens=_log_int(rng, 1, 64), top_k=rng.choice([4, 8]),
                    **shape)
    return dict(kind=kind, audio=audio, tokens=rng.choice([1, 1, 2]), **shape)


# ---- inputs ----------------------------------------------------------------------------------


def _rng(seed, tag):
    return torch.Generator(device="cuda").manual_seed((int(seed) * 64 + tag) % (1 << 62))


def _normal(g, *shape):
    return torch.randn(shape, generator=g, device="cuda")


def _roles(c, seed):
    """uint8 [L][H_kv]: 10 % anchors, 50 % tidal, the rest fixed (2 / 4 / 2 of a single layer's 8)."""
    n = c["layers"] * c["kv_heads"]
    a = max(2, round(0.1 * n))
    r = np.full(n, W.WNW_FIXED, np.uint8)
    perm = np.random.Generator(np.random.Philox(seed)).permutation(n)
    r[perm[:a]] = W.WNW_ANCHOR
    r[perm[a: a + round(0.5 * n)]] = W.WNW_TIDAL
    return r.reshape(c["layers"], c["kv_heads"])


def _importance(c, seed):
    if not c["per_head"]:
        return None
    return np.random.Generator(np.random.Philox(seed + 1)).random((c["layers"], c["kv_heads"]), dtype=np.float32)


LAMBDA = np.float32(0.4)


def _cache(c, seed, queries):
    """K, V bf16 [B][L][H_kv][T][d] and the queries bf16 [S][B][L][H_q][d] that attend to them.

    Keys: N(0, 1) plus a topic direction shared by TOPIC consecutive audio positions; the first 16
    are pushed towards the mean query (attention sink).  Queries: with fast drift, fresh noise plus
    twice the key of a position that jumps along the clip; else a direction that the head keeps, a
    little fresh noise, and a pull towards the topic at a position eight further on every step."""
    B, L, Hq, Hkv = c["batch"], c["layers"], c["q_heads"], c["kv_heads"]
    Ta, T, G = c["audio"], c["audio"] + c["text"], Hq // Hkv
    g = _rng(seed, 1)
    k = torch.empty((B, L, Hkv, T, D), dtype=torch.bfloat16, device="cuda")
    v = torch.empty_like(k)
    q = torch.empty((queries, B, L, Hq, D), dtype=torch.bfloat16, device="cuda")
    steps = np.arange(queries)
    host = np.random.Generator(np.random.Philox(seed + 2))
    nt = (Ta + TOPIC - 1) // TOPIC
    for b in range(B):
        if c["fast_drift"]:
            pos = np.minimum(steps * Ta // queries + host.integers(0, max(Ta // queries, 1), queries), Ta - 1)
        else:
            pos = (Ta // 3 + 8 * steps) % Ta
        pos = torch.from_numpy(pos).cuda()
        for l in range(L):
            kl = _normal(g, Hkv, T, D)
            topic = _normal(g, Hkv, nt, D)
            kl[:, :Ta] += topic.repeat_interleave(TOPIC, dim=1)[:, :Ta]
            kl *= math.sqrt(0.5)
            hold = _normal(g, Hkv, G, D)
            u = hold.mean(dim=1, keepdim=True)
            kl[:, : min(16, Ta)] += 3.0 * u / u.norm(dim=2, keepdim=True)
            z = _normal(g, queries, Hkv, G, D)
            if c["fast_drift"]:
                ql = z + 2.0 * kl[:, pos].transpose(0, 1).unsqueeze(2)
            else:
                ql = hold + 0.1 * z + 0.3 * topic[:, pos // TOPIC].transpose(0, 1).unsqueeze(2)
            k[b, l], v[b, l] = kl, _normal(g, Hkv, T, D)
            q[:, b, l] = ql.reshape(queries, Hq, D)
    return k, v, q


def _new_rows(c, seed):
    """The K and V rows of the tokens an "open" pass generates: bf16 [FIRST][B][L][H_kv][d] each."""
    g = _rng(seed, 2)
    shape = (FIRST, c["batch"], c["layers"], c["kv_heads"], D)
    return _normal(g, *shape).bfloat16(), _normal(g, *shape).bfloat16()


def _prefill(c, seed):
    return torch.rand((c["batch"], c["layers"], c["kv_heads"], c["audio"]), generator=_rng(seed, 3), device="cuda")


def _config(c):
    flags = 0
    for key, bit in (("next_step", W.WNW_F_SELECT_NEXT_STEP), ("copy_engines", W.WNW_F_RECALL_MEMCPY),
                     ("overlap", W.WNW_F_OVERLAP_CHUNKS), ("bf16_out", W.WNW_F_OUT_BF16)):
        flags |= bit if c[key] else 0
    return W.make_config(c["batch"], c["layers"], c["q_heads"], c["kv_heads"], c["audio"], c["text"], c["chunk"],
                         c["budget_bp"], flags=flags, max_new_tokens=FIRST if c["kind"] == "open" else 0)


class State:
    """What a program holds between calls; owns the library context, if there is one."""

    ctx = None

    def __init__(self, **kw):
        self.__dict__.update(kw)

    def __del__(self):
        if self.ctx is not None:
            W.wnw_destroy(self.ctx)


def _context(c, seed, k, v, scores):
    ctx = W.wnw_init_cache(_config(c), k, v)
    imp = _importance(c, seed)
    if imp is not None:
        W.wnw_set_retention(ctx, imp, float(LAMBDA))
    W.wnw_set_roles_device(ctx, _roles(c, seed), scores)
    return ctx


def _outputs(c, n_chunks, k):
    od = torch.bfloat16 if c["bf16_out"] else torch.float32
    B = c["batch"]
    return (torch.empty((B, c["layers"], c["q_heads"], D), dtype=od, device="cuda"),
            torch.empty((B, n_chunks), dtype=torch.float32, device="cuda"),
            torch.empty((B, k), dtype=torch.int32, device="cuda"))


def _chunks(c):
    """(segment length, segments, chunks, k) as include/wnw.h defines them."""
    cl = c["chunk"] // 2 if c["overlap"] else c["chunk"]
    nseg = -(-c["audio"] // cl)
    nchk = nseg - 1 if c["overlap"] and nseg >= 2 else nseg
    return cl, nseg, nchk, c["budget_bp"] * c["audio"] // (10000 * c["chunk"])


def prepare(c, seed):
    kind = c["kind"]
    if kind == "step":
        k, v, q = _cache(c, seed, RING)
        ctx = _context(c, seed, k, v, _prefill(c, seed))
        del k, v
        torch.cuda.empty_cache()
        s = State(kind=kind, ctx=ctx, q=list(q), at=0, outs=_outputs(c, *_chunks(c)[2:]))
        for _ in range(WARM):
            run(s)
        torch.cuda.synchronize()
        return s
    if kind == "open":
        k, v, q = _cache(c, seed, FIRST)
        kn, vn = _new_rows(c, seed)
        return State(kind=kind, c=c, seed=seed, k=k, v=v, q=list(q), kn=list(kn), vn=list(vn), scores=_prefill(c, seed),
                     outs=[_outputs(c, *_chunks(c)[2:]) for _ in range(FIRST)])
    if kind == "prefill":
        k, q = _prefill_inputs(c, seed)
        cfg = W.make_config(c["batch"], c["layers"], c["q_heads"], c["kv_heads"], c["audio"], c["text"], 64, 2000)
        ctx = W.wnw_init_cache(cfg, k, k)   # the scores read keys only
        p = torch.empty((c["batch"], c["layers"], c["kv_heads"], c["audio"]), device="cuda")
        return State(kind=kind, ctx=ctx, static=c["static"], k=k, q=q, p=p)
    if kind == "hits":
        g = _rng(seed, 4)
        L, Hq, Hkv, Ta, n = c["layers"], c["q_heads"], c["kv_heads"], c["audio"], c["tokens"]
        k = _normal(g, L, Hkv, Ta + c["text"], D).bfloat16()
        a = torch.randint(0, Ta - 12, (n,), generator=g, device="cuda", dtype=torch.int32)
        span = torch.stack([a, a + 12], dim=1).contiguous()
        # an answer token's queries lean towards a key of its aligned interval
        lean = k[:, :, (a + 4).long()].float().permute(2, 0, 1, 3).repeat_interleave(Hq // Hkv, dim=2)
        q = (_normal(g, n, L, Hq, D) + 0.7 * lean).bfloat16()
        return State(kind=kind, k=k, q=q, span=span, top_k=c["top_k"], audio=Ta,
                     hits=torch.empty((n, L, Hq), dtype=torch.int32, device="cuda"))
    grad = _sens_inputs(c, seed)
    return State(kind=kind, grad=grad, sens=torch.empty(grad.shape[:3], device="cuda"))


def _prefill_inputs(c, seed):
    g = _rng(seed, 5)
    B, L, Hq, Hkv, Tt = c["batch"], c["layers"], c["q_heads"], c["kv_heads"], c["text"]
    k = _normal(g, B, L, Hkv, c["audio"] + Tt, D).bfloat16()
    q = torch.empty((B, L, Hq, Tt, D), dtype=torch.bfloat16, device="cuda")
    for b in range(B):
        for l in range(L):
            # each text token leans towards the key of one audio position per q-head
            pos = torch.randint(0, c["audio"], (Hkv, Hq // Hkv * Tt, 1), generator=g, device="cuda")
            lean = k[b, l].gather(1, pos.expand(-1, -1, D)).reshape(Hq, Tt, D)
            q[b, l] = _normal(g, Hq, Tt, D) + 0.7 * lean.float()
    return k, q


def _sens_inputs(c, seed):
    g = _rng(seed, 6)
    shape = (c["tokens"], c["layers"], c["kv_heads"], c["audio"])
    # gradients: a scale per position over several orders of magnitude
    return _normal(g, *shape, D) * (1e-3 * torch.exp(_normal(g, *shape, 1)))


# ---- one pass --------------------------------------------------------------------------------


def run(s):
    if s.kind == "step":
        out, scores, selected = s.outs
        W.wnw_decode_step(s.ctx, s.q[s.at], out, scores, selected)
        s.at = (s.at + 1) % RING
        return s.outs
    if s.kind == "open":
        ctx = _context(s.c, s.seed, s.k, s.v, s.scores)
        try:
            for i in range(FIRST):
                W.wnw_append_kv(ctx, s.kn[i], s.vn[i])
                W.wnw_decode_step(ctx, s.q[i], *s.outs[i])
        finally:
            W.wnw_destroy(ctx)
        return s.outs
    if s.kind == "prefill":
        if s.static:
            W.wnw_prefill_scores_static(s.ctx, s.q, s.p)
        else:
            W.wnw_prefill_scores(s.ctx, s.q, s.p)
        return s.p
    if s.kind == "hits":
        W.wnw_voice_hits(s.k, s.q, s.span, s.top_k, s.audio, s.hits)
        return s.hits
    W.wnw_key_sensitivity(s.grad, s.sens)
    return s.sens


# ---- what a pass cannot do without -----------------------------------------------------------


def _rows(c):
    """Key rows a decode step reads (every sequence): anchors whole, kept rows and text of the others,
    and the complements of the k chunks selected last."""
    n = c["layers"] * c["kv_heads"]
    a = max(2, round(0.1 * n))
    tidal = round(0.5 * n)
    cl, nseg, _, k = _chunks(c)
    keep = c["audio"] * c["budget_bp"] // 10000     # per-head retention averages to the budget
    rows = a * (c["audio"] + c["text"]) + (n - a) * (keep + c["text"])
    rows += tidal * (min(k * c["chunk"], c["audio"]) * (10000 - c["budget_bp"]) // 10000)
    return rows * c["batch"]


def work(c):
    kind, L, Hq, Hkv = c["kind"], c["layers"], c["q_heads"], c["kv_heads"]
    G, Ta = Hq // Hkv, c["audio"]
    if kind in ("step", "open"):
        io = c["batch"] * L * Hq * D * (2 + (2 if c["bf16_out"] else 4))
        rows = _rows(c)
        w = {"bytes": rows * 2 * D * 2 + io, "flops": rows * G * 4 * D}
        if kind == "open":
            full = c["batch"] * L * Hkv * (Ta + c["text"]) * 2 * D * 2
            w = {"bytes": 2 * full + FIRST * w["bytes"], "flops": FIRST * w["flops"]}
        return w
    if kind == "prefill":
        B, Tt = c["batch"], c["text"]
        return {"bytes": B * L * (Hkv * (Ta + Tt) * D * 2 + Hq * Tt * D * 2 + Hkv * Ta * 4),
                "flops": B * L * Hq * Tt * (Ta + (Tt + 1) / 2) * 2 * D}
    if kind == "hits":
        n = c["tokens"]
        return {"bytes": L * Hkv * Ta * D * 2 + n * L * Hq * (D * 2 + 4), "flops": n * L * Hq * Ta * 2 * D}
    return {"bytes": c["tokens"] * L * Hkv * (Ta * D * 4 + 4), "flops": c["tokens"] * L * Hkv * Ta * 2 * D}


def tolerance(c):
    """About four times what the library's outputs differ by from exact()."""
    if c["kind"] == "hits":
        return "exact"    # whole numbers
    if c["kind"] == "prefill":
        return {"rel": 4e-6, "max": 1e-4}
    if c["kind"] == "sens":
        return {"rel": 2e-7, "max": 2e-6}
    if c["bf16_out"]:     # one rounding to bf16
        return {"rel": 7e-3, "max": 2e-2, "differ": 0.0}
    return {"rel": 1e-6, "max": 5e-5, "differ": 0.0}


# ---- the same in 64 bits ---------------------------------------------------------------------


def _keep_flags(c, seed, scores):
    """bool [B][L][H_kv][T_a]: per segment, the best positions by prefill score (ties: the lower)."""
    cl, nseg, _, _ = _chunks(c)
    Ta = c["audio"]
    pad = nseg * cl - Ta
    p = torch.nn.functional.pad(scores, (0, pad), value=-1.0).reshape(*scores.shape[:3], nseg, cl)
    rank = p.sort(dim=-1, descending=True, stable=True).indices.argsort(dim=-1)
    lens = torch.full((nseg,), cl, dtype=torch.int64)
    lens[-1] = cl - pad
    imp = _importance(c, seed)
    if imp is None:
        keep = (lens * c["budget_bp"] // 10000).expand(c["layers"], c["kv_heads"], nseg)
    else:
        r = np.minimum(imp.astype(np.float64) * np.float64(LAMBDA), 1.0)
        keep = torch.from_numpy(np.floor(r[..., None] * lens.numpy()).astype(np.int64))
    flags = rank < keep.cuda()[None, ..., None]
    return flags.reshape(*scores.shape[:3], nseg * cl)[..., :Ta]


def _exact_scores(c, k, q, roles, extra_k):
    """Chunk scores [B][n_chunks] of one step (Eq. 2 and the chunk mean), double."""
    cl, nseg, nchk, _ = _chunks(c)
    Ta, G = c["audio"], c["q_heads"] // c["kv_heads"]
    out = torch.zeros((c["batch"], nchk), dtype=torch.float64, device="cuda")
    lens = torch.full((nseg,), cl, dtype=torch.float64, device="cuda")
    lens[-1] = cl - (nseg * cl - Ta)
    for b in range(c["batch"]):
        mass = torch.zeros(nseg * cl, dtype=torch.float64, device="cuda")
        for l, h in zip(*np.nonzero(roles == W.WNW_ANCHOR)):
            kk = torch.cat([k[b, l, h], extra_k[:, b, l, h]]).double()
            x = q[b, l, h * G: (h + 1) * G].double() @ kk.T.contiguous() / math.sqrt(D)
            mass[:Ta] += x.softmax(dim=1)[:, :Ta].sum(dim=0)
        seg = mass.reshape(nseg, cl).sum(dim=1)
        if nchk < nseg:
            out[b] = (seg[:-1] + seg[1:]) / (lens[:-1] + lens[1:])
        else:
            out[b] = seg / lens
    return out


def _exact_out(c, k, v, q, roles, keep, resident, extra_k, extra_v):
    """Attention outputs [B][L][H_q][d] of one step, double; resident: bool [B][n_segments]."""
    cl, nseg, _, _ = _chunks(c)
    Ta, G = c["audio"], c["q_heads"] // c["kv_heads"]
    out = torch.empty((c["batch"], c["layers"], c["q_heads"], D), dtype=torch.float64, device="cuda")
    tail = torch.ones(c["text"] + extra_k.shape[0], dtype=torch.bool, device="cuda")
    for b in range(c["batch"]):
        res = resident[b].repeat_interleave(cl)[:Ta]
        for l in range(c["layers"]):
            for h in range(c["kv_heads"]):
                kk = torch.cat([k[b, l, h], extra_k[:, b, l, h]])
                vv = torch.cat([v[b, l, h], extra_v[:, b, l, h]])
                if roles[l, h] != W.WNW_ANCHOR:
                    on = keep[b, l, h]
                    at = torch.cat([on | res if roles[l, h] == W.WNW_TIDAL else on, tail]).nonzero().squeeze(1)
                    kk, vv = kk[at], vv[at]
                x = q[b, l, h * G: (h + 1) * G].double() @ kk.double().T.contiguous() / math.sqrt(D)
                out[b, l, h * G: (h + 1) * G] = x.softmax(dim=1) @ vv.double()
    return out


def _exact_steps(c, seed, first, last, queries):
    """(out, scores, selected) of the steps first .. last of a context that begins at step 0."""
    k, v, q = _cache(c, seed, queries)
    roles = _roles(c, seed)
    keep = _keep_flags(c, seed, _prefill(c, seed))
    _, nseg, nchk, top = _chunks(c)
    none = torch.empty((0, c["batch"], c["layers"], c["kv_heads"], D), device="cuda", dtype=k.dtype)
    kn, vn = _new_rows(c, seed) if c["kind"] == "open" else (none, none)
    picked, got = [], []
    for s in range(last + 1):
        ek, ev = kn[: s + 1], vn[: s + 1]
        scores = _exact_scores(c, k, q[s], roles, ek)
        order = scores.float().sort(dim=1, descending=True, stable=True).indices[:, :top]
        picked.append(order)
        if s < first:
            continue
        end = s if c["next_step"] else s + 1         # selections that serve step s: the lag's last three
        chunk = torch.zeros((c["batch"], nchk), dtype=torch.bool, device="cuda")
        for p in picked[max(0, end - 3): end]:
            chunk.scatter_(1, p, True)
        res = torch.zeros((c["batch"], nseg), dtype=torch.bool, device="cuda")
        res[:, :nchk] |= chunk
        if nchk < nseg:
            res[:, 1:] |= chunk
        got.append((_exact_out(c, k, v, q[s], roles, keep, res, ek, ev), scores, order.sort(dim=1).values.int()))
    return got


def exact(c, seed):
    kind = c["kind"]
    if kind == "step":
        return _exact_steps(c, seed, WARM, WARM, RING)[0]
    if kind == "open":
        return _exact_steps(c, seed, 0, FIRST - 1, FIRST)
    if kind == "prefill":
        k, q = _prefill_inputs(c, seed)
        B, L, Hq, Hkv, Ta, Tt = c["batch"], c["layers"], c["q_heads"], c["kv_heads"], c["audio"], c["text"]
        G = Hq // Hkv
        later = torch.ones((Tt, Tt), dtype=torch.bool, device="cuda").triu(1).repeat(G, 1)
        p = torch.empty((B, L, Hkv, Ta), dtype=torch.float64, device="cuda")
        for b in range(B):
            for l in range(L):
                for h in range(Hkv):
                    x = q[b, l, h * G: (h + 1) * G].reshape(G * Tt, D).double() @ k[b, l, h].double().T.contiguous()
                    x /= math.sqrt(D)
                    x[:, Ta:].masked_fill_(later, -math.inf)
                    p[b, l, h] = x.softmax(dim=1)[:, :Ta].sum(dim=0)
        return p
    if kind == "sens":
        return _sens_inputs(c, seed).double().norm(dim=-1).mean(dim=-1)
    return None     # hits: whole numbers
