"""The performance cases of the graded KV-cache path: what a serving program has it do.

Six kinds of work, each through the calls a program makes (``GradedCache``,
``LayerCaches`` and the observer functions of ``binding``):

* ``decode``: one layer's dense decode step over a graded cache, with the options it is
  served with (exact residual rows, values grouped per token, sequences of different
  lengths, the attention error certificate);
* ``quest``: one layer's Compressed-Quest decode step, page selection and sparse read;
* ``encode``: the prefill encode of one layer's cache (keys, values, page boxes);
* ``residual``: the prefill selection of the exact residual rows;
* ``observe``: the prefill attention-mass observer and the level allocation from it;
* ``serve``: a small model's decode loop, sequences admitted one after the other, every
  layer's append and ladder demotions in one call per step, every layer's attention,
  and the sequences retired at the end.

Keys and values are normal fp16 rows, four key channels of each (sequence, KV head) ten
times larger (outlier channels); queries are normal; the attention mass of the residual
selection is heavy-tailed.
"""
import math

import numpy as np
import torch

from paper_2608_23599_amd import binding as gkv

P, D = 64, 128
EXACT, INT8, INT4, INT2, CENTROID, MEAN = 16, 8, 4, 2, 1, 0
HEADS = ((8, 2), (32, 8), (28, 4), (40, 8), (16, 1), (6, 6))  # (query heads, KV heads)
MAX_UNIT_TOKENS = 8 * 4 * 131072  # tokens of all (sequence, KV head) units of the largest batch


# ---------------------------------------------------------------- the cases
def _decode(batch, heads, kv_heads, tokens, ladder="graded", residual=0, per_token=False, ragged=False,
            certificate=False, **more):
    return dict(kind="decode", batch=batch, heads=heads, kv_heads=kv_heads, tokens=tokens, ladder=ladder,
                residual=residual, per_token=per_token, ragged=ragged, certificate=certificate, **more)


def _quest(batch, heads, kv_heads, tokens, page, topk, residual=0, **more):
    return dict(kind="quest", batch=batch, heads=heads, kv_heads=kv_heads, tokens=tokens, ladder="graded",
                page=page, topk=topk, residual=residual, **more)


def _encode(batch, kv_heads, tokens, ladder, page, per_token=False, **more):
    return dict(kind="encode", batch=batch, heads=kv_heads, kv_heads=kv_heads, tokens=tokens, ladder=ladder,
                page=page, per_token=per_token, **more)


def _residual(batch, kv_heads, tokens, ladder, residual, per_token=False, **more):
    return dict(kind="residual", batch=batch, heads=kv_heads, kv_heads=kv_heads, tokens=tokens, ladder=ladder,
                residual=residual, per_token=per_token, **more)


def _observe(batch, heads, kv_heads, tokens, observed, **more):
    return dict(kind="observe", batch=batch, heads=heads, kv_heads=kv_heads, tokens=tokens, observed=observed, **more)


def _serve(layers, batch, heads, kv_heads, steps, stagger, **more):
    return dict(kind="serve", layers=layers, batch=batch, heads=heads, kv_heads=kv_heads, steps=steps,
                stagger=stagger, ladder="tiny", **more)


def listed():
    return [
        # the smallest call: one short conversation of a small model, where launches and latency count
        _decode(1, 8, 2, 2048, "tiny", name="dense 2k"),
        # one long-document conversation of an 8B-shaped model
        _decode(1, 32, 8, 16384, name="dense 16k"),
        # the headline: a batch of 128k contexts of a 7B-shaped model, 2% exact residual rows
        _decode(8, 28, 4, 131072, residual=20, name="dense 128k residual"),
        # a running batch of sequences of different lengths, values grouped per token
        _decode(6, 28, 4, 20011, per_token=True, ragged=True, name="dense ragged per token"),
        # the low-rate configuration: one-centroid base and 10.2% exact residual rows
        _decode(4, 28, 4, 50021, "rdv2", residual=102, name="dense low rate"),
        # sparse decode, one 32k conversation
        _quest(1, 32, 8, 32768, 16, 128, name="quest 32k"),
        # sparse decode, a batch of 128k contexts
        _quest(8, 32, 8, 131072, 16, 128, name="quest 128k batch"),
        # sparse decode, one million-token context
        _quest(1, 32, 8, 1048576, 16, 256, name="quest 1m"),
        # prefill of one 128k prompt: encode the layer's cache and its page boxes
        _encode(1, 8, 131072, "graded", 16, name="encode 128k"),
        # prefill of the headline batch: choose the exact residual rows
        _residual(8, 4, 131072, "graded", 20, name="residual 128k"),
        # prefill of one 128k prompt: attention mass of the last 64 queries, levels from it
        _observe(1, 28, 4, 131072, 64, name="observe 128k"),
        # the decode loop of a small served model, from admission to retirement
        _serve(4, 4, 28, 4, 896, 48, name="serve 4 layers"),
    ]


def _log(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(("decode", "decode", "decode", "quest", "quest", "encode", "residual", "observe", "serve"))
    heads, kv = rng.choice(HEADS)
    batch = rng.choice((1, 1, 2, 3, 4, 6, 8))
    most = MAX_UNIT_TOKENS // (batch * kv)
    if kind == "decode":
        tokens = _log(rng, 300, min(131072, most))
        ladder = rng.choice(("graded", "graded", "tiny", "rdv2"))
        ragged = batch > 1 and rng.random() < 0.4
        residual = 102 if ladder == "rdv2" else rng.choice((0, 20))
        return _decode(batch, heads, kv, tokens, ladder, 0 if ragged else residual, rng.random() < 0.3, ragged,
                       rng.random() < 0.2)
    if kind == "quest":
        tokens = _log(rng, 3000, min(1048576, most))
        return _quest(batch, heads, kv, tokens, rng.choice((16, 16, 32, 64)), _log(rng, 16, 256),
                      20 if tokens < 131072 and rng.random() < 0.25 else 0)
    if kind == "encode":
        return _encode(batch, kv, _log(rng, 500, min(131072, 8 * 131072 // (batch * kv))),
                       rng.choice(("graded", "graded", "tiny", "rdv2")), rng.choice((0, 16, 32, 64)),
                       rng.random() < 0.3)
    if kind == "residual":
        ladder = rng.choice(("graded", "graded", "rdv2"))
        return _residual(batch, kv, _log(rng, 1500, min(131072, most)), ladder, 102 if ladder == "rdv2" else 20,
                         rng.random() < 0.3)
    if kind == "observe":
        return _observe(batch, heads, kv, _log(rng, 500, min(131072, 4 * 131072 // (batch * kv))),
                        rng.choice((8, 16, 24, 32)))
    return _serve(rng.choice((1, 2, 3, 4)), min(batch, 4), heads, kv, _log(rng, 100, 896), rng.randrange(1, 64))


# ---------------------------------------------------------------- inputs
def _levels(ladder, tokens):
    """Levels of the age ladders by block, oldest first."""
    n = -(-tokens // P)
    age = np.arange(n)[::-1]
    if ladder == "tiny":
        lv = np.select([age < 4, age < 12, age < 24], [EXACT, INT8, INT4], INT2)
    elif ladder == "rdv2":
        lv = np.where(age < 16, EXACT, MEAN)
    else:
        rest = max(0, n - 16)
        lv = np.select([age < 16 + 25 * rest // 100, age < 16 + 60 * rest // 100], [INT8, INT4], INT2)
        lv = np.where(np.arange(n) < 10 * n // 100, CENTROID, lv)
        lv = np.where(age < 16, EXACT, lv)
    return lv.astype(np.int8)


def _generator(seed, *more):
    g = torch.Generator(device="cuda")
    g.manual_seed(hash((int(seed),) + tuple(int(m) for m in more)) % (1 << 62))
    return g


def _normal(g, *shape):
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32)


def _kv(case, seed):
    """Keys and values [batch][kv_heads][tokens][128] fp16."""
    B, H, T = case["batch"], case["kv_heads"], case["tokens"]
    k = torch.empty((B, H, T, D), dtype=torch.float16, device="cuda")
    v = torch.empty_like(k)
    for b in range(B):
        g = _generator(seed, 1, b)
        gain = torch.ones((H, 1, D), device="cuda")
        for h in range(H):
            gain[h, 0, torch.randperm(D, generator=g, device="cuda")[:4]] = 10.0
        k[b] = _normal(g, H, T, D) * gain
        v[b] = _normal(g, H, T, D)
    return k, v


def _queries(case, seed, *lead):
    shape = (*lead, case["heads"], D) if lead else (case["batch"], case["heads"], D)
    return _normal(_generator(seed, 2), *shape).half()


def _mass(case, seed):
    m = torch.exp(3.0 * _normal(_generator(seed, 3), case["batch"], case["kv_heads"], case["tokens"]))
    return m / m.sum(-1, keepdim=True)


def _lengths(case, seed):
    """Sequence lengths of a ragged batch; the first is the longest."""
    g = torch.Generator().manual_seed(int(seed) + 4)
    x = torch.rand(case["batch"], generator=g).tolist()
    lens = [max(1, int(case["tokens"] * (0.15 + 0.85 * f))) for f in x]
    lens[0] = case["tokens"]
    return lens


def _kept(case):
    return case["tokens"] * case.get("residual", 0) // 1000


def _level_table(case, lens):
    """[batch][kv_heads][blocks] levels, each sequence by the ladder at its own length."""
    n = -(-case["tokens"] // P)
    lv = np.full((case["batch"], case["kv_heads"], n), EXACT, np.int8)
    for b, t in enumerate(lens):
        own = _levels(case["ladder"], t)
        lv[b, :, :len(own)] = own
    return lv


def _build(case, seed, k, v):
    lens = _lengths(case, seed) if case.get("ragged") else None
    lv = _level_table(case, lens or [case["tokens"]] * case["batch"])
    return gkv.GradedCache.build(k.view(torch.int16), v.view(torch.int16), Hq=case["heads"], levels=lv,
                                 page=case.get("page", 0), nres_cap=_kept(case),
                                 v_per_token=case.get("per_token", False), seq_lens=lens)


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case}
    if kind == "serve":
        L, B, H, n = case["layers"], case["batch"], case["kv_heads"], case["steps"]
        blocks = -(-n // P)
        slots = {lv: 2 * B * H * (blocks + 1) for lv in (EXACT, INT8, INT4, INT2)}
        s["layers"] = [gkv.GradedCache(B, H, case["heads"], 0, blocks + 1, slots, seq_lens=[-1] * B)
                       for _ in range(L)]
        s["service"] = gkv.LayerCaches(s["layers"], case["ladder"])
        g = _generator(seed, 1)
        s["k"] = _normal(g, n, L, B, H, D).half().view(torch.int16)
        s["v"] = _normal(g, n, L, B, H, D).half().view(torch.int16)
        s["q"] = _queries(case, seed, n, L, B).view(torch.int16)
        s["out"] = torch.zeros((n, L, B, case["heads"], D), dtype=torch.float32, device="cuda")
        return s
    k, v = _kv(case, seed)
    if kind == "observe":
        s["k"] = k.view(torch.int16)
        s["q"] = _queries(case, seed, case["batch"], case["observed"]).view(torch.int16)
        return s
    s["cache"] = cache = _build(case, seed, k, v)
    if kind in ("encode", "residual"):
        s["k"], s["v"] = k.view(torch.int16), v.view(torch.int16)
    if kind == "encode":  # the run encodes into a cache whose slots are laid out
        cache.arena.zero_()
        cache.cert.zero_()
        if cache.boxes is not None:
            cache.boxes.zero_()
        return s
    if kind == "residual":
        s["mass"] = _mass(case, seed)
        return s
    if _kept(case):
        cache.rd_residual_select(k.view(torch.int16), v.view(torch.int16), _mass(case, seed), _kept(case))
    s["q"] = _queries(case, seed).view(torch.int16)
    return s


# ---------------------------------------------------------------- one pass
def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "serve":
        return _serve_pass(s)
    if kind == "observe":
        mass = gkv.observe_mass(s["q"], s["k"])
        norms = gkv.query_norms(s["q"], case["kv_heads"])
        levels = gkv.allocate_levels(s["k"], mass, norms, 1.0, 1e-3, 16)
        return {"mass": mass, "norms": norms, "levels": levels}
    cache = s["cache"]
    if kind == "decode":
        if case["certificate"]:
            out, bound = cache.decode_bound(s["q"])
            return {"out": out, "bound": bound}
        return {"out": cache.decode(s["q"])}
    if kind == "quest":
        pages = cache.quest_select(s["q"], case["topk"])
        return {"pages": pages, "out": cache.graded_decode_attn(s["q"], pages)}
    if kind == "encode":
        n = -(-case["tokens"] // P)
        cache.quantize_block(gkv.KEYS, s["k"], 0, n)
        cache.quantize_block(gkv.VALUES, s["v"], 0, n)
        out = {"records": cache.arena, "certificate": cache.cert}
        if case["page"]:
            cache.page_boxes(s["k"], 0, case["tokens"] // case["page"])
            out["boxes"] = cache.boxes
        return out
    cache.rd_residual_select(s["k"], s["v"], s["mass"], _kept(case))
    return {"tokens": cache.res_idx, "rows": cache.res_rows, "mask": cache.res_mask, "before": cache.res_off}


def _serve_pass(s):
    case, layers, service = s["case"], s["layers"], s["service"]
    k, v, q, out = s["k"], s["v"], s["q"], s["out"]
    for t in range(case["steps"]):
        if t % case["stagger"] == 0 and t // case["stagger"] < case["batch"]:
            for c in layers:
                c.admit(t // case["stagger"])
        service.step(k[t], v[t])
        for i, c in enumerate(layers):
            c.decode(q[t, i], out=out[t, i])
    for c in layers:
        for b in np.nonzero(c.lengths() >= 0)[0]:
            c.retire(int(b))
    return {"out": out}


# ---------------------------------------------------------------- the work of one pass
_BLOCK_BYTES = {EXACT: 16384, INT8: 512 + 8192, INT4: 512 + 4096, INT2: 512 + 2048, CENTROID: 1040, MEAN: 256}


def _record_bytes(case, lens):
    """Bytes of one KV head's key and value records, over the batch."""
    return sum(2 * _BLOCK_BYTES[int(x)] for t in lens for x in _levels(case["ladder"], t))


def work(case):
    B, H, Hq = case["batch"], case["kv_heads"], case["heads"]
    if case["kind"] == "serve":
        bytes_ = flops = 0
        for t in range(case["steps"]):
            lens = [t + 1 - b * case["stagger"] for b in range(B) if t >= b * case["stagger"]]
            bytes_ += H * (_record_bytes(case, lens) + 2 * 2 * D * 2 * len(lens)) + Hq * D * 6 * len(lens)
            flops += 4 * Hq * D * sum(lens)
        return {"bytes": bytes_ * case["layers"], "flops": flops * case["layers"]}
    T = case["tokens"]
    u = B * H
    io = B * Hq * D * (2 + 4)  # query in, output out
    if case["kind"] == "decode":
        # the mean length of a ragged batch stands for its sequences
        lens = [T] + [int(T * 0.575)] * (B - 1) if case["ragged"] else [T] * B
        rows = _kept(case)
        read = H * _record_bytes(case, lens) + u * rows * (2 * D * 2 + 4)
        return {"bytes": read + io, "flops": 4 * Hq * D * sum(lens)}
    if case["kind"] == "quest":
        pages = (T - 1) // case["page"]
        tokens = (min(case["topk"], pages) + 1) * case["page"]
        read = u * (pages * 4 * D + _record_bytes(case, [T]) * tokens // T)
        return {"bytes": read + io, "flops": B * Hq * D * (2 * pages + 4 * tokens)}
    if case["kind"] == "encode":
        boxes = T // case["page"] * 4 * D if case["page"] else 0
        return {"bytes": u * (2 * T * D * 2 + _record_bytes(case, [T]) + boxes), "flops": 8 * u * 2 * T * D}
    if case["kind"] == "residual":
        kept = _kept(case)
        read = T * D * 2 + T * 4 + _record_bytes(case, [T]) // 2 + kept * 2 * D * 2
        return {"bytes": u * (read + kept * (2 * D * 2 + 4) + T // 8), "flops": 5 * u * T * D}
    rows = case["observed"] * (Hq // H)
    return {"bytes": u * T * D * 2 + B * case["observed"] * Hq * D * 2 + u * (T // P) * 5,
            "flops": 2 * u * rows * T * D}


def tolerance(case):
    """About four times the error against 64 bits that was measured over the cases."""
    if case["kind"] in ("decode", "quest", "serve"):
        # probabilities enter the value product in fp16: 0.9e-4 to 2.3e-4, with the values'
        # scales multiplied into them (groups per token) 3.8e-4; the pages are exact
        return {"rel": 1.6e-3 if case.get("per_token") else 8e-4}
    if case["kind"] == "encode":
        return {"rel": 2e-7, "max": 5e-7}  # fp64 row errors rounded up to fp32 (0.5e-7); the records are bytes
    if case["kind"] == "residual":
        return "exact"
    # fp32 sums (1.2e-7); a level flips where its threshold lies within that of a block's value
    return {"rel": 1e-6, "differ": 5e-4}


# ---------------------------------------------------------------- the same in 64 bits
def _f16(x):
    """fp64 rounded once to fp16 (by way of fp32 rounded to odd), as fp64."""
    f = x.float()
    w = f.double()
    i = f.view(torch.int32)
    i = torch.where(w.abs() > x.abs(), i - 1, i)  # towards zero
    i = torch.where(i.view(torch.float32).double() != x, i | 1, i)
    return i.view(torch.float32).half().double()


def _lloyd(x, k):
    """x: [n][64][128]; the deterministic k-means of a centroid block, reconstructed."""
    if k == 1:
        return _f16(x.mean(1, keepdim=True)).expand_as(x)
    c = x[:, ::P // k].clone()

    def nearest(c):
        return torch.stack([(x - c[:, j:j + 1]).square().sum(-1) for j in range(k)], -1).argmin(-1)

    for _ in range(10):
        hot = torch.nn.functional.one_hot(nearest(c), k).double()  # [n][64][k]
        count = hot.sum(1)[..., None]
        c = torch.where(count > 0, hot.transpose(1, 2).contiguous() @ x / count.clamp(min=1), c)
    c = _f16(c)
    a = nearest(c)
    return torch.gather(c, 1, a[..., None].expand(-1, -1, D))


def _scalar(x, bits, axis):
    top = (1 << bits) - 1
    z, hi = x.amin(axis, keepdim=True), x.amax(axis, keepdim=True)
    s = _f16((hi - z) / top)
    z = _f16(z)
    code = torch.where(s > 0, torch.round((x - z) / torch.where(s > 0, s, 1.0)).clamp(0, top), 0.0)
    return code * s + z


def _rebuilt(x, levels, per_token=False):
    """x: [blocks][64][128] fp64; every block as its level stores it."""
    y = x.clone()
    levels = torch.as_tensor(np.ascontiguousarray(levels).astype(np.int64), device=x.device)
    for lv in (INT8, INT4, INT2, CENTROID, MEAN):
        at = torch.nonzero(levels == lv)[:, 0]
        for part in at.split(512):
            if len(part):
                b = x[part]
                y[part] = _lloyd(b, 4) if lv == CENTROID else _lloyd(b, 1) if lv == MEAN else _scalar(
                    b, lv, 2 if per_token else 1)
    return y


def _blocks(rows):
    """[T][128] as fp64 blocks, the last one filled with zeros."""
    n = -(-rows.shape[0] // P)
    x = torch.zeros((n * P, D), dtype=torch.float64, device=rows.device)
    x[:rows.shape[0]] = rows.double()
    return x.view(n, P, D)


def _chosen(case, mass, v, vr):
    """Mask of the residual tokens: the largest mass x squared value error, lower token first."""
    score = mass.double() * (v - vr).square().sum(-1)
    mask = torch.zeros(score.shape[0], dtype=torch.bool, device=v.device)
    mask[torch.sort(score, descending=True, stable=True).indices[:_kept(case)]] = True
    return mask


def _attend(q, k, v):
    a = torch.softmax(q @ k.transpose(0, 1).contiguous() / math.sqrt(D), -1)
    return a, a @ v


def exact(case, seed):
    kind = case["kind"]
    if kind == "residual":
        return None  # whole numbers and copied rows
    if kind == "serve":
        return {"out": _serve_exact(case, seed)}
    B, H, T = case["batch"], case["kv_heads"], case["tokens"]
    G = case["heads"] // H
    k, v = _kv(case, seed)
    if kind == "observe":
        q = _queries(case, seed, B, case["observed"]).double()
        n, blocks = case["observed"], -(-T // P)
        mass = torch.zeros((B, H, blocks), dtype=torch.float64, device="cuda")
        hidden = torch.arange(T, device="cuda")[None, :] > (T - n + torch.arange(n, device="cuda"))[:, None]
        for b in range(B):
            for h in range(H):
                kt = k[b, h].double().transpose(0, 1).contiguous()
                for g in range(G):
                    x = (q[b, :, h * G + g].contiguous() @ kt / math.sqrt(D)).masked_fill_(hidden, -math.inf)
                    w = torch.nn.functional.pad(torch.softmax(x, -1).sum(0), (0, blocks * P - T))
                    mass[b, h] += w.view(blocks, P).sum(-1) / (G * n)
        norms = q.square().sum(-1).sqrt().amax(1).view(B, H, G).amax(-1)
        return {"mass": mass, "norms": norms, "levels": None}
    lens = _lengths(case, seed) if case.get("ragged") else [T] * B
    per_token = case.get("per_token", False)
    if kind == "encode":
        lv = _levels(case["ladder"], T)
        cert = torch.zeros((B, H, len(lv), 4), dtype=torch.float64, device="cuda")
        for b in range(B):
            for h in range(H):
                cert[b, h] = _certificate(_blocks(k[b, h]), _blocks(v[b, h]), lv, per_token)
        return {"records": None, "certificate": cert, "boxes": None}
    q = _queries(case, seed).double()
    mass = _mass(case, seed) if _kept(case) else None
    out = torch.zeros((B, case["heads"], D), dtype=torch.float64, device="cuda")
    if kind == "quest":
        for b in range(B):
            for h in range(H):
                qs = q[b, h * G:(h + 1) * G].contiguous()
                out[b, h * G:(h + 1) * G] = _quest_exact(case, qs, k[b, h], v[b, h],
                                                         None if mass is None else mass[b, h])
        return {"pages": None, "out": out}
    bound = torch.zeros((B, case["heads"]), dtype=torch.float64, device="cuda")
    for b, t in enumerate(lens):
        lv = _levels(case["ladder"], t)
        for h in range(H):
            kb, vb = _blocks(k[b, h, :t]), _blocks(v[b, h, :t])
            kr, vr = _rebuilt(kb, lv).view(-1, D)[:t], _rebuilt(vb, lv, per_token).view(-1, D)[:t]
            kept = None
            if mass is not None:
                kept = _chosen(case, mass[b, h], vb.view(-1, D)[:t], vr)
                kr = torch.where(kept[:, None], kb.view(-1, D)[:t], kr)
                vr = torch.where(kept[:, None], vb.view(-1, D)[:t], vr)
            qs = q[b, h * G:(h + 1) * G].contiguous()
            a, out[b, h * G:(h + 1) * G] = _attend(qs, kr, vr)
            if case["certificate"]:
                bound[b, h * G:(h + 1) * G] = _bound(qs, a, kept, _certificate(kb, vb, lv, per_token))
    return {"out": out, "bound": bound} if case["certificate"] else {"out": out}


def _certificate(kb, vb, lv, per_token):
    """Per block: the largest key and value row error and the largest value row norm."""
    ke = (kb - _rebuilt(kb, lv)).norm(dim=-1).amax(-1)
    ve = (vb - _rebuilt(vb, lv, per_token)).norm(dim=-1).amax(-1)
    return torch.stack([ke, ve, vb.norm(dim=-1).amax(-1), torch.zeros_like(ke)], -1)


def _bound(q, a, kept, cert):
    """The attention error certificate of every head; residual rows count as exact."""
    n = cert.shape[0]
    exact_mass = torch.zeros(a.shape[0], dtype=torch.float64, device=a.device)
    if kept is not None:
        exact_mass = (a * kept).sum(-1)
        a = a * ~kept
    ab = torch.nn.functional.pad(a, (0, n * P - a.shape[1])).view(a.shape[0], n, P).sum(-1)
    eps = q.norm(dim=-1, keepdim=True) * cert[:, 0] / math.sqrt(D)
    up, down = (ab * eps.exp()).sum(-1) + exact_mass, (ab * (-eps).exp()).sum(-1) + exact_mass
    return (ab * cert[:, 1]).sum(-1) + (up / down - down / up).clamp(max=2.0) * cert[:, 2].amax()


def _quest_exact(case, q, k, v, mass):
    """One (sequence, KV head): the selected pages' rows and the current page's."""
    T, page = case["tokens"], case["page"]
    cur = (T - 1) // page
    lv = _levels(case["ladder"], T)
    rows = k[:cur * page].view(cur, page, D)
    lo, hi = rows.amin(1).float(), rows.amax(1).float()
    score = None
    for g in range(q.shape[0]):  # the bound is a 32-bit sum in channel order
        acc = torch.zeros(cur, device="cuda")
        for d, x in enumerate(q[g].tolist()):
            acc = acc + x * (hi if x >= 0 else lo)[:, d]
        score = acc if score is None else torch.maximum(score, acc)
    pages = torch.sort(score, descending=True, stable=True).indices[:case["topk"]]
    pages = torch.cat([pages.sort().values, torch.tensor([cur], device="cuda")])
    tok = (pages[:, None] * page + torch.arange(page, device="cuda")).view(-1)
    tok = tok[tok < T]
    if mass is not None:
        kb, vb = _blocks(k), _blocks(v)
        kr, vr = _rebuilt(kb, lv).view(-1, D)[:T], _rebuilt(vb, lv).view(-1, D)[:T]
        kept = _chosen(case, mass, vb.view(-1, D)[:T], vr)[:, None]
        kr, vr = torch.where(kept, kb.view(-1, D)[:T], kr)[tok], torch.where(kept, vb.view(-1, D)[:T], vr)[tok]
        return _attend(q, kr, vr)[1]
    blk, where = torch.unique(tok // P, return_inverse=True)  # only the touched blocks
    at = (blk[:, None] * P + torch.arange(P, device="cuda")).clamp(max=T - 1).view(-1)
    own = lv[blk.cpu().numpy()]
    kr = _rebuilt(k[at].double().view(-1, P, D), own)
    vr = _rebuilt(v[at].double().view(-1, P, D), own)
    return _attend(q, kr[where, tok % P], vr[where, tok % P])[1]


def _serve_exact(case, seed):
    L, B, H, n = case["layers"], case["batch"], case["kv_heads"], case["steps"]
    G = case["heads"] // H
    g = _generator(seed, 1)
    k = _normal(g, n, L, B, H, D).half().double()
    v = _normal(g, n, L, B, H, D).half().double()
    q = _queries(case, seed, n, L, B).double().view(n, L, B, H, G, D)
    out = torch.zeros((n, L, B, H, G, D), dtype=torch.float64, device="cuda")
    chain = (EXACT, INT8, INT4, INT2)  # a block steps down one level at a time
    for b in range(B):
        first = b * case["stagger"]
        t = n - first
        if t <= 0:
            continue
        blocks = -(-t // P)
        both = []
        for x in (k, v):
            rows = torch.zeros((L, H, blocks * P, D), dtype=torch.float64, device="cuda")
            rows[:, :, :t] = x[first:, :, b].permute(1, 2, 0, 3)
            x = rows.view(-1, P, D)
            steps = [x]
            for bits in chain[1:]:
                x = _scalar(x, bits, 1)
                steps.append(x)
            both.append(torch.stack(steps).view(len(chain), L, H, blocks, P, D))
        at = torch.arange(blocks, device="cuda")
        for i in range(t):
            lv = torch.as_tensor([chain.index(int(x)) for x in _levels(case["ladder"], i + 1)], device="cuda")
            kr, vr = (x[lv, :, :, at[:len(lv)]].permute(1, 2, 0, 3, 4).reshape(L * H, -1, D)[:, :i + 1] for x in both)
            s = q[first + i, :, b].reshape(L * H, G, D) @ kr.transpose(1, 2).contiguous() / math.sqrt(D)
            out[first + i, :, b] = (torch.softmax(s, -1) @ vr.contiguous()).view(L, H, G, D)
    return out.view(n, L, B, case["heads"], D)
