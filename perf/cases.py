"""The calls a serving program makes into this library, as measurable cases.

A case is one call (or, where K and V are separate calls, the two) of a
public entry point on one layer, with the pool, the page tables and the
buffers such a program keeps.  `listed` holds one case per direction of the
path (decode, verify, prefill, append, reconstruct; both stored formats) and,
for decode and prefill, several sizes; `draw` gives more of the same ranges.

Keys of a case:
  op          step       append one row per request, then attend (one launch)
              verify     2-4 causal query tokens per request over the cache
              prefill    a chunk of rows over a cached prefix, one request
              append     quantize rows of K and V into affine 4-bit pages
              tq4_append encode rows of K and of V into TQ4 pages
              tq4_decode single-query decode over TQ4 pages
              reconstruct  pages of a group of KV heads back to fp16 operands
  hq, hkv, d, group   heads, head size, elements per (scale, bias)
  positions   cached positions of the longest request, the step's included
  shortest    of the shortest one (the others lie evenly between)
  batch, shared   requests; positions of the prefix they share
  rows, prefix    new rows (append, prefill); positions before them
  queries     query tokens per request (verify)
  heads       KV heads of the group (reconstruct)
  tq4         the pages hold TQ4 vectors (reconstruct)
"""
import math

import torch

from paper_2609_17475_amd import jfkv

PAGE = 256    # positions per page
SPLITS = 64   # split cap of the decode calls
DEV = "cuda"
TD = 256      # head size of the TQ4 format

# 16-level minimum-distortion quantizer of a unit Gaussian (Max 1960, table I),
# the shape of the TQ4 codebook; coordinates of a rotated unit vector of 256
# elements have a standard deviation of 1 / 16.
_MAX16 = (0.1284, 0.3881, 0.6568, 0.9424, 1.256, 1.618, 2.069, 2.733)


def listed():
    wide = dict(hq=32, hkv=8, d=128, group=64)    # the 32/8-head geometry of the workloads
    paper = dict(hq=24, hkv=4, d=256)             # the paper's geometry (24/4 heads, d = 256)
    one = dict(batch=1, shared=0)
    return [
        # the smallest call: one decode step of a small model's layer over a
        # short context, where the launch and the latency chain count
        dict(name="step_4k", op="step", hq=4, hkv=1, d=128, group=64, positions=4097,
             shortest=4097, **one),
        # an ordinary decode step: part of the way through a 32K + 6K session
        dict(name="step_32k", op="step", positions=35841, shortest=35841, **wide, **one),
        # the headline: a decode step at the full 256K window
        dict(name="step_256k", op="step", positions=262145, shortest=262145, **wide, **one),
        # two long requests that share a 32K system prompt, batched
        dict(name="step_ragged_2", op="step", positions=196609, shortest=131073, batch=2,
             shared=32768, **wide),
        # speculative decoding: two proposed tokens and the bonus position
        dict(name="verify_256k", op="verify", positions=262144, shortest=262144, queries=3,
             **wide, **one),
        # a full prefill chunk deep into a long prompt
        dict(name="prefill_2k_64k", op="prefill", rows=2048, prefix=65536, **wide),
        # the paper's prefill probe: a 256-row chunk over a 192K history
        dict(name="prefill_256_192k", op="prefill", rows=256, prefix=196608, group=64, **paper),
        # a chat turn: a new message of 1,000 tokens after 7,000 cached ones
        dict(name="prefill_1k_7k", op="prefill", rows=1000, prefix=7000, **wide),
        # building the full-window cache from floating K and V
        dict(name="append_256k", op="append", rows=262143, prefix=0, batch=1, **wide),
        # the same in the paper's own format
        dict(name="tq4_append_256k", op="tq4_append", rows=262143, prefix=0, batch=1, hkv=4),
        # the paper's decode at its full native window
        dict(name="tq4_decode_256k", op="tq4_decode", positions=262144, shortest=262144, hq=24,
             hkv=4, **one),
        # operands of a two-head group for an SDPA-style prefill, 192K history
        dict(name="reconstruct_tq4_192k", op="reconstruct", tq4=True, positions=196608, heads=2,
             hkv=4, d=256, group=64),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    op = rng.choice(("step", "step", "verify", "prefill", "prefill", "append", "tq4_append",
                     "tq4_decode", "reconstruct"))
    hq, hkv, d, group = rng.choice(((32, 8, 128, 64), (32, 8, 128, 32), (16, 4, 128, 128),
                                    (4, 1, 128, 64), (24, 4, 256, 64), (16, 2, 64, 32)))
    case = dict(op=op)
    if op in ("step", "verify", "tq4_decode"):
        batch = rng.choice((1, 1, 2, 3, 8)) if op == "step" else rng.choice((1, 1, 2))
        positions = log_int(300, 250000 // batch)
        shortest = positions if batch == 1 else rng.randint(positions // 4, positions)
        shared = PAGE * rng.randint(0, (shortest - 64) // PAGE // 2) if batch > 1 and shortest > 64 else 0
        case.update(positions=positions, shortest=shortest, batch=batch, shared=shared)
        if op == "tq4_decode":
            case.update(hq=rng.choice((24, 16, 32)), hkv=4)
        else:
            case.update(hq=hq, hkv=hkv, d=d, group=group)
        if op == "verify":
            case.update(queries=rng.choice((2, 3, 4)))
    elif op == "prefill":
        rows = log_int(20, 2048)
        prefix = rng.choice((0, log_int(100, 30000), log_int(100, 60000)))
        prefix = min(prefix, 300_000_000_000 // (rows * hq * d))  # no costlier than those listed
        case.update(hq=hq, hkv=hkv, d=d, group=group, rows=rows, prefix=prefix)
    elif op in ("append", "tq4_append"):
        batch = rng.choice((1, 1, 2, 4))
        case.update(rows=max(batch, log_int(1, 200000)), prefix=rng.randint(0, 3000), batch=batch)
        if op == "append":
            case.update(hkv=hkv, d=d, group=group)
        else:
            case.update(hkv=rng.choice((4, 4, 2)))
    else:
        tq4 = rng.choice((True, False))
        case.update(tq4=tq4, positions=log_int(1000, 196608))
        if tq4:
            case.update(heads=rng.choice((1, 2, 4)), hkv=4, d=256, group=64)
        else:
            case.update(heads=min(2, hkv), hkv=hkv, d=d, group=group)
    return case


# ---------------------------------------------------------------- inputs
def _gen(seed, part):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed * 16 + part)
    return g


def _rows(seed, part, n, heads, d):
    """fp16 [n][heads][d]: unit Gaussian with 2 % outlier channels eight times
    as large (fixed across positions), as key and value activations have."""
    g = _gen(seed, part)
    x = torch.randn((n, heads, d), generator=g, device=DEV, dtype=torch.float32)
    n_out = max(1, round(0.02 * d))
    for h in range(heads):
        x[:, h, torch.randperm(d, generator=g, device=DEV)[:n_out]] *= 8.0
    return x.to(torch.float16)


def _queries(seed, part, *shape):
    x = torch.randn(shape, generator=_gen(seed, part), device=DEV, dtype=torch.float32)
    return (x / math.sqrt(shape[-1])).to(torch.float16)


def _lens(case):
    b, hi, lo = case["batch"], case["positions"], case["shortest"]
    return [hi if i == 0 else hi - (hi - lo) * i // (b - 1) for i in range(b)]


def _tables(seed, lens, shared):
    """Page tables of requests with `lens` positions whose first `shared` (a
    multiple of the page size) lie in the same pages; page IDs are a seeded
    permutation of a pool with a few pages to spare."""
    need = [-(-n // PAGE) for n in lens]
    sp = shared // PAGE
    total = sp + sum(n - sp for n in need) + 8
    g = torch.Generator()
    g.manual_seed(seed * 16 + 15)
    perm = torch.randperm(total, generator=g, dtype=torch.int32)
    t = torch.full((len(lens), max(need)), -1, dtype=torch.int32)
    at = sp
    for b, n in enumerate(need):
        t[b, :sp] = perm[:sp]
        t[b, sp:n] = perm[at:at + n - sp]
        at += n - sp
    return t.to(DEV), total


def _i32(v):
    return torch.tensor(v, dtype=torch.int32, device=DEV)


def _cache_rows(lens, shared):
    """How the rows of a cache are drawn: the shared prefix once, then each
    request's own rows; (rows in all, [(first row, start position, rows)])."""
    runs, at = [], shared
    for n in lens:
        runs.append((at, shared, n - shared))
        at += n - shared
    return at, runs


def _fill(write, k, v, lens, shared, tables):
    """Writes a cache drawn by _cache_rows: write(rows of k, of v, cu, start, tables)."""
    _, runs = _cache_rows(lens, shared)
    if shared:
        write(k[:shared], v[:shared], _i32([0, shared]), _i32([0]), tables[:1])
    cu = [0]
    for _, _, n in runs:
        cu.append(cu[-1] + n)
    write(k[shared:], v[shared:], _i32(cu), _i32([s for _, s, _ in runs]), tables)


def _signs(seed, part):
    return (torch.randint(0, 2, (TD,), generator=_gen(seed, part), device=DEV) * 2 - 1).float()


def _centroids():
    return torch.tensor([-c / 16 for c in reversed(_MAX16)] + [c / 16 for c in _MAX16],
                        dtype=torch.float32, device=DEV)


def _append_split(case):
    """Rows of each request of an append (all of `rows`, nearly even)."""
    b, n = case["batch"], case["rows"]
    return [n * (i + 1) // b - n * i // b for i in range(b)]


def prepare(case, seed):
    op = case["op"]
    s = {"case": case}
    if op in ("step", "verify"):
        lens = _lens(case)
        hq, hkv, d = case["hq"], case["hkv"], case["d"]
        tables, pages = _tables(seed, lens, case["shared"])
        pool = jfkv.KVPool(jfkv.layout(PAGE, hkv, d, case["group"], pages), fill=0)
        n, _ = _cache_rows(lens, case["shared"])
        k, v = _rows(seed, 0, n, hkv, d), _rows(seed, 1, n, hkv, d)
        _fill(lambda *a: jfkv.jf_kv_quantize_append(pool, *a), k, v, lens, case["shared"], tables)
        B, sq = case["batch"], case.get("queries", 1)
        ws = torch.zeros(jfkv.jf_decode_workspace_bytes(B, hq * sq, d, SPLITS), dtype=torch.uint8,
                         device=DEV)
        if op == "step":
            q = _queries(seed, 2, B, hq, d)
            out = torch.empty_like(q)
            kn, vn = _rows(seed, 3, B, hkv, d), _rows(seed, 4, B, hkv, d)
            s["call"] = jfkv.bind_decode_step(pool, kn, vn, q, tables, _i32(lens), 1.0, SPLITS, ws,
                                              out)
            # the step writes its row into the pool
            s["out"] = [out, pool.k_codes, pool.k_meta, pool.v_codes, pool.v_meta]
        else:
            q = _queries(seed, 2, B, sq, hq, d)
            out = torch.empty_like(q)
            s["call"] = jfkv.bind_verify(pool, q, tables, _i32(lens), 1.0, SPLITS, ws, out)
            s["out"] = [out]
    elif op == "prefill":
        hq, hkv, d, T, p0 = (case[k] for k in ("hq", "hkv", "d", "rows", "prefix"))
        tables, pages = _tables(seed, [p0 + T], 0)
        s["pool"] = pool = jfkv.KVPool(jfkv.layout(PAGE, hkv, d, case["group"], pages), fill=0)
        if p0:
            k, v = _rows(seed, 0, p0, hkv, d), _rows(seed, 1, p0, hkv, d)
            _fill(lambda *a: jfkv.jf_kv_quantize_append(pool, *a), k, v, [p0], 0, tables)
        s["q"] = _queries(seed, 2, T, hq, d)
        s["k"], s["v"] = _rows(seed, 3, T, hkv, d), _rows(seed, 4, T, hkv, d)
        s["table"], s["out"] = tables[0], torch.empty_like(s["q"])
    elif op in ("append", "tq4_append"):
        rows = _append_split(case)
        p0 = case["prefix"]
        s["tables"], pages = _tables(seed, [p0 + n for n in rows], 0)
        hkv = case["hkv"]
        d = case["d"] if op == "append" else TD
        s["k"], s["v"] = (_rows(seed, part, case["rows"], hkv, d) for part in (0, 1))
        cu = [0]
        for n in rows:
            cu.append(cu[-1] + n)
        s["cu"], s["start"] = _i32(cu), _i32([p0] * len(rows))
        if op == "append":
            s["pool"] = jfkv.KVPool(jfkv.layout(PAGE, hkv, d, case["group"], pages), fill=0)
        else:
            lay = jfkv.layout(PAGE, hkv, TD, 64, pages)
            s["pools"] = [jfkv.TQ4Pool(lay, fill=0) for _ in range(2)]
            s["signs"], s["cents"] = [_signs(seed, 5), _signs(seed, 6)], _centroids()
    elif op == "tq4_decode" or case["tq4"]:
        lens = _lens(case) if op == "tq4_decode" else [case["positions"]]
        shared = case.get("shared", 0)
        hkv = case["hkv"]
        tables, pages = _tables(seed, lens, shared)
        lay = jfkv.layout(PAGE, hkv, TD, 64, pages)
        kp, vp = (jfkv.TQ4Pool(lay, fill=0) for _ in range(2))
        ks, vs, cents = _signs(seed, 5), _signs(seed, 6), _centroids()
        n, _ = _cache_rows(lens, shared)

        def write(kr, vr, cu, start, tb):
            jfkv.jf_tq4_encode_append(kp, kr, ks, cents, cu, start, tb)
            jfkv.jf_tq4_encode_append(vp, vr, vs, cents, cu, start, tb)

        _fill(write, _rows(seed, 0, n, hkv, TD), _rows(seed, 1, n, hkv, TD), lens, shared, tables)
        if op == "tq4_decode":
            q = _queries(seed, 2, len(lens), case["hq"], TD)
            out = torch.empty_like(q)
            ws = torch.zeros(jfkv.jf_decode_workspace_bytes(len(lens), case["hq"], TD, SPLITS),
                             dtype=torch.uint8, device=DEV)
            s["call"] = jfkv.bind_tq4_decode(kp, vp, ks, vs, cents, q, tables, _i32(lens), 1.0,
                                             SPLITS, ws, out)
            s["out"] = [out]
        else:
            s["pools"], s["signs"], s["cents"], s["table"] = (kp, vp), (ks, vs), cents, tables[0]
            s["out"] = [torch.empty((case["heads"], lens[0], TD), dtype=torch.float16, device=DEV)
                        for _ in range(2)]
    else:
        n, hkv, d = case["positions"], case["hkv"], case["d"]
        tables, pages = _tables(seed, [n], 0)
        s["pool"] = pool = jfkv.KVPool(jfkv.layout(PAGE, hkv, d, case["group"], pages), fill=0)
        _fill(lambda *a: jfkv.jf_kv_quantize_append(pool, *a), _rows(seed, 0, n, hkv, d),
              _rows(seed, 1, n, hkv, d), [n], 0, tables)
        s["table"] = tables[0]
        s["out"] = [torch.empty((case["heads"], n, d), dtype=torch.float16, device=DEV)
                    for _ in range(2)]
    return s


def run(s):
    case = s["case"]
    op = case["op"]
    if "call" in s:  # decode loops keep their calls bound, the arguments marshalled once
        s["call"]()
        return s["out"]
    if op == "prefill":
        jfkv.jf_prefill_attn_q4(s["pool"], s["q"], s["k"], s["v"], s["table"], case["prefix"], 1.0,
                                s["out"])
        return [s["out"]]
    if op == "append":
        p = s["pool"]
        jfkv.jf_kv_quantize_append(p, s["k"], s["v"], s["cu"], s["start"], s["tables"])
        return [p.k_codes, p.k_meta, p.v_codes, p.v_meta]
    if op == "tq4_append":
        for p, x, sg in zip(s["pools"], (s["k"], s["v"]), s["signs"]):
            jfkv.jf_tq4_encode_append(p, x, sg, s["cents"], s["cu"], s["start"], s["tables"])
        return [t for p in s["pools"] for t in (p.words, p.norms)]
    if case["tq4"]:
        jfkv.jf_tq4_reconstruct(*s["pools"], *s["signs"], s["cents"], s["table"],
                                case["positions"], 0, case["heads"], *s["out"])
    else:
        jfkv.jf_reconstruct_q4(s["pool"], s["table"], case["positions"], 0, case["heads"],
                               *s["out"])
    return s["out"]


def work(case):
    op = case["op"]
    vec_tq4 = TD // 2 + 2
    if op in ("step", "verify", "tq4_decode"):
        lens = _lens(case)
        d = case.get("d", TD)
        vec = vec_tq4 if op == "tq4_decode" else d // 2 + 4 * d // case["group"]
        unique = sum(lens) - case["shared"] * (case["batch"] - 1)
        sq = case.get("queries", 1)
        nbytes = 2 * case["hkv"] * unique * vec + 4 * len(lens) * sq * case["hq"] * d
        if op == "step":
            nbytes += len(lens) * 2 * case["hkv"] * 2 * d
        return {"bytes": nbytes, "flops": 4 * d * case["hq"] * sq * sum(lens)}
    if op == "prefill":
        T, p0, d, hq, hkv = (case[k] for k in ("rows", "prefix", "d", "hq", "hkv"))
        vec = d // 2 + 4 * d // case["group"]
        return {"bytes": 2 * hkv * p0 * vec + 4 * T * (hq + hkv) * d,
                "flops": 4 * d * hq * (T * p0 + T * (T + 1) // 2)}
    if op == "append":
        d = case["d"]
        vecs = 2 * case["rows"] * case["hkv"]
        return {"bytes": vecs * (2 * d + d // 2 + 4 * d // case["group"]), "flops": 4 * vecs * d}
    if op == "tq4_append":  # 8 butterfly stages, the norm, the scaling
        vecs = 2 * case["rows"] * case["hkv"]
        return {"bytes": vecs * (2 * TD + vec_tq4), "flops": vecs * TD * 11}
    d = case["d"]
    vecs = 2 * case["positions"] * case["heads"]
    if case["tq4"]:
        return {"bytes": vecs * (2 * d + vec_tq4), "flops": vecs * d * 9}
    return {"bytes": vecs * (2 * d + d // 2 + 4 * d // case["group"]), "flops": 2 * vecs * d}


def tolerance(case):
    op = case["op"]
    # codes, scales, biases, indices, norms and the correctly rounded affine
    # operands are fixed to the bit by the formats' contracts
    if op in ("append", "tq4_append") or (op == "reconstruct" and not case["tq4"]):
        return "exact"
    # fp16 results of fp32 sums; probabilities enter the products as fp16.
    # About four times the distance from 64 bits that each path shows.
    return {"rel": {"step": 1.6e-3, "verify": 1.6e-3, "prefill": 1.2e-3, "tq4_decode": 2e-3,
                    "reconstruct": 8e-4}[op]}


# ------------------------------------------------- the same in 64 bits, plain torch
def _affine(x, group):
    """Scale, bias (fp32, fp16 values) and the stored values in 64 bits of rows
    x [n][d] under the affine 4-bit format."""
    n, d = x.shape
    g = x.float().reshape(n, d // group, group)
    bias, top = g.amin(2, keepdim=True), g.amax(2, keepdim=True)
    step = ((top - bias).double() / 15.0).float()  # (a float tensor / 15.0 is a product by 1 / 15)
    h = step.half()
    bits = h.view(torch.int16)
    h = torch.where(h.float() < step, (bits + 1).view(torch.float16), h).float()
    code = torch.where(h > 0, torch.round(((g - bias).double() / h.clamp_min(1e-30)).float()).clamp(0, 15),
                       torch.zeros_like(g))
    return h[..., 0], bias[..., 0], (h.double() * code.double() + bias.double()).reshape(n, d)


def _hadamard():
    m = torch.ones((1, 1), dtype=torch.float64, device=DEV)
    while m.shape[0] < TD:
        m = torch.cat([torch.cat([m, m], 1), torch.cat([m, -m], 1)], 0)
    return m


def _tq4(x, signs, cents):
    """The TQ4 format's stored values of rows x [n][256], in 64 bits."""
    x = x.double()
    h = _hadamard()
    rho = x.square().sum(1, keepdim=True).sqrt()
    y = (x * signs.double()) @ h / (16 * rho).clamp_min(1e-300)
    z = torch.bucketize(y, ((cents[:-1] + cents[1:]) * 0.5).double())
    return rho.float().half().double() * signs.double() * (cents.double()[z] @ h) / 16


def _attend(q, k, v, first_hidden):
    """Softmax attention in 64 bits of q [m][d] over k, v [n][d]; query i sees
    the positions below first_hidden[i]."""
    s = q.double() @ k.t()
    s.masked_fill_(torch.arange(k.shape[0], device=DEV)[None] >= first_hidden[:, None],
                   -float("inf"))
    return torch.softmax(s, 1) @ v


def exact(case, seed):
    op = case["op"]
    if op in ("step", "verify", "tq4_decode"):
        lens, shared, hq, hkv = _lens(case), case["shared"], case["hq"], case["hkv"]
        d, sq, B, gq = case.get("d", TD), case.get("queries", 1), case["batch"], case["hq"] // case["hkv"]
        n, runs = _cache_rows(lens, shared)
        k, v = _rows(seed, 0, n, hkv, d), _rows(seed, 1, n, hkv, d)
        if op == "tq4_decode":
            cents = _centroids()
            store = [lambda x, sg=_signs(seed, p): _tq4(x, sg, cents) for p in (5, 6)]
        else:
            store = [lambda x: _affine(x, case["group"])[2]] * 2
        if op == "step":
            for x, part in ((k, 3), (v, 4)):
                new = _rows(seed, part, B, hkv, d)
                for b, (at, _, m) in enumerate(runs):
                    x[at + m - 1] = new[b]
        q = _queries(seed, 2, B, sq, hq, d) if op == "verify" else _queries(seed, 2, B, hq, d).view(B, 1, hq, d)
        out = torch.empty((B, sq, hq, d), dtype=torch.float64, device=DEV)
        for h in range(hkv):
            kh, vh = store[0](k[:, h]), store[1](v[:, h])
            for b, (at, _, m) in enumerate(runs):
                kb, vb = (torch.cat([x[:shared], x[at:at + m]]) for x in (kh, vh))
                for t in range(sq):
                    sl = slice(h * gq, (h + 1) * gq)
                    lim = torch.full((gq,), lens[b] - sq + 1 + t, device=DEV)
                    out[b, t, sl] = _attend(q[b, t, sl], kb, vb, lim)
        if op == "verify":
            return [out]
        return [out.view(B, hq, d)] + [None] * (4 if op == "step" else 0)
    if op == "prefill":
        hq, hkv, d, T, p0 = (case[k] for k in ("hq", "hkv", "d", "rows", "prefix"))
        gq = hq // hkv
        q = _queries(seed, 2, T, hq, d)
        kv = [[_rows(seed, part, p0, hkv, d) if p0 else None, _rows(seed, part + 3, T, hkv, d)]
              for part in (0, 1)]
        out = torch.empty((T, hq, d), dtype=torch.float64, device=DEV)
        lim = p0 + 1 + torch.arange(T, device=DEV)
        for h in range(hkv):
            # the chunk's own rows are attended as they are, the prefix as it is stored
            k, v = (torch.cat(([] if old is None else [_affine(old[:, h], case["group"])[2]])
                              + [new[:, h].double()]) for old, new in kv)
            for i in range(h * gq, (h + 1) * gq):
                out[:, i] = _attend(q[:, i], k, v, lim)
        return [out]
    if op in ("append", "tq4_append"):
        # codes and indices are whole numbers; the (scale, bias) words and the
        # norms in 64 bits, at the places of their positions
        rows, p0, hkv = _append_split(case), case["prefix"], case["hkv"]
        tables, pages = _tables(seed, [p0 + n for n in rows], 0)
        pos = torch.cat([p0 + torch.arange(n, device=DEV) for n in rows])
        req = torch.cat([torch.full((n,), b, device=DEV) for b, n in enumerate(rows)])
        page = tables[req, pos // PAGE].long()
        res = []
        for part in (0, 1):
            if op == "tq4_append":
                norms = torch.zeros((pages, hkv, PAGE), dtype=torch.float64, device=DEV)
                x = _rows(seed, part, case["rows"], hkv, TD)
                for h in range(hkv):
                    norms[page, h, pos % PAGE] = x[:, h].double().square().sum(1).sqrt()
                res += [None, norms]
            else:
                d, group = case["d"], case["group"]
                meta = torch.zeros((pages, hkv, PAGE, d // group, 2), dtype=torch.float64,
                                   device=DEV)
                x = _rows(seed, part, case["rows"], hkv, d)
                for h in range(hkv):
                    g = x[:, h].double().reshape(-1, d // group, group)
                    lo, hi = g.amin(2), g.amax(2)
                    meta[page, h, pos % PAGE] = torch.stack([(hi - lo) / 15, lo], 2)
                res += [None, meta.reshape(-1)]
        return res
    n, hkv, d = case["positions"], case["hkv"], case["d"]
    res = []
    for part in (0, 1):
        x = _rows(seed, part, n, hkv, d)
        if case["tq4"]:
            sg, cents = _signs(seed, 5 + part), _centroids()
            res.append(torch.stack([_tq4(x[:, h], sg, cents) for h in range(case["heads"])]))
        else:
            res.append(torch.stack([_affine(x[:, h], case["group"])[2]
                                    for h in range(case["heads"])]))
    return res
