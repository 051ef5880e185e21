"""The work whose speed on one MI355X is tracked, as calls of the public entry
points: KV-cache appends (decode steps and prefills), attention logits against
the quantized cache, and compression of rows (round trip, quantize then
dequantize, with and without the stage-2 residual sketch).

listed() names twelve cases; draw() gives further cases of the same ranges:
widths 64 to 512 (the attention head widths, plus odd ones for plain rows),
2 to 4 bits, fp16 and fp32 rows, the Full, Fast and 2-D rotations, ragged row
counts and sequence lengths, multi-head and grouped-query attention.

prepare() makes a case's inputs on the GPU from the seed alone, run() is one
pass, exact() the same outputs in 64 bits from plain torch.
"""
import math

import numpy as np
import torch

import paper_2603_28430_amd as iq

DEV = "cuda"
F16, F32 = torch.float16, torch.float32
NEG_INF = float("-inf")

# d: the width of the rows; sets: "head" (one rotation set per head) or "one"
_DEFAULTS = dict(variant="fast", d=128, bits=3, dtype="f16", sets="head", block_size=16, m=0, group=1)


def _case(name, op, **kw):
    c = dict(_DEFAULTS, op=op, **kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one decode step of 32 sequences: their new K and V rows into the cache
        _case("append_decode", "append", tokens=32, heads=32),
        # one decode step of a small batch, grouped-query heads: append the new
        # token's rows, then the logits of its queries over the whole context
        _case("decode_step_gqa", "decode_step", seqs=4, heads=8, group=4, ctx=1900, variant="full"),
        # logits of a large batch over long contexts, one query head per key head
        _case("scores_mha_long", "scores", seqs=8, heads=32, ctx=32768, ragged=False, own_buffer=True),
        # the same with grouped-query heads, ragged contexts and 4 bits
        _case("scores_gqa_ragged", "scores", seqs=16, heads=8, group=4, ctx=16384, ragged=True, own_buffer=False,
              bits=4, variant="full"),
        # logits corrected by the residual sketch
        _case("scores_sketch", "scores", seqs=4, heads=32, ctx=16384, ragged=False, own_buffer=True, m=128),
        # a prefill: 8 prompts of 4,096 tokens
        _case("append_prefill", "append", tokens=8 * 4096, heads=32),
        # the same, keys with their residual sketch
        _case("append_prefill_sketch", "append_sketch", tokens=8 * 4096, heads=32, m=128),
        # a prefill at a head width that is not a power of two
        _case("append_prefill_d96", "append", tokens=2 * 2048 + 37, heads=32, d=96, bits=4),
        # offline compression of a block of rows with the residual sketch
        _case("quantize_sketch", "quantize_sketch", n=1000003, sets="one", m=128, variant="full"),
        # the fused quantize -> dequantize of many fp16 rows
        _case("roundtrip_f16", "roundtrip", n=1048576, sets="one", variant="full"),
        # and of wide fp32 rows
        _case("roundtrip_f32_d512", "roundtrip", n=262147, sets="one", d=512, dtype="f32"),
        # compress rows of an odd width and restore them
        _case("restore_d90", "restore", n=300007, sets="one", d=90, bits=4),
    ]


HEAD_WIDTHS = (64, 80, 96, 128, 128, 192, 256)


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["append", "append", "decode_step", "scores", "scores", "scores", "append_sketch",
                     "quantize_sketch", "roundtrip", "restore"])
    kw = dict(variant=rng.choice(["full", "fast", "2d"]), bits=rng.choice([2, 3, 4]), dtype="f16")
    if op in ("append", "append_sketch"):
        d = rng.choice(HEAD_WIDTHS)
        heads = rng.choice([4, 8, 12, 32])
        tokens = _log_int(rng, 1, 2 ** 27 // (heads * d))
        kw.update(d=d, heads=heads, tokens=tokens, block_size=rng.choice([16, 32, 64]))
        if op == "append_sketch":
            kw.update(m=64 if d > 192 else rng.choice([64, 128]))
    elif op in ("scores", "decode_step"):
        d = rng.choice(HEAD_WIDTHS)
        heads, group = rng.choice([(8, 1), (32, 1), (8, 4), (4, 8), (16, 2), (8, 5), (2, 8)])
        if kw["bits"] == 3 and d >= 192:   # larger groups are past the stated limit of the call
            group = min(group, 4)
        seqs = rng.choice([1, 2, 4, 8, 13])
        top = 4096 if op == "decode_step" else 2 ** 29 // (heads * seqs * d)
        kw.update(d=d, heads=heads, group=group, seqs=seqs, ctx=_log_int(rng, 200, min(top, 60000)),
                  block_size=rng.choice([16, 32, 64]))
        if op == "scores":
            kw.update(ragged=rng.random() < 0.5, own_buffer=rng.random() < 0.5,
                      m=0 if rng.random() < 0.6 else 64 if d > 192 else rng.choice([64, 128]))
    elif op == "quantize_sketch":
        d = rng.choice(HEAD_WIDTHS)
        kw.update(d=d, n=_log_int(rng, 100, 2 ** 27 // d), sets="one", m=64 if d > 192 else rng.choice([64, 128]))
    else:
        d = rng.choice(HEAD_WIDTHS + (90, 100, 384, 512))
        kw.update(d=d, n=_log_int(rng, 100, 2 ** 27 // d), sets="one", dtype=rng.choice(["f16", "f16", "f32"]))
    return _case(None, op, **kw)


# ---- inputs ------------------------------------------------------------------------

_codebooks = {}


def codebook(bits, d):
    """Lloyd-Max levels of N(0, 1/d), ascending and symmetric (numpy, 64 bits)."""
    if bits not in _codebooks:
        h = 1 << (bits - 1)
        c = (np.arange(h) + 0.5) * (3.0 / h)
        for _ in range(2000):
            t = np.concatenate([[0.0], 0.5 * (c[1:] + c[:-1]), [40.0]])
            pdf = np.exp(-0.5 * t * t) / math.sqrt(2 * math.pi)
            cdf = np.array([0.5 * (1 + math.erf(v / math.sqrt(2))) for v in t])
            c = (pdf[:-1] - pdf[1:]) / (cdf[1:] - cdf[:-1])
        _codebooks[bits] = np.concatenate([-c[::-1], c])
    return _codebooks[bits] / math.sqrt(d)


def padded_width(variant, d):
    return 2 * ((d + 1) // 2) if variant == "2d" else 4 * ((d + 3) // 4)


def record_bytes(case):
    return (padded_width(case["variant"], case["d"]) * case["bits"] + 7) // 8


def n_sets(case):
    return case["heads"] if case["sets"] == "head" else 1


def draws(case, seed):
    """Raw rotation draws [sets][...]: quaternions N(0, I_4) or planar angles."""
    rng = np.random.default_rng([seed, 11])
    s, d = n_sets(case), case["d"]
    if case["variant"] == "2d":
        return rng.uniform(0, 2 * math.pi, (s, (d + 1) // 2))
    return rng.standard_normal((s, (d + 3) // 4, 8 if case["variant"] == "full" else 4))


def projection(case, seed):
    return np.random.default_rng([seed, 13]).standard_normal((case["m"], case["d"]))


def generator(seed, stream):
    return torch.Generator(device=DEV).manual_seed(int(seed) * 64 + stream)


def rows(case, shape, seed, stream):
    """Key-, value- or query-like rows: Gaussian directions, norms spread around
    sqrt(d) from row to row, a few channels several times larger than the rest."""
    g = generator(seed, stream)
    x = torch.randn(shape, generator=g, device=DEV, dtype=F32)
    boost = torch.ones(shape[-1], device=DEV)
    boost[torch.randint(0, shape[-1], (3,), generator=g, device=DEV)] = 4.0
    x *= boost * torch.exp(0.3 * torch.randn(shape[:-1] + (1,), generator=g, device=DEV))
    return x.to(F32 if case["dtype"] == "f32" else F16)


def pack(idx, bits):
    """Records [..., ceil(w b / 8)] uint8 of indices [..., w] uint8, least significant bit first."""
    b = (idx.unsqueeze(-1) >> torch.arange(bits, device=idx.device, dtype=torch.uint8)) & 1
    b = b.reshape(idx.shape[:-1] + (-1,))
    pad = -b.shape[-1] % 8
    if pad:
        b = torch.nn.functional.pad(b, (0, pad))
    b = b.reshape(idx.shape[:-1] + (-1, 8))
    return (b << torch.arange(8, device=idx.device, dtype=torch.uint8)).sum(-1, dtype=torch.uint8)


def piece_major(rec):
    """[blocks, heads, block_size, R] records as the cache holds them: pieces of
    16 or 8 bytes (where that divides R) of consecutive positions adjacent."""
    nb, h, bs, r = rec.shape
    p = 16 if r % 16 == 0 else 8 if r % 8 == 0 else r
    return rec.reshape(nb, h, bs, r // p, p).transpose(2, 3).contiguous().reshape(nb, h, bs, r)


def random_indices(case, count, seed, stream):
    """Indices [count, padded width] as quantized keys have them: cells of Gaussian values."""
    t = torch.tensor(0.5 * (codebook(case["bits"], 1)[1:] + codebook(case["bits"], 1)[:-1]), device=DEV, dtype=F32)
    g = generator(seed, stream)
    w = padded_width(case["variant"], case["d"])
    out = torch.empty((count, w), device=DEV, dtype=torch.uint8)
    for s in range(0, count, 1 << 20):
        z = torch.randn((min(count - s, 1 << 20), w), generator=g, device=DEV, dtype=F32)
        out[s:s + z.shape[0]] = torch.bucketize(z, t, out_int32=True).to(torch.uint8)
    return out


def random_norms(case, count, seed, stream):
    z = torch.randn(count, generator=generator(seed, stream), device=DEV, dtype=F32)
    return math.sqrt(case["d"]) * torch.exp(0.3 * z)


def random_cache(case, blocks, seed):
    """A cache as earlier steps left it: idx (as indices), records, norms, signs, gammas."""
    h, bs = case["heads"], case["block_size"]
    count = blocks * h * bs
    # a quarter of the slots are drawn and the rest repeat them in another order
    base = max(1, count // 4)
    pick = torch.randint(0, base, (count,), generator=generator(seed, 21), device=DEV)
    idx = random_indices(case, base, seed, 22)
    c = dict(rec=pack(idx, case["bits"])[pick].reshape(blocks, h, bs, -1), base=idx, pick=pick,
             rho=random_norms(case, count, seed, 23).reshape(blocks, h, bs))
    if case["m"]:
        c["signs"] = torch.randint(0, 256, (blocks, h, bs, case["m"] // 8), generator=generator(seed, 24),
                                   device=DEV, dtype=torch.uint8)
        c["gamma"] = c["rho"] * 0.18
    return c


def lengths(case, seed):
    r = np.random.default_rng([seed, 17])
    if case["op"] == "decode_step" or case["ragged"]:
        return r.integers(max(1, case["ctx"] // 4), case["ctx"] + 1, case["seqs"])
    return np.full(case["seqs"], case["ctx"])


def block_layout(case, seed):
    """(blocks in the cache, block table [seqs, blocks per sequence]): blocks placed at random."""
    per = -(-case["ctx"] // case["block_size"])
    blocks = case["seqs"] * per + 7
    perm = np.random.default_rng([seed, 19]).permutation(blocks)[:case["seqs"] * per]
    return blocks, perm.reshape(case["seqs"], per).astype(np.int32)


def append_slots(case, seed):
    """(blocks in the cache, slot of each new token): prompts in whole blocks placed at random."""
    bs, n = case["block_size"], case["tokens"]
    per = -(-n // bs)
    r = np.random.default_rng([seed, 19])
    if n <= 256:   # a decode step: one token in each of n sequences, every block at its own fill
        blocks = max(64, 2 * n)
        return blocks, r.permutation(blocks)[:n] * bs + r.integers(0, bs, n)
    blocks = per + 5
    return blocks, (r.permutation(blocks)[:per, None] * bs + np.arange(bs)).reshape(-1)[:n]


def handle(case, seed):
    return iq.isoq_params_init(case["variant"], case["d"], case["bits"], n_sets(case), rot=draws(case, seed).reshape(-1),
                               codebook=codebook(case["bits"], case["d"]))


def prepare(case, seed):
    op, d = case["op"], case["d"]
    s = dict(op=op, p=handle(case, seed), sk=None)
    if case["m"]:
        s["sk"] = iq.isoq_sketch_init(s["p"], case["m"], S=projection(case, seed))
    if op in ("roundtrip", "restore", "quantize_sketch"):
        s["x"] = rows(case, (case["n"], d), seed, 1)
        s["dtype"] = s["x"].dtype
        return s
    r = record_bytes(case)
    if op in ("append", "append_sketch"):
        blocks, slots = append_slots(case, seed)
        h, bs = case["heads"], case["block_size"]
        s["slots"] = torch.from_numpy(np.ascontiguousarray(slots, np.int64)).to(DEV)
        s["k"] = rows(case, (case["tokens"], h, d), seed, 1)
        s["k_idx"] = torch.zeros((blocks, h, bs, r), dtype=torch.uint8, device=DEV)
        s["k_rho"] = torch.zeros((blocks, h, bs), device=DEV)
        if op == "append":
            s["pv"] = handle(case, seed + 1000003)
            s["v"] = rows(case, (case["tokens"], h, d), seed, 2)
            s["v_idx"], s["v_rho"] = torch.zeros_like(s["k_idx"]), torch.zeros_like(s["k_rho"])
        else:
            s["k_signs"] = torch.zeros((blocks, h, bs, case["m"] // 8), dtype=torch.uint8, device=DEV)
            s["k_gamma"] = torch.zeros_like(s["k_rho"])
        return s
    # logits (and a decode step before them)
    blocks, table = block_layout(case, seed)
    lens = lengths(case, seed)
    c = random_cache(case, blocks, seed)
    s.update(k_idx=piece_major(c["rec"]), k_rho=c["rho"], k_signs=c.get("signs"), k_gamma=c.get("gamma"),
             q=rows(case, (case["seqs"], case["heads"] * case["group"], d), seed, 3),
             table=torch.from_numpy(table).to(DEV), lens=torch.from_numpy(lens.astype(np.int32)).to(DEV),
             scale=1.0 / math.sqrt(d), out=None)
    if op == "decode_step":
        s["pv"] = handle(case, seed + 1000003)
        s["k"] = rows(case, (case["seqs"], case["heads"], d), seed, 1)
        s["v"] = rows(case, (case["seqs"], case["heads"], d), seed, 2)
        s["slots"] = torch.from_numpy(last_slots(case, table, lens)).to(DEV)
        s["v_idx"], s["v_rho"] = s["k_idx"].clone(), s["k_rho"].clone()
    elif case["own_buffer"]:
        s["out"] = torch.zeros((case["seqs"], case["heads"] * case["group"], table.shape[1] * case["block_size"]),
                               device=DEV)
    return s


def last_slots(case, table, lens):
    """The cache slot of each sequence's newest token."""
    bs = case["block_size"]
    i = np.arange(case["seqs"])
    return table[i, (lens - 1) // bs].astype(np.int64) * bs + (lens - 1) % bs


# ---- one pass ------------------------------------------------------------------------

def run(s):
    op = s["op"]
    if op == "roundtrip":
        return iq.isoq_roundtrip(s["p"], s["x"])
    if op == "restore":
        rec, rho = iq.isoq_quantize(s["p"], s["x"])
        return rec, rho, iq.isoq_dequantize(s["p"], rec, rho, dtype=s["dtype"])
    if op == "quantize_sketch":
        return iq.isoq_quantize_qjl(s["p"], s["sk"], s["x"])
    if op == "append_sketch":
        iq.isoq_kv_append_qjl(s["p"], s["sk"], s["k"], s["slots"], s["k_idx"], s["k_rho"], s["k_signs"], s["k_gamma"])
        return s["k_idx"], s["k_rho"], s["k_signs"], s["k_gamma"]
    if op in ("append", "decode_step"):
        iq.isoq_kv_append(s["p"], s["k"], s["slots"], s["k_idx"], s["k_rho"], s["pv"], s["v"], s["v_idx"], s["v_rho"])
        cache = (s["k_idx"], s["k_rho"], s["v_idx"], s["v_rho"])
        if op == "append":
            return cache
        return (iq.isoq_kv_scores(s["p"], s["q"], s["k_idx"], s["k_rho"], s["table"], s["lens"], scale=s["scale"]),
                ) + cache
    if s["sk"] is not None:
        return iq.isoq_kv_scores_qjl(s["p"], s["sk"], s["q"], s["k_idx"], s["k_rho"], s["k_signs"], s["k_gamma"],
                                     s["table"], s["lens"], scale=s["scale"], scores=s["out"])
    return iq.isoq_kv_scores(s["p"], s["q"], s["k_idx"], s["k_rho"], s["table"], s["lens"], scale=s["scale"],
                             scores=s["out"])


# ---- what a pass cannot do without, and how exact it is ---------------------------------

def work(case):
    op, d, r = case["op"], case["d"], record_bytes(case)
    es = 4 if case["dtype"] == "f32" else 2
    rot = 2 * d * {"full": 4, "fast": 4, "2d": 2}[case["variant"]]   # one block rotation of a row
    sketch = case["m"] // 8 + 4 if case["m"] else 0
    project = 2 * case["m"] * d
    if op == "roundtrip":
        return dict(bytes=case["n"] * 2 * d * es, flops=case["n"] * 2 * rot)
    if op == "restore":
        return dict(bytes=case["n"] * 2 * (d * es + r + 4), flops=case["n"] * 2 * rot)
    if op == "quantize_sketch":
        return dict(bytes=case["n"] * (d * es + r + 4 + sketch), flops=case["n"] * (rot + project))
    if op in ("append", "append_sketch"):
        n = case["tokens"] * case["heads"] * (2 if op == "append" else 1)
        return dict(bytes=n * (d * es + r + 4 + sketch) + case["tokens"] * 8, flops=n * (rot + project))
    frac = 0.625 if op == "decode_step" or case["ragged"] else 1.0   # mean length over ctx
    keys = frac * case["seqs"] * case["heads"] * case["ctx"]
    n = 0 if op != "decode_step" else 2 * case["seqs"] * case["heads"]
    return dict(bytes=keys * (r + 4 + sketch + 4 * case["group"]) + case["seqs"] * case["heads"] * case["group"] * d * es
                + case["seqs"] * (case["ctx"] // case["block_size"] * 4 + 4) + n * (d * es + r + 4),
                flops=keys * case["group"] * 2 * (d + case["m"]) + n * rot)


def tolerance(case):
    # records: a rotated coordinate within rounding of a threshold may take
    # either cell (about 5e-7 of the bytes against 64 bits, or one byte of a
    # small case), which moves a restored coordinate by up to a cell; signs: a
    # projection within rounding of zero may take either sign (7e-4 of the bytes)
    op = case["op"]
    if op in ("roundtrip", "restore"):
        return {"rel": 2e-3, "max": 0.9, "differ": 2e-6 + 1.5 / (case["n"] * record_bytes(case))}
    if op in ("append_sketch", "quantize_sketch"):
        return {"rel": 1e-5, "max": 1e-3, "differ": 3e-3}
    if op == "append":
        return {"rel": 1e-6, "max": 1e-5, "differ": 2e-6 + 1.5 / (case["tokens"] * case["heads"] * record_bytes(case))}
    return {"rel": 1e-6, "max": 1e-5, "differ": 1e-5}


# ---- the same outputs in 64 bits --------------------------------------------------------

def matrices(case, seed):
    """The block rotations [sets, blocks, k, k] in 64 bits (k = 4; 2 for planar pairs)."""
    u = draws(case, seed)
    if case["variant"] == "2d":
        c, s = np.cos(u), np.sin(u)
        m = np.stack([np.stack([c, -s], -1), np.stack([s, c], -1)], -2)
        return torch.from_numpy(m).to(DEV)

    def left(q):
        a, b, c, d = np.moveaxis(q, -1, 0)
        return np.stack([np.stack(v, -1) for v in ((a, -b, -c, -d), (b, a, -d, c), (c, d, a, -b), (d, -c, b, a))], -2)

    def right(q):
        a, b, c, d = np.moveaxis(q, -1, 0)
        return np.stack([np.stack(v, -1) for v in ((a, -b, -c, -d), (b, a, d, -c), (c, -d, a, b), (d, c, -b, a))], -2)

    ql = u[..., :4] / np.linalg.norm(u[..., :4], axis=-1, keepdims=True)
    m = left(ql)
    if case["variant"] == "full":
        qr = u[..., 4:] / np.linalg.norm(u[..., 4:], axis=-1, keepdims=True)
        m = m @ right(qr * np.array([1.0, -1.0, -1.0, -1.0]))
    return torch.from_numpy(np.ascontiguousarray(m)).to(DEV)


def rotate(m, x):
    """Block rotation m [blocks, k, k] of rows x [n, d], zero padded to whole blocks."""
    b, k = m.shape[0], m.shape[-1]
    x = torch.nn.functional.pad(x, (0, b * k - x.shape[-1])).reshape(-1, b, k)
    return sum(x[..., j, None] * m[:, :, j] for j in range(k)).reshape(-1, b * k)


def encode(case, m, x):
    """(indices, norms, levels selected, T x / norm) of rows x in 64 bits, one set."""
    lev = torch.tensor(codebook(case["bits"], case["d"]), device=DEV, dtype=torch.float64)
    x = x.double()
    rho = x.norm(dim=-1)
    y = rotate(m, x) / rho.clamp_min(1e-12)[:, None]
    idx = torch.bucketize(y, 0.5 * (lev[1:] + lev[:-1]))
    return idx, rho, lev[idx], y


def by_chunks(f, x, step=1 << 17):
    parts = [f(x[i:i + step]) for i in range(0, x.shape[0], step)]
    return [torch.cat(p) for p in zip(*parts)]


def exact(case, seed):
    op, d = case["op"], case["d"]
    ms = matrices(case, seed)
    if op in ("roundtrip", "restore"):
        x = rows(case, (case["n"], d), seed, 1)

        def there_and_back(xc):
            _, rho, c, _ = encode(case, ms[0], xc)
            return rho, (rho[:, None] * rotate(ms[0].transpose(-1, -2), c))[:, :d]
        rho, x_hat = by_chunks(there_and_back, x)
        return x_hat if op == "roundtrip" else (None, rho, x_hat)
    if op == "quantize_sketch":
        rho, gamma = by_chunks(lambda xc: norms_of(case, ms[0], xc), rows(case, (case["n"], d), seed, 1))
        return None, rho, None, gamma
    if op in ("append", "append_sketch"):
        blocks, slots = append_slots(case, seed)
        h, bs = case["heads"], case["block_size"]
        slots = torch.from_numpy(np.ascontiguousarray(slots, np.int64)).to(DEV)

        def cached(values):   # [tokens, heads] into [blocks, heads, block_size]
            c = torch.zeros((blocks, bs, h), device=DEV, dtype=torch.float64)
            c.view(-1, h)[slots] = values
            return c.transpose(1, 2).contiguous()

        def of(stream, want_gamma):
            x = rows(case, (case["tokens"], h, d), seed, stream)
            if not want_gamma:
                return cached(by_chunks(lambda xc: (xc.double().norm(dim=-1),), x, 1 << 12)[0]), None
            got = [by_chunks(lambda xc, i=i: norms_of(case, ms[i], xc), x[:, i].contiguous()) for i in range(h)]
            return tuple(cached(torch.stack([g[k] for g in got], 1)) for k in (0, 1))
        rho, gamma = of(1, op == "append_sketch")
        return (None, rho, None, gamma) if op == "append_sketch" else (None, rho, None, of(2, False)[0])
    return exact_scores(case, seed, ms)


def norms_of(case, m, x):
    _, rho, c, y = encode(case, m, x)
    return rho, rho * (y - c).norm(dim=-1)


def exact_scores(case, seed, ms):
    d, h, g, bs = case["d"], case["heads"], case["group"], case["block_size"]
    blocks, table = block_layout(case, seed)
    lens = lengths(case, seed)
    c = random_cache(case, blocks, seed)
    pick = c["pick"].reshape(blocks, h, bs)
    lev = torch.tensor(codebook(case["bits"], d), device=DEV, dtype=torch.float64)
    q = rows(case, (case["seqs"], h * g, d), seed, 3).double()
    scale = 1.0 / math.sqrt(d)
    step = case["op"] == "decode_step"
    if step:
        k = rows(case, (case["seqs"], h, d), seed, 1)
        rho_k = k.double().norm(dim=-1)
    fill = 0.0 if not step and case["own_buffer"] else NEG_INF
    out = torch.full((case["seqs"], h * g, table.shape[1] * bs), fill, device=DEV, dtype=torch.float64)
    if case["m"]:
        S = torch.from_numpy(projection(case, seed)).to(DEV)
        bits = torch.arange(8, device=DEV, dtype=torch.uint8)
    for s in range(case["seqs"]):
        t = torch.arange(int(lens[s]), device=DEV)
        blk = torch.from_numpy(table[s].astype(np.int64)).to(DEV)[t // bs]
        for i in range(h):
            qs = q[s, i * g:(i + 1) * g]
            keys = lev[c["base"][pick[blk, i, t % bs]].long()]
            rho = c["rho"][blk, i, t % bs].double()
            if step:   # the newest position holds the appended key
                _, _, ck, _ = encode(case, ms[i], k[s, i:i + 1])
                keys[-1], rho[-1] = ck[0], rho_k[s, i]
            val = rho * (rotate(ms[i], qs) @ keys.t().contiguous())
            if case["m"]:
                z = ((c["signs"][blk, i, t % bs].unsqueeze(-1) >> bits) & 1).reshape(-1, case["m"]).double() * 2 - 1
                sz = qs @ S.t().contiguous() @ z.t().contiguous()
                val += (math.sqrt(math.pi / 2) / case["m"]) * c["gamma"][blk, i, t % bs].double() * sz
            out[s, i * g:(i + 1) * g, :len(t)] = scale * val
    if not step:
        return out
    rho_v = rows(case, (case["seqs"], h, d), seed, 2).double().norm(dim=-1)
    slots = torch.from_numpy(last_slots(case, table, lens)).to(DEV)
    caches = []
    for new in (rho_k, rho_v):
        r = c["rho"].double().clone()
        r[slots // bs, :, slots % bs] = new
        caches += [None, r]
    return (out, *caches)
