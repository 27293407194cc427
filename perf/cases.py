"""Workloads by which this library's speed is judged: what a program that
uses it has it do, through the public entry points (the Python binding of the
C ABI and the block chain built on it), each with its work, a tolerance and a
64-bit value.

Sizes are those of the repository's configurations and benchmark (one GPU's
share of LLaMA-shaped blocks, the matrix chains, the fp32 matmul in 64-blocks,
the reductions and repartitions) and, in between, generic ones; draw() spreads
over the ranges they stand for, odd and ragged sizes included.

A pass returns whole output relations: the block-major storage, each block at
a 256-byte multiple, the padding between blocks zeroed once by prepare().
"""
from __future__ import annotations

import math

import torch

from paper_2609_03905_amd import ea
from paper_2609_03905_amd.block import LlamaBlockShare

TORCH = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
EPS = 1e-6


def listed():
    return [
        # The smallest call: the fp32 matmul of 256^3 in 4x4 blocks of 64x64
        # (four partial products per output block).  Latency counts.
        {"name": "matmul_f32_256", "kind": "matmul_f32", "m": 256, "k": 256, "n": 256, "block": 64, "kmajor": False},
        # An ordinary fp32 block product, ragged blocks on two letters.
        {"name": "matmul_f32_1536", "kind": "matmul_f32", "m": 1536, "k": 2048, "n": 1160, "block": 512,
         "kmajor": False},
        # A general einsum: the per-head scores of 8 heads, bf16 in, fp32 out
        # (two operands sharing a batch letter).
        {"name": "einsum_head_scores", "kind": "einsum", "spec": "hqd,hkd->hqk", "join": "mul", "agg": "sum",
         "b": 8, "i": 256, "j": 128, "k": 256, "block": 128, "dtype": "bf16", "out": "f32"},
        # One GPU's column share of a LLaMA-7B QKV projection and its
        # repartition to per-head blocks (prefill of 4096 tokens).
        {"name": "qkv_projection", "kind": "projection", "t": 4096, "j": 4096, "k": 1536, "block": 512, "head": 128},
        # A block GEMM of no round size: an odd number of tokens, a contracted
        # width that is a multiple of 8 only, weights stored [out, in], a
        # residual, fp16.
        {"name": "gemm_ragged_f16", "kind": "gemm", "t": 1001, "j": 2744, "k": 2008, "block": 512, "dtype": "f16",
         "kmajor": True, "residual": True},
        # The gated FFN product of a LLaMA-65B-shape share (width 22016 / 8).
        {"name": "swiglu_65b_share", "kind": "swiglu", "t": 2048, "j": 8192, "k": 2752, "block": 512,
         "dtype": "bf16", "kmajor": False},
        # One product of a matrix chain (about 8192^3 multiplies): the largest.
        {"name": "chain_product", "kind": "gemm", "t": 10240, "j": 16384, "k": 6144, "block": 512, "dtype": "bf16",
         "kmajor": False, "residual": False},
        # Causal attention, a head share of LLaMA-7B at batch 2, 2K tokens.
        {"name": "attention_2k", "kind": "attention", "b": 2, "h": 4, "g": 1, "s": 2048, "seq": 2048, "causal": True},
        # Causal grouped-query attention on one long sequence (4 query heads
        # over one key/value head, 8K tokens).
        {"name": "attention_gqa_8k", "kind": "attention", "b": 1, "h": 4, "g": 4, "s": 8192, "seq": 8192,
         "causal": True},
        # The row reductions on their own: RMSNorm over 4096-wide rows and
        # causal softmax over 2K scores, outputs streamed.
        {"name": "reductions", "kind": "reductions", "rows": 4096, "c": 4096, "cblock": 512, "h": 4, "s": 2048,
         "kblock": 256, "dtype": "bf16"},
        # A relation larger than the caches re-blocked: 256 MiB.
        {"name": "repartition_256m", "kind": "repartition", "m": 8192, "n": 16384, "am": 512, "an": 512, "bm": 128,
         "bn": 16384, "dtype": "bf16"},
        # The whole chain of one GPU's share of a LLaMA-65B-shape block.
        {"name": "block_65b_share", "kind": "block", "t": 2048, "hidden": 8192, "heads": 8, "heads_kv": 8,
         "ffn": 2752, "seq": 2048, "block": 512},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _mult(v, q):
    return max(q, v // q * q)


def draw(rng):
    kind = rng.choice(["matmul_f32", "einsum", "projection", "gemm", "gemm", "swiglu", "attention", "attention",
                       "rmsnorm", "softmax", "repartition", "block"])
    block = rng.choice([128, 256, 512])
    if kind == "matmul_f32":
        return {"kind": kind, "m": _log(rng, 64, 2048), "k": _log(rng, 64, 2048), "n": _log(rng, 64, 2048),
                "block": rng.choice([64, 100, 256, 512]), "kmajor": rng.random() < 0.5}
    if kind == "einsum":
        spec, join, agg = rng.choice([("hqd,hkd->hqk", "mul", "sum"), ("bij,bjk->bik", "mul", "sum"),
                                      ("tj,jk->tk", "mul", "sum"), ("ij->j", "mul", "sum"), ("ij->i", "mul", "max"),
                                      ("ij,ij->ij", "mul", "none"), ("ij,ij->ij", "add", "none")])
        if spec in ("hqd,hkd->hqk", "bij,bjk->bik"):
            b, i, j, k = rng.randint(2, 12), _log(rng, 33, 256), _log(rng, 32, 128), _log(rng, 33, 256)
        elif spec == "tj,jk->tk":  # extents that no vector width divides
            b, i, j, k = 1, _log(rng, 32, 512) | 1, _log(rng, 32, 256) | 1, _log(rng, 32, 512) | 1
        else:
            b, i, j, k = 1, _log(rng, 64, 4096), _log(rng, 64, 2048), 1
        dtype = rng.choice(["f32", "bf16"])
        return {"kind": kind, "spec": spec, "join": join, "agg": agg, "b": b, "i": i, "j": j, "k": k,
                "block": rng.choice([64, 128]), "dtype": dtype, "out": rng.choice(["f32", dtype])}
    if kind == "projection":
        return {"kind": kind, "t": _log(rng, 128, 8192), "j": _mult(_log(rng, 1024, 8192), 64),
                "k": 128 * rng.randint(3, 24), "block": 512, "head": 128}
    if kind in ("gemm", "swiglu"):
        c = {"kind": kind, "t": _log(rng, 64, 8192), "j": _mult(_log(rng, 256, 8192), rng.choice([8, 32, 128])),
             "k": _mult(_log(rng, 256, 8192), 8), "block": block, "dtype": rng.choice(["bf16", "bf16", "f16"]),
             "kmajor": rng.random() < 0.4}
        if kind == "gemm":
            c["residual"] = rng.random() < 0.4
        return c
    if kind == "attention":
        seq = 128 * _log(rng, 2, 64)
        n_seq = rng.choice([1, 1, rng.randint(2, 8)])
        while n_seq > 1 and n_seq * seq > 8192:
            n_seq -= 1
        g = rng.choice([1, 1, 4])
        return {"kind": kind, "b": rng.choice([1, 1, 2]), "h": g * rng.randint(1, 8 // g), "g": g, "s": n_seq * seq,
                "seq": seq, "causal": rng.random() < 0.8}
    if kind == "rmsnorm":
        c = _log(rng, 256, 8192)
        return {"kind": kind, "rows": _log(rng, 64, 8192), "c": c if rng.random() < 0.3 else _mult(c, 64),
                "cblock": rng.choice([512, 1024]), "dtype": rng.choice(["bf16", "bf16", "f32"]),
                "stream": rng.random() < 0.5}
    if kind == "softmax":
        s = _log(rng, 128, 4096)
        return {"kind": kind, "h": rng.randint(1, 4), "s": s if rng.random() < 0.3 else _mult(s, 64),
                "kblock": rng.choice([128, 256]), "dtype": rng.choice(["bf16", "bf16", "f32"]),
                "causal": rng.random() < 0.7, "stream": rng.random() < 0.5}
    if kind == "repartition":
        return {"kind": kind, "m": _log(rng, 256, 8192), "n": _log(rng, 256, 16384), "am": rng.choice([128, 500, 512]),
                "an": rng.choice([256, 500, 512]), "bm": rng.choice([64, 128, 300, 1024]),
                "bn": rng.choice([128, 300, 1024, 16384]), "dtype": rng.choice(["bf16", "f32"])}
    heads_kv = rng.choice([1, 2])
    t = 128 * _log(rng, 2, 16)
    n_seq = rng.choice([1, 2])
    return {"kind": "block", "t": n_seq * t, "hidden": 512 * rng.randint(2, 12), "heads": heads_kv * rng.choice([1, 4]),
            "heads_kv": heads_kv, "ffn": 64 * rng.randint(8, 40), "seq": t, "block": 512}


# ---- shapes and partitions ---------------------------------------------------
def _splits(n, b):
    return list(range(0, n, b)) + [n]


def _seq_ends(c):
    return list(range(c["seq"], c["s"] + 1, c["seq"])) if c["seq"] < c["s"] else None


def _einsum_parts(c):
    """Per operand of the spec (inputs, then output): shape and partition."""
    ext = dict(zip("hqdk", (c["b"], c["i"], c["j"], c["k"]))) if "h" in c["spec"] else \
        dict(zip("tjk", (c["i"], c["j"], c["k"]))) if "t" in c["spec"] else \
        dict(zip("bijk", (c["b"], c["i"], c["j"], c["k"])))
    lhs, out = c["spec"].split("->")
    return [(tuple(ext[x] for x in op), [_splits(ext[x], c["block"]) for x in op]) for op in lhs.split(",") + [out]]


def _attention_parts(c):
    hk = c["h"] // c["g"]
    part = lambda h: [_splits(c["b"], 1), _splits(h, 1), _splits(c["s"], 128), [0, 128]]
    return ((c["b"], c["h"], c["s"], 128), part(c["h"])), ((c["b"], hk, c["s"], 128), part(hk))


def _block_shapes(c):
    hd, wqkv = c["heads"] * 128, (c["heads"] + 2 * c["heads_kv"]) * 128
    return {"x": (c["t"], c["hidden"]), "n1": (c["hidden"],), "n2": (c["hidden"],), "wqkv": (c["hidden"], wqkv),
            "wo": (hd, c["hidden"]), "wg": (c["hidden"], c["ffn"]), "wu": (c["hidden"], c["ffn"]),
            "wd": (c["ffn"], c["hidden"])}


# ---- inputs, made from the seed alone ----------------------------------------
def _dense(c, seed):
    """The dense inputs of a case, on the GPU, in their storage type:
    activations N(0, 1), weights N(0, 0.02) (chain matrices N(0, 1/width)),
    norm weights U(0.5, 1.5)."""
    g = torch.Generator(device="cuda")
    g.manual_seed(7919 * int(seed) + 17)

    def normal(shape, dtype, std=1.0):
        return (torch.randn(shape, generator=g, device="cuda", dtype=torch.float32) * std).to(TORCH[dtype])

    def uniform(shape, dtype):
        return (torch.rand(shape, generator=g, device="cuda", dtype=torch.float32) + 0.5).to(TORCH[dtype])

    k = c["kind"]
    if k == "matmul_f32":
        return [normal((c["m"], c["k"]), "f32"), normal((c["n"], c["k"]) if c["kmajor"] else (c["k"], c["n"]), "f32")]
    if k == "einsum":
        return [normal(shape, c["dtype"]) for shape, _ in _einsum_parts(c)[:-1]]
    if k == "projection":
        return [normal((c["t"], c["j"]), "bf16"), normal((c["j"], c["k"]), "bf16", 0.02)]
    if k in ("gemm", "swiglu"):
        w = (c["k"], c["j"]) if c["kmajor"] else (c["j"], c["k"])
        std = 1.0 / c["j"] ** 0.5 if k == "gemm" else 0.02
        out = [normal((c["t"], c["j"]), c["dtype"])] + [normal(w, c["dtype"], std) for _ in range(1 + (k == "swiglu"))]
        if c.get("residual"):
            out.append(normal((c["t"], c["k"]), c["dtype"]))
        return out
    if k == "attention":
        (sq, _), (sk, _) = _attention_parts(c)
        return [normal(sq, "bf16"), normal(sk, "bf16"), normal(sk, "bf16")]
    if k == "rmsnorm":
        return [normal((c["rows"], c["c"]), c["dtype"]), uniform((c["c"],), c["dtype"])]
    if k == "softmax":
        return [normal((c["h"], c["s"], c["s"]), c["dtype"])]
    if k == "reductions":
        return [normal((c["rows"], c["c"]), c["dtype"]), uniform((c["c"],), c["dtype"]),
                normal((c["h"], c["s"], c["s"]), c["dtype"])]
    if k == "repartition":
        return [normal((c["m"], c["n"]), c["dtype"])]
    return {n: uniform(s, "bf16") if n in ("n1", "n2") else normal(s, "bf16", 1.0 if n == "x" else 0.02)
            for n, s in _block_shapes(c).items()}


def _out(shape, dtype, part):
    r = ea.Relation(shape, dtype, part)
    r.data.zero_()  # the padding between blocks
    return r


def prepare(case, seed):
    """Relations holding the inputs and zeroed outputs, and the planned
    configuration (a program plans once, at start-up)."""
    c, d = case, _dense(case, seed)
    k = c["kind"]
    calls = []  # the join-aggs of a pass: (positional arguments, keyword arguments)
    reparts = []  # then its repartitions: (source, destination, store)
    S = ea.AGG_SUM
    if k == "matmul_f32":
        pm, pk, pn = (_splits(c[x], c["block"]) for x in "mkn")
        A = ea.from_dense(d[0], "f32", [pm, pk])
        B = ea.from_dense(d[1], "f32", [pn, pk] if c["kmajor"] else [pk, pn])
        C = _out((c["m"], c["n"]), "f32", [pm, pn])
        calls.append((("ij,kj->ik" if c["kmajor"] else "ij,jk->ik", ea.JOIN_MUL, S, [A, B], C), {}))
        outs = [C]
    elif k == "einsum":
        parts = _einsum_parts(c)
        ins = [ea.from_dense(x, c["dtype"], p) for x, (_, p) in zip(d, parts)]
        C = _out(parts[-1][0], c["out"], parts[-1][1])
        join = ea.JOIN_MUL if c["join"] == "mul" else ea.JOIN_ADD
        agg = {"sum": S, "max": ea.AGG_MAX, "none": ea.AGG_NONE}[c["agg"]]
        calls.append(((c["spec"], join, agg, ins, C), {}))
        outs = [C]
    elif k == "projection":
        pt, pj, pk = (_splits(c[x], c["block"]) for x in "tjk")
        X, W = ea.from_dense(d[0], "bf16", [pt, pj]), ea.from_dense(d[1], "bf16", [pj, pk])
        Y = _out((c["t"], c["k"]), "bf16", [pt, pk])
        Yh = _out((c["t"], c["k"]), "bf16", [[0, c["t"]], _splits(c["k"], c["head"])])
        calls.append((("tj,jk->tk", ea.JOIN_MUL, S, [X, W], Y), {}))
        reparts.append((Y, Yh, ea.STORE_CACHED))
        outs = [Y, Yh]
    elif k in ("gemm", "swiglu"):
        pt, pj, pk = (_splits(c[x], c["block"]) for x in "tjk")
        pw = [pk, pj] if c["kmajor"] else [pj, pk]
        X = ea.from_dense(d[0], c["dtype"], [pt, pj])
        Ws = [ea.from_dense(w, c["dtype"], pw) for w in d[1:2 + (k == "swiglu")]]
        Y = _out((c["t"], c["k"]), c["dtype"], [pt, pk])
        kw = {"residual": ea.from_dense(d[2], c["dtype"], [pt, pk])} if c.get("residual") else {}
        spec = ("tj,kj" + ",kj" * (k == "swiglu") if c["kmajor"] else "tj,jk" + ",jk" * (k == "swiglu")) + "->tk"
        calls.append(((spec, ea.OP_SWIGLU if k == "swiglu" else ea.JOIN_MUL, S, [X] + Ws, Y), kw))
        outs = [Y]
    elif k == "attention":
        (sq, pq), (sk, pk) = _attention_parts(c)
        Q, K, V = ea.from_dense(d[0], "bf16", pq), ea.from_dense(d[1], "bf16", pk), ea.from_dense(d[2], "bf16", pk)
        O = _out(sq, "bf16", pq)
        kw = dict(scale=1.0 / 128 ** 0.5, causal=c["causal"], gqa_group=c["g"] if c["g"] > 1 else 0,
                  seq_ends=_seq_ends(c))
        calls.append((("bhqd,bgkd,bgkd->bhqd" if c["g"] > 1 else "bhqd,bhkd,bhkd->bhqd", ea.OP_ATTENTION, ea.AGG_LSE,
                       [Q, K, V], O), kw))
        outs = [O]
    elif k in ("rmsnorm", "softmax", "reductions"):
        outs = []
        store = ea.STORE_STREAM if c.get("stream", True) else ea.STORE_CACHED
        if k != "softmax":
            px = [[0, c["rows"]], _splits(c["c"], c["cblock"])]
            X, W = ea.from_dense(d[0], c["dtype"], px), ea.from_dense(d[1], c["dtype"], [px[1]])
            outs.append(_out((c["rows"], c["c"]), c["dtype"], px))
            calls.append((("tc,c->tc", ea.OP_RMSNORM, S, [X, W], outs[-1]), dict(eps=EPS, store=store)))
        if k != "rmsnorm":
            ps = [_splits(c["h"], 1), [0, c["s"]], _splits(c["s"], c["kblock"])]
            outs.append(_out((c["h"], c["s"], c["s"]), c["dtype"], ps))
            calls.append((("hqk->hqk", ea.OP_SOFTMAX, ea.AGG_LSE, [ea.from_dense(d[-1], c["dtype"], ps)], outs[-1]),
                          dict(causal=c.get("causal", True), store=store)))
    elif k == "repartition":
        A = ea.from_dense(d[0], c["dtype"], [_splits(c["m"], c["am"]), _splits(c["n"], c["an"])])
        B = _out((c["m"], c["n"]), c["dtype"], [_splits(c["m"], c["bm"]), _splits(c["n"], c["bn"])])
        reparts.append((A, B, ea.STORE_STREAM))
        outs = [B]
    else:
        ends = list(range(c["seq"], c["t"] + 1, c["seq"])) if c["seq"] < c["t"] else None
        blk = LlamaBlockShare(c["t"], c["hidden"], c["heads"], 128, c["ffn"], block=c["block"], eps=EPS,
                              heads_kv=c["heads_kv"], seq_ends=ends)
        blk.y.data.zero_()
        blk.load(d)
        return {"kind": k, "block": blk}
    for args, kw in calls:
        ea.joinagg_workspace(*args, **kw)
    for src, dst, _ in reparts:
        ea.repartition_plan(src, dst)
    return {"kind": k, "calls": calls, "reparts": reparts, "outs": outs}


def _values(rel, bits=False):
    """A relation's storage as values (or as integers of the same width)."""
    if bits:
        return rel.bytes().view(torch.int32 if rel.dtype == "f32" else torch.int16)
    return rel.bytes().view(TORCH[rel.dtype])


def run(state):
    if state["kind"] == "block":
        return [_values(state["block"].forward())]
    for args, kw in state["calls"]:
        ea.joinagg(*args, **kw)
    for src, dst, store in state["reparts"]:
        ea.repartition(src, dst, store=store)
    return [_values(r, bits=state["kind"] == "repartition") for r in state["outs"]]


# ---- work --------------------------------------------------------------------
def work(case):
    c, k = case, case["kind"]
    es = lambda dt: 4 if dt == "f32" else 2
    n = lambda shape: math.prod(shape)
    if k == "matmul_f32":
        m, kk, nn = c["m"], c["k"], c["n"]
        return {"bytes": 4 * (m * kk + kk * nn + m * nn), "flops": 2 * m * kk * nn}
    if k == "einsum":
        shapes = [s for s, _ in _einsum_parts(c)]
        ext = c["b"] * c["i"] * c["j"] * c["k"]
        terms = len(shapes) - 1  # one multiply or add per joined pair, one per aggregated term
        return {"bytes": sum(n(s) for s in shapes[:-1]) * es(c["dtype"]) + n(shapes[-1]) * es(c["out"]),
                "flops": ext * (terms - 1 + (c["agg"] != "none"))}
    if k == "projection":
        t, j, kk = c["t"], c["j"], c["k"]
        return {"bytes": 2 * (t * j + j * kk + 3 * t * kk), "flops": 2 * t * j * kk}
    if k in ("gemm", "swiglu"):
        t, j, kk, w = c["t"], c["j"], c["k"], 1 + (k == "swiglu")
        return {"bytes": 2 * (t * j + w * j * kk + t * kk * (1 + bool(c.get("residual")))),
                "flops": 2 * t * j * kk * w}
    if k == "attention":
        (sq, _), (sk, _) = _attention_parts(c)
        pairs = c["seq"] * (c["seq"] + 1) // 2 if c["causal"] else c["seq"] ** 2
        return {"bytes": 2 * (2 * n(sq) + 2 * n(sk)), "flops": 4 * 128 * pairs * (c["s"] // c["seq"]) * c["b"] * c["h"]}
    if k in ("rmsnorm", "softmax", "reductions"):
        b = f = 0
        e = es(c["dtype"])
        if k != "softmax":
            b += (2 * c["rows"] + 1) * c["c"] * e
            f += 4 * c["rows"] * c["c"]
        if k != "rmsnorm":
            seen = c["s"] * (c["s"] + 1) // 2 if c.get("causal", True) else c["s"] ** 2
            b += c["h"] * (seen + c["s"] ** 2) * e
            f += 5 * c["h"] * seen
        return {"bytes": b, "flops": f}
    if k == "repartition":
        return {"bytes": 2 * c["m"] * c["n"] * es(c["dtype"]), "flops": 0}
    s = _block_shapes(c)
    t, hd = c["t"], c["heads"] * 128
    pairs = c["seq"] * (c["seq"] + 1) // 2 * (t // c["seq"])
    weights = sum(n(v) for x, v in s.items() if x != "x")
    return {"bytes": 2 * (weights + 2 * n(s["x"])),
            "flops": 2 * t * (n(s["wqkv"]) + n(s["wo"]) + n(s["wg"]) + n(s["wu"]) + n(s["wd"]))
            + 4 * hd * pairs}


def tolerance(case):
    """About four times what an independent computation at the same precision
    (64-bit sums, the same storage types) is measured to differ by."""
    c, k = case, case["kind"]
    if k == "repartition":
        return "exact"
    if k == "block":
        return {"rel": 1.5e-2}  # bf16 at nine relation boundaries, softmax and SwiGLU between
    dtype = "f32" if k == "matmul_f32" else c.get("out", c.get("dtype", "bf16"))
    return {"f32": {"rel": 4e-6}, "f16": {"rel": 1e-3}, "bf16": {"rel": 7e-3}}[dtype]


# ---- 64-bit values -----------------------------------------------------------
def _packed(dense, part):
    """Block-major storage of a dense tensor: blocks row-major, each at a
    multiple of 256 bytes of its stored type (part[0] is that type)."""
    dtype, splits = part
    unit = 256 // (4 if dtype == "f32" else 2)
    pieces, pos = [], 0

    def walk(d, x):
        nonlocal pos
        if d == len(splits):
            pad = -pos % unit
            pieces.append(torch.zeros(pad, dtype=x.dtype, device=x.device))
            pieces.append(x.reshape(-1))
            pos += pad + x.numel()
            return
        for lo, hi in zip(splits[d], splits[d][1:]):
            walk(d + 1, x.narrow(d, lo, hi - lo))

    walk(0, dense)
    return torch.cat(pieces)


def _attend(q, k, v, causal, ends):
    """softmax(q k^T / sqrt(d)) v per head and sequence, in 64 bits; q [h, s, d], k and v [g, s, d]."""
    h, s, _ = q.shape
    out = torch.empty_like(q)
    for i in range(h):
        kv = i * k.shape[0] // h
        for lo, hi in zip([0] + ends[:-1], ends):
            x = q[i, lo:hi] @ k[kv, lo:hi].T / 128 ** 0.5
            if causal:
                x.masked_fill_(torch.ones_like(x, dtype=torch.bool).triu(1), -math.inf)
            out[i, lo:hi] = torch.softmax(x, -1) @ v[kv, lo:hi]
    return out


def _rmsnorm(x, w):
    return w * x / torch.sqrt((x * x).mean(-1, keepdim=True) + EPS)


def exact(case, seed):
    c, k, d = case, case["kind"], _dense(case, seed)
    if k == "repartition":
        return None
    if k == "block":
        return [_exact_block(c, {n: x.double() for n, x in d.items()})]
    d = [x.double() for x in d]
    if k == "matmul_f32":
        y = d[0] @ (d[1].T if c["kmajor"] else d[1])
        return [_packed(y, ("f32", [_splits(c["m"], c["block"]), _splits(c["n"], c["block"])]))]
    if k == "einsum":
        if c["agg"] == "max":
            y = d[0].amax(1)
        elif c["join"] == "add":
            y = d[0] + d[1]
        else:
            y = torch.einsum(c["spec"], *d)
        return [_packed(y, (c["out"], _einsum_parts(c)[-1][1]))]
    if k == "projection":
        y = d[0] @ d[1]
        return [_packed(y, ("bf16", [_splits(c["t"], c["block"]), _splits(c["k"], c["block"])])),
                _packed(y, ("bf16", [[0, c["t"]], _splits(c["k"], c["head"])]))]
    if k in ("gemm", "swiglu"):
        p = [d[0] @ (w.T if c["kmajor"] else w) for w in d[1:2 + (k == "swiglu")]]
        y = torch.nn.functional.silu(p[0]) * p[1] if k == "swiglu" else p[0] + d[2] if c.get("residual") else p[0]
        return [_packed(y, (c["dtype"], [_splits(c["t"], c["block"]), _splits(c["k"], c["block"])]))]
    if k == "attention":
        (_, pq), _ = _attention_parts(c)
        y = torch.stack([_attend(d[0][b], d[1][b], d[2][b], c["causal"], _seq_ends(c) or [c["s"]])
                         for b in range(c["b"])])
        return [_packed(y, ("bf16", pq))]
    out = []
    if k != "softmax":
        out.append(_packed(_rmsnorm(d[0], d[1]), (c["dtype"], [[0, c["rows"]], _splits(c["c"], c["cblock"])])))
    if k != "rmsnorm":
        x = d[-1]
        if c.get("causal", True):
            x = x.masked_fill(torch.ones(c["s"], c["s"], dtype=torch.bool, device=x.device).triu(1), -math.inf)
        out.append(_packed(torch.softmax(x, -1), (c["dtype"], [_splits(c["h"], 1), [0, c["s"]],
                                                               _splits(c["s"], c["kblock"])])))
    return out


def _exact_block(c, d):
    """The chain in 64 bits, every relation between two operators stored as
    bf16 (the chain's definition)."""
    r = lambda x: x.to(torch.bfloat16).double()
    heads = lambda x, n: x.reshape(c["t"], n, 128).transpose(0, 1).contiguous()
    h, g = c["heads"], c["heads_kv"]
    ends = list(range(c["seq"], c["t"] + 1, c["seq"]))
    qkv = r(r(_rmsnorm(d["x"], d["n1"])) @ d["wqkv"])
    q, k, v = qkv.split([h * 128, g * 128, g * 128], 1)
    o = r(_attend(heads(q, h), heads(k, g), heads(v, g), True, ends)).transpose(0, 1).reshape(c["t"], h * 128)
    x2 = r(d["x"] + o @ d["wo"])
    h2 = r(_rmsnorm(x2, d["n2"]))
    a = r(torch.nn.functional.silu(h2 @ d["wg"]) * (h2 @ d["wu"]))
    y = x2 + a @ d["wd"]
    return _packed(y, ("bf16", [_splits(c["t"], c["block"]), _splits(c["hidden"], c["block"])]))
