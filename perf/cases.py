"""The work of this library that its performance is measured on.

A user keeps each layer's KV cache and attention inputs in pinned host memory and decodes token by token.  The cases
are what such a program calls: one layer's decode (the latency path), one token through a stack of decoder layers with
the greedy step behind it (generation), the column schedule with the weights in host memory too (throughput), the
prefill stand-in that fills the store, and the entry points of the single kernels that serving code calls by
themselves: recompute GEMM, decode attention, 4-bit codec.  Shapes are those of the bench and the tests (hidden 768 to
7168, batch 1 to 64, contexts up to 4096), odd ones among them.

A case is a dict of plain values; "kind" says which entry points it takes.
"""
from __future__ import annotations

import ctypes
import math

import numpy as np
import torch

import paper_2411_17089_amd as kv

# hidden size -> (heads, head width); the widths the bench and the tests use
SHAPES = {768: (12, 64), 4096: (32, 128), 5120: (40, 128), 7168: (56, 128)}
LLAMA_FFN = {4096: 11008, 5120: 13824}
# the two rates of the cost model as the profiler reports them on this card; fixed, so that a plan depends on the case alone
LINK_BYTES_PER_S, GEMM_FLOPS_PER_S = 57.0e9, 1.25e15
STORE = {"f16": 0, "kv4": kv.KVPR_KV_INT4, "kv4x4": kv.KVPR_STORE_INT4}


def listed():
    return [
        # the smallest call: one attention block of the 768-wide test configuration, two short sequences
        {"name": "layer_768_b2_s96", "kind": "layer", "arch": "opt", "hidden": 768, "batch": 2, "seq": 96, "split": 40, "store": "f16"},
        # the bench's headline: the widest layer at batch 32, context 1024, at the split its plan gives
        {"name": "layer_7168_b32_s1024", "kind": "layer", "arch": "opt", "hidden": 7168, "batch": 32, "seq": 1024, "split": 768, "store": "f16"},
        # the 4-bit host store (cache and activations packed), at its planned split
        {"name": "layer_4096_int4_b32_s1024", "kind": "layer", "arch": "opt", "hidden": 4096, "batch": 32, "seq": 1024, "split": 576, "store": "kv4x4"},
        # interactive generation: one sequence, one token through decoder layers with resident weights, then the greedy step
        {"name": "token_4096_b1_s512", "kind": "token", "arch": "opt", "hidden": 4096, "batch": 1, "seq": 512, "layers": 4, "vocab": 50272, "granularity": 64},
        # the rotary family at an odd batch and an odd context, every split allowed
        {"name": "token_llama_4096_b3_s203", "kind": "token", "arch": "llama", "hidden": 4096, "batch": 3, "seq": 203, "layers": 3, "vocab": 32000, "granularity": 1},
        # throughput mode: weights in host memory as well, two GPU batches a layer, context of the bench's small-batch sweep
        {"name": "columns_4096_2xb4_s256", "kind": "columns", "arch": "opt", "hidden": 4096, "batch": 4, "seq": 256, "layers": 2, "gpu_batches": 2, "granularity": 64},
        # filling the store: prompt of 512 tokens, eight sequences
        {"name": "prefill_4096_b8_s512", "kind": "prefill", "arch": "opt", "hidden": 4096, "batch": 8, "seq": 512},
        # the recomputation of the headline layer by itself
        {"name": "gemm_7168_m24576", "kind": "gemm", "arch": "opt", "hidden": 7168, "batch": 32, "positions": 768},
        # ... and of a small ragged batch of the rotary family (1055 rows)
        {"name": "gemm_rope_5120_m1055", "kind": "gemm", "arch": "llama", "hidden": 5120, "batch": 5, "positions": 211},
        # attention over a batch of 32 at the bench's context
        {"name": "attention_5120_b32_s1025", "kind": "attention", "hidden": 5120, "batch": 32, "positions": 1025},
        # ... and over one long sequence
        {"name": "attention_4096_b1_s4097", "kind": "attention", "hidden": 4096, "batch": 1, "positions": 4097},
        # packing a 1024-position cache of 32 sequences and unpacking it again
        {"name": "codec_8192_r32768", "kind": "codec", "cols": 8192, "rows": 32768},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _plan_like(rng, hidden, seq):
    """A split near the one that balances the two arms of the cost model, sometimes well off it."""
    even = seq / (1.0 + hidden * LINK_BYTES_PER_S / GEMM_FLOPS_PER_S)
    return max(0, min(seq, int(even * rng.choice([1.0, 1.0, rng.uniform(0.3, 1.2)]))))


def draw(rng):
    """One more case.  Sizes stay within what the largest listed case of the same kind costs."""
    kind = rng.choice(["layer", "layer", "token", "token", "columns", "prefill", "gemm", "gemm", "attention", "attention", "codec"])
    arch = rng.choice(["opt", "llama"])
    hidden = rng.choice([4096, 5120] if arch == "llama" else [768, 4096, 5120, 7168])
    batch, seq = _log(rng, 1, 64), _log(rng, 40, 2048)
    fit = lambda halfs: max(16, min(seq, halfs // (batch * hidden)))          # noqa: E731  context so that a layer's X fits
    if kind == "layer":
        seq = fit(32 * 1024 * 7168)
        return {"kind": kind, "arch": arch, "hidden": hidden, "batch": batch, "seq": seq, "split": _plan_like(rng, hidden, seq),
                "store": rng.choice(["f16", "f16", "kv4", "kv4x4"])}
    if kind == "token":
        batch = min(batch, 32)
        hidden = min(hidden, 5120)
        layers = rng.randint(1, 4)
        seq = fit(32 * 1024 * 4096 // layers)
        return {"kind": kind, "arch": arch, "hidden": hidden, "batch": batch, "seq": seq, "layers": layers,
                "vocab": 32000 if arch == "llama" else 50272, "granularity": rng.choice([1, 64])}
    if kind == "columns":
        batch, hidden = min(batch, 32), min(hidden, 4096)
        seq = fit(4 * 1024 * 4096)
        return {"kind": kind, "arch": arch, "hidden": hidden, "batch": batch, "seq": seq, "layers": 2, "gpu_batches": rng.randint(1, 3),
                "granularity": rng.choice([1, 64])}
    if kind == "prefill":
        return {"kind": kind, "arch": arch, "hidden": hidden, "batch": batch, "seq": fit(16 * 512 * 4096)}
    if kind == "gemm":
        batch = min(batch, 32)
        return {"kind": kind, "arch": arch, "hidden": hidden, "batch": batch, "positions": max(1, min(seq, 24576 // batch))}
    if kind == "attention":
        hidden = rng.choice([768, 4096, 5120, 7168])
        return {"kind": kind, "hidden": hidden, "batch": batch, "positions": max(1, min(2 * seq + 1, 32 * 1025 * 7168 // (batch * hidden)))}
    cols = rng.choice([768, 4096, 5120, 8192, 10240, 14336])
    return {"kind": kind, "cols": cols, "rows": _log(rng, 1, 32768 * 8192 // cols)}


# ---- inputs ----

def _normal(g, shape, scale, mean=0.0):
    return (torch.randn(shape, generator=g, device="cuda", dtype=torch.float32) * scale + mean).half()


def _weights(g, arch, hidden, ffn):
    """Device parameters of one layer: weights N(0, 0.02), biases N(0, 0.01), norm gains around 1."""
    h = hidden
    t = {"wqkv": _normal(g, (3 * h, h), 0.02), "wo": _normal(g, (h, h), 0.02)}
    if arch == "opt":
        t.update(bqkv=_normal(g, (3 * h,), 0.01), bo=_normal(g, (h,), 0.01))
    if ffn:
        t.update(ln1_g=_normal(g, (h,), 0.05, 1.0), ln2_g=_normal(g, (h,), 0.05, 1.0),
                 w1=_normal(g, ((2 if arch == "llama" else 1) * ffn, h), 0.02), w2=_normal(g, (h, ffn), 0.02))
        if arch == "opt":
            t.update(ln1_b=_normal(g, (h,), 0.02), ln2_b=_normal(g, (h,), 0.02), b1=_normal(g, (ffn,), 0.01), b2=_normal(g, (h,), 0.01))
    return t


def _ffn(case):
    return LLAMA_FFN[case["hidden"]] if case["arch"] == "llama" else 4 * case["hidden"]


def _host(ctx, address, shape, dtype):
    """numpy view of pinned memory that a context owns; it keeps the context alive."""
    n = int(np.prod(shape)) * np.dtype(dtype).itemsize
    memory = (ctypes.c_ubyte * n).from_address(address)
    memory.owner = ctx
    return np.frombuffer(memory, dtype=dtype).reshape(shape)


class _Context:
    """A context and what has to live as long as it does."""

    def __init__(self, handle):
        self.handle = handle

    def __del__(self):
        kv.kvpr_destroy(self.handle)


def _context(case, layers, ffn, gpu_batches=0):
    heads, width = SHAPES[case["hidden"]]
    shape = (layers, case["hidden"], heads, width, ffn, case["batch"], case["seq"] + 2)
    more = {"dtype": kv.KVPR_F16 | STORE[case.get("store", "f16")], "arch": kv.KVPR_ARCH_LLAMA if case["arch"] == "llama" else kv.KVPR_ARCH_OPT}
    return _Context(kv.kvpr_create_offload(*shape, gpu_batches, **more) if gpu_batches else kv.kvpr_create(*shape, **more))


def _fill_store(case, ctx, slot, g, w):
    """Rows [0, seq) of a slot: activations N(0, 1) (what a norm layer gives), cache = their projection."""
    b, h, s = case["batch"], case["hidden"], case["seq"]
    x = torch.randn((s, b, h), generator=g, device="cuda", dtype=torch.float16)
    if case.get("store", "f16") == "kv4x4":
        kv.kvpr_store_write(ctx.handle, slot, 0, s, x.cpu(), None)
    else:
        torch.from_numpy(_host(ctx, kv.kvpr_store_ptrs(ctx.handle, slot)[0], (s, b, h), np.float16)).copy_(x)
    kv.kvpr_store_prefill_kv(ctx.handle, slot, s, w)


def _new_rows(case, ctx, slot):
    """Views of the host rows that a decode of this slot writes."""
    b, h, s = case["batch"], case["hidden"], case["seq"]
    rows = []
    for address, cols, packed in zip(kv.kvpr_store_ptrs(ctx.handle, slot), (h, 2 * h),
                                     (case.get("store") == "kv4x4", case.get("store", "f16") != "f16")):
        if packed:                                  # codes, then (scale, minimum) pairs, per sequence
            n = kv.kvpr_int4_row_bytes(cols)
            row = _host(ctx, address + s * b * n, (b, n), np.uint8)
            rows += [row[:, : cols // 2], row[:, cols // 2:].view(np.float16)]
        else:
            rows.append(_host(ctx, address + s * b * cols * 2, (b, cols), np.float16))
    return rows


def prepare(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    st = {"case": case}
    kind = case["kind"]
    if kind in ("layer", "prefill"):
        b, h = case["batch"], case["hidden"]
        st["tensors"] = _weights(g, case["arch"], h, 0)
        st["w"] = kv.make_weights(**st["tensors"])
        st["ctx"] = ctx = _context(case, 1, 0)
        _fill_store(case, ctx, 0, g, st["w"])
        st["x"] = _normal(g, (b, h), 1.0)
        st["out"] = torch.empty_like(st["x"])
        if kind == "layer":
            st["rows"] = _new_rows(case, ctx, 0)
        else:
            st["kv"] = _host(ctx, kv.kvpr_store_ptrs(ctx.handle, 0)[1], (case["seq"], b, 2 * h), np.float16)
    elif kind == "token":
        b, h, v = case["batch"], case["hidden"], case["vocab"]
        st["tensors"] = [_weights(g, case["arch"], h, _ffn(case)) for _ in range(case["layers"])]
        st["w"] = [kv.make_weights(**t) for t in st["tensors"]]
        st["ctx"] = ctx = _context(case, case["layers"], _ffn(case))
        for i, w in enumerate(st["w"]):
            _fill_store(case, ctx, i, g, w)
        kv.kvpr_set_profile(ctx.handle, kv.make_profile(LINK_BYTES_PER_S, GEMM_FLOPS_PER_S), kv.KVPR_COST_EQ10, case["granularity"])
        # output layer tied to the embedding, as this family ties them; the token's own embedding is the input
        st["emb"] = _normal(g, (v, h), 1.0)
        st["x"] = st["emb"][torch.randint(0, v, (b,), generator=g, device="cuda")].contiguous()
        st["x_out"], st["x_next"] = torch.empty_like(st["x"]), torch.empty_like(st["x"])
        st["logits"] = torch.empty((b, v), dtype=torch.float32, device="cuda")
        st["tokens"] = torch.empty((b,), dtype=torch.int32, device="cuda")
        st["rows"] = [_new_rows(case, ctx, i) for i in range(case["layers"])]
    elif kind == "columns":
        b, h, nb = case["batch"], case["hidden"], case["gpu_batches"]
        st["ctx"] = ctx = _context(case, case["layers"], _ffn(case), nb)
        for j in range(case["layers"]):
            t = _weights(g, case["arch"], h, _ffn(case))
            kv.kvpr_weights_write(ctx.handle, j, kv.make_weights(**(host := {n: a.cpu() for n, a in t.items()})))
            for q in range(nb):
                _fill_store(case, ctx, j * nb + q, g, kv.make_weights(**t))
            del t, host
        kv.kvpr_set_profile(ctx.handle, kv.make_profile(LINK_BYTES_PER_S, GEMM_FLOPS_PER_S), kv.KVPR_COST_EQ10, case["granularity"])
        st["slots"] = case["layers"] * nb
        st["x"] = _normal(g, (nb, b, h), 1.0)
        st["x_out"] = torch.empty_like(st["x"])
        st["rows"] = [_new_rows(case, ctx, i) for i in range(st["slots"])]
    elif kind == "gemm":
        h, b, n = case["hidden"], case["batch"], case["positions"]
        st["a"] = torch.randn((n * b, h), generator=g, device="cuda", dtype=torch.float16)
        st["wkv"], st["out"] = _normal(g, (2 * h, h), 0.02), torch.empty((n * b, 2 * h), dtype=torch.float16, device="cuda")
        if case["arch"] == "llama":
            st["table"] = torch.from_numpy(kv.kvpr_rope_table(n + 1, SHAPES[h][1])).cuda()
        else:
            st["bias"] = _normal(g, (2 * h,), 0.01)
    elif kind == "attention":
        h, b, n = case["hidden"], case["batch"], case["positions"]
        # q and K as projections of N(0, 1) activations by N(0, 0.02) weights give them
        spread = 0.02 * math.sqrt(h)
        st["q"] = torch.randn((b, h), generator=g, device="cuda") * spread
        st["kv"] = torch.randn((n, b, 2 * h), generator=g, device="cuda", dtype=torch.float16).mul_(spread)
        st["z"] = torch.empty((b, h), dtype=torch.float16, device="cuda")
        st["ws"] = torch.empty(kv.kvpr_attention_workspace_bytes(b, h, SHAPES[h][0], n), dtype=torch.uint8, device="cuda")
    else:
        rows, cols = case["rows"], case["cols"]
        st["src"] = torch.randn((rows, cols), generator=g, device="cuda", dtype=torch.float16)
        st["packed"] = torch.empty((rows, kv.kvpr_int4_row_bytes(cols)), dtype=torch.uint8, device="cuda")
        st["back"] = torch.empty_like(st["src"])
    return st


# ---- one pass ----

def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "layer":
        kv.kvpr_layer_decode(st["ctx"].handle, 0, case["seq"], case["split"], st["w"], st["x"], st["out"])
        return {"out": st["out"], "rows": st["rows"]}
    if kind == "token":
        kv.kvpr_decode_step(st["ctx"].handle, case["seq"], st["w"], st["x"], st["x_out"])
        kv.kvpr_greedy_next(st["x_out"], st["emb"], st["emb"], case["batch"], case["hidden"], case["vocab"], st["logits"], st["tokens"], st["x_next"])
        return {"hidden": st["x_out"], "logits": st["logits"], "tokens": st["tokens"], "next": st["x_next"], "rows": st["rows"]}
    if kind == "columns":
        kv.kvpr_decode_step_columns(st["ctx"].handle, case["seq"], st["slots"], st["x"], st["x_out"])
        return {"hidden": st["x_out"], "rows": st["rows"]}
    if kind == "prefill":
        kv.kvpr_store_prefill_kv(st["ctx"].handle, 0, case["seq"], st["w"])
        return st["kv"]
    if kind == "gemm":
        h, m = case["hidden"], case["positions"] * case["batch"]
        if case["arch"] == "llama":
            kv.kvpr_recompute_gemm_rope(st["a"], st["wkv"], None, st["out"], m, 2 * h, h, 2 * h, st["table"], case["positions"] + 1, h,
                                        SHAPES[h][1], case["batch"], 0)
        else:
            kv.kvpr_recompute_gemm(st["a"], st["wkv"], st["bias"], st["out"], m, 2 * h, h, 2 * h)
        return st["out"]
    if kind == "attention":
        h = case["hidden"]
        kv.kvpr_decode_attention(st["q"], st["kv"], st["z"], st["ws"], case["positions"], case["batch"], h, SHAPES[h][0])
        return st["z"]
    kv.kvpr_quant_int4(st["src"], st["packed"], case["rows"], case["cols"])
    kv.kvpr_dequant_int4(st["packed"], st["back"], case["rows"], case["cols"])
    return {"packed": st["packed"], "values": st["back"]}


# ---- what a pass cannot do without ----

def _attention_block(case, split):
    """(bytes, flops) of one layer's attention block without its weights: host rows in, the new row out; recomputation,
    projections, attention."""
    b, h, s = case["batch"], case["hidden"], case["seq"]
    store = case.get("store", "f16")
    x = b * (9 * h // 16 if store == "kv4x4" else 2 * h)
    c = b * (9 * h // 8 if store != "f16" else 4 * h)
    return (split * x + (s - split) * c + x + c,
            4.0 * b * split * h * h + 8.0 * b * h * h + 4.0 * b * h * (s + 1))


def _planned(case):
    p = kv.make_profile(LINK_BYTES_PER_S, GEMM_FLOPS_PER_S)
    return kv.kvpr_plan_split(p, kv.KVPR_COST_EQ10, case["batch"], case["seq"], case["hidden"], granularity=case["granularity"])[0]


def work(case):
    kind = case["kind"]
    if kind == "codec":
        n = case["rows"] * case["cols"]
        return {"bytes": n * 2 + 2 * (n * 9 // 16) + n * 2, "flops": 4.0 * n}
    h, b = case["hidden"], case["batch"]
    if kind == "gemm":
        m = case["positions"] * b
        return {"bytes": 2 * (m * h + 2 * h * h + 2 * m * h), "flops": 4.0 * m * h * h}
    if kind == "attention":
        n = case["positions"]
        return {"bytes": n * b * 4 * h + b * h * 6, "flops": 4.0 * n * b * h}
    if kind == "prefill":
        m = case["seq"] * b
        return {"bytes": 2 * (m * h + 2 * h * h + 2 * m * h), "flops": 4.0 * m * h * h}
    if kind == "layer":
        byt, flo = _attention_block(case, case["split"])
        return {"bytes": byt + 8 * h * h + 4 * b * h, "flops": flo}
    byt, flo = _attention_block(case, _planned(case))
    f = _ffn(case) * (3 if case["arch"] == "llama" else 2)              # FFN weights per hidden column
    layer_w = 2 * (4 * h * h + f * h)
    flo += 2.0 * b * f * h
    if kind == "columns":
        nb, n = case["gpu_batches"], case["layers"]
        return {"bytes": n * (layer_w + nb * byt) + 4 * nb * b * h, "flops": n * nb * flo}
    n, v = case["layers"], case["vocab"]
    return {"bytes": n * (layer_w + byt) + 2 * v * h + 4 * b * v + 6 * b * h, "flops": n * flo + 2.0 * b * v * h}


def tolerance(case):
    """About four times how far the float16 results are from the same path in 64 bits (relative 2-norm, then the largest
    single difference): 2.1e-4, 4.9e-4 where one kernel's float32 sums are rounded once; 5.3e-4, 2.0e-3 for an attention
    block, whose z is rounded before the output projection; 1.6e-3, 8e-3 for four decoder layers.  Whole values are codes
    of the packed rows (a value next to a rounding boundary may fall either way) and tokens."""
    kind = case["kind"]
    if kind == "codec":
        return "exact"
    if kind in ("gemm", "attention", "prefill"):
        return {"rel": 8e-4, "max": 2e-3}
    if kind == "layer":
        return {"rel": 2e-3, "max": 8e-3, "differ": 2e-3}
    return {"rel": 6e-3, "max": 3e-2, "differ": 2e-3}
