"""The layer pipeline where layers stream enough weights for the recomputation to run beside the previous one: ordering against
what the caller enqueued before the step, against the reuse of the two device buffers and between tokens, bit for bit against
the same steps waited for; per-layer timings and run-time adaptation; writes to the store behind a decode."""
import ctypes

import numpy as np
import pytest
import torch

import kvpr_inputs
from kvpr_testlib import dev, upload_layer

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def k():
    import paper_2411_17089_amd as k
    return k


class BigLayers:
    """A stack whose layers stream enough weights (more than 128 MB of FFN and output projection) for a recomputation of a few
    hundred rows to run beside them."""

    def __init__(self, k, arch, L, b, s, packed=False, seed=0):
        self.k, self.L, self.b, self.s, self.h, H = k, L, b, s, 1024, 8
        h, llama = self.h, arch == "llama"
        ffn = 20736 if llama else 31104
        g = torch.Generator(device="cuda").manual_seed(seed)
        self.t = t = lambda *shape, scale=0.02, mean=0.0: (torch.randn(shape, generator=g, device="cuda") * scale + mean).half()   # noqa: E731
        self.params, self.w = [], []
        for _ in range(L):
            d = dict(wqkv=t(3 * h, h), wo=t(h, h), ln1_g=t(h, mean=1.0), ln2_g=t(h, mean=1.0), w1=t((2 if llama else 1) * ffn, h), w2=t(h, ffn))
            if not llama:
                d.update(bqkv=t(3 * h), bo=t(h), ln1_b=t(h), ln2_b=t(h), b1=t(ffn), b2=t(h))
            self.params.append(d)
            self.w.append(k.make_weights(**d))
        self.ctx = k.kvpr_create(L, h, H, h // H, ffn, b, s + 4, dtype=k.KVPR_F16 | (k.KVPR_STORE_INT4 if packed else 0),
                                 arch=k.KVPR_ARCH_LLAMA if llama else k.KVPR_ARCH_OPT)
        for i in range(L):
            k.kvpr_store_write(self.ctx, i, 0, s, t(s, b, h, scale=1.0).cpu(), None)
            k.kvpr_store_prefill_kv(self.ctx, i, s, self.w[i])
        self.row_bytes = [b * (k.kvpr_int4_row_bytes(c) if packed else 2 * c) for c in (h, 2 * h)]

    def ahead(self):
        f = self.k.lib.kvpr_debug_layers_ahead
        f.restype, f.argtypes = ctypes.c_int64, [ctypes.c_void_p]
        return f(self.ctx)


@pytest.mark.parametrize("b,s", [(16, 40), (64, 10)])         # new rows stored on the compute stream, on the store stream
@pytest.mark.parametrize("poison", [False, True])
@pytest.mark.parametrize("arch,store,chunks", [("opt", "f16", 1), ("opt", "int4", 1), ("llama", "f16", 1), ("llama", "int4", 1), ("opt", "f16", 3), ("llama", "int4", 3)])
def test_tokens_back_to_back(k, arch, store, chunks, poison, b, s):
    """Three tokens enqueued one behind the other give what the same tokens give one at a time, outputs and host rows: the
    second reads the rows the first one stored, buffers and scratch rows are used again without a wait in between.  Most
    layers recompute beside the previous one; the weights are written just before the first step."""
    st = BigLayers(k, arch, 3, b, s, store == "int4", seed=b)
    h = st.h
    try:
        rows = [np.frombuffer((ctypes.c_ubyte * (3 * n)).from_address(a + s * n), np.uint8)
                for i in range(3) for a, n in zip(k.kvpr_store_ptrs(st.ctx, i), st.row_bytes)]
        xs = [st.t(b, h, scale=1.0) for _ in range(3)]
        splits = [[s - 1, s - 2, s], [s, s + 1, s - 1], [0, s + 2, s + 1]]
        final = [d["wqkv"].clone() for d in st.params]
        big = torch.randn(4096, 4096, device="cuda")
        k.kvpr_set_chunks(st.ctx, chunks)
        k.kvpr_set_debug(st.ctx, k.KVPR_DEBUG_POISON if poison else 0)
        got, before = {}, st.ahead()
        for mode in ("waited", "free", "free again"):
            for r in rows:
                r.setflags(write=True)
                r[:] = 0xFF                                     # NaN, packed or not
            outs = [torch.full((b, h), float("nan"), dtype=torch.float16, device="cuda") for _ in range(3)]
            for d in st.params:
                d["wqkv"].fill_(float("nan"))
            torch.cuda.synchronize()
            for _ in range(8):                                  # some milliseconds on the compute stream
                big = big @ big
                big /= big.abs().max()
            for d, f in zip(st.params, final):
                d["wqkv"].copy_(f)
            for j in range(3):
                if mode == "waited":
                    torch.cuda.synchronize()
                k.kvpr_decode_step(st.ctx, s + j, st.w, xs[j], outs[j], splits[j])
            torch.cuda.synchronize()
            got[mode] = [o.cpu().numpy() for o in outs] + [r.copy() for r in rows]
        assert st.ahead() - before == 3 * 8, "all but the split of nothing"
        assert all(np.isfinite(o.astype(np.float32)).all() for o in got["waited"][:3])
        for mode in ("free", "free again"):
            for a, w in zip(got[mode], got["waited"]):
                assert np.array_equal(a, w), mode
        # in line, as a timed step runs: the same bits again
        outs = [torch.empty((b, h), dtype=torch.float16, device="cuda") for _ in range(3)]
        before = st.ahead()
        for j in range(3):
            k.kvpr_decode_step(st.ctx, s + j, st.w, xs[j], outs[j], splits[j], timing=True)
        assert st.ahead() == before
        for o, w in zip(outs, got["waited"]):
            assert np.array_equal(o.cpu().numpy(), w)
    finally:
        k.kvpr_destroy(st.ctx)


@pytest.mark.parametrize("b,s", [(16, 40), (64, 10)])
def test_layer_timings_hang_together(k, b, s):
    """Times from a layer's first enqueue are not negative, the recomputation lies inside what assembles the cache, and that
    inside the layer: also where the link is ahead and a layer's inputs have landed before its turn."""
    st = BigLayers(k, "opt", 4, b, s, seed=1)
    try:
        x, out = st.t(b, st.h, scale=1.0), torch.empty((b, st.h), dtype=torch.float16, device="cuda")
        for splits in ([s - 1] * 4, [s] * 4, [5, s, 8, s]):
            for _ in range(3):
                _, tim = k.kvpr_decode_step(st.ctx, s, st.w, x, out, splits, timing=True)
                for i, t in enumerate(tim):
                    print(b, splits[i], i, "start %.4f recompute %.4f assemble %.4f total %.4f" % (t.ms_recompute_start, t.ms_recompute, t.ms_assemble, t.ms_total))
                    eps = 1e-3                                  # events are read to about a tenth of a microsecond
                    assert t.ms_recompute_start >= 0 and t.ms_recompute > 0
                    assert t.ms_recompute_start + t.ms_recompute <= t.ms_assemble + eps
                    assert t.ms_assemble <= t.ms_total + eps
    finally:
        k.kvpr_destroy(st.ctx)


def test_adaptation_in_a_stack_sees_the_product_alone(k):
    """The recomputation rate that a stack's layers report is that of the product, as single-layer calls report it, and not of
    a product that shares the chip with another layer."""
    L, b, s = 4, 16, 40
    st = BigLayers(k, "opt", L, b, s, seed=2)
    try:
        x, out = st.t(b, st.h, scale=1.0), torch.empty((b, st.h), dtype=torch.float16, device="cuda")
        rate, before = {}, st.ahead()
        for mode in ("layer", "stack", "layer", "stack"):
            for _ in range(12):
                k.kvpr_set_adaptive(st.ctx, 0.0)
                k.kvpr_set_profile(st.ctx, k.make_profile(57e9, 5e14), k.KVPR_COST_EQ10, 64)
                k.kvpr_set_adaptive(st.ctx, 1.0)
                if mode == "layer":
                    k.kvpr_layer_decode(st.ctx, 0, s, s, st.w[0], x, out)
                else:
                    k.kvpr_decode_step(st.ctx, s, st.w, x, out, [s] * L)
                torch.cuda.synchronize()
                rate.setdefault(mode, []).append(k.kvpr_get_profile(st.ctx).gemm_flops_per_s)       # alpha = 1: the last sample
        assert st.ahead() - before == 24 * (L - 1), "all but the first layer of a step"
        layer, stack = np.median(rate["layer"]), np.median(rate["stack"])
        print("recomputation rate, TFLOP/s: single-layer calls %.0f, stack %.0f" % (layer / 1e12, stack / 1e12))
        assert stack >= 0.85 * layer                            # the same launches; in a stack the clocks are no lower
    finally:
        k.kvpr_destroy(st.ctx)


@pytest.mark.parametrize("b,h,H", [(4, 512, 4), (64, 1024, 8)])     # new rows stored on the compute stream, on the store stream
def test_store_write_waits_for_decodes_only(k, b, h, H):
    """A row written right behind the decode that stores it holds what was written last, and the call does not wait for what
    the caller enqueued on the compute stream behind the decode."""
    s = 40
    L = kvpr_inputs.make_layer(760, b, s, h, H)
    d = upload_layer(L)
    w = k.make_weights(**{f: d[f] for f in ("wqkv", "bqkv", "wo", "bo")})
    ctx = k.kvpr_create(2, h, H, h // H, 0, b, s + 3)
    try:
        for i in range(2):
            k.kvpr_store_write(ctx, i, 0, s, np.ascontiguousarray(L["X"]), None)
            k.kvpr_store_prefill_kv(ctx, i, s, w)
        row_x, row_kv = np.full((1, b, h), 3.0, np.float16), np.full((1, b, 2 * h), 5.0, np.float16)
        out = torch.empty((b, h), dtype=torch.float16, device="cuda")
        big, done = torch.randn(8192, 8192, device="cuda"), torch.cuda.Event()
        big @ big
        torch.cuda.synchronize()
        for _ in range(3):
            for i in range(2):
                k.kvpr_layer_decode(ctx, i, s, s // 2, w, d["x_new"], out)
            for _ in range(20):                                     # some 200 ms
                big @ big
            done.record()
            k.kvpr_store_write(ctx, 1, s, s + 1, row_x, row_kv)
            early = not done.query()
            torch.cuda.synchronize()
            x, kv = (np.frombuffer((ctypes.c_ubyte * (b * c * 2)).from_address(a + s * b * c * 2), np.float16)
                     for a, c in zip(k.kvpr_store_ptrs(ctx, 1), (h, 2 * h)))
            assert (x == 3.0).all() and (kv == 5.0).all()
            assert early, "the call waited for unrelated work"
    finally:
        k.kvpr_destroy(ctx)
