"""Token GEMM for at most 8 rows, with the norm in front and the rotation behind: K in fewer pieces than waves, in even and uneven runs, in several segments and in runs of
4 KiB; outputs that are no multiple of 4, fewer than 4, and more than one workgroup's sums can hold.  (Of less than 1024 columns the
kernels for up to 64 rows take the products with 5 to 8 rows, and the narrow ones with fewer.)"""
import ctypes

import numpy as np
import pytest
import torch

import kvpr_inputs
from oracle import kvpr_llama_oracle as lo
from oracle import kvpr_oracle as ko
from kvpr_testlib import dev, rel_err, upload_layer
from test_gpu_llama import _lib_arrays, _llama_params

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def k():
    import paper_2411_17089_amd as k
    return k


@pytest.mark.parametrize("M", [1, 4, 5, 8])
@pytest.mark.parametrize("N,K,f32", [(3, 128, 0), (520, 768, 8), (1301, 1152, 1024), (1026, 2048, 0), (64, 7168, 64), (260, 7296, 0),
                                     (132, 8320, 4), (132, 11008, 0), (40, 16384, 8), (24, 32768, 0), (65536, 1024, 0), (140000, 256, 0)])
def test_product(k, M, N, K, f32):
    print(f"few tokens M={M} N={N} K={K} f32={f32}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(M * 1000 + N)
    x = torch.randn((M, K), generator=g, device="cuda").half()
    W = (torch.randn((N, K), generator=g, device="cuda") * 0.05).half()
    bias = (torch.randn((N,), generator=g, device="cuda") * 0.1).half()
    ld16 = N - f32 + 3
    y32 = torch.full((M, max(f32, 1)), float("nan"), dtype=torch.float32, device="cuda")
    y16 = torch.full((M, ld16), float("nan"), dtype=torch.float16, device="cuda")
    k.kvpr_token_gemm(x, W, bias, y32, y16, M, N, K, f32, ld16)
    torch.cuda.synchronize()
    want = x.double() @ W.double().T + bias.double()
    # float32 sums of K products in any order, then one rounding to float16 where that is the output
    sums = K * 2.0 ** -24 * (x.double().abs() @ W.double().abs().T + bias.double().abs())
    if f32:
        assert bool(((y32.double() - want[:, :f32]).abs() <= sums[:, :f32]).all())
    got = y16[:, : N - f32].double()
    assert bool(((got - want[:, f32:]).abs() <= sums[:, f32:] + 2.0 ** -11 * want[:, f32:].abs() + 2.0 ** -24).all())
    assert bool(torch.isnan(y16[:, N - f32:]).all()), "columns beyond the last feature must not be written"


@pytest.mark.parametrize("N,K", [(8192, 768), (8256, 768), (8300, 640), (8256, 512), (2304, 896)])
def test_product_of_few_columns(k, N, K):
    """Both sides of the rule for a product of less than 1024 columns."""
    for M in (1, 4):
        test_product(k, M, N, K, 8)


@pytest.mark.parametrize("b,ffn", [(3, 128), (4, 384), (5, 1152), (8, 11008), (8, 32768)])
def test_gated_decoder_layer(k, b, ffn):
    s, h, H = 12, 256, 2
    P = _llama_params(300 + b, b, h, H, ffn)
    layer = dict(P, X=kvpr_inputs._draw(np.random.default_rng(b), (s, b, h), 1.0))
    stored = lo.stored_kv(layer, "fp16").astype(np.float16)
    x = kvpr_inputs._draw(np.random.default_rng(ffn), (b, h), 1.0)
    d = {n: dev(a) for n, a in _lib_arrays(P).items()}
    ctx = k.kvpr_create(1, h, H, h // H, ffn, b, s + 2, arch=k.KVPR_ARCH_LLAMA)
    try:
        k.kvpr_store_write(ctx, 0, 0, s, np.ascontiguousarray(layer["X"]), stored)
        out = torch.empty((b, h), dtype=torch.float16, device="cuda")
        k.kvpr_decode_step(ctx, s, [k.make_weights(**d)], dev(x), out, [5])
        torch.cuda.synchronize()
        want = lo.decoder_stack_decode([layer], x, [5], [stored])[0]
        # gate, up, their product and the result are rounded to float16 (2^-11 each), as in the oracle; sums in another order
        assert rel_err(out.cpu().numpy(), want) <= 5e-3
    finally:
        k.kvpr_destroy(ctx)


# hidden 256: waves without columns; 1152: runs of 1 and 2 pieces; 2176: 2 and 3.  9 rows: the norm is a launch of its own
@pytest.mark.parametrize("h,H", [(256, 4), (1152, 9), (2176, 17)])
@pytest.mark.parametrize("b", [1, 4, 5, 8, 9])
@pytest.mark.parametrize("arch", ["opt", "llama"])
def test_norm_and_rotation_in_the_projection(k, arch, h, H, b):
    print(f"norm along arch={arch} h={h} b={b}", flush=True)
    s, ffn, llama = 7, 384, arch == "llama"
    if llama:
        P = _llama_params(70 + b, b, h, H, ffn)
        layer = dict(P, X=kvpr_inputs._draw(np.random.default_rng(b), (s, b, h), 1.0))
        stored, d = lo.stored_kv(layer, "fp16"), {n: dev(a) for n, a in _lib_arrays(P).items()}
    else:
        layer = dict(kvpr_inputs.make_layer(70 + b, b, s, h, H), **kvpr_inputs.make_ffn(70 + b, h, ffn))
        up = upload_layer(layer)
        stored, d = ko.stored_kv(layer, "fp16"), {n: up[n] for n in ("wqkv", "bqkv", "wo", "bo", "ln1_g", "ln1_b", "w1", "b1", "w2", "b2", "ln2_g", "ln2_b")}
    x = kvpr_inputs._draw(np.random.default_rng(h), (b, h), 1.0)
    want = (lo if llama else ko).decoder_stack_decode([layer], x, [3], [stored])[0]
    shifted = torch.empty((b * h + 1,), dtype=torch.float16, device="cuda")      # rows that start off a 16-byte boundary
    shifted[1:] = dev(x).view(-1)
    for x_in in (dev(x), shifted[1:].view(b, h)):
        ctx = k.kvpr_create(1, h, H, h // H, ffn, b, s + 2, arch=k.KVPR_ARCH_LLAMA if llama else k.KVPR_ARCH_OPT)
        try:
            k.kvpr_store_write(ctx, 0, 0, s, np.ascontiguousarray(layer["X"]), stored.astype(np.float16))
            outs = []
            for timing in (False, True):
                out = torch.empty((b, h), dtype=torch.float16, device="cuda")
                k.kvpr_decode_step(ctx, s, [k.make_weights(**d)], x_in, out, [3], timing=timing)
                torch.cuda.synchronize()
                outs.append(out.cpu().numpy())
            assert np.array_equal(outs[0], outs[1])
            assert rel_err(outs[0], want) <= 5e-3                                # the bound of the stack tests
            # the row that goes to the store: norm and rotation, one rounding each (3e-3, 5e-3 as in the stack tests)
            xp, kvp = k.kvpr_store_ptrs(ctx, 0)
            view = lambda p, n: np.ctypeslib.as_array(ctypes.cast(p, ctypes.POINTER(ctypes.c_uint16)), ((s + 1) * n,)).view(np.float16).reshape(s + 1, n)   # noqa: E731
            trace = (lo if llama else ko).decoder_stack_decode([layer], x, [3], [stored])[1][0]
            assert rel_err(view(xp, b * h)[s], np.asarray(trace["xn"]).reshape(-1)) <= 3e-3
            assert rel_err(view(kvp, b * 2 * h)[s], np.asarray(trace["kv_new"]).reshape(-1)) <= 5e-3
        finally:
            k.kvpr_destroy(ctx)


def _ffn_only(k, arch, b, h, width, ffn, seed):
    """One decoder layer whose attention block adds nothing (Wo = 0): result, stored rows of the new token, and what float64 gives for
    them with the roundings to float16 where the library rounds."""
    s, llama = 5, arch == "llama"
    g = torch.Generator(device="cuda").manual_seed(seed)
    rand = lambda *shape, scale, mean=0.0: (torch.randn(shape, generator=g, device="cuda") * scale + mean).half()   # noqa: E731
    w = {"wqkv": rand(3 * h, h, scale=0.02), "wo": torch.zeros((h, h), dtype=torch.float16, device="cuda"), "ln1_g": rand(h, scale=0.05, mean=1.0),
         "ln2_g": rand(h, scale=0.05, mean=1.0), "w1": rand((2 if llama else 1) * ffn, h, scale=0.02), "w2": rand(h, ffn, scale=0.02)}
    if not llama:
        w.update(bqkv=rand(3 * h, scale=0.1), ln1_b=rand(h, scale=0.02), ln2_b=rand(h, scale=0.02), b1=rand(ffn, scale=0.1), b2=rand(h, scale=0.1))
    x, rows = rand(b, h, scale=1.0), rand(s, b, h, scale=1.0).cpu().numpy()
    ctx = k.kvpr_create(1, h, h // width, width, ffn, b, s + 2, arch=k.KVPR_ARCH_LLAMA if llama else k.KVPR_ARCH_OPT)
    try:
        k.kvpr_store_write(ctx, 0, 0, s, rows, None)
        k.kvpr_store_prefill_kv(ctx, 0, s, k.make_weights(**w))
        out = torch.full((b, h), float("nan"), dtype=torch.float16, device="cuda")
        k.kvpr_decode_step(ctx, s, [k.make_weights(**w)], x, out, [3])
        torch.cuda.synchronize()
        xp, kvp = k.kvpr_store_ptrs(ctx, 0)
        row = lambda p, n: torch.from_numpy(np.frombuffer((ctypes.c_ubyte * (b * n * 2)).from_address(p + s * b * n * 2), np.float16).copy().reshape(b, n)).cuda()   # noqa: E731
        xn, kv_new = row(xp, h), row(kvp, 2 * h)
    finally:
        k.kvpr_destroy(ctx)
    d = {n: t.double() for n, t in w.items()}
    half = lambda t: t.half().double()   # noqa: E731

    def norm(i):
        t = x.double()
        t = t if llama else t - t.mean(1, keepdim=True)
        t = t * torch.rsqrt((t * t).mean(1, keepdim=True) + 1e-5) * d[f"ln{i}_g"]
        return t if llama else t + d[f"ln{i}_b"]
    a = half(norm(2)) @ d["w1"].T
    if llama:
        gate, up = half(a[:, :ffn]), half(a[:, ffn:])
        a = half(gate / (1.0 + torch.exp(-gate)) * up)
    else:
        a = half(torch.relu(a + d["b1"]))
    want = x.double() + half(a @ d["w2"].T + (0.0 if llama else d["b2"]))
    wv, bv = d["wqkv"][2 * h:], torch.zeros(h, device="cuda").double() if llama else d["bqkv"][2 * h:]
    v = xn.double() @ wv.T + bv
    sums = h * 2.0 ** -24 * (xn.double().abs() @ wv.abs().T + bv.abs())         # float32 sums of h products in any order
    return out.double(), want, xn.double(), norm(1), kv_new[:, h:].double(), v, sums


def _check_ffn_only(out, want, xn, xn_want, v, v_want, sums):
    # one rounding to float16; mean and variance of up to 8192 values of order 1 in float32, and four operations of 2^-24 on values
    # up to 6 (2e-5 is eight times that)
    assert bool(((xn - xn_want).abs() <= (2.0 ** -11 + 1e-5) * xn_want.abs() + 2e-5).all())
    # a product with the row that was stored, one rounding
    assert bool(((v - v_want).abs() <= sums + 2.0 ** -11 * v_want.abs() + 2.0 ** -24).all())
    # a value next to a rounding boundary may fall either way: 2^-11 of a normalised value or an activation, summed over the features
    assert rel_err(out.cpu().numpy(), want.cpu().numpy()) <= 5e-3                # the bound of the stack tests


@pytest.mark.parametrize("h", [4096, 5120, 6144, 7168, 8192])                    # 4 to 8 pieces of K a wave
@pytest.mark.parametrize("b", [1, 4, 5, 8])
@pytest.mark.parametrize("arch", ["opt", "llama"])
def test_norm_along_with_wide_rows(k, arch, h, b):
    print(f"norm along, wide rows: {arch} h={h} b={b}", flush=True)
    _check_ffn_only(*_ffn_only(k, arch, b, h, 128, 256, h + b))


# hidden 1024 and more: with 5 to 8 rows too the gated product is the kernel's.  63616 features are 63 units of rows for each of 256
# compute units: two workgroups of 32 would need more LDS than a launch gets
@pytest.mark.parametrize("h,ffn", [(1024, 128), (1152, 1152), (1024, 63616), (5120, 13824)])
@pytest.mark.parametrize("b", [4, 5, 8])
def test_gated_product(k, b, h, ffn):
    print(f"gated product h={h} ffn={ffn} b={b}", flush=True)
    _check_ffn_only(*_ffn_only(k, "llama", b, h, 128, ffn, ffn + b))
