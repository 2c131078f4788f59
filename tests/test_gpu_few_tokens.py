"""Token GEMM for at most 8 rows: K in fewer pieces than waves, in even and uneven runs, in several segments and in runs of
4 KiB; outputs that are no multiple of 4, fewer than 4, and more than one workgroup's sums can hold."""
import numpy as np
import pytest
import torch

import kvpr_inputs
from oracle import kvpr_llama_oracle as lo
from kvpr_testlib import dev, rel_err
from test_gpu_llama import _lib_arrays, _llama_params

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def k():
    import paper_2411_17089_amd as k
    return k


@pytest.mark.parametrize("M", [1, 4, 5, 8])
@pytest.mark.parametrize("N,K,f32", [(3, 128, 0), (520, 768, 8), (1301, 1152, 1024), (1026, 2048, 0), (64, 7168, 64), (260, 7296, 0),
                                     (132, 8320, 4), (132, 11008, 0), (40, 16384, 8), (24, 32768, 0), (140000, 256, 0)])
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


@pytest.mark.parametrize("b,ffn", [(3, 128), (4, 384), (5, 1152), (8, 11008)])
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
