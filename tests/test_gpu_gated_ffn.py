"""Gated FFN in one launch: the smallest width of its range and the one below it (two launches), every row-tile count."""
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


@pytest.mark.parametrize("ffn", [9088, 9216])
@pytest.mark.parametrize("b", [1, 17, 33, 64])
def test_decoder_layer(k, b, ffn):
    s, h, H = 12, 256, 2
    P = _llama_params(900 + b, b, h, H, ffn)
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
