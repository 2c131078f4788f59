"""How a layer was enqueued: in order on the compute stream or on three streams, where the cache comes in and where the new rows go
out, on both sides of the rules (256 compute units)."""
import numpy as np
import pytest
import torch

from kvpr_testlib import dev

pytestmark = pytest.mark.gpu
IN_ORDER, CACHE_BESIDE_RECOMPUTE, ROWS_BESIDE_ATTENTION = 1, 2, 4


@pytest.fixture(scope="module")
def k():
    import paper_2411_17089_amd as k
    return k


def _context(k, b, h, H, s, flags=0, ffn=0, layers=1):
    rng = np.random.default_rng(h + b)
    arrays = {"wqkv": rng.standard_normal((3 * h, h)) * 0.02, "wo": rng.standard_normal((h, h)) * 0.02}
    if ffn:
        arrays.update(ln1_g=np.ones(h), ln1_b=np.zeros(h), ln2_g=np.ones(h), ln2_b=np.zeros(h), w1=rng.standard_normal((ffn, h)) * 0.02, w2=rng.standard_normal((h, ffn)) * 0.02)
    w = {n: dev(a.astype(np.float16)) for n, a in arrays.items()}
    ctx = k.kvpr_create(layers, h, H, h // H, ffn, b, s + 2, dtype=k.KVPR_F16 | flags)
    x = rng.standard_normal((s, b, h)).astype(np.float16)
    for i in range(layers):
        k.kvpr_store_write(ctx, i, 0, s, x, None)
        k.kvpr_store_prefill_kv(ctx, i, s, k.make_weights(**w))
    return ctx, w, dev(rng.standard_normal((b, h)).astype(np.float16)), torch.empty((b, h), dtype=torch.float16, device="cuda")


ALL = IN_ORDER | CACHE_BESIDE_RECOMPUTE | ROWS_BESIDE_ATTENTION
BESIDE_PROJECTION = IN_ORDER | ROWS_BESIDE_ATTENTION


@pytest.mark.parametrize("b,h,H,s,l,mode", [
    (2, 768, 12, 96, 40, ALL), (2, 768, 12, 96, 0, BESIDE_PROJECTION), (56, 768, 12, 20, 10, ALL), (64, 768, 12, 20, 10, 0),
    (4, 1024, 8, 60, 60, ALL), (8, 1024, 8, 300, 50, ALL), (8, 1024, 8, 700, 100, 0), (3, 768, 12, 4000, 1000, 0), (1, 768, 12, 6000, 4000, BESIDE_PROJECTION),
    (8, 2048, 16, 40, 20, ALL), (4, 4096, 32, 100, 50, BESIDE_PROJECTION), (8, 4096, 32, 300, 100, 0),
    (3, 7168, 56, 40, 40, ALL), (3, 7168, 56, 217, 217, 0),                   # parts gain more
    (6, 7168, 56, 20, 0, BESIDE_PROJECTION), (6, 7168, 56, 50, 0, 0)])        # cache alone behind a long projection
def test_single_layer_call(k, b, h, H, s, l, mode):
    print(f"mode b={b} h={h} s={s} l={l}", flush=True)
    ctx, w, x, out = _context(k, b, h, H, s)
    try:
        k.kvpr_layer_decode(ctx, 0, s, l, k.make_weights(**w), x, out)
        torch.cuda.synchronize()
        assert k.lib.kvpr_debug_layer_mode(ctx) == mode
        k.kvpr_layer_decode(ctx, 0, s, l, k.make_weights(**w), x, out, timing=True)
        assert k.lib.kvpr_debug_layer_mode(ctx) == 0                   # timed: three streams
    finally:
        k.kvpr_destroy(ctx)


def test_unpacking_in_front_of_the_recomputation(k):
    """Packed activations of 13014 rows: unpacking and product take longer than a call in order saves, beside a cache that hides them."""
    b, h, H, s, l = 9, 768, 12, 1808, 1446
    ctx, w, x, out = _context(k, b, h, H, s, flags=k.KVPR_STORE_INT4)
    try:
        k.kvpr_layer_decode(ctx, 0, s, l, k.make_weights(**w), x, out)
        torch.cuda.synchronize()
        assert k.lib.kvpr_debug_layer_mode(ctx) == 0
    finally:
        k.kvpr_destroy(ctx)


@pytest.mark.parametrize("b,mode", [(4, ROWS_BESIDE_ATTENTION), (64, 0)])
def test_layer_of_a_step(k, b, mode):
    h, H, s = 1024, 8, 40
    ctx, w, x, out = _context(k, b, h, H, s, ffn=2048, layers=2)
    try:
        k.kvpr_decode_step(ctx, s, [k.make_weights(**w)] * 2, x, out, [10, 10])
        torch.cuda.synchronize()
        assert k.lib.kvpr_debug_layer_mode(ctx) == mode
    finally:
        k.kvpr_destroy(ctx)
