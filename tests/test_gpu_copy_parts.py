"""Single-layer decode whose activations come in by several parts: the same bits as in one part (a timed call), rows in the store
included, where the cache is shorter than the product, and one part where it is longer."""
import ctypes

import numpy as np
import pytest
import torch

from kvpr_testlib import dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def k():
    import paper_2411_17089_amd as k
    return k


@pytest.mark.parametrize("s,l,several", [(601, 601, True), (603, 590, True), (600, 100, False), (40, 9, False)])
@pytest.mark.parametrize("arch", ["opt", "llama"])
@pytest.mark.parametrize("packed", [False, True])
def test_parts_give_the_same_rows(k, s, l, several, arch, packed):
    b, h, H, llama = 64, 1024, 8, arch == "llama"
    print(f"parts s={s} l={l} {arch} packed={packed}", flush=True)
    rng = np.random.default_rng(s + l)
    x = rng.standard_normal((s, b, h)).astype(np.float16)
    arrays = {"wqkv": rng.standard_normal((3 * h, h)) * 0.03, "wo": rng.standard_normal((h, h)) * 0.03}
    if not llama:
        arrays.update(bqkv=rng.standard_normal(3 * h) * 0.1, bo=rng.standard_normal(h) * 0.1)
    w = {n: dev(a.astype(np.float16)) for n, a in arrays.items()}
    x_new = dev(rng.standard_normal((b, h)).astype(np.float16))
    got = []
    for timing in (True, False, False):
        ctx = k.kvpr_create(1, h, H, h // H, 0, b, s + 2, dtype=k.KVPR_F16 | (k.KVPR_STORE_INT4 if packed else 0),
                            arch=k.KVPR_ARCH_LLAMA if llama else k.KVPR_ARCH_OPT)
        try:
            k.kvpr_store_write(ctx, 0, 0, s, x, None)
            k.kvpr_store_prefill_kv(ctx, 0, s, k.make_weights(**w))
            out = torch.full((b, h), float("nan"), dtype=torch.float16, device="cuda")
            for _ in range(2):                                  # the second waits for the first one's buffers
                k.kvpr_layer_decode(ctx, 0, s, l, k.make_weights(**w), x_new, out, timing=timing)
            torch.cuda.synchronize()
            parts = k.lib.kvpr_debug_copy_parts(ctx)
            assert (parts > 1) == (several and not timing), parts
            row = b * (k.kvpr_int4_row_bytes(2 * h) if packed else 4 * h)
            address = k.kvpr_store_ptrs(ctx, 0)[1] + s * row
            got.append((out.cpu().numpy(), np.frombuffer((ctypes.c_ubyte * row).from_address(address), np.uint8).copy()))
        finally:
            k.kvpr_destroy(ctx)
    assert np.isfinite(got[0][0]).all()
    for o, r in got[1:]:
        assert np.array_equal(o, got[0][0]) and np.array_equal(r, got[0][1])
