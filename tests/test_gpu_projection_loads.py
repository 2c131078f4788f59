"""Single-layer decode with few rows: the projection reads W by ordinary loads where a recomputation follows and by non-temporal ones
where none does, with copies beside it or none.  The new token's rows have the same bits in all of them, and are right."""
import ctypes

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def k():
    import paper_2411_17089_amd as k
    return k


@pytest.mark.parametrize("h", [256, 1152, 4096, 7168, 8192])     # 0 / 1, 1 / 2, 4, 7 and 8 pieces of K a wave
@pytest.mark.parametrize("b", [1, 4, 5, 8])
@pytest.mark.parametrize("arch", ["opt", "llama"])
def test_new_rows_do_not_depend_on_the_split(k, arch, b, h):
    print(f"projection loads {arch} h={h} b={b}", flush=True)
    s, width = 9, 64 if h == 1152 else 128
    g = torch.Generator(device="cuda").manual_seed(h + b)
    rand = lambda *shape, scale: (torch.randn(shape, generator=g, device="cuda") * scale).half()   # noqa: E731
    w = {"wqkv": rand(3 * h, h, scale=0.02), "wo": rand(h, h, scale=0.02)}
    if arch == "opt":
        w["bqkv"] = rand(3 * h, scale=0.1)
    x_new, got = rand(b, h, scale=1.0), []
    x = rand(s, b, h, scale=1.0).cpu().numpy()
    for split, timing in ((0, False), (0, True), (5, False), (5, True), (s, False)):
        ctx = k.kvpr_create(1, h, h // width, width, 0, b, s + 2, arch=k.KVPR_ARCH_LLAMA if arch == "llama" else k.KVPR_ARCH_OPT)
        try:
            k.kvpr_store_write(ctx, 0, 0, s, x, None)
            k.kvpr_store_prefill_kv(ctx, 0, s, k.make_weights(**w))
            out = torch.full((b, h), float("nan"), dtype=torch.float16, device="cuda")
            k.kvpr_layer_decode(ctx, 0, s, split, k.make_weights(**w), x_new, out, timing=timing)
            torch.cuda.synchronize()
            address = k.kvpr_store_ptrs(ctx, 0)[1] + s * b * 4 * h
            got.append((np.frombuffer((ctypes.c_ubyte * (b * 4 * h)).from_address(address), np.float16).copy().reshape(b, 2 * h), out.cpu().numpy()))
        finally:
            k.kvpr_destroy(ctx)
    for row, out in got[1:]:
        assert np.array_equal(row, got[0][0])
        assert np.isfinite(out).all()
    # v is not rotated: float32 sums of h products in any order, one rounding to float16
    wv = w["wqkv"][2 * h:].double()
    want = x_new.double() @ wv.T + (w["bqkv"][2 * h:].double() if arch == "opt" else 0.0)
    sums = h * 2.0 ** -24 * (x_new.double().abs() @ wv.abs().T + 1.0)
    v = torch.from_numpy(got[0][0][:, h:]).cuda().double()
    assert bool(((v - want).abs() <= sums + 2.0 ** -11 * want.abs() + 2.0 ** -24).all())
