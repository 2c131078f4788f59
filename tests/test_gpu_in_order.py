"""Single-layer decode in order on the compute stream: copies beside the projection, the recomputation and the attention.  Both
sides of the rule, row counts of both token GEMMs, packed stores and unaligned rows, calls that follow one another in either
way and read the rows that the one before has stored."""
import numpy as np
import pytest
import torch

import kvpr_inputs
from kvpr_testlib import dev, rel_err, upload_layer
from oracle import kvpr_oracle as ko

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def k():
    import paper_2411_17089_amd as k
    return k


# (batch, hidden, heads): 8 and 9 rows at hidden 1024 are the two sides of the token GEMMs, at hidden 512 both take the one for up to
# 64 rows; hidden 384, batch 3 has packed rows of 8-byte pieces.  (test_gpu_layer_modes.py asserts which calls are in order.)
@pytest.mark.parametrize("b,h,H", [(2, 256, 2), (8, 512, 4), (9, 512, 4), (3, 384, 3), (8, 1024, 8), (5, 1024, 8), (9, 1024, 8)])
@pytest.mark.parametrize("packed", [False, True])
@pytest.mark.parametrize("s,l", [(70, 0), (70, 30), (70, 70), (1400, 300), (3000, 1500)])
def test_rows_written_and_read_in_either_order(k, b, h, H, packed, s, l):
    print(f"in order b={b} h={h} packed={packed} s={s} l={l}", flush=True)
    layer = kvpr_inputs.make_layer(s, b, s, h, H)
    stored = ko.stored_kv(layer, "fp16")
    d = upload_layer(layer)
    w = k.make_weights(**{f: d[f] for f in ("wqkv", "bqkv", "wo", "bo")})
    rng = np.random.default_rng(s + l)
    news = [dev(rng.standard_normal((b * h + 1,)).astype(np.float16))[1:].view(b, h) if i == 1 else
            dev(rng.standard_normal((b, h)).astype(np.float16)) for i in range(3)]
    got = {}
    for timed in ((False, False, False), (True, True, True), (False, True, False), (True, False, True)):   # a timed call takes the streams
        ctx = k.kvpr_create(1, h, H, h // H, 0, b, s + 4, dtype=k.KVPR_F16 | (k.KVPR_STORE_INT4 if packed else 0))
        try:
            k.kvpr_store_write(ctx, 0, 0, s, np.ascontiguousarray(layer["X"]), stored.astype(np.float16))
            outs = [torch.full((b, h), float("nan"), dtype=torch.float16, device="cuda") for _ in range(3)]
            for i in range(3):
                k.kvpr_layer_decode(ctx, 0, s + i, l + (i if l else 0), w, news[i], outs[i], timing=timed[i])
            torch.cuda.synchronize()
            got[timed] = [o.cpu().numpy() for o in outs]
        finally:
            k.kvpr_destroy(ctx)
    for timed, o in got.items():
        for i in range(3):
            assert np.array_equal(o[i], got[False, False, False][i]), (timed, i)
    if not packed:
        x0 = dict(layer, x_new=news[0].cpu().numpy().astype(np.float64))
        assert rel_err(got[False, False, False][0], ko.layer_decode(x0, l, stored)["o"]) <= 5e-3
