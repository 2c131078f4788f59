"""Single-layer decode where the way its rows come in changes (one kernel up to 1 MiB, 2 MiB for a float16 cache alone, copies
beyond): both sides of each limit against the oracle and, bit for bit, in the debug modes, with and without timing."""
import numpy as np
import pytest
import torch

import kvpr_inputs
from kvpr_testlib import dev, rel_err, upload_layer
from oracle import kvpr_int4_oracle as qo
from oracle import kvpr_oracle as ko

pytestmark = pytest.mark.gpu
B, H, HEADS = 4, 512, 4                                      # a position: 4 KiB of activations and 8 KiB of cache, packed 9/32 of it


@pytest.fixture(scope="module")
def k():
    import paper_2411_17089_amd as k
    return k


@pytest.mark.parametrize("s,l", [(128, 0), (129, 0), (256, 0), (257, 0), (256, 256), (257, 257), (170, 84), (171, 85), (700, 300), (1, 0), (1, 1)])
@pytest.mark.parametrize("packed", [False, True])
def test_modes_agree(k, s, l, packed):
    if packed and s > 1:                                    # the same bytes in packed rows, rounded down and up alike
        s, l = s * 32 // 9 + s % 2, l * 32 // 9
    layer = kvpr_inputs.make_layer(s, B, s, H, HEADS)
    stored = ko.stored_kv(layer, "fp16")
    d = upload_layer(layer)
    w = k.make_weights(**{f: d[f] for f in ("wqkv", "bqkv", "wo", "bo")})
    ctx = k.kvpr_create(1, H, HEADS, H // HEADS, 0, B, s + 2, dtype=k.KVPR_F16 | (k.KVPR_STORE_INT4 if packed else 0))
    try:
        k.kvpr_store_write(ctx, 0, 0, s, np.ascontiguousarray(layer["X"]), stored.astype(np.float16))
        outs = {}
        for mode, timing in ((0, False), (k.KVPR_DEBUG_POISON, False), (k.KVPR_DEBUG_POISON, True), (k.KVPR_DEBUG_POISON | k.KVPR_DEBUG_SYNC, False), (0, True)):
            k.kvpr_set_debug(ctx, mode)
            out = torch.full((B, H), float("nan"), dtype=torch.float16, device="cuda")
            for _ in range(2):                              # in a row: the second waits for the first one's buffers and rows
                k.kvpr_layer_decode(ctx, 0, s, l, w, d["x_new"], out, timing=timing)
            torch.cuda.synchronize()
            outs[mode, timing] = out.cpu().numpy()
        base = outs[0, False]
        for m, o in outs.items():
            assert np.array_equal(o, base), m
        if packed:                                          # what the store holds: rows through the codec and back
            layer, stored = dict(layer, X=qo.roundtrip(layer["X"]).astype(np.float64)), qo.roundtrip(stored.astype(np.float16)).astype(np.float64)
        assert rel_err(base, ko.layer_decode(layer, l, stored)["o"]) <= 5e-3                        # the bound of the layer tests
    finally:
        k.kvpr_destroy(ctx)
