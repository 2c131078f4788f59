"""Recomputations of 2 GFLOP and more in the layer pipeline, in line at these small FFNs: ordering against what the caller
enqueued before the step and against the reuse of the two device buffers, bit for bit against the same steps waited for.
Where they run beside the previous layer is in test_gpu_step_order.py."""
import numpy as np
import pytest
import torch

import kvpr_inputs
from kvpr_testlib import dev
from test_gpu_stack import Stack

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def k():
    import paper_2411_17089_amd as k
    return k


@pytest.mark.parametrize("b", [16, 64])                       # new rows stored on the compute stream, on the store stream
@pytest.mark.parametrize("n_layers,chunks", [(1, 1), (2, 1), (5, 1), (4, 3)])
def test_weights_written_just_before_the_step(k, n_layers, chunks, b):
    """The step is enqueued behind work that is still writing the weights: large products in the first token, some in the
    second and, beside splits of nothing, every other one in the third."""
    s, h, H, ffn = 64, 1024, 8, 1024
    st = Stack(k, n_layers, b, s, h, H, ffn, max_seq=s + 4, seed0=700)
    try:
        k.kvpr_set_chunks(st.ctx, chunks)
        final = [d["wqkv"].clone() for d in st.dev]
        xs = [dev(kvpr_inputs._draw(np.random.default_rng(t), (b, h), 1.0)) for t in range(3)]
        splits = [[s - 1] * n_layers, [(7 * i) % s for i in range(n_layers)], [(s + 2) * (i % 2) for i in range(n_layers)]]
        big = torch.randn(4096, 4096, device="cuda")
        got = {}
        for mode in ("waited", "free"):
            outs = [torch.empty((b, h), dtype=torch.float16, device="cuda") for _ in range(3)]
            for t in range(3):
                for d in st.dev:
                    d["wqkv"].fill_(float("nan"))
                torch.cuda.synchronize()
                for _ in range(8):                                  # some milliseconds on the compute stream
                    big = big @ big
                    big /= big.abs().max()
                for d, f in zip(st.dev, final):
                    d["wqkv"].copy_(f)
                if mode == "waited":
                    torch.cuda.synchronize()
                k.kvpr_decode_step(st.ctx, s + t, st.w, xs[t], outs[t], splits[t])
            torch.cuda.synchronize()
            got[mode] = [o.cpu().numpy() for o in outs]
        for t in range(3):
            assert np.isfinite(got["free"][t].astype(np.float32)).all()
            assert np.array_equal(got["free"][t], got["waited"][t]), t
    finally:
        st.close()
