"""Greedy step and norms where their vector paths can go wrong: rows that are no multiple of the vector width, tensors off a
16-byte boundary, ties across waves, rows without any token; a decoder step on unaligned hidden states."""
import numpy as np
import pytest
import torch

from kvpr_testlib import rel_err
from oracle import kvpr_oracle as ko
from test_gpu_stack import Stack

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def k():
    import paper_2411_17089_amd as k
    return k


def off(t, halfs):
    """The same values `halfs` elements past a 16-byte boundary."""
    room = torch.zeros(t.numel() + 16, dtype=t.dtype, device=t.device)
    view = room[halfs: halfs + t.numel()].view(t.shape)
    view.copy_(t)
    return view


@pytest.mark.parametrize("vocab", [1, 3, 64, 4095, 4096, 4097, 16388, 50272])
@pytest.mark.parametrize("shift", [0, 1])
def test_greedy(k, vocab, shift):
    """Logits come back whole, the token is their first maximum and the next input its embedding row."""
    b, h = 3, 128
    g = torch.Generator().manual_seed(vocab)
    hidden = torch.randn(b, h, generator=g).half().cuda()
    w = (torch.randn(vocab, h, generator=g) * 0.1).half()
    w[vocab // 2:] = w[: vocab - vocab // 2].clone()          # every logit of the first half again: ties far apart
    emb = torch.randn(vocab, h, generator=g).half().cuda()
    logits = off(torch.empty((b, vocab), dtype=torch.float32, device="cuda"), shift)
    tokens = torch.empty((b,), dtype=torch.int32, device="cuda")
    x_next = off(torch.empty((b, h), dtype=torch.float16, device="cuda"), shift)
    k.kvpr_greedy_next(hidden, w.cuda(), off(emb, shift), b, h, vocab, logits, tokens, x_next)
    lg = logits.cpu().numpy()
    assert np.array_equal(tokens.cpu().numpy(), lg.argmax(1))   # numpy's argmax takes the first as well
    assert torch.equal(x_next, emb[tokens.long()])


def test_greedy_rows_without_a_token(k):
    b, h, vocab = 2, 128, 320
    hidden = torch.zeros((b, h), dtype=torch.float16, device="cuda")
    hidden[0, 0], hidden[1, 0] = float("nan"), 1.0
    w = torch.zeros((vocab, h), dtype=torch.float16, device="cuda")
    w[7, 0] = 1.0
    emb = torch.ones((vocab, h), dtype=torch.float16, device="cuda")
    logits = torch.empty((b, vocab), dtype=torch.float32, device="cuda")
    tokens = torch.empty((b,), dtype=torch.int32, device="cuda")
    x_next = torch.empty((b, h), dtype=torch.float16, device="cuda")
    k.kvpr_greedy_next(hidden, w, emb, b, h, vocab, logits, tokens, x_next)
    assert tokens.tolist() == [0x7FFFFFFF, 7]
    assert (x_next[0] == 0).all() and (x_next[1] == 1).all()


@pytest.mark.parametrize("h,heads", [(128, 2), (640, 5), (8320, 65)])
def test_decoder_step_on_unaligned_hidden_states(k, h, heads):
    """Norm and residual read the caller's tensor: one piece per thread or several, on and off a 16-byte boundary."""
    st = Stack(k, 1, 2, 6, h, heads, 128)
    try:
        x = torch.from_numpy(st.x_in).cuda()
        outs = []
        for shift in (0, 1):
            out = off(torch.zeros_like(x), shift)
            k.kvpr_decode_step(st.ctx, st.s, st.w, off(x, shift), out, [3])
            torch.cuda.synchronize()
            outs.append(out.cpu().numpy())
        assert np.array_equal(outs[0], outs[1])
        ref, _ = ko.decoder_stack_decode(st.layers, st.x_in, [3], st.stored)
        assert rel_err(outs[0], ref) <= 5e-3                    # the bound of the decoder step tests
    finally:
        st.close()
