"""Every tile of the recompute GEMM at the edges of its range: row and column remainders, and K from one stage to past the
depth of its LDS ring; with and without the rotary epilogue of both head widths."""
import numpy as np
import pytest
import torch

from oracle import kvpr_oracle as ko
from kvpr_testlib import dev, rel_err

pytestmark = pytest.mark.gpu

# float32 sums of at most 576 products rounded once to float16: 2^-11 of the largest value, plus the sums' own error
TIGHT = 2e-3
TILES = range(1, 7)


@pytest.fixture(scope="module")
def k():
    import paper_2411_17089_amd as k
    return k


@pytest.fixture
def force(k):
    yield k.lib.kvpr_debug_set_gemm_variant
    k.lib.kvpr_debug_set_gemm_variant(0)


@pytest.mark.parametrize("tile", TILES)
@pytest.mark.parametrize("M,N,K", [(1, 8, 64), (64, 128, 128), (65, 136, 192), (193, 264, 384), (255, 520, 448), (257, 384, 576)])
def test_plain(k, force, tile, M, N, K):
    rng = np.random.default_rng(M * 3 + K)
    A = rng.standard_normal((M, K)).astype(np.float16)
    W = (rng.standard_normal((N, K)) * 0.05).astype(np.float16)
    bias = (rng.standard_normal(N) * 0.1).astype(np.float16)
    c = torch.full((M + 2, N + 8), float("nan"), dtype=torch.float16, device="cuda")
    force(tile)
    k.kvpr_recompute_gemm(dev(A), dev(W), dev(bias), c, M, N, K, N + 8)
    got = c.cpu().numpy()
    assert np.isnan(got[:M, N:]).all() and np.isnan(got[M:]).all(), "nothing outside the result may be written"
    assert rel_err(got[:M, :N], ko.project(A, W.T, bias)) <= TIGHT


@pytest.mark.parametrize("tile", TILES)
@pytest.mark.parametrize("heads,width", [(3, 128), (6, 64)])
def test_rotary(k, force, tile, heads, width):
    """The K half against the plain product rotated on the host, the V half against the plain product."""
    batch, l, pos0, h = 3, 71, 2, heads * width
    rng = np.random.default_rng(width)
    M, K = batch * l, h
    A = rng.standard_normal((M, K)).astype(np.float16)
    W = (rng.standard_normal((2 * h, K)) * 0.05).astype(np.float16)
    tab = k.kvpr_rope_table(pos0 + l, width)
    out = torch.full((M, 2 * h), float("nan"), dtype=torch.float16, device="cuda")
    force(tile)
    k.kvpr_recompute_gemm_rope(dev(A), dev(W), None, out, M, 2 * h, h, 2 * h, dev(tab, torch.float32), pos0 + l, h, width, batch, pos0)
    want = ko.project(A, W.T, None)
    t = np.asarray(tab, dtype=np.float64).reshape(pos0 + l, width // 2, 2)[pos0 + np.arange(M) // batch]     # cos, sin of a row's position
    half = want[:, :h].reshape(M, heads, 2, width // 2)
    cos, sin = t[:, None, :, 0], t[:, None, :, 1]
    want[:, :h] = np.stack([half[:, :, 0] * cos - half[:, :, 1] * sin, half[:, :, 1] * cos + half[:, :, 0] * sin], 2).reshape(M, h)
    assert rel_err(out.cpu().numpy(), want) <= TIGHT


def test_tiles_agree_bit_for_bit(k, force):
    """All tiles add the products of an output in the same order, so the choice between them never shows."""
    M, N, K = 300, 392, 320
    g = torch.Generator().manual_seed(1)
    A, W = torch.randn(M, K, generator=g).half().cuda(), torch.randn(N, K, generator=g).half().cuda()
    first = None
    for tile in TILES:
        c = torch.empty((M, N), dtype=torch.float16, device="cuda")
        force(tile)
        k.kvpr_recompute_gemm(A, W, None, c, M, N, K, N)
        first = c if first is None else first
        assert torch.equal(c, first), tile


@pytest.mark.parametrize("heads,width", [(3, 128), (6, 64)])
def test_rotary_tiles_agree_bit_for_bit(k, force, heads, width):
    batch, l, pos0, h = 3, 100, 2, heads * width
    g = torch.Generator().manual_seed(2)
    A, W = torch.randn(batch * l, h, generator=g).half().cuda(), (torch.randn(2 * h, h, generator=g) * 0.05).half().cuda()
    tab = dev(k.kvpr_rope_table(pos0 + l, width), torch.float32)
    first = None
    for tile in TILES:
        c = torch.empty((batch * l, 2 * h), dtype=torch.float16, device="cuda")
        force(tile)
        k.kvpr_recompute_gemm_rope(A, W, None, c, batch * l, 2 * h, h, 2 * h, tab, pos0 + l, h, width, batch, pos0)
        first = c if first is None else first
        assert torch.equal(c, first), tile
