"""The packing kernel at the edges of its arithmetic, bit for bit: any finite float16 values, one NaN among numbers,
infinities; row lengths that leave the last workgroup with one group of 4 lanes and ones that end inside a piece."""
import numpy as np
import pytest
import torch

from oracle import kvpr_int4_oracle as qo
from kvpr_testlib import dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def k():
    import paper_2411_17089_amd as k
    return k


def _pack(k, a):
    packed = torch.zeros((a.shape[0], k.kvpr_int4_row_bytes(a.shape[1])), dtype=torch.uint8, device="cuda")
    k.kvpr_quant_int4(dev(a), packed, *a.shape)
    return packed.cpu().numpy()


@pytest.mark.parametrize("rows,cols", [(1, 64), (129, 64), (3, 192), (65, 320), (127, 4160), (128, 4096), (513, 1024)])
def test_any_finite_values(k, rows, cols):
    rng = np.random.default_rng(rows + cols)
    a = rng.integers(0, 1 << 16, (rows, cols)).astype(np.uint16).view(np.float16)
    a = np.where(np.isfinite(a), a, np.float16(1.0))
    a[::3] = (rng.integers(0, 31, a[::3].shape) * 0.5).astype(np.float16)          # quotients on the rounding boundary
    a[1::3] = (rng.integers(0, 40, a[1::3].shape) * 2.0 ** -24).astype(np.float16)  # spans of a few subnormal steps
    assert np.array_equal(_pack(k, a), qo.pack_rows(*qo.quantize_rows(a)))


def test_nan_and_infinity(k):
    rng = np.random.default_rng(0)
    a = rng.standard_normal((4, 128)).astype(np.float16)
    a[0, 5] = a[0, 20] = np.nan              # skipped by the extremes, code 0
    a[1, 7], a[2, 9] = np.inf, -np.inf       # no finite scale: all codes 0
    a[3, :64] = np.nan
    got = _pack(k, a)
    codes, scale, mn = qo.quantize_rows(np.where(np.isfinite(a), a, a[:, 70:71]))
    filled = np.where(np.isnan(a[:1]), np.nanmin(a[0, :64]), a[:1])
    assert np.array_equal(got[:1], qo.pack_rows(*qo.quantize_rows(filled)))        # the minimum has code 0
    meta = got[:, 64:].copy().view(np.float16).reshape(4, 2, 2)                    # (scale, minimum) of the two groups
    assert not got[1:, :32].any(), "codes of a group without a finite scale"
    assert meta[1, 0, 0] == np.inf and meta[2, 0, 0] == np.inf and meta[2, 0, 1] == -np.inf and np.isnan(meta[3, 0]).all()
    want = qo.pack_rows(codes, scale, mn)
    assert np.array_equal(got[:, 32:64], want[:, 32:64]), "the group beside it is untouched"
