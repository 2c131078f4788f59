"""Decode attention where the choice of workgroups changes: chunks in whole rounds of the waves (rounded down, rounded up, a
remainder of one position), many partials to merge, one workgroup of 8 waves per sequence and column group, columns that
leave part of a wave idle."""
import numpy as np
import pytest
import torch

from kvpr_testlib import dev, rel_err
from oracle import kvpr_oracle as ko

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def k():
    import paper_2411_17089_amd as k
    return k


@pytest.mark.parametrize("S,b,h,H", [(128, 1, 128, 1), (129, 1, 128, 2), (513, 1, 1024, 8), (2049, 1, 512, 4), (4097, 1, 256, 4),
                                     (1000, 2, 192, 3), (31, 64, 640, 5), (200, 64, 640, 10), (70, 43, 1536, 12), (33, 7, 64, 1)])
def test_against_oracle(k, S, b, h, H):
    rng = np.random.default_rng(S + b)
    q = (rng.standard_normal((b, h)) * 1.5).astype(np.float32)
    kv = rng.standard_normal((S, b, 2 * h)).astype(np.float16)
    kv[S // 2, :, :h] *= 4                                  # one position that dominates some heads: partial maxima differ
    z = torch.full((b, h), float("nan"), dtype=torch.float16, device="cuda")
    ws = torch.empty(k.kvpr_attention_workspace_bytes(b, h, H, S), dtype=torch.uint8, device="cuda")
    k.kvpr_decode_attention(dev(q, torch.float32), dev(kv), z, ws, S, b, h, H)
    assert rel_err(z.cpu().numpy(), ko.decode_attention(q, kv, H)) <= 2e-3      # one float16 rounding is 4.9e-4
    z2 = torch.full_like(z, float("nan"))
    k.kvpr_decode_attention_static(dev(q, torch.float32), dev(kv), z2, S, b, h, H)
    assert torch.equal(z, z2)


@pytest.mark.parametrize("S,b", [(384, 128), (385, 128), (385, 129), (129, 255), (129, 256)])
def test_against_oracle_where_the_workgroup_changes(k, S, b):
    """Half the compute units busy without splits and one more, nearly all and all."""
    test_against_oracle(k, S, b, 64, 1)
