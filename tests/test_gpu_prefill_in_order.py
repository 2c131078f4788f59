"""The prefill helper in runs whose copies go along with the products and in one piece: one to seven runs, the last position count that
goes in runs and the first above them, against one product over all positions.  (test_gpu_prefill_rows.py asserts the number of
runs.)"""
import pytest

import test_gpu_prefill_runs as whole

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def k():
    import paper_2411_17089_amd as k
    return k


# hidden 512, float16: 96 MiB of rows are 768 positions at batch 64
@pytest.mark.parametrize("rotary", [False, True])
@pytest.mark.parametrize("packed", [False, True])
@pytest.mark.parametrize("b,s", [(64, 1), (64, 24), (64, 66), (1, 3000), (64, 768), (64, 769)])
def test_rows_equal_one_product(k, b, s, packed, rotary):
    print(f"prefill b={b} s={s} packed={packed} rotary={rotary}", flush=True)
    whole.test_rows_equal_one_product(k, b, s, packed, rotary)
