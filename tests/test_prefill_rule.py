"""When the prefill helper works in runs, as host arithmetic: both sides of each border of the rule, and what it was measured at."""
import ctypes as C

import pytest

F16, KV4, ALL4 = 0, 1, 2


@pytest.fixture(scope="module")
def runs():
    import paper_2411_17089_amd as k
    f = k.lib.kvpr_debug_prefill_rule
    f.restype, f.argtypes = C.c_int, [C.c_int, C.c_int, C.c_size_t, C.c_size_t, C.c_int]

    def call(hidden, batch, seq, store):
        x = batch * (k.kvpr_int4_row_bytes(hidden) if store == ALL4 else 2 * hidden)
        kv = batch * (4 * hidden if store == F16 else k.kvpr_int4_row_bytes(2 * hidden))
        return f(seq, hidden, x, kv, int(store != F16))
    return call


@pytest.mark.parametrize("hidden,batch,seq,store,want", [
    (512, 64, 24, F16, 1), (512, 64, 25, F16, 0),                                 # 3 MiB of rows in one run
    (768, 16, 198, F16, 0), (768, 8, 1150, F16, 0), (768, 8, 1190, F16, 4),       # narrow products: 27 MiB at hidden 768
    (1024, 32, 180, F16, 0), (1024, 32, 190, F16, 4), (256, 8, 4500, F16, 0), (256, 8, 4600, F16, 5),
    (2048, 32, 28, F16, 0), (2048, 32, 29, F16, 2), (4096, 8, 64, F16, 2), (7168, 2, 616, F16, 4), (4096, 8, 512, F16, 6),
    (768, 8, 700, KV4, 3), (256, 1, 4028, KV4, 1), (4096, 1, 1268, ALL4, 0), (768, 8, 1537, ALL4, 2),
    (7168, 32, 109, F16, 7), (7168, 32, 110, F16, 0)])                            # 96 MiB of rows
def test_rule(runs, hidden, batch, seq, store, want):
    assert runs(hidden, batch, seq, store) == want
