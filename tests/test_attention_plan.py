"""How the decode attention is cut into workgroups, as host arithmetic: where the rule changes over, that the pieces cover
the positions, and that their partial results fit the caller's workspace and the static array."""
import ctypes as C

import pytest


@pytest.fixture(scope="module")
def plan():
    import paper_2411_17089_amd as k
    f = k.lib.kvpr_debug_attention_plan
    f.restype, f.argtypes = C.c_int, [C.c_int, C.c_int, C.c_int] + [C.POINTER(C.c_int32)] * 3

    def call(batch, hidden, S):
        out = [C.c_int32() for _ in range(3)]
        assert f(batch, hidden, S, *out) == 0
        return tuple(v.value for v in out)                  # positions per workgroup, splits, waves per workgroup
    return call


# one column group at hidden 512: the batch is the number of workgroups without splits
@pytest.mark.parametrize("batch,S,splits,waves", [
    (127, 4097, 3, 4), (128, 4097, 2, 4), (128, 385, 2, 4), (128, 384, 1, 8), (128, 129, 1, 8),     # half the compute units
    (129, 4097, 1, 8), (255, 4097, 1, 8), (255, 129, 1, 8),                                       # more than half, not all
    (256, 4097, 1, 4), (256, 129, 1, 4), (257, 4097, 1, 4), (512, 4097, 1, 4),                    # one each and more
    (1, 128, 1, 8), (256, 128, 1, 8), (257, 128, 1, 4), (1, 129, 3, 4)])                          # two rounds to share
def test_rule(plan, batch, S, splits, waves):
    chunk, got_splits, got_waves = plan(batch, 512, S)
    assert (got_splits, got_waves) == (splits, waves)


def test_pieces_cover_the_positions_and_fit(plan):
    import paper_2411_17089_amd as k
    largest = 0
    for hidden in (64, 192, 512, 768, 1088, 4096, 5120, 7168, 16384):
        for batch in [*range(1, 65), 100, 128, 129, 200, 255, 256, 300]:
            for S in (1, 2, 31, 32, 33, 63, 64, 65, 100, 127, 128, 129, 191, 193, 255, 257, 500, 512, 513, 1000, 1025, 2049, 4097, 16000, 70000):
                chunk, splits, _ = plan(batch, hidden, S)
                assert chunk >= 1 and splits >= 1 and chunk * splits >= S > chunk * (splits - 1), (hidden, batch, S)
                need = splits * batch * hidden * 5 if splits > 1 else 0       # float32 sums and a (maximum, sum) pair per 8 columns
                assert need <= k.kvpr_attention_workspace_bytes(batch, hidden, hidden // 64, S)
                largest = max(largest, need)
    assert largest <= 1.3 * 2 ** 20 < k.KVPR_ATTENTION_STATIC_SCRATCH_BYTES, largest        # what the header promises
