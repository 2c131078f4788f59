"""How the token GEMM for few rows is cut into waves, pieces of K, segments and workgroups, as host arithmetic: the pieces cover K,
every workgroup has rows, and the sums of a workgroup fit the LDS that a launch gets."""
import ctypes as C

import pytest

PLAIN, GATED, ROTARY = 0, 1, 2
LDS = 64 * 1024


@pytest.fixture(scope="module")
def plan():
    import paper_2411_17089_amd as k
    f = k.lib.kvpr_debug_few_plan
    f.restype, f.argtypes = C.c_int, [C.c_int] * 5 + [C.POINTER(C.c_int32)] * 5

    def call(M, N, K, form=PLAIN, cus=256):
        out = [C.c_int32() for _ in range(5)]
        assert f(M, N, K, form, cus, *out) == 0
        return tuple(v.value for v in out)                  # waves, pieces, segments, workgroups, bytes of LDS
    return call


@pytest.mark.parametrize("M", [4, 8])
@pytest.mark.parametrize("form", [PLAIN, GATED, ROTARY])
@pytest.mark.parametrize("cus", [32, 80, 256, 304])
def test_sums_fit_beside_those_of_the_norm(plan, M, form, cus):
    tokens, parts = (4 if M <= 4 else 8), (1 if form == PLAIN else 2)
    for N in [*range(8, 4096, 8), *range(4096, 300000, 64 if cus < 256 else 128), 126976, 129024, 191488, 253952]:
        waves, _, _, grid, lds = plan(M, N, 1024, form, cus)
        units = (N + 3) // 4 if form == PLAIN else N // 8
        assert 1 <= grid <= units
        most = -(-units // grid)                            # of the first workgroups
        assert lds == most * parts * tokens * 4 * waves * 4
        assert lds + 2 * waves * tokens * 4 <= LDS, (N, grid, lds)     # two float32 sums of the norm for each wave and token


@pytest.mark.parametrize("M", [1, 4, 5, 8])
def test_pieces_cover_the_columns(plan, M):
    for K in range(128, 1 << 17, 128):
        waves, pieces, segments, _, _ = plan(M, 4096, K)
        assert waves == (4 if K % 16384 == 0 else 8)
        assert 1 <= pieces <= (8 if M <= 4 else 7) if waves == 8 else pieces == 7      # the only kernel of 4 waves
        runs = [K // 128 * (w + 1) // waves - K // 128 * w // waves for w in range(waves)]
        for run in set(runs):                               # a wave walks a segment of `pieces` or one less
            parts = {run * (s + 1) // segments - run * s // segments for s in range(segments)}
            assert parts <= {pieces, pieces - 1}, (K, run, parts)


@pytest.mark.parametrize("M,N,K,along,alone", [
    (1, 2304, 768, 1, 0), (4, 768, 768, 1, 0), (4, 8192, 768, 1, 0), (4, 8256, 768, 1, 1), (1, 50272, 640, 1, 1), (1, 50272, 512, 1, 0),
    (1, 768, 1024, 1, 1), (4, 128, 128, 1, 0), (5, 2304, 768, 0, 0), (5, 50272, 896, 0, 0), (5, 2304, 1024, 1, 1),
    (6, 4096, 11008, 1, 1), (7, 4096, 11008, 0, 0), (8, 4104, 11008, 1, 1), (8, 4096, 7168, 1, 1), (9, 12288, 4096, 0, 0)])
def test_rule(plan, M, N, K, along, alone):
    """With something along it saves a launch; alone it has to be the faster kernel."""
    import paper_2411_17089_amd as k
    assert (k.lib.kvpr_debug_few_tokens(M, N, K, 0), k.lib.kvpr_debug_few_tokens(M, N, K, 1)) == (along, alone)
