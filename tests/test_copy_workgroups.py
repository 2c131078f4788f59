"""Workgroups of the copy kernel between device memory and pinned host memory: one for each 4 KiB, and no more than the link needs."""
import ctypes as C

import pytest


@pytest.mark.parametrize("bytes_,bytes2,blocks", [(0, 0, 0), (1, 0, 1), (0, 4096, 1), (4096, 1, 2), (4096, 4096, 2), (200000, 45760, 60), (262144, 0, 64), (1 << 21, 0, 64),
                                                  (1 << 20, 1 << 20, 64)])
def test_workgroups(bytes_, bytes2, blocks):
    import paper_2411_17089_amd as k
    f = k.lib.kvpr_debug_copy_workgroups
    f.restype, f.argtypes = C.c_int, [C.c_size_t, C.c_size_t]
    assert f(bytes_, bytes2) == blocks
