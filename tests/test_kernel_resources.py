"""What the compiler reports of the library's kernels: no vector register is spilled to scratch memory.  (A token GEMM with 14 to 67
spilled was 3 - 5 % slower than the separate launches that it replaced.)"""
import struct

import msgpack


def _kernels(path):
    """Metadata of the kernels in the gfx950 code objects inside a shared library (ELF notes "AMDGPU", type 32: msgpack)."""
    data, out, at = open(path, "rb").read(), [], 1
    while (at := data.find(b"\x7fELF\x02", at)) > 0:
        machine, = struct.unpack_from("<H", data, at + 18)
        if machine == 224:                                             # EM_AMDGPU
            headers, = struct.unpack_from("<Q", data, at + 40)
            size, count = struct.unpack_from("<HH", data, at + 58)
            for i in range(count):
                kind, = struct.unpack_from("<I", data, at + headers + i * size + 4)
                offset, length = struct.unpack_from("<QQ", data, at + headers + i * size + 24)
                note, end = at + offset, at + offset + length
                while kind == 7 and note + 12 <= end:                  # SHT_NOTE
                    name, desc, type_ = struct.unpack_from("<III", data, note)
                    body = note + 12 + (name + 3) // 4 * 4
                    if type_ == 32 and data[note + 12:note + 12 + name].rstrip(b"\0") == b"AMDGPU":
                        out += msgpack.unpackb(data[body:body + desc])["amdhsa.kernels"]
                    note = body + (desc + 3) // 4 * 4
        at += 1
    return out


def test_no_spills():
    import paper_2411_17089_amd as k
    kernels = _kernels(k.lib._name)
    assert sum("few_tokens" in e[".name"] for e in kernels) > 100
    spilled = {e[".name"]: e[".vgpr_spill_count"] for e in kernels if e[".vgpr_spill_count"] or e[".private_segment_fixed_size"]}
    assert not spilled, spilled
