"""The built library's kernels keep what they compute on in registers: none has private memory or spills.  A loop that
the compiler could not unroll over a thread's elements would show here (its array lies in memory, at a third of the
speed), as would a kernel that needs more registers than there are."""
import os
import struct

import pytest

msgpack = pytest.importorskip("msgpack")


def _kernels(path):
    """The metadata of every kernel in the library's gfx950 code objects, by name."""
    data = open(path, "rb").read()
    out = {}
    at = data.find(b"__CLANG_OFFLOAD_BUNDLE__")
    while at >= 0:
        n, p = struct.unpack_from("<Q", data, at + 24)[0], at + 32
        for _ in range(n):
            off, size, ln = struct.unpack_from("<QQQ", data, p)
            triple, p = data[p + 24: p + 24 + ln], p + 24 + ln
            if b"gfx950" not in triple or not size:
                continue
            elf = data[at + off: at + off + size]
            sections, = struct.unpack_from("<Q", elf, 40)
            width, count = struct.unpack_from("<HH", elf, 58)
            for s in range(count):
                kind, = struct.unpack_from("<I", elf, sections + s * width + 4)
                start, = struct.unpack_from("<Q", elf, sections + s * width + 24)
                if kind != 7:                      # a note section
                    continue
                name, size, kind = struct.unpack_from("<III", elf, start)
                if kind == 32:                     # kernel metadata
                    first = start + 12 + (name + 3) // 4 * 4
                    for k in msgpack.unpackb(elf[first: first + size])["amdhsa.kernels"]:
                        out[k[".name"]] = k
        at = data.find(b"__CLANG_OFFLOAD_BUNDLE__", at + 24)
    return out


def test_no_kernel_keeps_its_values_in_memory():
    import paper_2506_10399_amd as pkg
    kernels = _kernels(os.path.join(os.path.dirname(pkg.__file__), "libficgcn.so"))
    assert len(kernels) > 200 and any("k_ntt_passILi9E" in n for n in kernels)
    assert [n for n, k in kernels.items() if k[".private_segment_fixed_size"] or k[".vgpr_spill_count"]] == []
