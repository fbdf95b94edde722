"""What the compiler gave the kernels of the built library: no scratch memory, and the registers that the measured numbers
of waves per SIMD need."""
import struct

import msgpack
import pytest

from paper_1804_08066_amd import build, mqgrad


def kernels():
    """The kernels' entries of the AMDGPU metadata notes in the library's embedded code objects."""
    with open(build.LIB, "rb") as f:
        blob = f.read()
    found = {}
    at = blob.find(b"\x7fELF", 1)          # the first one is the library itself
    while at >= 0:
        if struct.unpack_from("<H", blob, at + 18)[0] == 224:      # EM_AMDGPU
            phoff, = struct.unpack_from("<Q", blob, at + 32)
            entry, count = struct.unpack_from("<HH", blob, at + 54)
            for i in range(count):
                kind, _, offset, _, _, size = struct.unpack_from("<IIQQQQ", blob, at + phoff + i * entry)
                if kind != 4:                                      # PT_NOTE
                    continue
                note, end = at + offset, at + offset + size
                while note < end:
                    name, desc, type_ = struct.unpack_from("<III", blob, note)
                    body = note + 12 + (name + 3 & ~3)
                    if type_ == 32:                                # NT_AMDGPU_METADATA
                        for k in msgpack.unpackb(blob[body:body + desc])["amdhsa.kernels"]:
                            found[k[".name"]] = k
                    note = body + (desc + 3 & ~3)
        at = blob.find(b"\x7fELF", at + 4)
    return found


@pytest.fixture(scope="module")
def built():
    mqgrad.lib()
    found = kernels()
    assert len(found) > 150
    return found


def test_no_kernel_uses_scratch_memory(built):
    assert {n: k[".private_segment_fixed_size"] for n, k in built.items() if k[".private_segment_fixed_size"]} == {}


@pytest.mark.parametrize("kernel,waves", [("sum_range_minmax_tensor_kernel", 7), ("requantize_minmax_tensor_kernel", 7),
                                          ("requantize_minmax_kernel", 4)])
def test_waves_per_simd(built, kernel, waves):
    mine = {n: k for n, k in built.items() if kernel in n}
    assert mine
    for name, k in mine.items():
        assert k[".vgpr_count"] <= 512 // waves // 8 * 8, name
