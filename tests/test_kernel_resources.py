"""What the compiler gave the kernels of the built library: no scratch memory, the registers that the measured numbers
of waves per SIMD need, and the distance that stores it cannot see into must keep."""
import os
import re
import struct
import subprocess

import msgpack
import pytest

from paper_1804_08066_amd import build, mqgrad


def code_objects():
    """The code objects embedded in the library."""
    with open(build.LIB, "rb") as f:
        blob = f.read()
    at = blob.find(b"\x7fELF", 1)          # the first one is the library itself
    while at >= 0:
        if struct.unpack_from("<H", blob, at + 18)[0] == 224:      # EM_AMDGPU
            shoff, = struct.unpack_from("<Q", blob, at + 40)       # the section headers come last
            entry, count = struct.unpack_from("<HH", blob, at + 58)
            yield blob[at:at + shoff + entry * count]
        at = blob.find(b"\x7fELF", at + 4)


def kernels():
    """The kernels' entries of the code objects' AMDGPU metadata notes."""
    found = {}
    for obj in code_objects():
        phoff, = struct.unpack_from("<Q", obj, 32)
        entry, count = struct.unpack_from("<HH", obj, 54)
        for i in range(count):
            kind, _, offset, _, _, size = struct.unpack_from("<IIQQQQ", obj, phoff + i * entry)
            if kind != 4:                                          # PT_NOTE
                continue
            note, end = offset, offset + size
            while note < end:
                name, desc, type_ = struct.unpack_from("<III", obj, note)
                body = note + 12 + (name + 3 & ~3)
                if type_ == 32:                                    # NT_AMDGPU_METADATA
                    for k in msgpack.unpackb(obj[body:body + desc])["amdhsa.kernels"]:
                        found[k[".name"]] = k
                note = body + (desc + 3 & ~3)
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


def test_wide_scoped_stores_keep_two_wait_states(built, tmp_path):
    """The agent-scope 128-bit stores are inline assembly, so the compiler does not know that no vector operation may write
    their data in the two wait states behind them: each brings its own."""
    objdump = os.path.join(os.path.dirname(os.path.realpath(build.HIPCC)), "..", "llvm", "bin", "llvm-objdump")
    stores = 0
    for i, obj in enumerate(code_objects()):
        path = tmp_path / ("%d.o" % i)
        path.write_bytes(obj)
        text = subprocess.run([objdump, "-d", "--no-show-raw-insn", "--no-leading-addr", str(path)],
                              check=True, capture_output=True, text=True).stdout
        code = [line.split("//")[0].strip() for line in text.splitlines()]
        for store, behind in zip(code, code[1:]):
            if re.match(r"global_store_dwordx4 .* sc1$", store):
                stores += 1
                assert re.match(r"s_nop [1-9]", behind), (store, behind)
    assert stores > 100
