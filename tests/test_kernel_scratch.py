"""The persistent grouped-GEMM kernels keep what they need in registers: a kernel whose k loop goes through scratch memory waits
there for every load in flight.  Read from the kernel descriptors of the built library, so no GPU is needed."""
import struct

import pytest

import paper_2504_14960_amd as moe


def scratch_bytes(path):
    """Kernel name -> scratch bytes per lane, of all kernels in a library: a descriptor (symbol NAME.kd) starts with the
    kernel's fixed LDS and scratch sizes, 32 bits each (AMDGPU code object format)."""
    data = open(path, "rb").read()
    sizes = {}
    start = -1
    while (start := data.find(b"\x7fELF\x02\x01\x01\x40", start + 1)) >= 0:     # code objects inside the host library
        table, = struct.unpack_from("<Q", data, start + 0x28)
        width, count = struct.unpack_from("<HH", data, start + 0x3A)
        sections = [struct.unpack_from("<IIQQQQIIQQ", data, start + table + i * width) for i in range(count)]
        for kind, offset, size, link in ((s[1], s[4], s[5], s[6]) for s in sections):
            if kind != 11:                                                      # the dynamic symbols
                continue
            names = start + sections[link][4]
            for at in range(start + offset, start + offset + size, 24):
                name, _, _, index, value, _ = struct.unpack_from("<IBBHQQ", data, at)
                text = data[names + name:data.index(b"\0", names + name)].decode()
                if text.endswith(".kd"):
                    home = sections[index]
                    sizes[text[:-3]] = struct.unpack_from("<II", data, start + home[4] + value - home[3])[1]
    return sizes


@pytest.mark.parametrize("kernel", ["gemm_bf16_persist_kernel", "gemm_fp8_persist_kernel"])
def test_persistent_kernels_use_no_scratch_memory(kernel):
    sizes = {name: size for name, size in scratch_bytes(moe.lib_path()).items() if kernel in name}
    assert len(sizes) >= 8, "the library's kernels were not found"
    spilled = {name: size for name, size in sizes.items() if size}
    assert not spilled, spilled
