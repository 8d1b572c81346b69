"""What the compiler made of kernels that live on their last registers, read from the metadata of the built library."""
import os
import struct

import msgpack
import pytest

import paper_2010_02838_amd

NT_AMDGPU_METADATA, SHT_NOTE, EM_AMDGPU = 32, 7, 224


@pytest.fixture(scope="module")
def kernels():
    with open(os.path.join(os.path.dirname(paper_2010_02838_amd.__file__), "libcodistill.so"), "rb") as f:
        data = f.read()
    found, at = {}, data.find(b"\x7fELF", 1)
    while at >= 0:   # the device code objects inside the library
        if struct.unpack_from("<H", data, at + 18)[0] == EM_AMDGPU:
            shoff, shnum = struct.unpack_from("<Q", data, at + 40)[0], struct.unpack_from("<H", data, at + 60)[0]
            for k in range(shnum):
                header = at + shoff + 64 * k
                if struct.unpack_from("<I", data, header + 4)[0] != SHT_NOTE:
                    continue
                off = at + struct.unpack_from("<Q", data, header + 24)[0]
                names, size, kind = struct.unpack_from("<III", data, off)
                if kind == NT_AMDGPU_METADATA:
                    begin = off + 12 + (names + 3) // 4 * 4
                    found.update((q[".name"], q) for q in msgpack.unpackb(data[begin:begin + size])["amdhsa.kernels"])
        at = data.find(b"\x7fELF", at + 1)
    return found


def test_convolutions_spill_two_registers_at_most(kernels):
    """Two data gradients that hold a BatchNorm's input vectors through a loop of 128 accumulators are two registers short; no other convolution spills."""
    spills = {n: q[".vgpr_spill_count"] for n, q in kernels.items() if "igemm_kernel" in n or "wgrad" in n or "conv_generic" in n}
    assert len(spills) > 100
    short = {n: v for n, v in spills.items() if v}
    assert max(short.values(), default=0) <= 2
    assert all("igemm_kernelILi1ELi256ELi128ELi2ELi2ELb0ELi2E" in n or "igemm_kernelILi1ELi128ELi256ELi2ELi2ELb0ELi2E" in n for n in short)
