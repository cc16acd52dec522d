"""Register and LDS use of the state pass's kernels, read from the metadata
notes of the code objects in the built library: a value in scratch memory lies
within the serial chain of every chunk, and the launch rule counts on the
workgroups of some shapes sharing a compute unit."""

import os
import re
import struct

import msgpack
import pytest

import paper_2606_06034_amd as G

LIB = os.path.join(os.path.dirname(os.path.abspath(G.__file__)), "libgdninv.so")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"
NT_AMDGPU_METADATA = 32


def code_objects(blob):
    """The gfx950 code objects of the offload bundles in the library."""
    at = blob.find(MAGIC)
    while at >= 0:
        n, = struct.unpack_from("<Q", blob, at + len(MAGIC))
        if 0 < n <= 16:  # a bundle, not the name alone
            pos = at + len(MAGIC) + 8
            for _ in range(n):
                off, size, ln = struct.unpack_from("<QQQ", blob, pos)
                triple = blob[pos + 24:pos + 24 + ln].decode()
                pos += 24 + ln
                if triple.endswith("gfx950") and size:
                    yield blob[at + off:at + off + size]
        at = blob.find(MAGIC, at + 1)


def notes(elf):
    """The descriptors of an ELF file's AMDGPU metadata notes."""
    shoff, = struct.unpack_from("<Q", elf, 0x28)
    entsize, num = struct.unpack_from("<HH", elf, 0x3A)
    for i in range(num):
        kind, = struct.unpack_from("<I", elf, shoff + i * entsize + 4)
        pos, size = struct.unpack_from("<QQ", elf, shoff + i * entsize + 24)
        end = pos + size
        while kind == 7 and pos < end:  # SHT_NOTE
            nsz, dsz, typ = struct.unpack_from("<III", elf, pos)
            desc = pos + 12 + (nsz + 3) // 4 * 4
            if typ == NT_AMDGPU_METADATA:
                yield elf[desc:desc + dsz]
            pos = desc + (dsz + 3) // 4 * 4


@pytest.fixture(scope="module")
def kernels():
    with open(LIB, "rb") as f:
        blob = f.read()
    out = {}
    for elf in code_objects(blob):
        for d in notes(elf):
            for k in msgpack.unpackb(d)["amdhsa.kernels"]:
                out[k[".name"]] = k
    return out


# k_fwd_state<NB, DK, DV, F, TIO, NSL, RS, R, VARLEN>
NAME = re.compile(r"k_fwd_stateILi(\d+)ELi(\d+)ELi(\d+)EDv4_(ff|DF16bDF16b)"
                  r"Li(\d+)ELi(\d+)ELi(\d+)ELb([01])E")


def state_kernels(kernels, dt):
    out = {}
    for name, k in kernels.items():
        m = NAME.search(name)
        if m and (m[4] == "ff") == (dt == "f32"):
            out[tuple(int(m[i]) for i in (1, 2, 3, 5, 6, 7, 8))] = k
    assert len(out) >= 24  # 3 chunk sizes, 4 widths, plain and packed
    return out


def per_cu(k):
    """Workgroups a compute unit holds: 160 KiB of LDS, four SIMDs of 512
    registers a lane, given out in eights."""
    waves = k[".max_flat_workgroup_size"] // 64
    regs = (k[".vgpr_count"] + 7) // 8 * 8
    return min(160 * 1024 // k[".group_segment_fixed_size"], 4 * min(8, 512 // regs) // waves)


@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_state_pass_keeps_its_values_in_registers(kernels, dt):
    for shape, k in state_kernels(kernels, dt).items():
        assert k[".vgpr_spill_count"] == 0 and k[".private_segment_fixed_size"] == 0, shape


def test_fp32_one_slice_workgroups_share_a_cu(kernels):
    # past the CUs, C = 16 (ring of 2) and C = 64 with dk = 64 (ring of 1)
    seen = 0
    for (NB, DK, DV, NSL, RS, R, packed), k in state_kernels(kernels, "f32").items():
        if NSL == 1 and RS == 1 and (NB == 1 or (NB == 4 and DK == 64 and R == 1)):
            assert per_cu(k) >= 2, (NB, DK, DV, packed)
            seen += 1
    assert seen == 12
