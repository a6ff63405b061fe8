"""What the built kernels ask of a compute unit (512 registers per SIMD lane, four SIMDs, 160 KB of LDS), read from the
metadata that the compiler writes into the library: no GPU needed."""
import re
import struct

import msgpack
import pytest

from paper_2604_14825_amd import binding

REGISTERS, SIMDS, LDS = 512, 4, 160 << 10


def notes(elf):
    """Descriptors of the AMDGPU metadata notes (type 32) of a 64-bit code object."""
    shoff, = struct.unpack_from("<Q", elf, 0x28)
    shentsize, shnum = struct.unpack_from("<HH", elf, 0x3A)
    for i in range(shnum):
        base = shoff + i * shentsize
        kind, = struct.unpack_from("<I", elf, base + 4)
        if kind != 7:  # SHT_NOTE
            continue
        at, size = struct.unpack_from("<QQ", elf, base + 0x18)
        end = at + size
        while at + 12 <= end:
            namesz, descsz, ntype = struct.unpack_from("<III", elf, at)
            desc = at + 12 + (namesz + 3) // 4 * 4
            if ntype == 32:
                yield elf[desc : desc + descsz]
            at = desc + (descsz + 3) // 4 * 4


@pytest.fixture(scope="module")
def kernels():
    """Kernel name -> its metadata."""
    with open(binding.lib()._name, "rb") as f:
        data = f.read()
    found = {}
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    for m in re.finditer(magic, data):
        start = m.start()
        count, = struct.unpack_from("<Q", data, start + len(magic))
        at = start + len(magic) + 8
        for _ in range(count):
            offset, size, name_len = struct.unpack_from("<QQQ", data, at)
            name = data[at + 24 : at + 24 + name_len]
            at += 24 + name_len
            if b"gfx950" in name and size:
                for d in notes(data[start + offset : start + offset + size]):
                    for k in msgpack.unpackb(d)["amdhsa.kernels"]:
                        found[k[".name"]] = k
    assert found, "no gfx950 code object found in the library"
    return found


def work_groups_per_cu(k):
    waves = k[".max_flat_workgroup_size"] // 64
    registers = (k[".vgpr_count"] + 7) // 8 * 8
    return min(REGISTERS // registers * SIMDS // waves, LDS // k[".group_segment_fixed_size"])


def test_no_kernel_spills(kernels):
    for name, k in kernels.items():
        assert k[".private_segment_fixed_size"] == 0 and not k.get(".vgpr_spill_count", 0), name


@pytest.mark.parametrize("D,fp8,least", [(64, False, 4), (64, True, 4), (128, False, 2), (128, True, 2), (256, False, 2)])
def test_half_the_decode_wavefronts_share_a_cu(kernels, D, fp8, least):
    """Half the wavefronts of a split kernel keep half the bytes in flight: they are for work-groups that share a CU."""
    mark = "decode_split_fp8_kernelILi%dELi%dE" if fp8 else "decode_split_kernelILi%dELi[01]ELi%dE"
    mark %= (D, 2 if D > 128 else 4)
    forms = [k for name, k in kernels.items() if re.search(mark, name)]
    assert len(forms) == (1 if fp8 else 2), mark
    for k in forms:
        assert work_groups_per_cu(k) >= least, (k[".name"], k[".vgpr_count"], k[".group_segment_fixed_size"])
