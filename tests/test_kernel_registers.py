"""Wavefronts per SIMD that the built kernels leave room for, from the metadata that the compiler puts beside them."""
import re
import struct

import msgpack
import pytest

from paper_2502_16949_amd import binding as B

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _notes(elf):
    """(type, contents) of the notes of a 64-bit ELF file."""
    shoff, = struct.unpack_from("<Q", elf, 40)
    shentsize, shnum = struct.unpack_from("<HH", elf, 58)
    for i in range(shnum):
        kind, _, _, at, size = struct.unpack_from("<IQQQQ", elf, shoff + i * shentsize + 4)
        end = at + size
        while kind == 7 and at + 12 <= end:                # SHT_NOTE
            namesz, descsz, what = struct.unpack_from("<III", elf, at)
            desc = at + 12 + (namesz + 3) // 4 * 4
            yield what, elf[desc:desc + descsz]
            at = desc + (descsz + 3) // 4 * 4


@pytest.fixture(scope="module")
def kernels():
    """Mangled kernel name -> what the compiler says about it."""
    lib = open(B.LIB_PATH, "rb").read()
    out = {}
    for m in re.finditer(MAGIC, lib):
        at = m.end()
        n, = struct.unpack_from("<Q", lib, at)
        at += 8
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", lib, at)
            at += 24 + idlen
            if lib[at - idlen:at].endswith(b"gfx950"):
                for what, desc in _notes(lib[m.start() + off:m.start() + off + size]):
                    if what == 32:                         # NT_AMDGPU_METADATA
                        out.update((k[".name"], k) for k in msgpack.unpackb(desc)["amdhsa.kernels"])
    assert len(out) > 100
    return out


@pytest.fixture(scope="module")
def registers(kernels):
    """Mangled kernel name -> vector registers (of both kinds)."""
    return {name: k[".vgpr_count"] for name, k in kernels.items()}


def _waves(vgprs):
    return min(8, 512 // ((vgprs + 7) // 8 * 8))


# The fix-up of one row or one column slice per workgroup (the loop over slices is a kernel of its own): the registers of a
# row's sum, two to eight partial rows in flight, and with the update fused the table row and its new values.
@pytest.mark.parametrize("iters,fused,waves", [(1, 0, 8), (1, 1, 8), (2, 0, 8), (2, 1, 8), (3, 0, 8), (3, 1, 6), (4, 0, 7), (4, 1, 4)])
def test_fixup_of_single_slices(registers, iters, fused, waves):
    seen = [v for k, v in registers.items()
            if re.search(r"k_seg_fixupILi\d+ELi%dELi\d+ELb%dELi0E(Lb0E)?E" % (iters, fused), k)]
    assert seen and all(_waves(v) >= waves for v in seen), seen


# The fix-up whose workgroups take several column slices: 65 registers were a wavefront less, and 40.0 us in place of 34.3.
def test_fixup_of_many_slices(registers):
    seen = [v for k, v in registers.items() if re.search(r"k_seg_fixupILi16ELi1ELi16ELb[01]ELi0ELb1EE", k)]
    assert len(seen) == 2 and all(_waves(v) >= 8 for v in seen), seen


# Distances over rows of y of one float4 per lane (all that a projection can be wide): nothing of them goes to memory.
def test_distances_over_rows_of_y_do_not_spill(kernels):
    seen = [k[".vgpr_spill_count"] for name, k in kernels.items() if re.search(r"k_forward_yILi\d+ELi1E", name)]
    assert len(seen) == 20 and not any(seen), seen


# TransR's fused forward kernel for operand rows of up to 64 floats, which stages as many float4 a thread as they have.
def test_transr_fused_stages_narrow_rows(registers):
    seen = [v for k, v in registers.items() if re.search(r"k_transr_fusedILi\dELi[24]EE", k)]
    assert len(seen) == 10 and all(_waves(v) >= 4 for v in seen), seen
