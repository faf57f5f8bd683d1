"""Registers and scratch memory of the kernels in the built libplic.so, from the
metadata the compiler writes beside each.  No kernel spills and none has scratch
memory: a spilled register's reload inside a branch runs for the branch's lanes
only once the compiler has taken the execution mask's restore there for
redundant, and the other lanes go on with a stale value (the flag that keeps the
restores is checked too)."""
import os
import struct

import msgpack
import pytest

import paper_2006_12838_amd._build as build

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(data):
    """The gfx950 images in a shared library's offload bundles."""
    at = data.find(MAGIC)
    while at >= 0:
        count, = struct.unpack_from("<Q", data, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(count):
            offset, size, idlen = struct.unpack_from("<QQQ", data, p)
            name = data[p + 24:p + 24 + idlen]
            p += 24 + idlen
            if name.endswith(b"gfx950") and size:
                yield data[at + offset:at + offset + size]
        at = data.find(MAGIC, p)


def metadata(elf):
    """The kernels' metadata: the note of type 32 (msgpack) of an ELF image."""
    shoff, = struct.unpack_from("<Q", elf, 40)
    shentsize, shnum = struct.unpack_from("<HH", elf, 58)
    for k in range(shnum):
        kind, _, _, offset, size = struct.unpack_from("<IQQQQ", elf, shoff + k * shentsize + 4)
        end = offset + size
        while kind == 7 and offset < end:
            namesz, descsz, note = struct.unpack_from("<III", elf, offset)
            desc = offset + 12 + (namesz + 3) // 4 * 4
            if note == 32:
                yield from msgpack.unpackb(elf[desc:desc + descsz])["amdhsa.kernels"]
            offset = desc + (descsz + 3) // 4 * 4


@pytest.fixture(scope="module")
def kernels():
    if not os.path.exists(build.LIB):
        pytest.skip("libplic.so is not built")
    with open(build.LIB, "rb") as f:
        data = f.read()
    return {k[".name"]: k for elf in code_objects(data) for k in metadata(elf)}


def test_no_kernel_spills_or_has_scratch(kernels):
    assert sum("k_curv_quads" in n for n in kernels) == 96 and sum("k_offset" in n for n in kernels) > 50
    for name, k in kernels.items():
        assert k[".private_segment_fixed_size"] == 0 and not k[".uses_dynamic_stack"], name
        assert k[".vgpr_spill_count"] == 0, name   # (scalars spill to lanes of a vector register, read whatever the mask)


def test_execution_mask_restores_are_kept():
    at = build.FLAGS.index("-mllvm=-amdgpu-remove-redundant-endcf=0")
    assert build.FLAGS[at - 1] == "-Xarch_device"


def waves(kernel):
    """wavefronts per SIMD that a kernel's registers allow (512, by 8)"""
    return 512 // ((kernel[".vgpr_count"] + 7) // 8 * 8)


@pytest.mark.parametrize("solver,rows", [("sz", 0), ("sz", 1), ("analytic", 1)])
def test_closed_forms_in_fp64_keep_four_wavefronts(kernels, solver, rows):
    """float arrays, FP64 arithmetic, four problems a thread"""
    name = f"k_offsetILi{['analytic', 'sz'].index(solver)}EfddLi4ELb{rows}E"
    assert [waves(k) for n, k in kernels.items() if name in n] == [4]


@pytest.mark.parametrize("rows", [0, 1])
def test_unaligned_kawano_in_fp64_keeps_five_wavefronts(kernels, rows):
    """float arrays, FP64 arithmetic, one problem a thread"""
    assert [waves(k) for n, k in kernels.items() if f"k_offsetILi4EfddLi1ELb{rows}E" in n] == [5]
