"""What the built kernels ask for (the metadata that the compiler leaves in libmorlax.so's code objects): registers per lane where one
more would cost a workgroup of a CU, and no scratch memory where a kernel is meant to live in its registers."""
import os
import re
import struct

import pytest

from paper_2603_09237_amd import binding

msgpack = pytest.importorskip("msgpack")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(blob):
    """The gfx950 code objects of every offload bundle in a library."""
    for at in (m.start() for m in re.finditer(MAGIC, blob)):
        n, pos = struct.unpack_from("<Q", blob, at + len(MAGIC))[0], at + len(MAGIC) + 8
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", blob, pos)
            ident = blob[pos + 24:pos + 24 + idlen]
            pos += 24 + idlen
            if b"gfx950" in ident and size:
                yield blob[at + off:at + off + size]


def kernels(elf):
    """name -> metadata, from the AMDGPU note of one code object."""
    phoff, phentsize, phnum = struct.unpack_from("<Q", elf, 32)[0], *struct.unpack_from("<HH", elf, 54)
    for i in range(phnum):
        kind, _, off, _, _, size = struct.unpack_from("<IIQQQQ", elf, phoff + i * phentsize)
        if kind != 4:   # PT_NOTE
            continue
        namesz, descsz, note = struct.unpack_from("<III", elf, off)
        if note == 32:  # NT_AMDGPU_METADATA
            start = off + 12 + (namesz + 3) // 4 * 4
            return {k[".name"]: k for k in msgpack.unpackb(elf[start:start + descsz])["amdhsa.kernels"]}
    return {}


@pytest.fixture(scope="module")
def built():
    if not os.path.exists(binding.LIB_PATH):
        from paper_2603_09237_amd import build
        build.build(verbose=False)
    found = {}
    for elf in code_objects(open(binding.LIB_PATH, "rb").read()):
        found.update(kernels(elf))
    assert len(found) > 100
    return found


def of(built, pattern):
    hit = {n: k for n, k in built.items() if re.search(pattern, n)}
    assert hit, pattern
    return hit


@pytest.mark.parametrize("pattern", [r"k_ppo_loss_grad", r"k_hyper_dM_df", r"k_hyper_materialize"])
def test_no_scratch_memory(pattern, built):
    assert {n: k[".private_segment_fixed_size"] for n, k in of(built, pattern).items() if k[".private_segment_fixed_size"]} == {}


# pattern, registers: workgroups of eight waves, two of them to a CU; of four waves, four and three of them
@pytest.mark.parametrize("pattern, registers", [(r"k_hyper_dM_dfILi2E", 128), (r"k_hyper_materializeI(f|DF16b)Li[024]E", 128),
                                                (r"k_hyper_materializeI(f|DF16b)Li8E", 168)])
def test_registers_leave_room_for_the_workgroups_of_a_cu(pattern, registers, built):
    assert {n: k[".vgpr_count"] for n, k in of(built, pattern).items() if k[".vgpr_count"] > registers} == {}


@pytest.mark.parametrize("pattern", [r"k_hyper_dM_dfILi\dELb\dELi0E"])
def test_scalars_stay_scalar(pattern, built):
    """No table of kernel arguments is kept in the lanes of vector registers through a loop."""
    assert {n: k[".sgpr_spill_count"] for n, k in of(built, pattern).items() if k[".sgpr_spill_count"]} == {}
