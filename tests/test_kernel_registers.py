"""What the compiler made of the kernels, read from the code objects' metadata in libicv.so (no GPU needed)."""
import re
import struct

import msgpack

from paper_1907_02129_amd import binding as icv


def _code_objects(data: bytes):
    """The gfx950 ELF images of a library's offload bundles (one bundle per translation unit)."""
    at = data.find(b"__CLANG_OFFLOAD_BUNDLE__")
    while at >= 0:
        (n,) = struct.unpack_from("<Q", data, at + 24)
        pos = at + 32
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", data, pos)
            target = data[pos + 24:pos + 24 + idlen]
            pos += 24 + idlen
            if target.endswith(b"gfx950") and size:
                yield data[at + off:at + off + size]
        at = data.find(b"__CLANG_OFFLOAD_BUNDLE__", at + 24)


def _kernels(elf: bytes):
    """The kernel descriptions of one image: the AMDGPU metadata note (type 32), a msgpack map."""
    shoff, = struct.unpack_from("<Q", elf, 0x28)
    shentsize, shnum = struct.unpack_from("<HH", elf, 0x3A)
    for i in range(shnum):
        _, kind, _, _, off, size = struct.unpack_from("<IIQQQQ", elf, shoff + i * shentsize)
        if kind != 7:                                   # SHT_NOTE
            continue
        pos = off
        while pos < off + size:
            namesz, descsz, ntype = struct.unpack_from("<III", elf, pos)
            desc = pos + 12 + (namesz + 3) // 4 * 4
            if ntype == 32:
                yield from msgpack.unpackb(elf[desc:desc + descsz])["amdhsa.kernels"]
            pos = desc + (descsz + 3) // 4 * 4


def _all_kernels():
    with open(icv.LIB_PATH, "rb") as f:
        data = f.read()
    return {k[".name"]: k for elf in _code_objects(data) for k in _kernels(elf)}


def test_filter_in_registers_keeps_its_scalars():
    """A scalar spilled in this kernel is a vector lane read back in every pass, with one wavefront per SIMD to hide it.  With a
    batch-independent buffer and one row block per wavefront and pass none of the 3x3 ones spills; the others hold two
    copies of the output stage, 25 kernel elements or the whole batch's column mask."""
    spills = {}
    for name, k in _all_kernels().items():
        m = re.match(r"_ZN3icv12k_igemm_fregILi(\d)ELi(\d+)ELi(\d)ELi(\d)ELi(\d)ELb(\d)ELb(\d)E", name)
        if m:
            spills[tuple(map(int, m.groups()))] = k[".sgpr_spill_count"]
    assert len(spills) == 3 * 4 * 6 * 2 * 2             # types, shapes, column and row blocks, output stages, whole batch or one image
    most = {(9, 1, 1): 0, (9, 2, 1): 20, (25, 1, 1): 10, (25, 2, 1): 50, (9, 1, 0): 12, (9, 2, 0): 32, (25, 1, 0): 28, (25, 2, 0): 64}
    for (dt, T, KS, wn, mb, fused, img), n in spills.items():
        assert n <= most[T, mb, img], (dt, T, KS, wn, mb, fused, img, n)
