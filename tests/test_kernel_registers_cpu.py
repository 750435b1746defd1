"""Registers of the built kernels (CPU: read from libocc.so's own code object metadata).

A collective's workgroup runs beside a GEMM's on one CU, and with the device-side
counter it occupies its CU while it waits for GEMM workgroups that still have to be
placed: both must fit in a SIMD's 512 vector registers at once."""
import os
import struct

import pytest

from paper_2606_09200_amd import binding

msgpack = pytest.importorskip("msgpack")

SIMD_VGPRS, GRANULE = 512, 8


def code_objects(path):
    """The gfx950 code objects (ELF images) bundled in a shared library."""
    data = open(path, "rb").read()
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = data.find(magic)
    while at >= 0:
        n, = struct.unpack_from("<Q", data, at + 24)
        p = at + 32
        for _ in range(n):
            offset, size, idlen = struct.unpack_from("<QQQ", data, p)
            target = data[p + 24:p + 24 + idlen]
            p += 24 + idlen
            if target.endswith(b"gfx950") and size:
                yield data[at + offset:at + offset + size]
        at = data.find(magic, at + 1)


def kernels(elf):
    """amdhsa.kernels of a code object's metadata note (type 32 of "AMDGPU")."""
    shoff, = struct.unpack_from("<Q", elf, 0x28)
    entsize, count = struct.unpack_from("<HH", elf, 0x3A)
    for i in range(count):
        _, kind, _, _, offset, size = struct.unpack_from("<IIQQQQ", elf, shoff + i * entsize)
        if kind != 7:  # SHT_NOTE
            continue
        p = offset
        while p + 12 <= offset + size:
            namesz, descsz, ntype = struct.unpack_from("<III", elf, p)
            desc = p + 12 + (namesz + 3) // 4 * 4
            if ntype == 32 and elf[p + 12:p + 12 + 6] == b"AMDGPU":
                yield from msgpack.unpackb(elf[desc:desc + descsz])["amdhsa.kernels"]
            p = desc + (descsz + 3) // 4 * 4


@pytest.fixture(scope="module")
def built():
    if not os.path.exists(binding.LIB_PATH):
        pytest.skip("libocc.so is not built")
    found = [k for elf in code_objects(binding.LIB_PATH) for k in kernels(elf)]
    gemm = [k for k in found if "gemm_" in k[".name"]]
    comm = [k for k in found if "reduce_vec" in k[".name"] or "permute_vec" in k[".name"]]
    assert len(gemm) > 20 and len(comm) > 20
    return gemm, comm


def test_collective_fits_beside_every_gemm(built):
    gemm, comm = built

    def per_simd(k):
        waves = -(-k[".max_flat_workgroup_size"] // 64)
        return -(-waves // 4) * (-(-k[".vgpr_count"] // GRANULE) * GRANULE)

    beside = max(per_simd(k) for k in comm)
    for k in gemm:
        assert per_simd(k) + beside <= SIMD_VGPRS, (k[".name"], k[".vgpr_count"], beside)


def test_no_kernel_spills(built):
    for k in built[0] + built[1]:
        assert k.get(".vgpr_spill_count", 0) == 0 and k.get(".private_segment_fixed_size", 0) == 0, k[".name"]
