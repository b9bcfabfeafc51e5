"""Registers of the built kernels (CPU: the metadata notes of the library's
gfx950 code objects): no matrix-core matmul, row-attention or norm kernel
spills.  (The chunk-attention kernels may set aside a few outside their
loops.)"""
import struct

import pytest

from paper_2308_16369_amd import build

msgpack = pytest.importorskip("msgpack")


def _code_objects(lib):
    """The gfx950 ELF images of the library's offload bundles."""
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = lib.find(magic)
    while at >= 0:
        n, p = struct.unpack_from("<Q", lib, at + 24)[0], at + 32
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", lib, p)
            if b"gfx950" in lib[p + 24:p + 24 + idlen]:
                yield lib[at + off:at + off + size]
            p += 24 + idlen
        at = lib.find(magic, at + 24)


def _kernels(elf):
    """The kernels of one image: the AMDGPU metadata note of its note sections."""
    shoff, shentsize, shnum = struct.unpack_from("<Q", elf, 40)[0], *struct.unpack_from("<HH", elf, 58)
    for i in range(shnum):
        kind = struct.unpack_from("<I", elf, shoff + i * shentsize + 4)[0]
        off, size = struct.unpack_from("<QQ", elf, shoff + i * shentsize + 24)
        p, end = off, off + size
        while kind == 7 and p + 12 <= end:
            namesz, descsz, _ = struct.unpack_from("<III", elf, p)
            desc = p + 12 + (namesz + 3) // 4 * 4
            if elf[p + 12:p + 12 + namesz].rstrip(b"\0") == b"AMDGPU":
                yield from msgpack.unpackb(elf[desc:desc + descsz], raw=False)["amdhsa.kernels"]
            p = desc + (descsz + 3) // 4 * 4


def test_no_hot_kernel_spills_registers():
    with open(build.LIB, "rb") as f:
        lib = f.read()
    kernels = [k for elf in _code_objects(lib) for k in _kernels(elf)]
    names = ("gemm_ws", "gemm_quad", "gemm_bf16", "attn_rows", "norm_")
    hot = [k for k in kernels if any(n in k[".name"] for n in names)]
    assert len(hot) > 100
    spilled = {k[".name"]: (k[".sgpr_spill_count"], k[".vgpr_spill_count"]) for k in hot
               if k[".sgpr_spill_count"] or k[".vgpr_spill_count"] or k[".private_segment_fixed_size"]}
    assert not spilled
