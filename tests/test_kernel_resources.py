"""The built library's own account of its kernels (the metadata the compiler leaves with each): none uses scratch
memory -- a kernel that spills registers pays for it on every frame -- and the batched kernels keep the
occupancy they are compiled for (CPU only)."""
from __future__ import annotations

import re
import struct

import msgpack
import pytest

from paper_2510_03964_amd import build as lib_build


def _code_objects(blob: bytes):
    """The gfx950 code objects of the offload bundles in a shared library."""
    at = blob.find(b"__CLANG_OFFLOAD_BUNDLE__")
    while at >= 0:
        count, = struct.unpack_from("<Q", blob, at + 24)
        p = at + 32
        for _ in range(count):
            offset, size, n = struct.unpack_from("<QQQ", blob, p)
            triple = blob[p + 24:p + 24 + n]
            p += 24 + n
            if b"gfx950" in triple and size:
                yield blob[at + offset:at + offset + size]
        at = blob.find(b"__CLANG_OFFLOAD_BUNDLE__", at + 24)


def _kernels(elf: bytes):
    """amdhsa.kernels of a code object's AMDGPU metadata note."""
    shoff, = struct.unpack_from("<Q", elf, 0x28)
    entry, count = struct.unpack_from("<HH", elf, 0x3A)
    for i in range(count):
        kind, = struct.unpack_from("<I", elf, shoff + i * entry + 4)
        offset, size = struct.unpack_from("<QQ", elf, shoff + i * entry + 0x18)
        if kind != 7:                                        # SHT_NOTE
            continue
        p = offset
        while p < offset + size:
            names, descs, typ = struct.unpack_from("<III", elf, p)
            name = elf[p + 12:p + 12 + names].rstrip(b"\0")
            d = p + 12 + (names + 3) // 4 * 4
            if name == b"AMDGPU" and typ == 32:
                yield from msgpack.unpackb(elf[d:d + descs])["amdhsa.kernels"]
            p = d + (descs + 3) // 4 * 4


@pytest.fixture(scope="module")
def kernels():
    with open(lib_build.LIB, "rb") as f:
        found = {k[".name"]: k for obj in _code_objects(f.read()) for k in _kernels(obj)}
    assert any("frame_kernel" in n for n in found) and any("tick_args_kernel" in n for n in found)
    return found


def test_no_kernel_uses_scratch(kernels):
    bad = {n: (k[".private_segment_fixed_size"], k[".vgpr_spill_count"]) for n, k in kernels.items()
           if k[".private_segment_fixed_size"] or k[".vgpr_spill_count"]}
    assert not bad, bad


def test_batched_kernels_keep_their_occupancy(kernels):
    """Waves per SIMD by vector registers (512 a lane and SIMD, allocated in eights), by kind of tick."""
    for kind, waves in enumerate((8, 8, 7, 5, 7, 7, 7, 5)):
        for name in (f"_ZN4fwrs11tick_kernelILi{kind}E", f"_ZN4fwrs16tick_args_kernelILi{kind}E"):
            k = next(v for n, v in kernels.items() if n.startswith(name))
            assert 512 // ((k[".vgpr_count"] + 7) // 8 * 8) >= waves, (name, k[".vgpr_count"])


def test_the_frame_kernels_are_those_that_the_rules_launch(kernels):
    """frame_kernel<slots, op, per-slot mode, tiles>: every instantiation is one that some frame takes."""
    launched = {(k, op, 0, 1) for k in (0, 1, 2, 4, 8) for op in (1, 2, 3, 5, 7, 8, 9)}
    launched |= {(k, op, 0, 2) for k in (0, 1, 2, 4) for op in (1, 5)}
    launched |= {(k, op, 1, t) for k, t in ((0, 1), (1, 1), (2, 1), (3, 0), (4, 0), (5, 0), (8, 0)) for op in (1, 3, 5)}
    built = {tuple(map(int, m.groups())) for m in
             (re.match(r"_ZN4fwrs12frame_kernelILi(\d+)ELi(\d+)ELb([01])ELi(\d+)E", n) for n in kernels) if m}
    assert built == launched
