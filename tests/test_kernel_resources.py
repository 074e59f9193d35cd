"""Registers of the built kernels, from the notes of the code objects in libspa.so: how many workgroups of a kernel a unit
holds is part of its design, and a spill in a loop is paid on every turn."""
import os
import re
import struct

import pytest

from paper_2410_23608_amd import build as spa_build


@pytest.fixture(scope="module")
def kernels():
    """{demangled enough: (registers, spilled registers, scratch bytes, LDS bytes)}"""
    msgpack = pytest.importorskip("msgpack")
    b, out, at = open(spa_build.LIB_PATH, "rb").read(), {}, 0
    while (at := b.find(b"\x7fELF", at)) >= 0:
        if b[at + 4] == 2 and struct.unpack_from("<H", b, at + 18)[0] == 224:              # 64 bits, AMD GPU
            sections, count = struct.unpack_from("<Q", b, at + 40)[0], struct.unpack_from("<H", b, at + 60)[0]
            for o in (at + sections + 64 * i for i in range(count)):
                if struct.unpack_from("<I", b, o + 4)[0] == 7:                               # notes
                    p = at + struct.unpack_from("<Q", b, o + 24)[0]
                    name, size, kind = struct.unpack_from("<III", b, p)
                    if kind == 32:                                                           # the metadata
                        start = p + 12 + (name + 3) // 4 * 4
                        for k in msgpack.unpackb(b[start:start + size])["amdhsa.kernels"]:
                            out[k[".name"]] = (k[".vgpr_count"], k[".vgpr_spill_count"], k[".private_segment_fixed_size"],
                                               k[".group_segment_fixed_size"])
        at += 4
    assert len(out) > 100
    return out


def _waves(registers):                                                                       # of a SIMD, 512 registers a lane
    return 512 // ((registers + 7) // 8 * 8)


@pytest.mark.parametrize("pattern,count,waves", [
    (r"attn_fwd_bf16_tiled_kernelILi64E", 4, 3),
    (r"attn_fwd_bf16_tiled_kernelILi32ELi4ELi0E", 4, 4),                                # past 768 blocks
    (r"attn_fwd_bf16_tiled_kernelILi32ELi4ELi2E", 4, 3),
    (r"attn_fwd_bf16_group_kernel", 4, 4),
    (r"attn_fwd_bf16_wave_kernelILi1ELi32ELi64ELi[01]E", 2, 3),                              # 64-key steps, in order and gathered
    (r"attn_fwd_bf16_wave_kernelILi1ELi64ELi64ELi[01]E", 2, 2),
])
def test_waves_of_a_simd(kernels, pattern, count, waves):
    found = {n: k for n, k in kernels.items() if re.search(pattern, n)}
    assert len(found) == count
    for name, (registers, spilled, scratch, lds) in found.items():
        assert _waves(registers) >= waves and spilled == scratch == 0, name
        if "tiled" in name or "group" in name:                                               # four waves a workgroup
            assert waves * lds <= 160 * 1024, name


def test_no_kernel_spills(kernels):
    assert [n for n, k in kernels.items() if k[1] or k[2]] == []


def test_lanes_that_exchange_through_lds_order_their_memory():
    """A wave's LDS operations run in order, but __builtin_amdgcn_wave_barrier alone leaves the compiler free to move them across it:
    a fence of the wavefront stands before each."""
    found = 0
    for name in sorted(os.listdir(spa_build.CSRC)):
        with open(os.path.join(spa_build.CSRC, name)) as f:
            lines = f.read().splitlines()
        for before, line in zip(lines, lines[1:]):
            if "__builtin_amdgcn_wave_barrier()" in line:
                found += 1
                assert '__builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront")' in before, (name, line)
    assert found >= 3
