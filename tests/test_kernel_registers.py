"""The built kernels, from the code objects in the library.

* Vector registers: kernels that are bound by how many waves a SIMD holds stay within the 128 registers (or
  another bound) that their launch rule counts on, without spills.
* Cache write-backs and invalidations of the group kernels' exchange between XCDs: each is waited for before the
  next memory operation (the compiler's fence alone does not wait where it knows of nothing else in flight).
"""
import os
import re
import struct

import msgpack
import pytest

from paper_1806_08422_amd import build


@pytest.fixture(scope="module")
def code_objects():
    """The gfx950 code objects (ELF images) of libnmfa.so."""
    if not os.path.exists(build.LIB):
        build.build()
    with open(build.LIB, "rb") as f:
        blob = f.read()
    out = []
    for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", blob):
        n, = struct.unpack_from("<Q", blob, m.start() + 24)
        q = m.start() + 32
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", blob, q)
            target = blob[q + 24:q + 24 + length]
            q += 24 + length
            if b"gfx950" in target:
                out.append(blob[m.start() + off:m.start() + off + size])
    assert out
    return out


@pytest.fixture(scope="module")
def kernels(code_objects):
    """name -> (vector registers, spilled registers) of every kernel."""
    out = {}
    for elf in code_objects:
        out.update(_metadata(elf))
    return out


def _metadata(elf):
    shoff, = struct.unpack_from("<Q", elf, 0x28)
    shsize, shnum = struct.unpack_from("<HH", elf, 0x3A)
    for i in range(shnum):
        if struct.unpack_from("<I", elf, shoff + i * shsize + 4)[0] != 7:  # SHT_NOTE
            continue
        o, = struct.unpack_from("<Q", elf, shoff + i * shsize + 24)
        name, desc, _ = struct.unpack_from("<III", elf, o)
        o += 12 + (name + 3) // 4 * 4
        doc = msgpack.unpackb(elf[o:o + desc], strict_map_key=False)
        return {k[".name"]: (k[".vgpr_count"], k[".vgpr_spill_count"]) for k in doc["amdhsa.kernels"]}
    return {}


def _sparse(kernels, P, RB, DM, QP, unroll):
    name = f"anneal_sparse_rqILi{P}ELi{RB}ELi{DM}ELi{QP}ELb{int(unroll)}E"
    found = [v for k, v in kernels.items() if name in k]
    assert len(found) == 1, name
    return found[0]


# FP32 (P = 1), one quad per thread: a workgroup of 512 threads is two waves per SIMD, and two of them share a CU
@pytest.mark.parametrize("RB,DM,unroll", [
    (1, 4, True), (1, 6, True), (1, 8, False), (1, 10, True), (2, 3, True), (2, 4, True), (2, 6, True), (2, 8, False),
    (2, 10, False), (4, 3, True)])
def test_sparse_kernel_leaves_four_waves(kernels, RB, DM, unroll):
    vgprs, spills = _sparse(kernels, 1, RB, DM, 1, unroll)
    assert vgprs <= 128 and spills == 0


# the batched small-N kernel: registers of the largest job of a launch, not of the largest there is (operand
# reads NK: BF16 N = 32 NK, FP32 N = 16 NK), so that a CU holds at least as many waves per SIMD as given
@pytest.mark.parametrize("P,j8,nk,waves", [
    (2, 0, 1, 8), (2, 0, 3, 6), (2, 0, 4, 5), (2, 1, 3, 6), (1, 0, 2, 6), (1, 0, 5, 6), (1, 0, 7, 5), (0, 0, 4, 3)])
def test_batched_kernel_registers(kernels, P, j8, nk, waves):
    name = f"anneal_small_batchedILi{P}ELb{j8}ELi{nk}E"
    found = [v for k, v in kernels.items() if name in k]
    assert len(found) == 1, name
    assert -(-found[0][0] // 8) * 8 <= 512 // waves


# the small-N kernel in FP32: 80 registers for six waves per SIMD up to 96 spins (16 per operand read)
@pytest.mark.parametrize("nk", [3, 5, 6])
def test_small_fp32_registers(kernels, nk):
    found = [v for k, v in kernels.items() if f"anneal_smallILi1ELb0ELi{nk}ELi1ELb0ELi1E" in k]
    assert len(found) == 1 and found[0][0] <= 80


def test_cache_operations_are_waited_for(code_objects):
    wait = struct.pack("<I", 0xBF8C0F70)  # s_waitcnt vmcnt(0)
    found = 0
    # buffer_wbl2 sc1, buffer_inv sc1
    for op in (b"\x00\x80\xa0\xe0\x00\x00\x00\x00", b"\x00\x80\xa4\xe0\x00\x00\x00\x00"):
        for elf in code_objects:
            for m in re.finditer(re.escape(op), elf):
                assert elf[m.end():m.end() + 4] == wait
                found += 1
    assert found >= 40  # both in every group kernel
