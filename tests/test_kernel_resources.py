"""Registers and scratch memory of the built kernels, read from the metadata of
libppl.so's own code objects (no GPU needed)."""
import os
import struct

import pytest

msgpack = pytest.importorskip("msgpack")

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2010_08454_amd", "libppl.so")


def _code_objects(blob):
    """The gfx950 code objects of every offload bundle in a shared library."""
    magic, at = b"__CLANG_OFFLOAD_BUNDLE__", 0
    while (at := blob.find(magic, at)) >= 0:
        count, = struct.unpack_from("<Q", blob, at + len(magic))
        p = at + len(magic) + 8
        for _ in range(count):
            off, size, tlen = struct.unpack_from("<QQQ", blob, p)
            if b"gfx950" in blob[p + 24:p + 24 + tlen]:
                yield blob[at + off:at + off + size]
            p += 24 + tlen
        at += len(magic)


def _kernels(elf):
    """The kernel records of an ELF code object's metadata note."""
    sections, = struct.unpack_from("<Q", elf, 40)
    size, count = struct.unpack_from("<HH", elf, 58)
    for k in range(count):
        _, kind, _, _, off, _ = struct.unpack_from("<IIQQQQ", elf, sections + k * size)
        if kind == 7:                                  # SHT_NOTE
            nlen, dlen, _ = struct.unpack_from("<III", elf, off)
            at = off + 12 + (nlen + 3) // 4 * 4
            yield from msgpack.unpackb(elf[at:at + dlen])["amdhsa.kernels"]


@pytest.fixture(scope="module")
def kernels():
    with open(LIB, "rb") as f:
        blob = f.read()
    found = {k[".name"]: k for elf in _code_objects(blob) for k in _kernels(elf)}
    assert found, "no gfx950 kernels in the library"
    return found


def test_state_space_filter_keeps_its_state_in_registers(kernels):
    """Particles, log-weights and the noise drawn ahead stay in registers across
    the grid exchanges at every count of particles per lane."""
    mine = {n: k for n, k in kernels.items() if "smc_persistent_kernelINS_5LgssmE" in n}
    assert len(mine) == 8
    assert {n: k[".private_segment_fixed_size"] for n, k in mine.items()} == {n: 0 for n in mine}


def test_chains_keep_their_tables_in_registers(kernels):
    """Neither scratch memory nor an LDS table inside a Metropolis-Hastings
    iteration: the static LDS is the reduction's alone (30 sums of four waves, 8
    of four lanes for every row of 16)."""
    lds = {"mcmc_poly_kernelE": 30 * 4 * 8, "mcmc_poly_quad_kernelE": 16 * 4 * 8 * 8}
    for part, size in lds.items():
        k, = [k for n, k in kernels.items() if part in n]
        assert k[".private_segment_fixed_size"] == 0
        assert k[".group_segment_fixed_size"] == size
