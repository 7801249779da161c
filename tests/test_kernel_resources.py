"""Resources of the built kernels, from the code objects' own metadata (no GPU)."""

from __future__ import annotations

import os
import struct

import pytest

msgpack = pytest.importorskip("msgpack")

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                   "paper_2607_18253_amd", "liblar.so")
BUNDLE = b"__CLANG_OFFLOAD_BUNDLE__"
NT_AMDGPU_METADATA = 32


def _code_objects(blob):
    """The gfx950 ELF images of every offload bundle in the library."""
    at = blob.find(BUNDLE)
    while at >= 0:
        (n,) = struct.unpack_from("<Q", blob, at + len(BUNDLE))
        x = at + len(BUNDLE) + 8
        for _ in range(n):
            off, size, len_id = struct.unpack_from("<QQQ", blob, x)
            name = blob[x + 24:x + 24 + len_id]
            x += 24 + len_id
            if b"gfx950" in name and size:
                yield blob[at + off:at + off + size]
        at = blob.find(BUNDLE, at + 1)


def _kernels(elf):
    """Metadata of each kernel of one 64-bit little-endian ELF image."""
    shoff, = struct.unpack_from("<Q", elf, 0x28)
    shentsize, shnum = struct.unpack_from("<HH", elf, 0x3A)
    for s in range(shnum):
        kind, = struct.unpack_from("<I", elf, shoff + s * shentsize + 4)
        if kind != 7:   # SHT_NOTE
            continue
        off, size = struct.unpack_from("<QQ", elf, shoff + s * shentsize + 24)
        x, end = off, off + size
        while x < end:
            namesz, descsz, ntype = struct.unpack_from("<III", elf, x)
            desc = x + 12 + (namesz + 3) // 4 * 4
            if ntype == NT_AMDGPU_METADATA:
                yield from msgpack.unpackb(elf[desc:desc + descsz])["amdhsa.kernels"]
            x = desc + (descsz + 3) // 4 * 4


@pytest.fixture(scope="module")
def kernels():
    if not os.path.exists(LIB):
        pytest.skip("liblar.so not built")
    blob = open(LIB, "rb").read()
    out = {k[".name"]: k for elf in _code_objects(blob) for k in _kernels(elf)}
    assert len(out) > 50
    return out


def test_limits_queues_stay_in_registers(kernels):
    """A wave of the engine under limits keeps its queue in registers at every width:
    scratch memory holds spilled registers at most, no arrays."""
    names = [n for n in kernels if any(f"{len(k)}{k}I" in n for k in (
        "k_lfront", "k_lest", "k_lcommit", "k_ltrace", "k_ltrace_cl", "k_ldrain"))]
    assert len(names) >= 40
    for n in names:
        k = kernels[n]
        spilled = 4 * k[".vgpr_spill_count"]
        assert k[".private_segment_fixed_size"] <= spilled + 16, n


@pytest.mark.parametrize("slots,per_cu", [(1, 4), (2, 4), (4, 3), (8, 2)])
def test_limits_traces_share_a_cu(kernels, slots, per_cu):
    """4-wave workgroups of the clustered trace under limits that one CU holds: a SIMD has
    512 registers per lane for one wave of each, the CU 160 KiB of LDS."""
    names = [n for n in kernels if f"11k_ltrace_clILi{slots}ELi4E" in n]
    assert len(names) == 2
    for n in names:
        k = kernels[n]
        vgprs = -(-k[".vgpr_count"] // 8) * 8 + -(-k.get(".agpr_count", 0) // 8) * 8
        assert vgprs * per_cu <= 512, n
        assert k[".group_segment_fixed_size"] * per_cu <= 160 * 1024, n


@pytest.mark.parametrize("waves,per_cu", [(1, 5), (2, 2)])
def test_wide_traces_of_few_instances_share_a_cu(kernels, waves, per_cu):
    """A trace of one or two instances of up to 1024 sequences holds the LDS of its own
    waves, so that several scenarios share a CU."""
    names = [n for n in kernels if f"10k_trace_clILi16ELi{waves}ELi1E" in n]
    assert len(names) == 2
    for n in names:
        assert kernels[n][".group_segment_fixed_size"] * per_cu <= 160 * 1024, n
