"""Registers of the built kernels that count their global -> LDS loads themselves: a spilled register that is reloaded inside the loop
waits for every tile in flight, and copies between the two register files cost issue slots beside the MFMAs."""
import os
import struct
import subprocess

import msgpack
import pytest

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_15422_amd", "libdualkv.so")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"
NOTE_SEGMENT, NOTE_AMDGPU_METADATA = 4, 32


def _notes(elf):
    off, = struct.unpack_from("<Q", elf, 32)
    size, count = struct.unpack_from("<HH", elf, 54)
    for i in range(count):
        kind, _, at, _, _, n = struct.unpack_from("<IIQQQQ", elf, off + i * size)
        end = at + n
        while kind == NOTE_SEGMENT and at < end:
            name, desc, note = struct.unpack_from("<III", elf, at)
            at += 12 + (name + 3) // 4 * 4
            if note == NOTE_AMDGPU_METADATA:
                yield msgpack.unpackb(elf[at:at + desc])
            at += (desc + 3) // 4 * 4


@pytest.fixture(scope="module")
def kernels():
    """demangled name -> code object metadata, of every kernel in the library"""
    if not os.path.exists(LIB):
        pytest.skip("library not built")
    with open(LIB, "rb") as f:
        data = f.read()
    found, at = {}, data.find(MAGIC)
    while at >= 0:
        n, = struct.unpack_from("<Q", data, at + 24)
        entry = at + 32
        for _ in range(n):
            off, size, name = struct.unpack_from("<QQQ", data, entry)
            if b"gfx950" in data[entry + 24:entry + 24 + name]:
                for meta in _notes(data[at + off:at + off + size]):
                    found.update((k[".name"], k) for k in meta["amdhsa.kernels"])
            entry += 24 + name
        at = data.find(MAGIC, at + 24)
    names = subprocess.run(["c++filt"], input="\n".join(found), text=True, capture_output=True, check=True).stdout.split("\n")
    return {a.split("(")[0].replace("void dkv::", ""): k for a, k in zip(names, found.values())}


@pytest.mark.parametrize("d", [64, 96, 128])
@pytest.mark.parametrize("local", ["true", "false"])
def test_no_spills_and_one_register_file(kernels, d, local):
    mine = [k for n, k in kernels.items() if n.startswith(("fwd2_kernel<%d," % d, "dq2_kernel<%d," % d)) and n.endswith(local + ">")]
    assert len(mine) >= 3
    for k in mine:
        assert (k[".vgpr_spill_count"], k[".private_segment_fixed_size"], k.get(".agpr_count", 0)) == (0, 0, 0), k[".name"]


@pytest.mark.parametrize("local", ["true", "false"])
def test_three_dq_workgroups_on_a_cu(kernels, local):
    """Head dim 64: three waves a SIMD share its 512 registers, in units of eight"""
    assert kernels["dq2_kernel<64, 4, %s>" % local][".vgpr_count"] <= 168


@pytest.mark.parametrize("d", [64, 96, 128])
@pytest.mark.parametrize("local", ["true", "false"])
def test_shared_launch(kernels, d, local):
    """dK/dV and dQ in one launch: one register at most, which the dK/dV part spills for the partial last row block of a sequence"""
    assert kernels["dkdv4_kernel<%d, %s, true>" % (d, local)][".vgpr_spill_count"] <= 1
