"""Registers of the traversal kernels as the built library's own metadata states
them.  16 waves a CU, four a SIMD, leave a kernel 128 vector registers: one more
and a SIMD holds three waves, and what a kernel spills it stores and loads again."""
import re
import struct
import subprocess

import msgpack
import pytest

import paper_2305_01867_amd as rsi


def _notes(elf):
    """The kernels' metadata records of one AMD GPU code object."""
    sections, = struct.unpack_from("<Q", elf, 40)
    size, count = struct.unpack_from("<HH", elf, 58)
    for i in range(count):
        kind, = struct.unpack_from("<I", elf, sections + i * size + 4)
        if kind != 7:  # SHT_NOTE
            continue
        at, length = struct.unpack_from("<QQ", elf, sections + i * size + 24)
        end = at + length
        while at < end:
            name, desc, note = struct.unpack_from("<III", elf, at)
            at += 12 + (name + 3 & ~3)
            if note == 32:  # NT_AMDGPU_METADATA
                yield from msgpack.unpackb(elf[at:at + desc])["amdhsa.kernels"]
            at += desc + 3 & ~3


def _kernels(path):
    data = open(path, "rb").read()
    for bundle in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", data):
        at = bundle.start() + 32
        for _ in range(struct.unpack_from("<Q", data, bundle.start() + 24)[0]):
            offset, size, name = struct.unpack_from("<QQQ", data, at)
            target = data[at + 24:at + 24 + name]
            at += 24 + name
            if b"gfx950" in target:
                yield from _notes(data[bundle.start() + offset:bundle.start() + offset + size])


@pytest.fixture(scope="module")
def kernels():
    found = {k[".name"]: k for k in _kernels(rsi.library_path)}
    names = subprocess.run(["c++filt"], input="\n".join(found), capture_output=True, text=True, check=True).stdout
    short = [re.sub(r".*::(k_\w+)(<.*>)?\(.*", r"\1\2", n) for n in names.splitlines()]
    return dict(zip(short, found.values()))


# vector registers that may go to memory: in the certified lane forms of the
# count's 4-wide pass around a binary64 decision, in the barycentric pool once
# per refill
SPILLS = {"k_traverse_count<true, false, true>": 8, "k_pool<2, true, true>": 1, "k_pool<2, true, false>": 1}


def test_the_first_pass_keeps_four_waves_a_simd_and_its_registers(kernels):
    first = {n: k for n, k in kernels.items() if re.match(r"k_(traverse|traverse_count|pool)\b", n)}
    assert len(first) == 24 + 24 + 8 + 16  # modes, precisions, orders and widths, plain and counted; pools
    for name, k in first.items():
        assert k[".vgpr_count"] <= 128, (name, k[".vgpr_count"])
        stats = re.match(r"k_traverse(_count)?<(\d, )?\w+, true,", name)  # (the counting copies: diagnostics)
        if not stats:
            assert k[".vgpr_spill_count"] <= SPILLS.get(name, 0), (name, k[".vgpr_spill_count"])
