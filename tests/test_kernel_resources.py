"""Registers of the state-dependent map flushes, from the built library's own
kernel metadata: an instance past one of these lines loses a wave per SIMD
(512 registers shared out in eights), which the map flushes, off the memory bus
for part of their life, pay for in time."""
import re
import struct
import subprocess

import pytest

from paper_2609_33051_amd import build

msgpack = pytest.importorskip("msgpack")


def _code_objects(data):
    """The gfx950 code objects of the library's offload bundles."""
    at = -1
    while (at := data.find(b"__CLANG_OFFLOAD_BUNDLE__", at + 1)) >= 0:
        p = at + 32
        for _ in range(struct.unpack_from("<Q", data, at + 24)[0]):
            off, size, n = struct.unpack_from("<QQQ", data, p)
            triple = data[p + 24:p + 24 + n]
            p += 24 + n
            if b"gfx950" in triple and size:
                yield data[at + off:at + off + size]


def _metadata(elf):
    """The AMDGPU metadata notes (msgpack) of one code object."""
    shoff = struct.unpack_from("<Q", elf, 40)[0]
    size, num = struct.unpack_from("<HH", elf, 58)
    for k in range(num):
        _, kind, _, _, off, length = struct.unpack_from("<IIQQQQ", elf, shoff + k * size)
        p = off
        while kind == 7 and p < off + length:  # SHT_NOTE
            nsz, dsz, t = struct.unpack_from("<III", elf, p)
            desc = p + 12 + (nsz + 3) // 4 * 4
            if elf[p + 12:p + 18] == b"AMDGPU" and t == 32:
                yield msgpack.unpackb(elf[desc:desc + dsz])
            p = desc + (dsz + 3) // 4 * 4


@pytest.fixture(scope="module")
def kernels():
    """{"update_kernel<0, 128, ...>": (registers, spilled registers)}"""
    out = {}
    for elf in _code_objects(open(build.LIB, "rb").read()):
        for m in _metadata(elf):
            for k in m["amdhsa.kernels"]:
                out[k[".name"]] = (k[".vgpr_count"], k[".vgpr_spill_count"])
    names = subprocess.run(["c++filt"], input="\n".join(out), capture_output=True, text=True, check=True).stdout
    return {re.sub(r"^void skssm::|\(.*$", "", d): out[n] for n, d in zip(out, names.split("\n"))}


@pytest.mark.parametrize("sketch", ["float", "unsigned short"])
@pytest.mark.parametrize("io", ["float", "unsigned short"])
@pytest.mark.parametrize("shape,P,most", [
    ("0, 128, 64, 8, 16", -1, 80), ("0, 128, 64, 16, 16", -1, 80),  # Mamba-2, exact map: six waves
    ("0, 128, 64, 16, 16", 4, 80), ("0, 128, 64, 32, 16", 4, 96),   # P = 4: six, five
    ("0, 128, 128, 32, 16", 4, 128),                                # K = V = 128, rank 32: four
    ("1, 128, 128, 16, 16", 4, 128), ("2, 128, 128, 16, 16", 4, 128), ("2, 128, 128, 16, 16", -1, 128)])
def test_map_flush_registers(kernels, shape, P, most, io, sketch):
    regs, spilled = kernels[f"update_kernel<{shape}, {io}, {sketch}, {P}>"]
    assert regs <= most and spilled == 0
