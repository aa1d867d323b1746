"""Registers of the compiled kernels: the code objects in the library carry each
kernel's VGPRs and spills.  The DP kernels that fill the device keep every value
of a step in registers; a spilled one costs scratch traffic in every step.  No
GPU is touched here."""
import re
import struct

import pytest

from paper_2210_08052_amd import mpg

msgpack = pytest.importorskip("msgpack")


def _notes(elf):
    """(type, descriptor) of every note of an ELF64 image."""
    shoff = struct.unpack_from("<Q", elf, 0x28)[0]
    size, num = struct.unpack_from("<HH", elf, 0x3A)
    for s in range(num):
        head = shoff + s * size
        if struct.unpack_from("<I", elf, head + 4)[0] != 7:  # SHT_NOTE
            continue
        at, length = struct.unpack_from("<QQ", elf, head + 0x18)
        end = at + length
        while at < end:
            nlen, dlen, kind = struct.unpack_from("<III", elf, at)
            at += 12 + (nlen + 3 & ~3)
            yield kind, elf[at:at + dlen]
            at += dlen + 3 & ~3


@pytest.fixture(scope="module")
def kernels():
    """Metadata of every kernel of the library, by mangled name."""
    mpg.lib()
    data = open(mpg.LIB_PATH, "rb").read()
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    out = {}
    for m in re.finditer(re.escape(magic), data):
        at = m.end()
        count = struct.unpack_from("<Q", data, at)[0]
        at += 8
        for _ in range(count):
            off, size, tlen = struct.unpack_from("<QQQ", data, at)
            triple = data[at + 24:at + 24 + tlen]
            at += 24 + tlen
            if b"amdgcn" not in triple or not size:
                continue
            elf = data[m.start() + off:m.start() + off + size]
            for kind, desc in _notes(elf):
                if kind == 32:  # NT_AMDGPU_METADATA
                    for k in msgpack.unpackb(desc)["amdhsa.kernels"]:
                        out[k[".name"]] = k
    assert out, "no code object in %s" % mpg.LIB_PATH
    return out


def _select(kernels, template, args):
    """The kernels of a template whose arguments match (None: any)."""
    found = {}
    for name, k in kernels.items():
        m = re.search(r"%d%sI((?:L[ib]\d+E)+)E" % (len(template), template), name)
        if m:
            got = tuple(int(x) for x in re.findall(r"L[ib](\d+)E", m.group(1)))
            if all(a is None or a == g for a, g in zip(args, got)):
                found[got] = k
    assert found, (template, args)
    return found


@pytest.mark.parametrize("K", [1, 2])
def test_integer_form_without_spills(kernels, K):
    """<columns per lane, mode, traceback, no introns, no frameshifts, profile,
    fp32 form>: the integer form at widths 1 and 2."""
    for args, k in _select(kernels, "dp_kernel", (K, None, None, None, None, None, 0)).items():
        assert k[".vgpr_spill_count"] == 0, (args, k[".vgpr_count"], k[".vgpr_spill_count"])


@pytest.mark.parametrize("K", [1, 2])
def test_int16_without_spills(kernels, K):
    """<columns per lane, no introns, no frameshifts, three-input form>: both
    forms of the 16-bit kernel."""
    for args, k in _select(kernels, "dp16_kernel", (K, None, None, None)).items():
        assert k[".vgpr_spill_count"] == 0, (args, k[".vgpr_count"], k[".vgpr_spill_count"])
