"""Registers that the inverted-residual block kernels spill, as the built library's own code objects state them: a form that holds more than
fits does so by choice, and their number does not grow unseen."""
import re
import struct
import subprocess

import pytest

from paper_2207_01260_amd import binding as B
from paper_2207_01260_amd import build

READELF = "/opt/rocm/llvm/bin/llvm-readelf"


def _code_objects(path):
    """The gfx950 ELF images in the library's offload bundles."""
    data = open(path, "rb").read()
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = data.find(magic)
    while at >= 0:
        p = at + len(magic)
        (count,) = struct.unpack_from("<Q", data, p)
        p += 8
        for _ in range(count):
            offset, size, n = struct.unpack_from("<QQQ", data, p)
            triple = data[p + 24:p + 24 + n]
            p += 24 + n
            if b"gfx950" in triple and size:
                yield data[at + offset:at + offset + size]
        at = data.find(magic, at + len(magic))


@pytest.fixture(scope="module")
def spills(tmp_path_factory):
    """{(type, window, stride, filter blocks, expansion units, rows): spilled registers} of mbrow_kernel."""
    B.lib()
    found = {}
    image = tmp_path_factory.mktemp("code") / "image.o"
    for elf in _code_objects(build.library_path()):
        if b"mbrow_kernelI" not in elf:
            continue
        image.write_bytes(elf)
        notes = subprocess.run([READELF, "--notes", str(image)], capture_output=True, text=True, check=True).stdout
        name = None
        for line in notes.splitlines():
            m = re.match(r"\s+\.name:\s+(\S+)", line)
            if m and m[1].startswith("_Z"):
                name = m[1]
            m = re.match(r"\s+\.vgpr_spill_count:\s+(\d+)", line)
            if m and name:
                f = re.search(r"mbrow_kernelI(DF16_|DF16b|f)Li(\d)ELi(\d)ELi(\d)ELi(\d+)ELi(\d)ELb0", name)
                if f:
                    found[(f[1],) + tuple(int(v) for v in f.groups()[1:])] = int(m[1])
                name = None
    assert len(found) > 150
    return found


def test_fp32_strips_of_128_filters(spills):
    """What suits 16-bit data (operands read a row ahead) is not done in fp32, where it does not fit."""
    forms = {f: n for f, n in spills.items() if f[0] == "f" and f[1] == 3}
    assert len(forms) == 6
    assert all(n <= 4 for n in forms.values()), forms


@pytest.mark.parametrize("dtype,most_forms,most", [("DF16b", 8, 60), ("DF16_", 6, 30)])
def test_strips_of_16_bit_data(spills, dtype, most_forms, most):
    """3x3 windows: their weights are held as fp32, and operands read a row ahead, by the forms that have the registers."""
    forms = {f: n for f, n in spills.items() if f[0] == dtype and f[1] == 3}
    assert len(forms) == 43
    spilled = {f: n for f, n in forms.items() if n}
    assert len(spilled) <= most_forms and max(spilled.values()) <= most, spilled
    # two sums' blocks and fewer, and the lower of the heights: nothing
    assert not any(f[3] <= 2 for f in spilled), spilled


@pytest.mark.parametrize("form,most", [(("DF16b", 5, 1, 4, 2, 2), 8), (("DF16b", 5, 1, 4, 4, 2), 14), (("DF16_", 5, 1, 6, 6, 2), 8)])
def test_5x5_strips(spills, form, most):
    """Forms that spilled up to twice as much with the strip's place handed over in a struct."""
    assert spills[form] <= most
