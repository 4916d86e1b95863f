"""Vector registers of kernels whose speed rests on how many wavefronts a SIMD holds, read from the built library (no GPU needed)."""
import os
import re
import struct
import subprocess

import pytest

from paper_2205_14135_amd import build

READELF = "/opt/rocm/llvm/bin/llvm-readelf"


def _device_objects(data):
    """The code objects for the GPU inside the library's bytes (ELF files of machine 224)."""
    at = data.find(b"\x7fELF", 1)
    while at >= 0:
        if struct.unpack_from("<H", data, at + 18)[0] == 224:
            section_table, entry, count = struct.unpack_from("<Q", data, at + 40)[0], *struct.unpack_from("<HH", data, at + 58)
            yield data[at:at + section_table + entry * count]
        at = data.find(b"\x7fELF", at + 1)


@pytest.fixture(scope="module")
def registers(tmp_path_factory):
    """(kernel, template arguments) -> vector registers, both 16-bit types"""
    folder, out = tmp_path_factory.mktemp("objects"), {}
    with open(build.LIB, "rb") as f:
        for n, obj in enumerate(_device_objects(f.read())):
            path = os.path.join(str(folder), f"{n}.elf")
            with open(path, "wb") as g:
                g.write(obj)
            notes = subprocess.run([READELF, "--notes", path], capture_output=True, text=True, check=True).stdout
            for kernel in notes.split("- .agpr_count:")[1:]:
                name, count = re.search(r"\.name:\s+(\S+)", kernel).group(1), int(re.search(r"\.vgpr_count:\s+(\d+)", kernel).group(1))
                m = re.search(r"_GLOBAL__N_1\d+([a-z]\w*_kernel)I(?:DF16_|DF16b)((?:L[ib]\d+E)*)", name)
                if m:
                    key = (m.group(1), tuple(int(x) for x in re.findall(r"L[ib](\d+)E", m.group(2))))
                    out[key] = max(out.get(key, 0), count)
    return out


# <d, causal, dropout, block-sparse, wavefronts, groups>: three wavefronts per SIMD hold 168 registers each
@pytest.mark.parametrize("args", [(32, c, p, s, 4, 1) for c in (0, 1) for p in (0, 1) for s in (0, 1)] + [(32, c, p, 0, 2, 2) for c in (0, 1) for p in (0, 1)])
def test_dq_of_narrow_heads(registers, args):
    assert registers["dq_kernel", args] <= 168


@pytest.mark.parametrize("args", [(d, c, p, s, 4, 1) for d in (32, 64) for c in (0, 1) for p in (0, 1) for s in (0, 1)])
def test_forward_up_to_64_columns(registers, args):
    assert registers["fwd_kernel", args] <= 168
