"""Host side of the library's internals (csrc/attn_common.h) for tests that need no GPU: a shim the host half alone, compiled against the built
library, called through ctypes."""
import ctypes
import os
import subprocess

from paper_2205_14135_amd import binding, build


def compile_shim(source: str, folder) -> ctypes.CDLL:
    """`source`, which sees attn_common.h and defines extern "C" functions, as a loaded shared library."""
    binding.load()
    src, out = os.path.join(str(folder), "shim.cpp"), os.path.join(str(folder), "shim.so")
    with open(src, "w") as f:
        f.write('#include "attn_common.h"\n' + source)
    r = subprocess.run([build._hipcc(), "-O1", "-std=c++17", "-fPIC", "-shared", "-x", "hip", "--cuda-host-only", "--offload-arch=gfx950", f"-I{build.CSRC}", src,
                        "-x", "none", build.LIB, f"-Wl,-rpath,{build.HERE}", "-o", out], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return ctypes.CDLL(out)
