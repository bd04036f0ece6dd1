"""Host builds of small pieces of the library's C++ sources, for tests that need no GPU."""
import ctypes
import os
import subprocess

from paper_2309_14717_amd import build as b


def host_library(tmp_path, name, source):
    """Compile `source` (extern "C" functions; may include headers of csrc/) for the host alone."""
    src, so = str(tmp_path / (name + ".hip")), str(tmp_path / (name + ".so"))
    with open(src, "w") as f:
        f.write(source)
    subprocess.run([b.HIPCC, "--offload-host-only", "-std=c++17", "-O3", "-fPIC", "-shared", "-I", b.CSRC, src, "-o", so],
                   check=True, capture_output=True)
    return ctypes.CDLL(os.path.abspath(so))
