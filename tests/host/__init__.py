"""Host code of the library compiled for tests that need no GPU."""
import ctypes
import os
import subprocess
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(os.path.dirname(HERE))
CSRC = os.path.join(ROOT, "paper_2310_05037_amd", "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


def compile_host(*sources):
    """A shared library of C++ sources (paths from this folder, or library
    sources by name), loaded."""
    paths = [s if os.path.exists(s) else os.path.join(CSRC, s) for s in (os.path.join(HERE, s) if os.path.exists(
        os.path.join(HERE, s)) else s for s in sources)]
    out = os.path.join(tempfile.mkdtemp(prefix="rawalign_host_"), "host.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-ffp-contract=off", "-Wl,-Bsymbolic", "-D__HIP_PLATFORM_AMD__",
                    "-I", os.path.join(ROCM, "include"), "-I", os.path.join(ROOT, "include"), "-I", CSRC, *paths,
                    "-o", out], check=True)
    return ctypes.CDLL(out)
