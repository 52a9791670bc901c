"""Host code of the library compiled for tests that need no GPU."""
import atexit
import ctypes
import os
import shutil
import subprocess
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(os.path.dirname(HERE))
CSRC = os.path.join(ROOT, "paper_2310_05037_amd", "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


_built = {}


def _folder():
    path = tempfile.mkdtemp(prefix="rawalign_host_")
    atexit.register(shutil.rmtree, path, ignore_errors=True)
    return path


def compile_host(*sources):
    """A shared library of C++ sources (of this folder, or library sources by
    name), compiled once and loaded anew each time: no state of earlier loads."""
    if sources not in _built:
        paths = [p if os.path.exists(p) else os.path.join(CSRC, s) for s in sources for p in [os.path.join(HERE, s)]]
        out = os.path.join(_folder(), "host.so")
        subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-ffp-contract=off", "-Wl,-Bsymbolic", "-D__HIP_PLATFORM_AMD__",
                        "-I", os.path.join(ROCM, "include"), "-I", os.path.join(ROOT, "include"), "-I", CSRC, *paths,
                        "-o", out], check=True)
        _built[sources] = out
    copy = os.path.join(_folder(), "host.so")
    shutil.copy(_built[sources], copy)
    return ctypes.CDLL(copy)
