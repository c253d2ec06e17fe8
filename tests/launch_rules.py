"""launch_rules.cpp as a library (not collected by pytest)."""
import ctypes as C
import functools
import os
import subprocess
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))


@functools.lru_cache(maxsize=None)
def rules():
    with tempfile.TemporaryDirectory() as d:
        so = os.path.join(d, "launch_rules.so")
        subprocess.run([os.environ.get("CXX", "g++"), "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC",
                        os.path.join(HERE, "launch_rules.cpp"), "-o", so], check=True)
        return C.CDLL(so)
