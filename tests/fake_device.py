"""The library on fake_device.cpp, a HIP runtime without a device: a piece of Python is run
in a process of its own in which `fake` is that runtime and F, S are the package's modules."""
import os
import subprocess
import sys
import textwrap

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PROLOGUE = """
import ctypes as C, sys
sys.path.insert(0, {root!r})
fake = C.CDLL({lib!r}, mode=C.RTLD_GLOBAL)
fake.fake_capacity.argtypes = [C.c_size_t]
fake.fake_extend.argtypes = [C.c_ulonglong]
fake.fake_iteration.argtypes = [C.c_long] * 6
fake.fake_used.restype = C.c_size_t
for f in ("faults", "spawns", "graphs"):
    getattr(fake, "fake_" + f).restype = C.c_long
import numpy as np
from paper_1305_6981_amd import fciqmc as F
from paper_1305_6981_amd import systems as S

def error(call, *args):
    # the code of the call's error (0: none)
    try:
        call(*args)
    except F.FciqmcError as e:
        return e.code
    return 0
"""


def build(folder):
    lib = os.path.join(str(folder), "libfake_device.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-w", "-D__HIP_PLATFORM_AMD__",
                    "-I/opt/rocm/include", "-o", lib, os.path.join(HERE, "fake_device.cpp")], check=True)
    return lib


def run(lib, code):
    text = PROLOGUE.format(root=ROOT, lib=lib) + textwrap.dedent(code)
    done = subprocess.run([sys.executable, "-c", text], capture_output=True, text=True, timeout=120)
    assert done.returncode == 0, done.stdout + done.stderr
    return done.stdout
