"""Builds and loads tests/device_fmath.hip, device functions of the package on
their own, with the package's own flags."""
import ctypes
import os
import subprocess

from paper_2004_00304_amd import build as hipbuild

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(HERE, "device_fmath.so")


def build(force: bool = True) -> str:
    if force or not os.path.exists(LIB):
        subprocess.run(["hipcc", *hipbuild.FLAGS, "-shared", "-I", hipbuild.CSRC, "-o", LIB + ".tmp",
                        os.path.join(HERE, "device_fmath.hip")], check=True)
        os.replace(LIB + ".tmp", LIB)
    return LIB


def load():
    lib = ctypes.CDLL(build(force=False))
    p = ctypes.c_void_p
    lib.device_terms.argtypes = [ctypes.c_uint32, ctypes.c_uint32, p, p, p, p, p]
    return lib
