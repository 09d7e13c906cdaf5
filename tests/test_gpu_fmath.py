"""The binary32 functions of the Box-Muller transform as the device computes them
(hardware reciprocal and reciprocal root with Newton steps instead of the IEEE
division and root): on all 2^24 arguments that the generator produces they are
the oracle's to the bit, whose every step is an IEEE binary32 operation."""
import ctypes
import os
import shutil
import subprocess

import pytest

from tests import device_lib

pytestmark = pytest.mark.gpu

CHECK = r"""
#include <math.h>
#include <stdint.h>
#include <string.h>
extern "C" float orc_ln32(float x);
extern "C" void orc_sincos32(float u, float* sn, float* cs);
static uint32_t bits(float v) { uint32_t b; memcpy(&b, &v, 4); return b; }
extern "C" void differ(uint32_t n, const float* ln, const float* radius, const float* sn, const float* cs, long* bad) {
    for (uint32_t k = 0; k < n; ++k) {
        const float a = (float)k * 0x1p-24f, l = orc_ln32(1.0f - a);
        float s, c;
        orc_sincos32(a, &s, &c);
        bad[0] += bits(ln[k]) != bits(l);
        bad[1] += bits(radius[k]) != bits(sqrtf(-2.0f * l));
        bad[2] += bits(sn[k]) != bits(s) || bits(cs[k]) != bits(c);
    }
}
"""


def test_binary32_pair_equals_the_oracle_bit_for_bit(tmp_path):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not found")
    from oracle import oracle as O
    n = 1 << 24
    lib = device_lib.load()
    out = torch.empty((4, n), dtype=torch.float32, device="cuda")
    at = [ctypes.c_void_p(out[i].data_ptr()) for i in range(4)]
    assert lib.device_terms(0, n, *at, ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0
    host = out.cpu()
    so = O.build(force=False)
    src, exe = tmp_path / "c.cpp", tmp_path / "c.so"
    src.write_text(CHECK)
    subprocess.run([gxx, "-O2", "-ffp-contract=off", "-fno-fast-math", "-fPIC", "-shared", str(src), so, "-o", str(exe),
                    "-lm", f"-Wl,-rpath,{os.path.dirname(so)}"], check=True)
    check = ctypes.CDLL(str(exe))
    bad = (ctypes.c_long * 3)()
    check.differ(ctypes.c_uint32(n), *[ctypes.c_void_p(host[i].data_ptr()) for i in range(4)], bad)
    assert list(bad) == [0, 0, 0], list(bad)
