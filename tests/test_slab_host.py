"""The exchange's buffer test for binary32 particles (csrc/slab.hpp, compiled for
the host with g++) against the rule it stands for: the particle's fine row,
clamped into the slab, lies in a buffer (the oracle's buffer_cell)."""
import os
import shutil
import subprocess

import numpy as np
import pytest

HDR = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2004_00304_amd", "csrc")

DRIVER = r"""
#include <stdio.h>
#include "slab.hpp"
int main() {
    int ylo, yhi, lo, hi;
    float below, from;
    while (scanf("%d %d %d %d", &ylo, &yhi, &lo, &hi) == 4) {
        lbmpcd::buffer_bounds(ylo, yhi, lo, hi, &below, &from);
        printf("%a %a\n", (double)below, (double)from);
    }
    return 0;
}
"""


@pytest.fixture(scope="module")
def bounds(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not found")
    d = tmp_path_factory.mktemp("slab")
    src, exe = d / "s.cpp", d / "s"
    src.write_text(DRIVER)
    subprocess.run([gxx, "-O2", "-I", HDR, str(src), "-o", str(exe)], check=True)

    def call(cases):
        out = subprocess.run([str(exe)], input="\n".join(" ".join(map(str, c)) for c in cases), capture_output=True,
                             text=True, check=True).stdout.split()
        return [tuple(np.float32(float.fromhex(t)) for t in out[2 * i:2 * i + 2]) for i in range(len(cases))]
    return call


def test_bounds_equal_the_rows_rule(bounds):
    f = np.float32
    slabs = [(0, 1), (0, 8), (8, 16), (5, 6), (126, 130), (0, 70000)]
    cases = [(ylo, yhi, lo, hi) for ylo, yhi in slabs for lo in (0, 1, 2, yhi - ylo) for hi in (0, 1, 3, yhi - ylo)
             if lo + hi <= yhi - ylo]
    rng = np.random.default_rng(3)
    for (ylo, yhi, lo, hi), (below, frm) in zip(cases, bounds(cases)):
        edges = np.array([ylo, ylo + lo, yhi - hi, yhi, ylo - 3, yhi + 3, -0.0, 0.25, 1e-30], f)
        y = np.concatenate([edges, np.nextafter(edges, f(-np.inf)), np.nextafter(edges, f(np.inf)),
                            rng.uniform(ylo - 1, yhi + 1, 4000).astype(f), [f(np.inf), f(-np.inf)]])
        got = (y < below) | (y >= frm)
        for r in (1, 2, 3, 4, 7):
            R = (yhi - ylo) * r
            J = np.clip(np.floor((y.astype(np.float64) - ylo) * r), 0, R - 1)
            want = (J < lo * r) | (J >= R - hi * r)
            assert np.array_equal(got, want), (ylo, yhi, lo, hi, r, y[got != want])
