"""Cell sums with and without replicas at 512 threads: channels of sparse cells
(none), of dense cells (replicated), and a context that holds both, whose one
kernel serves either."""
import pytest

from paper_2004_00304_amd import workloads as W
from tests.gpu_util import RTOL32, RTOL64, assert_parity, banner, compare_state
from tests.test_gpu_parity import env  # noqa: F401

pytestmark = pytest.mark.gpu


def sparse(**kw):
    return W.make(n=(24, 24, 1), ylo=0, yhi=12, buf_lo=0, buf_hi=2, refine=1, substeps=1, ppc=10, wg_threads=512,
                  tile=(16, 8, 0), **kw)


def dense(**kw):
    return W.make(n=(9, 12, 1), ylo=0, yhi=6, buf_lo=0, buf_hi=2, refine=1, substeps=1, ppc=180, wg_threads=512,
                  tile=(2, 1, 0), **kw)


@pytest.mark.parametrize("fp", [64, 32])
@pytest.mark.parametrize("mode", [{}, dict(collision=1), dict(reinject=1), dict(collision=1, deterministic=1)],
                         ids=["srd", "at", "ce", "at_deterministic"])
@pytest.mark.parametrize("which", ["sparse", "dense", "both"])
def test_parity(env, which, mode, fp):  # noqa: F811
    O, lbmpcd = env
    mk = {"sparse": [sparse], "dense": [dense], "both": [sparse, dense]}[which]
    ps = [f(part_fp=fp, instance=i, **mode) for i, f in enumerate(mk)]
    banner(f"replicas {which} {mode} binary{fp}")
    sim = lbmpcd.Sim(ps)
    sim.step(4)
    b = [sim.binning(i) for i in range(len(ps))]
    rtol = RTOL64 if fp == 64 else RTOL32
    for i, p in enumerate(ps):
        orc = O.Oracle(p)
        orc.step(4)
        assert_parity(compare_state(sim, orc, p, rtol, inst=i, binning=b[i]), rtol)
