"""Parity with the oracle at the edges of the default tile size (grids of just
under and over 128 and 512 tiles of 1280 particles, alone and as a batch) and of
the replicated cell sums (tiles of one, two, four and eight dense cells at 512
threads), both collision rules, with the deterministic sums too."""
import pytest

from paper_2004_00304_amd import workloads as W
from tests.gpu_util import RTOL32, RTOL64, assert_parity, banner, compare_state
from tests.test_gpu_parity import env  # noqa: F401


pytestmark = pytest.mark.gpu


def dense(tile, **kw):
    return W.paper_centreline(180, n=(9, 12, 1), yhi=6, tile=(*tile, 0), wg_threads=512, **kw)


CASES = {
    "tiles_under_128": (W.make(n=(116, 32, 1)), 4),
    "tiles_over_128": (W.make(n=(128, 32, 1)), 4),
    "tiles_under_512": (W.make(n=(480, 32, 1), part_fp=32), 3),
    "tiles_over_512": (W.make(n=(509, 32, 1), part_fp=32), 3),
    "dense_1": (dense((1, 1)), 5),
    "dense_2": (dense((2, 1)), 5),
    "dense_4": (dense((2, 2)), 5),
    "dense_8": (dense((4, 2)), 5),
    "dense_srd": (dense((1, 1), collision=0), 5),
    "dense_fp32": (dense((2, 1), part_fp=32), 5),
    "dense_deterministic": (dense((2, 2), deterministic=1), 5),
}


@pytest.mark.parametrize("name", list(CASES))
def test_parity(env, name):  # noqa: F811
    O, lbmpcd = env
    p, steps = CASES[name]
    banner(f"tile rule {name}")
    sim, orc = lbmpcd.Sim(p), O.Oracle(p)
    sim.step(steps)
    orc.step(steps)
    rtol = RTOL64 if p["part_fp"] == 64 else RTOL32
    assert_parity(compare_state(sim, orc, p, rtol), rtol)


def test_batch_counts_all_channels(env):  # noqa: F811
    """Two channels whose tiles together pass the edge take the larger tile
    and agree with the oracle channel by channel."""
    O, lbmpcd = env
    ps = [W.make(n=(64, 32, 1), instance=i) for i in range(2)]
    sim = lbmpcd.Sim(ps)
    sim.step(4)
    b = [sim.binning(i) for i in range(2)]
    for i, p in enumerate(ps):
        orc = O.Oracle(p)
        orc.step(4)
        assert_parity(compare_state(sim, orc, p, RTOL64, inst=i, binning=b[i]), RTOL64)
