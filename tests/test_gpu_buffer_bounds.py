"""Binary32 particles on the slab's upper face, y = yhi: initial positions are
rounded to binary32, which lands a few of them there, and a caller may put
them there.  The fine row of such a particle is the last one, so it is in a
buffer only where the upper face has one."""
import numpy as np
import pytest

from paper_2004_00304_amd import workloads as W
from tests.gpu_util import RTOL32, assert_parity, banner, compare_state
from tests.test_gpu_parity import env  # noqa: F401

pytestmark = pytest.mark.gpu

SLABS = {
    "walled_2d": W.walled_2d(part_fp=32), "periodic_2d": W.periodic_2d(part_fp=32),
    "no_buffer_3d": W.small_3d(part_fp=32, buf_lo=0, buf_hi=0, feedback=0),
    "lower_buffer_2d": W.small_2d(part_fp=32, buf_lo=2, buf_hi=0, feedback=0),
    "top_wall_2d": W.small_2d(part_fp=32, ylo=16, yhi=24, buf_lo=2, buf_hi=0, feedback=0),
    "upper_buffer_3d": W.small_3d(part_fp=32, buf_lo=0, buf_hi=1, feedback=0),
    "all_buffer_2d": W.small_2d(part_fp=32, buf_lo=8, buf_hi=0, feedback=0),
    "at_top_wall_2d": W.small_2d(part_fp=32, ylo=16, yhi=24, buf_lo=2, buf_hi=0, feedback=0, collision=1),
}


@pytest.mark.parametrize("slab", list(SLABS))
def test_particles_on_the_upper_face(env, slab):  # noqa: F811
    O, lbmpcd = env
    p = SLABS[slab]
    banner(f"upper face {slab}")
    sim, orc = lbmpcd.Sim(p), O.Oracle(p)
    pos, vel = orc.particles()
    # one in fifty of the particles of the upper node row (their tile's window
    # holds the face's rows) and a few from anywhere else in the slab
    rng = np.random.default_rng(8)
    pick = np.flatnonzero((pos[1] > p["yhi"] - 1) & (rng.random(pos.shape[1]) < 0.02))
    pick = np.union1d(pick, rng.choice(pos.shape[1], 5, replace=False))
    pos[1, pick] = p["yhi"]
    pos = pos.astype(np.float32).astype(np.float64)
    orc.set_particles(pos, vel)
    sim.set_state("pos", pos.reshape(-1))
    sim.step(2)
    orc.step(2)
    assert_parity(compare_state(sim, orc, p, RTOL32), RTOL32)
