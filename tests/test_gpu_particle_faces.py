"""Particles that land on or next to the faces where the step kernel's range tests
decide: the ends of the periodic axes, the slab's faces and the buffers' edges,
and velocities that are not finite in every kind of slab (reflecting, walled,
periodic)."""
import numpy as np
import pytest

from paper_2004_00304_amd import workloads as W
from tests.gpu_util import RTOL32, RTOL64, assert_parity, banner, compare_state
from tests.test_gpu_parity import env  # noqa: F401


pytestmark = pytest.mark.gpu

SLABS = {
    "reflecting_2d": W.small_2d, "reflecting_3d": W.small_3d, "walled_2d": W.walled_2d, "periodic_2d": W.periodic_2d,
    "refine3_3d": lambda **kw: W.small_3d(refine=3, **kw), "no_buffer_2d": lambda **kw: W.small_2d(buf_lo=0, buf_hi=0, **kw),
}


@pytest.mark.parametrize("part_fp", [64, 32])
@pytest.mark.parametrize("slab", list(SLABS))
def test_landing_on_faces(env, slab, part_fp):  # noqa: F811
    O, lbmpcd = env
    p = SLABS[slab](part_fp=part_fp, feedback=0, g=(0.0, 0.0, 0.0))
    banner(f"faces {slab} binary{part_fp}")
    sim, orc = lbmpcd.Sim(p), O.Oracle(p)
    pos, vel = orc.particles()
    cast = np.float32 if part_fp == 32 else np.float64
    rng = np.random.default_rng(5)
    ends = {0: [0.0, p["n"][0]], 1: [p["ylo"], p["yhi"], p["ylo"] + p["buf_lo"], p["yhi"] - p["buf_hi"]], 2: [0.0, p["n"][2]]}
    for q in range(p["dim"]):
        # one in twenty of the particles within half a node of a face (more
        # would overfill the tiles at the faces)
        face = np.array(ends[q])[np.abs(pos[q][:, None] - np.array(ends[q])).argmin(1)]
        near = np.flatnonzero((np.abs(pos[q] - face) < 0.5) & (rng.random(pos.shape[1]) < 0.05))
        face = face[near]
        off = rng.choice([-1e-7, 0.0, 1e-7], near.size)
        vel[q, near] = ((face + off - pos[q, near]) * p["substeps"]).astype(cast)
    vel = vel.astype(cast).astype(np.float64)
    orc.set_particles(pos, vel)
    sim.set_state("vel", vel.reshape(-1))
    sim.step(2)
    orc.step(2)
    rtol = RTOL64 if part_fp == 64 else RTOL32
    assert_parity(compare_state(sim, orc, p, rtol), rtol)


@pytest.mark.parametrize("part_fp", [64, 32])
@pytest.mark.parametrize("bad", [(0.0, np.inf), (0.0, -np.inf), (0.0, np.nan), (-np.inf, 0.0), (np.nan, 1e30), (3e38, 0.0)])
@pytest.mark.parametrize("slab", ["reflecting_2d", "walled_2d", "periodic_2d"])
def test_invalid_velocity_is_parked(env, slab, bad, part_fp):  # noqa: F811
    _, lbmpcd = env
    p = SLABS[slab](part_fp=part_fp, feedback=0)
    banner(f"invalid {slab} {bad} binary{part_fp}")
    sim = lbmpcd.Sim(p)
    pos, vel = sim.particles()
    inside = (pos[1] > p["ylo"] + p["buf_lo"] + 0.2) & (pos[1] < p["yhi"] - p["buf_hi"] - 0.2)
    vel[:, int(np.flatnonzero(inside)[0])] = bad
    sim.set_state(lbmpcd.PART_VEL, vel.reshape(-1))
    sim.step(1)
    with pytest.raises(lbmpcd.LbmpcdError) as e:
        sim.sync()
    assert e.value.code == 5 and "invalid" in str(e.value), str(e.value)
    st = sim.stats()
    assert st["bad_state"] >= 1 and st["dropped"] == 0, st
    pos, vel = sim.particles()
    assert np.isfinite(pos).all() and np.isfinite(vel).all()
