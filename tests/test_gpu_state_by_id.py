"""Particle state by id through every record layout and both ways of reading
it (scattered components below 2^18 binary32 or 2^24 binary64 particles, the
inverse map from there on): after some steps have mixed the tiles, velocities
and positions written by set_state come back exactly, and reading them twice
gives the same, with the state's cells unchanged by the reads."""
import pytest

from paper_2004_00304_amd import workloads as W
from tests.gpu_util import banner
from tests.test_gpu_parity import env  # noqa: F401

pytestmark = pytest.mark.gpu

CASES = {
    "2d_fp32_small": W.small_2d(part_fp=32),
    "2d_fp32_map": W.small_2d(part_fp=32, n=(256, 24, 1), ppc=12),      # 393,216 particles
    "2d_fp64": W.small_2d(),
    "3d_fp32_small": W.small_3d(part_fp=32),
    "3d_fp32_map": W.small_3d(part_fp=32, n=(48, 16, 40), ppc=5),       # 384,000
    "3d_fp64": W.small_3d(),
    "3d_fp64_map": W.small_3d(n=(192, 16, 200), ppc=12),                # 18,432,000
}


@pytest.mark.parametrize("name", list(CASES))
def test_state_roundtrip(env, name):  # noqa: F811
    _, lbmpcd = env
    import torch
    p = CASES[name]
    banner(f"state by id {name}: {W.sizes(p)['particles']} particles")
    sim = lbmpcd.Sim(p)
    sim.step(3)
    cells = sim.moments("cell_id")
    pos = sim.get_state("pos")
    assert torch.equal(pos, sim.get_state("pos")) and torch.equal(cells, sim.moments("cell_id"))
    gen = torch.Generator(device="cuda").manual_seed(5)
    vel = torch.randn(pos.numel(), dtype=torch.float64, device="cuda", generator=gen)
    if p["part_fp"] == 32:
        vel = vel.float().double()
    sim.set_state("vel", vel)
    assert torch.equal(sim.get_state("vel"), vel)
    sim.set_state("pos", pos)
    assert torch.equal(sim.get_state("pos"), pos)
    d = p["dim"]
    x = pos.reshape(d, -1)
    hi = [p["n"][0], p["yhi"], p["n"][2]]
    lo = [0, p["ylo"], 0]
    for k in range(d):
        assert bool((x[k] >= lo[k]).all()) and bool((x[k] < hi[k]).all())
