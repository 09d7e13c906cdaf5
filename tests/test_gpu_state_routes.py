"""Particle state by id on both sides of the sizes at which its routes change:
reads through the inverse map from 2^19 binary32 particles in 3D and 2^24
otherwise, writes in the tiles' order from 2^25.  After some steps have mixed
the tiles, positions and velocities written by set_state come back exactly."""
import pytest

from paper_2004_00304_amd import workloads as W
from tests.gpu_util import banner
from tests.test_gpu_parity import env  # noqa: F401

pytestmark = pytest.mark.gpu

CASES = {
    "3d_fp32_below": W.small_3d(part_fp=32, n=(64, 16, 40)),             # 512,000
    "3d_fp32_map": W.small_3d(part_fp=32, n=(67, 16, 41)),               # 549,400
    "2d_fp32_below": W.small_2d(part_fp=32, n=(14563, 24, 1), ppc=9),    # 16,776,576
    "2d_fp32_map": W.small_2d(part_fp=32, n=(14567, 24, 1), ppc=9),      # 16,781,184
    "2d_fp64_map": W.small_2d(n=(14567, 24, 1), ppc=9),
    "2d_fp32_in_order": W.small_2d(part_fp=32, n=(21847, 24, 1), ppc=12),  # 33,556,992
}


@pytest.mark.parametrize("name", list(CASES))
def test_state_roundtrip(env, name):  # noqa: F811
    _, lbmpcd = env
    import torch
    p = CASES[name]
    banner(f"state routes {name}: {W.sizes(p)['particles']} particles")
    sim = lbmpcd.Sim(p)
    sim.step(2)
    cells = sim.moments("cell_id")
    pos = sim.get_state("pos")
    gen = torch.Generator(device="cuda").manual_seed(5)
    vel = torch.randn(pos.numel(), dtype=torch.float64, device="cuda", generator=gen)
    if p["part_fp"] == 32:
        vel = vel.float().double()
    sim.set_state("vel", vel)
    assert torch.equal(sim.get_state("vel"), vel)
    # the same positions by another route of the particle, mirrored and back
    x = pos.reshape(p["dim"], -1)
    sim.set_state("pos", x.flip(1).contiguous())
    assert torch.equal(sim.get_state("pos").reshape(x.shape), x.flip(1))
    sim.set_state("pos", pos)
    assert torch.equal(sim.get_state("pos"), pos) and torch.equal(sim.moments("cell_id"), cells)


def test_second_channel_of_a_batch(env):  # noqa: F811
    """The map of a channel whose slots do not start the buffer."""
    _, lbmpcd = env
    import torch
    ps = [W.small_3d(part_fp=32, n=(20 + 3 * i, 16, 10 + i), instance=i) for i in range(2)] + [CASES["3d_fp32_map"]]
    sim = lbmpcd.Sim(ps)
    sim.step(2)
    gen = torch.Generator(device="cuda").manual_seed(6)
    want = [torch.randn(3 * W.sizes(p)["particles"], device="cuda", generator=gen).double() for p in ps]
    for i, v in enumerate(want):
        sim.set_state("vel", v, inst=i)
    for i in (2, 0, 1, 2):
        assert torch.equal(sim.get_state("vel", inst=i), want[i]), i
