"""Reading the state by id after tiles have overflowed: an id whose particle was
dropped has no slot, and its place in the caller's memory is left untouched,
with the scattered reads (small channels) and through the inverse map alike.
Which ids are lost is told by the cells, which are always scattered."""
import ctypes as C

import pytest

from paper_2004_00304_amd import workloads as W
from tests.gpu_util import banner
from tests.test_gpu_parity import env  # noqa: F401

pytestmark = pytest.mark.gpu

# capacity 0.9 and tiles of about 1,000 particles: their slots are full at the start
KW = dict(part_fp=32, capacity_factor=0.9, tile_target=1000, feedback=0)
CASES = {
    "scattered_3d": W.small_3d(n=(24, 16, 20), ppc=8, **KW),
    "map_3d": W.small_3d(n=(48, 16, 40), ppc=8, **KW),
    "scattered_2d": W.small_2d(n=(320, 24, 1), ppc=9, **KW),
    "map_2d": W.small_2d(n=(14600, 24, 1), ppc=9, **KW),
}


@pytest.mark.parametrize("name", list(CASES))
def test_lost_ids_are_left_untouched(env, name):  # noqa: F811
    _, lbmpcd = env
    import torch
    p = CASES[name]
    sim = lbmpcd.Sim(p)
    n, d = W.sizes(p)["particles"], p["dim"]

    def read(field, fill, dtype, per):
        out = torch.full((per, n), fill, dtype=dtype, device="cuda")
        with torch.cuda.device(sim.device):
            rc = lbmpcd._lib.lbmpcd_moments(sim._h, field, 0, C.c_void_p(out.data_ptr()),
                                            out.numel() * out.element_size(), 1)
        assert rc == 0
        return out

    lost_all = 0
    for steps in (1, 2, 3):
        sim.step(1)
        # a read before the step's own leaves its map in the idle buffer
        for field in (lbmpcd.PART_POS, lbmpcd.PART_VEL_PENDING, lbmpcd.PART_VEL, lbmpcd.PART_POS):
            lost = read(lbmpcd.CELL_ID, -7, torch.int32, 1)[0] == -7
            got = read(field, 1e300, torch.float64, d)
            assert bool((got[:, lost] == 1e300).all()), (steps, field, int(lost.sum()))
            assert bool((got[:, ~lost].abs() < 1e6).all()), (steps, field)
        lost_all = int(lost.sum())
    banner(f"lost ids {name}: {lost_all} of {n}")
    assert lost_all == sim.stats()["dropped"] > 0
