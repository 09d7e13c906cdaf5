"""The sampled profile against the oracle where particles re-wrapped across
the slab, short slabs and tall tiles meet the tile's LDS window of profile
rows: each row's count is exact, its velocity sums within 1e-11 of the count
(binary64) or 2e-6 (binary32 stores)."""
import numpy as np
import pytest

from paper_2004_00304_amd import workloads as W
from tests.gpu_util import banner
from tests.test_gpu_parity import env  # noqa: F401

pytestmark = pytest.mark.gpu

CASES = {
    # LB on both faces: particles leave one face and enter at the other
    "rewrap_2d": W.small_2d(feedback=0),
    "rewrap_2d_fp32": W.small_2d(feedback=0, part_fp=32),
    "rewrap_3d_feedback": W.small_3d(),
    "rewrap_3d_deterministic": W.small_3d(deterministic=1, feedback=0),
    # slabs of fewer rows than the window, down to one fine row
    "short_slab": W.small_2d(ylo=8, yhi=9, buf_lo=0, buf_hi=0, feedback=0),
    "one_row": W.small_2d(ylo=8, yhi=9, buf_lo=0, buf_hi=0, refine=1, feedback=0, ppc=20),
    # windows of more than eight rows, of the most rows, and of too many
    "rows_12": W.small_2d(tile=(4, 8, 0), feedback=0),
    "rows_over_16": W.small_2d(tile=(4, 16, 0), feedback=0),
    # 512 threads, and walls (no re-wrap)
    "wg512": W.small_2d(wg_threads=512, feedback=0),
    "walls": W.walled_2d(),
    "periodic": W.periodic_2d(),
}


@pytest.mark.parametrize("name", list(CASES))
def test_profile_rows(env, name):  # noqa: F811
    O, lbmpcd = env
    p = CASES[name]
    banner(f"profile window {name}")
    sim, orc = lbmpcd.Sim(p), O.Oracle(p)
    sim.sample(1)
    orc.sample(1)
    sim.step(5)
    orc.step(5)
    pg, (po, _) = sim.profile(), orc.profile()
    d = 1 + p["dim"]
    tol = 1e-11 if p["part_fp"] == 64 else 2e-6
    assert (pg[:, 0] == po[:, 0]).all()
    assert np.abs(pg[:, 1:d] - po[:, 1:d]).max() <= tol * np.abs(po[:, 0]).max()
