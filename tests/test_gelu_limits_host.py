"""GELU at the ends of binary32: x for large x and for infinity, 0 for large
negative x, and NaN only for NaN (csrc/gelu.hpp, compiled for the host)."""
import math

import numpy as np

from tests.test_gelu_host import run  # noqa: F401


def test_limits(run):  # noqa: F811
    big = [1e2, 1e10, 1e18, 1e19, 3.4e38, math.inf]
    g = run(big + [-b for b in big] + [math.nan])[2]
    x = np.array(big, np.float32).astype(np.float64)
    assert np.array_equal(g[:6], x), g[:6]
    assert np.all(g[6:12] == 0.0), g[6:12]
    assert math.isnan(g[12])
