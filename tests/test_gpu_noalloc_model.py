"""lbmpcd_closure_forward_noalloc against the FP64 model of oracle/mlp.py at the
edges of its 32-row tiles and at its largest call.  Tolerances as in
test_gpu_closure_net.py."""
import numpy as np
import pytest

from tests.gpu_util import banner
from tests.test_gpu_closure import env, rel_l2  # noqa: F401
from tests.test_gpu_closure_net import net  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [1, 31, 33, 1000, 8192])
def test_noalloc_forward(net, rows):  # noqa: F811
    torch, M, sim, X, Y, P, Xs, Ys, my, sy = net
    out = sim.closure_forward_noalloc(torch.tensor(X[:rows], device="cuda")).cpu().numpy().astype(np.float64)
    want = M.physical_outputs(X[:rows], M.forward(P, Xs[:rows])[0] * sy + my)
    el, nr = np.abs(out - want).max() / np.abs(want).max(), rel_l2(out, want)
    banner(f"no-alloc forward, {rows} rows: max {el:.2e}, norm {nr:.2e}")
    assert out.shape == want.shape and el <= 1e-2 and nr <= 1e-3
