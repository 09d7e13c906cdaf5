"""The closure network's fused kernels at the edges of their tiles, against
the FP64 model of oracle/mlp.py on identical BF16 operands: batches around the
32-row tile, the 128-row split of the weight gradients (one split, two, an
uneven last one), the largest batch with 128-row splits and one beyond it, and
the forward pass's change of tile at 8,192 rows.  Tolerances as in
test_gpu_closure.py: the accumulation is FP32 over at most 288 products
forward (BF16 rounding of the activations, 2^-8, flips rarely) and the
gradients sum up to 9,000 rows in FP32."""
import numpy as np
import pytest

from tests.gpu_util import banner
from tests.test_gpu_closure import channel, env, random_block, raw_data, rel_l2  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def net(env):  # noqa: F811
    torch, M, lbmpcd = env
    rng = np.random.default_rng(3)
    sim = lbmpcd.Sim(channel())
    block = random_block(M, rng)
    sim.closure_weights(block)
    X, Y = raw_data(M, rng, block, 9000)
    P = block[:M.NPARAM].astype(np.float64)
    st = block[M.NPARAM:].astype(np.float64)
    _, _, my, sy = M.split_stats(st)
    return torch, M, sim, X, Y, P, M.standardise(X, st), (M.network_targets(X, Y) - my) / sy, my, sy


@pytest.mark.parametrize("rows", [1, 31, 32, 33, 127, 129, 300, 8192, 8193, 9000])
def test_forward_and_gradient_at_tile_edges(net, rows):
    torch, M, sim, X, Y, P, Xs, Ys, my, sy = net
    Xt, Yt = torch.tensor(X[:rows], device="cuda"), torch.tensor(Y[:rows], device="cuda")
    out = sim.closure_forward(Xt).cpu().numpy().astype(np.float64)
    want = M.physical_outputs(X[:rows], M.forward(P, Xs[:rows])[0] * sy + my)
    el, nr = np.abs(out - want).max() / np.abs(want).max(), rel_l2(out, want)
    loss, G = sim.closure_loss_grad(Xt, Yt)
    lo, Go = M.loss_grad(P, Xs[:rows], Ys[:rows])
    ge = rel_l2(G, Go)
    banner(f"{rows} rows: forward max {el:.2e}, norm {nr:.2e}; loss {loss:.6g} (oracle {lo:.6g}); gradient {ge:.2e}")
    assert out.shape == want.shape and el <= 1e-2 and nr <= 1e-3
    assert abs(loss - lo) <= 1e-3 * lo
    assert ge <= 1e-2
