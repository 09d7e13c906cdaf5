"""Device memory that a caller hands over need only have the alignment of its
elements: a workspace 8 bytes past an aligned address and training scratch and
data 4 bytes past one give the results of aligned memory, although records,
node moments and training operands move in 16-byte vectors."""
import ctypes as C

import numpy as np
import pytest

from paper_2004_00304_amd import workloads as W
from tests.gpu_util import RTOL32, RTOL64, assert_parity, banner, compare_state
from tests.test_gpu_closure import channel, env, random_block, raw_data  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.fixture()
def shifted(env, monkeypatch):  # noqa: F811
    """Sim whose workspace starts 8 bytes past an aligned address."""
    torch, M, lbmpcd = env

    def make(p):
        empty = torch.empty

        def off(n, *a, **kw):
            return empty(n + 8, *a, **kw)[8:] if kw.get("dtype") == torch.uint8 else empty(n, *a, **kw)
        with monkeypatch.context() as m:
            m.setattr(torch, "empty", off)
            sim = lbmpcd.Sim(p)
        assert sim.workspace.data_ptr() % 16 == 8
        return sim
    return torch, M, lbmpcd, make


@pytest.mark.parametrize("p", [W.small_2d(), W.small_2d(part_fp=32), W.small_3d(), W.small_3d(part_fp=32, lb_fp=32)],
                         ids=["2d_fp64", "2d_fp32", "3d_fp64", "3d_fp32"])
def test_workspace(shifted, p):
    from oracle import oracle as O
    sim, orc = shifted[3](p), O.Oracle(p)
    banner(f"workspace 8 bytes off, {p['dim']}D binary{p['part_fp']}")
    sim.step(3)
    orc.step(3)
    rtol = RTOL64 if p["part_fp"] == 64 else RTOL32
    assert_parity(compare_state(sim, orc, p, rtol), rtol)


def test_closure(shifted):
    torch, M, lbmpcd, make = shifted
    rng = np.random.default_rng(2)
    block = random_block(M, rng)
    X, Y = raw_data(M, rng, block, 300)
    Xt, Yt = torch.tensor(X, device="cuda"), torch.tensor(Y, device="cuda")
    banner("closure 4 and 8 bytes off")
    res = []
    for sim, off in ((lbmpcd.Sim(channel()), 0), (make(channel()), 4)):
        sim.closure_weights(block)
        xs, ys = (torch.empty(t.numel() + 1, device="cuda")[off // 4:][:t.numel()] for t in (Xt, Yt))
        xs.copy_(Xt.reshape(-1))
        ys.copy_(Yt.reshape(-1))
        scr = torch.empty(lbmpcd.scratch_size(300, 300) + 4, dtype=torch.uint8, device="cuda")[off:]
        loss, G = C.c_double(), np.zeros(lbmpcd.CLOSURE_NPARAM, np.float32)
        assert lbmpcd._lib.lbmpcd_closure_loss_grad(
            sim._h, C.c_void_p(xs.data_ptr()), C.c_void_p(ys.data_ptr()), 300, C.c_void_p(scr.data_ptr()), scr.numel(),
            C.byref(loss), G.ctypes.data_as(C.c_void_p)) == 0
        out = torch.empty(300 * 9 + 1, device="cuda")[off // 4:]
        assert lbmpcd._lib.lbmpcd_closure_forward_noalloc(sim._h, C.c_void_p(xs.data_ptr()), 300, C.c_void_p(out.data_ptr())) == 0
        res.append((G, out[:2700].cpu().numpy(), sim.closure_predict().cpu().numpy()))
    for a, b in zip(*res):
        assert np.isfinite(a).all() and np.array_equal(a, b)
