"""The default tile size (host logic): on either side of each of the rule's edges
the workspace is that of the tile size which the rule names, for one channel,
for a batch that is counted together, and with a workgroup chosen by the caller."""
import pytest

from paper_2004_00304_amd import lbmpcd
from paper_2004_00304_amd import workloads as W

SIZES = (160, 320, 640, 1280)


def chosen(ps):
    """The tile size whose workspace the default has."""
    def size(t):
        return lbmpcd.workspace_size([{**p, "tile_target": t} for p in ps])
    sizes = {size(t): t for t in SIZES}
    assert len(sizes) == len(SIZES)
    return sizes[size(0)]


def channel(columns, **kw):
    """Tiles of 1280 are 64 x 2 cells: 17 on the 33 rows of every 16 nodes of length."""
    return W.make(n=(16 * columns, 32, 1), **kw)


F32, CE, AT = dict(part_fp=32), dict(reinject=1), dict(collision=1)


@pytest.mark.parametrize("kw,edges", [
    ({}, {128: (160, 320), 512: (320, 640), 2560: (640, 1280)}),
    (AT, {128: (160, 320), 512: (320, 640), 2560: (640, 1280)}),
    (CE, {512: (320, 640), 2560: (640, 1280)}),
    (F32, {128: (160, 320), 512: (320, 640), 1536: (640, 1280)}),
    ({**F32, **AT}, {512: (320, 640), 2560: (640, 1280)}),
    ({**F32, **CE}, {128: (160, 320), 384: (320, 1280)}),
    ({**F32, **CE, **AT}, {512: (320, 640), 1152: (640, 1280)}),
    (dict(wg_threads=256), {128: (160, 320), 2560: (640, 1280)}),
])
def test_edges(kw, edges):
    for edge, (below, above) in edges.items():
        assert chosen([channel((edge - 1) // 17, **kw)]) == below, (edge, kw)
        assert chosen([channel(-(-edge // 17), **kw)]) == above, (edge, kw)


@pytest.mark.parametrize("fp", [32, 64])
def test_3d(fp):
    # one tile of 4 x 2 x 8 cells in the channel's 512 x 65 x 256 cells cut in x and z
    assert chosen([W.channel_3d_scaled(16, 32, part_fp=fp)]) == 640
    assert chosen([W.channel_3d_scaled(8, 8, part_fp=fp)]) == 640
    assert chosen([W.channel_3d_scaled(8, 4, part_fp=fp)]) == 1280


def test_a_batch_is_counted_together():
    ps = [W.make(n=(64, 32, 1), instance=i) for i in range(2)]  # 68 tiles of 1280 each
    assert chosen(ps[:1]) == 160 and chosen(ps) == 320
    assert chosen([W.make(n=(64, 32, 1), instance=i) for i in range(8)]) == 640


@pytest.mark.parametrize("p", [channel(4), channel(16, **F32), W.channel_3d_scaled(8, 8)])
def test_a_callers_512_threads_take_full_tiles(p):
    assert chosen([{**p, "wg_threads": 512}]) == 1280
