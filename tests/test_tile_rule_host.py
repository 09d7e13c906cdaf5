"""The default tile size (host logic): the workspace is that of the tile size
which the rule names, on either side of each of its edges, for one channel, for
a batch that is counted together, and with a workgroup chosen by the caller."""
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
    """33 rows of 64 cells for every 16 nodes of length, 10 particles in each:
    136, 68, 34 and 17 tiles of 160, 320, 640 and 1280 particles."""
    return W.make(n=(16 * columns, 32, 1), **kw)


@pytest.mark.parametrize("fp", [32, 64])
@pytest.mark.parametrize("at", [0, 1])
@pytest.mark.parametrize("substeps,sizes", [
    (4, {1: 160, 5: 160, 6: 320, 11: 320, 12: 640, 22: 640, 23: 1280, 200: 1280}),   # at most 768 tiles
    (8, {5: 160, 6: 320, 23: 1280}),
    (2, {1: 160, 2: 320, 3: 320, 4: 640, 7: 640, 8: 1280}),                          # at most 256
    (3, {1: 160, 2: 320, 8: 1280}),
    (1, {1: 160, 2: 320, 3: 640, 5: 640, 6: 1280}),                                  # at most 192
])
def test_edges(substeps, sizes, at, fp):
    for columns, size in sizes.items():
        assert chosen([channel(columns, substeps=substeps, collision=at, part_fp=fp)]) == size, columns


def test_chapman_enskog_in_binary64():
    for columns, size in {5: 160, 6: 320, 23: 640, 150: 640, 151: 1280}.items():   # 150 columns: 2,550 full tiles
        assert chosen([channel(columns, reinject=1)]) == size, columns
    assert chosen([channel(23, reinject=1, part_fp=32)]) == 1280
    assert chosen([channel(23, reinject=1, substeps=1)]) == 1280


@pytest.mark.parametrize("fp", [32, 64])
def test_3d(fp):
    assert chosen([W.channel_3d_scaled(32, 64, part_fp=fp)]) == 320
    assert chosen([W.channel_3d_scaled(16, 32, part_fp=fp)]) == 640
    assert chosen([W.channel_3d_scaled(16, 16, part_fp=fp)]) == 1280


def test_3d_without_refinement():
    assert chosen([W.small_3d(n=(48, 16, 40), refine=1, ppc=20)]) == 640
    assert chosen([W.small_3d(n=(24, 16, 20), refine=2, ppc=10)]) == 320


def test_a_batch_is_counted_together():
    ps = [channel(4, instance=i) for i in range(6)]   # 544 tiles of 160 each
    assert [chosen(ps[:k]) for k in (1, 2, 3, 5, 6)] == [160, 320, 640, 640, 1280]


def test_dense_cells_keep_full_tiles():
    """60 particles per cell: 160 and 320 would be tiles of eight cells."""
    p = W.make(n=(32, 32, 1), ppc=60)
    assert lbmpcd.workspace_size([p]) == lbmpcd.workspace_size([{**p, "tile_target": 640}])
    assert lbmpcd.workspace_size([p]) != lbmpcd.workspace_size([{**p, "tile_target": 320}])


@pytest.mark.parametrize("p", [channel(4), channel(16, part_fp=32), W.channel_3d_scaled(16, 32)])
def test_a_callers_512_threads_take_full_tiles(p):
    assert chosen([{**p, "wg_threads": 512}]) == 1280
    assert chosen([{**p, "wg_threads": 256}]) < 1280
