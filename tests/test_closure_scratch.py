"""Scratch sizes of the closure's training and forward calls (host logic): scratch
that serves some rows serves fewer as well, and the size of any row count is
computed at once."""
import time

from paper_2004_00304_amd import lbmpcd


def test_size_grows_with_the_rows():
    rows = sorted({*range(1, 2000, 13), *range(8000, 20000, 7), *range(8160, 8260), *(2 ** k + d for k in range(40) for d in (-1, 0, 1))} - {0})
    sizes = [lbmpcd.scratch_size(n) for n in rows]
    assert all(a <= b for a, b in zip(sizes, sizes[1:])), [(n, s) for n, s, t in zip(rows, sizes, sizes[1:]) if s > t][:4]
    # a batch takes what its own rows take, and no more than all of them
    assert lbmpcd.scratch_size(9000, 4096) == lbmpcd.scratch_size(4096) <= lbmpcd.scratch_size(9000)


def test_size_of_many_rows_is_computed_at_once():
    t0 = time.perf_counter()
    lbmpcd.scratch_size(1 << 44)
    assert time.perf_counter() - t0 < 1.0
