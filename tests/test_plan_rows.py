"""What the planner lays down for rows that are no multiple of 16 bytes (how a receiving tile's lanes are dealt over the runs it
meets) and for elements a few apart, on the CPU."""
import ctypes as C

import numpy as np
import pytest

from tests.cases import Case, contig
from tests.test_plan_host import describe, interp  # noqa: F401


def lanes(interp, rb, col0, n):  # noqa: F811
    """(lanes, rounds of the kernel)"""
    interp.run_lanes_check.restype = C.c_int64
    rounds = C.c_uint32(0)
    return interp.run_lanes_check(C.c_uint32(rb), C.c_uint32(col0), C.c_uint32(n), C.byref(rounds)), rounds.value


@pytest.mark.parametrize("rb", [16, 17, 31, 32, 33, 202, 4099, 16383, 16384, 16385, 40001, 300007, (1 << 30) - 1])
def test_lanes_of_a_tile_are_those_of_its_bytes(interp, rb):  # noqa: F811
    """Inside one run, over the end of one and over many; parts of less than a vector, of whole vectors and not.  No more
    lanes than the parts have vectors begun (one a part beyond the tile's own), however long the runs are."""
    rng = np.random.default_rng(rb)
    starts = {0, 1, 15, 16, rb - 1, rb - 15, rb - 16, rb - 17, rb // 2, rb // 3} | {int(x) for x in rng.integers(0, rb, 6)}
    for col0 in sorted(c for c in starts if 0 <= c < rb):
        left = rb - col0
        for n in sorted({1, 15, 16, 17, 256, 8448, 16384, left, left - 1, left + 1, left + 15, left + 16, left + 17}):
            if 0 < n <= 1 << 16:
                runs = (col0 + n - 1) // rb + 1
                got = lanes(interp, rb, col0, n)[0]
                assert 0 < got <= n // 16 + runs, (rb, col0, n, got)


@pytest.mark.parametrize("rb", [64, 65, 79, 101, 202, 204, 404, 2006, 4099, 8193, 16385, 100514])
def test_a_whole_tile_takes_one_round(interp, rb):  # noqa: F811
    """However it lies in its runs, a tile of 16 KiB: a second round would be for a few dozen lanes alone."""
    for col0 in range(0, rb, max(1, rb // 97)):
        assert lanes(interp, rb, col0, 16384)[1] == 1, (rb, col0)


# (elements of a run, distance between them, element size, runs): the ones sent as elements a few apart.  Runs that are not whole
# numbers of the neighbours read at once only if they are long: a wave with such a group reads its elements one by one.
@pytest.mark.parametrize("views,sizes", [
    (((32, 2, 2),), 2), (((32, 4, 1),), 1), (((32, 2, 2), (32, 2, 1)), 3),
    (((31, 2, 2),), 0), (((32, 3, 2),), 0), (((32, 2, 4),), 0), (((32, 8, 1),), 0),
    (((31, 2, 2), (40, 4, 1)), 1),                           # of one size, a launch of the other has none
    (((31, 2, 2), (100, 2, 2)), 2),                          # one of them is enough for a launch
    (((33, 2, 2),), 0), (((101, 2, 2),), 0), (((4095, 2, 2),), 0), (((4097, 2, 2),), 2),
    (((36, 2, 1),), 0), (((1004, 2, 1),), 0), (((4097, 2, 1),), 1), (((102, 4, 1),), 0), (((4097, 4, 1),), 1),
    (((8, 2, 2),), 0), (((12, 2, 2),), 2), (((8, 2, 1),), 0), (((16, 2, 1),), 1), (((12, 4, 1),), 1),
    (((1024, 4, 2),), 0), (((5000, 4, 2),), 0),              # two at a time
    (((1499, 2, 2, 2200),), 0), (((1501, 2, 2, 2090),), 0), (((1501, 2, 2, 2100),), 2),        # either side of 6 MiB
    (((1501, 2, 1, 4190),), 0), (((1501, 2, 1, 4200),), 1), (((1024, 4, 2, 3071),), 0), (((1024, 4, 2, 3072),), 2), (((5001, 4, 2, 700),), 0),
    (((401, 2, 2, 31370),), 0), (((401, 2, 2, 31390),), 2), (((399, 2, 2, 32000),), 0),        # of 24 MiB
])
def test_the_plan_says_which_launches_have_elements_a_few_apart(interp, views, sizes):  # noqa: F811
    case = Case("apart", tuple(((rows[0] if rows else 9, n), (n * step + 5, step), es) for n, step, es, *rows in views) + (contig((100,), 2),), 3, 4096)
    descs, keep = describe(case)
    assert interp.apart_sizes(descs, len(case.tensors), case.k, C.c_uint64(case.B)) == sizes


@pytest.mark.parametrize("n,step,es,sizes", [(31, 2, 2, 0), (33, 2, 2, 2), (35, 4, 2, 2), (101, 2, 1, 1), (1 << 20, 4, 1, 1), (101, 3, 1, 0)])
def test_one_run_of_elements_a_few_apart(interp, n, step, es, sizes):  # noqa: F811
    descs, keep = describe(Case("run", (((n,), (step,), es),), 3, 4096))
    assert interp.apart_sizes(descs, 1, 3, C.c_uint64(4096)) == sizes
