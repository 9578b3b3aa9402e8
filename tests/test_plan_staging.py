"""The pieces in which the CPU-forwarding stream stages a message, on the CPU."""
import ctypes as C

import pytest

from oracle import hxt_oracle as ho
from tests.cases import Case, contig
from tests.test_plan_host import describe, interp, oracle_msg  # noqa: F401

KiB, MiB = 1 << 10, 1 << 20


def copies_of(interp, case, window):  # noqa: F811
    """[(offset, bytes, piece)] and the ranges of the packed buffer"""
    descs, keep = describe(case)
    out, ranges = (C.c_uint64 * 32)(), C.c_int(0)
    n = interp.staging_copies_of(descs, len(case.tensors), case.k, C.c_uint64(case.B), C.c_int(window), out, C.byref(ranges))
    assert 0 <= n <= 4
    return [tuple(out[3 * i:3 * i + 3]) for i in range(n)], ranges.value


def used_ranges(case):
    """The packed bytes that chunks use, neighbours merged."""
    m, out = oracle_msg(case), []
    infos = [ho.chunk_info(m, case.B, case.k, c) for c in range(ho.num_chunks(m, case.B))]
    for off, n in sorted((i["packed_off"], i["padded"]) for i in infos):
        if out and out[-1][0] + out[-1][1] == off:
            out[-1][1] += n
        else:
            out.append([off, n])
    return out


# Two ranges wherever the last chunk is short and not in the last lane.
@pytest.mark.parametrize("lanes,chunk", [(1, 4 * MiB), (3, 640 * KiB), (4, 2 * MiB), (8, 4 * MiB), (5, 256 * KiB), (8, 25 * MiB)])
@pytest.mark.parametrize("nbytes", [256, 5 * MiB + 300, 10 * MiB - 256, 10 * MiB, 14 * MiB - 256, 14 * MiB, 24 * MiB - 256, 24 * MiB, 25 * MiB + 300, 28 * MiB + 4096,
                                    4000 * 2 * 3584 * 2, 56 * MiB])
def test_pieces_cover_the_message_and_keep_to_the_copies_of_a_window(interp, lanes, chunk, nbytes):  # noqa: F811
    for last in range(lanes + 1):                            # a short last chunk in every lane
        case = Case("contig", (contig((nbytes + last * chunk,), 1),), lanes, chunk)
        want = used_ranges(case)
        total = sum(n for _, n in want)
        for window in (1, 2, 3, 4, 5, 6, 7, 8, 9, 16, 17, 1000):
            copies, ranges = copies_of(interp, case, window)
            assert ranges == len(want)
            pieces = [sum(n for _, n, q in copies if q == k) for k in range(copies[-1][2] + 1)]
            assert [q for _, _, q in copies] == sorted(q for _, _, q in copies)
            if window <= 4:
                want_pieces = 3 if total >= 14 * MiB else 2 if total >= 10 * MiB else 1
            else:
                want_pieces = max(1, min(3, 16 // window - (ranges - 1))) if total >= 24 * MiB else 1
            assert len(pieces) == want_pieces, (case, window, copies)
            assert len(copies) * window <= 16 or len(copies) == ranges, (case, window, copies)
            assert max(pieces) - min(pieces) <= 256 * len(pieces), (case, window, pieces)        # equal, but for the rounding
            assert all(off % 256 == 0 and n > 0 for off, n, _ in copies)
            merged = []
            for off, n, _ in copies:                         # in order, without gap or overlap inside a range
                if merged and merged[-1][0] + merged[-1][1] == off:
                    merged[-1][1] += n
                else:
                    merged.append([off, n])
            assert merged == want, (case, window, copies)
