"""GPU parity at the sizes where a rule of the launch code changes: either side of each limit, against the oracle."""
import pytest

from tests.cases import Case, contig, make_storages
from tests.test_gpu_parity import NT, round_trip_check, say

pytestmark = pytest.mark.gpu
MiB = 1 << 20


@pytest.mark.parametrize("nbytes", [32 * MiB, 32 * MiB + 8, 64 * MiB, 64 * MiB + 24])
def test_cache_hints_either_side_of_their_limits(nbytes):
    """Tensor loads stop being cacheable above 32 MiB, packed loads above 64 MiB of packed bytes."""
    case = Case("contig_%d" % nbytes, (contig((nbytes // 8,), 8),), 3, MiB)
    say("case", case.name)
    round_trip_check(case, make_storages(case, 5), nthreads=NT)


@pytest.mark.parametrize("chunk", [1024, 1 << 16, 1 << 20], ids=lambda b: "chunks_of_%d" % b)
@pytest.mark.parametrize("esize", [1, 2, 4, 8])
def test_transpose_tiles_at_their_edges(esize, chunk):
    """Tiles that are full, one element short or long, narrower than a vector, and rows that meet chunk borders inside a
    vector (odd lengths and pitches), in one message of many small matrices."""
    T, V = (128 if esize <= 2 else 64), 16 // esize
    sizes = sorted({2, V - 1, V, V + 1, T - 1, T, T + 1, T + V + 1} - {0, 1})
    tensors = tuple(((r, c), (1, r + (r + c) % 3), esize) for r in sizes for c in sizes)
    case = Case("edges_%d_%d" % (esize, chunk), tensors, 3, chunk)
    say("case", case.name, len(tensors), "tensors")
    round_trip_check(case, make_storages(case, 17), nthreads=NT)
