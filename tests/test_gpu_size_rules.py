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
