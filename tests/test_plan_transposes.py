"""The work tables of large transposes, executed on the CPU: tiles inside chunks where these hold whole numbers of tile rows,
across chunks where they would be clipped."""
import numpy as np
import pytest

from oracle import hxt_oracle as ho
from tests.cases import CLIPPED_TRANSPOSES, Case, make_storages
from tests.test_plan_host import interp, oracle_msg, run_interp  # noqa: F401

INSIDE, ACROSS = 3, 7


@pytest.mark.parametrize("view,kind", list(zip(CLIPPED_TRANSPOSES, [ACROSS, INSIDE, ACROSS, INSIDE, ACROSS, ACROSS, INSIDE, ACROSS, INSIDE, ACROSS])))
def test_large_transposes(interp, view, kind):  # noqa: F811
    shape, strides, esize, chunk = view
    case = Case("transpose", ((shape, strides, esize),), 3, chunk)
    m, raws = oracle_msg(case), make_storages(case, 5)
    want = ho.pack(m, raws, chunk, 3, fill=0x99, nthreads=4)
    got = np.full(want.size, 0x99, np.uint8)
    rc, _, kinds = run_interp(interp, case, raws, got, 0, 16384)
    assert rc == 0 and np.array_equal(got, want)
    assert kinds[0] == kind
    dst_o = [np.full(r.size, 0x42, np.uint8) for r in raws]
    dst = [np.full(r.size, 0x42, np.uint8) for r in raws]
    ho.unpack(m, want, chunk, 3, dst_o, nthreads=4)
    assert run_interp(interp, case, dst, want.copy(), 1, 16384)[0] == 0
    assert np.array_equal(dst[0], dst_o[0])
