"""GPU parity of the strided copy kernels at the shapes where their work is split: edges of vectors, runs and tiles, plain
sums and tags, against the oracle."""
import numpy as np
import pytest
import torch

from oracle import hxt_oracle as ho
from paper_2602_18007_amd import hxt
from tests.cases import CLIPPED_TRANSPOSES as CLIPPED, Case, make_storages
from tests.test_gpu_parity import DEV, oracle_msg, plan_of, round_trip_check, say, to_dev

pytestmark = pytest.mark.gpu
KiB = 1 << 10


def check(shape, strides, esize, lanes, chunk, base_offset=0):
    """Plain sums (round_trip_check) and tags, both directions."""
    case = Case("view", ((shape, strides, esize),), lanes, chunk)
    raws = make_storages(case, 11)
    say(shape, strides, esize, lanes, chunk, base_offset)
    round_trip_check(case, raws, base_offset=base_offset)
    m, p = oracle_msg(case), plan_of(case)
    C = p.num_chunks
    want = ho.pack(m, raws, chunk, lanes, fill=0xA5)
    src = [to_dev(r, base_offset) for r in raws]
    packed = torch.full((want.size,), 0xA5, dtype=torch.uint8, device=DEV)
    tags = torch.zeros(64 * C, dtype=torch.uint8, device=DEV)
    hxt.hxt_pack_seal(p, src, packed, 5, 2, tags)
    assert np.array_equal(packed.cpu().numpy(), want)
    assert np.array_equal(tags.cpu().numpy().reshape(C, 64), ho.seal(m, want, chunk, lanes, 5, 2))
    if not p.tensor_unpack_safe(0):
        return
    dst_o = [np.full(r.size, 0x3C, np.uint8) for r in raws]
    ho.unpack(m, want, chunk, lanes, dst_o)
    dst = [to_dev(d * 0 + 0x3C, base_offset) for d in dst_o]
    status = torch.full((C + 1,), 7, dtype=torch.int32, device=DEV)
    hxt.hxt_unpack_verify(p, packed, tags, 5, 2, dst, status)
    assert np.array_equal(dst[0].cpu().numpy(), dst_o[0])
    assert not status.any()


# (run length in elements, gap behind it, element size, base off by): one vector and its neighbours, runs that end anywhere
# in a vector, pieces of 8 and 4 bytes and vectors, each side of the rule between them.
RUNS = [(16, 1, 1, 0), (17, 0, 1, 1), (31, 9, 1, 0), (8, 1, 2, 0), (9, 4, 2, 2), (100, 28, 2, 0), (100, 28, 2, 2), (101, 3, 2, 0),
        (102, 2, 2, 0), (1003, 1, 2, 0), (5, 1, 4, 0), (6, 2, 4, 4), (101, 19, 4, 0), (3, 1, 8, 0), (4099, 5, 1, 3)]


@pytest.mark.parametrize("run,gap,esize,off", RUNS)
def test_rows_that_are_no_multiple_of_a_vector(run, gap, esize, off):
    pitch = run + gap
    rows = 70 * KiB // (run * esize) + 3
    check((rows, run), (pitch, 1), esize, 3, 8 * KiB + 256, off)
    check((rows // 4, 4, run), (pitch, (rows // 4) * pitch + 1, 1), esize, 2, 64 * KiB, off)       # neighbours far apart in storage
    check((4, rows // 4, run), ((rows // 4) * pitch + 3, pitch, 1), esize, 2, 64 * KiB, off)
    check((rows, run), (max(run - 3, 0), 1), esize, 2, 16 * KiB, off)                              # runs that overlap: a source only
    check((7, run), (0, 1), esize, 1, 512, off)                                                    # the same run over and over


# Runs longer than a tile of 16 KiB (bytes, gap): tiles inside one run, over the end of one with less and more than a vector
# on either side.
@pytest.mark.parametrize("run,gap,off", [(16385, 1, 0), (16399, 4, 1), (16401, 2, 0), (40001, 10, 3), (300007, 57, 0)])
def test_rows_longer_than_a_tile(run, gap, off):
    pitch = run + gap
    for chunk in (256 * KiB, 40 * KiB + 256):
        check((4, run), (pitch, 1), 1, 3, chunk, off)
        check((2, 2, run), (pitch, 2 * pitch + 1, 1), 1, 2, chunk, off)       # the next run below this one in storage
    check((3, run // 2), (pitch, 1), 2, 2, 64 * KiB, 2 * off)


# (elements of a run, distance between them, element size, base off by): runs either side of 32 elements, the shortest and
# the long ones, whole numbers of groups and not, distances with a path of their own (2 and 4, of 1 and 2 bytes) and without.
APART = [(31, 2, 2, 0), (32, 2, 2, 0), (33, 2, 2, 2), (101, 2, 2, 0), (67, 4, 2, 6), (128, 4, 2, 0), (100, 3, 2, 0), (45, 2, 1, 1),
         (77, 4, 1, 3), (64, 5, 1, 0), (50, 2, 4, 4), (40, 4, 4, 0), (37, 2, 8, 8),
         (16, 2, 1, 1), (24, 2, 1, 0), (12, 4, 1, 3), (12, 2, 2, 2), (4097, 2, 2, 2), (4099, 2, 1, 1), (4098, 4, 1, 0)]


@pytest.mark.parametrize("run,step,esize,off", APART)
def test_elements_a_few_apart(run, step, esize, off):
    n = 70 * KiB // (run * esize) + 3
    check((n * run + 5,), (step,), esize, 3, 8 * KiB + 256, off)
    check((n, run), (run * step + 1, step), esize, 2, 64 * KiB, off)
    check((n // 3, 3, run), (run * step, (n // 3) * run * step + 3, step), esize, 2, 64 * KiB, off)
    check((n, run), (step, step), esize, 2, 16 * KiB, off)             # runs over each other: a source only


# Either side of 10 MiB, chunks that hold whole numbers of tile rows and not: tiles inside chunks or across them.
@pytest.mark.parametrize("shape,strides,esize,chunk", CLIPPED)
def test_transposes_that_chunks_would_clip(shape, strides, esize, chunk):
    check(shape, strides, esize, 3, chunk)
