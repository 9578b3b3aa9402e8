"""GPU parity at the sizes where a rule of the launch code changes: either side of each limit, against the oracle."""
import numpy as np
import pytest
import torch

from oracle import hxt_oracle as ho
from paper_2602_18007_amd import hxt
from tests.cases import ONE_LAUNCH_LIMITS, SMALL_CASES, Case, contig, make_storages
from tests.test_gpu_parity import NT, DEV, oracle_msg, round_trip_check, say, to_dev

pytestmark = pytest.mark.gpu
MiB = 1 << 20


@pytest.mark.parametrize("nbytes", [32 * MiB, 32 * MiB + 8, 64 * MiB, 64 * MiB + 24, 128 * MiB, 128 * MiB + 24])
def test_cache_hints_either_side_of_their_limits(nbytes):
    """Packed loads stop being cacheable above 128 MiB of packed bytes."""
    case = Case("contig_%d" % nbytes, (contig((nbytes // 8,), 8),), 3, MiB)
    say("case", case.name)
    round_trip_check(case, make_storages(case, 5), nthreads=NT)


@pytest.mark.parametrize("nbytes", [64 * MiB, 64 * MiB + 256])
@pytest.mark.parametrize("view", ["contig", "rows", "two_contig"])
def test_sends_from_bases_off_by_an_element(view, nbytes):
    """Loads from tensors that do not start on 16 bytes are cacheable up to 64 MiB, non-temporal above: plain sums and tags,
    one tensor, rows and a message of two tensors of which one is aligned."""
    n = nbytes // 2
    if view == "rows":
        tensors, off = [((n // 4096, 4096), (4104, 1), 2)] + ([((n % 4096,), (1,), 2)] if n % 4096 else []), [2, 0]
    elif view == "two_contig":
        tensors, off = [((n // 2,), (1,), 2), ((n - n // 2,), (1,), 2)], [0, 2]
    else:
        tensors, off = [((n,), (1,), 2)], [2]
    case = Case(view, tuple(tensors), 4, MiB)
    m, raws = oracle_msg(case), make_storages(case, 5)
    p = hxt.hxt_plan_multi(tensors, 4, MiB)
    C = p.num_chunks
    want = ho.pack(m, raws, MiB, 4, fill=0xA5, nthreads=NT)
    src = []
    for r, o in zip(raws, off):
        t = torch.empty(r.size + 64, dtype=torch.uint8, device=DEV)[o:]
        t[:r.size] = torch.from_numpy(r).to(DEV)
        src.append(t)
    say(view, nbytes)
    for tagged in (False, True):
        packed = torch.full((want.size,), 0xA5, dtype=torch.uint8, device=DEV)
        if tagged:
            tags = torch.zeros(64 * C, dtype=torch.uint8, device=DEV)
            hxt.hxt_pack_seal(p, src, packed, 7, 1, tags)
            assert np.array_equal(tags.cpu().numpy().reshape(C, 64), ho.seal(m, want, MiB, 4, 7, 1))
        else:
            sums = torch.zeros(C, dtype=torch.int64, device=DEV)
            hxt.hxt_pack(p, src, packed, sums)
            assert np.array_equal(sums.cpu().numpy().view(np.uint64), ho.checksum(m, want, MiB, 4))
        assert np.array_equal(packed.cpu().numpy(), want)


@pytest.mark.parametrize("nbytes", [12 * MiB, 12 * MiB + 4096, 64 * MiB, 64 * MiB + 4096])
@pytest.mark.parametrize("esize", [1, 2, 4, 8])
def test_elements_written_through_either_side_of_their_limits(esize, nbytes):
    """Every other element of rows: packed elements are written through above 12 MiB, single bytes up to 64 MiB."""
    cols = 4096 // esize
    case = Case("columns_%d_%d" % (esize, nbytes), (((nbytes // 4096, cols), (2 * cols, 2), esize),), 3, MiB)
    say("case", case.name)
    round_trip_check(case, make_storages(case, 5), nthreads=NT)


@pytest.mark.parametrize("hint", [0, 1])
@pytest.mark.parametrize("rows", [((300, 101, 107, 1),), ((300, 101, 107, 2), (70, 33, 40, 2)), ((300, 101, 107, 1), (70, 101, 107, 4)),
                                  ((300, 102, 106, 2), (41, 35, 36, 1)), ((300, 102, 106, 8),),
                                  ((300, 100, 104, 2), (41, 35, 36, 1)), ((300, 100, 104, 2), (70, 102, 106, 2))], ids=lambda r: "rows_of_" + "_".join(str(x[1] * x[3]) for x in r))
def test_rows_of_odd_lengths_by_the_pieces_they_go_in(rows, hint):
    """Runs go in pieces of 8 bytes (sending, of 4 too) or in vectors; messages whose runs all go in pieces have a kernel of
    their own, and with others among them they don't."""
    case = Case("odd_rows", tuple(((n, c), (p, 1), e) for n, c, p, e in rows), 3, 1 << 16)
    say("case", rows)
    round_trip_check(case, make_storages(case, 5), hint=hint)
    tagged_round_trip(case, hint)


@pytest.mark.parametrize("esize", [1, 2, 4, 8])
@pytest.mark.parametrize("nbytes", [8 * MiB, 25 * MiB])
def test_transposed_tensors_at_any_base(esize, nbytes):
    """Receiving transposes store rows that do not start on 16 bytes cacheable, by size of element and launch: bases one
    element off, pitches of whole vectors and not, against the oracle."""
    rows = 1021
    cols = nbytes // (rows * esize)
    for pitch in (rows + 3, rows + 6):                   # 1024 elements, and an odd number of elements to a vector
        base, ends = 1, (cols - 1) * pitch + rows
        m = ho.Message([ho.TensorSpec((rows, cols), (1, pitch), esize)])
        raw = np.random.default_rng(3).integers(0, 256, size=ends * esize, dtype=np.uint8)
        p = hxt.hxt_plan_multi([((rows, cols), (1, pitch), esize)], 4, MiB)
        assert p.tensor_kind(0).startswith("transpose")
        at = torch.empty(ends * esize + 64, dtype=torch.uint8, device=DEV)[base * esize:]
        at[:raw.size] = torch.from_numpy(raw).to(DEV)
        want = ho.pack(m, [raw], MiB, 4, fill=0xA5, nthreads=NT)
        packed = torch.full((want.size,), 0xA5, dtype=torch.uint8, device=DEV)
        say("pitch", pitch)
        hxt.hxt_pack(p, [at], packed)
        assert np.array_equal(packed.cpu().numpy(), want)
        dst_o = [np.full(raw.size, 0x3C, np.uint8)]
        ho.unpack(m, want, MiB, 4, dst_o, nthreads=NT)
        at.fill_(0x3C)
        hxt.hxt_unpack(p, packed, [at])
        assert np.array_equal(at.cpu().numpy()[:raw.size], dst_o[0])


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


def tagged_round_trip(case, hint):
    """pack + seal, then unpack + verify of the intact bytes and of a damaged last chunk, against the oracle."""
    m = oracle_msg(case)
    p = hxt.hxt_plan_multi([(s, st, e) for s, st, e in case.tensors], case.k, case.B)
    hxt.hxt_plan_set_option(p, hxt.HXT_OPT_PACKED_HINT, hint)
    raws, C = make_storages(case, 23), p.num_chunks
    want = ho.pack(m, raws, case.B, case.k, fill=0xA5, nthreads=NT)
    want_tags = ho.seal(m, want, case.B, case.k, 77, 5)
    packed = torch.full((max(want.size, 16),), 0xA5, dtype=torch.uint8, device=DEV)
    tags = torch.full((max(C, 1) * 64,), 0xEE, dtype=torch.uint8, device=DEV)
    hxt.hxt_pack_seal(p, [to_dev(r) for r in raws], packed, 77, 5, tags)
    assert np.array_equal(packed.cpu().numpy()[:want.size], want)
    assert np.array_equal(tags.cpu().numpy()[:C * 64].reshape(C, 64), want_tags)
    if not C or not all(p.tensor_unpack_safe(t) for t in range(len(case.tensors))):
        return
    damaged = want.copy()
    damaged[p.chunk_info(C - 1)["packed_off"] + 5] ^= 0x40
    for pk in (want, damaged):
        dst_o = [np.full(r.size, 0x3C, np.uint8) for r in raws]
        ho.unpack(m, pk, case.B, case.k, dst_o, nthreads=NT)
        dst = [to_dev(np.full(r.size, 0x3C, np.uint8)) for r in raws]
        status = torch.full((C + 1,), 0x7FFFFFFF, dtype=torch.int32, device=DEV)
        hxt.hxt_unpack_verify(p, to_dev(pk), to_dev(want_tags.reshape(-1)), 77, 5, dst, status)
        assert np.array_equal(status.cpu().numpy().view(np.uint32), ho.verify(m, pk, want_tags, case.B, case.k, 77, 5))
        for a, b in zip(dst_o, dst):
            assert np.array_equal(b.cpu().numpy()[:a.size], a)


# The packed hint "non-temporal" keeps a message out of the one launch for several kinds, so both routes are compared.
@pytest.mark.parametrize("hint", [0, 1], ids=["one_launch", "a_launch_per_kind"])
@pytest.mark.parametrize("case", SMALL_CASES, ids=lambda c: c.name)
def test_both_routes_of_small_messages(case, hint):
    say("case", case.name)
    round_trip_check(case, make_storages(case, 5), hint=hint)
    tagged_round_trip(case, hint)


@pytest.mark.parametrize("hint", [0, 1], ids=["one_launch", "a_launch_per_kind"])
@pytest.mark.parametrize("chunk", [1024, 1 << 16], ids=lambda b: "chunks_of_%d" % b)
@pytest.mark.parametrize("esize", [1, 2, 4, 8])
def test_tags_of_transposes_at_their_edges(esize, chunk, hint):
    """Weights of vectors that start inside a word or meet a chunk border; 36 matrices, the pads between them and a run
    of rows whose length is no multiple of 16 bytes."""
    T, V = (128 if esize <= 2 else 64), 16 // esize
    sizes = [V + 1, T - 1, T, T + 1, T + V + 1, 2 * T + 3]
    tensors = tuple(((r, c), (1, r + (r + c) % 3), esize) for r in sizes for c in sizes) + (((37, 2 * V + 1), (2 * V + 4, 1), esize),)
    case = Case("tagged_edges_%d_%d" % (esize, chunk), tensors, 3, chunk)
    say("case", case.name)
    tagged_round_trip(case, hint)


@pytest.mark.parametrize("rows", [2054, 2055, 2056, 16430, 16440])
def test_one_launch_either_side_of_its_limits(rows):
    """Padded rows of 4082 bytes with pads, which ride in the launch of the rows at any size, and the same with a mask and a
    transposed matrix (three launches: one up to 64 MiB, 16432 rows)."""
    padded = ((rows, 2041), (2048, 1), 2)
    for tensors in ((padded,), (padded, contig((rows,), 1), ((64, 40), (1, 64), 4))):
        case = Case("limit_%d_%d" % (rows, len(tensors)), tensors, 4, MiB)
        say("case", case.name)
        round_trip_check(case, make_storages(case, 5), nthreads=NT)
        tagged_round_trip(case, -1)


@pytest.mark.parametrize("over", [0, 256])
@pytest.mark.parametrize("make", list(ONE_LAUNCH_LIMITS), ids=["two_launches", "three_launches"])
def test_messages_of_several_kinds_either_side_of_their_limit(make, over):
    """The planner's tests check that these take one launch up to the limit and one per kind beyond it."""
    case = make(ONE_LAUNCH_LIMITS[make] + over)
    say("case", case.name)
    round_trip_check(case, make_storages(case, 5), nthreads=NT)
    tagged_round_trip(case, -1)
