"""Performance cases of the boundary transfer: the messages a pipeline stage sends and receives, through the
library's Python entry points.

A pass is one whole transfer on one GPU: every message is packed into its chunk buffer and unpacked again (or added
to what the receiver holds), with the integrity check that the case names.  Sizes come from the benchmark messages in
paper_2602_18007_amd/workloads.py and from bench.py; draw() spreads them over the ranges these stand for.

Everything the library moves is compared bit for bit: packed bytes, destinations (with the bytes between the elements
of strided views), checksums, tags and verification results.
"""
from __future__ import annotations

import math

import torch

from paper_2602_18007_amd import hxt

DEV = "cuda:0"
KiB, MiB = 1 << 10, 1 << 20
DTYPES = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32, "u8": torch.uint8}
ESIZE = {"bf16": 2, "f16": 2, "f32": 4, "u8": 1}
CAP_BYTES = 512 * MiB          # most tensor bytes of a drawn case


# ---- the cases ----------------------------------------------------------------------

def listed():
    return [
        # One small activation (a short decode step, or a toy model): launches and host time count, not bytes.
        dict(name="tiny_message", path="message", view="contig", dtype="bf16", seq=128, mb=1, hidden=512, offset=0,
             messages=1, checks="sums", lanes=2, chunk_kib=16),
        # The benchmark's headline step: forward activation and backward gradient of an 8B model's boundary at once.
        dict(name="boundary_pair", path="message", view="contig", dtype="bf16", seq=4096, mb=1, hidden=4096, offset=0,
             messages=2, checks="sums", lanes=4, chunk_kib=1024),
        # One 56 MiB activation of a 7B model, with chunk tags sealed and verified inside the copies.
        dict(name="tagged_activation", path="message", view="contig", dtype="bf16", seq=4096, mb=2, hidden=3584, offset=0,
             messages=1, checks="tags", lanes=8, chunk_kib=4096),
        # The same activation as training frameworks hold it: a [seq, mb, hidden] view of [mb, seq, hidden] storage.
        dict(name="sequence_first_view", path="message", view="rows", dtype="bf16", seq=4096, mb=2, hidden=3584, offset=0,
             messages=1, checks="sums", lanes=8, chunk_kib=4096),
        # A padded matrix: runs that are not multiples of 16 bytes.
        dict(name="padded_rows", path="message", view="padded", dtype="bf16", rows=327680, cols=100, pitch=128,
             messages=1, checks="sums", lanes=4, chunk_kib=1024),
        # A transposed weight gradient or activation.
        dict(name="transposed", path="message", view="transposed", dtype="bf16", batch=1, rows=4096, cols=4096, pad=0,
             messages=1, checks="sums", lanes=4, chunk_kib=1024),
        # The same with packed rows that are long against the chunk.
        dict(name="transposed_wide", path="message", view="transposed", dtype="bf16", batch=1, rows=256, cols=65536, pad=0,
             messages=1, checks="sums", lanes=4, chunk_kib=1024),
        # Every other column of a matrix (interleaved pairs): no unit stride anywhere.
        dict(name="every_other_column", path="message", view="columns", dtype="bf16", rows=4096, cols=4096, step=2,
             messages=1, checks="sums", lanes=4, chunk_kib=1024),
        # What a boundary carries beside the activation: a byte mask, f32 side values taken out of a larger buffer, a
        # transposed projection and rows with padding, all in one tagged message of odd sizes.
        dict(name="mixed_bundle", path="message", view="mixed", dtype="bf16", seq=1021, mb=2, hidden=1024,
             messages=1, checks="tags", lanes=4, chunk_kib=256),
        # Gradients of four layers of an 8B model crossing in 25 MiB buckets and added to the receiver's own.
        dict(name="gradient_buckets", path="grads", dtype="bf16", layers=4, hidden=4096, kv=1024, ffn=14336, odd=0,
             checks="sums", lanes=8, chunk_kib=25600),
        # 1F1B: a stream of micro-batches through two buffer sets, device to device.
        dict(name="microbatch_stream", path="stream", dtype="bf16", seq=4096, mb=1, hidden=4096, messages=32, buffers=2,
             checks="sums", lanes=4, chunk_kib=2048),
        # The compatibility path: the same stream through pinned host memory (bound by the host link).
        dict(name="host_forwarded_stream", path="forward", dtype="bf16", seq=4096, mb=2, hidden=3584, messages=8, buffers=2,
             checks="sums", lanes=8, chunk_kib=4096),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    lanes = rng.choice([1, 2, 4, 4, 8, 8])
    checks = rng.choice(["sums", "sums", "tags"])
    chunk_kib = rng.choice([256, 512, 1024, 1024, 2048, 4096, 8192])
    path = rng.choice(["contig", "contig", "contig", "rows", "padded", "transposed", "transposed", "columns", "mixed",
                       "grads", "stream", "forward"])
    dtype = rng.choice(["bf16", "bf16", "bf16", "f16", "f32"])
    es = ESIZE[dtype]
    if path == "contig":
        messages = rng.choice([1, 1, 2, 3, 4])
        hidden = rng.choice([_log(rng, 64, 8192), 64 * rng.randint(1, 128)])
        size = _log(rng, 16 * KiB, CAP_BYTES // messages)
        seq, mb = max(1, size // (hidden * es)), rng.choice([1, 1, 2, 4])
        return dict(path="message", view="contig", dtype=dtype, seq=max(1, seq // mb), mb=mb, hidden=hidden,
                    offset=rng.choice([0, 0, 0, rng.randint(1, 63)]), messages=messages, checks=checks, lanes=lanes,
                    chunk_kib=chunk_kib if size > MiB else rng.choice([16, 64]))
    if path == "rows":
        mb, hidden = rng.randint(2, 8), 8 * rng.randint(8, 1024)
        seq = max(2, _log(rng, MiB, 256 * MiB) // (mb * hidden * es))
        return dict(path="message", view="rows", dtype=dtype, seq=seq, mb=mb, hidden=hidden, offset=0, messages=1,
                    checks=checks, lanes=lanes, chunk_kib=chunk_kib)
    if path == "padded":
        cols = _log(rng, 16, 4000)
        rows = max(2, _log(rng, MiB, 128 * MiB) // (cols * es))
        return dict(path="message", view="padded", dtype=dtype, rows=rows, cols=cols, pitch=cols + rng.randint(1, 64),
                    messages=1, checks=checks, lanes=lanes, chunk_kib=chunk_kib)
    if path == "transposed":
        batch, size, rows = rng.choice([1, 1, 4]), _log(rng, MiB, 256 * MiB), _log(rng, 64, 16384)
        cols = max(16, size // (batch * rows * es))
        if rng.random() < 0.6:                          # most real extents are multiples of 64
            rows, cols = max(64, rows // 64 * 64), max(64, cols // 64 * 64)
        return dict(path="message", view="transposed", dtype=dtype, batch=batch, rows=rows, cols=cols,
                    pad=rng.choice([0, 0, 8, 5]), messages=1, checks=checks, lanes=lanes, chunk_kib=chunk_kib)
    if path == "columns":
        rows = _log(rng, 64, 8192)
        cols = max(32, _log(rng, MiB, 64 * MiB) // (rows * es))
        return dict(path="message", view="columns", dtype=dtype, rows=rows, cols=cols, step=rng.choice([2, 2, 3, 4]),
                    messages=1, checks=checks, lanes=lanes, chunk_kib=chunk_kib)
    if path == "mixed":
        return dict(path="message", view="mixed", dtype="bf16", seq=_log(rng, 32, 8192), mb=rng.choice([1, 2, 4]),
                    hidden=64 * rng.randint(4, 64), messages=1, checks=checks, lanes=lanes,
                    chunk_kib=rng.choice([64, 256, 1024]))
    if path == "grads":
        hidden = 128 * rng.randint(4, 24)
        return dict(path="grads", dtype=rng.choice(["bf16", "f32"]), layers=rng.randint(1, 3), hidden=hidden,
                    kv=max(64, hidden // 4), ffn=hidden * 7 // 2, odd=rng.choice([0, 0, 1, 3]), checks="sums", lanes=lanes,
                    chunk_kib=rng.choice([1024, 4096, 25600]))
    hidden = 128 * rng.randint(4, 40)
    size = _log(rng, 512 * KiB, 48 * MiB)
    if path == "stream":
        messages = max(2, min(_log(rng, 4, 32), 1024 * MiB // size))
        return dict(path="stream", dtype="bf16", seq=max(8, size // (hidden * 2)), mb=1, hidden=hidden, messages=messages,
                    buffers=rng.choice([2, 2, 3, 4]), checks=checks, lanes=lanes, chunk_kib=chunk_kib)
    return dict(path="forward", dtype="bf16", seq=max(8, size // (hidden * 4)), mb=2, hidden=hidden,
                messages=rng.randint(2, 8), buffers=2, checks=checks, lanes=lanes, chunk_kib=chunk_kib)


# ---- message geometry -----------------------------------------------------------------

def _tensors(case):
    """The tensors of one message: (shape, strides or None, dtype name, elements of storage, first element)."""
    dt = case["dtype"]

    def contig(shape, d=dt, offset=0):
        n = math.prod(shape)
        return (tuple(shape), None, d, n + offset, offset)

    def strided(shape, strides, d=dt):
        return (tuple(shape), tuple(strides), d, sum((s - 1) * t for s, t in zip(shape, strides)) + 1, 0)

    if case["path"] == "grads":
        h, kv, f, odd = case["hidden"], case["kv"], case["ffn"] + case["odd"], case["odd"]
        layer = [(h,), (h, h), (kv, h), (kv, h), (h, h), (h,), (f, h), (f, h), (h + odd, f)]
        return [contig(s) for _ in range(case["layers"]) for s in layer]
    if case["path"] in ("stream", "forward"):           # [seq, mb, hidden]; for mb = 1 a view of [mb, seq, hidden]
        s, m, h = case["seq"], case["mb"], case["hidden"]
        return [strided((s, m, h), (h, s * h, 1)) if m == 1 else contig((s, m, h))]
    view = case["view"]
    if view == "contig":
        return [contig((case["seq"], case["mb"], case["hidden"]), offset=case["offset"])]
    if view == "rows":
        s, m, h = case["seq"], case["mb"], case["hidden"]
        return [strided((s, m, h), (h, s * h, 1))]
    if view == "padded":
        return [strided((case["rows"], case["cols"]), (case["pitch"], 1))]
    if view == "transposed":
        b, r, c = case["batch"], case["rows"], case["cols"]
        pitch = r + case["pad"]
        return [strided((b, r, c), (c * pitch, 1, pitch))]
    if view == "columns":
        r, c, k = case["rows"], case["cols"], case["step"]
        return [strided((r, c), (c * k, k))]
    s, m, h = case["seq"], case["mb"], case["hidden"]
    return [
        strided((s, m, h), (h, s * h, 1)),              # activation, sequence first
        contig((m, s), "u8"),                           # attention mask
        contig((s, m, 3), "f32", offset=1),             # side values, a slice of a larger buffer
        strided((h, s), (1, h)),                        # a projection, transposed
        strided((s, 100), (128, 1)),                    # logits of a small head, padded pitch
        contig((h,), "f32"),
    ]


def _bytes(case):
    return sum(math.prod(s) * ESIZE[d] for s, _, d, _, _ in _tensors(case))


def _storages(case, gen, fill):
    """One storage tensor per tensor of a message: values as they are met in training, or zeros for a receiver."""
    out = []
    for _, _, d, n, _ in _tensors(case):
        if not fill:
            out.append(torch.zeros(n, dtype=DTYPES[d], device=DEV))
        elif d == "u8":
            out.append(torch.randint(0, 2, (n,), generator=gen, device=DEV, dtype=torch.uint8))
        else:
            std = 0.02 if case["path"] == "grads" else 1.0
            out.append(torch.randn(n, generator=gen, device=DEV, dtype=torch.float32).mul_(std).to(DTYPES[d]))
    return out


def _first(case, storages):
    """The tensors a call is given: each storage from its first element on."""
    return [x[o:] for x, (_, _, _, _, o) in zip(storages, _tensors(case))]


def _plan(case):
    descr = [(s, st, DTYPES[d]) for s, st, d, _, _ in _tensors(case)]
    return hxt.hxt_plan_multi(descr, case["lanes"], case["chunk_kib"] * KiB)


def _packed(plan):
    return torch.zeros(max(plan.packed_bytes, 256), dtype=torch.uint8, device=DEV)


_streams = []


def _three_streams():
    """The streams a program keeps for its micro-batch pipeline (pack, staging, unpack)."""
    if not _streams:
        _streams.extend(torch.cuda.Stream() for _ in range(3))
    return _streams


# ---- one case -----------------------------------------------------------------------------

def prepare(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    n = case["messages"] if case["path"] != "grads" else 1
    st = {"case": case, "n": n, "tags": case["checks"] == "tags"}
    st["src"] = [_storages(case, gen, True) for _ in range(n)]
    st["dst"] = [_storages(case, gen, case["path"] == "grads") for _ in range(n)]
    src, dst = [_first(case, x) for x in st["src"]], [_first(case, x) for x in st["dst"]]
    if case["path"] in ("stream", "forward"):
        return _prepare_stream(case, st, src, dst)
    plans = [_plan(case) for _ in range(n)]
    C = plans[0].num_chunks
    st["plan"], st["from"], st["to"] = plans[0], src[0], dst[0]
    st["packed"] = [_packed(p) for p in plans]
    if st["tags"]:
        st["sent"] = [torch.zeros(64 * C, dtype=torch.uint8, device=DEV) for _ in range(n)]
        st["got"] = [torch.zeros(C + 1, dtype=torch.int32, device=DEV) for _ in range(n)]
        st["seq"], st["micro_batch"] = [seed % 1000003 + i for i in range(n)], list(range(n))
        if n > 1:
            st["pack"] = hxt.TagBatch(plans, src, st["packed"], st["sent"])
            st["unpack"] = hxt.TagBatch(plans, dst, st["packed"], st["sent"], st["got"])
    else:
        st["sent"] = [torch.zeros(C, dtype=torch.int64, device=DEV) for _ in range(n)]
        st["got"] = [torch.zeros(C, dtype=torch.int64, device=DEV) for _ in range(n)]
        if n > 1:
            st["pack"] = hxt.Batch(plans, src, st["packed"], st["sent"])
            st["unpack"] = hxt.Batch(plans, dst, st["packed"], st["got"])
    return st


def _prepare_stream(case, st, src, dst):
    n, nb, forward = st["n"], case["buffers"], case["path"] == "forward"
    plan = _plan(case)
    C = plan.num_chunks
    pinned = lambda size: torch.zeros(size, dtype=torch.uint8, pin_memory=True)
    st["plan"] = plan
    st["packed"] = [_packed(plan) for _ in range(nb)]
    st["landed"] = [_packed(plan) for _ in range(nb)] if forward else []
    kw = {}
    if forward:
        # drained every few messages inside the call, as the library advises for this path
        kw.update(path=hxt.HXT_CPU_FORWARD, packed_recv=st["landed"], drain_every=4,
                  host_pinned=[pinned(max(plan.packed_bytes, 256)) for _ in range(nb)])
    if st["tags"]:
        st["sent"] = [torch.zeros(64 * C, dtype=torch.uint8, device=DEV) for _ in range(nb)]
        st["got"] = torch.zeros(n * (C + 1), dtype=torch.int32, device=DEV)
        kw.update(tags_send=st["sent"], status=st["got"], seq_base=7)
        if forward:
            kw.update(tags_recv=[torch.zeros(64 * C, dtype=torch.uint8, device=DEV) for _ in range(nb)],
                      tags_pinned=[pinned(64 * C) for _ in range(nb)])
    else:
        st["sent"] = torch.zeros(n * C, dtype=torch.int64, device=DEV)
        st["got"] = torch.zeros(n * C, dtype=torch.int64, device=DEV)
        kw.update(send_sums=st["sent"], recv_sums=st["got"])
    a, b, c = _three_streams()
    st["exchange"] = hxt.Exchange(src, dst, st["packed"], stream_pack=a, stream_stage=b, stream_unpack=c, **kw)
    return st


def run(st):
    path, plan = st["case"]["path"], st["plan"]
    if path in ("stream", "forward"):
        hxt.hxt_exchange_stream(plan, st["exchange"])
        return [_joined(st["dst"]), st["packed"], st["landed"], st["sent"], st["got"]]
    if path == "grads":
        hxt.hxt_pack(plan, st["from"], st["packed"][0], st["sent"][0])
        hxt.hxt_unpack_accumulate(plan, st["packed"][0], st["to"], st["got"][0])
    elif st["tags"] and st["n"] > 1:
        hxt.hxt_pack_seal_batch(st["pack"], st["seq"], st["micro_batch"])
        hxt.hxt_unpack_verify_batch(st["unpack"], st["seq"], st["micro_batch"])
    elif st["tags"]:
        seq, mb = st["seq"][0], st["micro_batch"][0]
        hxt.hxt_pack_seal(plan, st["from"], st["packed"][0], seq, mb, st["sent"][0])
        hxt.hxt_unpack_verify(plan, st["packed"][0], st["sent"][0], seq, mb, st["to"], st["got"][0])
    elif st["n"] > 1:
        hxt.hxt_pack_batch(st["pack"])
        hxt.hxt_unpack_batch(st["unpack"])
    else:
        hxt.hxt_pack(plan, st["from"], st["packed"][0], st["sent"][0])
        hxt.hxt_unpack(plan, st["packed"][0], st["to"], st["got"][0])
    return [_joined(st["dst"]), st["packed"], st["sent"], st["got"]]


def _joined(messages):
    return [x for tensors in messages for x in tensors]


def work(case):
    """Bytes that have to move.  Pack reads the tensors and writes the packed bytes, unpack reads these and writes the
    tensors; adding on arrival reads the old values too, forwarding through the host reads and writes the packed bytes
    once more on the device.  Additions are the only arithmetic on values."""
    n = case.get("messages", 1) if case["path"] != "grads" else 1
    b = n * _bytes(case)
    if case["path"] == "grads":
        return {"bytes": 5 * b, "flops": b // ESIZE[case["dtype"]]}
    return {"bytes": (6 if case["path"] == "forward" else 4) * b, "flops": 0}


def tolerance(case):
    return "exact"
