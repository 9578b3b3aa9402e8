// Internal structures shared by the host planner and the HIP kernels of libhxt.
// Not part of the ABI.
#ifndef HXT_INTERNAL_H
#define HXT_INTERNAL_H

#include <cstdint>
#include <vector>

#include "hxt.h"

#if defined(__HIPCC__)
#define HXT_HD __host__ __device__ inline
#else
#define HXT_HD inline
#endif

namespace hxt {

// Which kernel family moves a piece of the stream.
enum Kind : uint16_t {
    K_NONE = 0,
    K_CONTIG = 1,     // tensor bytes are contiguous in memory: straight 128-bit copy
    K_ROWS = 2,       // innermost dimension contiguous, 16-byte friendly rows: gather of runs
    K_TRANSPOSE = 3,  // innermost logical dim strided, second innermost contiguous: LDS tile transpose
    K_GENERIC = 4,    // anything else: one element at a time
    K_ZERO = 5,       // pad bytes between tensors / after the last one (byte granular, < 256 bytes)
    K_ROWS_SPLIT = 6, // innermost dimension contiguous, runs of 16 bytes or more whose length or pitch is not a
                      // multiple of 16: a 16-byte packed vector may end one run and begin the next
    K_TRANSPOSE_SPAN = 7  // the transpose when a chunk holds fewer rows of the packed side than a tile is high: a tile
                          // is a full block of the logical matrix and its rows may lie in different chunks
};

// One unit of work for one workgroup.  64 bytes of 32/64-bit fields, read with scalar loads.
//   linear kinds (CONTIG, ROWS, GENERIC, ZERO):
//     packed_off : first packed byte of the piece (CONTIG/ROWS/GENERIC: multiple of 256)
//     src_off    : logical byte offset inside the tensor (equals the storage offset for CONTIG)
//     n0         : bytes of the piece
//     a          : byte offset of the piece inside its chunk
//   TRANSPOSE (a 2-D block of ni logical rows x nj logical columns inside one chunk):
//     packed_off : packed byte of element (i0, j0);  b = packed row pitch in bytes
//     src_off    : storage byte of element (i0, j0); a = storage pitch between columns in bytes
//     n0 = ni (rows, contiguous in storage), n1 = nj (columns, contiguous in the packed stream)
//   TRANSPOSE_SPAN (the same block, not confined to one chunk): as TRANSPOSE, except
//     packed_off : byte of element (i0, j0) in the logical stream (the kernel finds every row's chunk from it)
//     chunk      : index of the tile's first entry in Plan::inc;  ordinal = number of entries (chunks it touches)
struct Tile {
    uint64_t packed_off;
    uint64_t src_off;
    uint64_t a;
    uint64_t b;
    uint32_t chunk;
    uint32_t tensor;   // index relative to the launch group's first tensor
    uint32_t kind;
    uint32_t n0;
    uint32_t n1;
    uint32_t ordinal;  // position of this tile among the tiles of its chunk (0 .. chunk_tiles[chunk] - 1)
    uint32_t estep;    // TRANSPOSE: bytes between neighbouring elements along the tensor side's fast direction
    uint32_t reserved;
};
static_assert(sizeof(Tile) == 64, "Tile must stay 64 bytes");

// Exact unsigned division of n < 2^31 by a fixed d < 2^31: q = (n * mul) >> (31 + shift).
struct FastDiv {
    uint32_t mul;
    uint32_t shift;
};
FastDiv make_fastdiv(uint32_t d);
HXT_HD uint32_t fast_div(uint32_t n, FastDiv d) { return uint32_t((uint64_t(n) * d.mul) >> (31 + d.shift)); }

// Chunk/lane geometry in closed form, for work that is uniform over the packed stream (a
// message made of one contiguous tensor; the stand-alone checksum of any message).  The
// stream is cut into chunks of B bytes and every chunk into tpc = ceil(B / tile) tiles;
// tile number t belongs to chunk t / tpc.  Lane l holds q + (l < r) chunks, so its region
// starts at (l*q + min(l, r)) * B.
struct ChunkGeom {
    uint64_t N;          // tensor bytes (uniform-copy path only)
    uint64_t L;          // stream bytes (multiple of 256)
    uint64_t B;          // chunk bytes
    uint32_t k, C;       // lanes, chunks
    uint32_t tile;       // bytes per tile (multiple of 256)
    uint32_t tpc;        // tiles per full chunk
    uint32_t q, r;       // C / k, C % k
    uint32_t ntiles;     // (C - 1) * tpc + tiles of the last chunk
    uint32_t last_tiles; // tiles of the last chunk
    FastDiv div_tpc, div_k;
    FastDiv div_b256;    // division by B / 256, for chunk_at
};

struct TileSpan {
    uint32_t chunk;
    uint32_t ordinal;    // position of the tile inside its chunk
    uint32_t expected;   // tiles that make up this chunk
    uint64_t stream_off; // first stream byte of the tile
    uint64_t packed_off; // where it lives in the packed buffer
    uint32_t len;        // stream bytes in the tile (multiple of 256)
};

HXT_HD TileSpan locate_tile(const ChunkGeom &g, uint32_t t)
{
    TileSpan s;
    const uint32_t c = fast_div(t, g.div_tpc), j = t - c * g.tpc;
    const uint32_t slot = fast_div(c, g.div_k), lane = c - slot * g.k;
    const uint64_t in_chunk = uint64_t(j) * g.tile;
    const uint64_t chunk_len = (c + 1 == g.C) ? g.L - uint64_t(c) * g.B : g.B;
    const uint64_t left = chunk_len - in_chunk;
    s.chunk = c;
    s.ordinal = j;
    s.expected = (c + 1 == g.C) ? g.last_tiles : g.tpc;
    s.stream_off = uint64_t(c) * g.B + in_chunk;
    s.packed_off = (uint64_t(lane) * g.q + (lane < g.r ? lane : g.r) + slot) * g.B + in_chunk;
    s.len = left < g.tile ? uint32_t(left) : g.tile;
    return s;
}

// Where byte s of the stream (below 2^40, the largest message) lies: its chunk and its position in it.
struct ChunkAt {
    uint32_t chunk;
    uint64_t rem;
};

HXT_HD ChunkAt chunk_at(const ChunkGeom &g, uint64_t s)
{
    // s and B are divided in units of 256 bytes.  The quotient is exact below 2^31 units and at most one too high from
    // there to 2^32 (the error term of make_fastdiv doubles), which the remainder shows.
    uint32_t c = fast_div(uint32_t(s >> 8), g.div_b256);
    uint64_t rem = s - uint64_t(c) * g.B;
    if (int64_t(rem) < 0) {
        --c;
        rem += g.B;
    }
    return ChunkAt{c, rem};
}

// Per-tensor view description for the ROWS and GENERIC kernels (merged dims, logical order).
struct TensorDev {
    int32_t ndim;                      // merged dims; for ROWS the last one is the contiguous run
    int32_t esize;
    uint32_t row_bytes;                // ROWS: bytes of one contiguous run
    uint32_t all_div;                  // 1: dim_div is valid for every dim and every shape[d] <= 2^30
    uint32_t low_or;                   // ROWS_SPLIT: OR of the run length and the outer strides in bytes (their low bits
                                       // give the widest naturally aligned piece the tensor side can be accessed in)
    uint32_t apart;                    // GENERIC: takes_apart is true for it
    FastDiv row_div;                   // ROWS: division by row_bytes
    FastDiv lane_div;                  // ROWS_SPLIT: division by the 16-byte vectors begun in a run
    FastDiv dim_div[HXT_MAX_DIMS];     // division by shape[d]: for the outer dims of a ROWS tensor, for all dims if all_div
    int64_t shape[HXT_MAX_DIMS];
    int64_t stride_b[HXT_MAX_DIMS];    // bytes
};

// Receiving rows in 16-byte vectors: a tile of n bytes that starts at byte col0 of a run of rb bytes deals lanes over the part
// of every run that lies in it, as many as the part has vectors begun; the last one of a part ends with it.  By run, not by
// tile, because a run's store must not be split into bursts; by the part, because a run can be much longer than a tile.
// A part that is no multiple of 16 bytes has a vector begun more than its bytes have: a tile of kDefaultTileBytes is done in one
// round of the kernel's 256 threads and 5 vectors each with runs of 64 bytes or more (4, as sends have, would leave a second
// round to a few dozen lanes.  Unpack, 4 against 5: rows of 204 bytes 8 MiB 6.9 -> 6.5 us, 32 MiB 20.2 -> 18.6, of 202 bytes
// 16 MiB 12.1 -> 11.5).
struct RunLanes {
    static constexpr uint32_t PER_THREAD = 5;
    uint32_t rb, col0, n, first, lanes, all;           // lanes of the first run's part, of a whole run, of the tile
    FastDiv div;                                       // by lanes
    struct Lane {
        uint32_t dr, at, skip;     // run (counted from the tile's first), the vector's byte of the tile, its bytes that the lane
    };                             // before has too (16: nothing to move, the part is shorter than a vector)
    // runs: those the tile meets
    HXT_HD RunLanes(uint32_t rb_, uint32_t col0_, uint32_t n_, uint32_t runs, FastDiv by_lanes) : rb(rb_), col0(col0_), n(n_), div(by_lanes)
    {
        const uint32_t part = rb - col0 < n ? rb - col0 : n;
        lanes = (rb + 15) >> 4;
        first = (part + 15) >> 4;
        all = first + (runs > 1 ? (runs - 2) * lanes + ((n - ((runs - 1) * rb - col0) + 15) >> 4) : 0);
    }
    HXT_HD Lane lane(uint32_t i) const
    {
        const uint32_t q = i < first ? 0 : fast_div(i - first, div), dr = i < first ? 0 : q + 1;
        const uint32_t k = i < first ? i : i - first - q * lanes;
        const uint32_t start = dr * rb - col0;         // (below zero, wrapped, for the first run)
        const uint32_t lo = dr ? start : 0, hi = start + rb < n ? start + rb : n, y = lo + 16 * k;
        const uint32_t at = y + 16 < hi ? y : hi - 16;
        return hi - lo < 16 ? Lane{dr, 0, 16} : Lane{dr, at, y - at};
    }
};

constexpr int kMaxGroupTensors = 64;   // base pointers passed by value per launch

struct TensorPlan {
    int ndim = 0;                      // merged
    int64_t shape[HXT_MAX_DIMS] = {0};
    int64_t stride[HXT_MAX_DIMS] = {0};  // elements
    int esize = 1;
    hxt_dtype_t dtype = HXT_U8;
    uint64_t elems = 0, bytes = 0, stream_off = 0;
    Kind kind = K_NONE;
    bool unpack_safe = true;
};

// Whether a tensor of the per-element kernel is sent by send_apart, which takes 16 / step neighbours of the last dim, `step` bytes
// apart, at a time.  Where these are not all of one run it reads them one by one, and a wave with one such lane waits for all
// of them: views of several dims go this way if runs are whole numbers of neighbours, or so long that few waves meet the end of
// one, which matters the less the more tiles there are.  Sends of 2, 8 and 32 MiB element by element against this, pitches 3
// elements more:
//   whole numbers: bytes every other, runs of 16 9.7 -> 7.2, 15.8 -> 9.1, 44 -> 24 us, every fourth, of 12 11.6 -> 9.4, 16.8 -> 13.1,
//     48 -> 38; bf16 every other, of 12 7.2 -> 7.3, 10.5 -> 9.0, 27 -> 24, of 200 7.1 -> 7.1, 10.3 -> 8.4, 27 -> 22 (runs of 8 were not
//     measured); every fourth, of 1024 7.9 -> 9.2, 11.8 -> 11.4, 34.2 -> 34.2;
//   others: bytes every other, runs of 101 11.2 -> 17.9, 15.6 -> 20.3, 44 -> 43, of 404 10.6 -> 15.0, 15.7 -> 16.7, 46 -> 37, of 1501
//     10.2 -> 10.4, 15.4 -> 12.1, 44 -> 29, of 2002 11.0 -> 12.6, 15.5 -> 14.5, 44 -> 34, of 4098 10.9 -> 9.8, 15.4 -> 11.4, 44 -> 28; every
//     fourth, of 101 12.1 -> 20.0, 16.8 -> 25.7, 47 -> 58, of 403 11.8 -> 15.4, 16.5 -> 18.9, 46.8 -> 46.4, of 1501 11.8 -> 11.7, 16.4 -> 14.7,
//     47 -> 39; bf16 every other, of 101 7.7 -> 12.0, 10.4 -> 14.9, 27 -> 34, of 403 7.4 -> 9.8, 10.5 -> 11.4, 29.0 -> 28.9, of 1501 7.1 -> 8.0,
//     10.3 -> 9.6, 26 -> 25, of 4098 7.5 -> 7.3, 10.3 -> 8.6, 26 -> 22; every fourth, of 4097 and more, never (30001 7.6 -> 8.8, 11.7 -> 12.3,
//     34 -> 35).
inline bool takes_apart(const TensorPlan &t)
{
    const int64_t run = t.shape[t.ndim - 1], step = t.stride[t.ndim - 1] * t.esize;
    if (t.esize > 2 || (step != 2 * t.esize && step != 4 * t.esize)) return false;
    if (t.ndim == 1) return run >= 32;
    const int64_t m = 16 / step;
    const bool some = t.bytes >= (uint64_t(6) << 20), many = t.bytes >= (uint64_t(24) << 20);       // tiles
    if (run >= 12 && run % m == 0) return m > 2 || some;
    return m > 2 && run >= (many ? 400 : (some ? 1500 : 4096));
}

struct Group {          // one kernel launch
    Kind kernel;        // K_CONTIG (serves ZERO tiles too), K_ROWS, K_ROWS_SPLIT, K_TRANSPOSE, K_GENERIC
    uint32_t first;     // first tile
    uint32_t count;
    uint32_t tensor_base;
    uint32_t n_tensors; // tensors addressed: [tensor_base, tensor_base + n_tensors)
    uint32_t apart;     // K_GENERIC: element sizes of tensors that takes_apart is true for, ORed
};

struct Plan {
    std::vector<TensorPlan> tensors;
    uint64_t N = 0, L = 0, B = 0, C = 0;
    int k = 1;
    std::vector<uint64_t> lane_off;      // k + 1 entries
    std::vector<uint64_t> lane_chunks;   // k
    uint32_t tile_bytes = 0;
    std::vector<Tile> tiles;             // grouped by kernel family, stream order inside a group
    std::vector<Group> groups;
    std::vector<uint32_t> chunk_tiles;   // arrivals each chunk's checksum expects: its tiles, plus one per TRANSPOSE_SPAN
                                         // tile that touches it
    std::vector<uint32_t> inc;           // TRANSPOSE_SPAN tiles: pairs (chunk, ordinal of this arrival among the chunk's),
                                         // a tile's pairs consecutive and ascending by chunk
    std::vector<TensorDev> tdev;
    bool all_unpack_safe = true;
    bool can_accumulate = true;          // every non-empty tensor is contiguous bf16 or f32
    ChunkGeom geom;                      // closed-form geometry of the packed stream
    bool uniform = false;                // the message is one contiguous tensor: geom alone describes the copy
    uint32_t uniform_tensor = 0;         // index of that tensor
    bool pads_ride = false;              // the contiguous group holds nothing but pads and there is one other group, of one
                                         // element size: one launch takes the tiles of both (they lie next to each other)
    uint32_t launches = 0;               // launches the groups take, one per group and element size

    uint64_t chunk_padded(uint64_t c) const;
    uint64_t chunk_packed_off(uint64_t c) const { return lane_off[c % k] + (c / k) * B; }
};

// Host-only, allocation-free: the closed-form geometry alone.  Returns an hxt_status.
int make_geom(uint64_t N, uint64_t L, uint64_t B, uint32_t k, uint32_t tile_bytes, ChunkGeom &g);

// Host-only construction of every table (no HIP call).  Returns an hxt_status.
int build_plan(const hxt_tensor_desc_t *tensors, int n_tensors, int n_lanes, size_t chunk_bytes,
               uint32_t tile_bytes, Plan &out);

constexpr uint32_t kDefaultTileBytes = 16384;  // bytes of the stream one workgroup moves (linear kinds)
// A TRANSPOSE tile is at most T x T elements, T chosen so that a tile row is 128-512 bytes.
HXT_HD constexpr uint32_t transpose_tile(uint32_t esize) { return esize <= 2 ? 128u : 64u; }

}  // namespace hxt

#endif
