// Rules of the launch code that only look at sizes: no HIP, so that they can be tested without a GPU.
#ifndef HXT_RULES_H
#define HXT_RULES_H

#include <algorithm>

#include "hxt_internal.h"

namespace hxt {

// Cache hints, chosen per launch from the stream bytes it moves, whatever chunks they are cut into (HXT_NT_USER /
// HXT_NT_PACKED, 0 or 1, override).
//   Packed side, stores: written through to the last-level cache, where the wire or hxt_unpack reads them
//     (store_packed16).  Better than non-temporal stores up to 1 GiB (pack + unpack with sums: 128 MiB 81 against 92 us,
//     288 MiB 171 against 197, 512 MiB 338 against 356); above, nothing of the buffer's start is left when it is read
//     and non-temporal stores are as good or better (1.7 GB pack + accumulate 1407 against 1401 us).  Buffers of 8 to
//     16 MiB that are unpacked right away on the same GPU would be faster left in the L2s (8 MiB 9.9 against 10.4 us, 16 MiB
//     16.0 against 16.6), which no wire reads; after the kernel that writes the tensor even those are not (16.5 against 15.8).
//   Packed side, loads: cacheable up to 128 MiB, where the buffer still is in the last-level cache when it is read
//     (unpack of one of two buffers in turn, cacheable against non-temporal: 80 MiB 26.8 against 30.6 us, 96 MiB 31.1
//     against 35.8, 128 MiB 41.0 against 46.5; accumulated 62.8 against 72.9; rows of 101 bf16 elements 81.9 against 102).
//     Buffers that have left the cache lose less by it (128 MiB, pack + unpack 82.8 against 81.1).  Non-temporal above:
//     what has been read only pushes out what is still to be read (pack + unpack 160 MiB 98.8 against 106.4, 256 MiB 153
//     against 158).  The stand-alone passes, which take nothing but the buffer through the cache, already from 64 MiB on
//     (pack + hxt_checksum 96 MiB 45.2 against 50.2 us, 128 MiB 57.7 against 67.6).
//   Tensor side, loads and stores: non-temporal.  A message's tensors are new each time: keeping their lines pays only
//     where the very same tensor is sent again (32 MiB over and over, pack + unpack: 24.8 us non-temporal, 22.6 cacheable;
//     three in turn 26.4 and 24.7) and costs where it has just been written or has left the cache (through two packed
//     buffers, 8 MiB 10.4 against 11.5 us, 16 MiB 16.6 against 17.1, a transposed 32 MiB matrix 26.8 against 27.9).
//   But loads from tensors at bases that are not multiples of 16 bytes are cacheable up to 64 MiB: neighbouring vectors
//     share bursts there (base one element off, tensor just written, pack + unpack: 32 MiB 36.1 us non-temporal, 32.7
//     cacheable; 64 MiB 63.6 and 56.6; but pack of a 128 MiB tensor that is not in the cache 43.5 and 49.4).
constexpr uint64_t kCacheableMisalignedLoads = uint64_t(64) << 20;
constexpr uint64_t kCacheablePackedLoads = uint64_t(128) << 20, kCacheablePackedPasses = uint64_t(64) << 20;
constexpr uint64_t kWrittenThroughLimit = uint64_t(1) << 30;

// Bytes a launch over the message moves on the packed side (its packed buffer, whole chunks, can be much longer).
inline uint64_t launch_bytes(const Plan &p) { return p.L; }

// hint: HXT_OPT_PACKED_HINT of the plan that decides; bytes: those of the launch; load: it reads the packed side.
inline bool packed_nontemporal(int hint, uint64_t bytes, bool load)
{
    return hint >= 0 ? hint != 0 : bytes > (load ? kCacheablePackedLoads : kWrittenThroughLimit);
}

// forced: HXT_NT_USER; send: the launch reads tensors; low: all their base addresses ORed.
inline bool user_nontemporal(int forced, bool send, uintptr_t low, uint64_t bytes)
{
    return forced >= 0 ? forced != 0 : !(send && low % 16 != 0 && bytes <= kCacheableMisalignedLoads);
}

inline bool pass_nontemporal(int hint, uint64_t bytes) { return hint >= 0 ? hint != 0 : bytes > kCacheablePackedPasses; }

// Packed elements of the per-element kernel: written through in messages of more than 12 MiB (of bytes: up to 64); smaller
// ones find them in the L2 when they are unpacked here, and those of 8 bytes are left there always.  Every other column,
// pack + unpack, through against not: bf16 4 MiB 17.0 and 14.3 us, 8 MiB 20.9 and 19.2, 16 MiB 32.0 and 34.2, 32 MiB 56.3
// and 59.8; f32 8 MiB 18.2 and 16.6, 32 MiB 53.0 and 54.8; bytes 4 MiB 24.3 and 19.9, 32 MiB 74.2 and 76.2, 96 MiB just
// written 215 and 207; f64 16 MiB 30.3 and 29.0.
constexpr uint64_t kElementsThrough = uint64_t(12) << 20, kBytesThrough = uint64_t(64) << 20;

inline bool elements_through(int esize, uint64_t bytes)
{
    return esize < 8 && bytes > kElementsThrough && (esize > 1 || bytes <= kBytesThrough);
}

// Stream bytes up to which a message that would take several launches goes out in one (k_message, 4 workgroups per CU).
// Measured, pack + unpack with sums, launches of their own against one:
//   three launches or more: six tensors of five kinds 16 MiB 64 -> 28 us, 48 MiB 92 -> 59, 64 MiB 105 -> 70 (with tags 128 ->
//     79), 80 MiB 121 -> 86; three transposes of different element sizes 4 MiB 33 -> 15, 48 MiB 76 -> 63, 64 MiB 90 -> 78, 80 MiB
//     112 -> 95; every other column, odd rows and a mask 16 MiB 40 -> 27, 64 MiB 83 -> 75, but the pack alone 38.3 -> 38.4 there
//     and 43.9 -> 48.0 at 80 MiB (98 -> 90 a pair): the line lies where sending alone would lose.
//   two, where the gain is one launch each way: odd rows and a mask 8 MiB 19 -> 15, 12 MiB 22 -> 17; two transposes 12 MiB 28 ->
//     18; every third column and a mask 12 MiB 38 -> 33.  Every other column and a mask, where k_message goes without send_apart:
//     4 MiB 18.2 -> 16.0, 12 MiB 28.9 -> 27.4 (with tags 33.4 -> 30.7) with the pack alone 12.1 -> 13.2, 16 MiB 35.4 -> 33.7 and
//     14.6 -> 15.7, 24 MiB 45.0 -> 48.2 and 18.4 -> 23.9.  Other pairs would gain beyond the line too (16 MiB: odd rows and a mask
//     28 -> 21, two transposes 25 -> 17).
constexpr uint64_t kOneLaunchLimit = uint64_t(64) << 20;
constexpr uint64_t kOneLaunchForTwoLimit = uint64_t(12) << 20;

inline bool one_launch(const Plan &p)
{
    return p.launches > 1 && p.tensors.size() <= size_t(kMaxGroupTensors) &&
           launch_bytes(p) <= (p.launches > 2 ? kOneLaunchLimit : kOneLaunchForTwoLimit);
}

// Byte ranges of the packed buffer that staging moves for a lane selection.
inline int stage_ranges(const Plan &p, int lane, uint64_t (*r)[2])
{
    auto used = [&](int l) -> uint64_t {
        uint64_t n = p.lane_chunks[l];
        if (n == 0) return 0;
        return (n - 1) * p.B + p.chunk_padded((n - 1) * p.k + l);
    };
    if (lane >= 0) {
        r[0][0] = p.lane_off[lane];
        r[0][1] = used(lane);
        return r[0][1] ? 1 : 0;
    }
    // all lanes: regions are adjacent; only the lane holding the last chunk can end short
    if (p.C == 0) return 0;
    const int ls = int((p.C - 1) % p.k);
    const uint64_t cut = p.lane_off[ls] + used(ls), total = p.lane_off[p.k];
    r[0][0] = 0;
    if (cut == p.lane_off[ls + 1]) {
        r[0][1] = total;
        return 1;
    }
    r[0][1] = cut;
    if (p.lane_off[ls + 1] == total) return 1;
    r[1][0] = p.lane_off[ls + 1];
    r[1][1] = total - p.lane_off[ls + 1];
    return 2;
}

// The copies in which the CPU-forwarding stream stages a message, in pieces of equal bytes: the host-to-device copies of a
// piece start when that piece is on the host, so that fewer bytes go with the other direction idle when a window of messages
// (drain_every, or all of them) begins and ends.  Whole against in pieces, windows of 4: 8 x 56 MiB in three 11.91 -> 10.92 ms,
// 16 x 24 MiB in three 10.63 -> 9.81, 16 x 19 MiB in three 8.65 -> 8.08 (in two 8.20), 8 x 12 MiB in two 2.79 -> 2.66 (in three
// 2.73), 16 x 10 MiB in two 4.73 -> 4.55; 8 MiB in two 3.93 -> 3.83, but also 4.07 -> 4.26 and 1.97 -> 2.19.
// Cut only as far as the runtime still overlaps the two directions: with more outstanding a stream takes up to twice as long,
// now and then or always.  No more than 16 copies a direction and window (a piece that lies in both ranges of the packed
// buffer is two; 20 to 32: 13 MiB 5.65 -> 11.2 ms, 17 MiB 7.15 -> 13.3, 25 MiB 10.2 -> 11.4), and windows of more than 4
// messages only from 24 MiB on (two pieces in windows of 8: 24 MiB 9.74 -> 9.33; of 5 to 8: 10 MiB 5.71 -> 5.99, 6.70 -> 8.54,
// 7.66 -> 10.9, 4.36 -> 7.41, 16 MiB 8.81 -> 8.40 and 10.3 -> 9.93, but 11.7 -> 14.0 and 6.62 -> 8.54).
constexpr int kMostPieces = 3, kMostCopies = kMostPieces + 1, kShortWindow = 4;
constexpr uint64_t kTwoPieces = uint64_t(10) << 20, kThreePieces = uint64_t(14) << 20, kPiecesInLongWindows = uint64_t(24) << 20;

struct StagedCopy {
    uint64_t off, bytes;
    int piece;
};

inline int staging_copies(const Plan &p, int window, StagedCopy *out)
{
    uint64_t r[2][2];
    const int n = stage_ranges(p, -1, r);
    if (n == 0) return 0;
    const uint64_t total = r[0][1] + (n > 1 ? r[1][1] : 0);
    int pieces = total >= kThreePieces ? kMostPieces : (total >= kTwoPieces ? 2 : 1);
    if (window > kShortWindow) pieces = total >= kPiecesInLongWindows ? std::max(1, std::min(kMostPieces, 16 / window - (n - 1))) : 1;
    const uint64_t step = (total / uint64_t(pieces) + HXT_ALIGN - 1) / HXT_ALIGN * HXT_ALIGN;
    int m = 0;
    uint64_t before = 0;                                   // bytes of the ranges ahead
    for (int i = 0; i < n; ++i) {
        for (uint64_t o = 0; o < r[i][1]; ++m) {
            const uint64_t piece = (before + o) / step, end = std::min(r[i][1], (piece + 1) * step - before);
            out[m] = StagedCopy{r[i][0] + o, end - o, int(piece)};
            o = end;
        }
        before += r[i][1];
    }
    return m;
}

}  // namespace hxt

#endif
