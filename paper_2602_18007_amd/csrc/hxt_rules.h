// Rules of the launch code that only look at sizes: no HIP, so that they can be tested without a GPU.
#ifndef HXT_RULES_H
#define HXT_RULES_H

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

// Stream bytes up to which a message that would take several launches goes out in one (k_message).  Measured, pack + unpack
// with sums, launches of their own against one:
//   three launches or more: six tensors of five kinds 4 MiB 33 -> 14 us, 16 MiB 46 -> 25, 48 MiB 64 -> 50, 64 MiB 75 -> 64,
//     80 MiB 84 -> 76; three transposes of different element sizes 4 MiB 30 -> 16, 48 MiB 53 -> 48, 64 MiB 77 -> 77, but
//     80 MiB 90 -> 94.
//   two, where the gain is one launch each way and k_message's residency (3 or 4 workgroups per CU) soon costs more: padded
//     rows and a mask 4 MiB 16 -> 11, 12 MiB 23 -> 17; two transposes 12 MiB 27 -> 19; every other column and a mask 12 MiB
//     34 -> 28 (with tags 39 -> 34), but its pack alone 16 MiB with tags 20.4 -> 22.5 and 24 MiB 21.4 -> 24.7.
constexpr uint64_t kOneLaunchLimit = uint64_t(64) << 20;
constexpr uint64_t kOneLaunchForTwoLimit = uint64_t(12) << 20;

inline bool one_launch(const Plan &p)
{
    return p.launches > 1 && p.tensors.size() <= size_t(kMaxGroupTensors) &&
           launch_bytes(p) <= (p.launches > 2 ? kOneLaunchLimit : kOneLaunchForTwoLimit);
}

}  // namespace hxt

#endif
