// HIP kernels (gfx950) of libhxt: device code only, included by hxt_device.hip.
//
// Data plane of the paper's Section 2.2 transfer: user buffer -> chunk buffer on
// the sender (pack), chunk buffer -> user buffer on the receiver (unpack), and a
// per-chunk integrity sum.  Every kernel is a pure byte mover: data is handled as
// unsigned integers so that any bit pattern survives unchanged.
//
// Work decomposition: the host planner cuts the message into tiles (one per
// workgroup, never crossing a tensor, and never a chunk except in
// k_transpose_span); a workgroup reads its 64-byte tile record with scalar
// loads and moves the bytes with 128-bit vector accesses where the view allows.
// Checksums are accumulated per thread in 64-bit integers, reduced across the
// 64-lane wavefront with shuffles, across the four waves through LDS, and added
// to the chunk's total with one 64-bit atomic per workgroup (k_transpose_span:
// one per chunk its tile touches); integer addition makes the result
// independent of the order of arrival.
#ifndef HXT_KERNELS_H
#define HXT_KERNELS_H

#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "hxt_internal.h"

namespace hxt {

constexpr int kThreads = 256;
constexpr int kUnroll = 4;
constexpr uint32_t kTagMagic = 0x31545848u;     // 'H','X','T','1' in memory order

struct BasePtrs {
    uint8_t *p[kMaxGroupTensors];
};

struct ElemKinds {                     // per tensor of a launch group: 1 = 32-bit float, 0 = bf16
    uint8_t f32[kMaxGroupTensors];
};

// Accumulator slot of a checksum in flight.  Every operation of a plan (pack, unpack, the
// stand-alone passes, ...) owns its own set of slots, SumCtx::stride bytes apart (256 unless the
// plan has very many chunks) so that neighbouring slots' atomics land in different memory
// channels.  Always zero between kernels.
struct Acc {
    unsigned long long sum;
    uint32_t cnt;
    uint32_t pad;
};

struct SumCtx {
    uint64_t *sums;      // caller's array, one entry per chunk
    uint8_t *acc;        // plan-owned Acc slots: C * fan first-level slots, then C second-level slots
    uint32_t stride;     // bytes between slots
    uint32_t sum_bits;   // > 0: a chunk's total fits this many bits and the arrival count rides above it
    uint32_t fan;        // first-level slots per chunk (power of two); 1 = second level only
    uint32_t chunks;     // C
};

// ---- small device helpers ----------------------------------------------------

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

template <bool NT>
__device__ __forceinline__ u32x4 load16(const u32x4 *p)
{
    if constexpr (NT) return __builtin_nontemporal_load(p);
    else return *p;
}

template <bool NT>
__device__ __forceinline__ void store16(u32x4 *p, u32x4 v)
{
    if constexpr (NT) __builtin_nontemporal_store(v, p);
    else *p = v;
}

template <bool NT, typename E>
__device__ __forceinline__ E load_elem(const E *p)
{
    if constexpr (NT) return __builtin_nontemporal_load(p);
    else return *p;
}

template <bool NT, typename E>
__device__ __forceinline__ void store_elem(E *p, E v)
{
    if constexpr (NT) __builtin_nontemporal_store(v, p);
    else *p = v;
}

// Stores to the packed buffer.  Not non-temporal means written through the XCD's L2 (device scope): the bytes are
// kept by the memory-side last-level cache, where the wire or hxt_unpack on any XCD finds them, and no dirty lines
// are left in eight L2s for the end of the kernel to write back.  Measured, pack + unpack of one message with sums:
// 56 MiB 40.5 us written back, 39.1 us written through; 2 x 32 MiB 46.2 -> 44.3 us.
template <bool NT>
__device__ __forceinline__ void store_packed16(u32x4 *p, u32x4 v)
{
    if constexpr (NT) __builtin_nontemporal_store(v, p);
    else __builtin_amdgcn_global_store_b128((__attribute__((address_space(1))) u32x4 *)p, v, "agent");
}

// THROUGH = false: element by element, where writing through does not pay, and left to the L2.
template <bool NT, bool THROUGH = true, typename E>
__device__ __forceinline__ void store_packed_elem(E *p, E v)
{
    if constexpr (NT) __builtin_nontemporal_store(v, p);
    else if constexpr (THROUGH) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else *p = v;
}

// 16 bytes at any address: the hardware takes misaligned vector accesses, and 64 lanes of them next to each other
// still cost little more than aligned ones.
typedef u32x4 u32x4_any __attribute__((aligned(1)));

template <bool NT>
__device__ __forceinline__ u32x4 load16_any(const uint8_t *p)
{
    if constexpr (NT) return __builtin_nontemporal_load(reinterpret_cast<const u32x4_any *>(p));
    else return *reinterpret_cast<const u32x4_any *>(p);
}

template <bool NT>
__device__ __forceinline__ void store16_any(uint8_t *p, u32x4 v)
{
    if constexpr (NT) __builtin_nontemporal_store(v, reinterpret_cast<u32x4_any *>(p));
    else *reinterpret_cast<u32x4_any *>(p) = v;
}

// The same, cacheable, for one side of a branch whose other side is non-temporal (as one store the hint would be lost).
__device__ __forceinline__ void store16_cached(uint8_t *p, u32x4 v)
{
    __builtin_amdgcn_global_store_b128((__attribute__((address_space(1))) u32x4 *)reinterpret_cast<u32x4 *>(p), v, "wavefront");
}

// The first n elements of a vector, one at a time.
template <typename E>
__device__ __forceinline__ void store_elems(uint8_t *p, u32x4 v, uint32_t n)
{
    union {
        u32x4 x;
        E e[16 / sizeof(E)];
    } o{v};
#pragma unroll
    for (uint32_t q = 0; q < 16 / sizeof(E); ++q)
        if (q < n) reinterpret_cast<E *>(p)[q] = o.e[q];
}

// Vector v of a span of nvec (>= 1) vectors, zeros beyond its end.  The load itself is unconditional (the
// index is clamped into the span): the loads of an unrolled round are then all issued before the first
// of them is waited for, where guarded loads are waited for one by one.
template <bool NT>
__device__ __forceinline__ u32x4 load16_or_zero(const u32x4 *s, uint32_t v, uint32_t nvec)
{
    const u32x4 x = load16<NT>(s + min(v, nvec - 1));
    return v < nvec ? x : u32x4{0, 0, 0, 0};
}

__device__ __forceinline__ uint64_t words_sum(u32x4 v)
{
    return (uint64_t(v.x) + uint64_t(v.y)) + (uint64_t(v.z) + uint64_t(v.w));
}

// The sum of the packed words that 16 bytes at packed position pos contribute to: byte k weighs 256^((pos + k) mod 4),
// so a vector that starts inside a word is summed as words rotated by its phase.
__device__ __forceinline__ uint64_t rotated_sum(u32x4 v, uint32_t pos)
{
    const uint32_t by = 8 * (pos & 3u);
    return words_sum(u32x4{__builtin_rotateleft32(v.x, by), __builtin_rotateleft32(v.y, by), __builtin_rotateleft32(v.z, by),
                           __builtin_rotateleft32(v.w, by)});
}

// Bytes [from, to) of a vector, zeros elsewhere.
__device__ __forceinline__ u32x4 keep_bytes(u32x4 v, uint32_t from, uint32_t to)
{
    auto below = [](uint32_t word, uint32_t k) {         // mask of the bytes of a word that lie below byte k of the vector
        const uint32_t lo = 4 * word;
        return k <= lo ? 0u : (k >= lo + 4 ? ~0u : (1u << (8 * (k - lo))) - 1u);
    };
    return u32x4{v.x & below(0, to) & ~below(0, from), v.y & below(1, to) & ~below(1, from),
                 v.z & below(2, to) & ~below(2, from), v.w & below(3, to) & ~below(3, from)};
}

__device__ __forceinline__ u32x4 shift_bytes_down(u32x4 v, uint32_t by)         // by < 16: byte k of the result is byte k + by
{
    const unsigned __int128 x = __builtin_bit_cast(unsigned __int128, v) >> (8 * by);
    return __builtin_bit_cast(u32x4, x);
}

__device__ __forceinline__ u32x4 shift_bytes_up(u32x4 v, uint32_t by)
{
    const unsigned __int128 x = __builtin_bit_cast(unsigned __int128, v) << (8 * by);
    return __builtin_bit_cast(u32x4, x);
}

// Sum over every LANES lanes in a DPP row of 16, in the last of them (the others hold partial sums).  Inactive lanes count
// as zero.
template <int CTRL, int ROWS = 0xF>
__device__ __forceinline__ uint64_t dpp_plus(uint64_t v)
{
    const uint32_t lo = uint32_t(__builtin_amdgcn_update_dpp(0, int(uint32_t(v)), CTRL, ROWS, 0xF, false));
    const uint32_t hi = uint32_t(__builtin_amdgcn_update_dpp(0, int(uint32_t(v >> 32)), CTRL, ROWS, 0xF, false));
    return v + (uint64_t(hi) << 32 | lo);
}

template <uint32_t LANES>
__device__ __forceinline__ uint64_t lanes_sum(uint64_t v)
{
    static_assert(LANES == 8 || LANES == 16);
    v = dpp_plus<0x111>(v);                              // row_shr 1, 2, 4, 8
    v = dpp_plus<0x112>(v);
    v = dpp_plus<0x114>(v);
    return LANES == 16 ? dpp_plus<0x118>(v) : v;
}

// One arrival at an accumulator slot that expects `expected` of them: adds `value` and reports
// whether this was the last arrival, in which case `value` becomes the slot's total and the
// slot is zero again.  Only relaxed device-scope atomics touch a slot (no cache write-back).
//   sum_bits > 0: totals stay below 2^sum_bits (a chunk has at most B/4 words of 32 bits) and
//     the arrival count fits in the bits above, so one atomic adds and takes the ticket at once.
//   sum_bits == 0: sum and ticket are two words; the ticket is taken after the wave has seen
//     its own addition return, which orders the two.
__device__ __forceinline__ bool slot_arrive(Acc *a, unsigned long long &value, uint32_t expected, uint32_t sum_bits)
{
    if (expected == 1) return true;
    if (sum_bits) {
        const unsigned long long one = 1ull << sum_bits;
        const unsigned long long before = __hip_atomic_fetch_add(&a->sum, one + value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if ((before >> sum_bits) != expected - 1) return false;
        __hip_atomic_store(&a->sum, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        value = (before + value) & (one - 1);
        return true;
    }
    const unsigned long long before = __hip_atomic_fetch_add(&a->sum, value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::"v"(uint32_t(before)) : "memory");
    const uint32_t ticket = __hip_atomic_fetch_add(&a->cnt, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (ticket != expected - 1) return false;
    value = __hip_atomic_exchange(&a->sum, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&a->cnt, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return true;
}

// Adds this workgroup's partial sum to its chunk.  A chunk made of many tiles spreads its
// arrivals over `fan` first-level slots (tile ordinal mod fan) so that they do not queue on
// one address; the last arrival of a first-level slot carries that slot's total to the chunk's
// second-level slot, and the last arrival there writes sums[chunk].
// One arrival, made by one thread: `s` is a finished partial sum for `chunk`, this being arrival number
// `ordinal` of the `expected` the chunk gets.
__device__ __forceinline__ void commit_total(unsigned long long s, uint32_t chunk, uint32_t ordinal, uint32_t expected,
                                             const SumCtx &cx)
{
    Acc *top = reinterpret_cast<Acc *>(cx.acc + (size_t(cx.chunks) * cx.fan + chunk) * cx.stride);
    bool last;
    if (cx.fan == 1 || expected < 2 * cx.fan) {
        last = slot_arrive(top, s, expected, cx.sum_bits);
    } else {
        const uint32_t sub = ordinal & (cx.fan - 1);
        const uint32_t share = expected / cx.fan + (sub < (expected & (cx.fan - 1)) ? 1u : 0u);
        Acc *first = reinterpret_cast<Acc *>(cx.acc + (size_t(chunk) * cx.fan + sub) * cx.stride);
        last = slot_arrive(first, s, share, cx.sum_bits) && slot_arrive(top, s, cx.fan, cx.sum_bits);
    }
    if (last) cx.sums[chunk] = s;
}

__device__ __forceinline__ void chunk_commit(uint64_t acc, uint32_t chunk, uint32_t ordinal, uint32_t expected,
                                             const SumCtx &cx)
{
    __shared__ uint64_t part[kThreads / 64];
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_down(acc, o, 64);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) part[wave] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long s = 0;
#pragma unroll
        for (int w = 0; w < kThreads / 64; ++w) s += part[w];
        commit_total(s, chunk, ordinal, expected, cx);
    }
}

// Copy `bytes` contiguous bytes between a user tensor and the packed buffer (pack: user ->
// packed, unpack: packed -> user) in 16-byte vectors, UNROLL independent loads in flight per
// thread before the first store; a last partial vector goes byte by byte.  NTU / NTP mark
// the user-side / packed-side accesses non-temporal.  The tensor may start at any address: with a base that is only
// element aligned the same instructions cost up to 8 % (32 MiB, pack + unpack, all buffers cold: 27.0 us aligned, 29.1 two
// bytes off; putting vectors together from narrower aligned accesses took 31.0).
template <bool UNPACK, bool CSUM, bool NTU, bool NTP>
__device__ __forceinline__ uint64_t copy_span(uint8_t *user, uint8_t *pk, uint32_t bytes)
{
    const uint32_t nvec = bytes >> 4;
    constexpr uint32_t STEP = kThreads * kUnroll;
    const uint32_t full = nvec / STEP * STEP;            // uniform: blocks that need no bounds checks
    auto load = [&](uint32_t v) {
        if constexpr (UNPACK) return load16<NTP>(reinterpret_cast<const u32x4 *>(pk) + v);
        else return load16_any<NTU>(user + (size_t(v) << 4));
    };
    auto store = [&](uint32_t v, u32x4 r) {
        if constexpr (UNPACK) store16_any<NTU>(user + (size_t(v) << 4), r);
        else store_packed16<NTP>(reinterpret_cast<u32x4 *>(pk) + v, r);
    };
    uint64_t acc = 0;
    for (uint32_t v = threadIdx.x; v < full; v += STEP) {
        u32x4 r[kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) r[u] = load(v + u * kThreads);
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            store(v + u * kThreads, r[u]);
            if constexpr (CSUM) acc += words_sum(r[u]);
        }
    }
    for (uint32_t v = full + threadIdx.x; v < nvec; v += kThreads) {
        const u32x4 r = load(v);
        store(v, r);
        if constexpr (CSUM) acc += words_sum(r);
    }
    const uint32_t tail = bytes & 15;                    // only at the very end of a tensor
    if (threadIdx.x < tail) {
        const uint32_t i = (nvec << 4) + threadIdx.x;
        const uint8_t b = (UNPACK ? pk : user)[i];
        (UNPACK ? user : pk)[i] = b;
        if constexpr (CSUM) acc += uint64_t(b) << (8 * (i & 3));
    }
    return acc;
}

// ---- receive and accumulate -----------------------------------------------------
// new = round(old + arriving) per element.  bf16: both operands widened exactly to binary32,
// added in binary32, the sum rounded to bf16 to nearest with ties to even.  f32: binary32
// addition.  Every NaN result becomes the canonical quiet NaN, so that the outcome does not
// depend on NaN payload propagation.
__device__ __forceinline__ uint32_t f32_to_bf16_rne(float f)
{
    const uint32_t u = __float_as_uint(f);
    if ((u & 0x7FFFFFFFu) > 0x7F800000u) return 0x7FC0u;
    return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}

__device__ __forceinline__ uint32_t add_bf16x2(uint32_t old, uint32_t in)
{
    const float lo = __uint_as_float(old << 16) + __uint_as_float(in << 16);
    const float hi = __uint_as_float(old & 0xFFFF0000u) + __uint_as_float(in & 0xFFFF0000u);
    return f32_to_bf16_rne(lo) | (f32_to_bf16_rne(hi) << 16);
}

__device__ __forceinline__ uint32_t add_f32(uint32_t old, uint32_t in)
{
    const uint32_t u = __float_as_uint(__uint_as_float(old) + __uint_as_float(in));
    return (u & 0x7FFFFFFFu) > 0x7F800000u ? 0x7FC00000u : u;
}

template <bool F32>
__device__ __forceinline__ u32x4 add_vec(u32x4 old, u32x4 in)
{
    if constexpr (F32) return u32x4{add_f32(old.x, in.x), add_f32(old.y, in.y), add_f32(old.z, in.z), add_f32(old.w, in.w)};
    else return u32x4{add_bf16x2(old.x, in.x), add_bf16x2(old.y, in.y), add_bf16x2(old.z, in.z), add_bf16x2(old.w, in.w)};
}

// Adds `bytes` arriving contiguous bytes at pk to the tensor bytes at user (element aligned; a last partial vector goes
// element by element).  Returns the checksum
// contribution of the packed bytes read.
template <bool F32, bool CSUM, bool NTU, bool NTP>
__device__ __forceinline__ uint64_t accumulate_span(uint8_t *user, const uint8_t *pk, uint32_t bytes)
{
    const u32x4 *in = reinterpret_cast<const u32x4 *>(pk);
    const uint32_t nvec = bytes >> 4;
    constexpr int U = 2;                                   // two vectors of each operand in flight per thread
    constexpr uint32_t STEP = kThreads * U;
    const uint32_t full = nvec / STEP * STEP;
    uint64_t acc = 0;
    for (uint32_t v = threadIdx.x; v < full; v += STEP) {
        u32x4 a[U], b[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            a[u] = load16<NTP>(in + v + u * kThreads);
            b[u] = load16_any<NTU>(user + (size_t(v + u * kThreads) << 4));
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            store16_any<NTU>(user + (size_t(v + u * kThreads) << 4), add_vec<F32>(b[u], a[u]));
            if constexpr (CSUM) acc += words_sum(a[u]);
        }
    }
    for (uint32_t v = full + threadIdx.x; v < nvec; v += kThreads) {
        const u32x4 a = load16<NTP>(in + v);
        uint8_t *at = user + (size_t(v) << 4);
        store16_any<NTU>(at, add_vec<F32>(load16_any<NTU>(at), a));
        if constexpr (CSUM) acc += words_sum(a);
    }
    constexpr uint32_t ES = F32 ? 4 : 2;
    const uint32_t tail = (bytes & 15) / ES;               // whole elements in the last partial vector
    if (threadIdx.x < tail) {
        const uint32_t off = (nvec << 4) + threadIdx.x * ES;
        if constexpr (F32) {
            const uint32_t a = *reinterpret_cast<const uint32_t *>(pk + off);
            uint32_t *d = reinterpret_cast<uint32_t *>(user + off);
            *d = add_f32(*d, a);
            if constexpr (CSUM) acc += a;
        } else {
            const uint32_t a = *reinterpret_cast<const uint16_t *>(pk + off);
            uint16_t *d = reinterpret_cast<uint16_t *>(user + off);
            *d = uint16_t(add_bf16x2(*d, a));
            if constexpr (CSUM) acc += uint64_t(a) << (8 * (off & 3));
        }
    }
    return acc;
}

// Pad bytes (fewer than 256): pack writes zeros, unpack only reads them for the sum.
// `phase` is the position of pk[0] within its 32-bit word.
template <bool UNPACK, bool CSUM>
__device__ __forceinline__ uint64_t pad_span(uint8_t *pk, uint32_t bytes, uint32_t phase)
{
    uint64_t acc = 0;
    for (uint32_t i = threadIdx.x; i < bytes; i += kThreads) {
        if constexpr (!UNPACK) pk[i] = 0;
        if constexpr (UNPACK && CSUM) acc += uint64_t(pk[i]) << (8 * ((phase + i) & 3));
    }
    return acc;
}

// ---- uniform copy: messages that are one contiguous tensor each -------------------
// No table: tile -> (chunk, lane, slot, offsets) in closed form from the kernel arguments.
// One launch can serve several such messages (the forward activation and the backward
// gradient that cross a stage boundary at the same point of the schedule): workgroups
// [first_tile, first_tile + ntiles) belong to message i.
constexpr int kMaxBatch = 4;

struct UniformItem {
    ChunkGeom g;
    uint8_t *user;
    uint8_t *packed;
    SumCtx cx;
    uint32_t first_tile;
    uint32_t unpack;       // direction of this item; only read by the mixed-direction instantiation
};

enum Direction { DIR_PACK = 0, DIR_UNPACK = 1, DIR_MIXED = 2 };

struct UniformArgs {
    UniformItem it[kMaxBatch];
    uint32_t n;
};

template <bool UNPACK, bool CSUM, bool NTU, bool NTP>
__device__ __forceinline__ void uniform_tile(const UniformItem &it, uint32_t tile)
{
    const ChunkGeom &g = it.g;
    const TileSpan t = locate_tile(g, tile);
    const uint64_t left = g.N > t.stream_off ? g.N - t.stream_off : 0;     // tensor bytes from here on
    const uint32_t data = left < t.len ? uint32_t(left) : t.len;
    uint8_t *pk = it.packed + t.packed_off;
    uint64_t acc = copy_span<UNPACK, CSUM, NTU, NTP>(it.user + t.stream_off, pk, data);
    if (data < t.len) acc += pad_span<UNPACK, CSUM>(pk + data, t.len - data, data);
    if constexpr (CSUM) chunk_commit(acc, t.chunk, t.ordinal, t.expected, it.cx);
}

// DIR: all items pack, all unpack, or each item says which (a micro-batch stream overlaps the
// unpack of one message with the pack of the next inside one launch).
template <int DIR, bool CSUM, bool NTU, bool NTP>
__global__ __launch_bounds__(kThreads) void k_uniform(UniformArgs a)
{
    uint32_t m = 0;
#pragma unroll
    for (uint32_t i = 1; i < kMaxBatch; ++i)
        if (i < a.n && blockIdx.x >= a.it[i].first_tile) m = i;
    const UniformItem &it = a.it[m];
    const uint32_t tile = blockIdx.x - it.first_tile;
    if constexpr (DIR == DIR_MIXED) {
        if (it.unpack) uniform_tile<true, CSUM, NTU, NTP>(it, tile);
        else uniform_tile<false, CSUM, NTU, NTP>(it, tile);
    } else {
        uniform_tile<DIR == DIR_UNPACK, CSUM, NTU, NTP>(it, tile);
    }
}

// ---- contiguous tensors of a multi-tensor message: table driven ---------------------
template <bool UNPACK, bool CSUM, bool NTU, bool NTP>
__global__ __launch_bounds__(kThreads) void k_contig(const Tile *__restrict__ tiles,
                                                     const uint32_t *__restrict__ chunk_tiles, BasePtrs bases,
                                                     uint8_t *__restrict__ packed, SumCtx cx)
{
    const Tile t = tiles[blockIdx.x];
    uint64_t acc;
    if (t.kind == K_ZERO)
        acc = pad_span<UNPACK, CSUM>(packed + t.packed_off, t.n0, uint32_t(t.packed_off));
    else
        acc = copy_span<UNPACK, CSUM, NTU, NTP>(bases.p[t.tensor] + t.src_off, packed + t.packed_off, t.n0);
    if constexpr (CSUM) chunk_commit(acc, t.chunk, t.ordinal, chunk_tiles[t.chunk], cx);
}

// ---- receive and accumulate: the uniform and the table-driven contiguous kernels -----
template <bool CSUM, bool NTU, bool NTP>
__global__ __launch_bounds__(kThreads) void k_uniform_accumulate(UniformArgs a)
{
    uint32_t m = 0;                                    // up to kMaxBatch messages per launch, as in k_uniform
#pragma unroll
    for (uint32_t i = 1; i < kMaxBatch; ++i)
        if (i < a.n && blockIdx.x >= a.it[i].first_tile) m = i;
    const UniformItem &it = a.it[m];
    const ChunkGeom &g = it.g;
    const TileSpan t = locate_tile(g, blockIdx.x - it.first_tile);
    const uint64_t left = g.N > t.stream_off ? g.N - t.stream_off : 0;
    const uint32_t data = left < t.len ? uint32_t(left) : t.len;
    uint8_t *pk = it.packed + t.packed_off;
    uint64_t acc = it.unpack ? accumulate_span<true, CSUM, NTU, NTP>(it.user + t.stream_off, pk, data)
                             : accumulate_span<false, CSUM, NTU, NTP>(it.user + t.stream_off, pk, data);
    if (data < t.len) acc += pad_span<true, CSUM>(pk + data, t.len - data, data);
    if constexpr (CSUM) chunk_commit(acc, t.chunk, t.ordinal, t.expected, it.cx);
}

template <bool CSUM, bool NTU, bool NTP>
__global__ __launch_bounds__(kThreads) void k_contig_accumulate(const Tile *__restrict__ tiles,
                                                                const uint32_t *__restrict__ chunk_tiles,
                                                                BasePtrs bases, ElemKinds kinds,
                                                                uint8_t *__restrict__ packed, SumCtx cx)
{
    const Tile t = tiles[blockIdx.x];
    uint64_t acc;
    if (t.kind == K_ZERO)
        acc = pad_span<true, CSUM>(packed + t.packed_off, t.n0, uint32_t(t.packed_off));
    else if (kinds.f32[t.tensor])
        acc = accumulate_span<true, CSUM, NTU, NTP>(bases.p[t.tensor] + t.src_off, packed + t.packed_off, t.n0);
    else
        acc = accumulate_span<false, CSUM, NTU, NTP>(bases.p[t.tensor] + t.src_off, packed + t.packed_off, t.n0);
    if constexpr (CSUM) chunk_commit(acc, t.chunk, t.ordinal, chunk_tiles[t.chunk], cx);
}

// ---- strong check: plain sum and position-weighted sum of every chunk -----------------
// out[2c] = sum of the chunk's words, out[2c+1] = sum of (j+1) * word j, both mod 2^64.
// A logical accumulator is a pair of slots (2s: plain sum and arrival count, 2s+1: weighted
// sum); the ticket is taken after both additions have returned.  Same two-level fan-out as
// chunk_commit: first-level pairs C*fan, then one second-level pair per chunk.
// sum_bits > 0 (see slot_arrive): the plain sum and the arrival count share one word, so the arrival is
// the weighted sum's addition, then one addition that also takes the ticket; sum_bits == 0: three steps.
__device__ __forceinline__ bool pair_arrive(uint8_t *acc, uint32_t stride, size_t s, unsigned long long &a,
                                            unsigned long long &b, uint32_t expected, uint32_t sum_bits)
{
    if (expected == 1) return true;
    Acc *sa = reinterpret_cast<Acc *>(acc + (2 * s) * stride);
    Acc *sb = reinterpret_cast<Acc *>(acc + (2 * s + 1) * stride);
    const unsigned long long rb = __hip_atomic_fetch_add(&sb->sum, b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (sum_bits) {
        asm volatile("s_waitcnt vmcnt(0)" ::"v"(uint32_t(rb)) : "memory");
        const unsigned long long one = 1ull << sum_bits;
        const unsigned long long before = __hip_atomic_fetch_add(&sa->sum, one + a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if ((before >> sum_bits) != expected - 1) return false;
        __hip_atomic_store(&sa->sum, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        a = (before + a) & (one - 1);
        b = __hip_atomic_exchange(&sb->sum, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return true;
    }
    const unsigned long long ra = __hip_atomic_fetch_add(&sa->sum, a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::"v"(uint32_t(ra)), "v"(uint32_t(rb)) : "memory");
    const uint32_t ticket = __hip_atomic_fetch_add(&sa->cnt, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (ticket != expected - 1) return false;
    a = __hip_atomic_exchange(&sa->sum, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    b = __hip_atomic_exchange(&sb->sum, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&sa->cnt, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return true;
}

// MODE says what the workgroup that completes a chunk does with the two sums:
//   SUMS   out = uint64[2C]: writes the pair.
//   SEAL   out = C tags: writes the chunk's 64-byte tag (hxt_chunk_tag_t) at its packed-slot index.
//   VERIFY out = uint32[C + 1], tags = C tags: compares the tag found at the chunk's slot with the
//          receiver's own layout, the expected message identity and the recomputed sums, and
//          writes the bit mask to out[chunk].
enum Sum2Mode { SUM2_SUMS = 0, SUM2_SEAL = 1, SUM2_VERIFY = 2 };

struct TagWork {
    const uint8_t *tags;     // VERIFY: the received tags
    uint64_t seq;            // SEAL: value to write; VERIFY: value expected
    uint32_t micro_batch;
    uint32_t sum_bits;       // see pair_arrive; set by the launch code
};

// The received tag of a workgroup's chunk, loaded by thread 0 when the workgroup starts so that the load's
// latency is long past when (and if) this workgroup turns out to complete the chunk.
struct TagRegs {
    u32x4 r[4];
};

__device__ __forceinline__ uint64_t tag_place(const ChunkGeom &g, uint32_t c)     // packed offset of chunk c / B
{
    const uint32_t slot = fast_div(c, g.div_k), lane = c - slot * g.k;
    return uint64_t(lane) * g.q + (lane < g.r ? lane : g.r) + slot;
}

__device__ __forceinline__ TagRegs load_tag(const ChunkGeom &g, uint32_t chunk, const TagWork &w)
{
    TagRegs t{};
    if (!w.tags) return t;                               // nothing to compare with: a tag is being written
    const u32x4 *tag = reinterpret_cast<const u32x4 *>(w.tags + tag_place(g, chunk) * 64);
#pragma unroll
    for (int i = 0; i < 4; ++i) t.r[i] = tag[i];
    return t;
}

__device__ __forceinline__ TagRegs prefetch_tag(int mode, const ChunkGeom &g, uint32_t chunk, const TagWork &w)
{
    if (mode == SUM2_VERIFY && threadIdx.x == 0) return load_tag(g, chunk, w);
    return TagRegs{};
}

__device__ __forceinline__ void finish_chunk(int mode, const ChunkGeom &g, uint32_t c, uint64_t sum,
                                             uint64_t wsum, void *out, const TagWork &w, const TagRegs &got,
                                             uint8_t *acc, uint32_t stride, uint32_t fan)
{
    if (mode == SUM2_SUMS) {
        uint64_t *o = static_cast<uint64_t *>(out);
        o[2 * size_t(c)] = sum;
        o[2 * size_t(c) + 1] = wsum;
        return;
    }
    const uint32_t slot = fast_div(c, g.div_k), lane = c - slot * g.k;
    const uint64_t place = tag_place(g, c);
    const uint64_t padded = (c + 1 == g.C) ? g.L - uint64_t(c) * g.B : g.B;
    const u32x4 q0{kTagMagic, c, lane, slot};
    const u32x4 q1{uint32_t(w.seq), uint32_t(w.seq >> 32), w.micro_batch, g.C};
    const u32x4 q2{uint32_t(padded), uint32_t(padded >> 32), uint32_t(sum), uint32_t(sum >> 32)};
    const u32x4 q3{uint32_t(wsum), uint32_t(wsum >> 32), 0u, 0u};
    if (mode == SUM2_SEAL) {
        u32x4 *tag = reinterpret_cast<u32x4 *>(static_cast<uint8_t *>(out) + place * 64);
        tag[0] = q0;
        tag[1] = q1;
        tag[2] = q2;
        tag[3] = q3;
        return;
    }
    const u32x4 r0 = got.r[0], r1 = got.r[1], r2 = got.r[2], r3 = got.r[3];
    uint32_t m = 0;
    if (r0.x != q0.x) m |= HXT_TAG_BAD_MAGIC;
    if (r0.y != q0.y || r0.z != q0.z || r0.w != q0.w || r1.w != q1.w || r2.x != q2.x || r2.y != q2.y) m |= HXT_TAG_BAD_PLACE;
    if (r1.x != q1.x || r1.y != q1.y) m |= HXT_TAG_BAD_SEQ;
    if (r1.z != q1.z) m |= HXT_TAG_BAD_MICRO_BATCH;
    if (r2.z != q2.z || r2.w != q2.w) m |= HXT_TAG_BAD_SUM;
    if (r3.x != q3.x || r3.y != q3.y) m |= HXT_TAG_BAD_WSUM;
    if (r3.z != 0 || r3.w != 0) m |= HXT_TAG_BAD_RESERVED;
    static_cast<uint32_t *>(out)[c] = m;
    // One more slot, after the chunks' own pairs, counts the chunks that are done (upper half of the word)
    // and the rejected ones among them (lower half) with one addition; the chunk that completes the
    // message writes the total to out[C] and clears the slot.
    const unsigned long long mine = (1ull << 32) | (m != 0 ? 1u : 0u);
    unsigned long long total = mine;
    if (g.C > 1) {
        Acc *done = reinterpret_cast<Acc *>(acc + 2 * (size_t(g.C) * (fan + 1)) * stride);
        const unsigned long long before = __hip_atomic_fetch_add(&done->sum, mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (uint32_t(before >> 32) != g.C - 1) return;
        __hip_atomic_store(&done->sum, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        total = before + mine;
    }
    static_cast<uint32_t *>(out)[g.C] = uint32_t(total);
}

// One arrival, made by one thread (as commit_total): the one that completes the chunk finishes it with the received
// tag that tag() returns.
template <class GetTag>
__device__ __forceinline__ void pair_commit_total(int mode, const ChunkGeom &g, uint32_t chunk, uint32_t ordinal, uint32_t expected,
                                                  unsigned long long a, unsigned long long b, void *out, uint8_t *acc,
                                                  uint32_t stride, uint32_t fan, const TagWork &work, GetTag &&tag)
{
    const size_t top = size_t(g.C) * fan + chunk;
    bool last;
    if (fan == 1 || expected < 2 * fan) {
        last = pair_arrive(acc, stride, top, a, b, expected, work.sum_bits);
    } else {
        const uint32_t sub = ordinal & (fan - 1);
        const uint32_t share = expected / fan + (sub < (expected & (fan - 1)) ? 1u : 0u);
        last = pair_arrive(acc, stride, size_t(chunk) * fan + sub, a, b, share, work.sum_bits) &&
               pair_arrive(acc, stride, top, a, b, fan, work.sum_bits);
    }
    if (last) finish_chunk(mode, g, chunk, a, b, out, work, tag(), acc, stride, fan);
}

using PairParts = uint64_t[2][kThreads / 64];          // in LDS

// Workgroup-wide: reduces every thread's (a, b), adds the pair to the chunk's accumulators (two-level
// fan-out as in chunk_commit); the workgroup that completes the chunk finishes it.
__device__ __forceinline__ void pair_commit(int mode, const ChunkGeom &g, const TileSpan &t, unsigned long long a,
                                            unsigned long long b, void *out, uint8_t *acc, uint32_t stride,
                                            uint32_t fan, const TagWork &work, const TagRegs &got, PairParts &part)
{
    for (int o = 32; o > 0; o >>= 1) {
        a += __shfl_down(a, o, 64);
        b += __shfl_down(b, o, 64);
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) {
        part[0][wave] = a;
        part[1][wave] = b;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        a = b = 0;
#pragma unroll
        for (int w = 0; w < kThreads / 64; ++w) {
            a += part[0][w];
            b += part[1][w];
        }
        pair_commit_total(mode, g, t.chunk, t.ordinal, t.expected, a, b, out, acc, stride, fan, work, [&] { return got; });
    }
}

struct Sums2 {
    uint64_t s, w;
};

// A thread's vectors are numbers tid + 256 n (n = 0, 1, ...) of the tile; with S_n the sum of vector n's words and
// I_n = y + 2z + 3w, the tile-local weighted sum is
//   sum (i + 1) w_i = (4 tid + 1) * sum_n S_n + 1024 * sum_n n S_n + sum_n I_n,
// so the loop only adds (as in k_checksum2) and each thread multiplies once at the end.
struct Partial2 {
    uint64_t S, nS, I;
    __device__ __forceinline__ void add(u32x4 r, uint64_t n)
    {
        const uint64_t zw = uint64_t(r.z) + r.w, yzw = zw + r.y, sv = yzw + r.x;
        S += sv;
        nS += n * sv;
        I += yzw + zw + r.w;
    }
};

template <bool UNPACK, bool NTU, bool NTP>
__device__ __forceinline__ Sums2 copy_span2(uint8_t *user, uint8_t *pk, uint32_t bytes)
{
    auto load = [&](uint32_t v) {
        if constexpr (UNPACK) return load16<NTP>(reinterpret_cast<const u32x4 *>(pk) + v);
        else return load16_any<NTU>(user + (size_t(v) << 4));
    };
    auto store = [&](uint32_t v, u32x4 r) {
        if constexpr (UNPACK) store16_any<NTU>(user + (size_t(v) << 4), r);
        else store_packed16<NTP>(reinterpret_cast<u32x4 *>(pk) + v, r);
    };
    const uint32_t nvec = bytes >> 4;
    constexpr uint32_t STEP = kThreads * kUnroll;
    const uint32_t full = nvec / STEP * STEP;
    Partial2 p{0, 0, 0};
    uint64_t n0 = 0;                                     // n of the current block's first vector
    uint32_t v = threadIdx.x;
    for (; v < full; v += STEP, n0 += kUnroll) {
        u32x4 r[kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) r[u] = load(v + u * kThreads);
        uint64_t blockS = 0, blockN = 0, blockI = 0;     // this block's sum_u S_u, sum_u u * S_u, sum_u I_u
#pragma unroll
        for (int u = kUnroll - 1; u >= 0; --u) {
            store(v + u * kThreads, r[u]);
            const uint64_t zw = uint64_t(r[u].z) + r[u].w, yzw = zw + r[u].y;
            blockN += blockS;                            // after the loop: sum_u u * S_u
            blockS += yzw + r[u].x;
            blockI += yzw + zw + r[u].w;
        }
        p.S += blockS;
        p.nS += blockN + n0 * blockS;
        p.I += blockI;
    }
    for (; v < nvec; v += kThreads, ++n0) {
        const u32x4 r = load(v);
        store(v, r);
        p.add(r, n0);
    }
    Sums2 acc{p.S, uint64_t(4 * threadIdx.x + 1) * p.S + 4ull * kThreads * p.nS + p.I};
    const uint32_t tail = bytes & 15;                    // only at the very end of the tensor
    if (threadIdx.x < tail) {
        const uint32_t i = (nvec << 4) + threadIdx.x;
        const uint8_t b = (UNPACK ? pk : user)[i];
        (UNPACK ? user : pk)[i] = b;
        const uint64_t val = uint64_t(b) << (8 * (i & 3));
        acc.s += val;
        acc.w += uint64_t((i >> 2) + 1) * val;
    }
    return acc;
}

// Pad bytes after the tensor's last byte, `first` = their byte position in the tile: pack writes zeros
// (which add nothing to either sum), unpack adds what it finds there.
template <bool UNPACK>
__device__ __forceinline__ Sums2 pad_span2(uint8_t *pk, uint32_t bytes, uint64_t first)
{
    Sums2 acc{0, 0};
    for (uint32_t i = threadIdx.x; i < bytes; i += kThreads) {
        if constexpr (!UNPACK) {
            pk[i] = 0;
        } else {
            const uint64_t pos = first + i;
            const uint64_t val = uint64_t(pk[i]) << (8 * (pos & 3));
            acc.s += val;
            acc.w += uint64_t((pos >> 2) + 1) * val;
        }
    }
    return acc;
}

template <typename E>
__device__ __forceinline__ uint64_t elem_weighted(E v, uint64_t packed_pos)
{
    if constexpr (sizeof(E) == 8) {
        return uint64_t(uint32_t(v)) + uint64_t(uint32_t(uint64_t(v) >> 32));
    } else {
        return uint64_t(v) << (8 * (packed_pos & 3));
    }
}

// ---- what a copy checks on the way ------------------------------------------------
// NONE: nothing.  SUMS: the plain sum of every chunk.  TAGS: both sums, sealed into a tag by a pack and compared with
// the received tag by an unpack, so that tags cost no pass of their own whatever the views of the message.
enum Check { CHECK_NONE = 0, CHECK_SUMS = 1, CHECK_TAGS = 2 };

template <int CHECK>
struct CheckArgs {
    SumCtx cx;
};

template <>
struct CheckArgs<CHECK_TAGS> {
    SumCtx cx;             // the pair-of-sums slots; cx.sums is not used
    ChunkGeom g;
    void *out;             // pack: the message's tags; unpack: its status words
    TagWork work;
};

template <bool UNPACK, int CHECK>
__device__ __forceinline__ TagRegs prefetch_check(const CheckArgs<CHECK> &ck, uint32_t chunk)
{
    if constexpr (CHECK == CHECK_TAGS) return prefetch_tag(UNPACK ? SUM2_VERIFY : SUM2_SEAL, ck.g, chunk, ck.work);
    else return TagRegs{};
}

template <bool UNPACK>
__device__ __forceinline__ void commit_tags(Sums2 v, const Tile &t, const uint32_t *__restrict__ chunk_tiles,
                                            const CheckArgs<CHECK_TAGS> &ck, const TagRegs &got, PairParts &part)
{
    TileSpan span{};
    span.chunk = t.chunk;
    span.ordinal = t.ordinal;
    span.expected = chunk_tiles[t.chunk];
    pair_commit(UNPACK ? SUM2_VERIFY : SUM2_SEAL, ck.g, span, v.s, v.w, ck.out, ck.cx.acc, ck.cx.stride, ck.cx.fan, ck.work, got, part);
}

// Workgroup-wide: the tile's sums (weights counted from the chunk's first word) go to its chunk.
template <bool UNPACK, int CHECK>
__device__ __forceinline__ void commit_tile(Sums2 v, const Tile &t, const uint32_t *__restrict__ chunk_tiles,
                                            const CheckArgs<CHECK> &ck, const TagRegs &got)
{
    if constexpr (CHECK == CHECK_SUMS) chunk_commit(v.s, t.chunk, t.ordinal, chunk_tiles[t.chunk], ck.cx);
    if constexpr (CHECK == CHECK_TAGS) {
        __shared__ PairParts part;
        commit_tags<UNPACK>(v, t, chunk_tiles, ck, got, part);
    }
}

// The pads behind a tensor.  Every table-driven kernel takes them, so that they ride in the launch of the tensor's own
// tiles where the message has no other contiguous piece (see Plan::pads_ride).
template <bool UNPACK, int CHECK>
__device__ __forceinline__ Sums2 pad_tile(const Tile &t, uint8_t *packed)
{
    if constexpr (CHECK == CHECK_TAGS) return pad_span2<UNPACK>(packed + t.packed_off, t.n0, t.a);
    else return Sums2{pad_span<UNPACK, CHECK == CHECK_SUMS>(packed + t.packed_off, t.n0, uint32_t(t.packed_off)), 0};
}

// Adds an element of 8 bytes or less that starts at byte `pos` of a chunk (or of a tile that starts on a word).
template <int CHECK, typename E>
__device__ __forceinline__ void count_elem(Sums2 &acc, E v, uint64_t pos)
{
    if constexpr (CHECK != CHECK_NONE) acc.s += elem_weighted(v, pos);
    if constexpr (CHECK == CHECK_TAGS) {
        const uint64_t j = pos >> 2;
        if constexpr (sizeof(E) == 8) acc.w += (j + 1) * uint32_t(v) + (j + 2) * uint32_t(uint64_t(v) >> 32);
        else acc.w += (j + 1) * (uint64_t(v) << (8 * (pos & 3)));
    }
}

// Adds 16 bytes that start at byte `pos` (a multiple of the element size ES; ES = 16: any vector of the packed side's own) of a chunk.
template <int CHECK, int ES>
__device__ __forceinline__ void count_vector(Sums2 &acc, u32x4 v, uint64_t pos)
{
    if constexpr (CHECK == CHECK_SUMS) {
        acc.s += ES == 16 ? words_sum(v) : rotated_sum(v, uint32_t(pos));
    } else if constexpr (CHECK == CHECK_TAGS) {
        uint32_t w0 = v.x, w1 = v.y, w2 = v.z, w3 = v.w, w4 = 0;
        if constexpr (ES < 4) {                          // a vector that starts inside a word: moved up by its phase, into five words
            const uint32_t down = 32 - 8 * (uint32_t(pos) & 3u);
            w4 = uint32_t(uint64_t(v.w) >> down);
            w3 = uint32_t((uint64_t(v.w) << 32 | v.z) >> down);
            w2 = uint32_t((uint64_t(v.z) << 32 | v.y) >> down);
            w1 = uint32_t((uint64_t(v.y) << 32 | v.x) >> down);
            w0 = uint32_t((uint64_t(v.x) << 32) >> down);
        }
        const uint64_t t4 = w4, t3 = t4 + w3, t2 = t3 + w2, t1 = t2 + w1, s = t1 + w0;
        acc.s += s;
        acc.w += ((pos >> 2) + 1) * s + (t1 + t2) + (t3 + t4);
    }
}

// ---- rows: innermost dimension contiguous, outer dimensions strided -------------
// A 16-byte vector never straddles a run (run length and strides are multiples of 16; the base need not be).
// Logical byte -> (row, column) and row -> outer indices use multiply-shift division.
template <bool UNPACK, int CHECK, bool NTU, bool NTP>
__device__ __forceinline__ Sums2 rows_tile(const Tile &t, const TensorDev &td, uint8_t *user, uint8_t *pk)
{
    const uint32_t row_bytes = td.row_bytes;
    const uint64_t row0 = t.src_off / row_bytes;                    // uniform
    const uint32_t col0 = uint32_t(t.src_off - row0 * row_bytes);
    const int outer = td.ndim - 1;
    const uint32_t nvec = t.n0 >> 4;
    Sums2 acc{0, 0};
    for (uint32_t v0 = threadIdx.x; v0 < nvec; v0 += kThreads * kUnroll) {
        u32x4 r[kUnroll];
        uint64_t off[kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const uint32_t v = v0 + u * kThreads;
            const uint32_t x = col0 + (v << 4);
            const uint32_t dr = fast_div(x, td.row_div);
            uint32_t row = uint32_t(row0) + dr;
            uint64_t o = x - dr * row_bytes;
            for (int d = outer - 1; d > 0; --d) {
                const uint32_t q = fast_div(row, td.dim_div[d]);
                o += uint64_t(row - q * uint32_t(td.shape[d])) * uint64_t(td.stride_b[d]);
                row = q;
            }
            o += uint64_t(row) * uint64_t(td.stride_b[0]);
            off[u] = o;
            if (v < nvec) {
                if constexpr (UNPACK) r[u] = load16<NTP>(reinterpret_cast<const u32x4 *>(pk + (uint64_t(v) << 4)));
                else r[u] = load16_any<NTU>(user + o);
            }
        }
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const uint32_t v = v0 + u * kThreads;
            if (v < nvec) {
                if constexpr (UNPACK) store16_any<NTU>(user + off[u], r[u]);
                else store_packed16<NTP>(reinterpret_cast<u32x4 *>(pk + (uint64_t(v) << 4)), r[u]);
                count_vector<CHECK, 16>(acc, r[u], t.a + (uint64_t(v) << 4));
            }
        }
    }
    return acc;
}

template <bool UNPACK, int CHECK, bool NTU, bool NTP>
__global__ __launch_bounds__(kThreads) void k_rows(const Tile *__restrict__ tiles,
                                                   const uint32_t *__restrict__ chunk_tiles,
                                                   const TensorDev *__restrict__ tensors, uint32_t tensor_base,
                                                   BasePtrs bases, uint8_t *__restrict__ packed, CheckArgs<CHECK> ck)
{
    const Tile t = tiles[blockIdx.x];
    const TagRegs got = prefetch_check<UNPACK, CHECK>(ck, t.chunk);
    const Sums2 acc = t.kind == K_ZERO ? pad_tile<UNPACK, CHECK>(t, packed)
                                       : rows_tile<UNPACK, CHECK, NTU, NTP>(t, tensors[tensor_base + t.tensor], bases.p[t.tensor], packed + t.packed_off);
    commit_tile<UNPACK, CHECK>(acc, t, chunk_tiles, ck, got);
}

// ---- rows whose length or pitch is not a multiple of 16 bytes ----------------------
// Still a gather of contiguous runs (of 16 bytes or more), but a 16-byte vector of the packed stream may end one run and
// begin the next.  A byte finds its run with one multiply-shift division and the run's storage offset from the outer
// indices.
// TWO_D: the view has two dims (the usual padded-pitch matrix) and needs no index decomposition.  Otherwise the outer dims
// are held in registers (the loops store through byte pointers, which may alias the descriptor, so anything read through it
// inside them would be read again every time).
template <bool TWO_D>
struct RunsOf {
    static constexpr int D = TWO_D ? 1 : HXT_MAX_DIMS - 1;          // dims outside the run
    uint32_t shape[D], mul[D], shift[D];
    uint64_t stride[D];
    uint32_t row_bytes, row0, col0;                                 // the tile starts at byte col0 of run row0
    int outer;
    FastDiv row_div;
    __device__ __forceinline__ RunsOf(const Tile &t, const TensorDev &td)
        : row_bytes(td.row_bytes), outer(TWO_D ? 1 : td.ndim - 1), row_div(td.row_div)
    {
        const uint64_t r = t.src_off / row_bytes;                   // uniform
        row0 = uint32_t(r);
        col0 = uint32_t(t.src_off - r * row_bytes);
#pragma unroll
        for (int d = 0; d < D; ++d) {
            shape[d] = 1, mul[d] = 0, shift[d] = 0, stride[d] = 0;
            if (d < outer) {
                shape[d] = uint32_t(td.shape[d]);
                mul[d] = td.dim_div[d].mul;
                shift[d] = td.dim_div[d].shift;
                stride[d] = uint64_t(td.stride_b[d]);
            }
        }
    }
    // Storage offset of run row0 + dr.
    __device__ __forceinline__ uint64_t run(uint32_t dr) const
    {
        uint32_t row = row0 + dr;
        uint64_t o = 0;
#pragma unroll
        for (int d = D - 1; d > 0; --d) {
            if (d < outer) {
                const uint32_t q = fast_div(row, FastDiv{mul[d], shift[d]});
                o += uint64_t(row - q * shape[d]) * stride[d];
                row = q;
            }
        }
        return o + uint64_t(row) * stride[0];
    }
    // Storage offset of byte x of run row0 (x counted on into run row0 + dr, where it lies).
    __device__ __forceinline__ uint64_t place(uint32_t x, uint32_t dr) const
    {
        if constexpr (TWO_D) return uint64_t(row0) * stride[0] + x + uint64_t(dr) * (stride[0] - row_bytes);      // (modulo 2^64)
        else return run(dr) + uint64_t(int64_t(int32_t(x - dr * row_bytes)));
    }
    // Bytes from the first to the last byte of the view.
    __device__ __forceinline__ uint64_t extent() const
    {
        uint64_t e = row_bytes;
#pragma unroll
        for (int d = 0; d < D; ++d) e += uint64_t(shape[d] - 1) * stride[d];
        return e;
    }
};

template <int G> struct PieceOf;
template <> struct PieceOf<8> { using type = uint64_t; };
template <> struct PieceOf<4> { using type = uint32_t; };

// In pieces of G bytes, naturally aligned on both sides, consecutive lanes taking consecutive pieces of the tile: a wave's
// access is contiguous on the packed side and contiguous within each run on the tensor side (64 lanes x 8 bytes = 512 bytes
// per instruction).  Guarded loads are issued without waits here, interleaved with the address arithmetic, and that order
// measures 10 % faster than eight loads in one burst.
template <bool UNPACK, int CHECK, bool NTP, int G, bool TWO_D>
__device__ __forceinline__ Sums2 rows_split_pieces(const Tile &t, const TensorDev &td, uint8_t *user, uint8_t *pk)
{
    using P = typename PieceOf<G>::type;
    const RunsOf<TWO_D> runs(t, td);
    const uint32_t npiece = t.n0 / G;
    constexpr int U = G == 8 ? 8 : 16;                              // pieces in flight per thread: a 16 KiB tile in one go
    auto user_piece = [&](uint32_t i) {                             // piece i of the tile -> its place in storage
        const uint32_t x = runs.col0 + i * G, dr = fast_div(x, runs.row_div);
        return reinterpret_cast<P *>(user + runs.place(x, dr));
    };
    P *pieces = reinterpret_cast<P *>(pk);
    Sums2 acc{0, 0};
    for (uint32_t i0 = threadIdx.x; i0 < npiece; i0 += kThreads * U) {
        P r[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t i = i0 + u * kThreads;
            r[u] = 0;
            if (i < npiece) {
                if constexpr (UNPACK) r[u] = load_elem<NTP>(pieces + i);
                else r[u] = __builtin_nontemporal_load(user_piece(i));
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t i = i0 + u * kThreads;
            if (i < npiece) {
                if constexpr (UNPACK) __builtin_nontemporal_store(r[u], user_piece(i));
                else store_packed_elem<NTP>(pieces + i, r[u]);
                count_elem<CHECK>(acc, r[u], t.a + i * G);
            }
        }
    }
    return acc;
}

// In 16-byte vectors.
// Sending, a vector of the packed side that ends one run and begins the next is put together from two loads, one where it
// would lie if its first run went on and one where it would lie if its second run had begun earlier.  Both stay within the
// view's extent unless the second run lies below the first one (or over it) in storage; the loads are then taken from within
// the runs and shifted.
// Receiving, every run (the part of it that is in this tile) gets as many lanes as it has vectors begun (RunLanes); the last of
// them ends with the run, so that it stores some bytes a second time, with the same values, and a wave's store covers every run
// whole: each burst of the tensor side is written once, which counts as much as the width (stored with their last pieces
// apart, 32 MiB of rows of 37 elements took 109 us instead of 27).  Only what a tile holds of its first or last run can be
// shorter than a vector and goes byte by byte.
// Rows of bf16 at odd pitches, 32 MiB, pack / unpack, in pieces of 2 bytes against vectors (tensors of three messages in
// turn): 37 elements 18.8 / 36.8 -> 18.9 / 24.8 us, 101 elements 17.3 / 24.2 -> 16.1 / 18.5, 1003 elements 17.3 / 19.3 ->
// 15.4 / 14.8.  Pieces of 4 bytes: 101 f32 15.0 / 18.2 against 16.0 / 15.7, 102 bf16 unpack 21.2 against 18.6 (8 MiB 6.4 and
// 6.5; short runs lose at small sizes, 5 f32 8 MiB 8.4 and 9.1, 9 f32 7.8 and 8.2, and gain from there on, 32 MiB 30.6 and 28.6, 27.2
// and 24.7); of 8 bytes: 100 bf16 15.1 / 17.2 against 16.1 / 18.8: sending, pieces of 4 and 8 bytes are the faster ones, receiving,
// those of 8.  Rows much longer than a tile, 66 MB of bf16 at odd pitches, unpack in pieces of 2 bytes against vectors: 50257
// elements 29.6 -> 23.6 us, 151643 30.4 -> 23.6, a million 30.2 -> 23.0 (with tags 36.6 -> 25.3, 36.2 -> 25.5, 36.7 -> 24.9).
template <bool UNPACK, int CHECK, bool NTP, bool TWO_D>
__device__ __forceinline__ Sums2 rows_split_vectors(const Tile &t, const TensorDev &td, uint8_t *user, uint8_t *pk)
{
    const RunsOf<TWO_D> runs(t, td);
    const uint32_t rb = runs.row_bytes, n = t.n0;
    Sums2 acc{0, 0};
    constexpr uint32_t U = UNPACK ? RunLanes::PER_THREAD : kUnroll;
    auto byte = [&](uint32_t i) {                                   // byte i of the tile alone
        const uint32_t x = runs.col0 + i, dr = fast_div(x, runs.row_div);
        uint8_t *at = user + runs.place(x, dr);
        const uint8_t v = UNPACK ? pk[i] : *at;
        if constexpr (UNPACK) *at = v;
        else pk[i] = v;
        count_elem<CHECK>(acc, v, t.a + i);
    };
    if constexpr (!UNPACK) {
        const uint32_t nvec = n >> 4;
        const uint64_t extent = runs.extent();
        for (uint32_t v0 = threadIdx.x; v0 < nvec; v0 += kThreads * U) {
            u32x4 r[U], s[U];
            uint32_t k[U];
            bool apart[U];
#pragma unroll
            for (uint32_t u = 0; u < U; ++u) {
                const uint32_t x = runs.col0 + (min(v0 + u * kThreads, nvec - 1) << 4);
                const uint32_t dr = fast_div(x, runs.row_div);
                uint64_t o = runs.place(x, dr);
                k[u] = rb - (x - dr * rb);                                      // bytes of the run from here on
                s[u] = u32x4{0, 0, 0, 0};
                apart[u] = false;
                if (k[u] < 16) {
                    uint64_t o2 = runs.place(x, dr + 1);                 // (below run dr + 1 by k)
                    apart[u] = o + 16 > extent || int64_t(o2) < 0;
                    if (apart[u]) o -= 16 - k[u], o2 += k[u];       // the run's last bytes, the next one's first
                    s[u] = load16_any<true>(user + o2);
                }
                r[u] = load16_any<true>(user + o);
            }
#pragma unroll
            for (uint32_t u = 0; u < U; ++u) {
                const uint32_t v = v0 + u * kThreads;
                if (v < nvec) {
                    if (apart[u]) {
                        r[u] = shift_bytes_down(r[u], 16 - k[u]);
                        s[u] = shift_bytes_up(s[u], k[u]);
                    }
                    const u32x4 w = k[u] < 16 ? keep_bytes(r[u], 0, k[u]) | keep_bytes(s[u], k[u], 16) : r[u];
                    store_packed16<NTP>(reinterpret_cast<u32x4 *>(pk) + v, w);
                    count_vector<CHECK, 16>(acc, w, t.a + (uint64_t(v) << 4));
                }
            }
        }
        if (threadIdx.x < (n & 15u)) byte((nvec << 4) + threadIdx.x);            // only at the very end of the tensor
    } else {
        const uint32_t last = fast_div(runs.col0 + n - 1, runs.row_div);         // the tile meets runs row0 .. row0 + last
        const RunLanes deal(rb, runs.col0, n, last + 1, td.lane_div);
        for (uint32_t i0 = threadIdx.x; i0 < deal.all; i0 += kThreads * U) {
            u32x4 r[U];
            uint32_t at[U], skip[U];
            uint8_t *to[U];
#pragma unroll
            for (uint32_t u = 0; u < U; ++u) {
                const uint32_t i = i0 + u * kThreads;
                const RunLanes::Lane l = deal.lane(min(i, deal.all - 1));
                at[u] = l.at;
                skip[u] = i < deal.all ? l.skip : 16;
                to[u] = user + runs.place(at[u] + runs.col0, l.dr);
                r[u] = load16_any<NTP>(pk + at[u]);
            }
#pragma unroll
            for (uint32_t u = 0; u < U; ++u)
                if (skip[u] < 16) {
                    store16_any<true>(to[u], r[u]);
                    count_vector<CHECK, 1>(acc, keep_bytes(r[u], skip[u], 16), t.a + at[u]);
                }
        }
        auto piece = [&](uint32_t lo, uint32_t hi) {
            if (hi - lo < 16 && threadIdx.x < hi - lo) byte(lo + threadIdx.x);
        };
        piece(0, min(rb - runs.col0, n));
        if (last) piece(last * rb - runs.col0, n);
    }
    return acc;
}

// Whether a tensor goes in pieces: low is its base address and TensorDev::low_or ORed.
template <bool UNPACK>
HXT_HD bool in_pieces(uint32_t low) { return (low & (UNPACK ? 7u : 3u)) == 0; }

template <bool UNPACK, int CHECK, bool NTP, bool PIECES_LIKELY, bool ALL_PIECES = false>
__device__ __forceinline__ Sums2 rows_split_any(const Tile &t, const TensorDev &td, uint8_t *user, uint8_t *pk)
{
    // widest piece that is naturally aligned everywhere: low bits of the base address, the run length and the pitches
    const uint32_t low = (uint32_t(reinterpret_cast<uintptr_t>(user)) | td.low_or) & 7u;
    auto pieces = [&]<int G>() {
        return td.ndim == 2 ? rows_split_pieces<UNPACK, CHECK, NTP, G, true>(t, td, user, pk)
                            : rows_split_pieces<UNPACK, CHECK, NTP, G, false>(t, td, user, pk);
    };
    if constexpr (ALL_PIECES && UNPACK) return pieces.template operator()<8>();
    if (PIECES_LIKELY ? __builtin_expect(low == 0, 1) : low == 0) return pieces.template operator()<8>();
    if constexpr (ALL_PIECES) return pieces.template operator()<4>();
    if constexpr (!UNPACK)
        if (in_pieces<UNPACK>(low)) return pieces.template operator()<4>();
    return td.ndim == 2 ? rows_split_vectors<UNPACK, CHECK, NTP, true>(t, td, user, pk)
                        : rows_split_vectors<UNPACK, CHECK, NTP, false>(t, td, user, pk);
}

// ALL_PIECES: every tensor of the launch goes in pieces.  (A kernel of their own, as the code of the vectors beside them slows
// them down: rows of 200 bytes, 8 MB, pack / unpack, 6.00 / 6.18 -> 5.81 / 5.95 us; with tags 16 MB 10.37 / 12.68 -> 9.97 /
// 12.41; in three dims 4 MB 5.54 / 6.03 -> 5.41 / 5.56.)
template <bool UNPACK, int CHECK, bool NTP, bool ALL_PIECES>
__global__ __launch_bounds__(kThreads) void k_rows_split(const Tile *__restrict__ tiles,
                                                         const uint32_t *__restrict__ chunk_tiles,
                                                         const TensorDev *__restrict__ tensors, uint32_t tensor_base,
                                                         BasePtrs bases, uint8_t *__restrict__ packed, CheckArgs<CHECK> ck)
{
    const Tile t = tiles[blockIdx.x];
    const TagRegs got = prefetch_check<UNPACK, CHECK>(ck, t.chunk);
    const Sums2 acc = t.kind == K_ZERO ? pad_tile<UNPACK, CHECK>(t, packed) : rows_split_any<UNPACK, CHECK, NTP, false, ALL_PIECES>(t, tensors[tensor_base + t.tensor], bases.p[t.tensor], packed + t.packed_off);
    commit_tile<UNPACK, CHECK>(acc, t, chunk_tiles, ck, got);
}

// ---- transpose: logical inner dimension strided, the one before it contiguous ----
// A tile is ni x nj elements (at most T x T: 128 x 128 for 1- and 2-byte elements, 64 x 64 otherwise).  The tensor
// stores nj rows of ni contiguous elements, the packed stream has ni rows of nj.  A thread loads a block of V x V
// elements (V = 16 bytes' worth: V rows of one vector each), transposes it in registers and leaves V vectors in LDS;
// after the barrier the tile's rows leave LDS as whole vectors, 16 lanes (256 contiguous bytes) to a row.  So LDS is
// touched by 16-byte accesses only, once each way; gathering elements out of it instead kept the LDS pipe busy for
// about 1.7 us of a 14 us launch (64 two-byte reads per thread).  32 MiB of bf16, pack + unpack, new tensors through two
// packed buffers: 28.4 -> 26.8 us (a plain copy of the same bytes: 26.2); the gain is all on the sending side.
// Vectors need no alignment beyond the element's: the hardware takes misaligned 16-byte accesses, and even with both
// row pitches odd (bf16, pitches of 8198 bytes) they beat element accesses, 30 against 31-38 us per pair.
template <typename E>
struct TransposeShape {
    static constexpr uint32_t T = transpose_tile(sizeof(E)), V = 16 / sizeof(E);
    static constexpr uint32_t NB = T / V;                        // vectors per tile row
    // Source rows of a thread's block: as many as a vector has elements, so that LDS takes whole vectors.  Not for bytes:
    // 64 such blocks make up a tile, three waves of four would have none and the fourth all the sums to take; a block is 4
    // rows, LDS takes words.  32 MiB of bytes, receiving: 13.8 -> 11.9 us, with tags 25.3 -> 14.0, across chunks 22.2 -> 14.5.
    static constexpr uint32_t R = sizeof(E) == 1 ? 4 : V;
    static constexpr uint32_t BLOCKS = NB * (T / R);
};

// x[r] holds V elements of source row r; afterwards x[c] holds the V elements of source column c (bytes: word c & 3 of
// x[c / 4] holds the 4 elements of source column c).
template <typename E>
__device__ __forceinline__ void transpose_block(u32x4 (&x)[TransposeShape<E>::R])
{
    constexpr int V = TransposeShape<E>::R;
    u32x4 y[V];
    if constexpr (sizeof(E) == 8) {
        y[0] = u32x4{x[0].x, x[0].y, x[1].x, x[1].y};
        y[1] = u32x4{x[0].z, x[0].w, x[1].z, x[1].w};
    } else if constexpr (sizeof(E) == 4) {
#pragma unroll
        for (int c = 0; c < 4; ++c) y[c] = u32x4{x[0][c], x[1][c], x[2][c], x[3][c]};
    } else if constexpr (sizeof(E) == 2) {
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t a = x[2 * q][c], b = x[2 * q + 1][c];
                y[2 * c][q] = __builtin_amdgcn_perm(b, a, 0x05040100u);
                y[2 * c + 1][q] = __builtin_amdgcn_perm(b, a, 0x07060302u);
            }
    } else {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const uint32_t lo01 = __builtin_amdgcn_perm(x[1][c], x[0][c], 0x05010400u);       // bytes 0 0' 1 1'
            const uint32_t hi01 = __builtin_amdgcn_perm(x[1][c], x[0][c], 0x07030602u);       // bytes 2 2' 3 3'
            const uint32_t lo23 = __builtin_amdgcn_perm(x[3][c], x[2][c], 0x05010400u);
            const uint32_t hi23 = __builtin_amdgcn_perm(x[3][c], x[2][c], 0x07030602u);
            y[c] = u32x4{__builtin_amdgcn_perm(lo23, lo01, 0x05040100u), __builtin_amdgcn_perm(lo23, lo01, 0x07060302u),
                         __builtin_amdgcn_perm(hi23, hi01, 0x05040100u), __builtin_amdgcn_perm(hi23, hi01, 0x07060302u)};
        }
    }
#pragma unroll
    for (int i = 0; i < V; ++i) x[i] = y[i];
}

// Where the rows of a tile lie on the packed side.
// PitchRows: a tile inside one chunk, rows a fixed pitch apart, one sum for the tile.
struct PitchRows {
    static constexpr bool kSpan = false;
    uint8_t *base;                 // element (0, 0) of the tile
    uint64_t pitch;
    uint64_t pos;                  // its position in the chunk (for the weights of sums)
    __device__ __forceinline__ uint8_t *at(uint32_t row, uint32_t byte) const { return base + row * pitch + byte; }
    template <int CHECK>
    __device__ __forceinline__ uint64_t position(uint32_t row, uint32_t byte) const
    {
        if constexpr (CHECK == CHECK_SUMS) return uint32_t(pos) + row * uint32_t(pitch) + byte;
        return pos + row * pitch + byte;
    }
};
// SpanRows: every row placed on its own (k_transpose_span keeps the placement in LDS): bytes below first[row] lie from
// p0[row] on in the packed buffer, the rest at p1[row]; sums go to the partial sum of the chunk they fall into.
struct SpanRows {
    static constexpr bool kSpan = true;
    uint8_t *packed;
    const uint64_t *p0, *p1;
    const uint16_t *first, *entry;
    const uint64_t *rem;           // position of the row's first byte in its chunk
    unsigned long long *part, *wpart;
    bool may_cross;                // a vector may straddle a chunk border (rows are not 16-byte aligned against it)
    __device__ __forceinline__ uint8_t *at(uint32_t row, uint32_t byte) const
    {
        return packed + (byte < first[row] ? p0[row] : p1[row]) + byte;
    }
    // (chunks are multiples of 256 bytes, so the phase in a word, all that plain sums ask for, is the same on both sides)
    template <int CHECK>
    __device__ __forceinline__ uint64_t position(uint32_t row, uint32_t byte) const
    {
        if constexpr (CHECK == CHECK_SUMS) return uint32_t(rem[row]) + byte;
        return byte < first[row] ? rem[row] + byte : byte - first[row];
    }
    __device__ __forceinline__ bool crosses(uint32_t row, uint32_t byte) const
    {
        return may_cross && byte < first[row] && byte + 16 > first[row];
    }
    template <int CHECK>
    __device__ __forceinline__ void count(uint32_t row, bool second, Sums2 v) const
    {
        const uint32_t at = entry[row] + (second ? 1u : 0u);
        __hip_atomic_fetch_add(&part[at], (unsigned long long)v.s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if constexpr (CHECK == CHECK_TAGS)
            __hip_atomic_fetch_add(&wpart[at], (unsigned long long)v.w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
};

// The elements of a vector on the packed side that straddles a chunk border (bytes below `first` of the row lie from
// `before` on, the rest from `after` on), one at a time.
template <typename E, bool NTP>
__device__ __forceinline__ void store_crossing(uint8_t *before, uint8_t *after, uint32_t first, uint32_t byte, uint32_t n, u32x4 v)
{
    constexpr uint32_t ES = sizeof(E);
#pragma unroll
    for (uint32_t q = 0; q < 16 / ES; ++q) {
        const uint32_t at = byte + q * ES;
        const E e = E(ES == 8 ? uint64_t(v[q * ES / 4]) | uint64_t(v[(q * ES / 4 + 1) & 3]) << 32 : uint64_t(v[q * ES / 4]) >> (8 * (q * ES & 3)));
        if (q < n) store_packed_elem<NTP>(reinterpret_cast<E *>((at < first ? before : after) + at), e);
    }
}

template <typename E>
__device__ __forceinline__ u32x4 load_crossing(const uint8_t *before, const uint8_t *after, uint32_t first, uint32_t byte)
{
    union {
        E e[16 / sizeof(E)];
        u32x4 x;
    } o;
#pragma unroll
    for (uint32_t q = 0; q < 16 / sizeof(E); ++q) {
        const uint32_t at = byte + q * uint32_t(sizeof(E));
        o.e[q] = *reinterpret_cast<const E *>((at < first ? before : after) + at);
    }
    return o.x;
}

// Adds the sum of a vector of packed bytes (n of them from byte `skip` on count) to the tile's sum, or to the partial sum
// of its chunk.  SpanRows: called by all lanes of a wave, 16 lanes next to each other (8 for bytes) holding
// vectors of one tile row (live: this lane's vector counts); the row is summed across those lanes first, so that one lane
// goes to LDS.
template <typename E, int CHECK, class Rows>
__device__ __forceinline__ void count_packed(const Rows &rows, uint32_t row, uint32_t byte, u32x4 v, uint32_t skip, uint32_t n,
                                             bool live, Sums2 &acc)
{
    const u32x4 kept = live ? keep_bytes(v, skip, n) : u32x4{0, 0, 0, 0};
    if constexpr (!Rows::kSpan) {
        count_vector<CHECK, sizeof(E)>(acc, kept, rows.template position<CHECK>(row, byte));
    } else {
        const uint32_t border = rows.first[row];
        const bool crossing = rows.crosses(row, byte);
        if (crossing && live) {                          // split at the border: rare, and only where rows are misaligned
            const uint32_t before = border - byte;
            Sums2 ahead{0, 0}, behind{0, 0};
            count_vector<CHECK, sizeof(E)>(ahead, keep_bytes(kept, 0, before), rows.template position<CHECK>(row, byte));
            // (the bytes behind the border start the next chunk: weights counted from its first word)
#pragma unroll
            for (uint32_t q = 0; q < 16 / sizeof(E); ++q) {
                const uint32_t at = q * uint32_t(sizeof(E));
                const E e = E(sizeof(E) == 8 ? uint64_t(kept[at / 4]) | uint64_t(kept[(at / 4 + 1) & 3]) << 32 : uint64_t(kept[at / 4]) >> (8 * (at & 3)));
                if (at >= before) count_elem<CHECK>(behind, e, uint64_t(at - before));
            }
            rows.template count<CHECK>(row, false, ahead);
            rows.template count<CHECK>(row, true, behind);
        }
        Sums2 v2{0, 0};
        if (!crossing) count_vector<CHECK, sizeof(E)>(v2, kept, rows.template position<CHECK>(row, byte));
        constexpr uint32_t LANES = TransposeShape<E>::NB < 16 ? TransposeShape<E>::NB : 16;     // of a DPP row that hold one tile row
        const bool whole = border >= TransposeShape<E>::T * uint32_t(sizeof(E));     // the row meets no border in this tile
        Sums2 total{lanes_sum<LANES>(v2.s), 0};
        if constexpr (CHECK == CHECK_TAGS) total.w = lanes_sum<LANES>(v2.w);
        if (whole && (threadIdx.x & (LANES - 1)) == LANES - 1) rows.template count<CHECK>(row, false, total);
        if (!whole && v2.s) rows.template count<CHECK>(row, byte >= border, v2);
    }
}

// Moves one tile.  Source rows are the tensor's (pack) or the packed side's (unpack): nb rows of na elements.
// place() puts into LDS what `rows` reads there; a pack does that while its loads from the tensor are on their way.
// fetch() asks for what the caller needs at the end.
template <typename E, bool UNPACK, int CHECK, bool NTU, bool NTP, bool FULL, class Rows, class Place, class Fetch>
__device__ __forceinline__ Sums2 transpose_tile_vectors(uint8_t *user, uint64_t user_pitch, uint32_t na_in, uint32_t nb_in,
                                                           const Rows &rows, u32x4 *lds, Place &&place, Fetch &&fetch)
{
    using Sh = TransposeShape<E>;
    constexpr uint32_t T = Sh::T, V = Sh::V, R = Sh::R, NB = Sh::NB, ES = sizeof(E);
    constexpr uint32_t PER = Sh::BLOCKS < uint32_t(kThreads) ? 1 : Sh::BLOCKS / kThreads;      // blocks per thread
    const uint32_t na = FULL ? T : na_in, nb = FULL ? T : nb_in;
    auto slot_of = [](uint32_t row, uint32_t slot) { return row * NB + (slot ^ ((row / V) & (NB - 1))); };
    Sums2 acc{0, 0};
    if constexpr (Rows::kSpan && UNPACK) {
        place();
        __syncthreads();
    }
#pragma unroll
    for (uint32_t k = 0; k < PER; ++k) {
        const uint32_t id = threadIdx.x + k * kThreads, la = id & (NB - 1), lb = id / NB;
        const uint32_t a0 = la * V, b0 = lb * R;
        constexpr bool kAll = FULL && Sh::BLOCKS >= uint32_t(kThreads);      // every thread has a whole block
        const bool live = kAll || (id < Sh::BLOCKS && a0 < na && b0 < nb);
        auto row_of = [&](uint32_t r) { return kAll ? b0 + r : min(b0 + r, nb - 1); };
        // The last block of a row that is no multiple of V starts early enough to end with it (its first columns are
        // then moved twice, with the same values); rows beyond the tile repeat the last one.
        const uint32_t as = FULL || a0 + V <= na ? a0 : (na >= V ? na - V : 0);
        const bool narrow = !FULL && na < V;
        u32x4 x[R];
        if (live && !narrow) {
#pragma unroll
            for (uint32_t r = 0; r < R; ++r) {
                const uint32_t b = row_of(r);
                if constexpr (!UNPACK) {
                    x[r] = load16_any<NTU>(user + b * user_pitch + as * ES);
                } else if constexpr (!Rows::kSpan) {
                    x[r] = load16_any<NTP>(rows.at(b, as * ES));
                } else {
                    // (a vector across a chunk border is read from the 16 bytes that end there, and put right below)
                    const uint32_t byte = rows.crosses(b, as * ES) ? rows.first[b] - 16u : as * ES;
                    x[r] = load16_any<NTP>(rows.packed + (as * ES < rows.first[b] ? rows.p0[b] : rows.p1[b]) + int32_t(byte));
                }
            }
            if constexpr (UNPACK && Rows::kSpan) {
                if (rows.may_cross)
#pragma unroll
                    for (uint32_t r = 0; r < R; ++r) {
                        const uint32_t b = row_of(r);
                        if (rows.crosses(b, as * ES)) x[r] = load_crossing<E>(rows.packed + rows.p0[b], rows.packed + rows.p1[b], rows.first[b], as * ES);
                    }
            }
        } else if (live) {                               // fewer than V columns in the whole tile
#pragma unroll
            for (uint32_t r = 0; r < R; ++r) {
                const uint32_t b = row_of(r);
                union {
                    E e[V];
                    u32x4 v;
                } o{};
#pragma unroll
                for (uint32_t q = 0; q < V; ++q)
                    if (q < na) {
                        if constexpr (!UNPACK) o.e[q] = *reinterpret_cast<const E *>(user + b * user_pitch + q * ES);
                        else o.e[q] = *reinterpret_cast<const E *>(rows.at(b, q * ES));
                    }
                x[r] = o.v;
            }
        }
        if constexpr (CHECK != CHECK_NONE && UNPACK) {
            const uint32_t skip = (a0 - as) * ES, n = narrow ? na * ES : 16;
#pragma unroll
            for (uint32_t r = 0; r < R; ++r)
                count_packed<E, CHECK>(rows, row_of(r), as * ES, x[r], FULL ? 0 : skip, FULL ? 16 : n,
                                live && (kAll || b0 + r < nb), acc);
        }
        if (k == 0) {
            if constexpr (!UNPACK) place();
            fetch();
        }
        if (live) {
            transpose_block<E>(x);
#pragma unroll
            for (uint32_t c = 0; c < V; ++c)
                if (!narrow || c < na) {
                    if constexpr (R == V) lds[slot_of(as + c, lb)] = x[c];
                    else reinterpret_cast<uint32_t *>(lds + slot_of(as + c, lb / (V / R)))[lb % (V / R)] = x[c / R][c % R];
                }
        }
    }
    __syncthreads();
    // Receiving, rows that do not start on 16 bytes are left in the cache: non-temporal, the bursts they share with their
    // neighbours go out in parts.  A base one element off, 32 MiB: bytes 27.2 -> 13.7 us, two bytes 16.6 -> 13.0, four
    // 17.7 -> 12.1, across chunks 30 -> 17.4, 22.8 -> 16.0, 22.5 -> 14.9; 96 MiB of bytes 110 -> 71.  Not in launches of up
    // to 24 MiB of wider elements, which would have it all to write back at their end (two bytes, 8 MiB 5.0 against 5.7 us,
    // 12 MiB 8.9 against 11.8; 24 MiB even; bytes, 8 MiB 6.6 against 5.8), and not of eight bytes, whose rows of 512 bytes
    // have few such bursts (96 MiB across chunks 54.6 against 57.1).
    const bool large = ES == 1 || (ES < 8 && uint64_t(gridDim.x) * (T * T * ES) > (24u << 20));
    const bool cached = large && ((uint32_t(reinterpret_cast<uintptr_t>(user)) | uint32_t(user_pitch)) & 15u) != 0;
#pragma unroll
    for (uint32_t k = 0; k < T * NB / kThreads; ++k) {
        const uint32_t id = threadIdx.x + k * kThreads, row = id / NB, slot = id & (NB - 1);
        const bool live = FULL || (row < na && slot * V < nb);
        const uint32_t r = FULL ? row : min(row, na - 1), n = FULL ? V : min(V, nb - min(slot * V, nb));
        const u32x4 v = lds[slot_of(r, slot)];
        if constexpr (CHECK != CHECK_NONE && !UNPACK) count_packed<E, CHECK>(rows, r, slot * 16, v, 0, n * ES, live, acc);
        if (!live) continue;
        if constexpr (UNPACK) {
            uint8_t *to = user + r * user_pitch + slot * 16;
            if (!(FULL || n == V)) store_elems<E>(to, v, n);
            else if (cached) store16_cached(to, v);
            else store16_any<true>(to, v);
        } else if constexpr (!Rows::kSpan) {
            uint8_t *to = rows.at(r, slot * 16);
            if (FULL || n == V) store_packed16<NTP>(reinterpret_cast<u32x4 *>(to), v);
            else store_elems<E>(to, v, n);
        } else {
            if ((FULL || n == V) && !rows.crosses(r, slot * 16)) store_packed16<NTP>(reinterpret_cast<u32x4 *>(rows.at(r, slot * 16)), v);
            else store_crossing<E, NTP>(rows.packed + rows.p0[r], rows.packed + rows.p1[r], rows.first[r], slot * 16, n, v);
        }
    }
    return acc;
}

// The tensor's fast direction has a stride of a few elements (es bytes from element to element): element by element,
// through an LDS tile padded by one element.  Thread (tx, ty) holds elements of packed row tx only while it is on the
// tensor side and sums them there: sum(row, v, j) for element j of its row.  Eight global loads per thread are issued
// before the first of them is needed (row and column numbers are clamped into the tile, so the loads need no guard).
template <typename E, bool UNPACK, bool NTP, class Rows, class Sum>
__device__ __forceinline__ void transpose_tile_elements(uint8_t *user, uint64_t user_pitch, uint32_t es, uint32_t ni, uint32_t nj,
                                                        const Rows &rows, uint8_t *lds_raw, Sum &&sum)
{
    constexpr uint32_t T = TransposeShape<E>::T, TY = kThreads / T, U = 8;
    E(*lds)[T + 1] = reinterpret_cast<E(*)[T + 1]>(lds_raw);
    const uint32_t tx = threadIdx.x & (T - 1), ty = threadIdx.x / T;
    auto tensor_side = [&]() {
        if (tx >= ni) return;
        for (uint32_t j0 = ty; j0 < nj; j0 += TY * U) {
            E v[U];
#pragma unroll
            for (uint32_t u = 0; u < U; ++u) {
                const uint32_t j = min(j0 + u * TY, nj - 1);
                if constexpr (!UNPACK) v[u] = __builtin_nontemporal_load(reinterpret_cast<const E *>(user + j * user_pitch + tx * es));
                else v[u] = lds[j][tx];
            }
#pragma unroll
            for (uint32_t u = 0; u < U; ++u) {
                const uint32_t j = j0 + u * TY;
                if (j < nj) {
                    if constexpr (!UNPACK) lds[j][tx] = v[u];
                    else __builtin_nontemporal_store(v[u], reinterpret_cast<E *>(user + j * user_pitch + tx * es));
                    sum(tx, v[u], j);
                }
            }
        }
    };
    auto packed_side = [&]() {
        const uint32_t txc = min(tx, nj - 1);
        for (uint32_t i0 = ty; i0 < ni; i0 += TY * U) {
            E *p[U];
            E v[U];
#pragma unroll
            for (uint32_t u = 0; u < U; ++u) {
                p[u] = reinterpret_cast<E *>(rows.at(min(i0 + u * TY, ni - 1), txc * uint32_t(sizeof(E))));
                if constexpr (UNPACK) v[u] = load_elem<NTP>(p[u]);
            }
#pragma unroll
            for (uint32_t u = 0; u < U; ++u) {
                const uint32_t i = i0 + u * TY;
                if (i < ni && tx < nj) {
                    if constexpr (UNPACK) lds[tx][i] = v[u];
                    else store_packed_elem<NTP>(p[u], lds[tx][i]);
                }
            }
        }
    };
    if constexpr (!UNPACK) {
        tensor_side();
        __syncthreads();
        packed_side();
    } else {
        packed_side();
        __syncthreads();
        tensor_side();
    }
}

template <typename E>
constexpr uint32_t transpose_lds_bytes() { return TransposeShape<E>::T * (TransposeShape<E>::T + 1) * sizeof(E); }

template <typename E, bool UNPACK, int CHECK, bool NTU, bool NTP>
__device__ __forceinline__ Sums2 transpose_any(const Tile &t, uint8_t *base, uint8_t *packed, const CheckArgs<CHECK> &ck, uint8_t *lds_raw)
{
    constexpr uint32_t T = TransposeShape<E>::T;
    uint8_t *user = base + t.src_off;
    const uint32_t ni = t.n0, nj = t.n1;
    uint64_t in_chunk = t.packed_off & 255u;           // plain sums only need the position within a word
    if constexpr (CHECK == CHECK_TAGS) in_chunk = t.packed_off - tag_place(ck.g, t.chunk) * ck.g.B;
    const PitchRows rows{packed + t.packed_off, t.b, in_chunk};
    u32x4 *lds = reinterpret_cast<u32x4 *>(lds_raw);
    const uint32_t na = UNPACK ? nj : ni, nb = UNPACK ? ni : nj;
    Sums2 acc{0, 0};
    if (t.estep != sizeof(E))
        transpose_tile_elements<E, UNPACK, NTP>(user, t.a, t.estep, ni, nj, rows, lds_raw, [&](uint32_t i, E v, uint32_t j) {
            count_elem<CHECK>(acc, v, rows.template position<CHECK>(i, j * sizeof(E)));
        });
    else if (ni == T && nj == T)
        acc = transpose_tile_vectors<E, UNPACK, CHECK, NTU, NTP, true>(user, t.a, na, nb, rows, lds, [] {}, [] {});
    else
        acc = transpose_tile_vectors<E, UNPACK, CHECK, NTU, NTP, false>(user, t.a, na, nb, rows, lds, [] {}, [] {});
    return acc;
}

template <typename E, bool UNPACK, int CHECK, bool NTP>
__global__ __launch_bounds__(kThreads) void k_transpose(const Tile *__restrict__ tiles,
                                                        const uint32_t *__restrict__ chunk_tiles, BasePtrs bases,
                                                        uint8_t *__restrict__ packed, CheckArgs<CHECK> ck)
{
    __shared__ __attribute__((aligned(16))) uint8_t lds_raw[transpose_lds_bytes<E>()];
    const Tile t = tiles[blockIdx.x];
    const TagRegs got = prefetch_check<UNPACK, CHECK>(ck, t.chunk);
    const Sums2 acc = t.kind == K_ZERO ? pad_tile<UNPACK, CHECK>(t, packed) : transpose_any<E, UNPACK, CHECK, true, NTP>(t, bases.p[t.tensor], packed, ck, lds_raw);
    commit_tile<UNPACK, CHECK>(acc, t, chunk_tiles, ck, got);
}

// ---- transpose whose tiles span chunks -------------------------------------------
// For matrices whose packed rows are long against the chunk: a tile is a full block of the logical matrix
// (so that every memory burst of the tensor side is used whole) and row i of it starts at stream byte
// s0 + i * b, wherever that falls; a tile row is shorter than a chunk, so it meets at most one chunk
// border.  Thread i places row i (its chunk, the packed address of its first byte, how many of its
// bytes lie before the border and where the rest go) and leaves that in LDS, so that the copy only
// reads it back.  Placing takes no division and no memory access but for rows farther apart than a chunk is long, and
// what the commit at the end reads is loaded at the start.  Sums go to the tile's per-chunk partial sums in LDS; at the
// end one thread per chunk touched makes that chunk's arrival (inc holds the tile's chunks, ascending, and the ordinal
// of each arrival).
// [256, 65536] bf16 (8 packed rows per 1 MiB chunk), pack + unpack: 33.2 -> 27.8 us.

// What k_transpose_span keeps in LDS beside the tile, for tiles of T rows.  Per row: packed offset of byte x is p0 + x for
// x < first, p1 + x from there on (first is a whole tile row or more where the row meets no border); at: entry of the
// row's first chunk; rem: position of its first byte in that chunk (for the weights of the sums).
// A tile's rows meet at most 2 T chunks.  SPARE entries more change nothing but where the rest lies, and no reason is known for
// what that does to transposes with tags (sums do not change): pack + unpack of two bytes, without them against with them, [143,
// 96522] 54.1 and 52.7 us, [500, 33000] 52.3 and 51.7, [256, 65536] 34.6 and 35.2, [4000, 4000] 34.3 and 34.7; of one byte [256,
// 65536] 23.6 and 23.3.  k_transpose_span keeps the layout that it has always had; k_message has no room for them.
template <uint32_t T, int CHECK, uint32_t SPARE = 2>
struct SpanLds {
    static constexpr uint32_t MAXC = 2 * T + SPARE;
    unsigned long long part[MAXC];                      // partial sum per chunk touched
    unsigned long long wpart[CHECK == CHECK_TAGS ? MAXC : 1];       // and the weighted one
    uint64_t p0[T], p1[T], rem[T];
    uint16_t first[T], at[T];                           // (16 bits: four workgroups of bf16 tiles with tags just fit a CU's LDS)
};

template <typename E, bool UNPACK, int CHECK, bool NTU, bool NTP, class Lds>
__device__ __forceinline__ void transpose_span_any(const Tile &t, const uint32_t *__restrict__ chunk_tiles,
                                                   const uint32_t *__restrict__ inc, const ChunkGeom &g, uint8_t *base,
                                                   uint8_t *packed, const CheckArgs<CHECK> &ck, uint8_t *lds_raw, Lds &sp)
{
    constexpr uint32_t T = TransposeShape<E>::T;
    static_assert(T <= kThreads, "one thread places one row");
    uint64_t *const row_p0 = sp.p0, *const row_p1 = sp.p1, *const row_rem = sp.rem;
    uint16_t *const row_first = sp.first, *const row_at = sp.at;
    unsigned long long *const part = sp.part, *const wpart = sp.wpart;
    uint8_t *user = base + t.src_off;
    const uint32_t ni = t.n0, nj = t.n1, n_inc = t.ordinal;
    const uint32_t *my = inc + 2 * size_t(t.chunk);
    uint32_t my_chunk = 0, my_ordinal = 0, my_expected = 0;      // this thread's arrival at the end
    auto fetch = [&]() {                                // asked for behind the tile's own loads, so that it is there then
        if (CHECK == CHECK_NONE || threadIdx.x >= n_inc) return;
        my_chunk = my[2 * threadIdx.x];
        my_ordinal = my[2 * threadIdx.x + 1];
        my_expected = chunk_tiles[my_chunk];
    };
    auto place = [&]() {                                // row threadIdx.x; the partial sums start at zero
        for (uint32_t i = threadIdx.x; i < n_inc; i += kThreads) {
            part[i] = 0;
            if constexpr (CHECK == CHECK_TAGS) wpart[i] = 0;
        }
        if (threadIdx.x >= ni) return;
        const uint64_t B = g.B, s0 = t.packed_off;
        const auto [c, rem] = chunk_at(g, s0 + uint64_t(threadIdx.x) * t.b);
        const uint32_t c0 = chunk_at(g, s0).chunk;
        uint32_t at = c - c0;                           // rows no farther apart than a chunk is long meet every chunk in turn
        if (t.b > B) {                                  // else: look for the entry that names chunk c (it is there)
            uint32_t lo = 0, hi = n_inc - 1;
            while (lo < hi) {
                const uint32_t mid = (lo + hi) / 2;
                if (my[2 * mid] < c) lo = mid + 1;
                else hi = mid;
            }
            at = lo;
        }
        auto chunk_base = [&](uint32_t ch) {
            const uint32_t slot = fast_div(ch, g.div_k), lane = ch - slot * g.k;
            return (uint64_t(lane) * g.q + (lane < g.r ? lane : g.r) + slot) * B;
        };
        const uint64_t room = B - rem;                  // bytes of chunk c from the row's start on
        const bool whole = room >= uint64_t(nj) * sizeof(E);
        row_at[threadIdx.x] = uint16_t(at);
        row_first[threadIdx.x] = uint16_t(whole ? T * uint32_t(sizeof(E)) : uint32_t(room));
        row_rem[threadIdx.x] = rem;
        row_p0[threadIdx.x] = chunk_base(c) + rem;
        row_p1[threadIdx.x] = whole ? 0 : chunk_base(c + 1) + rem - B;          // (+ x >= B - rem for those bytes)
    };
    const SpanRows rows{packed, row_p0, row_p1, row_first, row_at, row_rem, part, wpart, ((t.packed_off | t.b) & 15u) != 0};
    u32x4 *lds = reinterpret_cast<u32x4 *>(lds_raw);
    const uint32_t na = UNPACK ? nj : ni, nb = UNPACK ? ni : nj;
    if (t.estep != sizeof(E)) {
        // one thread holds elements of one row: the part before the chunk border and the part after it are summed in
        // registers and go to LDS once
        Sums2 a0{0, 0}, a1{0, 0};
        place();
        fetch();
        __syncthreads();
        transpose_tile_elements<E, UNPACK, NTP>(user, t.a, t.estep, ni, nj, rows, lds_raw, [&](uint32_t i, E v, uint32_t j) {
            if constexpr (CHECK != CHECK_NONE) {
                Sums2 x{0, 0};
                count_elem<CHECK>(x, v, rows.template position<CHECK>(i, j * sizeof(E)));
                const bool ahead = j * sizeof(E) < row_first[i];
                a0.s += ahead ? x.s : 0, a0.w += ahead ? x.w : 0;
                a1.s += ahead ? 0 : x.s, a1.w += ahead ? 0 : x.w;
            }
        });
        if constexpr (CHECK != CHECK_NONE) {
            const uint32_t tx = threadIdx.x & (T - 1);
            if (a0.s) rows.template count<CHECK>(tx, false, a0);
            if (a1.s) rows.template count<CHECK>(tx, true, a1);
        }
    } else if (ni == T && nj == T) {
        transpose_tile_vectors<E, UNPACK, CHECK, NTU, NTP, true>(user, t.a, na, nb, rows, lds, place, fetch);
    } else {
        transpose_tile_vectors<E, UNPACK, CHECK, NTU, NTP, false>(user, t.a, na, nb, rows, lds, place, fetch);
    }
    if constexpr (CHECK != CHECK_NONE) {
        __syncthreads();
        auto arrive = [&](uint32_t i, uint32_t chunk, uint32_t ordinal, uint32_t expected) {
            if constexpr (CHECK == CHECK_SUMS) commit_total(part[i], chunk, ordinal, expected, ck.cx);
            else pair_commit_total(UNPACK ? SUM2_VERIFY : SUM2_SEAL, g, chunk, ordinal, expected, part[i], wpart[i], ck.out, ck.cx.acc, ck.cx.stride, ck.cx.fan, ck.work, [&] { return load_tag(g, chunk, ck.work); });
        };
        if (threadIdx.x < n_inc) arrive(threadIdx.x, my_chunk, my_ordinal, my_expected);
        for (uint32_t i = threadIdx.x + kThreads; i < n_inc; i += kThreads) arrive(i, my[2 * i], my[2 * i + 1], chunk_tiles[my[2 * i]]);
    }
}

template <typename E, bool UNPACK, int CHECK, bool NTP>
__global__ __launch_bounds__(kThreads) void k_transpose_span(const Tile *__restrict__ tiles,
                                                             const uint32_t *__restrict__ chunk_tiles,
                                                             const uint32_t *__restrict__ inc, ChunkGeom g,
                                                             BasePtrs bases, uint8_t *__restrict__ packed, CheckArgs<CHECK> ck)
{
    __shared__ __attribute__((aligned(16))) uint8_t lds_raw[transpose_lds_bytes<E>()];
    __shared__ SpanLds<TransposeShape<E>::T, CHECK> sp;
    const Tile t = tiles[blockIdx.x];
    if (t.kind == K_ZERO) {
        const TagRegs got = prefetch_check<UNPACK, CHECK>(ck, t.chunk);
        commit_tile<UNPACK, CHECK>(pad_tile<UNPACK, CHECK>(t, packed), t, chunk_tiles, ck, got);
        return;
    }
    transpose_span_any<E, UNPACK, CHECK, true, NTP>(t, chunk_tiles, inc, g, bases.p[t.tensor], packed, ck, lds_raw, sp);
}

// ---- generic: any strides, one element at a time -------------------------------
// Every element's address is recomputed from its logical index.  Only used for views the
// other kernels do not take (no dimension with stride one, or runs shorter than 16 bytes).
// The elements [e0, e0 + nel) of one tensor, every dim within reach of the multiply-shift division.
// ND > 0: the tensor has exactly ND merged dims; ND == 0: any number, read from the descriptor.
// The dims are copied into registers first: the loop below stores through byte pointers, which
// may alias anything, so values read through the descriptor inside it would be read again for
// every element.  Consecutive lanes take consecutive elements, U of them in flight per thread:
// a wave's access is contiguous on the packed side and as dense on the tensor side as the view
// allows.  The loads of a round are unconditional (the index is clamped into the tile), so that
// all of them are issued before the first is waited for; only the stores are guarded.
template <int ND>
struct ElementsOf {
    static constexpr int D = ND ? ND : HXT_MAX_DIMS;
    int nd;
    uint32_t shape[D], mul[D], shift[D], first[D];
    uint64_t stride[D];
    __device__ __forceinline__ ElementsOf(const TensorDev &td, uint64_t e0) : nd(ND ? ND : td.ndim)
    {
        uint64_t idx = e0;                                  // coordinates of the span's first element
#pragma unroll
        for (int d = D - 1; d >= 0; --d) {
            shape[d] = 1, mul[d] = 0, shift[d] = 0, first[d] = 0, stride[d] = 0;
            if (d < nd) {
                shape[d] = uint32_t(td.shape[d]);
                mul[d] = td.dim_div[d].mul;
                shift[d] = td.dim_div[d].shift;
                stride[d] = uint64_t(td.stride_b[d]);
                const uint64_t q = idx / uint64_t(td.shape[d]);
                first[d] = uint32_t(idx - q * uint64_t(td.shape[d]));
                idx = q;
            }
        }
    }
    // Storage offset of element el of the span.  An element's coordinates are the first element's plus its number within
    // the span, carried from the last dim upwards in 32 bits (a span has fewer than 2^30 elements and so has every dim).
    // left: elements of the last dim from this one to its end.
    __device__ __forceinline__ uint64_t at(uint32_t el, uint32_t *left = nullptr) const
    {
        uint64_t off = 0;
        uint32_t x = el;
        if (left && nd == 1) *left = shape[0] - (first[0] + el);
#pragma unroll
        for (int d = D - 1; d > 0; --d) {
            if (d < nd) {
                x += first[d];
                const uint32_t q = fast_div(x, FastDiv{mul[d], shift[d]});
                if (left && d == nd - 1) *left = shape[d] - (x - q * shape[d]);
                off += uint64_t(x - q * shape[d]) * stride[d];
                x = q;
            }
        }
        return off + uint64_t(x + first[0]) * stride[0];
    }
};

template <typename E, bool UNPACK, int CHECK, bool NTP, bool THROUGH, int ND>
__device__ __forceinline__ Sums2 generic_span(const TensorDev &td, uint64_t e0, uint32_t nel, uint8_t *user, E *p, uint64_t in_chunk)
{
    const ElementsOf<ND> els(td, e0);
    auto locate = [&](uint32_t el) { return reinterpret_cast<E *>(user + els.at(el)); };
    constexpr int U = 8;
    Sums2 acc{0, 0};
    const uint32_t last = nel - 1;
    for (uint32_t e1 = threadIdx.x; e1 < nel; e1 += kThreads * U) {
        E val[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t el = min(e1 + u * kThreads, last);
            if constexpr (UNPACK) val[u] = load_elem<NTP>(p + el);
            else val[u] = load_elem<true>(locate(el));
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t el = e1 + u * kThreads;
            if (el < nel) {
                if constexpr (UNPACK) store_elem<true>(locate(el), val[u]);
                else store_packed_elem<NTP, THROUGH>(p + el, val[u]);
                count_elem<CHECK>(acc, val[u], in_chunk + uint64_t(el) * sizeof(E));
            }
        }
    }
    return acc;
}

// Sending elements (of 1 or 2 bytes) that lie S = 2 or 4 apart: M = 16 / (S * element size) neighbours of a run are read as one vector, so that
// a wave's load is contiguous, picked out of the registers and stored side by side, 16 / S bytes.  The vector starts with the
// first of them; where they are the last of their run it ends with the last of them instead (what lies behind need not be
// the view's); neighbours that are not of one run are read one by one.
// What it saves is instructions, a load of 2 bytes for every element.  Pack alone with sums, element by element against this:
// every other of 16.8 M bf16 25.5 -> 21.3 us (tensors not in the cache 27.5 -> 24.1), of 8 M 15.3 -> 11.3, of 6 M with tags
// 14.4 -> 9.9, of 33.5 M bytes 42.0 -> 21.2; every fourth of 4 M bf16 11.4 -> 10.1, of 16.8 M 33.0 -> 32.6, of 33.5 M bytes
// 44.1 -> 33.0.  Not for elements of 4 bytes, whose own loads are wide enough (every other of 8.4 M f32 21.4 -> 23.0, every
// fourth 33.2 -> 37.9).  The packed side is written through by the rule for single elements (every fourth of 1.2 M bf16, pack +
// unpack, 14.2 us through, 12.6 not; 14.0 element by element).  Every third goes element by element: read as whole vectors, lanes 48 bytes apart, 29.3 -> 33.5.
template <typename E, uint32_t S>
struct Apart {
    static constexpr uint32_t ES = sizeof(E), M = 16 / (S * ES), BYTES = M * ES, BEHIND = (S - 1) * ES;
    using P = std::conditional_t<BYTES == 8, uint64_t, uint32_t>;
    static_assert(ES <= 2 && BYTES == sizeof(P));
    // The elements at bytes 0, S * ES, 2 * S * ES ... of a vector.
    static __device__ __forceinline__ P pick(u32x4 v)
    {
        auto two = [](uint32_t a, uint32_t b) {             // the elements that start in each of two words, side by side
            if constexpr (ES == 2) return __builtin_amdgcn_perm(b, a, 0x05040100u);
            else return S == 2 ? __builtin_amdgcn_perm(b, a, 0x06040200u) : __builtin_amdgcn_perm(b, a, 0x0C0C0400u);      // (0x0C: zero)
        };
        if constexpr (ES == 2) {
            if constexpr (S == 2) return uint64_t(two(v.z, v.w)) << 32 | two(v.x, v.y);
            else return two(v.x, v.z);
        } else {
            if constexpr (S == 2) return uint64_t(two(v.z, v.w)) << 32 | two(v.x, v.y);
            else return two(v.x, v.y) | two(v.z, v.w) << 16;
        }
    }
};

template <typename E, uint32_t S, int CHECK, bool NTP, bool THROUGH, int ND>
__device__ __forceinline__ Sums2 send_apart(const TensorDev &td, uint64_t e0, uint32_t nel, const uint8_t *user, E *p, uint64_t in_chunk)
{
    using A = Apart<E, S>;
    using P = typename A::P;
    constexpr uint32_t ES = sizeof(E), M = A::M, U = 8;
    const ElementsOf<ND> els(td, e0);
    const uint32_t groups = nel / M;
    P *const out = reinterpret_cast<P *>(p);
    Sums2 acc{0, 0};
    for (uint32_t g0 = threadIdx.x; g0 < groups; g0 += kThreads * U) {
        u32x4 r[U];
        uint32_t left[U];
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
            // (of two runs: what the first run ends with is read, which is not used)
            uint64_t off = els.at(min(g0 + u * kThreads, groups - 1) * M, &left[u]);
            if (left[u] <= M) off -= A::BEHIND + (M - left[u]) * (S * ES);
            r[u] = load16_any<true>(user + off);
        }
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
            const uint32_t g = g0 + u * kThreads;
            if (g >= groups) continue;
            if (left[u] == M) r[u] = shift_bytes_down(r[u], A::BEHIND);
            P v = A::pick(r[u]);
            if (left[u] < M) {
                union {
                    E e[M];
                    P x;
                } o;
#pragma unroll
                for (uint32_t q = 0; q < M; ++q) o.e[q] = *reinterpret_cast<const E *>(user + els.at(g * M + q));
                v = o.x;
            }
            store_packed_elem<NTP, THROUGH>(out + g, v);
            count_elem<CHECK>(acc, v, in_chunk + uint64_t(g) * A::BYTES);
        }
    }
    if (threadIdx.x < nel - groups * M) {                   // only at the very end of the tensor
        const uint32_t el = groups * M + threadIdx.x;
        const E v = *reinterpret_cast<const E *>(user + els.at(el));
        p[el] = v;
        count_elem<CHECK>(acc, v, in_chunk + uint64_t(el) * ES);
    }
    return acc;
}

// The same for tensors with a dim beyond the reach of the multiply-shift division: every element's
// index is divided out in 64 bits.
template <typename E, bool UNPACK, int CHECK, bool NTP, bool THROUGH>
__device__ __noinline__ Sums2 generic_span_wide(const TensorDev &td, uint64_t e0, uint32_t nel, uint8_t *user, E *p, uint64_t in_chunk)
{
    const int nd = td.ndim;
    Sums2 acc{0, 0};
    for (uint32_t el = threadIdx.x; el < nel; el += kThreads) {
        uint64_t idx = e0 + el, off = 0;
        for (int d = nd - 1; d >= 0; --d) {
            const uint64_t q = idx / uint64_t(td.shape[d]);
            off += (idx - q * uint64_t(td.shape[d])) * uint64_t(td.stride_b[d]);
            idx = q;
        }
        E *at = reinterpret_cast<E *>(user + off);
        E v;
        if constexpr (UNPACK) {
            v = load_elem<NTP>(p + el);
            store_elem<true>(at, v);
        } else {
            v = load_elem<true>(at);
            store_packed_elem<NTP, THROUGH>(p + el, v);
        }
        count_elem<CHECK>(acc, v, in_chunk + uint64_t(el) * sizeof(E));
    }
    return acc;
}

// APART: with send_apart, where takes_apart finds use for it.  Elsewhere its registers (65 to 79 instead of 44 to 51: 6 or 7 waves
// per SIMD instead of 8) only slow the others down: sends of every third and fifth element, without it and with it, bytes with
// tags 1 MB 10.6 -> 11.1, 11.2 -> 11.8, 11.5 -> 12.0, 4 MB 13.6 -> 14.0, 13.4 -> 13.8, 14.1 -> 14.5, bf16 1 MB 7.1 -> 7.3, with tags
// 8.1 -> 8.3; from 16 MB on there is no difference.  A bundle of 7 MB with tags in k_message, which has no room for it, 23.0 ->
// 24.4 a pair.
template <typename E, bool UNPACK, int CHECK, bool NTP, bool THROUGH, bool APART>
__device__ __forceinline__ Sums2 generic_any(const Tile &t, const TensorDev &td, uint8_t *user, uint8_t *packed)
{
    E *p = reinterpret_cast<E *>(packed + t.packed_off);
    const uint32_t nel = t.n0 / sizeof(E);
    const uint64_t e0 = t.src_off / sizeof(E);
    if (nel == 0) return Sums2{0, 0};
    if (!td.all_div) return generic_span_wide<E, UNPACK, CHECK, NTP, THROUGH>(td, e0, nel, user, p, t.a);
    if constexpr (!UNPACK && APART && sizeof(E) <= 2) {
        const uint64_t step = uint64_t(td.stride_b[td.ndim - 1]);
        auto apart = [&]<uint32_t S>() {
            return td.ndim == 1 ? send_apart<E, S, CHECK, NTP, THROUGH, 1>(td, e0, nel, user, p, t.a)
                                : send_apart<E, S, CHECK, NTP, THROUGH, 0>(td, e0, nel, user, p, t.a);
        };
        if (td.apart) {
            if (step == 2 * sizeof(E)) return apart.template operator()<2>();
            return apart.template operator()<4>();
        }
    }
    switch (td.ndim) {
    case 1: return generic_span<E, UNPACK, CHECK, NTP, THROUGH, 1>(td, e0, nel, user, p, t.a);
    case 2: return generic_span<E, UNPACK, CHECK, NTP, THROUGH, 2>(td, e0, nel, user, p, t.a);
    case 3: return generic_span<E, UNPACK, CHECK, NTP, THROUGH, 3>(td, e0, nel, user, p, t.a);
    case 4: return generic_span<E, UNPACK, CHECK, NTP, THROUGH, 4>(td, e0, nel, user, p, t.a);
    default: return generic_span<E, UNPACK, CHECK, NTP, THROUGH, 0>(td, e0, nel, user, p, t.a);
    }
}

template <typename E, bool UNPACK, int CHECK, bool NTP, bool THROUGH, bool APART>
__global__ __launch_bounds__(kThreads) void k_generic(const Tile *__restrict__ tiles,
                                                      const uint32_t *__restrict__ chunk_tiles,
                                                      const TensorDev *__restrict__ tensors, uint32_t tensor_base,
                                                      BasePtrs bases, uint8_t *__restrict__ packed, CheckArgs<CHECK> ck)
{
    const Tile t = tiles[blockIdx.x];
    const TagRegs got = prefetch_check<UNPACK, CHECK>(ck, t.chunk);
    const Sums2 acc = t.kind == K_ZERO ? pad_tile<UNPACK, CHECK>(t, packed) : generic_any<E, UNPACK, CHECK, NTP, THROUGH, APART>(t, tensors[tensor_base + t.tensor], bases.p[t.tensor], packed);
    commit_tile<UNPACK, CHECK>(acc, t, chunk_tiles, ck, got);
}

// ---- a whole message of several kinds of view in one launch --------------------------
// Messages that mix views (an activation, a mask, a transposed projection, the pads between them) are small more often
// than not, and one launch per kind then costs more than the bytes: each has to fill the chip and drain it again for a
// few dozen tiles.  Here every workgroup looks at its tile's kind.  The kernel needs the registers and the LDS of its
// hungriest branch, which a large message would feel: see kOneLaunchLimit.
struct MessageArgs {
    BasePtrs bases;                    // of all tensors of the message
    uint32_t first[6], base[6];        // per launch group of the plan: its first tile, its first tensor
    uint32_t n;
};

template <bool UNPACK, int CHECK>
__global__ __launch_bounds__(kThreads) void k_message(const Tile *__restrict__ tiles, const uint32_t *__restrict__ chunk_tiles,
                                                      const TensorDev *__restrict__ tensors, const uint32_t *__restrict__ inc,
                                                      ChunkGeom g, MessageArgs a, uint8_t *__restrict__ packed, CheckArgs<CHECK> ck)
{
    // The hints of a small message.  (Loads from the tensors cacheable, unlike in kernels of their own: the tiles of one
    // tensor share memory bursts and run far apart in time here.  7 MB in four kinds of view, pack, through two packed
    // buffers: 8.5 us, non-temporal 10.4; 34 MB 22.9 and 21.8.)
    constexpr bool NTU = UNPACK, NTP = false;
    constexpr uint32_t kLds = transpose_lds_bytes<uint64_t>() > transpose_lds_bytes<uint16_t>() ? transpose_lds_bytes<uint64_t>()
                                                                                                : transpose_lds_bytes<uint16_t>();
    __shared__ __attribute__((aligned(16))) uint8_t lds_raw[kLds];
    __shared__ SpanLds<TransposeShape<uint16_t>::T, CHECK, 0> sp;
    const Tile t = tiles[blockIdx.x];
    uint32_t first_tensor = a.base[0];
#pragma unroll
    for (uint32_t i = 1; i < 6; ++i)
        if (i < a.n && blockIdx.x >= a.first[i]) first_tensor = a.base[i];
    const TensorDev &td = tensors[first_tensor + t.tensor];
    uint8_t *base = a.bases.p[first_tensor + t.tensor], *pk = packed + t.packed_off;
    auto by_size = [&](auto &&f) {
        switch (td.esize) {
        case 1: return f.template operator()<uint8_t>();
        case 2: return f.template operator()<uint16_t>();
        case 4: return f.template operator()<uint32_t>();
        default: return f.template operator()<uint64_t>();
        }
    };
    if (t.kind == K_TRANSPOSE_SPAN) {                  // (its field `chunk` is no chunk; it commits by itself)
        by_size([&]<typename E>() { transpose_span_any<E, UNPACK, CHECK, NTU, NTP>(t, chunk_tiles, inc, g, base, packed, ck, lds_raw, sp); });
        return;
    }
    const TagRegs got = prefetch_check<UNPACK, CHECK>(ck, t.chunk);
    Sums2 acc{0, 0};
    switch (t.kind) {
    case K_ZERO:
        acc = pad_tile<UNPACK, CHECK>(t, packed);
        break;
    case K_CONTIG:
        if constexpr (CHECK == CHECK_TAGS) {
            acc = copy_span2<UNPACK, NTU, NTP>(base + t.src_off, pk, t.n0);
            acc.w += (t.a >> 2) * acc.s;
        } else {
            acc.s = copy_span<UNPACK, CHECK == CHECK_SUMS, NTU, NTP>(base + t.src_off, pk, t.n0);
        }
        break;
    case K_ROWS: acc = rows_tile<UNPACK, CHECK, NTU, NTP>(t, td, base, pk); break;
    case K_ROWS_SPLIT:
        // (receiving, pieces are named as the likely way, or the code of the vectors around them slows them down: 7 MB in four
        // kinds of view with tags, unpack 10.7 us against 10.2; sending it is the other way round, 10.5 against 11.1)
        acc = rows_split_any<UNPACK, CHECK, NTP, UNPACK>(t, td, base, pk);
        break;
    case K_TRANSPOSE:
        acc = by_size([&]<typename E>() { return transpose_any<E, UNPACK, CHECK, NTU, NTP>(t, base, packed, ck, lds_raw); });
        break;
    default: acc = by_size([&]<typename E>() { return generic_any<E, UNPACK, CHECK, NTP, false, false>(t, td, base, packed); }); break;
    }
    // (with tags, what the sums are reduced in lies where a spanning tile keeps its own: 40960 bytes of LDS are four
    // workgroups per CU, 64 more were three.  Pack + unpack with
    // tags of bundles of four kinds: 24 MB 41.7 -> 39.0 us, 31 MB 44.1 -> 40.8; 7 MB, one round of tiles, 22.9 and 23.1)
    if constexpr (CHECK == CHECK_TAGS) commit_tags<UNPACK>(acc, t, chunk_tiles, ck, got, reinterpret_cast<PairParts &>(sp.part));
    else commit_tile<UNPACK, CHECK>(acc, t, chunk_tiles, ck, got);
}

// ---- stand-alone checksum of packed chunks (closed-form geometry, no table) ----------
template <bool NTP>
__global__ __launch_bounds__(kThreads) void k_checksum(ChunkGeom g, const uint8_t *__restrict__ packed, SumCtx cx)
{
    const TileSpan t = locate_tile(g, blockIdx.x);
    const u32x4 *s = reinterpret_cast<const u32x4 *>(packed + t.packed_off);
    const uint32_t nvec = t.len >> 4;
    uint64_t acc = 0;
    for (uint32_t v = threadIdx.x; v < nvec; v += kThreads * kUnroll) {
        u32x4 r[kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u)
            r[u] = load16_or_zero<NTP>(s, v + u * kThreads, nvec);
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) acc += words_sum(r[u]);
    }
    chunk_commit(acc, t.chunk, t.ordinal, t.expected, cx);
}

// ---- stand-alone strong check: the pass over the packed chunks -------------------------
// Word j of the chunk sits at tile word i = j - j0.  A thread's vectors start at tile words
// 4 * (tid + 256 * n), n = 0, 1, ...; with S_n the sum of vector n's words and I_n = y + 2z + 3w,
//   sum (j+1) w_j = (j0 + 4 tid + 1) * sum_n S_n + 1024 * sum_n n S_n + sum_n I_n,
// so the loop needs additions only (sum_n n S_n is kept as a running suffix sum) and each
// thread multiplies once.
template <int MODE, bool NTP>
__global__ __launch_bounds__(kThreads) void k_checksum2(ChunkGeom g, const uint8_t *__restrict__ packed,
                                                        void *__restrict__ out, uint8_t *acc, uint32_t stride,
                                                        uint32_t fan, TagWork work)
{
    const TileSpan t = locate_tile(g, blockIdx.x);
    const TagRegs got = prefetch_tag(MODE, g, t.chunk, work);
    const u32x4 *s = reinterpret_cast<const u32x4 *>(packed + t.packed_off);
    const uint64_t j0 = (t.stream_off - uint64_t(t.chunk) * g.B) >> 2;
    const uint32_t nvec = t.len >> 4;
    uint64_t S = 0, nS = 0, I = 0;          // sum_n S_n, sum_n n*S_n, sum_n I_n
    uint64_t n0 = 0;                         // n of the current block of vectors
    for (uint32_t v = threadIdx.x; v < nvec; v += kThreads * kUnroll, n0 += kUnroll) {
        u32x4 r[kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u)
            r[u] = load16_or_zero<NTP>(s, v + u * kThreads, nvec);
        uint64_t blockS = 0, blockN = 0;     // this block's sum_u S_u and sum_u u*S_u
#pragma unroll
        for (int u = kUnroll - 1; u >= 0; --u) {
            const uint64_t zw = uint64_t(r[u].z) + r[u].w;
            const uint64_t yzw = zw + r[u].y;
            blockN += blockS;                // after the loop: sum_u u * S_u
            blockS += yzw + r[u].x;
            I += yzw + zw + r[u].w;
        }
        S += blockS;
        nS += blockN + n0 * blockS;
    }
    __shared__ PairParts part;
    pair_commit(MODE, g, t, S, (j0 + 4ull * threadIdx.x + 1) * S + 4ull * kThreads * nS + I, out, acc, stride, fan, work, got, part);
}

// ---- pack + seal and unpack + verify in one pass (messages that are one contiguous tensor) ----
// The copy of k_uniform with both sums of the packed words taken on the way, so that tags cost no
// extra pass over the message.  Weights are tile-local here (word i of the tile weighs i + 1);
// the tile's position in its chunk is applied once per workgroup.
// One launch serves up to kMaxBatch such messages (workgroups [first_tile, first_tile + ntiles) belong to
// message i), as k_uniform does for the plain sums.
struct UniformTagItem {
    ChunkGeom g;
    uint8_t *user;
    uint8_t *packed;
    void *out;             // SEAL: the message's tags; VERIFY: its status words
    uint8_t *acc;          // the plan's pair-of-sums accumulator slots
    uint32_t stride, fan;
    TagWork work;
    uint32_t first_tile;
};

struct UniformTagArgs {
    UniformTagItem it[kMaxBatch];
    uint32_t n;
};

template <bool UNPACK, int MODE, bool NTU, bool NTP>
__global__ __launch_bounds__(kThreads) void k_uniform_tag(UniformTagArgs a)
{
    uint32_t m = 0;
#pragma unroll
    for (uint32_t i = 1; i < kMaxBatch; ++i)
        if (i < a.n && blockIdx.x >= a.it[i].first_tile) m = i;
    const UniformTagItem &it = a.it[m];
    const ChunkGeom &g = it.g;
    const TileSpan t = locate_tile(g, blockIdx.x - it.first_tile);
    const TagRegs got = prefetch_tag(MODE, g, t.chunk, it.work);
    const uint64_t left = g.N > t.stream_off ? g.N - t.stream_off : 0;
    const uint32_t data = left < t.len ? uint32_t(left) : t.len;
    uint8_t *pk = it.packed + t.packed_off;
    Sums2 sums = copy_span2<UNPACK, NTU, NTP>(it.user + t.stream_off, pk, data);
    if (data < t.len) {
        const Sums2 pad = pad_span2<UNPACK>(pk + data, t.len - data, data);
        sums.s += pad.s;
        sums.w += pad.w;
    }
    const uint64_t j0 = (t.stream_off - uint64_t(t.chunk) * g.B) >> 2;       // the tile's first word in its chunk
    __shared__ PairParts part;
    pair_commit(MODE, g, t, sums.s, j0 * sums.s + sums.w, it.out, it.acc, it.stride, it.fan, it.work, got, part);
}

// The same for the contiguous tensors of a multi-tensor message (gradient buckets): the table-driven copy
// of k_contig with both sums taken on the way.  A tile's record says where it starts inside its chunk.
template <bool UNPACK, int MODE, bool NTU, bool NTP>
__global__ __launch_bounds__(kThreads) void k_contig_tag(const Tile *__restrict__ tiles,
                                                         const uint32_t *__restrict__ chunk_tiles, BasePtrs bases,
                                                         uint8_t *__restrict__ packed, ChunkGeom g, void *out,
                                                         uint8_t *acc, uint32_t stride, uint32_t fan, TagWork work)
{
    const Tile t = tiles[blockIdx.x];
    const TagRegs got = prefetch_tag(MODE, g, t.chunk, work);
    TileSpan span{};
    span.chunk = t.chunk;
    span.ordinal = t.ordinal;
    span.expected = chunk_tiles[t.chunk];
    Sums2 sums;
    uint64_t j0 = 0;
    if (t.kind == K_ZERO) {                                  // byte granular: weights taken from the chunk's start
        sums = pad_span2<UNPACK>(packed + t.packed_off, t.n0, t.a);
    } else {
        sums = copy_span2<UNPACK, NTU, NTP>(bases.p[t.tensor] + t.src_off, packed + t.packed_off, t.n0);
        j0 = t.a >> 2;
    }
    __shared__ PairParts part;
    pair_commit(MODE, g, span, sums.s, j0 * sums.s + sums.w, out, acc, stride, fan, work, got, part);
}

}  // namespace hxt

#endif
