// Launches of the kernels that are compiled in files of their own, so that the library builds on several processors.
#ifndef HXT_LAUNCH_H
#define HXT_LAUNCH_H

#include "hxt_kernels.h"

namespace hxt {

// Calls f.template operator()<NTU, NTP>() for the chosen cache hints.
template <typename F>
void with_hints(bool nt_user, bool nt_packed, F &&f)
{
    if (nt_user) {
        if (nt_packed) f.template operator()<true, true>();
        else f.template operator()<true, false>();
    } else {
        if (nt_packed) f.template operator()<false, true>();
        else f.template operator()<false, false>();
    }
}

// Cache hints of a launch: the tensor side's and the packed side's accesses are non-temporal.
struct Hints {
    bool user, packed;
};

// The hints of the strided kernels, whose stores to the tensors are always non-temporal: a receiving launch has one hint.
template <bool UNPACK, typename F>
void with_strided_hints(Hints h, F &&f)
{
    if constexpr (UNPACK) {
        if (h.packed) f.template operator()<true, true>();
        else f.template operator()<true, false>();
    } else {
        with_hints(h.user, h.packed, f);
    }
}

template <bool UNPACK, int CHECK>
void launch_transpose(Hints h, const Tile *tiles, uint32_t count, int esize, const uint32_t *chunk_tiles, const BasePtrs &b,
                      uint8_t *packed, const CheckArgs<CHECK> &ck, hipStream_t st);

template <bool UNPACK, int CHECK>
void launch_transpose_span(Hints h, const Tile *tiles, uint32_t count, int esize, const uint32_t *chunk_tiles,
                           const uint32_t *inc, const ChunkGeom &g, const BasePtrs &b, uint8_t *packed,
                           const CheckArgs<CHECK> &ck, hipStream_t st);

template <bool UNPACK, int CHECK>
void launch_message(const Tile *tiles, uint32_t count, const uint32_t *chunk_tiles, const TensorDev *tensors, const uint32_t *inc,
                    const ChunkGeom &g, const MessageArgs &a, uint8_t *packed, const CheckArgs<CHECK> &ck, hipStream_t st);

}  // namespace hxt

#endif
