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

// (The strided kernels take the packed side's hint alone: ntp.)
template <bool UNPACK, int CHECK>
void launch_transpose(bool ntp, const Tile *tiles, uint32_t count, int esize, const uint32_t *chunk_tiles, const BasePtrs &b,
                      uint8_t *packed, const CheckArgs<CHECK> &ck, hipStream_t st);

template <bool UNPACK, int CHECK>
void launch_transpose_span(bool ntp, const Tile *tiles, uint32_t count, int esize, const uint32_t *chunk_tiles,
                           const uint32_t *inc, const ChunkGeom &g, const BasePtrs &b, uint8_t *packed,
                           const CheckArgs<CHECK> &ck, hipStream_t st);

template <bool UNPACK, int CHECK>
void launch_message(const Tile *tiles, uint32_t count, const uint32_t *chunk_tiles, const TensorDev *tensors, const uint32_t *inc,
                    const ChunkGeom &g, const MessageArgs &a, uint8_t *packed, const CheckArgs<CHECK> &ck, hipStream_t st);

}  // namespace hxt

#endif
