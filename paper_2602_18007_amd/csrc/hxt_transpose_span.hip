// Launches of k_transpose_span.
#include "hxt_launch.h"

namespace hxt {

template <bool UNPACK, int CHECK>
void launch_transpose_span(bool ntp, const Tile *tiles, uint32_t count, int esize, const uint32_t *chunk_tiles,
                           const uint32_t *inc, const ChunkGeom &g, const BasePtrs &b, uint8_t *packed,
                           const CheckArgs<CHECK> &ck, hipStream_t st)
{
    auto go = [&]<bool NTP>() {
        switch (esize) {
        case 1: k_transpose_span<uint8_t, UNPACK, CHECK, NTP><<<count, kThreads, 0, st>>>(tiles, chunk_tiles, inc, g, b, packed, ck); break;
        case 2: k_transpose_span<uint16_t, UNPACK, CHECK, NTP><<<count, kThreads, 0, st>>>(tiles, chunk_tiles, inc, g, b, packed, ck); break;
        case 4: k_transpose_span<uint32_t, UNPACK, CHECK, NTP><<<count, kThreads, 0, st>>>(tiles, chunk_tiles, inc, g, b, packed, ck); break;
        default: k_transpose_span<uint64_t, UNPACK, CHECK, NTP><<<count, kThreads, 0, st>>>(tiles, chunk_tiles, inc, g, b, packed, ck); break;
        }
    };
    if (ntp) go.template operator()<true>();
    else go.template operator()<false>();
}

template void launch_transpose_span<false, CHECK_NONE>(bool, const Tile *, uint32_t, int, const uint32_t *, const uint32_t *, const ChunkGeom &, const BasePtrs &, uint8_t *, const CheckArgs<CHECK_NONE> &, hipStream_t);
template void launch_transpose_span<false, CHECK_SUMS>(bool, const Tile *, uint32_t, int, const uint32_t *, const uint32_t *, const ChunkGeom &, const BasePtrs &, uint8_t *, const CheckArgs<CHECK_SUMS> &, hipStream_t);
template void launch_transpose_span<false, CHECK_TAGS>(bool, const Tile *, uint32_t, int, const uint32_t *, const uint32_t *, const ChunkGeom &, const BasePtrs &, uint8_t *, const CheckArgs<CHECK_TAGS> &, hipStream_t);
template void launch_transpose_span<true, CHECK_NONE>(bool, const Tile *, uint32_t, int, const uint32_t *, const uint32_t *, const ChunkGeom &, const BasePtrs &, uint8_t *, const CheckArgs<CHECK_NONE> &, hipStream_t);
template void launch_transpose_span<true, CHECK_SUMS>(bool, const Tile *, uint32_t, int, const uint32_t *, const uint32_t *, const ChunkGeom &, const BasePtrs &, uint8_t *, const CheckArgs<CHECK_SUMS> &, hipStream_t);
template void launch_transpose_span<true, CHECK_TAGS>(bool, const Tile *, uint32_t, int, const uint32_t *, const uint32_t *, const ChunkGeom &, const BasePtrs &, uint8_t *, const CheckArgs<CHECK_TAGS> &, hipStream_t);

}  // namespace hxt
