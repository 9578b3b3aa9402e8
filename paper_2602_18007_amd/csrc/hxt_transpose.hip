// Launches of k_transpose.
#include "hxt_launch.h"

namespace hxt {

template <bool UNPACK, int CHECK>
void launch_transpose(bool ntp, const Tile *tiles, uint32_t count, int esize, const uint32_t *chunk_tiles, const BasePtrs &b,
                      uint8_t *packed, const CheckArgs<CHECK> &ck, hipStream_t st)
{
    auto go = [&]<bool NTP>() {
        switch (esize) {
        case 1: k_transpose<uint8_t, UNPACK, CHECK, NTP><<<count, kThreads, 0, st>>>(tiles, chunk_tiles, b, packed, ck); break;
        case 2: k_transpose<uint16_t, UNPACK, CHECK, NTP><<<count, kThreads, 0, st>>>(tiles, chunk_tiles, b, packed, ck); break;
        case 4: k_transpose<uint32_t, UNPACK, CHECK, NTP><<<count, kThreads, 0, st>>>(tiles, chunk_tiles, b, packed, ck); break;
        default: k_transpose<uint64_t, UNPACK, CHECK, NTP><<<count, kThreads, 0, st>>>(tiles, chunk_tiles, b, packed, ck); break;
        }
    };
    if (ntp) go.template operator()<true>();
    else go.template operator()<false>();
}

template void launch_transpose<false, CHECK_NONE>(bool, const Tile *, uint32_t, int, const uint32_t *, const BasePtrs &, uint8_t *, const CheckArgs<CHECK_NONE> &, hipStream_t);
template void launch_transpose<false, CHECK_SUMS>(bool, const Tile *, uint32_t, int, const uint32_t *, const BasePtrs &, uint8_t *, const CheckArgs<CHECK_SUMS> &, hipStream_t);
template void launch_transpose<false, CHECK_TAGS>(bool, const Tile *, uint32_t, int, const uint32_t *, const BasePtrs &, uint8_t *, const CheckArgs<CHECK_TAGS> &, hipStream_t);
template void launch_transpose<true, CHECK_NONE>(bool, const Tile *, uint32_t, int, const uint32_t *, const BasePtrs &, uint8_t *, const CheckArgs<CHECK_NONE> &, hipStream_t);
template void launch_transpose<true, CHECK_SUMS>(bool, const Tile *, uint32_t, int, const uint32_t *, const BasePtrs &, uint8_t *, const CheckArgs<CHECK_SUMS> &, hipStream_t);
template void launch_transpose<true, CHECK_TAGS>(bool, const Tile *, uint32_t, int, const uint32_t *, const BasePtrs &, uint8_t *, const CheckArgs<CHECK_TAGS> &, hipStream_t);

}  // namespace hxt
