// Launches of k_message, receiving side.
#include "hxt_launch.h"

namespace hxt {

template <bool UNPACK, int CHECK>
void launch_message(const Tile *tiles, uint32_t count, const uint32_t *chunk_tiles, const TensorDev *tensors, const uint32_t *inc,
                    const ChunkGeom &g, const MessageArgs &a, uint8_t *packed, const CheckArgs<CHECK> &ck, hipStream_t st)
{
    k_message<UNPACK, CHECK><<<count, kThreads, 0, st>>>(tiles, chunk_tiles, tensors, inc, g, a, packed, ck);
}

template void launch_message<true, CHECK_NONE>(const Tile *, uint32_t, const uint32_t *, const TensorDev *, const uint32_t *, const ChunkGeom &, const MessageArgs &, uint8_t *, const CheckArgs<CHECK_NONE> &, hipStream_t);
template void launch_message<true, CHECK_SUMS>(const Tile *, uint32_t, const uint32_t *, const TensorDev *, const uint32_t *, const ChunkGeom &, const MessageArgs &, uint8_t *, const CheckArgs<CHECK_SUMS> &, hipStream_t);
template void launch_message<true, CHECK_TAGS>(const Tile *, uint32_t, const uint32_t *, const TensorDev *, const uint32_t *, const ChunkGeom &, const MessageArgs &, uint8_t *, const CheckArgs<CHECK_TAGS> &, hipStream_t);

}  // namespace hxt
