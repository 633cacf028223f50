// The wave tiles for 16-bit operands off the 16-byte grid, in place of the general family's 128x128 tiles.
#include "tile_wavek_kernel.hpp"

namespace gemm {
hipError_t launch_wave_any(const Args& a, int rows, int group_m, hipStream_t stream) {
    return rows == 16 ? tile::launch_wavek_variant<tile::WaveK<16, 1, 3, true>>(a, group_m, stream)
                                   : tile::launch_wavek_variant<tile::WaveK<64, 1, 2, true>>(a, group_m, stream);
}
}  // namespace gemm
