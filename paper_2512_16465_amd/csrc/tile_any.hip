// The register-staged 128x128 macro-tile kernel for 16-bit operands of any alignment.
#include "tile_kernel.hpp"

namespace gemm {
hipError_t launch_any_tile(const Args& a, int group_m, hipStream_t stream) { return tile::launch_variant<tile::Cfg<128, 128, 64, 2, 2>, true>(a, group_m, stream); }
}  // namespace gemm
