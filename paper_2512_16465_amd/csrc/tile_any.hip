// The kernels of the general family on the matrix cores: the register-staged 128x128 macro-tile kernel for 16-bit operands
// of any alignment, and the 64x64 fp32 tile with the sums of each slab folded.
#include "tile_f32_kernel.hpp"

namespace gemm {
namespace {
template <bool FOLD>
hipError_t launch_any(const Args& a, int group_m, hipStream_t stream, int64_t slice_len) {
    using C = tile::Cfg<128, 128, 64, 2, 2>;
    return slice_len ? tile::launch_variant<C, true, FOLD, true>(a, group_m, stream, slice_len) : tile::launch_variant<C, true, FOLD>(a, group_m, stream);
}
}  // namespace
hipError_t launch_any_tile(const Args& a, int group_m, hipStream_t stream, int64_t slice_len, bool fold) {
    return fold ? launch_any<true>(a, group_m, stream, slice_len) : launch_any<false>(a, group_m, stream, slice_len);
}
hipError_t launch_any_f32_tile(const Args& a, int group_m, hipStream_t stream, int64_t slice_len) {
    using C = tile::F32CfgT<64, 64, 2, 2, true>;
    return slice_len ? tile::launch_f32_tiles<C, true>(a, group_m, stream, slice_len) : tile::launch_f32_tiles<C>(a, group_m, stream);
}
}  // namespace gemm
