// The kernels of the general family on the matrix cores: the register-staged 128x128 macro-tile kernel for 16-bit operands
// of any alignment, and the 64x64 fp32 tile with the sums of each slab folded.
//
// Bound of the first: unaligned loads through the registers (2049x2051x2045 bf16 NT 57 us, NN 53, TT 53, TN 66; the plain kernel
// 1245 to 1340).  With A stored K x M it spills (48 and 108 bytes a thread) to fit two workgroups on a unit, which is still
// the better choice: with one, and nothing spilled, TN takes 108 us and TT 86; 511x513x1023 TN 17.3 against 17.9.  With folded
// sums (an fp32 C) the second set of sums does not fit beside a second workgroup: 92 to 124 us.
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
