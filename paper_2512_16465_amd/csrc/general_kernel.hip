// The general family: calls whose operands are not on the 16-byte grid, or whose contiguous dimension is not a
// multiple of 8.  Most of them go on to matrix-core kernels that need no alignment; the general kernel proper, one
// thread per output element, any shape, leading dimension, alignment and element type, is the correctness floor under
// them, and it also serves K == 0 and alpha == 0 where only the epilogue is left.
#include "common.hpp"

namespace gemm {

namespace {

constexpr int GT = 16;   // 16 x 16 threads per workgroup

// A small LDS-tiled contraction in fp32: each workgroup computes a 16 x 16 block of C, staging
// 16 x 16 blocks of op(A) and op(B).  Partial sums are folded every 16 terms, which keeps the
// rounding error of long fp32 sums near sqrt-like growth rather than linear in K.
__global__ __launch_bounds__(GT * GT) void general_kernel(Args a) {
    __shared__ float sa[GT][GT + 1];
    __shared__ float sb[GT][GT + 1];
    select_batch(a);
    const int tx = threadIdx.x, ty = threadIdx.y;
    const int64_t tiles_n = (a.N + GT - 1) / GT;
    const int64_t tiles_m = (a.M + GT - 1) / GT;
    const bool skip_product = (a.alpha == 0.0f);
    for (int64_t t = blockIdx.x; t < tiles_m * tiles_n; t += gridDim.x) {
        const int64_t i0 = (t / tiles_n) * GT, j0 = (t % tiles_n) * GT;
        const int64_t i = i0 + ty, j = j0 + tx;
        float acc = 0.0f;
        if (!skip_product) {
            for (int64_t k0 = 0; k0 < a.K; k0 += GT) {
                // sa[r][c] = op(A)(i0 + r, k0 + c); sb[r][c] = op(B)(k0 + r, j0 + c)
                {
                    const int64_t ai = i0 + ty, ak = k0 + tx;
                    float v = 0.0f;
                    if (ai < a.M && ak < a.K)
                        v = load_elem(a.A, a.dtype, a.transA ? ak * a.lda + ai : ai * a.lda + ak);
                    sa[ty][tx] = v;
                    const int64_t bk = k0 + ty, bj = j0 + tx;
                    float w = 0.0f;
                    if (bk < a.K && bj < a.N)
                        w = load_elem(a.B, a.dtype, a.transB ? bj * a.ldb + bk : bk * a.ldb + bj);
                    sb[ty][tx] = w;
                }
                __syncthreads();
                float s = 0.0f;
#pragma unroll
                for (int kk = 0; kk < GT; ++kk) s = fmaf(sa[ty][kk], sb[kk][tx], s);
                acc += s;
                __syncthreads();
            }
        }
        if (i < a.M && j < a.N) {
            const int64_t ci = i * a.ldc + j;
            const float c_in = (a.beta != 0.0f) ? load_elem(a.C, a.out_dtype, ci) : 0.0f;
            const float bj = a.bias ? load_elem(a.bias, a.bias_dtype, j) : 0.0f;
            store_elem(a.C, a.out_dtype, ci, epilogue_value(acc, a.alpha, a.beta, c_in, bj, a.act));
        }
    }
}

}  // namespace

const char* general_variant_name(int variant) {
    static const char* const names[kGeneralVariants] = {"general_16x16", "general_128x128x64_w2x2",
                                                        "general_f32_64x64x32_w2x2", "general_wavek_64x64x64_w4",
                                                        "general_wavek_16x64x64_w4"};
    return variant >= 0 && variant < kGeneralVariants ? names[variant] : nullptr;
}

bool general_variant_supports(const Args& a, int variant) {
    if (variant == 0) return true;
    if (variant < 0 || variant >= kGeneralVariants) return false;
    if ((a.dtype == DT_F32) != (variant == 2) || a.M < 1 || a.N < 1 || a.K < 1) return false;
    const uintptr_t off = a.dtype == DT_F32 ? 3 : 1;                    // elements at their natural alignment
    if (((uintptr_t)a.A & off) || ((uintptr_t)a.B & off)) return false;
    // 32-bit byte offsets inside a slab, a 32-bit workgroup count
    if (a.lda > (1 << 22) || a.ldb > (1 << 22) || a.K > (1 << 30)) return false;
    if (((a.M + 63) / 64) * ((a.N + 63) / 64) > (int64_t)1 << 30) return false;
    // the wave tiles' movers start the last chunk of a row 8 elements ahead of its end and mask with an offset of 2 GiB - 16; a k-row of
    // 16 elements of an A stored K x M is no whole line
    if (variant >= kGeneralWave64) {
        if (((!a.transA || a.transB) && a.K < 8) || (variant == kGeneralWave16 && a.transA)) return false;
        if ((a.transA ? a.K : a.M) * a.lda * 2 >= 0x7ffffff0ll || (a.transB ? a.N : a.K) * a.ldb * 2 >= 0x7ffffff0ll) return false;
    }
    // the 16-bit mover of an m/n-contiguous operand fetches eight rows at a time
    return a.dtype == DT_F32 || ((!a.transA || a.M >= 8) && (a.transB || a.N >= 8));
}

hipError_t launch_general(const Args& a, int variant, int group_m, hipStream_t stream, bool fold, int64_t slice_len) {
    if (!general_variant_supports(a, variant)) return hipErrorInvalidValue;
    if (variant == 1) return launch_any_tile(a, group_m, stream, slice_len, fold);
    if (variant == 2) return launch_any_f32_tile(a, group_m, stream, slice_len);
    if (variant >= kGeneralWave64) return launch_wave_any(a, variant == kGeneralWave16 ? 16 : 64, group_m, stream);
    const int64_t tiles = ((a.M + GT - 1) / GT) * ((a.N + GT - 1) / GT);
    if (tiles == 0) return hipSuccess;
    const int64_t grid = tiles < (1 << 20) ? tiles : (1 << 20);
    hipLaunchKernelGGL(general_kernel, dim3((unsigned)grid, (unsigned)a.batch), dim3(GT, GT), 0, stream, a);
    return hipGetLastError();
}

}  // namespace gemm
