// fp32 tiles of 32x32 and 16x32 whose k range is divided among the eight waves of the workgroup (gfx950), for calls whose grid
// of 64x64 tiles leaves compute units idle.
//
// Such a call is bound by one workgroup's chain: launch, first slab, a barrier per slab of 32 (0.57 us of which 0.2 are work,
// 64x64 alone on its unit), sums, stores, and a second launch where slices are to shorten it.  Here each wave computes the
// whole small tile over every eighth slab: it loads its slabs into LDS as they are (fp32), takes the fragments apart in
// registers, each element once in the workgroup, and waits for nobody; the eight sums are added once.  Per slab and wave 208
// vector instructions take the four fragments of a 32x32 tile apart for 24 matrix instructions: the vector ALUs bound it, 2
// waves to a SIMD filling each other's waits, at 0.0046 us per element of k alone on a unit.  The code that runs once is short
// on purpose (8 KB; a first form with 64x64 tiles and 20 KB took 6.6 us for one slab where this takes 4): a wave waits for the
// instruction cache for all of it. The products and their order, the scale and the way out for what overflows are those of
// tile_f32_kernel.hpp; every slab is summed by itself and added by the vector ALUs, so the error is a third to a tenth (256^3
// 2.3e-7 -> 7.0e-8, 64x460x1152 5.2e-7 -> 8.9e-8 of the result's norm). Measured, the 64x64 tiles (in slices where it was so) /
// these, us: 256^3 8.2 / 7.2 (the rate of launches), 512^3 10.5 / 7.0, 64x460x1152 23.7 / 7.6, 268x228x3592 TN 69 / 18,
// 16x1024x1024 9.9 / 7.2, 64x1800x3008 15.7 / 15.2, 1024^3 24.1 to 25.3 / 25.6.
#pragma once
#include "tile_f32_kernel.hpp"
#include "tile_wavek_kernel.hpp"

namespace gemm {
namespace tile {

constexpr uint32_t kPastSlab = 0x7ffffff0u;      // past the end of any slab's descriptor, which starts at the slab and ends there at the latest

template <int ROWS>
struct WaveKF32 {
    static constexpr int BM = ROWS, BN = 32, BK = 32, WAVES = 8, NT = WAVES * 64;
    static constexpr int TM = BM / 16, TN = BN / 16;
    static constexpr int A_SLAB = BM * BK * 4, SLAB = A_SLAB + BN * BK * 4;      // bytes, of one wave
    static constexpr int LDS_BYTES = WAVES * SLAB;
    static_assert(BM * BN * 4 <= SLAB, "a wave parks its sums where its slab was");
};

// k-contiguous operand: a slab is rows of 128 bytes, chunk c (four k) of row r at r*128 + (c xor hash(r))*16; a fragment, 8
// consecutive k of a row per lane, is two chunks.  (The placement of the 16-bit tiles, and no more free of conflicts: 0.30 to
// 0.41 of the active LDS cycles.)
template <int ROWS>
struct WaveKCF32 {
    static constexpr int L = ROWS / 8;
    uint32_t voff[L];
    static __device__ __forceinline__ uint32_t chunk(int q, int lane) { return (uint32_t)(lane & 7) ^ WaveKC<64>::hash((uint32_t)(8 * q + (lane >> 3))); }
    __device__ __forceinline__ void init(int lane, int64_t ld, int valid_rows) {
        const uint32_t ld_bytes = (uint32_t)ld * 4;
#pragma unroll
        for (int q = 0; q < L; ++q) {
            const int row = 8 * q + (lane >> 3);
            const int rc = row < valid_rows ? row : valid_rows - 1;      // rows past the edge re-read a valid row and are never stored
            voff[q] = (uint32_t)rc * ld_bytes + chunk(q, lane) * 16;
        }
    }
    // for a slab of which `k_left` < 32 elements are inside K: the chunks behind them are fetched as zeros
    __device__ __forceinline__ void mask(int lane, int k_left) {
#pragma unroll
        for (int q = 0; q < L; ++q)
            if ((int)chunk(q, lane) * 4 >= k_left) voff[q] = kPastSlab;
    }
    static __device__ __forceinline__ const char* tile_base(const void* p, int64_t first_row, int64_t ld) { return (const char*)p + first_row * ld * 4; }
    static __device__ __forceinline__ int64_t k_step_bytes(int64_t /*ld*/) { return 128; }
    static __device__ __forceinline__ int64_t total_bytes(int64_t rows, int64_t K, int64_t ld) { return ((rows - 1) * ld + K) * 4; }

    struct Raw { u32x4 q[2]; };
    static constexpr int ADDRESSES = 2;
    static __device__ __forceinline__ uint32_t address(int half, int lane) {
        const uint32_t r = lane & 15, g = lane >> 4;
        return r * 128 + (((2 * g + (uint32_t)half) ^ WaveKC<64>::hash(r)) << 4);
    }
    template <int TILE>
    static __device__ __forceinline__ void read(const uint32_t (&addr)[ADDRESSES], Raw& r) {
        asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(r.q[0]) : "v"(addr[0]), "n"(TILE * 2048));
        asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(r.q[1]) : "v"(addr[1]), "n"(TILE * 2048));
    }
    static __device__ __forceinline__ void wait(Raw& r) { asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(r.q[0]), "+v"(r.q[1])); }
    template <int E> static __device__ __forceinline__ float get(const Raw& r) { return __uint_as_float(r.q[E / 4][E % 4]); }
};

// m- or n-contiguous operand: k-row 8g + e of a slab at position 4e + g, so that the four lane groups of a fragment read (g = 0 .. 3)
// find theirs side by side; with 32 columns the two halves of a row change places for g = 2 and 3, and the four 64-byte
// pieces fall on different quarters of a bank line.
template <int ROWS>
struct WaveMCF32 {
    static constexpr int L = ROWS / 8, ROW = ROWS * 4, PER_LOAD = 1024 / ROW, LANES = 64 / PER_LOAD;      // bytes of a k-row; k-rows of a load, lanes of a k-row
    static_assert(ROWS == 16 || ROWS == 32, "a half or a whole line");
    uint32_t voff[L];
    static __device__ __forceinline__ uint32_t position(int q, int lane) { return (uint32_t)(q * PER_LOAD + lane / LANES); }
    static __device__ __forceinline__ int row_of(int q, int lane) { return (int)(8 * (position(q, lane) & 3) + (position(q, lane) >> 2)); }
    __device__ __forceinline__ void init(int lane, int64_t ld, int valid_rows) {
        const uint32_t ld_bytes = (uint32_t)ld * 4;
#pragma unroll
        for (int q = 0; q < L; ++q) {
            const uint32_t c = (uint32_t)(lane % LANES) ^ (ROWS == 32 ? ((position(q, lane) & 2) << 1) : 0u);
            const uint32_t c4 = (int)(c * 4 + 4) <= valid_rows ? c * 4 : (uint32_t)(valid_rows - 4);      // past the edge: the last valid chunk, never stored
            voff[q] = (uint32_t)row_of(q, lane) * ld_bytes + c4 * 4;
        }
    }
    __device__ __forceinline__ void mask(int lane, int k_left) {
#pragma unroll
        for (int q = 0; q < L; ++q)
            if (row_of(q, lane) >= k_left) voff[q] = kPastSlab;
    }
    static __device__ __forceinline__ const char* tile_base(const void* p, int64_t first_row, int64_t /*ld*/) { return (const char*)p + first_row * 4; }
    static __device__ __forceinline__ int64_t k_step_bytes(int64_t ld) { return 128 * ld; }
    static __device__ __forceinline__ int64_t total_bytes(int64_t rows, int64_t K, int64_t ld) { return ((K - 1) * ld + rows) * 4; }

    struct Raw { u32x2 q[4]; };
    static constexpr int ADDRESSES = 2;
    static __device__ __forceinline__ uint32_t address(int tile, int lane) {
        const uint32_t r = lane & 15, g = lane >> 4;
        return g * ROW + (ROWS == 32 ? (((uint32_t)tile ^ (g >> 1)) << 6) : 0u) + r * 4;
    }
    template <int TILE>
    static __device__ __forceinline__ void read(const uint32_t (&addr)[ADDRESSES], Raw& r) {
        constexpr int S = ROW / 64;      // 256-byte steps from e to e + 1
        asm volatile("ds_read2st64_b32 %0, %1 offset0:%2 offset1:%3" : "=v"(r.q[0]) : "v"(addr[TILE]), "n"(0), "n"(S));
        asm volatile("ds_read2st64_b32 %0, %1 offset0:%2 offset1:%3" : "=v"(r.q[1]) : "v"(addr[TILE]), "n"(2 * S), "n"(3 * S));
        asm volatile("ds_read2st64_b32 %0, %1 offset0:%2 offset1:%3" : "=v"(r.q[2]) : "v"(addr[TILE]), "n"(4 * S), "n"(5 * S));
        asm volatile("ds_read2st64_b32 %0, %1 offset0:%2 offset1:%3" : "=v"(r.q[3]) : "v"(addr[TILE]), "n"(6 * S), "n"(7 * S));
    }
    static __device__ __forceinline__ void wait(Raw& r) { asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(r.q[0]), "+v"(r.q[1]), "+v"(r.q[2]), "+v"(r.q[3])); }
    template <int E> static __device__ __forceinline__ float get(const Raw& r) { return __uint_as_float(r.q[E / 2][E % 2]); }
};

struct Pieces { u32x4 hi, mid, lo; };

// eight elements times `scale`, taken apart (see tile_f32_kernel.hpp)
template <class L>
__device__ __forceinline__ void wavek_split(const typename L::Raw& r, float scale, Pieces& p) {
    static_for<4>([&](auto d) {
        constexpr int i = decltype(d)::value;
        float x = L::template get<2 * i>(r) * scale, y = L::template get<2 * i + 1>(r) * scale;
        const uint32_t h = pack_bf16(x, y);
        x -= low_bf16(h);
        y -= high_bf16(h);
        const uint32_t m = pack_bf16(x, y);
        x -= low_bf16(m);
        y -= high_bf16(m);
        p.hi[i] = h;
        p.mid[i] = m;
        p.lo[i] = pack_bf16(x, y);
    });
}

template <class C, bool A_KC, bool B_KC>
__global__ __launch_bounds__(C::NT, 4) void tile_wavek_f32_kernel(Args a, int tiles_m, int tiles_n, int group_m) {
    constexpr int TM = C::TM, TN = C::TN;
    __shared__ __attribute__((aligned(1024))) char lds[C::LDS_BYTES];
    __shared__ uint32_t beyond[C::WAVES];
    select_batch(a);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int tm, tn;
    tile_of_workgroup(blockIdx.x, tiles_m, tiles_n, group_m, tm, tn);
    const int64_t m0 = (int64_t)tm * C::BM, n0 = (int64_t)tn * C::BN;
    const int K = (int)a.K, slabs = (K + C::BK - 1) / C::BK;

    using LA = typename std::conditional<A_KC, WaveKCF32<C::BM>, WaveMCF32<C::BM>>::type;
    using LB = typename std::conditional<B_KC, WaveKCF32<C::BN>, WaveMCF32<C::BN>>::type;
    const char* const pa = LA::tile_base(a.A, m0, a.lda);
    const char* const pb = LB::tile_base(a.B, n0, a.ldb);
    const int64_t a_step = LA::k_step_bytes(a.lda), b_step = LB::k_step_bytes(a.ldb);
    const int64_t a_bytes = LA::total_bytes(a.M, a.K, a.lda) - (pa - (const char*)a.A);
    const int64_t b_bytes = LB::total_bytes(a.N, a.K, a.ldb) - (pb - (const char*)a.B);

    char* const slab = lds + wave * C::SLAB;
    const uint32_t slab_at = (uint32_t)(uintptr_t)GEMM_LDS_PTR(slab);
    uint32_t fa[LA::ADDRESSES], fb[LB::ADDRESSES];
#pragma unroll
    for (int i = 0; i < LA::ADDRESSES; ++i) fa[i] = slab_at + LA::address(i, lane);
#pragma unroll
    for (int j = 0; j < LB::ADDRESSES; ++j) fb[j] = slab_at + C::A_SLAB + LB::address(j, lane);

    RawBias bias;      // (asked for ahead of the k loop: behind it the loads would be a trip to memory more)
    ask_bias(a, n0 + 4 * (lane & 7), bias);
    f32x4 acc[TM][TN];

    // The slabs of this wave, every eighth from `wave` on: `multiply` gets the elements as they lie in LDS.  The first trip only
    // asks (the code is there once).
    auto for_my_slabs = [&](auto&& multiply) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        LA la;
        LB lb;
        la.init(lane, a.lda, (int)(a.M - m0 < C::BM ? a.M - m0 : C::BM));
        lb.init(lane, a.ldb, (int)(a.N - n0 < C::BN ? a.N - n0 : C::BN));
#pragma unroll 1
        for (int t = wave - C::WAVES; t < slabs; t += C::WAVES) {
            typename LA::Raw ar[TM];
            typename LB::Raw br[TN];
            if (t >= 0) {
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                static_for<TN>([&](auto j) { LB::template read<decltype(j)::value>(fb, br[decltype(j)::value]); });
                static_for<TM>([&](auto i) { LA::template read<decltype(i)::value>(fa, ar[decltype(i)::value]); });
#pragma unroll
                for (int j = 0; j < TN; ++j) LB::wait(br[j]);
#pragma unroll
                for (int i = 0; i < TM; ++i) LA::wait(ar[i]);
            }
            const int next = t + C::WAVES, k_left = K - next * C::BK;
            if (k_left > 0) {
                if (k_left < C::BK) {      // (the last slab that this wave asks for)
                    la.mask(lane, k_left);
                    lb.mask(lane, k_left);
                }
                const int64_t left_a = a_bytes - next * a_step, left_b = b_bytes - next * b_step;
                const __amdgpu_buffer_rsrc_t ra = make_rsrc(pa + next * a_step, left_a < kPastSlab ? left_a : kPastSlab),
                                             rb = make_rsrc(pb + next * b_step, left_b < kPastSlab ? left_b : kPastSlab);
#pragma unroll
                for (int q = 0; q < LA::L; ++q) load_to_lds_b128(ra, slab + q * 1024, la.voff[q], 0);
#pragma unroll
                for (int q = 0; q < LB::L; ++q) load_to_lds_b128(rb, slab + C::A_SLAB + q * 1024, lb.voff[q], 0);
            }
            if (t >= 0) multiply(ar, br);
        }
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    };
    // every wave's sums where its slab was, chunk c of row r at place c xor (r mod 8)
    auto park = [&]() {
        const int r = lane & 15, g = lane >> 4;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) *(f32x4*)(slab + (16 * i + r) * 128 + (((4 * j + g) ^ (r & 7)) << 4)) = acc[i][j];
        __syncthreads();
    };

    for_my_slabs([&](const typename LA::Raw (&ar)[TM], const typename LB::Raw (&br)[TN]) {
        Pieces pb[TN];
#pragma unroll
        for (int j = 0; j < TN; ++j) wavek_split<LB>(br[j], kSplitScale, pb[j]);
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            Pieces pa;
            wavek_split<LA>(ar[i], kSplitScale, pa);
            f32x4 t[TN];
#define GEMM_WAVEK_STEP(PA, PB, FROM) _Pragma("unroll") for (int j = 0; j < TN; ++j) t[j] = wavek_mfma<true>(pb[j].PB, pa.PA, FROM)
            GEMM_WAVEK_STEP(lo, hi, (f32x4{0.0f, 0.0f, 0.0f, 0.0f}));
            GEMM_WAVEK_STEP(hi, lo, t[j]);
            GEMM_WAVEK_STEP(mid, mid, t[j]);
            GEMM_WAVEK_STEP(mid, hi, t[j]);
            GEMM_WAVEK_STEP(hi, mid, t[j]);
            GEMM_WAVEK_STEP(hi, hi, t[j]);
#undef GEMM_WAVEK_STEP
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[i][j] += t[j];
        }
    });

    // Whatever overflowed in the scaled split is not finite any more, and the eight sums together must stay finite too.
    uint32_t largest = 0;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const uint32_t magnitude = __float_as_uint(acc[i][j][v]) & 0x7fffffffu;
                largest = magnitude > largest ? magnitude : largest;
            }
    const bool mine = __builtin_amdgcn_ballot_w64(largest >= __float_as_uint(0x1p123f)) != 0;
    if (lane == 0) beyond[wave] = mine;
    park();
    float unscale = kSplitUnscale;
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(lane < C::WAVES && beyond[lane & (C::WAVES - 1)] != 0) != 0, 0)) {
        __syncthreads();      // (nobody reads the flags or the sums any more)
        unscale = 1.0f;
        for_my_slabs([&](const typename LA::Raw (&ar)[TM], const typename LB::Raw (&br)[TN]) {
            static_for<8>([&](auto e) {      // (the order of k is free as long as both operands agree)
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(LB::template get<decltype(e)::value>(br[j]), LA::template get<decltype(e)::value>(ar[i]),
                                                                         acc[i][j], 0, 0, 0);
            });
        });
        park();
    }

    // The sums of the eight waves, added in their order, and the epilogue: eight rows to a wave, four columns to a lane.
    const int rr = lane >> 3, cc = lane & 7, r = 8 * wave + rr;
    const int64_t row = m0 + r, col = n0 + 4 * cc;
    if (r >= C::BM || row >= a.M || col >= a.N) return;
    const char* const at = lds + r * 128 + ((cc ^ (r & 7)) << 4);
    f32x4 o[1] = {*(const f32x4*)at};
#pragma unroll
    for (int w = 1; w < C::WAVES; ++w) o[0] += *(const f32x4*)(at + w * C::SLAB);
    o[0] = a.alpha * (unscale * o[0]);
    float* const p = (float*)a.C + row * a.ldc + col;
    const int columns = a.N - col < 4 ? (int)(a.N - col) : 4;
    if (a.beta != 0.0f) {
        f32x4 c;
        if (columns == 4) c = OutVec<DT_F32>::load4(p);
        else {
#pragma unroll
            for (int e = 0; e < 4; ++e) c[e] = p[e < columns ? e : 0];
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) o[0][e] = fmaf(a.beta, c[e], o[0][e]);
    }
    o[0] += bias_values(a, bias);
    if (a.act != ACT_NONE) apply_act4(o, a.act);
    if (columns == 4) {
        OutVec<DT_F32>::store4(p, o[0]);
    } else {
#pragma unroll
        for (int e = 0; e < 3; ++e)
            if (e < columns) p[e] = o[0][e];
    }
}

template <class C>
hipError_t launch_wavek_f32(const Args& a, int group_m, hipStream_t stream) {
    const int tiles_m = (int)((a.M + C::BM - 1) / C::BM), tiles_n = (int)((a.N + C::BN - 1) / C::BN);
    const dim3 grid((unsigned)(tiles_m * tiles_n), (unsigned)a.batch), block(C::NT);
    const bool akc = !a.transA, bkc = a.transB != 0;
#define GEMM_TILE_LAUNCH(AKC, BKC) hipLaunchKernelGGL((tile_wavek_f32_kernel<C, AKC, BKC>), grid, block, 0, stream, a, tiles_m, tiles_n, group_m)
    if (akc && bkc) GEMM_TILE_LAUNCH(true, true);
    else if (akc && !bkc) GEMM_TILE_LAUNCH(true, false);
    else if (!akc && bkc) GEMM_TILE_LAUNCH(false, true);
    else GEMM_TILE_LAUNCH(false, false);
#undef GEMM_TILE_LAUNCH
    return hipGetLastError();
}

}  // namespace tile
}  // namespace gemm
