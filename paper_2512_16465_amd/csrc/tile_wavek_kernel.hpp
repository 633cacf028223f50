// Tiles of 64x64 and 16x64 whose k range is divided among the waves of the workgroup (bf16 / fp16, gfx950), for calls whose
// grid of 128x128 tiles leaves compute units idle.
//
// Such a call is bound by what one workgroup takes: the way of its operands from the L2 into LDS (about 50 bytes per clock and
// unit) and, with a few dozen slabs of k, the time from the launch to the first product and from the last one to the stores.  A
// 128x128 tile on 4 waves that share every slab walks k at 0.0066 us per element alone on its unit (two barriers' worth of
// waiting per 32 elements; its LDS traffic, 12 clocks per element, is above the 8 of its products) and needs 11 us around it,
// and dividing its k range over workgroups costs a second launch.  Here a wave computes the whole tile over every fourth slab
// of 64: it loads its own slabs into its own ring, waits for nobody, and the four sums are added through LDS once, at the end.
// A tile of 64x64 reads half as many bytes per element as one of 128x128, 0.0026 us each, and four times as many units work on
// it; with 16 rows 0.0013 us. Two workgroups share a unit (64 KiB of LDS with one slab per wave, 80 KiB with two of the 16-row
// tile), one waits while the other multiplies.  Slabs of 64 are whole 128-byte lines of a k-contiguous operand, and of an
// m/n-contiguous one.
//
// Measured, the 128x128 tiles (whole, or divided over workgroups and a second launch) / these, us: 832x512x768 12.3 / 8.2 (the
// rate of launches from Python), 145x4864x2816 17.5 / 12.3, 960x2048x1280 19.1 / 13.0, 1024x1024x2048 18.2 / 10.6, 104x560x1768
// 12.6 / 8.3, 896x896x6592 TN 23.4 / 23; 16 rows: 48x1024x4096 14.4 / 9.3, 256x512x4864 15.7 / 11.5, 15x16128x2048 17.1 / 12.8.
// Tried: 128x64 (one workgroup per unit: behind the other tiles everywhere), 32x64 (at most 14 % ahead on a few shapes), two
// slabs per wave and one workgroup per unit with 64x64 (up to 16 % ahead at k beyond 4000 with under 100 tiles, half the speed
// beyond 256 tiles).
#pragma once
#include "tile_dma16_kernel.hpp"
#include "tile_f32_kernel.hpp"

namespace gemm {
namespace tile {

// ROWS x 64 tile, 64 of k per slab and wave, NS places for slabs per wave.  WGS: workgroups that share a unit.
// ANY: operands off the 16-byte grid.
template <int ROWS, int NS_, int WGS_, bool ANY_ = false>
struct WaveK {
    static constexpr bool ANY = ANY_;
    static_assert(!ANY || NS_ == 1, "the registers hold the slab behind");
    static constexpr int BM = ROWS, BN = 64, BK = 64, WAVES = 4, NT = WAVES * 64, NS = NS_, WGS = WGS_;
    static constexpr int TM = BM / 16;                                                        // blocks of 16 rows
    static constexpr int A_SLAB = BM * BK * 2, SLAB = A_SLAB + BN * BK * 2, RING = NS * SLAB;      // bytes, of one wave
    static constexpr int LDS_BYTES = WAVES * RING;
    static constexpr int LOADS = SLAB / 1024;      // direct-to-LDS loads per slab and wave
    static_assert(LDS_BYTES * WGS <= 160 * 1024, "the workgroups of a unit share its LDS");
    static_assert(BM * BN * 4 <= RING, "a wave parks its sums in its own ring");
};

// k-contiguous operand: a slab is 64 rows of 128 bytes (whole cache lines); 16-byte chunk c of row r at r*128 + (c xor
// hash(r))*16. The hash puts the 16 rows that 16 consecutive lanes read on 16 distinct places of a 256-byte bank line.  Those
// lanes are not the ones served together: 0.33 to 0.48 of the active LDS cycles are conflicts with both operands k-contiguous
// (0.16 to 0.29 with one; the quartered kernel, whose rows of 64 bytes are placed otherwise, 0.04), so a fragment read takes
// about two turns.
template <int ROWS>
struct WaveKC {
    static constexpr int L = ROWS / 8;
    static __device__ __forceinline__ uint32_t hash(uint32_t r) { return (r ^ ((r >> 3) & 1u)) & 7u; }
    uint32_t voff[L];
    __device__ __forceinline__ void init(int lane, int64_t ld, int valid_rows) {
        const uint32_t ld_bytes = (uint32_t)ld * 2;
#pragma unroll
        for (int q = 0; q < L; ++q) {
            const int row = 8 * q + (lane >> 3);
            const int rc = row < valid_rows ? row : valid_rows - 1;      // rows past the edge re-read a valid row and are never stored
            voff[q] = (uint32_t)rc * ld_bytes + chunk(q, lane) * 16;
        }
    }
    static __device__ __forceinline__ uint32_t chunk(int q, int lane) { return (uint32_t)(lane & 7) ^ hash((uint32_t)(8 * q + (lane >> 3))); }
    // for a slab of which `k_left` < 64 elements are inside K: the chunks behind them are fetched as zeros
    __device__ __forceinline__ void mask(int lane, int k_left) {
#pragma unroll
        for (int q = 0; q < L; ++q)
            if ((int)chunk(q, lane) * 8 >= k_left) voff[q] = 0x7ffffff0u;
    }
    static __device__ __forceinline__ const char* tile_base(const void* p, int64_t first_row, int64_t ld) { return (const char*)p + first_row * ld * 2; }
    static __device__ __forceinline__ int64_t k_step_bytes(int64_t /*ld*/) { return 128; }
    static __device__ __forceinline__ int64_t total_bytes(int64_t rows, int64_t K, int64_t ld) { return ((rows - 1) * ld + K) * 2; }

    typedef Frag16RawKC Raw;
    static constexpr int ADDRESSES = 2;      // one per 32 of k
    static __device__ __forceinline__ uint32_t address(int ks, int lane) {
        const uint32_t r = lane & 15, g = lane >> 4;
        return r * 128 + ((((uint32_t)ks * 4 + g) ^ hash(r)) << 4);
    }
    // fragment of the 16 rows of block TILE, k 32*KS .. +31
    template <int TILE, int KS>
    static __device__ __forceinline__ void read(const uint32_t (&addr)[ADDRESSES], uint32_t slab, Raw& r) {
        asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(r.q) : "v"(addr[KS] + slab), "n"(TILE * 2048));
    }
};

// m- or n-contiguous operand: a slab is 64 k-rows of 128 bytes; chunk c (8 columns) of k-row k at k*128 + (c xor swizzle(k))*16.  A
// transposing read takes 32 bytes from each of four consecutive k-rows per 16 lanes; 32 lanes (k-rows 0-3 and 8-11 of a
// block) are served together and fall on distinct places: two rows per 256-byte bank line, bits 1 and 3 of k spread the others.
template <int ROWS>
struct WaveMC {
    static constexpr int L = 8;
    static_assert(ROWS == 64, "a whole line of a k-row");
    static __device__ __forceinline__ uint32_t swizzle(uint32_t k) { return (k & 2u) | (((k >> 3) & 1u) << 2); }
    uint32_t voff[L];
    __device__ __forceinline__ void init(int lane, int64_t ld, int valid_rows) {
        const uint32_t ld_bytes = (uint32_t)ld * 2;
#pragma unroll
        for (int q = 0; q < L; ++q) {
            const uint32_t k = 8 * q + (lane >> 3);
            const uint32_t c = (uint32_t)(lane & 7) ^ swizzle(k);
            const uint32_t c8 = (int)(c * 8 + 8) <= valid_rows ? c * 8 : (uint32_t)(valid_rows - 8);      // past the edge: the last valid chunk, never stored
            voff[q] = k * ld_bytes + c8 * 2;
        }
    }
    __device__ __forceinline__ void mask(int lane, int k_left) {
#pragma unroll
        for (int q = 0; q < L; ++q)
            if (8 * q + (lane >> 3) >= k_left) voff[q] = 0x7ffffff0u;
    }
    static __device__ __forceinline__ const char* tile_base(const void* p, int64_t first_row, int64_t /*ld*/) { return (const char*)p + first_row * 2; }
    static __device__ __forceinline__ int64_t k_step_bytes(int64_t ld) { return 128 * ld; }
    static __device__ __forceinline__ int64_t total_bytes(int64_t rows, int64_t K, int64_t ld) { return ((K - 1) * ld + rows) * 2; }

    typedef Frag16RawMC Raw;
    static constexpr int ADDRESSES = 4;      // one per block (the swizzle reaches the block's bits)
    static __device__ __forceinline__ uint32_t address(int tile, int lane) {
        const uint32_t j = lane & 15, g = lane >> 4;
        const uint32_t k = 8 * g + (j >> 2), col = 16 * tile + 4 * (j & 3);
        return k * 128 + (((col >> 3) ^ swizzle(k)) << 4) + (col & 7) * 2;
    }
    template <int TILE, int KS>
    static __device__ __forceinline__ void read(const uint32_t (&addr)[ADDRESSES], uint32_t slab, Raw& r) {
        asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(r.lo) : "v"(addr[TILE] + slab), "n"(KS * 4096));
        asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(r.hi) : "v"(addr[TILE] + slab), "n"(KS * 4096 + 512));
    }
};

// Waits for every LDS read and names the fragments that it has brought.
__device__ __forceinline__ void wait_frags(Frag16RawKC (&r)[1]) { asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(r[0].q)); }
template <class Raw>
__device__ __forceinline__ void wait_frags(Raw (&r)[4]) { wait_raw8(r); }

template <bool IS_BF16>
__device__ __forceinline__ f32x4 wavek_mfma(u32x4 a, u32x4 b, f32x4 c) {
    if constexpr (IS_BF16) return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    else return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}

// ---- the same operands off the 16-byte grid: through registers, to the same places in LDS ----
// A 16-byte buffer load takes any element's address.  Chunks that would cross the end of a row are loaded from 8 elements ahead of the
// end and moved down by `s` elements (wave-uniform), so that nothing outside the operand is ever asked for.

__device__ __forceinline__ u32x4 drop_elements(u32x4 v, int s) {
    if (s & 1) {
        v.x = __builtin_amdgcn_alignbit(v.y, v.x, 16);
        v.y = __builtin_amdgcn_alignbit(v.z, v.y, 16);
        v.z = __builtin_amdgcn_alignbit(v.w, v.z, 16);
        v.w >>= 16;
    }
    if (s & 2) v = u32x4{v.y, v.z, v.w, 0u};
    if (s & 4) v = u32x4{v.z, v.w, 0u, 0u};
    return v;
}

template <int ROWS>
struct WaveAnyKC : WaveKC<ROWS> {
    using Base = WaveKC<ROWS>;
    u32x4 r[Base::L];
    static __device__ __forceinline__ const char* tile_base(const void* p, int64_t first_row, int64_t ld) { return Base::tile_base(p, first_row, ld); }
    __device__ __forceinline__ void init(int lane, int64_t ld, int64_t /*first_row*/, int valid_rows) { Base::init(lane, ld, valid_rows); }
    // slab `t`; `bytes`: from `base` to the end of the operand
    __device__ __forceinline__ void load(const char* base, int64_t bytes, int64_t step, int t, int k_left, int lane) {
        if (k_left >= 64) {
            const __amdgpu_buffer_rsrc_t rsrc = make_rsrc(base, bytes);
#pragma unroll
            for (int q = 0; q < Base::L; ++q) r[q] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, Base::voff[q], (uint32_t)(t * step), 0);
            return;
        }
        // the last slab: the chunk with the row's last element in it, zeros behind it (the matrix has at least 8 k, so only a later
        // slab than the first can start a load ahead of itself)
        const int s = -k_left & 7, ahead = t > 0 ? 16 : 0;
        const __amdgpu_buffer_rsrc_t rsrc = make_rsrc(base + t * step - ahead, bytes - t * step + ahead);
#pragma unroll
        for (int q = 0; q < Base::L; ++q) {
            const int k = (int)Base::chunk(q, lane) * 8;
            const uint32_t off = Base::voff[q] + (uint32_t)(ahead - (k + 8 > k_left ? 2 * s : 0));
            r[q] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, k < k_left ? off : 0x7ffffff0u, 0, 0);
        }
        if (s) {
#pragma unroll
            for (int q = 0; q < Base::L; ++q) {
                const int k = (int)Base::chunk(q, lane) * 8;
                const u32x4 moved = drop_elements(r[q], s);
                r[q] = k + 8 > k_left ? moved : r[q];
            }
        }
    }
    __device__ __forceinline__ void store(char* slab, int lane) const {
#pragma unroll
        for (int q = 0; q < Base::L; ++q) *(u32x4*)(slab + q * 1024 + lane * 16) = r[q];
    }
};

template <int ROWS>
struct WaveAnyMC : WaveMC<ROWS> {
    using Base = WaveMC<ROWS>;
    static_assert(ROWS == 64, "one sub-slab");
    u32x4 r[Base::L];
    int edge;      // columns of the tile inside the operand where they end inside a chunk, 0: they do not
    // the base of a later tile is 8 columns ahead of it
    static __device__ __forceinline__ const char* tile_base(const void* p, int64_t first_row, int64_t /*ld*/) {
        return (const char*)p + (first_row - (first_row > 0 ? 8 : 0)) * 2;
    }
    __device__ __forceinline__ void init(int lane, int64_t ld, int64_t first_row, int valid_rows) {
        const int ahead = first_row > 0 ? 8 : 0;
        const uint32_t ld_bytes = (uint32_t)ld * 2;
        edge = valid_rows & 7 ? valid_rows : 0;
#pragma unroll
        for (int q = 0; q < Base::L; ++q) {
            const uint32_t k = 8 * q + (lane >> 3);
            const int c8 = (int)((uint32_t)(lane & 7) ^ Base::swizzle(k)) * 8;
            Base::voff[q] = k * ld_bytes + (uint32_t)((c8 + 8 <= valid_rows ? c8 : valid_rows - 8) + ahead) * 2;
        }
    }
    __device__ __forceinline__ void load(const char* base, int64_t bytes, int64_t step, int t, int k_left, int lane) {
        const __amdgpu_buffer_rsrc_t rsrc = make_rsrc(base, bytes);
        if (k_left < 64) Base::mask(lane, k_left);      // (the last slab that this wave asks for)
#pragma unroll
        for (int q = 0; q < Base::L; ++q) r[q] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, Base::voff[q], (uint32_t)(t * step), 0);
    }
    __device__ __forceinline__ void store(char* slab, int lane) {
        if (edge) {
            const int s = -edge & 7;
#pragma unroll
            for (int q = 0; q < Base::L; ++q) {
                const int c8 = (int)((uint32_t)(lane & 7) ^ Base::swizzle(8 * q + (lane >> 3))) * 8;
                const u32x4 moved = drop_elements(r[q], s);
                r[q] = c8 == (edge & ~7) ? moved : r[q];
            }
        }
#pragma unroll
        for (int q = 0; q < Base::L; ++q) *(u32x4*)(slab + q * 1024 + lane * 16) = r[q];
    }
};

// The sums of the waves are added in the order of the waves: every wave parks its own in its ring as rows of 16 chunks, chunk c
// of row r at place c xor (r mod 16), then adds its share of the rows.
template <int TM>
__device__ __forceinline__ void wavek_park(char* ring, const f32x4 (&acc)[TM][4], int lane) {
    const int r = lane & 15, g = lane >> 4;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) *(f32x4*)(ring + (16 * i + r) * 256 + (((4 * j + g) ^ r) << 4)) = acc[i][j];
}

// ... and the epilogue of those rows, four columns to a lane.  `unscale`: factor on the sums.  A wave runs this code once, and code run
// for the first time waits for the instruction cache, so what an activation takes is there once, for a row at a time, and a
// ragged edge goes element by element in a loop (all of it unrolled, bias and GELU cost a 512x512x256 call 5.5 us).
template <class C, int OUT>
__device__ __forceinline__ void wavek_finish(char* lds, const Args& a, int64_t m0, int64_t n0, int wave, int lane, const RawBias& bias, float unscale = 1.0f) {
    using OV = OutVec<OUT>;
    constexpr int SHARE = C::BM / C::WAVES, T = SHARE >= 4 ? SHARE / 4 : 1;      // rows of a wave; of a lane
    const int rr = lane >> 4, cc = lane & 15, first = SHARE * wave;
    const int64_t row0 = m0 + first + rr, col = n0 + 4 * cc;
    if ((SHARE < 4 && rr >= SHARE) || row0 >= a.M || col >= a.N) return;
    const int rows = a.M - row0 < 4 * T ? (int)(a.M - row0 + 3) / 4 : T;          // of this lane inside C
    const int columns = a.N - col < 4 ? (int)(a.N - col) : 4;
    const float alpha = a.alpha, beta = a.beta;
    typename OV::elem* const p0 = (typename OV::elem*)a.C + row0 * a.ldc + col;
    const int64_t step = 4 * a.ldc;
    const f32x4 bias4 = bias_values(a, bias);
    auto place = [&](int t) {
        const int r = first + 4 * t + rr;
        return lds + r * 256 + ((cc ^ (r & 15)) << 4);
    };
    auto sum = [&](int t) {
        const char* const at = place(t);
        f32x4 s = *(const f32x4*)at;
#pragma unroll
        for (int w = 1; w < C::WAVES; ++w) s += *(const f32x4*)(at + w * C::RING);
        return alpha * (unscale * s);
    };
    if (__builtin_amdgcn_ballot_w64(columns != 4) == 0) {
        f32x4 s[T], cin[T];
        if (beta != 0.0f) {
#pragma unroll
            for (int t = 0; t < T; ++t)
                if (t < rows) cin[t] = OV::load4(p0 + t * step);
        }
#pragma unroll
        for (int t = 0; t < T; ++t) s[t] = sum(t);
        if (beta != 0.0f) {
#pragma unroll
            for (int t = 0; t < T; ++t)
#pragma unroll
                for (int e = 0; e < 4; ++e) s[t][e] = fmaf(beta, cin[t][e], s[t][e]);
        }
#pragma unroll
        for (int t = 0; t < T; ++t) s[t] += bias4;
        if (a.act == ACT_NONE) {
#pragma unroll
            for (int t = 0; t < T; ++t)
                if (t < rows) OV::store4(p0 + t * step, s[t]);
            return;
        }
#pragma unroll
        for (int t = 0; t < T; ++t) *(f32x4*)place(t) = s[t];
#pragma unroll 1
        for (int t = 0; t < rows; ++t) {
            f32x4 o[1] = {*(const f32x4*)place(t)};
            apply_act4(o, a.act);
            OV::store4(p0 + t * step, o[0]);
        }
        return;
    }
#pragma unroll 1
    for (int t = 0; t < rows; ++t) {
        f32x4 o[1] = {sum(t)};
        typename OV::elem* const p = p0 + t * step;
        if (beta != 0.0f) {
            float c[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) c[e] = OV::load1(p + (e < columns ? e : 0));
#pragma unroll
            for (int e = 0; e < 4; ++e) o[0][e] = fmaf(beta, c[e], o[0][e]);
        }
        o[0] += bias4;
        if (a.act != ACT_NONE) apply_act4(o, a.act);
        if (columns == 4) {
            OV::store4(p, o[0]);
        } else {
#pragma unroll
            for (int e = 0; e < 3; ++e)
                if (e < columns) OV::store1(p + e, o[0][e]);
        }
    }
}

template <class C, bool IS_BF16, bool A_KC, bool B_KC>
__global__ __launch_bounds__(C::NT, C::WGS) void tile_wavek_kernel(Args a, int tiles_m, int tiles_n, int group_m) {
    __shared__ __attribute__((aligned(1024))) char lds[C::LDS_BYTES];
    select_batch(a);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int tm, tn;
    tile_of_workgroup(blockIdx.x, tiles_m, tiles_n, group_m, tm, tn);
    const int64_t m0 = (int64_t)tm * C::BM, n0 = (int64_t)tn * C::BN;
    const int K = (int)a.K, slabs = (K + C::BK - 1) / C::BK;

    using LA = typename std::conditional<C::ANY, typename std::conditional<A_KC, WaveAnyKC<C::BM>, WaveAnyMC<C::BM>>::type,
                                         typename std::conditional<A_KC, WaveKC<C::BM>, WaveMC<C::BM>>::type>::type;
    using LB = typename std::conditional<C::ANY, typename std::conditional<B_KC, WaveAnyKC<C::BN>, WaveAnyMC<C::BN>>::type,
                                         typename std::conditional<B_KC, WaveKC<C::BN>, WaveMC<C::BN>>::type>::type;
    LA la;
    LB lb;
    const int valid_m = (int)(a.M - m0 < C::BM ? a.M - m0 : C::BM), valid_n = (int)(a.N - n0 < C::BN ? a.N - n0 : C::BN);
    if constexpr (C::ANY) {
        la.init(lane, a.lda, m0, valid_m);
        lb.init(lane, a.ldb, n0, valid_n);
    } else {
        la.init(lane, a.lda, valid_m);
        lb.init(lane, a.ldb, valid_n);
    }
    const char* const pa = LA::tile_base(a.A, m0, a.lda);
    const char* const pb = LB::tile_base(a.B, n0, a.ldb);
    const int64_t a_step = LA::k_step_bytes(a.lda), b_step = LB::k_step_bytes(a.ldb);
    const int64_t a_bytes = LA::total_bytes(a.M, a.K, a.lda) - (pa - (const char*)a.A);
    const int64_t b_bytes = LB::total_bytes(a.N, a.K, a.ldb) - (pb - (const char*)a.B);

    char* const ring = lds + wave * C::RING;
    const uint32_t ring_at = (uint32_t)(uintptr_t)GEMM_LDS_PTR(ring);
    uint32_t fa[LA::ADDRESSES], fb[LB::ADDRESSES];
#pragma unroll
    for (int i = 0; i < LA::ADDRESSES; ++i) fa[i] = ring_at + LA::address(i, lane);
#pragma unroll
    for (int j = 0; j < LB::ADDRESSES; ++j) fb[j] = ring_at + C::A_SLAB + LB::address(j, lane);

    // Requests slab `t` of the call into place `p`.  A slab past the end is requested through descriptors of length zero: it
    // fetches nothing but counts like any other, so the waits below can be exact.
    auto request = [&](int t, int p) {
        const int k_left = K - t * C::BK;
        if constexpr (C::ANY) {
            if (k_left > 0) {
                la.load(pa, a_bytes, a_step, t, k_left, lane);
                lb.load(pb, b_bytes, b_step, t, k_left, lane);
            }
            return;
        } else {
            const __amdgpu_buffer_rsrc_t ra = make_rsrc(pa, k_left > 0 ? a_bytes : 0), rb = make_rsrc(pb, k_left > 0 ? b_bytes : 0);
            const uint32_t sa = (uint32_t)(t * a_step), sb = (uint32_t)(t * b_step);
            char* const dst = ring + p * C::SLAB;
            if (k_left > 0 && k_left < C::BK) {      // (the last slab that this wave asks for)
                la.mask(lane, k_left);
                lb.mask(lane, k_left);
            }
#pragma unroll
            for (int q = 0; q < LA::L; ++q) load_to_lds_b128(ra, dst + q * 1024, la.voff[q], sa);
#pragma unroll
            for (int q = 0; q < LB::L; ++q) load_to_lds_b128(rb, dst + C::A_SLAB + q * 1024, lb.voff[q], sb);
        }
    };

    RawBias bias;      // (asked for ahead of the k loop: behind it the loads would be a trip to memory more)
    ask_bias(a, n0 + 4 * (lane & 15), bias);
    constexpr int TM = C::TM;
    f32x4 acc[TM][4];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    typename LA::Raw af[2][TM];
    typename LB::Raw bf[2][4];
    auto read = [&](auto ks_c, uint32_t slab) {
        constexpr int ks = decltype(ks_c)::value;
        LA::template read<0, ks>(fa, slab, af[ks][0]);
        LB::template read<0, ks>(fb, slab, bf[ks][0]);
        LB::template read<1, ks>(fb, slab, bf[ks][1]);
        LB::template read<2, ks>(fb, slab, bf[ks][2]);
        LB::template read<3, ks>(fb, slab, bf[ks][3]);
        static_for<TM - 1>([&](auto i) { LA::template read<decltype(i)::value + 1, ks>(fa, slab, af[ks][decltype(i)::value + 1]); });
    };

    // Wave w takes slabs w, w + 4, ...; no wave waits for another before the sums are added.  The products of a slab are summed by
    // themselves and added by the vector ALUs, which rounds a sum half as often at full magnitude: an fp32 result is no further off
    // than from more and shorter sums (of 240 random calls with an fp32 C none but by chance, half the error in the
    // median), at no cost that could be measured.
    const int mine = slabs > wave ? (slabs - wave + C::WAVES - 1) / C::WAVES : 0;
#pragma unroll 1
    for (int i = -C::NS; i < mine; ++i) {      // (the first NS trips only ask: the code is there once)
        const int place = C::NS == 1 ? 0 : i & (C::NS - 1);
        if (i >= 0) {
            if constexpr (C::ANY) {
                la.store(ring, lane);
                lb.store(ring + C::A_SLAB, lane);
                asm volatile("" ::: "memory");      // (a wave's LDS operations take effect in their order)
            } else {
                asm volatile("s_waitcnt vmcnt(%0)" ::"n"((C::NS - 1) * C::LOADS) : "memory");
            }
            read(std::integral_constant<int, 0>{}, (uint32_t)(place * C::SLAB));
            read(std::integral_constant<int, 1>{}, (uint32_t)(place * C::SLAB));
            wait_frags(af[0]);
            wait_frags(bf[0]);
            wait_frags(af[1]);
            wait_frags(bf[1]);
        }
        request(wave + C::WAVES * (i + C::NS), place);
        if (i >= 0) {
#pragma unroll
            for (int m = 0; m < TM; ++m) {
                f32x4 t[4];      // (B's fragment first: a lane's four registers are four consecutive columns of a row)
#pragma unroll
                for (int j = 0; j < 4; ++j) t[j] = wavek_mfma<IS_BF16>(frag16_value(bf[0][j]), frag16_value(af[0][m]), f32x4{0.0f, 0.0f, 0.0f, 0.0f});
#pragma unroll
                for (int j = 0; j < 4; ++j) t[j] = wavek_mfma<IS_BF16>(frag16_value(bf[1][j]), frag16_value(af[1][m]), t[j]);
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[m][j] += t[j];
            }
        }
    }
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");      // (nothing lands in the ring any more)

    wavek_park<TM>(ring, acc, lane);
    __syncthreads();
    if (a.out_dtype == DT_F32) wavek_finish<C, DT_F32>(lds, a, m0, n0, wave, lane, bias);
    else if (a.out_dtype == DT_BF16) wavek_finish<C, DT_BF16>(lds, a, m0, n0, wave, lane, bias);
    else wavek_finish<C, DT_F16>(lds, a, m0, n0, wave, lane, bias);
}

template <class C>
hipError_t launch_wavek_variant(const Args& a, int group_m, hipStream_t stream) {
    const int tiles_m = (int)((a.M + C::BM - 1) / C::BM), tiles_n = (int)((a.N + C::BN - 1) / C::BN);
    const dim3 grid((unsigned)(tiles_m * tiles_n), (unsigned)a.batch), block(C::NT);
    const bool bf = a.dtype == DT_BF16, akc = !a.transA, bkc = a.transB != 0;
#define GEMM_TILE_LAUNCH(BF, AKC, BKC) hipLaunchKernelGGL((tile_wavek_kernel<C, BF, AKC, BKC>), grid, block, 0, stream, a, tiles_m, tiles_n, group_m)
    if (akc) {
        if (bf) { if (bkc) GEMM_TILE_LAUNCH(true, true, true); else GEMM_TILE_LAUNCH(true, true, false); }
        else { if (bkc) GEMM_TILE_LAUNCH(false, true, true); else GEMM_TILE_LAUNCH(false, true, false); }
    } else if constexpr (C::BM % 64 == 0) {
        if (bf) { if (bkc) GEMM_TILE_LAUNCH(true, false, true); else GEMM_TILE_LAUNCH(true, false, false); }
        else { if (bkc) GEMM_TILE_LAUNCH(false, false, true); else GEMM_TILE_LAUNCH(false, false, false); }
    } else {
        return hipErrorInvalidValue;
    }
#undef GEMM_TILE_LAUNCH
    return hipGetLastError();
}

}  // namespace tile
}  // namespace gemm
