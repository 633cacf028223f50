// Macro-tile kernel for fp32 operands on the bf16 matrix instruction (gfx950).
//
// The fp32 matrix instructions run at a sixteenth of the bf16 rate (157 against 2500 TFLOP/s), so the product is
// formed from bf16 ones without giving up fp32 accuracy.  Every operand element is taken apart, exactly, as
//   x = hi + mid + lo,   hi = bf16(x), mid = bf16(x - hi), lo = x - hi - mid
// (8 significant bits each and the signs of the remainders: 24 bits), and of the nine products of the pieces the
// six largest are summed,
//   hi*hi + hi*mid + mid*hi + mid*mid + hi*lo + lo*hi,
// each exact in fp32 and added in the fp32 accumulators of v_mfma_f32_16x16x32_bf16.  The three left out are at most
// 2^-24 |a b| together (|mid| <= 2^-8 |x|, |lo| <= 2^-17 |x|).  (Sums of products of an exact split in shorter floats: Dekker 1971;
// three bf16 for one fp32: Henry, Tang and Heinecke 2019.)  Against 64-bit sums the results are closer than the
// fp32 instruction's, which rounds an accumulator once per two products where this one does six times per 32 (2-norm, Gaussian data: K = 4
// 3.2e-8 against 4.0e-8, K = 32 3.7e-8 against 1.0e-7, K = 256 2.3e-7 against 2.9e-7, K = 4096 1.0e-6 against 1.1e-6).
//
// Structure: one stage of a slab is three planes of bf16 per operand in LDS, two stages; while a wave multiplies slab
// kt it takes apart slab kt+1, which is in registers, into the other stage, and asks for slab kt+2 as registers come free.
// One barrier per slab, a sixth of its instructions ahead of its end: the last pair of planes is in registers by then, so
// the matrix pipe has work on both sides of the barrier.  Everything is placed by slots, one behind each matrix
// instruction.
//
// Bound: the issue port.  Next to a matrix instruction (16 cycles) there is room for about two vector instructions, and taking
// an element apart costs 6.5, so a tile's ratio of staged elements to products decides: 1.6 vector instructions per
// matrix instruction with 256x128, 2.2 with 128x128.  Beyond that the power limit: at 4096^3 the pairs run at 2.0 GHz with the
// matrix pipe 67 % busy and 1.84 vector instructions per matrix instruction over the whole kernel.  Measured, this kernel / one
// on the fp32 instruction before: 4096^3 580 to 616 us (237 to 223 TFLOP/s) / 1054 to 1209, 2048^3 86 to 93 / 137 to 146, 1024^3 20.5 to
// 22.3 / 27.2 to 27.8, 512^3 11.1 / 11.5, 256^3 8.1 / 8.9, 4096x4096x64 27.2 to 28.1 / 30.
//
// What the split cannot take.  The pieces of an element are multiples of its last bit, 2^-149 for the smallest floats, and a bf16
// number's last bit is 2^-133 at least: both operands are multiplied by 2^16 first (one instruction per element, exact), which
// makes the split exact for every float down to the subnormal ones, and the sums by 2^-32 in the end.  Zeros, tiny elements and
// sums that cancel cost nothing.  Left are values so large that something overflows: a scaled element, a product of two or a sum
// (results from 2^96 on), and infinities and NaN themselves.  All of these end in a sum that is not finite, whatever comes
// after, so a tile with such a sum is computed again, unscaled, the slabs that hold an element above 2^40 or below
// 2^-110 by v_mfma_f32_16x16x4_f32.  Only elements of the operands count there, not what lies past their edges and is
// loaded with them.  Such a tile takes about three times its time (every one, 4096^3: 1714 us); the same time for all other data
// (a zero row, triangular, ternary, one element of 2^50, all of them 1e15, subnormal elements: 1024^3 21.6 to 23.5 us).
//
// Edges: loads past the end of an operand return zero dword by dword through the buffer descriptor's range check;
// elements of a k-contiguous operand past K are cleared when they are staged.  Nothing needs more than the natural
// alignment of a float.
#pragma once
#include <utility>
#include "tile_kernel.hpp"

namespace gemm {
namespace tile {

// BM x BN workgroup tile, WM x WN waves.  FOLD: each slab is summed by itself and added to the accumulators by the vector
// ALUs, which rounds a sum once per 32 elements of k at full magnitude (without: six times, on the matrix unit).  The general
// family takes it, whose plain kernel sums sixteen at a time: 2-norm error against 64 bits, Gaussian data, K = 128 / 1024 /
// 4095, plain kernel 9.3e-8 / 1.65e-7 / 2.98e-7, folded 5.6e-8 / 1.18e-7 / 2.21e-7, not folded 1.5e-7 / 4.9e-7 / 1.0e-6
// (the fp32 instruction is behind all three).  2049x2051x2045 143 us, a sixth less without the folds.
template <int BM_, int BN_, int WM_, int WN_, bool FOLD_ = false>
struct F32CfgT {
    static constexpr bool FOLD = FOLD_;
    static constexpr int BM = BM_, BN = BN_, BK = 32, WM = WM_, WN = WN_;
    static constexpr int NT = WM * WN * 64;
    static constexpr int WTM = BM / WM, WTN = BN / WN;
    static constexpr int TM = WTM / 32, TN = WTN / 32;   // 32-row bands of the epilogue
    static constexpr int TI = WTM / 16, TJ = WTN / 16;   // 16x16 accumulators of the wave sub-block
    static constexpr int A_PLANE = BM * BK * 2, B_PLANE = BN * BK * 2;   // one piece (hi, mid or lo) of a slab: rows of 32 bf16, chunks placed by swz<4>
    static constexpr int B_REGION = 3 * A_PLANE, STAGE = 3 * (A_PLANE + B_PLANE);
    static constexpr int RAW_STRIDE = BK + 4;            // floats per row of a slab staged as fp32
    static_assert(BM * RAW_STRIDE * 4 <= 3 * A_PLANE && BN * RAW_STRIDE * 4 <= 3 * B_PLANE, "the fp32 form of a slab fits the region of the three planes");
    static constexpr int WGS_PER_CU = 2 * STAGE > 80 * 1024 ? 1 : 3;
    static constexpr int WAVES_PER_SIMD = WGS_PER_CU * NT / 256;
    static_assert(!FOLD || WAVES_PER_SIMD > 1, "the additions need matrix instructions whose wait states the compiler supplies");
};

// f(0), f(1) .. f(N - 1) with the numbers as types: the bodies are placed slot by slot and name registers
template <class F, int... I>
__device__ __forceinline__ void static_for_each(F&& f, std::integer_sequence<int, I...>) { (f(std::integral_constant<int, I>{}), ...); }
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) { static_for_each(f, std::make_integer_sequence<int, N>{}); }

constexpr float kSplitScale = 0x1p16f, kSplitUnscale = 0x1p-32f;          // of each operand, of a product
constexpr float kSplitLargest = 0x1p40f, kSplitSmallest = 0x1p-110f;      // what the split takes without the scale

// bf16 pair of two floats (round to nearest even), and its two values widened again
__device__ __forceinline__ uint32_t pack_bf16(float x, float y) {
    typedef __attribute__((ext_vector_type(2))) float f32x2;
    typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{x, y}, bf16x2));
}
__device__ __forceinline__ float low_bf16(uint32_t p) { return __uint_as_float(p << 16); }
__device__ __forceinline__ float high_bf16(uint32_t p) { return __uint_as_float(p & 0xffff0000u); }

// One operand's slab: ROWS rows x 32 k.  A thread holds L quads of elements that it can take apart and stage without
// moving anything between lanes.  k-contiguous operand: a quad is one 16-byte load, four consecutive k of one row.
// m/n-contiguous operand: G = L or four loads of four rows each at consecutive k make a block; with four loads quad i of
// the block is row i (four k), with two it is rows 2i and 2i + 1 (two k each).
template <bool KC, int ROWS, class C>
struct F32Mover {
    static constexpr int L = ROWS * C::BK / 4 / C::NT, G = L < 4 ? L : 4;
    static_assert(L == 2 || L == 4 || L == 8, "64, 128 or 256 rows");
    static constexpr int PLANE = ROWS * C::BK * 2;
    static constexpr int KQ = C::BK / 4, RB = ROWS / 4;                     // quads per row (k-contiguous); blocks of four rows
    uint32_t goff[L];      // byte offset of the load from the slab's first byte
    uint32_t loff[L];      // byte offset of the quad (of its first row's part) in a plane
    f32x4 r[L];

    // first row and first k of quad i
    static __device__ __forceinline__ uint32_t quad_row(int i, int tid) {
        return KC ? (i * C::NT + tid) / KQ : (((i / G) * C::NT + tid) % RB) * 4 + (i % G) * (4 / G);
    }
    static __device__ __forceinline__ uint32_t quad_k(int i, int tid) { return KC ? (i * C::NT + tid) % KQ * 4 : ((i / G) * C::NT + tid) / RB * G; }
    __device__ __forceinline__ void init(int tid, int64_t ld) {
#pragma unroll
        for (int i = 0; i < L; ++i) {
            const uint32_t row = quad_row(i, tid), k = quad_k(i, tid);
            goff[i] = (uint32_t)((KC ? row * ld + k : (k + i % G) * ld + (row & ~3u)) * 4);
            loff[i] = swz<4>(row, k >> 3) + (k & 7) * 2;
        }
    }
    static __device__ __forceinline__ const char* tile_base(const void* p, int64_t first_row, int64_t ld) {
        return KC ? (const char*)p + first_row * ld * 4 : (const char*)p + first_row * 4;
    }
    static __device__ __forceinline__ int64_t k_step_bytes(int64_t ld) { return KC ? (int64_t)C::BK * 4 : (int64_t)C::BK * ld * 4; }
    // bytes of the operand from the first element of a slab of k elements of a tile with `rows` rows of it to the last one
    static __device__ __forceinline__ uint32_t slab_bytes(int rows, int k, int64_t ld) {
        return (uint32_t)((KC ? (rows - 1) * ld + k : (k - 1) * ld + rows) * 4);
    }
    // Every load is issued (past the end of the slab it reads as zero); what a k-contiguous operand holds past K is
    // cleared when it is staged -- clearing it here would be a write to a register with a load in flight, which waits for it.
    __device__ __forceinline__ void gload_one(int i, __amdgpu_buffer_rsrc_t rsrc) {
        r[i] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, goff[i], 0, 0));
    }
    __device__ __forceinline__ void gload(__amdgpu_buffer_rsrc_t rsrc) {
#pragma unroll
        for (int i = 0; i < L; ++i) gload_one(i, rsrc);
    }
    // the loads whose registers are free once quad i (taken in order) has been taken apart
    __device__ __forceinline__ void gload_after(int i, __amdgpu_buffer_rsrc_t rsrc) {
        if (KC) {
            gload_one(i, rsrc);
        } else if (i % G == G - 1) {
#pragma unroll
            for (int j = 0; j < G; ++j) gload_one(i - i % G + j, rsrc);
        }
    }
    // Element e of pair h of quad i, where it lies in the registers.
    template <int I, int H, int E> static constexpr int reg_of() { return KC ? I : (G == 4 ? I - I % G + 2 * H + E : E); }
    template <int I, int H, int E> static constexpr int lane_of() { return KC ? 2 * H + E : (G == 4 ? I % G : 2 * I + H); }
    template <int I, int H, int E> __device__ __forceinline__ float get() const { return r[reg_of<I, H, E>()][lane_of<I, H, E>()]; }
    template <int I, int H, int E> __device__ __forceinline__ void set(float x) { r[reg_of<I, H, E>()][lane_of<I, H, E>()] = x; }
    // the last slab of a k-contiguous operand: clear what lies past K (`left` = k values of the slab inside K)
    __device__ __forceinline__ void clear_past(int left, int tid) {
        if (!KC) return;
#pragma unroll
        for (int i = 0; i < L; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) r[i][e] = (int)quad_k(i, tid) + e < left ? r[i][e] : 0.0f;
    }
    // Pair h of quad i, scaled and taken apart in six parts of one to three instructions (in place: the elements become what is
    // left of them).  The empty assembly keeps a part where it is called: the compiler would move all of it behind
    // the matrix instructions, to where the pieces are stored.
    static constexpr int PARTS = 6;
    float wide[2];
    u32x2 piece[3];        // of the quad at hand
    template <int PART, int I, int H>
    __device__ __forceinline__ void split_part(float scale) {
        float x = get<I, H, 0>(), y = get<I, H, 1>();
        if constexpr (PART == 5) {
            uint32_t w = pack_bf16(x, y);
            asm volatile("" ::"v"(w));
            piece[2][H] = w;
        } else if constexpr (PART % 2 == 1) {
            uint32_t w = pack_bf16(x, y);
            wide[0] = low_bf16(w); wide[1] = high_bf16(w);
            asm volatile("" ::"v"(w), "v"(wide[0]), "v"(wide[1]));
            piece[PART / 2][H] = w;
        } else {
            if constexpr (PART == 0) { x *= scale; y *= scale; }
            else { x -= wide[0]; y -= wide[1]; }
            asm volatile("" ::"v"(x), "v"(y));
            set<I, H, 0>(x); set<I, H, 1>(y);
        }
    }
    // the quad's pieces to their planes
    __device__ __forceinline__ void store_pieces(char* region, int i) const {
#pragma unroll
        for (int p = 0; p < 3; ++p) {
            if constexpr (KC || G == 4) {
                *(u32x2*)(region + p * PLANE + loff[i]) = piece[p];
            } else {          // two rows of a 128-byte line: the second one's chunks sit 64 bytes across
                *(uint32_t*)(region + p * PLANE + loff[i]) = piece[p].x;
                *(uint32_t*)(region + p * PLANE + (loff[i] ^ 64u)) = piece[p].y;
            }
        }
    }
    __device__ __forceinline__ void split_and_store(char* region, float scale) {
        static_for<L>([&](auto i) {
            constexpr int I = decltype(i)::value;
            static_for<2 * PARTS>([&](auto w) { split_part<decltype(w)::value % PARTS, I, decltype(w)::value / PARTS>(scale); });
            store_pieces(region, I);
        });
    }
    // an element of the operand that the split cannot take as it is, not scaled (an m/n-contiguous operand is loaded past its
    // edge as well: `rows` = rows of the tile inside it)
    __device__ __forceinline__ bool outside(int rows, int tid) const {
        bool out = false;
#pragma unroll
        for (int i = 0; i < L; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float m = __builtin_fabsf(r[i][e]);
                out = out || ((m > kSplitLargest || (m < kSplitSmallest && m != 0.0f)) && (KC || ((int)quad_row(i, tid) & ~3) + e < rows));
            }
        return out;
    }
    __device__ __forceinline__ void store_raw(char* region, int tid) const {
        static_for<L>([&](auto i) {
            constexpr int I = decltype(i)::value;
            float* p = (float*)region + quad_row(I, tid) * C::RAW_STRIDE + quad_k(I, tid);
            const f32x4 x = {get<I, 0, 0>(), get<I, 0, 1>(), get<I, 1, 0>(), get<I, 1, 1>()};
            if constexpr (KC || G == 4) {
                *(f32x4*)p = x;
            } else {
                p[0] = x[0]; p[1] = x[1];
                p[C::RAW_STRIDE] = x[2]; p[C::RAW_STRIDE + 1] = x[3];
            }
        });
    }
};

// c += a * b.  With one workgroup per compute unit the accumulators live in the accumulation registers, and the
// instruction is written as assembly: left to itself the compiler moves them (or the fragments) between the two register
// files in the loop.  No accumulator is touched twice within four of them; the kernel supplies the wait states
// before it reads one.
template <bool ASM>
__device__ __forceinline__ void f32_mfma_bf16(f32x4& c, u32x4 a, u32x4 b) {
    if constexpr (ASM) asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
    else c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
template <bool ASM>
__device__ __forceinline__ void f32_mfma_f32(f32x4& c, float a, float b) {
    if constexpr (ASM) asm volatile("v_mfma_f32_16x16x4_f32 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
    else c = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
// the wait states between the last such instruction and the first read of an accumulator
template <bool ASM, int N>
__device__ __forceinline__ void f32_settle(f32x4 (&c)[N]) {
    if constexpr (ASM) {
        asm volatile("s_nop 15");
#pragma unroll
        for (int i = 0; i < N; ++i) asm volatile("" : "+a"(c[i]));
    }
}

// Which planes (0 = hi, 1 = mid, 2 = lo) the six steps of a slab multiply.  hi*hi comes last: in the first slab the small
// products are then summed among themselves (a K of one slab is rounded once at full magnitude).  The first step needs
// neither hi, so that it can be fetched while the last step of the slab before still multiplies those.
template <class C>
struct F32Planes {
    static constexpr int of_a(int s) { return s < 2 ? 1 : (s == 2 ? 2 : 0); }
    static constexpr int of_b(int s) { return s == 0 || s == 4 ? 1 : (s == 3 ? 2 : 0); }
    // the steps that use a plane of the operand for the first time
    static constexpr bool new_a(int s) { return s == 0 || s == 2 || s == 3; }
    static constexpr bool new_b(int s) { return s == 0 || s == 1 || s == 3; }
    // a step of four instructions is shorter than the LDS takes: all planes of a slab at once
    static constexpr bool EARLY = C::TI * C::TJ < 8;
};

// The accumulators of one tile of op(A) * op(B); every wave is done with `lds` when it returns.
// Accumulator (i, j): B's fragment is the instruction's first operand, so lane (c16, g4) holds row 16 i + c16 and
// columns 16 j + 4 g4 .. + 3 of the wave sub-block.
template <class C, bool A_KC, bool B_KC>
__device__ __forceinline__ void f32_tile_product(const Args& a, int64_t m0, int64_t n0, char* lds, uint32_t* flag,
                                                 f32x4 (&acc)[C::TI][C::TJ]) {
    constexpr int TI = C::TI, TJ = C::TJ;
    constexpr bool ASM = C::WAVES_PER_SIMD == 1;
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int c16 = lane & 15, g4 = lane >> 4;
    const int wm = wave % C::WM, wn = wave / C::WM;
    const int rows_a = (int)(a.M - m0 < C::BM ? a.M - m0 : C::BM), rows_b = (int)(a.N - n0 < C::BN ? a.N - n0 : C::BN);
    const int K = (int)a.K;

    using LA = F32Mover<A_KC, C::BM, C>;
    using LB = F32Mover<B_KC, C::BN, C>;
    LA la;
    LB lb;
    la.init(tid, a.lda);
    lb.init(tid, a.ldb);
    const char* pa = LA::tile_base(a.A, m0, a.lda);
    const char* pb = LB::tile_base(a.B, n0, a.ldb);
    const int64_t a_step = LA::k_step_bytes(a.lda), b_step = LB::k_step_bytes(a.ldb);

    auto clear_acc = [&]() {
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
            for (int j = 0; j < TJ; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    };
    clear_acc();
    // what the matrix instructions add to: the accumulators, or the sums of one slab
    constexpr bool FOLD = C::FOLD;
    f32x4 slab_sum[FOLD ? TI : 1][FOLD ? TJ : 1];
    auto sum = [&](int m) -> f32x4& {
        if constexpr (FOLD) return slab_sum[m / TJ][m % TJ];
        else return acc[m / TJ][m % TJ];
    };
    auto fold = [&](int m) {
        if constexpr (FOLD) acc[m / TJ][m % TJ] += slab_sum[m / TJ][m % TJ];
    };
    auto clear_sum = [&](int m) {
        if constexpr (FOLD) slab_sum[m / TJ][m % TJ] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    };
    if constexpr (FOLD) static_for<TI * TJ>([&](auto m) { clear_sum(decltype(m)::value); });

    uint32_t fa[TI], fb[TJ];                              // this lane's fragment of 16 rows in a plane: row c16, k = 8 g4 .. + 7
#pragma unroll
    for (int i = 0; i < TI; ++i) fa[i] = swz<4>(wm * C::WTM + i * 16 + c16, g4);
#pragma unroll
    for (int j = 0; j < TJ; ++j) fb[j] = C::B_REGION + swz<4>(wn * C::WTN + j * 16 + c16, g4);

    // The order of the slabs is free: a partial one comes first, so that the loop only sees whole ones.  Past the last
    // slab the loop asks twice more and gets zeros (what lies there in memory is not the operand's).
    const int partial = K % C::BK, k_tiles = K / C::BK + (partial ? 1 : 0);
    auto slab_of = [&](int t) { return (int64_t)(partial ? (t == 0 ? k_tiles - 1 : t - 1) : t); };
    auto slab_k = [&](int t) { return partial && t == 0 ? partial : C::BK; };
    auto slab_a = [&](int t) { return make_rsrc(pa + slab_of(t) * a_step, t < k_tiles ? LA::slab_bytes(rows_a, slab_k(t), a.lda) : 0); };
    auto slab_b = [&](int t) { return make_rsrc(pb + slab_of(t) * b_step, t < k_tiles ? LB::slab_bytes(rows_b, slab_k(t), a.ldb) : 0); };
    auto load_slab = [&](int t) {
        la.gload(slab_a(t));
        lb.gload(slab_b(t));
    };
    auto clear_past = [&](int t) {
        if (t == 0 && partial) { la.clear_past(partial, tid); lb.clear_past(partial, tid); }
    };

    constexpr int STEPS = 6;
    using Planes = F32Planes<C>;
    constexpr int NM = TI * TJ;
    u32x4 af[3][TI], bf[3][TJ];
    auto read_a = [&](const char* stage, int p, int i) { af[p][i] = *(const u32x4*)(stage + p * C::A_PLANE + fa[i]); };
    auto read_b = [&](const char* stage, int p, int j) { bf[p][j] = *(const u32x4*)(stage + p * C::B_PLANE + fb[j]); };

    if (k_tiles > 0) {
        LA la1 = la;                  // the first two slabs in one trip to memory
        LB lb1 = lb;
        load_slab(0);
        la1.gload(slab_a(1));
        lb1.gload(slab_b(1));
        __builtin_amdgcn_sched_barrier(0);
        clear_past(0);
        la.split_and_store(lds, kSplitScale);
        lb.split_and_store(lds + C::B_REGION, kSplitScale);
#pragma unroll
        for (int i = 0; i < LA::L; ++i) la.r[i] = la1.r[i];
#pragma unroll
        for (int i = 0; i < LB::L; ++i) lb.r[i] = lb1.r[i];
    }
    if (tid < 2) flag[tid] = 0;       // (read after the loop)
#pragma unroll
    for (int i = 0; i < TI; ++i) af[0][i] = u32x4{0u, 0u, 0u, 0u};       // the step ahead of the first slab adds nothing
#pragma unroll
    for (int j = 0; j < TJ; ++j) bf[0][j] = u32x4{0u, 0u, 0u, 0u};
    const char *next_a = pa + slab_of(2) * a_step, *next_b = pb + slab_of(2) * b_step;      // slab kt+2: a whole one
    const uint32_t whole_a = LA::slab_bytes(rows_a, C::BK, a.lda), whole_b = LB::slab_bytes(rows_b, C::BK, a.ldb);
    float scale = kSplitScale;
    asm("" : "+s"(scale));                                // (in a register: the instruction is half as long)
    auto iteration = [&](int kt, auto stage_) {
        constexpr int stage = decltype(stage_)::value;
        const char* cur = lds + stage * C::STAGE;
        char* nxt = lds + (1 - stage) * C::STAGE;
        const __amdgpu_buffer_rsrc_t ra = make_rsrc(next_a, kt + 2 < k_tiles ? whole_a : 0), rb = make_rsrc(next_b, kt + 2 < k_tiles ? whole_b : 0);
        next_a += a_step;
        next_b += b_step;
        __syncthreads();              // slab kt is staged; every wave has the last planes of slab kt-1 in registers
        // step 5 of slab kt-1, then steps 0 to 4 of slab kt
        constexpr int PAIRS = 2 * (LA::L + LB::L), WORK = PAIRS * LA::PARTS, SLOTS = STEPS * NM, LAST = SLOTS - SLOTS / 16;
        static_for<SLOTS>([&](auto slot_) {
            constexpr int slot = decltype(slot_)::value, n = slot / NM, s = (n + STEPS - 1) % STEPS, m = slot % NM, i = m / TJ, j = m % TJ;
            // (the sums of slab kt-1 are added NM - 1 instructions after their last product, just before slab kt needs them)
            if constexpr (slot >= NM - 1 && slot < 2 * NM - 1) fold(slot - (NM - 1));
            if constexpr (n == 1) clear_sum(m);
            f32_mfma_bf16<ASM>(sum(m), bf[Planes::of_b(s)][j], af[Planes::of_a(s)][i]);
            // the planes that the next step, step n of slab kt, is the first to need
            if constexpr (Planes::EARLY) {
                if constexpr (slot == 0) {
#pragma unroll
                    for (int i = 0; i < TI; ++i) read_a(cur, Planes::of_a(0), i);
#pragma unroll
                    for (int j = 0; j < TJ; ++j) read_b(cur, Planes::of_b(0), j);
                }
                if constexpr (slot == NM - 1) {
                    static_for<STEPS - 1>([&](auto t) {
                        constexpr int next = decltype(t)::value + 1;
#pragma unroll
                        for (int j = 0; j < TJ; ++j)
                            if (Planes::new_b(next)) read_b(cur, Planes::of_b(next), j);
#pragma unroll
                        for (int i = 0; i < TI; ++i)
                            if (Planes::new_a(next)) read_a(cur, Planes::of_a(next), i);
                    });
                }
            } else {
                if constexpr (Planes::new_b(n) && m < TJ) read_b(cur, Planes::of_b(n), m);
                if constexpr (Planes::new_a(n) && m >= NM - TI - TJ && m < NM - TJ) read_a(cur, Planes::of_a(n), m - (NM - TI - TJ));
            }
            // the next slab: a share of taking it apart (A's quads first), its stores, the loads behind it
            constexpr int w0 = slot * WORK / LAST < WORK ? slot * WORK / LAST : WORK;
            constexpr int w1 = (slot + 1) * WORK / LAST < WORK ? (slot + 1) * WORK / LAST : WORK;
            static_for<w1 - w0>([&](auto w_) {
                constexpr int w = w0 + decltype(w_)::value, pair = w / LA::PARTS, part = w % LA::PARTS, quad = pair / 2;
                constexpr bool done = part == LA::PARTS - 1 && pair % 2 == 1;
                if constexpr (quad < LA::L) {
                    la.template split_part<part, quad, pair % 2>(scale);
                    if constexpr (done) { la.store_pieces(nxt, quad); la.gload_after(quad, ra); }
                } else {
                    lb.template split_part<part, quad - LA::L, pair % 2>(scale);
                    if constexpr (done) { lb.store_pieces(nxt + C::B_REGION, quad - LA::L); lb.gload_after(quad - LA::L, rb); }
                }
            });
            __builtin_amdgcn_sched_barrier(0);
        });
    };
#pragma unroll 1
    for (int kt = 0; kt < k_tiles; kt += 2) {
        iteration(kt, std::integral_constant<int, 0>{});
        if (kt + 1 < k_tiles) iteration(kt + 1, std::integral_constant<int, 1>{});
    }
#pragma unroll
    for (int m = 0; m < NM; ++m) f32_mfma_bf16<ASM>(sum(m), bf[0][m % TJ], af[0][m / TJ]);
#pragma unroll
    for (int m = 0; m < NM; ++m) fold(m);
#pragma unroll
    for (int i = 0; i < TI; ++i) f32_settle<ASM>(acc[i]);

#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TJ; ++j) acc[i][j] *= kSplitUnscale;

    // Has anything overflowed?  (see above; only what is inside C counts: past its edge there are products of what lies past an
    // operand's edge)
    auto set_if = [&](int word, bool mine) { if (mine) flag[word] = 1; };
    auto is_set = [&](int word) { return __builtin_amdgcn_readfirstlane(flag[word]) != 0; };      // (behind a barrier)
    float nan = 0.0f;                                     // not a number as soon as it has met one that is not finite
    if (rows_a == C::BM && rows_b == C::BN) {
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
            for (int j = 0; j < TJ; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v) nan = fmaf(acc[i][j][v], 0.0f, nan);
    } else {
        const int rows = rows_a - (wm * C::WTM + c16), cols = rows_b - (wn * C::WTN + 4 * g4);
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
            for (int j = 0; j < TJ; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v) nan = fmaf(16 * i < rows && 16 * j + v < cols ? acc[i][j][v] : 0.0f, 0.0f, nan);
    }
    if (k_tiles == 0) __syncthreads();
    set_if(0, nan != nan);
    __syncthreads();
    if (__builtin_expect(is_set(0), 0)) {
        clear_acc();
        __syncthreads();
        if (tid == 0) flag[0] = 0;
        __syncthreads();
        load_slab(0);
#pragma unroll 1
        for (int kt = 0; kt < k_tiles; ++kt) {
            clear_past(kt);
#pragma unroll
            for (int m = 0; m < NM; ++m) clear_sum(m);
            set_if(kt & 1, la.outside(rows_a, tid) || lb.outside(rows_b, tid));
            __syncthreads();                              // (the last slab has been read as well)
            const bool as_fp32 = is_set(kt & 1);
            if (as_fp32) {
                la.store_raw(lds, tid);
                lb.store_raw(lds + C::B_REGION, tid);
            } else {
                la.split_and_store(lds, 1.0f);
                lb.split_and_store(lds + C::B_REGION, 1.0f);
            }
            load_slab(kt + 1);
            __syncthreads();
            if (tid == 0) flag[kt & 1] = 0;
            if (as_fp32) {
                // lane group g4 takes k = 4 g4 .. + 3 of sixteen, one per instruction (the order of k is free as long as
                // both operands agree)
#pragma unroll 1
                for (int s = 0; s < C::BK / 16; ++s) {
                    f32x4 ar[TI], br[TJ];
                    const int k = (16 * s + 4 * g4) * 4;
#pragma unroll
                    for (int i = 0; i < TI; ++i) ar[i] = *(const f32x4*)(lds + (wm * C::WTM + i * 16 + c16) * C::RAW_STRIDE * 4 + k);
#pragma unroll
                    for (int j = 0; j < TJ; ++j) br[j] = *(const f32x4*)(lds + C::B_REGION + (wn * C::WTN + j * 16 + c16) * C::RAW_STRIDE * 4 + k);
#pragma unroll
                    for (int q = 0; q < 4; ++q)
#pragma unroll
                        for (int m = 0; m < NM; ++m)
                            f32_mfma_f32<ASM>(sum(m), br[m % TJ][q], ar[m / TJ][q]);
                }
            } else {
#pragma unroll 1
                for (int s = 0; s < STEPS; ++s) {
                    const int p = Planes::of_a(s), q = Planes::of_b(s);
                    u32x4 ar[TI], br[TJ];
#pragma unroll
                    for (int i = 0; i < TI; ++i) ar[i] = *(const u32x4*)(lds + p * C::A_PLANE + fa[i]);
#pragma unroll
                    for (int j = 0; j < TJ; ++j) br[j] = *(const u32x4*)(lds + q * C::B_PLANE + fb[j]);
#pragma unroll
                    for (int m = 0; m < NM; ++m) f32_mfma_bf16<ASM>(sum(m), br[m % TJ], ar[m / TJ]);
                }
            }
#pragma unroll
            for (int m = 0; m < NM; ++m) fold(m);
        }
    }
#pragma unroll
    for (int i = 0; i < TI; ++i) f32_settle<ASM>(acc[i]);
    __syncthreads();                                      // LDS is reused by the epilogue
}

// IN_TURN: as for the 16-bit tile_kernel, the k slices of the call one after another
template <class C, bool A_KC, bool B_KC, bool IN_TURN>
__global__ __launch_bounds__(C::NT, C::WAVES_PER_SIMD) void tile_f32_kernel(Args a, int tiles_m, int tiles_n, int group_m, int64_t slice_len) {
    using EL = EpiLayout<C>;
    constexpr int TI = C::TI, TJ = C::TJ;
    constexpr int LDS_BYTES = 2 * C::STAGE > EL::BYTES ? 2 * C::STAGE : EL::BYTES;
    __shared__ __attribute__((aligned(128))) char lds[LDS_BYTES];
    __shared__ uint32_t flag[2];
    select_batch(a);
    int tm, tn;
    tile_of_workgroup(blockIdx.x, tiles_m, tiles_n, group_m, tm, tn);
    const int64_t m0 = (int64_t)tm * C::BM, n0 = (int64_t)tn * C::BN;
    f32x4 acc[TI][TJ];
    if constexpr (IN_TURN) {
        f32x4 part[TI][TJ];
        for_each_slice(a, slice_len, [&](const Args& s, bool first) {
            f32_tile_product<C, A_KC, B_KC>(s, m0, n0, lds, flag, part);
#pragma unroll
            for (int i = 0; i < TI; ++i)
#pragma unroll
                for (int j = 0; j < TJ; ++j)
#pragma unroll
                    for (int v = 0; v < 4; ++v) acc[i][j][v] = (first ? 0.0f : acc[i][j][v]) + part[i][j][v];
        });
    } else {
        f32_tile_product<C, A_KC, B_KC>(a, m0, n0, lds, flag, acc);
    }
    const int lane = threadIdx.x & 63, c16 = lane & 15, g4 = lane >> 4;
    tile_epilogue_bands<C>(
        [&](auto band, char* region) {
            constexpr int b = decltype(band)::value;
#pragma unroll
            for (int i2 = 0; i2 < 2; ++i2)
#pragma unroll
                for (int j = 0; j < TJ; ++j) *(f32x4*)(region + ((16 * i2 + c16) * EL::RS + j * 16 + 4 * g4) * 4) = acc[2 * b + i2][j];
        },
        lds, a, m0, n0, INT64_MAX, !IN_TURN);
}

template <class C, bool IN_TURN = false>
inline hipError_t launch_f32_tiles(const Args& a, int group_m, hipStream_t stream, int64_t slice_len = 0) {
    const int tiles_m = (int)((a.M + C::BM - 1) / C::BM), tiles_n = (int)((a.N + C::BN - 1) / C::BN);
    const dim3 grid((unsigned)(tiles_m * tiles_n), (unsigned)a.batch), block(C::NT);
    const bool akc = !a.transA, bkc = a.transB != 0;
#define GEMM_TILE_LAUNCH(AKC, BKC) \
    hipLaunchKernelGGL((tile_f32_kernel<C, AKC, BKC, IN_TURN>), grid, block, 0, stream, a, tiles_m, tiles_n, group_m, slice_len)
    if (akc && bkc) GEMM_TILE_LAUNCH(true, true);
    else if (akc && !bkc) GEMM_TILE_LAUNCH(true, false);
    else if (!akc && bkc) GEMM_TILE_LAUNCH(false, true);
    else GEMM_TILE_LAUNCH(false, false);
#undef GEMM_TILE_LAUNCH
    return hipGetLastError();
}

// (kF32PairAbove: why the 128x128 variant takes its tiles in pairs)
template <int BM, int BN, int WM, int WN>
inline hipError_t launch_f32_variant(const Args& a, int group_m, hipStream_t stream) {
    if constexpr (BM == 128) {
        const int64_t tiles = ((a.M + 127) / 128) * ((a.N + 127) / 128) * a.batch;
        if (tiles > kF32PairAbove) return launch_f32_tiles<F32CfgT<256, 128, 4, 2>>(a, group_m, stream);
    }
    return launch_f32_tiles<F32CfgT<BM, BN, WM, WN>>(a, group_m, stream);
}

}  // namespace tile
}  // namespace gemm
