// Table of macro-tile variants and the preconditions of the family.
#include "tile_kernel.hpp"

namespace gemm {

#define GEMM_TILE_VARIANT(IDX, NAME, KIND, BM, BN, BK, WM, WN, NS) \
    hipError_t launch_tile_variant_##IDX(const Args& a, int group_m, const TileSplit& split, hipStream_t stream);
#include "tile_variants.def"
#undef GEMM_TILE_VARIANT

namespace {

typedef hipError_t (*launch_fn)(const Args&, int, const TileSplit&, hipStream_t);

const TileVariantInfo kInfo[] = {
#define GEMM_TILE_VARIANT(IDX, NAME, KIND, BM, BN, BK, WM, WN, NS) {NAME, BM, BN, BK, (WM) * (WN) * 64, KIND},
#include "tile_variants.def"
#undef GEMM_TILE_VARIANT
};

const launch_fn kLaunch[] = {
#define GEMM_TILE_VARIANT(IDX, NAME, KIND, BM, BN, BK, WM, WN, NS) launch_tile_variant_##IDX,
#include "tile_variants.def"
#undef GEMM_TILE_VARIANT
};

constexpr int kNum = (int)(sizeof(kInfo) / sizeof(kInfo[0]));

}  // namespace

int tile_num_variants() { return kNum; }

const TileVariantInfo* tile_variant_info(int variant) {
    return (variant >= 0 && variant < kNum) ? &kInfo[variant] : nullptr;
}

// 16-byte vector loads along the contiguous dimension of each operand (8 elements of 16 bits,
// 4 of 32), 32-bit byte offsets inside a tile, and a 32-bit workgroup count.
bool tile_supports(const Args& a) {
    if (a.dtype != DT_BF16 && a.dtype != DT_F16 && a.dtype != DT_F32) return false;
    const int64_t chunk = a.dtype == DT_F32 ? 4 : 8;
    if (a.M <= 0 || a.N <= 0 || a.K <= 0) return false;
    if (((uintptr_t)a.A & 15) || ((uintptr_t)a.B & 15)) return false;
    if ((a.lda % chunk) || (a.ldb % chunk)) return false;
    if (a.lda > (1 << 22) || a.ldb > (1 << 22)) return false;
    if (a.K > (1 << 30)) return false;
    // the contiguous dimension of each operand must be whole 16-byte chunks
    if ((!a.transA ? a.K : a.M) % chunk) return false;
    if ((a.transB ? a.K : a.N) % chunk) return false;
    const int64_t tiles = ((a.M + 127) / 128) * ((a.N + 127) / 128);
    if (tiles > (int64_t)1 << 30) return false;
    return true;
}

// A variant takes either 16-bit or 32-bit operands.  The direct-to-LDS variants mask lanes with a
// fixed out-of-range offset of 2 GiB - 16.
bool tile_variant_supports(const Args& a, int variant) {
    if (variant < 0 || variant >= kNum) return false;
    const bool fp32 = kInfo[variant].kind == 4 || kInfo[variant].kind == 7;
    if (fp32 != (a.dtype == DT_F32)) return false;
    if (kInfo[variant].kind == 0 || fp32) return true;
    if (kInfo[variant].kind == 5 && !shortk_call_fits(a)) return false;
    const int64_t a_bytes = ((a.transA ? a.K : a.M) * a.lda) * 2, b_bytes = ((a.transB ? a.N : a.K) * a.ldb) * 2;
    return a_bytes < 0x7ffffff0ll && b_bytes < 0x7ffffff0ll;
}

// The persistent short-k kernel (kind 5): whole slabs, K <= 128 (the operands of a tile inside 64 KiB of LDS),
// C write-only, no bias, stored in 16-byte pieces.  (Restated here from
// tile_shortk_kernel.hpp, which only the variant's own translation unit includes.)
bool shortk_call_fits(const Args& a) {
    if (a.K % 32 != 0 || a.K > 128 || a.beta != 0.0f || a.bias != nullptr || a.k_total != 0) return false;
    const int64_t ob = elem_bytes(a.out_dtype);
    if (a.N % 8 != 0 || a.ldc % (16 / ob) != 0 || ((uintptr_t)a.C & 15)) return false;
    if (a.batch > 1 && (a.strideC * ob) % 16 != 0) return false;
    return true;
}

bool tile_variant_splits(int variant) { return variant >= 0 && variant < kNum && kInfo[variant].kind == 3; }
bool tile_variant_slices(int variant) { return variant >= 0 && variant < kNum && kInfo[variant].kind != 3 && kInfo[variant].kind != 5; }

namespace {

// Estimates in us of the wave tiles, fitted to 490 random calls (M 1 to 4000, N and K 64 to 16384, all layouts, batches; half
// of the calls within 7 %, nine of ten within 20 %).  Per element of k: a workgroup alone on its unit, or each round of
// them; both grow where an operand's rows start inside a 128-byte line, so that a slab's 128 bytes of a row lie in two.
struct WaveTile { int variant, bm; double per_k_alone, per_k, straddling, fixed, per_round, store_rate, weight_rate; };
constexpr WaveTile kWaveTiles[] = {{18, 64, 0.00255, 0.00258, 0.15, 4.2, 0.96, 6.7e6, 22e6}, {19, 16, 0.00131, 0.00143, 0.21, 4.1, 0.6, 22e6, 11e6}};
// Up to two workgroups of 64x64 per unit: those are resident at once.  Beyond, the 128x128 tile reads half as much per product
// (1392x2816x1024, 968 tiles of 64x64: 21.9 us against 17.5; 960x2048x1280, 480 tiles: 13.0 against 19.1).  Operands of more
// than 128 MiB stream from memory, which few short-lived workgroups do not keep busy (14x3840x14336 60 us in 16-row tiles, 40
// cut along k).
constexpr int64_t kWaveTilesPerUnit = 2, kWaveTileBytes = (int64_t)128 << 20;

}  // namespace

int wave_tile_for(const Args& a, int64_t cus, double* estimate) {
    if ((a.M + a.N) * a.K * a.batch * 2 > kWaveTileBytes) return -1;
    if (((a.M + 63) / 64) * ((a.N + 63) / 64) * a.batch > kWaveTilesPerUnit * cus) return -1;
    int best = -1;
    double best_time = 0.0;
    for (const WaveTile& t : kWaveTiles) {
        if (!tile_variant_supports(a, t.variant) || (a.transA && t.bm != 64)) continue;
        const int64_t rounds = (((a.M + t.bm - 1) / t.bm) * ((a.N + 63) / 64) * a.batch + cus - 1) / cus;
        const int straddling = ((a.transA ? a.M : a.K) % 64 != 0) + ((a.transB ? a.K : a.N) % 64 != 0);
        const double per_k = (rounds == 1 ? t.per_k_alone : t.per_k * (double)rounds) * (1.0 + t.straddling * straddling);
        const double stored = (double)(a.M * a.N * a.batch) * (double)elem_bytes(a.out_dtype) * (a.beta != 0.0f ? 2.0 : 1.0);
        const double time = t.fixed + t.per_round * (double)rounds + per_k * (double)a.K + stored / t.store_rate + (double)(a.N * a.K * a.batch) * 2.0 / t.weight_rate;
        if (best < 0 || time < best_time) { best = t.variant; best_time = time; }
    }
    if (estimate) *estimate = best_time;
    return best;
}

// Whole 128x128 tiles that have no wave tile: with both operands k-contiguous and K from 1280 on they run on the quartered
// kernel (variant 16, 16x16x32 products, its slabs requested in pairs), which waits less per slab and has the longer fill
// (1216x2752x1024 14.6 -> 15.3); the sums are the same to the bit (a test holds them together).  Of 165 random calls of 512 to
// 1600 64x64 tiles it is 1.07 times as fast on average for K 1024 to 1536 and 1.10 beyond (600x4024x4264 59.7 -> 51 us,
// 1648x1872x6224 80.8 -> 68, 2120x1376x3304 53.7 -> 44; 6 % slower on one of 58), 1.02 for K 512 to 768, 1.02 to 1.04 with a
// row-major B (two of 32 4 % slower), 0.94 to 0.97 with A stored KxM.  With more than two and up to two and a half tiles to a
// unit it is level (20 random calls) and loses where few of the third are there (1856x80x1856, batch of 39, 69.6 -> 80.7 us, of
// 43 1696x80x1696 65 -> 71): variant 5 stays.
constexpr int64_t kLongK = 1280;
// Up to 64 columns to a matrix the 128x128 tile is at least half empty, and the 64x64 wave tile is ahead at any number of
// tiles, with A row-major and K from 768 on: 17 random calls, batches of attention's second product most of them, 1.09 times as
// fast on average (1160x64x1160 NN, batch of 57, 59.4 -> 46.2 us, 1512x64x1512 NT, 26, 39.6 -> 32.2, 1864x64x1864 NN, 29, 65.4
// -> 57.4; 2 % behind on one).  With A stored KxM 0.91 to 1.1, with a shorter k 0.88 to 1.2.
constexpr int64_t kNarrowK = 768;

// C = alpha op(A) op(B) and nothing else on whole 128x128 tiles leaves that kernel straight from its registers.  There the wave
// tiles, which add their sums through LDS first, are level at best up to K = 128 (batch of 21 256x256x64 NT 4.8 us against 6.0,
// of 5 512x512x128 5.2 against 6.2), and beyond one of them to a unit up to K = 1536 in a batch (of 17 512x128x512 NN 7.9 against
// 9.8), up to 512 in a single matrix (168 random calls 1.02 times as long on them out of the last-level cache, 0.97 from memory;
// with A stored K x M and B row-major up to 1024, 100 calls 1.07 and 1.02).  From there on the wave tiles are ahead (168 calls 0.94
// and 0.80: 5632x256x1280 NN 14.6 us against 16.7).  Ragged tiles, a C that is read, a bias or an activation take the staged
// epilogue, and the wave tiles are ahead of it.
constexpr int64_t kWholeShortK = 128, kWholeK = 512, kWholeKTN = 1024, kWholeKBatch = 1536;

bool whole_128_tiles_ahead(const Args& a, int64_t cus) {
    if (a.beta != 0.0f || a.bias || a.act != ACT_NONE || a.M % 128 || a.N % 128) return false;
    if (a.M / 64 * (a.N / 64) * a.batch <= cus) return a.K <= kWholeShortK;
    return a.K < (a.batch > 1 ? kWholeKBatch : a.transA && !a.transB ? kWholeKTN : kWholeK);
}

namespace {

// With A stored K x M, B row-major, the rows of both starting inside a 128-byte line, more than one 64x64 tile to a unit, K from
// 2400 on and a C of 16 bits that is only written the wave tiles are behind: 37 random calls 1.11 times as long on them with the
// operands in the last-level cache (none ahead), 0.985 from memory (264x5904x2824 25.5 us against 31.3, 296x4968x2456 23.2 against
// 26.9).  With an fp32 C that is read they are ahead (155 calls, 0.99 and 0.92).
constexpr int64_t kLongTN = 2400;

bool long_straddling_tn(const Args& a, int64_t cus) {
    if (a.batch != 1 || !a.transA || a.transB || a.M % 64 == 0 || a.N % 64 == 0 || a.K < kLongTN || a.beta != 0.0f || a.out_dtype == DT_F32) return false;
    return ((a.M + 63) / 64) * ((a.N + 63) / 64) > cus;
}

// The tiles of a matrix of a batch lie on as many XCDs as there are of them, and each XCD's L2 fetches the matrix's operands for
// itself: 64x64 tiles spread a small matrix over more of them than 128x128 tiles do.  Beyond one wave tile to a unit, where that
// is 90 MB more to fetch (or 93 MB in all with A stored K x M, B row-major and K beyond 700), the 128x128 tiles of at most a round
// (three quarters of one) stay: 239 of 1708 random batches 1.22 times as long on the wave tiles with the operands in the
// last-level cache and 1.10 from memory (42 x 360x120x1696 NN 22.0 us against 37.4, 29 x 120x264x1544 TN 18.9 against 30.6),
// three of them ahead; of the others 90 are more than 5 % behind, 0.85 of the time on average.  Level, and left: both operands
// k-contiguous (1.01 and 0.87), and a row-major B of up to 64 columns (0.93 and 0.90 as attention's second product).  A C that is
// read or has 32 bits costs the 128x128 tiles more; three times its further bytes are taken off (66 of 428 batches with an fp32
// C and beta = 1: 1.12 and 1.02).
constexpr int64_t kXcds = 8, kSpreadBytes = 90000000, kSpreadBytesTN = 93000000, kSpreadKTN = 700;

bool spread_batch(const Args& a, int64_t cus) {
    const int64_t wave = ((a.M + 63) / 64) * ((a.N + 63) / 64), whole = ((a.M + 127) / 128) * ((a.N + 127) / 128);
    if (a.batch == 1 || wave * a.batch <= cus || whole * a.batch > cus || (!a.transA && (a.transB || a.N <= 64))) return false;
    const int64_t operands = (a.M + a.N) * a.K * a.batch * 2, on = wave < kXcds ? wave : kXcds, before = whole < kXcds ? whole : kXcds;
    const int64_t more_of_c = (a.M * a.N * a.batch) * (elem_bytes(a.out_dtype) * (a.beta != 0.0f ? 2 : 1) - 2);
    if (operands * (on - before) - 3 * more_of_c >= kSpreadBytes) return true;
    return a.transA && !a.transB && a.K > kSpreadKTN && 4 * whole * a.batch <= 3 * cus && operands * on - 3 * more_of_c > kSpreadBytesTN;
}

}  // namespace

int whole_tile_variant(const Args& a, int variant, int64_t cus) {
    if (variant != 5 && variant != 12) return -1;
    const int wave_tile = whole_128_tiles_ahead(a, cus) || long_straddling_tn(a, cus) || spread_batch(a, cus) ? -1 : wave_tile_for(a, cus, nullptr);
    if (wave_tile >= 0) return wave_tile;
    if (variant == 5 && !a.transA && a.N <= 64 && a.K >= kNarrowK && tile_variant_supports(a, 18)) return 18;
    const int64_t tiles = ((a.M + 127) / 128) * ((a.N + 127) / 128) * a.batch;
    const bool thin_third_round = tiles > 2 * cus && 2 * tiles <= 5 * cus;
    return !a.transA && a.transB && a.K >= kLongK && !thin_third_round && tile_variant_supports(a, 16) ? 16 : -1;
}

int tile_variant_for_layout(const Args& a, int variant) { return variant == 19 && a.transA ? 18 : variant; }

hipError_t launch_tile(const Args& a, int variant, int group_m, const TileSplit& split, hipStream_t stream) {
    if (variant < 0 || variant >= kNum) return hipErrorInvalidValue;
    if (split.parts > 1 && !tile_variant_splits(variant)) return hipErrorInvalidValue;
    return kLaunch[variant](a, group_m < 1 ? 1 : group_m, split, stream);
}

namespace {

// Adds the partial tiles of a split in the order of their k shares and applies the epilogue:
// one thread per four consecutive columns of a tile row.  The kernel is one round trip to memory
// long, so the loads of all shares (P > 0: their number is fixed at compile time; P == 0: any
// number, four at a time) and of C_in and bias are issued before the first use.
template <int P>
__global__ __launch_bounds__(256) void tile_split_reduce_kernel(Args a, int tiles_m, int tiles_n, int group_m, int first_tile,
                                                                int parts, const float* partials, int BM, int BN) {
    int tm, tn;
    tile::tile_of_workgroup(first_tile + (int)blockIdx.x, tiles_m, tiles_n, group_m, tm, tn);
    const int idx = (int)blockIdx.y * 256 + (int)threadIdx.x;          // one of BM * BN / 4 vectors
    const int r = idx / (BN / 4), c = (idx % (BN / 4)) * 4;
    const int64_t row = (int64_t)tm * BM + r, col = (int64_t)tn * BN + c;
    if (row >= a.M || col >= a.N) return;
    const size_t tile_floats = (size_t)BM * BN;
    const float* p = partials + ((size_t)blockIdx.x * parts) * tile_floats + (size_t)r * BN + c;
    float c_in[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    tile::RawBias bias;
    auto load_inputs = [&]() {
        tile::ask_bias(a, col, bias);
        const bool vec = col + 3 < a.N;
        if (vec && a.beta != 0.0f) {
            const int64_t ci = row * a.ldc + col;
            f32x4 v;
            if (a.out_dtype == DT_F32) v = tile::OutVec<DT_F32>::load4((const float*)a.C + ci);
            else if (a.out_dtype == DT_BF16) v = tile::OutVec<DT_BF16>::load4((const uint16_t*)a.C + ci);
            else v = tile::OutVec<DT_F16>::load4((const uint16_t*)a.C + ci);
#pragma unroll
            for (int e = 0; e < 4; ++e) c_in[e] = v[e];
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (vec || col + e >= a.N) break;
            if (a.beta != 0.0f) c_in[e] = load_elem(a.C, a.out_dtype, row * a.ldc + col + e);
        }
    };
    f32x4 s;
    if constexpr (P > 0) {
        f32x4 v[P];
#pragma unroll
        for (int q = 0; q < P; ++q) v[q] = *(const f32x4*)(p + (size_t)q * tile_floats);
        load_inputs();
        s = v[0];
#pragma unroll
        for (int q = 1; q < P; ++q) s += v[q];
    } else {
        load_inputs();
        s = *(const f32x4*)p;
        int q = 1;
        for (; q + 4 <= parts; q += 4) {
            f32x4 v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = *(const f32x4*)(p + (size_t)(q + u) * tile_floats);
#pragma unroll
            for (int u = 0; u < 4; ++u) s += v[u];
        }
        for (; q < parts; ++q) s += *(const f32x4*)(p + (size_t)q * tile_floats);
    }
    const f32x4 bj = tile::bias_values(a, bias);
    f32x4 one[1];
#pragma unroll
    for (int e = 0; e < 4; ++e) one[0][e] = epilogue_value(s[e], a.alpha, a.beta, c_in[e], bj[e], ACT_NONE);
    if (a.act != ACT_NONE) apply_act4(one, a.act);
    const f32x4 o = one[0];
    if (col + 3 < a.N) {          // four outputs in one store
        const int64_t ci = row * a.ldc + col;
        if (a.out_dtype == DT_F32) tile::OutVec<DT_F32>::store4((float*)a.C + ci, o);
        else if (a.out_dtype == DT_BF16) tile::OutVec<DT_BF16>::store4((uint16_t*)a.C + ci, o);
        else tile::OutVec<DT_F16>::store4((uint16_t*)a.C + ci, o);
        return;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        if (col + e >= a.N) break;
        store_elem(a.C, a.out_dtype, row * a.ldc + col + e, o[e]);
    }
}

}  // namespace

hipError_t launch_tile_split_reduce(const Args& a, int variant, int group_m, const TileSplit& split, hipStream_t stream) {
    if (variant < 0 || variant >= kNum || split.parts <= 1) return hipErrorInvalidValue;
    const int BM = kInfo[variant].BM, BN = kInfo[variant].BN;
    const int tiles_m = (int)((a.M + BM - 1) / BM), tiles_n = (int)((a.N + BN - 1) / BN);
    const int tail = tiles_m * tiles_n - split.first_tile;
    if (tail <= 0) return hipSuccess;
    const dim3 grid((unsigned)tail, (unsigned)(BM * BN / 4 / 256)), block(256);
    const int gm = group_m < 1 ? 1 : group_m;
#define GEMM_REDUCE_LAUNCH(P)                                                                                       \
    hipLaunchKernelGGL(tile_split_reduce_kernel<P>, grid, block, 0, stream, a, tiles_m, tiles_n, gm, split.first_tile, \
                       split.parts, (const float*)split.partials, BM, BN)
    switch (split.parts) {
        case 2: GEMM_REDUCE_LAUNCH(2); break;
        case 3: GEMM_REDUCE_LAUNCH(3); break;
        case 4: GEMM_REDUCE_LAUNCH(4); break;
        case 6: GEMM_REDUCE_LAUNCH(6); break;
        case 8: GEMM_REDUCE_LAUNCH(8); break;
        default: GEMM_REDUCE_LAUNCH(0); break;
    }
#undef GEMM_REDUCE_LAUNCH
    return hipGetLastError();
}

}  // namespace gemm
