// C ABI of libgemm: argument validation, kernel choice, workspace ownership.
#include <new>

#include "../../include/gemm.h"
#include "common.hpp"

#define GEMM_EXPORT extern "C" __attribute__((visibility("default")))

// A workspace grows by at least doubling, so 48 replaced buffers cover any sequence of sizes.
constexpr int kMaxRetired = 48;

// Split-K scratch of gemm_run_noalloc: device memory that exists from the moment the library is
// loaded, so that entry point never allocates.  Every GPU holds its own copy at its own address;
// the name below is only the host-side handle of the symbol, never an address to hand to a kernel:
// gemm_create looks the address up once per device (scratch_of_device) and everything else uses that.
constexpr size_t kScratchBytes = (size_t)32 << 20;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];
constexpr int kMaxDevices = 64;

struct gemm_handle_s {
    int device;
    int num_cus;
    float* workspace;
    size_t workspace_bytes;
    // Buffers that a larger one has replaced.  Work enqueued earlier may still use them, so they are
    // kept until the caller vouches for the streams (gemm_reserve_workspace, gemm_destroy).
    void* retired[kMaxRetired];
    int num_retired;
    float* scratch;          // this device's copy of the static split-K scratch
    bool forced;
    gemm_plan_t plan;        // forced plan (valid when forced)
    gemm_plan_t last;        // plan of the last successful run
    gemm_plan_t launched;    // ... and the kernel it was launched on
};

namespace {

using gemm::Args;

bool valid_dtype(int d) { return d == GEMM_F32 || d == GEMM_F16 || d == GEMM_BF16; }

// Picks a tile variant for the macro-tile family by comparing two estimates of the run time in
// microseconds.  A workgroup of the 256x256 tile (16x16x32 MFMA, direct-to-LDS, one workgroup per
// compute unit) takes 0.0203 us * K for its k loop plus 12 us for filling the pipeline
// and for the epilogue, which nothing overlaps; the 128x128 tile (two workgroups per compute
// unit, each other's epilogue hidden behind the other's k loop) takes kSmallPerK * K + kSmallFixed
// per tile and compute unit.  Measured: 8192^3 in 744 us with the large tile (4 rounds) and
// 1235 us with the small one (16 tiles per compute unit); 32 x 2048x2048x128 in 122 us (8
// rounds) and 83 us (32 tiles per compute unit).  So long k loops favour the large tile (2.2x
// the flops per cycle), short ones (K below about 560) the small one, and so does a grid that
// leaves most of the chip idle or a dimension that would waste half of every large tile.
// The constants of all estimates below were calibrated by timing the automatic plan against every
// forced combination of tile variant and split over a few hundred shapes.
// Operands of 2 GiB or more take the register-staged siblings (the direct loads mask lanes with
// a fixed 2 GiB - 16 offset).
constexpr int kLargeTileVariant = 10, kLargeTileFallback = 0, kSmallTileVariant = 5, kSmallTileFallback = 3;
// short k loops: the small tile with a ring of three stages (48 KiB of LDS: three workgroups per
// compute unit instead of two; faster up to K = 256 - 8192x8192x256: 53 against 63 us - slower from
// K = 512 on: 4096x4096x512 27 against 25, 256x4096x512 7.4 against 6.7; slices take the ring of four)
constexpr int kSmallTileShortK = 12;
constexpr int64_t kShortK = 256;
// ... and for K <= 128 with at least a tile per compute unit the persistent kernel, which keeps a panel of B in
// LDS, writes C from the registers and lets two workgroups per compute unit take turns (32 x 2048x2048x128: the
// bench row X8; level with the small tile from 256 tiles on, ahead from 512)
constexpr int kPersistentShortK = 17;
constexpr double kSmallPerK = 0.0094, kSmallFixed = 1.4;     // (the large tile's 0.0203 us per k and 12 us fixed: kFullTile below)
// A last round that fills less than this fraction of the compute units is split along K (when the
// variant can): each of its tiles goes to several workgroups, each over a share of the k slabs of
// at least kMinSlabsPerPart, and a second kernel adds the parts.  The number of parts minimises
// k loop / parts + the cost of the second kernel, which moves parts x tiles partial tiles of
// 256 KiB (0.1 us each, write and read: 1024x4096x14336 on 128 half tiles in 2 parts, 106 us) and
// adds them one after the other (0.3 us per part).  Measured: 512x512x65536 (4 tiles) 89 / 67 /
// 86 us with 16 / 32 / 64 parts, 256x256x131072 (1 tile) 147 / 94 / 78 us, 1024x1024x16384
// (16 tiles) 67 / 53 us with 16 / 12 parts.
constexpr double kSplitBelow = 0.6, kReducePerPartTile = 0.1, kReducePerPart = 0.3, kReduceLaunch = 3.0;
constexpr int kMinSlabsPerPart = 16;
constexpr int kPartChoices[] = {2, 3, 4, 6, 8, 12, 16, 24, 32, 48, 64};
// Tile rows per band of the workgroup -> tile map: the 32 workgroups resident on an XCD then cover 4 x 8
// tiles (8 x 4 with bands of 8 measured 0.5 % slower on 8192^3 and 8192x28672x8192, bands of 16 3 % slower).
constexpr int kTileBandRows = 4;
// most rows of C for which the automatic choice takes the skinny family
constexpr int64_t kSkinnyAutoRows = 32, kSkinnyAutoBytes = (int64_t)128 << 20, kSkinnyAutoBytesF32 = (int64_t)16 << 20;

// The 16x16x32 kernel with its tile halved along one side (256x128, 128x256): half the MFMAs per
// slab and 12 instead of 16 fragment reads, so LDS rather than the matrix pipe bounds it
// (4096^3: 116 us on either against 94 on the full tile = 0.0117 us per k and tile, 10 us fixed).
// It pays where the full tile would be half empty: 65536x128x4096 100 us against 120 on the
// 128x128 tile and 146 on the full tile, 32768x256x4096 75 against 87.
struct Dma16Tile { int variant; int bm, bn; double per_k, fixed, hbm_rate; int min_slabs; };   // min_slabs: shortest share of a split, in slabs of 32
constexpr Dma16Tile kFullTile{10, 256, 256, 0.0203, 12.0, 4.4e6, kMinSlabsPerPart};      // (8192^3: 709 us in four rounds; 4096^3: 92; 4096x4096x512: 21)
constexpr Dma16Tile kTallTile{14, 256, 128, 0.0117, 9.0, 5.8e6, kMinSlabsPerPart};
constexpr Dma16Tile kWideTile{15, 128, 256, 0.0117, 9.0, 5.8e6, kMinSlabsPerPart};
// ... and quartered (128x128, 16 MFMAs per step): 1024x4096x4096 in 38.5 us on 256 tiles; with its split it is
// the tile for small grids with long k loops (48x4096x4096: 15 us in 8 shares against 19 on sliced 32x32x16 tiles).
constexpr Dma16Tile kQuarterTile{16, 128, 128, 0.0082, 3.0, 5.0e6, 4};       // (its steps are short: 64x4096x512 11 us in 4 shares of 4 slabs, 14 whole)
constexpr double kHalfTileMargin = 0.9, kUnfavouredHalfTile = 1.15;
constexpr int64_t kQuarterTileRows = 64, kQuarterTileLongK = 16384;
constexpr double kQuarterTileMargin = 0.92;

// A round that leaves compute units idle runs its tiles faster than a full one: the clock of the busy units is
// higher and the caches and memory are less contended.  4096x6144x4096 (one full round and 128 tiles) takes 165 us
// unsplit where two full rounds would take 190; 4096x14336x4096 and 2048x28672x4096 (three and a half rounds) 358:
// the half round costs 0.74 to 0.77 of a full one.  Factor on the k loop of an unsplit trailing round of `tail`
// tiles behind at least one full round (the rates of a grid that is one partly filled round were fitted on such
// grids and stay as they are); the shares of a split round fill the chip and get none.
constexpr double kIdleRoundBase = 0.5;
double idle_round_factor(int64_t tail, int64_t cus, bool behind_full_rounds) {
    const double fill = (double)tail / (double)cus;
    return (fill >= 1.0 || !behind_full_rounds) ? 1.0 : kIdleRoundBase + (1.0 - kIdleRoundBase) * fill;
}

// time of the k loops of a round whose tiles are cut in `parts`, plus the second kernel (us)
double split_round_time(const Dma16Tile& t, int64_t tail, int parts, int64_t K, int64_t cus, bool behind_full_rounds, double live = 1.0) {
    const double loop = t.per_k * (double)K / parts;
    if (parts <= 1) return loop * idle_round_factor(tail, cus, behind_full_rounds);
    const double area = live * (double)(t.bm * t.bn) / 65536.0;      // (rows of a tile below the last row of C are not moved)
    const double move = kReducePerPartTile * area * parts * (double)tail, add = kReducePerPart * parts;
    return loop + (move > add ? move : add) + kReduceLaunch;
}

// parts per tile of the trailing `tail` tiles (1 = no split)
int tail_parts(const Dma16Tile& t, int64_t tail, int64_t cus, int64_t K, bool behind_full_rounds, double live = 1.0) {
    if (tail <= 0 || (double)tail >= kSplitBelow * (double)cus) return 1;
    const int64_t slabs = (K + 31) / 32;
    int best = 1;
    double best_t = split_round_time(t, tail, 1, K, cus, behind_full_rounds, live);
    for (int parts : kPartChoices) {
        if (parts * tail > cus || slabs / parts < t.min_slabs) break;
        const double tt = split_round_time(t, tail, parts, K, cus, behind_full_rounds, live);
        if (tt < best_t) { best_t = tt; best = parts; }
    }
    return best;
}

// whole call on one of the 16x16x32 tiles: full rounds, then the trailing round with its split
double dma16_time(const Dma16Tile& t, const Args& a, int64_t cus, bool may_split, int* parts_out, int64_t* first_split) {
    const int64_t tiles = ((a.M + t.bm - 1) / t.bm) * ((a.N + t.bn - 1) / t.bn) * a.batch;
    const int64_t tail = tiles % cus;
    const int64_t rows = ((a.M + t.bm - 1) / t.bm) * t.bm;
    const double live = (double)a.M / (double)rows;
    const bool behind = tiles >= cus;
    const int parts = may_split ? tail_parts(t, tail, cus, a.K, behind, live) : 1;
    double time = (double)(tiles / cus) * (t.per_k * (double)a.K + t.fixed);
    if (tail) time += split_round_time(t, tail, parts, a.K, cus, behind, live) + t.fixed;
    // operands that stream from HBM: not faster than this tile pulls them
    const double bytes = (double)(a.M + a.N) * (double)a.K * 2.0 * (double)a.batch;
    // (a thousandth of the unbounded estimate on top, so that of two tiles at the same bound the one with less to do wins)
    if (bytes > (double)((int64_t)256 << 20) && bytes / t.hbm_rate + t.fixed > time) time = bytes / t.hbm_rate + t.fixed + 1e-3 * time;
    *parts_out = parts;
    *first_split = tiles - tail;
    return time;
}

// The 128x128 tile has no such split; a grid of it that leaves compute units idle is cut in k
// slices instead (a strided batch over k ranges into fp32 partial results, added by the reduce
// kernel of the skinny family).  Time of the small tile with `slices` (1 = none), us.  A workgroup
// that has its compute unit to itself walks k at a rate set by where its operands come from:
// 0.0055 us per k for a handful of workgroups out of the L2 (512x512x4096: 23 us), 0.008 with 64
// (1024x1024x4096: 31 us), 0.0093 with one on every unit (1024x4096x14336: 134 us), 0.0122 when the operands exceed the
// last-level cache and come from HBM (128 ... 256 x 16384 x 16384: 186 to 200 us) - its ring keeps
// 48 KiB in flight against the large tile's 128 KiB.  Two workgroups per unit: kSmallPerK per round.
// The whole call is not faster than HBM delivers (4.7 TB/s reached by the sliced small tile).
// Slices add the second kernel: launch + the partial results written and read once.
constexpr double kSmallAloneFew = 0.0055, kSmallAloneMany = 0.008, kSmallAloneAll = 0.0093, kSmallAloneHbm = 0.0122;
constexpr double kSmallHbmRate = 4.7e6, kSliceMoveRate = 4.5e6;      // bytes per us
constexpr int kSliceChoices[] = {2, 4, 8, 16};
constexpr int64_t kMinSliceK = 512;          // shorter k ranges spend their time filling the pipeline (256x512x4096: 8 slices 12 us, 16 slices 15)
constexpr int64_t kMinSliceKF32 = 128;      // (64x1024x1024 11 us in 8 slices, 18 in 2)
constexpr double kSliceMargin = 0.9;          // slices must promise 10 % (384x2048x2048: 14 us whole, 18 in 4 slices, estimated equal)
constexpr double kSliceLaunchF32 = 3.5, kSliceMarginF32 = 0.92;      // (512^3 fp32: 11 us in 4 slices, 13 whole; 3072^3 within 8 %)
constexpr double kF32StoreRate = 3.75e6;
constexpr double kSliceLaunch = 5.0;          // the second kernel of a sliced call: launch, gap, one round trip (512x2048x2048: 14 us whole, 19 in 4 slices)
// Operands beyond the last-level cache stream from HBM on every call; there the large tile with its split
// stays ahead of the sliced small tile (128x16384x16384: 114 against 125 us, 128x8192x28672: 104
// against 119), so slices are considered only below this size (96...256 x 8192 x 8192, 134 to 138 MB:
// 33 to 44 us sliced against 46 to 56 on the large tile).
constexpr int64_t kLastLevelCacheBytes = (int64_t)256 << 20;

double small_tile_time(const Args& a, int64_t tiles, int slices, int64_t cus) {
    const double k = (double)a.K / slices;
    const int64_t wgs = tiles * slices, rounds = (wgs + cus - 1) / cus;
    const double bytes = (double)(a.M + a.N) * (double)a.K * 2.0 * (double)a.batch;
    const bool hbm = bytes > (double)kLastLevelCacheBytes;
    double loop;
    if (wgs <= cus) {
        const double crowd = wgs >= 64 ? 1.0 : (double)wgs / 64.0, full = wgs <= 64 ? 0.0 : (double)(wgs - 64) / (double)(cus - 64);
        loop = (hbm ? kSmallAloneHbm : kSmallAloneFew + (kSmallAloneMany - kSmallAloneFew) * crowd + (kSmallAloneAll - kSmallAloneMany) * full) * k;
    } else {
        loop = (double)rounds * kSmallPerK * k;
    }
    if (hbm && bytes / kSmallHbmRate > loop) loop = bytes / kSmallHbmRate;
    double t = loop + (double)rounds * kSmallFixed;
    if (slices > 1) t += kSliceLaunch + (double)slices * (double)(a.M * a.N) * 8.0 / kSliceMoveRate;
    return t;
}

// The slices an fp32 call is cut in: what its workspace has always been sized for.  A caller that reserved the
// workspace for a call, captures it on a handle that has none, or makes it through gemm_run_noalloc must not find that a
// faster kernel needs more of it, and fewer of them would round longer sums (532x1296x1296 3.3e-7 of the result's norm in
// 4, 5.5e-7 whole), so this rule (the estimate for the fp32 instruction: 0.0275 / 0.085 us per element of k for a 64x64 /
// 128x128 tile alone on its unit, 0.02 / 0.068 per tile otherwise) stays as it was when the kernel changed.  Its counts are
// still good ones: 532x1296x1296 25.1 us in 4 slices against 30.6 whole, 3072x312x1984 37.9 in 2 against 44.1.
int f32_slices(const Args& a, int64_t cus) {
    int most = 1;
    double best = 0.0;
    for (int big = 0; big < 2; ++big) {
        const int64_t side = big ? 128 : 64;
        const int64_t tiles = ((a.M + side - 1) / side) * ((a.N + side - 1) / side) * a.batch;
        for (int sl : {1, 2, 4, 8, 16}) {
            if (sl > 1 && (a.batch != 1 || a.N % 8 != 0 || a.K / sl < kMinSliceKF32)) break;
            const int64_t wgs = tiles * sl;
            double t = (wgs <= cus ? (big ? 0.085 : 0.0275) : (big ? 0.068 : 0.02) * (double)((wgs + cus - 1) / cus)) * ((double)a.K / sl) + 4.0;
            if (sl > 1) t = (t + kSliceLaunch + (double)sl * (double)(a.M * a.N) * 8.0 / kSliceMoveRate) / kSliceMargin;
            if (best == 0.0 || t < best) { best = t; most = sl; }
        }
    }
    return most;
}

struct TileChoice { int variant; int first_split_tile; int parts; double time; };   // time: the estimate behind the choice, us (0: none)
// fp32: the 128x128 or the 64x64 tile, whichever leaves the busiest compute unit less to do (see
// choose_tile).  The small tile is at least as fast as the general kernel down to a single tile
// (256^3: 8.6 against 10.2 us, 64^3: 4.6 against 5.9), so every aligned fp32 call takes a tile kernel.
constexpr int kF32TileVariant = 11, kF32SmallTileVariant = 13;
constexpr int64_t kF32MinTiles = 1;

// fp32: the 128x128 tile (beyond one per compute unit in pairs, see kF32PairAbove) or the 64x64 tile (up to three
// workgroups per unit), whole or in `slices` of k.  Estimate in us, fitted to both tiles on 350 random calls (M, N up to 4096,
// K from 8 to 4096, batches; the rule's choice is within 8 % of the faster one on all of them and 0.05 % behind on average):
//   64x64: 5.5 fixed; per element of k a unit's one, two or three workgroups 0.0177, 0.0262, 0.0374 (1024^3 21.6 us, 3072^3 360);
//   128x128: 10.8 fixed, 0.0435 per element with one per unit (2048^3 92 us); in pairs 4.7 more per full round behind the first, 0.0714
//   per element for a full round, 0.0543 for one that leaves 40 % of the units idle, in between in proportion;
//   the results leave at 3.75 TB/s.
// The fixed part decides at short k: 4001x895x16 12.5 us on the small tile, 15.3 on the large one, 2044x1940x104 14.7 / 17.9.
// Slices add the second kernel.  Deep k on a small grid gains most from them: 256x256x4096 74 -> 15 us in
// 16, 64x4096x4096 78 -> 23 in 8.
double f32_time(const Args& a, bool big, int slices, int64_t cus) {
    const int64_t side = big ? 128 : 64;
    const int64_t wgs = ((a.M + side - 1) / side) * ((a.N + side - 1) / side) * a.batch * slices, per_unit = (wgs + cus - 1) / cus;
    double per_k, fixed;
    if (!big) {
        per_k = (double)(per_unit / 3) * 0.0374 + (per_unit % 3 == 0 ? 0.0 : (per_unit % 3 == 1 ? 0.0177 : 0.0262));
        fixed = 5.5;
    } else if (wgs <= gemm::kF32PairAbove) {
        per_k = (double)per_unit * 0.0435;
        fixed = 10.8;
    } else {
        const double n = (double)(((a.M + 255) / 256) * ((a.N + 127) / 128) * a.batch * slices) / (double)cus;
        const double whole = (double)(int64_t)n, fill = n - whole;
        per_k = whole * 0.0714 + (fill > 0.0 ? 0.0543 + 0.0171 * (fill > 0.6 ? (fill - 0.6) / 0.4 : 0.0) : 0.0);
        fixed = 6.1 + 4.7 * (whole > 1.0 ? whole : 1.0) + (fill > 0.0 && whole > 0.0 ? 1.3 : 0.0);
    }
    const double t = fixed + per_k * ((double)a.K / slices) + (double)(a.M * a.N * a.batch) * 4.0 / kF32StoreRate;
    return slices > 1 ? (t + kSliceLaunchF32 + (double)slices * (double)(a.M * a.N) * 8.0 / kSliceMoveRate) / kSliceMarginF32 : t;
}

// Where the choice below comes to a 128x128 tile, the tiles with the k range divided among the waves (see wave_tile_for) are
// compared with it, whole or in parts: by their own estimate against that of the split or the slices, and in place of a whole
// 128x128 tile wherever wave_tile_for gives one and whole_128_tiles_ahead does not keep it.  On the device, on random calls of
// the sizes that a 128x128 tile used to take, they are 1.7 times as fast on average (geometric) in place of whole tiles (4600
// calls, eleven more than 5 % behind, 14 % the worst; with A stored K x M and more than one 64x64 tile to a unit 1.03 times on
// 739, 117 behind) and 1.5 in place of shares and slices (2149; three, 9 %), with the weights from memory 1.32 (134, 33 %: a k
// beyond 2800 with rows off the line or beyond 5500 on few units, the same calls level or ahead out of the last-level cache).
// Cut as before: long k ranges in slices, which put them on more units than a tile's waves are (128x1024x8192: 15 against
// 19.8), and a single strip or two of 33 to 64 rows, whose weights three or four tiles of 16 rows would each read. With a
// row-major weight, fewer 16-row tiles than half the units and K beyond 5000 (4096 where rows start inside a line) the shares
// draw more from memory than these few workgroups do (26 random calls: 1.24 times as long here from memory, 0.91 out of the
// last-level cache); so do they from K = 3000 on with fewer tiles than a quarter of the units and a pitch of whole 512 bytes, the
// k-rows of a slab on few memory channels (23 calls: 1.25 and 0.87; 10x2560x3328 13.8 us against 22.5 from memory, 12.3 against
// 14.4).  With A stored K x M the shares are ahead beyond K = 4096 (3584x256x6144 TN 21 us against 24.9, 904x1024x5632 TT 20.4
// against 23.5).
constexpr int64_t kLongSlicedK = 4096, kFewWaveTiles = 16, kLongRowMajorK = 5000;

bool row_major_stream_on_few_units(const Args& a, int64_t tiles, int64_t cus) {
    if (!a.transB && 4 * tiles < cus && a.ldb % 256 == 0 && a.K >= 3000) return true;
    return !a.transB && 2 * tiles < cus && a.K > (a.K % 64 || a.N % 64 ? kLongSlicedK : kLongRowMajorK);
}

TileChoice choose_shared_k_tile(const Args& a, int num_cus) {
    const int64_t cus = num_cus > 0 ? num_cus : 256;
    if (a.dtype == gemm::DT_F32) {
        const int slices = f32_slices(a, cus);
        const bool big = f32_time(a, true, slices, cus) < f32_time(a, false, slices, cus);
        return TileChoice{big ? kF32TileVariant : kF32SmallTileVariant, 0, slices, 0.0};
    }
    // a batch multiplies the number of workgroups; its trailing round is never split along K
    const int64_t small = ((a.M + 127) / 128) * ((a.N + 127) / 128) * a.batch;
    const bool large_ok = gemm::tile_variant_supports(a, kLargeTileVariant);
    const Dma16Tile* best_tile = &kFullTile;
    int parts = 1;
    int64_t first_split = 0;
    double t_large = dma16_time(kFullTile, a, cus, large_ok && a.batch == 1, &parts, &first_split);
    if (large_ok && a.batch == 1) {      // (in batched calls they were 4 to 16 % behind the 128x128 tile wherever they were chosen)
        // A half tile (a) where every full tile would be at least half empty (N <= 128 or M <= 128), or
        // (b) where it fills the chip better than the full tile does - 2048x4096x4096 is 128 full tiles
        // but 256 tiles of 256x128: 56 us against 80 on 128x128 tiles; 1024x8192x8192: 103 against 122 -
        // for operands inside the last-level cache and by a margin of 10 %: the estimates are not
        // sharper than that (4096x4224x4096: 131 us on the full tile, 145 to 170 on 256x128, estimated
        // 151 and 141), and from HBM the full tile with its split stays ahead (640x16384x16384: 319
        // against 369 to 388).
        const double t_full = t_large;
        const bool in_cache = (a.M + a.N) * a.K * 2 * a.batch <= kLastLevelCacheBytes;
        // On equal tile counts the half tile whose long side lies along the longer side of C is ahead
        // (1024x512x65536: 256x128 69 us, 128x256 101; 512x512x65536: 63 and 47; 1024x1024x32768: 82 and 72).
        const Dma16Tile* favoured = a.M > a.N ? &kTallTile : &kWideTile;
        for (const Dma16Tile* t : {&kWideTile, &kTallTile, &kQuarterTile}) {
            const int64_t halves = t == &kTallTile ? (a.N + 127) / 128 : (t == &kWideTile ? (a.M + 127) / 128 : 0);
            int p = 1;
            int64_t f = 0;
            const double tt = dma16_time(*t, a, cus, a.batch == 1, &p, &f) * (t == favoured || t == &kQuarterTile ? 1.0 : kUnfavouredHalfTile);
            // the quartered tile: for at most 64 rows of C, where it was ahead of every other plan on all 32 shapes
            // tried (48 x N x K; by 10 to 38 % over the sliced 32x32x16 tile); elsewhere the estimates at 10 to 20 us are
            // not sharp enough to place it (128x2048x2048: 14 us against 12), and it is left to forced plans
            const bool allowed = t == &kQuarterTile ? (a.M <= kQuarterTileRows && in_cache) : (halves == 1 || (in_cache && tt < kHalfTileMargin * t_full));
            if (allowed && tt < t_large) { t_large = tt; best_tile = t; parts = p; first_split = f; }
        }
    }
    const bool small_ok = gemm::tile_variant_supports(a, kSmallTileVariant);
    const double t_whole = small_tile_time(a, small, 1, cus);
    double t_small = t_whole;
    int slices = 1;
    if (small_ok && a.batch == 1 && a.N % 8 == 0 && (a.M + a.N) * a.K * 2 <= kLastLevelCacheBytes) {
        for (int sl : kSliceChoices) {
            if (a.K / sl < kMinSliceK || small * sl > 2 * cus) break;
            const double t = small_tile_time(a, small, sl, cus);
            if (t < t_small && t < kSliceMargin * t_whole) { t_small = t; slices = sl; }
        }
    }
    // (the sliced 32x32x16 tile is estimated too well for so few rows - 48x4096x4096: estimated 14 us, measured 19;
    // the quartered tile in 8 shares: estimated 15, measured 15 - so it does not compete there)
    if (best_tile == &kQuarterTile) t_small = t_large + 1.0;
    // The quartered tile against whatever won so far, for operands inside the last-level cache: with the last
    // steps of its k loop pipelined it is ahead of the sliced 32x32x16 tile on grids of one to two hundred small
    // tiles (128x4096x4096: 17 us in 6 shares against 20 in 8 slices; 512x4096x4096: 28 in 2 shares against 33
    // whole), where its estimate says so by 8 %.
    if (large_ok && a.batch == 1 && best_tile != &kQuarterTile && (a.M + a.N) * a.K * 2 <= kLastLevelCacheBytes) {
        int p = 1;
        int64_t f = 0;
        const double tq = dma16_time(kQuarterTile, a, cus, true, &p, &f);
        if (tq < kQuarterTileMargin * t_small && tq < kQuarterTileMargin * t_large) return TileChoice{kQuarterTile.variant, (int)f, p, tq};
    }
    if (t_large <= t_small) {
        if (!large_ok) return TileChoice{kLargeTileFallback, 0, 1, 0.0};
        return TileChoice{best_tile->variant, (int)first_split, parts, t_large};
    }
    if (!small_ok) return TileChoice{kSmallTileFallback, 0, 1, 0.0};
    // Where the 128x128 grid would be sliced along a long k, the quartered 16x16x32 tile with its own split does
    // the same job 3 to 23 % faster (256x1024x32768: 31 against 38 us, 512x1024x16384: 29 against 33); with shorter
    // k loops the sliced 32x32x16 tile stays ahead (128x1024x8192: 15 against 18).
    if (slices > 1 && a.K >= kQuarterTileLongK && large_ok && (a.M + a.N) * a.K * 2 <= kLastLevelCacheBytes) {
        int p = 1;
        int64_t f = 0;
        const double tq = dma16_time(kQuarterTile, a, cus, true, &p, &f);
        if (p > 1) return TileChoice{kQuarterTile.variant, (int)f, p, tq};
    }
    if (slices == 1 && small >= cus && gemm::tile_variant_supports(a, kPersistentShortK)) return TileChoice{kPersistentShortK, 0, 1, t_small};
    return TileChoice{slices == 1 && a.K <= kShortK ? kSmallTileShortK : kSmallTileVariant, 0, slices, t_small};
}

// An fp32 call that a plan gives to the 64x64 tiles, in whatever slices, runs in one launch on the tiles whose eight waves
// divide the k range, 32x32 (variant 20) or 16x32 (21), where those promise to be ahead (-1: neither).  Estimates in us, fitted
// to 240 random calls each (half within 4 %, nine of ten within 12 %).  On the device, on 2000 random calls (M, N to 3000, K
// to 6000) the choice is 1.80 times as fast as before on average (geometric), more than 5 % behind on four (8 %):
// 268x228x3592 TN 69 -> 18 us, 64x460x1152 23.7 -> 7.6 (N no multiple of 8, so never cut in slices), 512^3 10.5 -> 7.0,
// 64x168x2752 16.8 -> 12.6, 256^3 8.2 -> 7.2.  Two workgroups of 32x32 to a unit are resident at once; beyond, the 64x64 tile
// stages half as many elements per product (1016x2352x868 39 us against 48), and few columns with a long k are faster in
// slices.
int wave_f32_variant(const Args& a, int slices, int num_cus) {
    const int64_t cus = num_cus > 0 ? num_cus : 256;
    constexpr int64_t kTwoSlabs = 64;      // (up to here one launch takes as long as another: 39x588x64 6.6 us on either)
    constexpr double kSlicedMargin = 0.8; // (f32_time has a margin of its own against slices; 207x1328x3164: 27 us in 8 slices, 35 here)
    if (a.dtype != gemm::DT_F32 || a.K <= kTwoSlabs || ((a.M + 31) / 32) * ((a.N + 31) / 32) * a.batch > 2 * cus) return -1;
    struct Tile { int variant, rows; double per_k_half, per_k, per_k_more, fixed, per_round, weight_rate, activation, rows_of_a, rows_of_b; };
    static const Tile tiles[] = {{20, 32, 0.00462, 0.00998, 0.00957, 3.4, 0.37, 19e6, 0.3, 0.056, 0.017}, {21, 16, 0.00294, 0.00702, 0.00597, 2.66, 1.21, 17e6, 0.18, 0.086, 0.0}};
    double best = slices > 1 ? kSlicedMargin * f32_time(a, false, slices, cus) : f32_time(a, false, 1, cus);
    int variant = -1;
    for (const Tile& t : tiles) {
        const double wgs = (double)(((a.M + t.rows - 1) / t.rows) * ((a.N + 31) / 32) * a.batch) / (double)(2 * cus), rounds = wgs > 1.0 ? wgs : 1.0;
        const double per_k = (wgs <= 0.5 ? t.per_k_half : t.per_k + t.per_k_more * (rounds - 1.0)) * (1.0 + (a.transA ? t.rows_of_a : 0.0) + (a.transB ? 0.0 : t.rows_of_b));
        const double time = t.fixed + t.per_round * rounds + per_k * (double)a.K + (double)(a.M * a.N * a.batch) * 4.0 / 1.0e6 +
                            (double)(a.N * a.K * a.batch) * 4.0 / t.weight_rate + (a.act != gemm::ACT_NONE ? t.activation : 0.0);
        if (time < best) { best = time; variant = t.variant; }
    }
    return variant;
}

// Few rows whose plan is the narrow streaming kernel (one launch), a wide streaming kernel in slices or the quartered tile in
// shares run, in one launch, on the 16x64 or 64x64 tile whose waves divide the k range, where that is ahead (-1: it isn't): a
// workgroup of it reads 64 columns of the weight once, where the narrow kernel's has 16 (four times as many workgroups, the
// first products 5 us after the launch) and slices and shares need a second launch.  A unit streams about 30 GB/s from memory
// however many waves ask, so what has fewer than 48 workgroups (64 with a row-major weight, 96 with fewer than 96 columns of
// tiles and K beyond 4096; 80 of 64 rows, 200 for the wide kernels) or more than one to a unit is left where it is, and so is K
// beyond 8192 (NN 5000), where four waves' walk is the longer one.  A row-major weight with a pitch of whole 512 bytes is too,
// from K = 3000 on (the wide kernel's slices: 5000): the k-rows of a slab fall on few memory channels (31x2560x4864 18.8 us
// here, 15 in shares).
// - streaming kernels in slices, up to 16 rows: from 200 workgroups on, always (30 random calls, 1.13 to 1.20 times as fast on
//   average; 7 % ahead at the least up to K = 7000: 16x16384x4096 NN 32.4 -> 29, 8x15296x5184 NN 35.7 -> 27.5, 12x12288x4096 NT
//   24.8 -> 24).
// - the others by estimates in us, fitted to 423 random calls with 16-row tiles and 514 with 64-row tiles (half within 5 to 7
//   %, nine of ten within 11 to 17 %), by a margin of 5 %.  On such calls 1.17 to 1.18 times as fast on average with 16 rows
//   (the faster one in hindsight 1.18 to 1.19) and 1.06 to 1.10 with 64: 12x8192x2048 12 -> 8, 7x9920x2176 15.9 -> 9.6,
//   46x8128x2944 NN 18.1 -> 13.3, 61x2624x4480 NN 16.2 -> 11; with fewer than 64 workgroups of a long k or a row-major weight a
//   unit's own rate shows (26x3304x4544 NN 15.3 against 13.1, 5x5120x5120 NT 19.1 against 17.8 on 80).  Those were timed with
//   the weights in the caches.  On a weight that the caches do not hold the narrow kernel's four times as many workgroups draw
//   more: with fewer than 128 here and a long k (149 of 1010 random calls; with K no multiple of 64 each visit's lines are
//   asked for twice) these tiles took 1.19 times as long from memory and 0.95 from the last-level cache, and it stays:
//   9x6693x4656 19.7 us, 25.6 here, 13x4045x3840 12.2 / 16.6, 16x6696x4112 12 % longer here out of the caches too.  Of 884
//   random calls that leave the narrow kernel none is more than 5 % behind with the weight in the L2, six (12 % the worst) out
//   of the last-level cache, 120 (32 %) from memory: 1.38, 1.32 and 1.11 times as fast on average.
// Workgroups are counted against the 256 units of the whole part, on which all of this was measured; on a partition of it the
// plan stays.
constexpr int64_t kFewRowsUnits = 256;
int few_rows_wave_tile(const Args& a, const gemm_plan_t& plan, int64_t cus) {
    constexpr int kQuarter = 16, kNarrow = 5, kWideRowMajor = 0, kWide = 1, kFewRows = 19, kManyRows = 18;
    if (cus != kFewRowsUnits || a.transA || a.batch != 1 || a.M > 64 || a.K > (a.transB ? 8192 : 5000 + 3192 * (plan.kernel == GEMM_KERNEL_SKINNY))) return -1;
    if (a.dtype == gemm::DT_F32 || !gemm::tile_supports(a) || !gemm::tile_variant_supports(a, kManyRows)) return -1;
    const int64_t columns = (a.N + 63) / 64, tiles = ((a.M + 15) / 16) * columns;
    const bool pitch = !a.transB && a.ldb % 256 == 0;
    const double weight = (double)(a.N * a.K) * 2e-6, k = (double)a.K;
    if (plan.kernel == GEMM_KERNEL_SKINNY && (plan.variant == kWideRowMajor || plan.variant == kWide))
        return plan.split_k > 1 && a.M <= 16 && tiles >= 200 && tiles <= 256 && a.K <= 7000 && !(pitch && a.K >= 5000) ? kFewRows : -1;
    const bool narrow = plan.kernel == GEMM_KERNEL_SKINNY;
    if (narrow && columns < 128 && (a.K % 64 ? a.K >= 1500 : columns < 64 && a.K >= 2500)) return -1;
    if (narrow ? plan.variant != kNarrow || plan.split_k != 1 || !a.transB : plan.variant != kQuarter || plan.split_k == 1) return -1;
    if ((pitch && a.K >= 3000) || row_major_stream_on_few_units(a, tiles, cus)) return -1;
    const int straddling = (a.K % 64 != 0) + ((a.transB ? a.K : a.N) % 64 != 0);      // operands whose 128-byte pieces lie in two lines
    const double beyond = weight > 30.0 ? weight - 30.0 : 0.0, uncached = weight > 72.0 ? weight - 72.0 : 0.0;
    const double partial = (double)(a.M * a.N * plan.split_k) * 8e-6;
    double time, wave;
    if (tiles >= (a.K > 4096 && a.transB && columns < 96 ? 96 : a.transB ? 48 : 64) && tiles <= 256 && weight <= 100.0) {
        const double grid = (double)tiles / 256.0;
        time = narrow ? 4.96 + 0.00072 * k + 0.0311 * weight + 0.0776 * beyond + 6.98 * grid
               : a.transB ? 10.3 + 0.00051 * k + 0.119 * beyond + 1.78 * grid + 0.109 * partial
                          : 11.7 + 0.00027 * k + 0.159 * beyond + 0.276 * partial;
        wave = a.transB ? 2.94 + 0.00143 * k * (1.0 + 0.25 * straddling) + 0.2 * uncached + 4.41 * grid
                        : 3.10 + 0.00159 * k * (1.0 + 0.28 * straddling) + 0.2 * uncached + 2.09 * grid;
        return wave < 0.95 * time ? kFewRows : -1;
    }
    if (a.M <= 16 || columns < 80 || columns > 256 || weight > 130.0) return -1;
    const double grid = (double)columns / 256.0;
    time = a.transB ? 10.7 + 3.3 * grid + 0.232 * partial + 0.234 * beyond : 12.1 + 1.2 * grid + 0.164 * partial + 0.209 * beyond;
    wave = a.transB ? 4.3 + 0.00275 * k * (1.0 + 0.2 * straddling) + 0.25 * uncached + 0.5 * grid : 5.0 + 0.00272 * k * (1.0 + 0.19 * straddling) + 0.226 * uncached;
    return wave < 0.93 * time ? kManyRows : -1;
}

// Whether a call is cut along k does not depend on beta, the bias or the activation, so the wave tiles are estimated for one
// epilogue per type of C, a C of 32 bits as read and one of 16 as written only: a caller that made a call without reading C, so
// that the workspace is there, and then captures it with beta = 1 must not find that the second one needs a workspace and the
// first did not (112x6664x2712 TT was such a call: one launch with C written only, 4 shares with C read).
TileChoice choose_tile(const Args& call, int num_cus) {
    TileChoice c = choose_shared_k_tile(call, num_cus);      // (which asks the epilogue only whether the persistent kernel takes it)
    Args a = call;
    a.beta = a.out_dtype == gemm::DT_F32 ? 1.0f : 0.0f; a.bias = nullptr; a.act = gemm::ACT_NONE;
    const int64_t cus = num_cus > 0 ? num_cus : 256;
    if (a.dtype == gemm::DT_F32 || c.time <= 0.0 || c.variant == kPersistentShortK) return c;
    double time = 0.0;
    const int wave_tile = gemm::wave_tile_for(a, cus, &time);
    if (wave_tile < 0) return c;
    if (c.variant == kSmallTileVariant || c.variant == kSmallTileShortK) {
        if (c.parts == 1) {      // (launched on the wave tile: kernel_of)
            if (!gemm::whole_128_tiles_ahead(a, cus)) c.time = time;
            return c;
        }
        if (a.K >= kLongSlicedK) return c;
    } else if (c.variant != kQuarterTile.variant || (c.parts > 1 && a.transA && a.K > kLongSlicedK)) {
        return c;
    }
    if (c.parts > 1 && !a.transA && row_major_stream_on_few_units(a, ((a.M + 15) / 16) * ((a.N + 63) / 64), cus)) return c;
    if (c.parts > 1 && a.M > 32 && ((a.M + 63) / 64) * ((a.N + 63) / 64) <= kFewWaveTiles) return c;
    return c.parts == 1 || time < c.time ? TileChoice{wave_tile, 0, 1, time} : c;
}

// Makes the workspace at least `bytes` large without waiting for anything: a buffer that is too
// small is set aside (launches already enqueued, on this or another stream, may still be using it)
// and a new one of at least twice its size is allocated.
gemm_status_t ensure_workspace(gemm_handle_s* h, size_t bytes) {
    if (bytes <= h->workspace_bytes) return GEMM_OK;
    if (h->workspace && h->num_retired >= kMaxRetired) return GEMM_ERR_ALLOC;
    size_t want = bytes < ((size_t)32 << 20) ? ((size_t)32 << 20) : bytes;
    if (want < 2 * h->workspace_bytes) want = 2 * h->workspace_bytes;
    void* p = nullptr;
    if (hipMalloc(&p, want) != hipSuccess) {
        (void)hipGetLastError();
        if (want == bytes || hipMalloc(&p, bytes) != hipSuccess) { (void)hipGetLastError(); return GEMM_ERR_ALLOC; }
        want = bytes;
    }
    if (h->workspace) h->retired[h->num_retired++] = h->workspace;
    h->workspace = (float*)p;
    h->workspace_bytes = want;
    return GEMM_OK;
}

// Address of the static scratch on `device`, which must be current; looked up on first use.
gemm_status_t scratch_of_device(int device, float** out) {
    static void* table[kMaxDevices];          // (written once per device; a race writes the same value twice)
    if (device < 0 || device >= kMaxDevices) return GEMM_ERR_HIP;
    if (!table[device]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) { (void)hipGetLastError(); return GEMM_ERR_HIP; }
        table[device] = p;
    }
    *out = (float*)table[device];
    return GEMM_OK;
}

// Where a call's partial results go: the handle's own buffer, which may grow, or the static scratch,
// which may not.
struct Workspace {
    gemm_handle_s* h;
    bool fixed;
    float* ptr() const { return fixed ? h->scratch : h->workspace; }
    gemm_status_t ensure(size_t bytes) const {
        if (fixed) return bytes <= kScratchBytes ? GEMM_OK : GEMM_ERR_SCRATCH_LIMIT;
        return ensure_workspace(h, bytes);
    }
    // the same for a plan that can do without: false where there is nothing to be had (never: the static scratch)
    bool obtain(size_t bytes, hipStream_t stream) const {
        if (fixed || bytes <= h->workspace_bytes) return ensure(bytes) == GEMM_OK;
        hipStreamCaptureStatus capturing = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(stream, &capturing) != hipSuccess) { (void)hipGetLastError(); return false; }
        return capturing == hipStreamCaptureStatusNone && ensure(bytes) == GEMM_OK;
    }
};

gemm_status_t free_retired(gemm_handle_s* h) {
    gemm_status_t st = GEMM_OK;
    for (int i = 0; i < h->num_retired; ++i)
        if (hipFree(h->retired[i]) != hipSuccess) { (void)hipGetLastError(); st = GEMM_ERR_HIP; }
    h->num_retired = 0;
    return st;
}

}  // namespace

GEMM_EXPORT gemm_status_t gemm_create(gemm_handle_t* out) {
    if (!out) return GEMM_ERR_INVALID_ARG;
    *out = nullptr;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) { (void)hipGetLastError(); return GEMM_ERR_HIP; }
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) {
        (void)hipGetLastError();
        return GEMM_ERR_HIP;
    }
    gemm_handle_s* h = new (std::nothrow) gemm_handle_s();
    if (!h) return GEMM_ERR_ALLOC;
    h->device = dev;
    h->num_cus = cus > 0 ? cus : 256;
    h->workspace = nullptr;
    h->workspace_bytes = 0;
    h->num_retired = 0;
    h->scratch = nullptr;
    {
        const gemm_status_t st = scratch_of_device(dev, &h->scratch);
        if (st != GEMM_OK) { delete h; return st; }
    }
    h->forced = false;
    h->plan = gemm_plan_t{GEMM_KERNEL_AUTO, -1, 0};
    h->last = gemm_plan_t{GEMM_KERNEL_AUTO, -1, 0};
    h->launched = h->last;
    *out = h;
    return GEMM_OK;
}

GEMM_EXPORT gemm_status_t gemm_destroy(gemm_handle_t h) {
    if (!h) return GEMM_OK;
    gemm_status_t st = free_retired(h);
    if (h->workspace && hipFree(h->workspace) != hipSuccess) {
        (void)hipGetLastError();
        st = GEMM_ERR_HIP;
    }
    delete h;
    return st;
}

GEMM_EXPORT gemm_status_t gemm_reserve_workspace(gemm_handle_t h, size_t bytes) {
    if (!h) return GEMM_ERR_INVALID_ARG;
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) { (void)hipGetLastError(); return GEMM_ERR_HIP; }
    if (dev != h->device) return GEMM_ERR_INVALID_ARG;
    // the caller has synchronised: nothing uses the replaced buffers any more
    gemm_status_t st = free_retired(h);
    if (st != GEMM_OK) return st;
    st = ensure_workspace(h, bytes);
    if (st != GEMM_OK) return st;
    return free_retired(h);
}

GEMM_EXPORT gemm_status_t gemm_workspace_size(gemm_handle_t h, size_t* bytes) {
    if (!h || !bytes) return GEMM_ERR_INVALID_ARG;
    *bytes = h->workspace_bytes;
    return GEMM_OK;
}

GEMM_EXPORT const char* gemm_status_string(gemm_status_t s) {
    switch (s) {
        case GEMM_OK: return "success";
        case GEMM_ERR_INVALID_ARG: return "invalid argument";
        case GEMM_ERR_UNSUPPORTED: return "unsupported combination";
        case GEMM_ERR_ALLOC: return "workspace allocation failed";
        case GEMM_ERR_HIP: return "HIP call or kernel launch failed";
        case GEMM_ERR_SCRATCH_LIMIT: return "the call needs more split-K scratch than the static buffer of gemm_run_noalloc holds";
    }
    return "unknown status";
}

GEMM_EXPORT gemm_status_t gemm_set_plan(gemm_handle_t h, const gemm_plan_t* plan) {
    if (!h) return GEMM_ERR_INVALID_ARG;
    if (!plan) { h->forced = false; return GEMM_OK; }
    if (plan->kernel < GEMM_KERNEL_AUTO || plan->kernel > GEMM_KERNEL_SKINNY) return GEMM_ERR_INVALID_ARG;
    if (plan->split_k < 0 || plan->split_k > 64) return GEMM_ERR_INVALID_ARG;
    if (plan->variant < -1) return GEMM_ERR_INVALID_ARG;
    if (plan->kernel == GEMM_KERNEL_MFMA_TILE && plan->variant >= gemm::tile_num_variants()) return GEMM_ERR_INVALID_ARG;
    h->forced = plan->kernel != GEMM_KERNEL_AUTO;
    h->plan = *plan;
    return GEMM_OK;
}

GEMM_EXPORT gemm_status_t gemm_get_last_plan(gemm_handle_t h, gemm_plan_t* out) {
    if (!h || !out) return GEMM_ERR_INVALID_ARG;
    *out = h->last;
    return GEMM_OK;
}

GEMM_EXPORT gemm_status_t gemm_get_last_launch(gemm_handle_t h, gemm_plan_t* out) {
    if (!h || !out) return GEMM_ERR_INVALID_ARG;
    *out = h->launched;
    return GEMM_OK;
}

GEMM_EXPORT const char* gemm_variant_name(gemm_kernel_t kernel, int32_t variant) {
    if (kernel == GEMM_KERNEL_MFMA_TILE) {
        const gemm::TileVariantInfo* info = gemm::tile_variant_info(variant);
        return info ? info->name : nullptr;
    }
    if (kernel == GEMM_KERNEL_GENERAL) return gemm::general_variant_name(variant);
    if (kernel == GEMM_KERNEL_SKINNY) return gemm::skinny_variant_name(variant);
    return nullptr;
}

namespace {

// The product `a` as a strided batch of `slices` ranges of k, `len` elements each but the last, into fp32 partial results
// whose rows are `ld` apart.
Args slices_of(const Args& a, int slices, int64_t len, float* partials, int64_t ld) {
    Args p = a;
    p.K = len; p.k_total = a.K;
    p.batch = slices;
    p.strideA = a.transA ? len * a.lda : len;
    p.strideB = a.transB ? len : len * a.ldb;
    p.C = partials; p.ldc = ld; p.strideC = a.M * ld;
    p.out_dtype = gemm::DT_F32; p.alpha = 1.0f; p.beta = 0.0f; p.bias = nullptr; p.act = gemm::ACT_NONE;
    return p;
}

int64_t general_slice_len(int64_t K, int& slices);
int wave_any_rows(const Args& a, int slices, int num_cus);

// The kernel that an automatic plan is launched on.  The plan says which family takes the call, in how many slices and with how much
// workspace; several are launched, whatever their slices, as one kernel whose waves divide the k range, or on another pipeline
// of the same tile, at the sizes at which that is faster.  A forced plan is launched as it stands.
gemm_plan_t kernel_of(const Args& a, const gemm_plan_t& plan, int split_first, int num_cus) {
    int variant = -1;
    if (plan.kernel == GEMM_KERNEL_GENERAL) {
        const int rows = plan.variant == 1 ? wave_any_rows(a, plan.split_k, num_cus) : 0;
        return rows ? gemm_plan_t{GEMM_KERNEL_GENERAL, rows == 16 ? gemm::kGeneralWave16 : gemm::kGeneralWave64, 1} : plan;
    }
    if (plan.kernel == GEMM_KERNEL_MFMA_TILE && plan.variant == kF32SmallTileVariant) variant = wave_f32_variant(a, plan.split_k, num_cus);
    else if (plan.kernel == GEMM_KERNEL_MFMA_TILE && plan.split_k == 1) variant = gemm::whole_tile_variant(a, plan.variant, num_cus);
    else if (plan.kernel == GEMM_KERNEL_SKINNY || split_first == 0) variant = few_rows_wave_tile(a, plan, num_cus);
    return variant >= 0 ? gemm_plan_t{GEMM_KERNEL_MFMA_TILE, variant, 1} : plan;
}

bool same_plan(const gemm_plan_t& x, const gemm_plan_t& y) { return x.kernel == y.kernel && x.variant == y.variant && x.split_k == y.split_k; }

// Launches the kernels of a plan for the (validated) call `a`; may lower plan.split_k to what the
// call can take.  split_first: first tile of a split trailing round (macro-tile family).
// automatic: the library chose the plan, and kernel_of it is launched.  `launched`: what was.
// allocate_only: stop after making the workspace large enough for the plan (whatever kernel_of it is: another call of these
// sizes, with another epilogue, may need it where nothing can be allocated).
gemm_status_t launch_plan(const Workspace& ws, const Args& a, gemm_plan_t& plan, int split_first, hipStream_t stream, bool automatic,
                          gemm_plan_t* launched, bool allocate_only = false) {
    const int64_t M = a.M, N = a.N, K = a.K, batch = a.batch;
    const int64_t in_bytes = gemm::elem_bytes(a.dtype);
    const gemm_plan_t kernel = automatic ? kernel_of(a, plan, split_first, ws.h->num_cus) : plan;
    const bool in_one_launch = !same_plan(kernel, plan);
    const int variant = plan.kernel == GEMM_KERNEL_MFMA_TILE ? gemm::tile_variant_for_layout(a, plan.variant) : plan.variant;
    hipError_t e = hipSuccess;
    gemm_status_t st = GEMM_OK;
    bool side_by_side = true;
    int64_t slice_len = 0;
    // ---- the slices that there are, and the workspace ----
    if (plan.kernel == GEMM_KERNEL_SKINNY) {
        const int max_split = gemm::skinny_max_split(a, plan.variant);
        if (plan.split_k > max_split) plan.split_k = max_split;
        const size_t need = gemm::skinny_workspace_bytes(a, plan.split_k);
        if (need) st = ws.ensure(need);
    } else if (plan.kernel == GEMM_KERNEL_MFMA_TILE && plan.split_k > 1) {
        const int64_t slabs = (K + 31) / 32;
        if (plan.split_k > slabs) plan.split_k = (int)slabs;
        if (plan.split_k > 1 && !gemm::tile_variant_splits(variant)) {
            // k slices: ranges of whole 32-element slabs, all of one length but the last
            slice_len = ((slabs + plan.split_k - 1) / plan.split_k) * 32;
            plan.split_k = (int)((K + slice_len - 1) / slice_len);
            if (plan.split_k > 1) st = ws.ensure((size_t)plan.split_k * (size_t)M * (size_t)N * sizeof(float));
        } else if (plan.split_k > 1) {
            const gemm::TileVariantInfo* info = gemm::tile_variant_info(variant);
            const int64_t tiles = ((a.M + info->BM - 1) / info->BM) * ((a.N + info->BN - 1) / info->BN);
            st = ws.ensure((size_t)(tiles - split_first) * plan.split_k * info->BM * info->BN * sizeof(float));
        }
    } else if (plan.kernel == GEMM_KERNEL_GENERAL && plan.split_k > 1) {
        // k slices, as above; a call of this family has never failed for want of a workspace, so where there is none to
        // be had (the stream is being captured, memory is out) its slices are computed one after another, to the same bits
        slice_len = general_slice_len(K, plan.split_k);
        if (plan.split_k > 1) {
            const size_t need = (size_t)plan.split_k * (size_t)M * (size_t)((N + 7) / 8 * 8) * sizeof(float);
            if (ws.fixed && need > kScratchBytes) return GEMM_ERR_SCRATCH_LIMIT;
            side_by_side = ws.obtain(need, stream);
        }
    }
    if (st != GEMM_OK || allocate_only) return st;
    // ---- launch ----
    *launched = in_one_launch ? kernel : gemm_plan_t{plan.kernel, variant, plan.split_k};
    const gemm::TileSplit whole{0, 1, nullptr};
    if (kernel.kernel == GEMM_KERNEL_MFMA_TILE && (in_one_launch || plan.split_k == 1)) {
        e = gemm::launch_tile(a, launched->variant, kTileBandRows, whole, stream);
    } else if (kernel.kernel == GEMM_KERNEL_MFMA_TILE && slice_len > 0) {
        e = gemm::launch_tile(slices_of(a, plan.split_k, slice_len, ws.ptr(), N), variant, kTileBandRows, whole, stream);
        if (e == hipSuccess) e = gemm::launch_splitk_reduce(a, plan.split_k, ws.ptr(), stream);
    } else if (kernel.kernel == GEMM_KERNEL_MFMA_TILE) {
        const gemm::TileSplit split{split_first, plan.split_k, ws.ptr()};
        e = gemm::launch_tile(a, variant, kTileBandRows, split, stream);
        if (e == hipSuccess) e = gemm::launch_tile_split_reduce(a, variant, kTileBandRows, split, stream);
    } else if (kernel.kernel == GEMM_KERNEL_SKINNY) {
        // one matrix per launch (the slices of a split share the workspace, in stream order)
        Args one = a;
        one.batch = 1;
        for (int64_t b = 0; b < batch && e == hipSuccess; ++b) {
            one.A = (const char*)a.A + b * a.strideA * in_bytes;
            one.B = (const char*)a.B + b * a.strideB * in_bytes;
            one.C = (char*)a.C + b * a.strideC * gemm::elem_bytes(a.out_dtype);
            e = gemm::launch_skinny(one, plan.split_k, ws.ptr(), stream, plan.variant);
        }
    } else {
        const bool fold = a.out_dtype == gemm::DT_F32;
        if (in_one_launch || plan.split_k == 1) {
            e = gemm::launch_general(a, kernel.variant, kTileBandRows, stream, fold);
        } else if (!side_by_side) {
            e = gemm::launch_general(a, plan.variant, kTileBandRows, stream, fold, slice_len);
        } else {
            const int64_t P = (N + 7) / 8 * 8;
            e = gemm::launch_general(slices_of(a, plan.split_k, slice_len, ws.ptr(), P), plan.variant, kTileBandRows, stream, fold);
            if (e == hipSuccess) e = gemm::launch_splitk_reduce(a, plan.split_k, ws.ptr(), stream);
        }
    }
    return e == hipSuccess ? GEMM_OK : GEMM_ERR_HIP;
}

// Remainder peeling.  A C whose last column (or row) of 256-wide tiles is nearly empty pays a whole
// tile's k loop for a few columns there, and that column of tiles can cost a round of its own
// (8000x8200x8136: 33 tile columns for 8 columns of C, 1056 tiles = four rounds and 32 tiles).  The
// call is then made in two: the whole tiles, and the remaining thin strip as a call of its own, which
// the choice above sends to small tiles cut along K.  Taken when the two estimates together are 3 %
// below the estimate for the whole; a strip is at most 64 wide.  `rest` starts where `main_part` ends.
constexpr int64_t kPeelWidest = 64;
constexpr double kPeelGain = 0.97, kSecondLaunch = 3.0;

bool peel_remainder(const Args& a, int num_cus, double whole_time, Args* main_part, Args* rest, TileChoice* main_choice,
                    TileChoice* rest_choice) {
    if (a.batch != 1 || whole_time <= 0.0) return false;
    const int64_t in_bytes = gemm::elem_bytes(a.dtype), out_bytes = gemm::elem_bytes(a.out_dtype);
    bool found = false;
    double best = kPeelGain * whole_time;
    for (int side = 0; side < 2; ++side) {                  // 0: columns, 1: rows
        const int64_t extent = side == 0 ? a.N : a.M, whole = (extent / 256) * 256, strip = extent - whole;
        if (whole < 256 || strip <= 0 || strip > kPeelWidest) continue;
        Args m = a, r = a;
        if (side == 0) {
            m.N = whole; r.N = strip;
            r.B = (const char*)a.B + (a.transB ? whole * a.ldb : whole) * in_bytes;
            r.C = (char*)a.C + whole * out_bytes;
            if (a.bias) r.bias = (const char*)a.bias + whole * gemm::elem_bytes(a.bias_dtype);
        } else {
            m.M = whole; r.M = strip;
            r.A = (const char*)a.A + (a.transA ? whole : whole * a.lda) * in_bytes;
            r.C = (char*)a.C + whole * a.ldc * out_bytes;
        }
        if (!gemm::tile_supports(m) || !gemm::tile_supports(r)) continue;
        const TileChoice cm = choose_tile(m, num_cus), cr = choose_tile(r, num_cus);
        if (cm.time <= 0.0 || cr.time <= 0.0) continue;
        const double t = cm.time + cr.time + kSecondLaunch;
        if (t < best) { best = t; found = true; *main_part = m; *rest = r; *main_choice = cm; *rest_choice = cr; }
    }
    return found;
}

// The roofline rule of the paper (Section 4.3) as arithmetic.  A kernel is placed by its arithmetic
// intensity, flop per byte of compulsory traffic: left of the point where the roof of the
// lowest-throughput unit (the fp32 vector ALUs) meets the memory roof it is memory-bound, right of the
// point where the roof of the highest-throughput unit that can do the work (the matrix cores for the
// operand type) meets it, compute-bound, in between in the middle zone.  The class names the resource
// to optimise for: memory-bound and middle-zone calls are candidates for the streaming (skinny)
// family, whose objective is bytes per second on one pass over B; compute-bound calls go to the
// macro-tile family, whose objective is matrix-core occupancy, and never to the streaming family.
// For fp32 that unit's roof is taken at the fp32 instruction's rate, which is the vector ALUs' too, although products of bf16 pieces
// reach up to 417 TFLOP/s (2.5e15 / 6): the streaming fp32 kernels multiply on the vector ALUs, so where those meet the
// memory roof is where streaming ends, and fp32 has no middle zone.
constexpr double kPeakVectorFlops = 157.3e12, kPeakMatrixFlops16 = 2.5e15, kPeakMatrixFlops32 = 157.3e12, kPeakMemoryBytes = 8.0e12;

struct Roofline { double intensity; gemm_roofline_t cls; };

Roofline roofline_of(int64_t batch, int64_t M, int64_t N, int64_t K, int dtype, int out_dtype, bool reads_c, int bias_dtype) {
    const double in_b = (double)gemm::elem_bytes(dtype), out_b = (double)gemm::elem_bytes(out_dtype);
    double bytes = ((double)M * (double)K + (double)K * (double)N) * in_b + (double)M * (double)N * out_b * (reads_c ? 2.0 : 1.0);
    bytes *= (double)batch;
    if (bias_dtype >= 0) bytes += (double)N * (double)gemm::elem_bytes(bias_dtype);
    const double flops = 2.0 * (double)M * (double)N * (double)K * (double)batch;
    Roofline r;
    r.intensity = bytes > 0.0 ? flops / bytes : 0.0;
    const double ridge_low = kPeakVectorFlops / kPeakMemoryBytes;
    const double ridge_high = (dtype == gemm::DT_F32 ? kPeakMatrixFlops32 : kPeakMatrixFlops16) / kPeakMemoryBytes;
    r.cls = r.intensity < ridge_low ? GEMM_MEMORY_BOUND : (r.intensity > ridge_high ? GEMM_COMPUTE_BOUND : GEMM_MIDDLE_ZONE);
    return r;
}

Roofline roofline_of(const Args& a) {
    return roofline_of(a.batch, a.M, a.N, a.K, a.dtype, a.out_dtype, a.beta != 0.0f, a.bias ? a.bias_dtype : -1);
}

// Inside the two classes that may stream, measurements break the tie between the families.  16-bit
// operands: the skinny kernels are ahead where B is a long stream - up to 32 rows, B of 128 MiB or
// more, K >= 4096, N >= 4096 (fewer than 16 column groups need more than 16 slices: 16x2048x32768 36
// to 38 us against 31 to 32 on sliced tiles; 32x16384x16384: 94 against 99 us on the 128x256 tile
// with a K split, 16x28672x8192 with B stored N x K: 79 against 92).  Smaller weights run as fast or
// faster as sliced 128x128 tiles or split quarter tiles (1...8 x 4096 x 4096: 11.5 to 12 us against
// 11.5 to 15; 32x2048x2048: 15 to 20 against 19 to 21), and with 33 to 64 rows the 128x256 tile wins
// everywhere (64x16384x16384: 107 against 112 / 126 us).  fp32 operands: up to 8 rows on a B of 16 MiB
// or more take the fp32 streaming kernels (vector ALUs: at half a flop per byte and row the matrix
// cores have nothing to add), everything else the fp32 tiles.
struct AutoPlan {
    gemm_plan_t plan;          // of the call, or of its whole tiles when it is made in two
    int split_first;
    bool peeled;               // made in two: main_part with `plan`, then rest with rest_plan
    Args main_part, rest;
    gemm_plan_t rest_plan;
    int rest_split_first;
};

// Operands off the 16-byte grid: the general kernel for the smallest calls, the matrix cores for the rest, in k slices where
// the tiles leave the chip idle.  Slices have to fit the static scratch, so that every entry point takes the same ones.
// Estimates in us, fitted to all plans on 1250 random calls (M, N 1 to 3072, K 24 to 4096, the four layouts, batches):
// the choice is 0.3 % behind the fastest plan on average, by more than 10 % on 9 of them, and with 16 bits never by more than 6 %
// behind the general kernel.  Nine calls of ten are within 7 % of their estimates.
constexpr int64_t kGeneralMinSliceK = 48;
// (2.6 to 3.1 on the device, more for the call: 33x43x223 fp32 10.2 us plain, 10.8 in 4 slices; none / SiLU / GELU on the
// 16-bit tile 215x127x181 11.7 / 12.4 / 13.8, 335x75x629 20.3 / 21.1 / 22.4; on the fp32 one 0.1 to 0.4 more than none; 1.5
// there too left 65x23x223 with GELU at 11.3 in 4 slices where one takes 8.9 and the general kernel 10.2)
constexpr double kSecondKernel = 3.4, kActivation = 1.5, kActivationF32 = 0.3;
constexpr double kGeneralMargin = 1.08;       // what the 16-bit tiles must promise (without it up to 22 % behind the general kernel); the fp32 ones round less

// The general kernel: 0.55 us per step of 16 along k, and its throughput (beyond four blocks per unit less each).
double general_time(const Args& a) {
    const double blocks = (double)((a.M + 15) / 16) * (double)((a.N + 15) / 16) * (double)a.batch;
    return 2.2 + (double)((a.K + 15) / 16) * (0.55 + 0.00031 * blocks + 0.00026 * (blocks > 1024.0 ? blocks - 1024.0 : 0.0)) + 0.0004 * blocks;
}

// The tiles in `slices` of `len` elements of k.  An operand contiguous along m or n costs more instructions per slab than a
// k-contiguous one, so a slab's time goes by layout (1023x1025x1021 22 us NT, 25 NN, 31 TN).  The epilogue is in proportion to
// a tile's live rows up to 64; a number of slices that the reduction has no instance for costs a round trip each.
double general_tile_time(const Args& a, int slices, int64_t len, int64_t cus) {
    const bool f32 = a.dtype == gemm::DT_F32, fold = !f32 && a.out_dtype == gemm::DT_F32;
    const double elements = (double)a.M * (double)a.N * (double)a.batch;
    double moved = elements * (f32 || fold || slices > 1 ? 4.0 : 2.0), t = 0.0;
    if (a.act != gemm::ACT_NONE && slices == 1) t = f32 ? kActivationF32 : kActivation;
    if (slices > 1) {
        moved += (double)slices * (double)a.M * (double)((a.N + 7) / 8 * 8) * 4.0;
        t = kSecondKernel + (slices == 2 || slices == 4 || slices == 8 || slices == 16 ? 0.0 : 0.36 * slices);
    }
    if (f32) {      // 64x64 tiles with folded sums, up to three workgroups per unit
        const int64_t per_unit = (((a.M + 63) / 64) * ((a.N + 63) / 64) * a.batch * slices + cus - 1) / cus;
        const double per_k = (double)(per_unit / 3) * 0.037 + (per_unit % 3 == 0 ? 0.0 : (per_unit % 3 == 1 ? 0.0185 : 0.0281));
        return t + 4.6 + per_k * (double)len + moved / 2.6e6;
    }
    // 128x128 tiles, two workgroups per unit (one with folded sums); per slab of 64 and layout: up to half a workgroup per unit,
    // up to one, and per round
    static const double few[4] = {0.77, 1.10, 1.01, 1.48}, one[4] = {0.97, 1.27, 1.24, 1.58}, full[4] = {1.22, 1.47, 1.54, 1.89};
    static const double few_folded[4] = {1.15, 1.42, 1.34, 1.78}, full_folded[4] = {1.19, 1.49, 1.33, 1.69};
    const int layout = (a.transA ? 2 : 0) + (a.transB ? 0 : 1);                  // NT, NN, TT, TN
    const int64_t wgs = ((a.M + 127) / 128) * ((a.N + 127) / 128) * a.batch * slices, places = fold ? cus : 2 * cus;
    const double rounds = (double)((wgs + places - 1) / places), slabs = (double)((len + 63) / 64);
    const double live = (double)(a.M < 64 ? a.M : 64) / 64.0;
    if (fold) return t + 5.25 + 4.2 * live + (wgs <= cus / 2 ? few_folded : full_folded)[layout] * slabs * rounds + 4.2 * (rounds - 1.0) + moved / 3.6e6;
    return t + 4.7 + 4.0 * live + (wgs <= cus / 2 ? few : (wgs <= cus ? one : full))[layout] * slabs * rounds + 0.9 * (rounds - 1.0) + moved / 3.3e6;
}

// The length of the `slices` slices a general plan cuts K into (whole 32-element slabs); `slices` becomes what there are.
int64_t general_slice_len(int64_t K, int& slices) {
    const int64_t slabs = (K + 31) / 32, len = ((slabs + slices - 1) / slices) * 32;
    slices = (int)((K + len - 1) / len);
    return slices > 1 ? len : K;
}

// A call that a plan gives to the 16-bit tiles of the general family, in whatever slices, runs in one launch on the tiles whose
// waves divide the k range, 64 or 16 (returned; 0: neither) rows by 64 columns, where those promise to be ahead.  Estimates in
// us, fitted to 210 random calls each (half within 5 %, nine of ten within 14 %).  On the device, on 1150 random calls with
// more than 64 rows the choice is 1.63 times as fast as before on average (eight more than 5 % behind, 17 % the worst), on 1556
// with fewer 1.74 times out of the last-level cache (eight, 16 %) and 1.64 from memory (76, 39 %).  At 2049x2051x2045 the
// three are level (53 to 54 us); at 4095^3 the large tile, which reads half as many bytes, is ahead (255 us against 328), as are
// slices with few columns and a long k (9x979x4043 16.4 against 29.4).  Results of 16 bits only: for an fp32 C slices and folds
// have the smaller error.
constexpr int kMostSlices = 16;
constexpr int64_t kSlicedLongK = 3600;
int wave_any_rows(const Args& a, int slices, int num_cus) {
    const int64_t cus = num_cus > 0 ? num_cus : 256;
    if (a.out_dtype == gemm::DT_F32 || !gemm::general_variant_supports(a, gemm::kGeneralWave64)) return 0;
    struct Tile { int rows; double per_k_alone, per_k, fixed, per_round, store_rate, activation, weight_rate, layout[4]; };
    static const Tile tiles[] = {{64, 0.0041, 0.0038, 5.1, 0.6, 3.4e6, 1.3, 41e6, {1.0, 1.12, 1.34, 1.37}},      // NT, NN, TT, TN
                                 {16, 0.00256, 0.0024, 4.2, 0.0, 1.0e6, 0.6, 23e6, {1.0, 1.05, 0.0, 0.0}}};
    const int layout = (a.transA ? 2 : 0) + (a.transB ? 0 : 1);
    // (slices of a weight stored N x K draw more from memory than few workgroups with a long k do: 40 random calls 1.14 times
    // as long here, 0.92 out of the last-level cache)
    if (slices > 1 && !a.transA && a.transB && a.K > 4096 && ((a.M + 15) / 16) * ((a.N + 63) / 64) * 8 < cus * 3) return 0;
    int sl = slices > 1 ? slices : 1, rows = 0;
    const int64_t len = sl > 1 ? general_slice_len(a.K, sl) : a.K;
    double best = general_tile_time(a, sl, len, cus);
    for (const Tile& t : tiles) {
        if (t.layout[layout] == 0.0) continue;      // (a k-row of 16 elements of an A stored K x M is no whole line)
        const int64_t rounds = (((a.M + t.rows - 1) / t.rows) * ((a.N + 63) / 64) * a.batch + cus - 1) / cus;
        const double time = t.fixed + t.per_round * (double)rounds + (rounds == 1 ? t.per_k_alone : t.per_k * (double)rounds) * t.layout[layout] * (double)a.K +
                            (double)(a.M * a.N * a.batch) * 2.0 / t.store_rate + (a.act != gemm::ACT_NONE ? t.activation : 0.0) +
                            (double)(a.N * a.K * a.batch) * 2.0 / t.weight_rate;
        // (10 % promised beyond what is resident at once: with 7 to 10 nine random calls were 1.06 times as long here,
        // 2711x1985x131 NN 18.0 against 16.4 us)
        if (time < best * (rounds > 2 ? 0.9 : 1.0)) { best = time; rows = t.rows; }
    }
    // (sixteen slices of a long k, where the 16-row tiles would leave half of the units idle: those stay.  140 random calls 1.10 times
    // as long here from memory, 1.01 out of the last-level cache: 57x982x3883 NT 16.8 us against 21.0 and 15.5 against 17.7)
    const int64_t strips = ((a.M + 15) / 16) * ((a.N + 63) / 64);
    if (rows == 16 && slices == kMostSlices && a.M <= 128 && a.K >= kSlicedLongK && 2 * strips <= cus) return 0;
    return rows;
}

gemm_plan_t general_plan(const Args& a, int num_cus) {
    const int64_t cus = num_cus > 0 ? num_cus : 256;
    gemm_plan_t plan{GEMM_KERNEL_GENERAL, 0, 1};
    const bool f32 = a.dtype == gemm::DT_F32;
    const int variant = f32 ? 2 : 1;
    if (!gemm::general_variant_supports(a, variant)) return plan;
    double best = general_time(a) / (f32 ? 1.0 : kGeneralMargin);
    for (int cut : {1, 2, 4, 8, 16}) {
        if (cut > 1 && (a.batch != 1 || a.K / cut < kGeneralMinSliceK || (int64_t)cut * a.M * ((a.N + 7) / 8 * 8) * 4 > (int64_t)kScratchBytes)) break;
        int slices = cut;
        const int64_t len = general_slice_len(a.K, slices);
        const double t = general_tile_time(a, slices, len, cus);
        if (t < best) { best = t; plan.variant = variant; plan.split_k = slices; }
    }
    return plan;
}

AutoPlan automatic_plan(const Args& a, int num_cus, bool batch_aligned) {
    AutoPlan ap;
    ap.plan = gemm_plan_t{GEMM_KERNEL_GENERAL, 0, 1};
    ap.split_first = -1;
    ap.peeled = false;
    ap.rest_plan = ap.plan;
    ap.rest_split_first = -1;
    const Roofline roof = roofline_of(a);
    const bool may_stream = roof.cls != GEMM_COMPUTE_BOUND && gemm::skinny_supports(a) && batch_aligned;
    // fp32: B stored N x K from 16 MiB on; a row-major B from 16 MiB per row of C on (its kernel spends vector
    // instructions per row: 8 x 4096 x 4096 43 us against 29 on the fp32 tiles, 8 x 8192 x 8192 73 against 85)
    const bool long_stream = a.dtype == gemm::DT_F32
                                 ? (a.N * a.K * 4 >= kSkinnyAutoBytesF32 * (a.transB ? 1 : a.M) && a.K >= 1024 && a.N >= 1024)
                                 : (a.M <= kSkinnyAutoRows && a.N * a.K * 2 >= kSkinnyAutoBytes && a.K >= 4096 && a.N >= 4096 && !a.transA);
    // An A stored K x M costs the streaming kernels a copy (3 to 4 us: 8 x 8192 x 8192 33 us against 30 on split
    // quarter tiles, 32 x 16384 x 16384 98 against 93), so they take it only where the macro tiles cannot: a row
    // count that is no multiple of 8, which would otherwise fall to the general kernel.
    const bool only_stream = a.transA && !gemm::tile_supports(a);
    // up to four rows on a 16-bit weight stored N x K: one launch of the vector-ALU kernel, at every size
    // (1 x 4096 x 4096 6.4 us against 12.0 on split tiles, 1 x 512 x 512 5.8 against 8.0); a batch would be
    // one launch per matrix and stays with the tiles
    // ... and up to 16 rows on such a weight with at most 4096 stored rows and below 128 MiB: one launch of the
    // MFMA kernel with 16 columns per workgroup (8 x 4096 x 4096 8.7 us against 12.3)
    const bool few_rows = a.dtype != gemm::DT_F32 && a.batch == 1 && gemm::skinny_supports(a) &&
                          (gemm::skinny_variant_of(a) == 4 || gemm::skinny_variant_of(a) == 5);
    // ... the same two kernels where only the number of stored rows (columns of C) is no multiple of 8: without a split
    // nothing in them works on groups of columns
    const int ragged = batch_aligned && roof.cls != GEMM_COMPUTE_BOUND ? gemm::skinny_ragged_columns_variant(a) : -1;
    if (ragged >= 0) {
        ap.plan = gemm_plan_t{GEMM_KERNEL_SKINNY, ragged, 1};
    } else if (may_stream && (long_stream || only_stream || few_rows)) {
        ap.plan = gemm_plan_t{GEMM_KERNEL_SKINNY, gemm::skinny_variant_of(a), gemm::skinny_default_split(a, num_cus)};
    } else if (gemm::tile_supports(a) && batch_aligned &&
               (a.dtype != gemm::DT_F32 || ((a.M + 63) / 64) * ((a.N + 63) / 64) * a.batch >= kF32MinTiles)) {
        const TileChoice c = choose_tile(a, num_cus);
        ap.plan = gemm_plan_t{GEMM_KERNEL_MFMA_TILE, c.variant, c.parts};
        ap.split_first = c.first_split_tile;
        TileChoice cm, cr;
        if (peel_remainder(a, num_cus, c.time, &ap.main_part, &ap.rest, &cm, &cr)) {
            ap.peeled = true;
            ap.plan = gemm_plan_t{GEMM_KERNEL_MFMA_TILE, cm.variant, cm.parts};
            ap.split_first = cm.first_split_tile;
            ap.rest_plan = gemm_plan_t{GEMM_KERNEL_MFMA_TILE, cr.variant, cr.parts};
            ap.rest_split_first = cr.first_split_tile;
        }
    } else {
        ap.plan = general_plan(a, num_cus);
    }
    return ap;
}

// Largest number of matrices one launch takes (the y dimension of a grid).
constexpr int64_t kMaxBatchPerLaunch = 65535;

gemm_status_t run_batch(gemm_handle_t h, bool fixed_scratch, int64_t batch, int64_t M, int64_t N, int64_t K,
                        gemm_op_t transA, gemm_op_t transB, gemm_dtype_t dtype,
                        float alpha, const void* A, int64_t lda, int64_t strideA,
                        const void* B, int64_t ldb, int64_t strideB,
                        float beta, void* C, int64_t ldc, int64_t strideC,
                        const gemm_epilogue_t* epilogue, void* stream_) {
    // ---- validation: nothing is launched and C is untouched on any error below ----
    if (!h) return GEMM_ERR_INVALID_ARG;
    if (M < 0 || N < 0 || K < 0 || batch < 0) return GEMM_ERR_INVALID_ARG;
    if (strideA < 0 || strideB < 0 || strideC < 0) return GEMM_ERR_INVALID_ARG;
    if ((transA != GEMM_OP_N && transA != GEMM_OP_T) || (transB != GEMM_OP_N && transB != GEMM_OP_T)) return GEMM_ERR_INVALID_ARG;
    if (!valid_dtype(dtype)) return GEMM_ERR_INVALID_ARG;
    gemm_epilogue_t epi;
    if (epilogue) epi = *epilogue;
    else epi = gemm_epilogue_t{dtype, nullptr, dtype, GEMM_ACT_NONE};
    if (!valid_dtype(epi.out_dtype)) return GEMM_ERR_INVALID_ARG;
    if (epi.bias && !valid_dtype(epi.bias_dtype)) return GEMM_ERR_INVALID_ARG;
    if ((int)epi.act < (int)GEMM_ACT_NONE || (int)epi.act > (int)GEMM_ACT_GELU_TANH) return GEMM_ERR_INVALID_ARG;
    const int64_t a_cols = transA == GEMM_OP_N ? K : M, b_cols = transB == GEMM_OP_N ? N : K;
    if (lda < (a_cols > 1 ? a_cols : 1) || ldb < (b_cols > 1 ? b_cols : 1) || ldc < (N > 1 ? N : 1)) return GEMM_ERR_INVALID_ARG;
    if (M > 0 && N > 0 && !C) return GEMM_ERR_INVALID_ARG;
    if (M > 0 && K > 0 && !A) return GEMM_ERR_INVALID_ARG;
    if (N > 0 && K > 0 && !B) return GEMM_ERR_INVALID_ARG;
    if (epi.out_dtype != dtype && epi.out_dtype != GEMM_F32) return GEMM_ERR_UNSUPPORTED;
    // the matrices of C must not overlap one another
    if (batch > 1 && M > 0 && N > 0 && strideC < (M - 1) * ldc + N) return GEMM_ERR_INVALID_ARG;
    if (M == 0 || N == 0 || batch == 0) return GEMM_OK;
    {   // the handle (its workspace, its compute-unit count) belongs to the device it was created on
        int dev = -1;
        if (hipGetDevice(&dev) != hipSuccess) { (void)hipGetLastError(); return GEMM_ERR_HIP; }
        if (dev != h->device) return GEMM_ERR_INVALID_ARG;
    }
    if (batch > kMaxBatchPerLaunch) {
        // more matrices than one grid holds: consecutive launches over consecutive parts of the batch
        const int64_t ea = gemm::elem_bytes((int)dtype), ec = gemm::elem_bytes((int)epi.out_dtype);
        for (int64_t b0 = 0; b0 < batch; b0 += kMaxBatchPerLaunch) {
            const int64_t nb = batch - b0 < kMaxBatchPerLaunch ? batch - b0 : kMaxBatchPerLaunch;
            const gemm_status_t st = run_batch(h, fixed_scratch, nb, M, N, K, transA, transB, dtype, alpha,
                                               A ? (const char*)A + b0 * strideA * ea : nullptr, lda, strideA,
                                               B ? (const char*)B + b0 * strideB * ea : nullptr, ldb, strideB, beta,
                                               (char*)C + b0 * strideC * ec, ldc, strideC, epilogue, stream_);
            if (st != GEMM_OK) return st;
        }
        return GEMM_OK;
    }

    hipStream_t stream = (hipStream_t)stream_;
    const Workspace ws{h, fixed_scratch};
    Args a;
    a.M = M; a.N = N; a.K = K;
    a.transA = transA == GEMM_OP_T; a.transB = transB == GEMM_OP_T;
    a.dtype = (int)dtype; a.out_dtype = (int)epi.out_dtype; a.bias_dtype = (int)epi.bias_dtype; a.act = (int)epi.act;
    a.alpha = alpha; a.beta = beta;
    a.A = A; a.lda = lda; a.B = B; a.ldb = ldb; a.C = C; a.ldc = ldc;
    a.bias = epi.bias;
    a.batch = (int32_t)batch;
    a.k_total = 0;
    a.strideA = batch > 1 ? strideA : 0; a.strideB = batch > 1 ? strideB : 0; a.strideC = batch > 1 ? strideC : 0;
    // the matrix-core kernels read 16-byte vectors: every matrix of the batch must start on a 16-byte boundary
    const int64_t in_bytes = gemm::elem_bytes(a.dtype);
    const bool batch_aligned = batch == 1 || ((strideA * in_bytes) % 16 == 0 && (strideB * in_bytes) % 16 == 0);

    // ---- plan ----
    gemm_plan_t plan{GEMM_KERNEL_GENERAL, 0, 1};
    int split_first = -1;          // first tile of a split trailing round (macro-tile family)
    bool automatic = false;        // whether the library chose the kernel, not the caller
    gemm_plan_t launched = plan;
    const bool product = (K > 0 && alpha != 0.0f);
    if (!product) {
        plan = gemm_plan_t{GEMM_KERNEL_GENERAL, 0, 1};      // only the epilogue is left
    } else if (h->forced) {
        plan = h->plan;
        if (plan.kernel == GEMM_KERNEL_MFMA_TILE) {
            if (!gemm::tile_supports(a) || !batch_aligned) return GEMM_ERR_UNSUPPORTED;
            if (plan.variant < 0) {
                automatic = plan.split_k <= 1;
                const TileChoice c = choose_tile(a, h->num_cus);
                plan.variant = c.variant;
                if (plan.split_k == 0) { plan.split_k = c.parts; split_first = c.first_split_tile; }
            }
            if (!gemm::tile_variant_supports(a, plan.variant)) return GEMM_ERR_UNSUPPORTED;
            if (plan.split_k < 1) plan.split_k = 1;
            if (plan.split_k > 1 && batch > 1) return GEMM_ERR_UNSUPPORTED;
            if (plan.split_k > 1 && !gemm::tile_variant_splits(plan.variant) && N % 8 != 0) return GEMM_ERR_UNSUPPORTED;
            if (plan.split_k > 1 && gemm::tile_variant_splits(plan.variant) && split_first < 0) {
                // a forced split applies to the trailing partial round, or to every tile of a grid smaller than one round
                const gemm::TileVariantInfo* info = gemm::tile_variant_info(plan.variant);
                const int64_t tiles = ((a.M + info->BM - 1) / info->BM) * ((a.N + info->BN - 1) / info->BN);
                const int64_t cus = h->num_cus > 0 ? h->num_cus : 256;
                split_first = (int)(tiles - tiles % cus);
                if (split_first == tiles) plan.split_k = 1;
            }
        } else if (plan.kernel == GEMM_KERNEL_SKINNY && plan.variant >= 4 && plan.split_k == 1 && batch_aligned &&
                   plan.variant == gemm::skinny_ragged_columns_variant(a)) {
            // (a plan that the automatic choice reported can be forced)
        } else if (plan.kernel == GEMM_KERNEL_SKINNY) {
            if (!gemm::skinny_supports(a) || !batch_aligned) return GEMM_ERR_UNSUPPORTED;
            if (!gemm::skinny_variant_serves(a, plan.variant)) return GEMM_ERR_UNSUPPORTED;
            if (plan.variant < 0) plan.variant = gemm::skinny_variant_of(a);
            if (plan.split_k == 0) plan.split_k = gemm::skinny_default_split(a, h->num_cus, plan.variant);
        } else if (plan.variant < 1 || !gemm::general_variant_supports(a, plan.variant) || plan.variant >= gemm::kGeneralVariants) {
            plan = gemm_plan_t{GEMM_KERNEL_GENERAL, 0, 1};      // (the one that takes everything)
        } else if (plan.split_k < 1 || batch > 1 || plan.variant >= gemm::kGeneralWave64) {
            plan.split_k = 1;
        }
    } else {
        const AutoPlan ap = automatic_plan(a, h->num_cus, batch_aligned);
        plan = ap.plan;
        split_first = ap.split_first;
        automatic = true;
        if (ap.peeled) {
            gemm_plan_t pm = ap.plan, pr = ap.rest_plan;
            // the workspace of both parts first: a failed allocation must leave C untouched
            gemm_plan_t rest_launched = pr;
            gemm_status_t st = launch_plan(ws, ap.main_part, pm, ap.split_first, stream, automatic, &launched, true);
            if (st == GEMM_OK) st = launch_plan(ws, ap.rest, pr, ap.rest_split_first, stream, automatic, &rest_launched, true);
            if (st != GEMM_OK) return st;
            st = launch_plan(ws, ap.main_part, pm, ap.split_first, stream, automatic, &launched);
            if (st == GEMM_OK) st = launch_plan(ws, ap.rest, pr, ap.rest_split_first, stream, automatic, &rest_launched);
            if (st != GEMM_OK) return st;
            h->last = pm;         // the plan of the whole tiles
            h->launched = launched;
            return GEMM_OK;
        }
    }

    // ---- launch ----
    const gemm_status_t st = launch_plan(ws, a, plan, split_first, stream, automatic, &launched);
    if (st != GEMM_OK) return st;
    h->last = plan;
    h->launched = launched;
    return GEMM_OK;
}

}  // namespace

GEMM_EXPORT gemm_status_t gemm_roofline_class(int64_t batch, int64_t M, int64_t N, int64_t K, gemm_dtype_t dtype, gemm_dtype_t out_dtype,
                                              int32_t reads_c, int32_t has_bias, gemm_dtype_t bias_dtype, gemm_roofline_t* cls,
                                              double* intensity) {
    if (!cls || batch < 1 || M < 1 || N < 1 || K < 1) return GEMM_ERR_INVALID_ARG;
    if (!valid_dtype(dtype) || !valid_dtype(out_dtype) || (has_bias && !valid_dtype(bias_dtype))) return GEMM_ERR_INVALID_ARG;
    const Roofline r = roofline_of(batch, M, N, K, (int)dtype, (int)out_dtype, reads_c != 0, has_bias ? (int)bias_dtype : -1);
    *cls = r.cls;
    if (intensity) *intensity = r.intensity;
    return GEMM_OK;
}

namespace {

// The automatic plan of a call on aligned operands that are never looked at; `call`: the call.
gemm_status_t query(int32_t compute_units, int64_t batch, int64_t M, int64_t N, int64_t K, gemm_op_t transA, gemm_op_t transB, gemm_dtype_t dtype,
                    gemm_dtype_t out_dtype, int64_t lda, int64_t ldb, int64_t ldc, bool reads_c, gemm_act_t act, Args* call, AutoPlan* plan) {
    if (compute_units < 1 || batch < 1 || M < 1 || N < 1 || K < 1) return GEMM_ERR_INVALID_ARG;
    if ((transA != GEMM_OP_N && transA != GEMM_OP_T) || (transB != GEMM_OP_N && transB != GEMM_OP_T)) return GEMM_ERR_INVALID_ARG;
    if (!valid_dtype(dtype) || !valid_dtype(out_dtype)) return GEMM_ERR_INVALID_ARG;
    if ((int)act < (int)GEMM_ACT_NONE || (int)act > (int)GEMM_ACT_GELU_TANH) return GEMM_ERR_INVALID_ARG;
    if (out_dtype != dtype && out_dtype != GEMM_F32) return GEMM_ERR_UNSUPPORTED;
    const int64_t a_cols = transA == GEMM_OP_N ? K : M, b_cols = transB == GEMM_OP_N ? N : K;
    if (lda < a_cols || ldb < b_cols || ldc < N) return GEMM_ERR_INVALID_ARG;
    if (batch > kMaxBatchPerLaunch) batch = kMaxBatchPerLaunch;      // larger batches run in parts of this size
    Args& a = *call;
    a.M = M; a.N = N; a.K = K;
    a.transA = transA == GEMM_OP_T; a.transB = transB == GEMM_OP_T;
    a.dtype = (int)dtype; a.out_dtype = (int)out_dtype; a.bias_dtype = (int)dtype; a.act = (int)act;
    a.alpha = 1.0f; a.beta = reads_c ? 1.0f : 0.0f;
    // stand-ins for aligned operands (never dereferenced: nothing is launched)
    a.A = (const void*)(uintptr_t)0x100000; a.B = (const void*)(uintptr_t)0x100000; a.C = (void*)(uintptr_t)0x100000;
    a.lda = lda; a.ldb = ldb; a.ldc = ldc;
    a.bias = nullptr;
    a.batch = (int32_t)batch;
    a.k_total = 0;
    const int64_t rows_a = transA == GEMM_OP_N ? M : K, rows_b = transB == GEMM_OP_N ? K : N;
    a.strideA = batch > 1 ? rows_a * lda : 0; a.strideB = batch > 1 ? rows_b * ldb : 0; a.strideC = batch > 1 ? M * ldc : 0;
    const int64_t in_bytes = gemm::elem_bytes(a.dtype);
    const bool batch_aligned = batch == 1 || ((a.strideA * in_bytes) % 16 == 0 && (a.strideB * in_bytes) % 16 == 0);
    *plan = automatic_plan(a, compute_units, batch_aligned);
    return GEMM_OK;
}

}  // namespace

GEMM_EXPORT gemm_status_t gemm_plan_query(int32_t compute_units, int64_t batch, int64_t M, int64_t N, int64_t K,
                                          gemm_op_t transA, gemm_op_t transB, gemm_dtype_t dtype, gemm_dtype_t out_dtype,
                                          int64_t lda, int64_t ldb, int64_t ldc, gemm_plan_t* out) {
    if (!out) return GEMM_ERR_INVALID_ARG;
    Args a;
    AutoPlan ap;
    const gemm_status_t st = query(compute_units, batch, M, N, K, transA, transB, dtype, out_dtype, lda, ldb, ldc, false, GEMM_ACT_NONE, &a, &ap);
    if (st == GEMM_OK) *out = ap.plan;
    return st;
}

GEMM_EXPORT gemm_status_t gemm_launch_query(int32_t compute_units, int64_t batch, int64_t M, int64_t N, int64_t K,
                                            gemm_op_t transA, gemm_op_t transB, gemm_dtype_t dtype, gemm_dtype_t out_dtype,
                                            int64_t lda, int64_t ldb, int64_t ldc, int32_t reads_c, gemm_act_t act, gemm_plan_t* out) {
    if (!out) return GEMM_ERR_INVALID_ARG;
    Args a;
    AutoPlan ap;
    const gemm_status_t st = query(compute_units, batch, M, N, K, transA, transB, dtype, out_dtype, lda, ldb, ldc, reads_c != 0, act, &a, &ap);
    if (st == GEMM_OK) *out = kernel_of(ap.peeled ? ap.main_part : a, ap.plan, ap.split_first, compute_units);
    return st;
}

GEMM_EXPORT gemm_status_t gemm_run(gemm_handle_t h, int64_t M, int64_t N, int64_t K,
                                   gemm_op_t transA, gemm_op_t transB, gemm_dtype_t dtype,
                                   float alpha, const void* A, int64_t lda,
                                   const void* B, int64_t ldb,
                                   float beta, void* C, int64_t ldc,
                                   const gemm_epilogue_t* epilogue, void* stream) {
    return run_batch(h, false, 1, M, N, K, transA, transB, dtype, alpha, A, lda, 0, B, ldb, 0, beta, C, ldc, 0, epilogue, stream);
}

GEMM_EXPORT gemm_status_t gemm_run_noalloc(gemm_handle_t h, int64_t M, int64_t N, int64_t K,
                                           gemm_op_t transA, gemm_op_t transB, gemm_dtype_t dtype,
                                           float alpha, const void* A, int64_t lda,
                                           const void* B, int64_t ldb,
                                           float beta, void* C, int64_t ldc,
                                           const gemm_epilogue_t* epilogue, void* stream) {
    return run_batch(h, true, 1, M, N, K, transA, transB, dtype, alpha, A, lda, 0, B, ldb, 0, beta, C, ldc, 0, epilogue, stream);
}

GEMM_EXPORT gemm_status_t gemm_run_batched(gemm_handle_t h, int64_t batch, int64_t M, int64_t N, int64_t K,
                                           gemm_op_t transA, gemm_op_t transB, gemm_dtype_t dtype,
                                           float alpha, const void* A, int64_t lda, int64_t strideA,
                                           const void* B, int64_t ldb, int64_t strideB,
                                           float beta, void* C, int64_t ldc, int64_t strideC,
                                           const gemm_epilogue_t* epilogue, void* stream) {
    return run_batch(h, false, batch, M, N, K, transA, transB, dtype, alpha, A, lda, strideA, B, ldb, strideB, beta, C, ldc, strideC,
                     epilogue, stream);
}
