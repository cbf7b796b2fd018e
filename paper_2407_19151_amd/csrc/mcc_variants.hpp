// mcc_variants.hpp -- kernel variants (threads per cell, cell capacity) and
// the cell-size buckets they serve.  Shared by the host runtime and the
// instantiation units.
#pragma once

namespace mcc {

// precision / physics modes compiled
// MODE_TAN: FP64 step carrying the tangent of the velocities (forward mode);
// the *_DIAG modes also measure the residual momentum and energy (separate
// kernels, so the step without diagnostics carries none of their registers)
enum Mode {
  MODE_FP64 = 0,
  MODE_FP32 = 1,
  MODE_REL = 2,
  MODE_TAN = 3,
  MODE_FP64_DIAG = 4,
  MODE_FP32_DIAG = 5,
  MODE_REL_DIAG = 6,
  // N x N pairing (Sec. 3.1) in the FP64, FP32 and relativistic forms
  MODE_FP64_NXN = 7,
  MODE_FP32_NXN = 8,
  MODE_REL_NXN = 9,
  // duplicity pairing (Higginson et al.'s s) in the same three forms
  MODE_FP64_DUP = 10,
  MODE_FP32_DUP = 11,
  MODE_REL_DUP = 12,
  NMODE = 13
};

// layout: 1 LDS (compact: keys and pair energies aliased, above 1024 particles
// the weights read from the input; 40-42 B per particle of capacity where
// separate arrays took 56, so more cells are resident per CU: relativistic
// cells of 576 + 448, 484 us per step of 4096 cells at three waves per SIMD,
// 593 with separate arrays at two; cells of 3000, 254 us per 400 in LDS, 608
// in global scratch);
// 2 per-workgroup global scratch (one wave per cell, or several waves for
// the plain FP64 and FP32 modes)
struct Variant {
  int tpc;     // threads per cell (workgroup size)
  int cap;     // largest cell the variant holds
  int layout;  // 1 LDS, 2 global scratch
};

constexpr int NVARIANT = 16;
constexpr Variant kVariants[NVARIANT] = {
    {64, 128, 1},    {64, 256, 1},   {128, 256, 1},  {128, 512, 1},  {256, 512, 1},
    {256, 1024, 1},  {512, 1024, 1}, {512, 2048, 1}, {1024, 2048, 1}, {1024, 4096, 1},
    {64, 32768, 2},  {256, 2048, 1}, {512, 4096, 1}, {256, 4096, 1},
    {256, 32768, 2}, {512, 32768, 2}};
// the one-wave global variant, which the modes without multi-wave global
// kernels use in place of variants 14 and 15
constexpr int kGlobalOneWave = 10;

// cell-size buckets: bucket b holds cells with kBucketCap[b-1] < n <= kBucketCap[b]
constexpr int NBUCKET = 7;
constexpr int kBucketCap[NBUCKET] = {128, 256, 512, 1024, 2048, 4096, 32768};
// default variant per bucket (the fastest measured on lognormal cell-size
// mixes; the autotuner may pick another candidate).  The compact layouts
// take 256 threads for the 2048 bucket (under the 2-wave register cap the
// FP64 512-thread kernel holds one workgroup per CU: 0.55 against 0.43 ms on
// the 65,536-cell mix).  Cells above 4096 particles take 8 waves in
// global scratch (measured on cells of 4 400 to 8 200 particles: 5.1-5.3x the
// one-wave variant, 1.5x the 4-wave).  The tangent form: two waves for cells
// of 129-256 (3000 of 200: 141 against 147 us) and eight for 1025-2048, whose
// registers hold twice the snapshot.
constexpr int kDefaultVariant[NBUCKET] = {0, 1, 3, 5, 11, 12, 15};
constexpr int kDefaultVariantTan[NBUCKET] = {0, 2, 3, 5, 7, 12, 15};
// With at most as many cells as the device has compute units, every cell has
// a CU to itself: resident cells per CU no longer matter, the latency of one
// cell does, and four waves per cell shorten it (16 cells, FP64 N97, kernel
// time against the table above: 200 particles 35 against 45 us, 400 37
// against 47; eight waves for 1500: 63 against 81).  Cells of 60 are slower
// (36 against 34), but one variant up to 1024 particles lets a call without a
// plan launch one kernel for the first four buckets (kFewBucket takes their
// cells); a plan of such cells takes the one wave (mcc_plan_create).
constexpr int kFewVariant[NBUCKET] = {5, 5, 5, 5, 7, 12, 15};
constexpr int kFewBucket = 3;
static_assert(kFewVariant[0] == kFewVariant[kFewBucket] &&
                  kFewVariant[1] == kFewVariant[kFewBucket] &&
                  kFewVariant[2] == kFewVariant[kFewBucket],
              "the merged buckets share a variant");
// candidates the autotuner times per bucket (-1 terminated)
constexpr int kCandidates[NBUCKET][5] = {
    {0, 1, 2, 5, -1}, {1, 2, 3, 4, 5}, {3, 4, 5, 6, -1}, {5, 6, 7, 11, -1},
    {7, 11, 8, -1, -1}, {12, 13, 9, -1, -1}, {15, 14, 10, -1, -1}};

// the tangent form keeps three more doubles per particle and one per pair: in
// LDS (compact layout) up to 2048 particles, above that in global scratch.
// With separate arrays and the tangent's snapshot in LDS it held two cells of
// 512 per CU instead of four (1024 cells of 512: 139 against 95 us per step)
// and none above 1024 (400 cells of 1800: 1312 against 204 us).
constexpr Variant kTanVariantBig = {64, 4096, 2};
// the most threads a tangent kernel takes: the reverse mode, which follows it,
// would spill half its registers at sixteen waves
constexpr Variant kTanVariantWide = {512, 2048, 1};

// few: no more cells than compute units
inline constexpr int default_variant(int mode, int bucket, bool few) {
  return few ? kFewVariant[bucket]
         : mode == MODE_TAN ? kDefaultVariantTan[bucket]
                            : kDefaultVariant[bucket];
}

// multi-wave global-scratch kernels: the FP64, FP32 and relativistic modes
// of every pairing (the waves of a workgroup share their CU's L1, so the
// barrier orders their scratch accesses as it does for LDS)
inline constexpr bool multiwave_global(int m) {
  return m == MODE_FP64 || m == MODE_FP32 || m == MODE_REL || m == MODE_FP64_NXN ||
         m == MODE_FP32_NXN || m == MODE_REL_NXN || m == MODE_FP64_DUP || m == MODE_FP32_DUP ||
         m == MODE_REL_DUP;
}
inline constexpr Variant variant_of(int mode, int v) {
  return (kVariants[v].layout == 2 && kVariants[v].tpc > 64 && !multiwave_global(mode))
             ? kVariants[kGlobalOneWave]
         : (mode == MODE_TAN && kVariants[v].cap > 2048 && kVariants[v].layout != 2)
             ? kTanVariantBig
         : (mode == MODE_TAN && kVariants[v].tpc > 512) ? kTanVariantWide
             : kVariants[v];
}

// Minimum waves per SIMD the compiler must leave room for (it then caps the
// registers, spilling a little): measured on the lognormal cell-size mix,
// where 2 waves per SIMD (the uncapped allocation) left the cell kernels
// waiting on LDS and barriers most of the time.  Cells of 2048 and 4096
// particles, whose LDS use allows at most 8 waves per CU, ask for 2: an
// uncapped allocation that reaches 256 registers leaves room for one.
// The tangent form's LDS leaves room for two per SIMD above 256 particles (an
// uncapped 512 kernel takes 270 registers, one wave: 1024 cells 136 against 96
// us) and pays for three below (6000 cells of 60: 150, 128 and 150 us at two,
// three and four).  1: no cap (the global-scratch forms).
constexpr int min_waves(int tpc, int cap, int layout, bool tangent) {
  if (layout == 2) return 1;
  if (tangent) return cap <= 256 ? 3 : 2;
  if (cap >= 2048) return 2;
  if (tpc == 64 && cap == 128) return 4;
  return 3;
}

// global scratch bytes per workgroup of a global-layout variant:
// 8 CAP doubles (v, w, snapshot, pair buffer), 2 CAP u32 (keys, slots),
// 6 CAP u16 (lists, orders, bucket members, weight order)
// (tangent form: 7 more CAP doubles for the tangent, its snapshot and the
// per-pair tangents)
constexpr unsigned long long big_stride_bytes(int cap, bool tan = false) {
  return ((unsigned long long)cap * (8 * 8 + 2 * 4 + 6 * 2 + (tan ? 7 * 8 : 0)) + 255ull) &
         ~255ull;
}

}  // namespace mcc
