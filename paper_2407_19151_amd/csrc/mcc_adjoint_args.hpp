// mcc_adjoint_args.hpp -- argument block of the reverse-mode kernels
// (mcc_collide_adjoint), shared by the host runtime and the kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mcc_kernel_args.hpp"
#include "mcc_variants.hpp"

namespace mcc {

struct AdjointArgs {
  const int64_t *offsets;
  const double *w;
  const double *vx, *vy, *vz;  // the step's input (read)
  double *gx, *gy, *gz;        // in: adjoint of the output; out: of the input
  const double *cell_volume;
  double dV;
  int64_t n;
  int32_t n_cells, S, n_coll;
  int32_t method, corr, sortw, keep;
  double fE;
  double inv_lnl;  // 1 / lnL (0 when lnL = 0: no pair scatters)
  uint64_t seed, step;
  double mass[MCC_MAX_SPECIES];
  CollConst coll[MCC_MAX_COLLISIONS];
  const int32_t *cell_list;
  const uint32_t *cell_count;
  double *lnl_part;  // [n_cells]: per-cell adjoint of lnL
  int32_t *err;
  const double2 *n97;    // as in CollideArgs
  const double *n97seg;
  char *scratch;    // per-workgroup scratch, `stride` bytes each
  uint64_t stride;
  int32_t slots;    // record slots in it
};

// record slots per workgroup: the collisions a forward pass records before
// the sweep back over them (longer lists are taken in groups).  Six cover
// three species; three for the global scratch, whose slots are up to 2.6 MB.
constexpr int ADJ_MAX_SLOTS = 6, ADJ_BIG_SLOTS = 3;

// one record slot: 9 doubles, half a double, half a u32 and a u16 per
// particle of capacity, and 32 doubles
constexpr unsigned long long adj_slot_bytes(int cap) {
  return ((unsigned long long)cap * (9 * 8 + 4 + 2 + 2) + 32 * 8 + 255ull) & ~255ull;
}
// per-workgroup scratch: the slots, and for the cells in global scratch 7.5
// doubles, 2 u32 and 5 u16 per particle of capacity
constexpr unsigned long long adj_stride_bytes(int cap, int slots, bool global) {
  return adj_slot_bytes(cap) * (unsigned)slots +
         (global ? (((unsigned long long)cap * (7 * 8 + 4 + 2 * 4 + 5 * 2) + 255ull) & ~255ull)
                 : 0ull);
}

// The reverse-mode kernel of a size bucket (largest cell `most`) beside a
// tangent kernel of tpc threads per cell: as many threads, so that the two
// split a cell's sums alike (the sums still round by their own expressions: at
// a switch, where a cell's correction just fails, the two forms' factors f_E
// differ by a few units in the last place).  In LDS up to 2048 particles,
// above that, and for one wave above 256, in global scratch.
struct AdjointForm {
  int tpc, cap;
  bool global;
};
inline constexpr AdjointForm adjoint_form(int tpc, int most) {
  if (most > 4096) return {64, 32768, true};
  if (tpc == 512) return {512, 2048, false};
  if (tpc == 256) return most <= 1024 ? AdjointForm{256, 1024, false} : AdjointForm{256, 2048, false};
  if (tpc == 128) return {128, 512, false};
  if (most <= 128) return {64, 128, false};
  if (most <= 256) return {64, 256, false};
  return {64, 4096, true};
}
// (every variant that a bucket can run, the caller's included)
inline constexpr bool adjoint_forms_match() {
  for (int b = 0; b < NBUCKET; ++b)
    for (int v = 0; v < NVARIANT; ++v) {
      if (kVariants[v].cap < kBucketCap[b]) continue;
      const AdjointForm f = adjoint_form(variant_of(MODE_TAN, v).tpc, kBucketCap[b]);
      if (f.tpc != variant_of(MODE_TAN, v).tpc || f.cap < kBucketCap[b]) return false;
    }
  return true;
}
static_assert(adjoint_forms_match(), "the reverse mode takes the tangent's threads per cell");

// a compiled reverse-mode kernel
struct AdjointKernel {
  const void *fn = nullptr;
  AdjointForm form{};
};

}  // namespace mcc
