// mcc_api.hip -- host runtime behind include/mcc.h: context and workspace,
// argument checks, per-collision constants, size-bucketed launches of the
// collide kernel variants, the unsorted entry (binning + gather/scatter),
// and the batched plan (device work lists, autotuned variants, HIP graph).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <mutex>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include <vector>

#include "../../include/mcc.h"
#include "mcc_kernel_args.hpp"
#include "mcc_variants.hpp"

const void *const *mcc_kernel_table_fp64();
const void *const *mcc_kernel_table_fp32();
const void *const *mcc_kernel_table_rel();
const void *const *mcc_kernel_table_tan();
const void *const *mcc_kernel_table_fp64_diag();
const void *const *mcc_kernel_table_fp32_diag();
const void *const *mcc_kernel_table_rel_diag();
const void *const *mcc_kernel_table_fp64_nxn();
const void *const *mcc_kernel_table_fp32_nxn();
const void *const *mcc_kernel_table_rel_nxn();
const void *const *mcc_kernel_table_fp64_dup();
const void *const *mcc_kernel_table_fp32_dup();
const void *const *mcc_kernel_table_rel_dup();

namespace mcc {
hipError_t launch_zero_stats(mcc_stats *st, hipStream_t s);
hipError_t launch_set_u64(uint64_t *p, uint64_t v, hipStream_t s);
hipError_t launch_inc_u64(uint64_t *p, hipStream_t s);
hipError_t launch_flag_nonzero(const uint32_t *count, int32_t code, int32_t *err,
                               hipStream_t s);
hipError_t launch_front(const int64_t *offsets, int32_t n_cells, int32_t S, int64_t n,
                        const double *w, int32_t *lists, uint32_t *counts, int32_t *cell_corr,
                        mcc_stats *stats, double *zero, int64_t nzero, int first_bucket,
                        int32_t *err, hipStream_t s);
int64_t scan_tiles_needed(int64_t m);
int64_t bin_hist_entries(int64_t n);
hipError_t launch_bin(int64_t n, const int32_t *cells, const int32_t *species, int32_t n_cells,
                      int32_t S, uint32_t *keys0, uint32_t *keys1, int32_t *vals0,
                      int32_t *vals1, uint32_t *hist, uint32_t *pos, int64_t *tiles,
                      int64_t *offsets, int32_t *perm, int32_t *err, hipStream_t s);
hipError_t launch_sample_angles(int method, int precision, int64_t n, const double *s,
                                const uint32_t *a0, const uint32_t *a1, double *oc, double *st,
                                double *A, const double2 *tab, const double *seg,
                                hipStream_t st_);
hipError_t launch_n97_table(double2 *tab, hipStream_t s);
const double *n97_segments_host();
size_t rebin_scratch_bytes(int64_t n, int64_t m);
int64_t rebin_tiles_needed(int64_t n, int64_t m);
hipError_t launch_rebin(int64_t n, int64_t m, int32_t S, int32_t n_cells, const int64_t *off,
                        const int32_t *cells_new, int64_t *off_new, int32_t *perm,
                        void *scratch, int64_t *tiles, int32_t *err, hipStream_t s);
int bin_passes(int64_t m);
hipError_t launch_bin_move(int64_t n, const int32_t *cells, const int32_t *species,
                           int32_t n_cells, int32_t S, uint32_t *keys0, uint32_t *keys1,
                           uint32_t *const *place, uint16_t *const *local, uint32_t *hist,
                           uint32_t *pos, int64_t *tiles, int64_t *offsets,
                           const double *const *payload, double *g, double *rec, int64_t n_pad,
                           int32_t *err, hipStream_t s);
hipError_t launch_move_back(int64_t n, int64_t m, uint32_t *const *place, uint16_t *const *local,
                            double *g, double *rec, int64_t n_pad, double *const *v,
                            hipStream_t s);
hipError_t launch_gather_rec(int64_t n, const int32_t *perm, const double *const *payload,
                             double *rec, double *const *g, hipStream_t s);
hipError_t launch_scatter_back_rec(int64_t n, const int32_t *perm, double *const *g, double *rec,
                                   double *const *v, hipStream_t s);
hipError_t launch_gather(int64_t n, const int32_t *perm, const double *w, const double *vx,
                         const double *vy, const double *vz, double *gw, double *gx, double *gy,
                         double *gz, hipStream_t s);
struct AdjointArgs;
struct AdjointKernel;
AdjointKernel adjoint_kernel_for(bool fp32, int tpc, int most);
hipError_t launch_adjoint(const AdjointKernel &k, const AdjointArgs &base, const int32_t *lists,
                          const uint32_t *counts, int32_t n_cells, int b, int grid,
                          hipStream_t s);
hipError_t launch_sum_f64(const double *x, int64_t n, double *out, hipStream_t s);
}  // namespace mcc
#include "mcc_adjoint_args.hpp"

using namespace mcc;

namespace {

struct DevBuf {
  void *p = nullptr;
  size_t bytes = 0;
  bool ensure(size_t want) {
    if (want <= bytes) return true;
    if (p) (void)hipFree(p);
    p = nullptr;
    bytes = 0;
    if (hipMalloc(&p, want) != hipSuccess) {
      p = nullptr;
      return false;
    }
    bytes = want;
    return true;
  }
  void release() {
    if (p) (void)hipFree(p);
    p = nullptr;
    bytes = 0;
  }
  template <class T>
  T *as() const {
    return reinterpret_cast<T *>(p);
  }
};

// global scratch of the large-cell (GLOBAL layout) variants.  A context
// owns one for its direct calls and every plan owns its own: a plan's graph
// holds the scratch address, so a buffer the context later grows (and
// reallocates) must never be the one a plan replays against.
// One buffer per kernel footprint (the tangent's arrays are larger), so none
// ever moves: a caller's graph may hold it too.
struct BigScratch {
  DevBuf big32k, tan4k, tan32k;
  DevBuf &of(const Variant &V, bool tan) { return !tan ? big32k : V.cap > 4096 ? tan32k : tan4k; }
  const DevBuf &of(const Variant &V, bool tan) const {
    return const_cast<BigScratch *>(this)->of(V, tan);
  }
  void release() {
    big32k.release();
    tan4k.release();
    tan32k.release();
  }
};
// (the step's global variants are all of the largest capacity)
constexpr bool step_globals_are_32k() {
  for (int m = 0; m < NMODE; ++m)
    for (int v = 0; v < NVARIANT; ++v)
      if (m != MODE_TAN && variant_of(m, v).layout == 2 && variant_of(m, v).cap != MCC_MAX_CELL)
        return false;
  return true;
}
static_assert(step_globals_are_32k(), "one scratch size per buffer");

const void *const *kernel_table(int mode) {
  switch (mode) {
    case MODE_FP64: return mcc_kernel_table_fp64();
    case MODE_FP32: return mcc_kernel_table_fp32();
    case MODE_TAN: return mcc_kernel_table_tan();
    case MODE_FP64_DIAG: return mcc_kernel_table_fp64_diag();
    case MODE_FP32_DIAG: return mcc_kernel_table_fp32_diag();
    case MODE_REL_DIAG: return mcc_kernel_table_rel_diag();
    case MODE_FP64_NXN: return mcc_kernel_table_fp64_nxn();
    case MODE_FP32_NXN: return mcc_kernel_table_fp32_nxn();
    case MODE_REL_NXN: return mcc_kernel_table_rel_nxn();
    case MODE_FP64_DUP: return mcc_kernel_table_fp64_dup();
    case MODE_FP32_DUP: return mcc_kernel_table_fp32_dup();
    case MODE_REL_DUP: return mcc_kernel_table_rel_dup();
    default: return mcc_kernel_table_rel();
  }
}

}  // namespace

// Side streams and events (default priority) on which the kernels of some size
// buckets run beside those of the others.  A context makes one, which calls
// take; the second, which only plans do, is made when a plan first needs it (25
// us each, of 75 that creating a context takes).
struct Branches {
  static constexpr int N = 2;
  hipStream_t side[N] = {};
  hipEvent_t fork = nullptr, join[N] = {};
  int ready = 0;  // side streams there are
  // makes k side streams; false: not to be had (the caller then takes fewer)
  bool create(int k) {
    if (ready >= k) return true;
    hipError_t e = hipSuccess;
    if (!fork) e = hipEventCreateWithFlags(&fork, hipEventDisableTiming);
    while (ready < k && e == hipSuccess) {
      if (!join[ready]) e = hipEventCreateWithFlags(&join[ready], hipEventDisableTiming);
      if (e == hipSuccess) e = hipStreamCreateWithFlags(&side[ready], hipStreamNonBlocking);
      if (e == hipSuccess) ++ready;
    }
    if (e != hipSuccess) (void)hipGetLastError();
    return ready >= k;
  }
  void release() {
    for (int i = 0; i < N; ++i) {
      if (join[i]) (void)hipEventDestroy(join[i]);
      if (side[i]) (void)hipStreamDestroy(side[i]);
      join[i] = nullptr;
      side[i] = nullptr;
    }
    if (fork) (void)hipEventDestroy(fork);
    fork = nullptr;
    ready = 0;
  }
};

struct mcc_ctx {
  int device = 0;
  hipStream_t stream = nullptr;
  Branches branches;  // the steps' other streams (launch_buckets; a plan's capture)
  int n_cu = 0;
  bool validate = false;
  int32_t *err = nullptr;  // device error word
  DevBuf lists, counts;
  BigScratch big;  // large-cell scratch of the direct (non-plan) calls
  DevBuf n97;                      // N97 table of the FP32 form (built once)
  const double *n97seg = nullptr;  // of the FP64 form (the device's)
  // per size bucket: the collide kernels' cell-claim and finished-workgroup
  // counters (zero between launches: each launch resets them at its end, so
  // launches of one context must not overlap)
  DevBuf work;
  // unsorted entry: the payload in grouped order and between the passes (or in
  // records), and where a pass's items went, or the permutation (mcc_rebin uses
  // `grouped` for its copy)
  DevBuf tiles, off, grouped, rec, place[2], local;
  DevBuf word;  // the calls' weight order of large cells (PREP_KEEP)
  DevBuf bin_k0, bin_k1, bin_v0, bin_v1, bin_hist, bin_pos;  // radix-sort scratch
  // reverse-mode form: per-workgroup scratch (cells up to 4096 particles,
  // and above), per-cell lnL adjoints
  DevBuf adj_small, adj_big, adj_part;
  // incremental re-binning
  DevBuf rb;
  int grid[NMODE][NVARIANT] = {};
  int variant[NBUCKET] = {};
};

namespace {
// The kernel variant of every bucket for one call, and the first bucket that
// takes cells (the ones below hand theirs to it).
struct Variants {
  int v[NBUCKET];
  int first = 0;
  // The most cells bucket b can hold of n particles in n_cells cells: each
  // has more than the bucket below holds.  0: the bucket is empty whatever
  // the offsets hold (a segment inside [0, n) cannot be that large), and its
  // kernel need not be launched; otherwise a bound for its grid, exact for
  // well-formed offsets (a longer list is still worked off).
  int64_t most_cells(int64_t n, int32_t n_cells, int b) const {
    if (b < first) return 0;
    const int64_t least = b > first ? (int64_t)kBucketCap[b - 1] + 1 : 1;
    return std::min<int64_t>(n_cells, n / least);
  }
};
}  // namespace

struct mcc_plan {
  mcc_ctx *ctx = nullptr;
  CollideArgs args{};
  int mode = 0;
  int32_t n_cells = 0;
  Variants pick;
  uint32_t hcount[NBUCKET] = {};  // cells per bucket (fixed for the plan)
  DevBuf lists, counts, step;
  BigScratch big;          // large-cell scratch of this plan's kernels (its graph holds it)
  DevBuf prep, prep_word;  // weight data of the bound population (PREP_READ)
  mcc_stats *stats = nullptr;
  int32_t *cell_corr = nullptr;
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
  double tuned_ms[NBUCKET][NVARIANT] = {};
};

namespace {

mcc_status from_hip(hipError_t e) {
  if (e == hipSuccess) return MCC_OK;
  if (e == hipErrorOutOfMemory || e == hipErrorMemoryAllocation) return MCC_ERR_OOM;
  return MCC_ERR_DEVICE;
}

#define HIP_TRY(expr)                         \
  do {                                        \
    hipError_t e_ = (expr);                   \
    if (e_ != hipSuccess) return from_hip(e_); \
  } while (0)

// kernel family of a step: precision / physics, and whether diagnostics are
// measured (A.diag, set by fill_args)
int mode_of(const mcc_params *p, const CollideArgs &A) {
  if (p->pairing == MCC_PAIRING_NXN)
    return p->relativistic ? MODE_REL_NXN
           : p->precision == MCC_FP32_KINEMATICS ? MODE_FP32_NXN : MODE_FP64_NXN;
  if (p->pairing == MCC_PAIRING_DUPLICITY)
    return p->relativistic ? MODE_REL_DUP
           : p->precision == MCC_FP32_KINEMATICS ? MODE_FP32_DUP : MODE_FP64_DUP;
  if (p->relativistic) return A.diag ? MODE_REL_DIAG : MODE_REL;
  if (p->precision == MCC_FP32_KINEMATICS) return A.diag ? MODE_FP32_DIAG : MODE_FP32;
  return A.diag ? MODE_FP64_DIAG : MODE_FP64;
}

// host checks of the step arguments shared by every entry point
mcc_status check_step(int64_t n, int32_t n_cells, int32_t n_species, const double *w,
                      const double *vx, const double *vy, const double *vz,
                      const double *cell_volume, double dVs, const mcc_species *sp,
                      int32_t n_coll, const mcc_collision *coll, double dt, double lnL,
                      const mcc_params *p) {
  if (n < 0 || n_cells < 0 || n_species < 1 || n_species > MCC_MAX_SPECIES) return MCC_ERR_INVALID;
  if (n_coll < 0 || n_coll > MCC_MAX_COLLISIONS) return MCC_ERR_INVALID;
  if (n > 0 && (!w || !vx || !vy || !vz)) return MCC_ERR_INVALID;
  if (n > (int64_t)INT32_MAX) return MCC_ERR_UNSUPPORTED;
  if (!sp || (n_coll > 0 && !coll) || !p) return MCC_ERR_INVALID;
  for (int s = 0; s < n_species; ++s)
    if (!(sp[s].mass > 0.0) || !std::isfinite(sp[s].mass) || !std::isfinite(sp[s].charge))
      return MCC_ERR_INVALID;
  for (int k = 0; k < n_coll; ++k)
    if (coll[k].a < 0 || coll[k].a >= n_species || coll[k].b < 0 || coll[k].b >= n_species)
      return MCC_ERR_INVALID;
  if (!std::isfinite(dt) || dt < 0.0 || !std::isfinite(lnL) || lnL < 0.0) return MCC_ERR_INVALID;
  if (p->method != MCC_TA77 && p->method != MCC_N97 && p->method != MCC_HARD_SPHERE)
    return MCC_ERR_INVALID;
  if (p->method == MCC_HARD_SPHERE)
    for (int k = 0; k < n_coll; ++k)
      if (!(coll[k].cross_section >= 0.0) || !std::isfinite(coll[k].cross_section))
        return MCC_ERR_INVALID;
  if (p->precision != MCC_FP64 && p->precision != MCC_FP32_KINEMATICS) return MCC_ERR_INVALID;
  if (p->on_failure != MCC_FAIL_RESET && p->on_failure != MCC_FAIL_KEEP) return MCC_ERR_INVALID;
  if (p->max_passes < 1) return MCC_ERR_INVALID;
  if (p->pairing != MCC_PAIRING_ORDER_N && p->pairing != MCC_PAIRING_NXN &&
      p->pairing != MCC_PAIRING_DUPLICITY)
    return MCC_ERR_INVALID;
  if (p->pairing != MCC_PAIRING_ORDER_N && p->diagnostics) return MCC_ERR_UNSUPPORTED;
  if (!(p->f_E > 0.0 && p->f_E < 1.0)) return MCC_ERR_INVALID;
  if (!(p->eps0 > 0.0) || !std::isfinite(p->eps0)) return MCC_ERR_INVALID;
  if (p->relativistic && !(p->c > 0.0 && std::isfinite(p->c))) return MCC_ERR_INVALID;
  if (p->relativistic && p->precision != MCC_FP64) return MCC_ERR_UNSUPPORTED;
  if (p->method == MCC_HARD_SPHERE && (p->relativistic || p->precision != MCC_FP64))
    return MCC_ERR_UNSUPPORTED;
  if (!cell_volume && !(dVs > 0.0 && std::isfinite(dVs))) return MCC_ERR_INVALID;
  return MCC_OK;
}

void fill_args(CollideArgs &A, int64_t n, int32_t n_cells, int32_t S, const int64_t *offsets,
               const double *w, double *vx, double *vy, double *vz, const double *cell_volume,
               double dVs, const mcc_species *sp, int32_t n_coll, const mcc_collision *coll,
               double dt, double lnL, uint64_t seed, uint64_t step, const mcc_params *p,
               mcc_stats *stats, int32_t *cell_corr, const mcc_ctx *ctx) {
  std::memset(&A, 0, sizeof(A));
  A.offsets = offsets;
  A.w = w;
  A.vx = vx;
  A.vy = vy;
  A.vz = vz;
  A.cell_volume = cell_volume;
  A.dV = dVs;
  A.n = n;
  A.n_cells = n_cells;
  A.S = S;
  A.n_coll = n_coll;
  A.method = p->method;
  A.corr = p->moment_correction ? 1 : 0;
  A.sortw = p->sort_by_weight ? 1 : 0;
  A.max_passes = p->max_passes;
  A.keep = p->on_failure == MCC_FAIL_KEEP ? 1 : 0;
  A.diag = (p->diagnostics && stats) ? 1 : 0;
  A.fE = p->f_E;
  A.c = p->relativistic ? p->c : 1.0;
  A.seed = seed;
  A.step = step;
  A.step_dev = nullptr;
  for (int s = 0; s < S; ++s) A.mass[s] = sp[s].mass;
  const double pi = 3.14159265358979323846;
  for (int k = 0; k < n_coll; ++k) {
    const int a = coll[k].a, b = coll[k].b;
    const double ma = sp[a].mass, mb = sp[b].mass, qa = sp[a].charge, qb = sp[b].charge;
    const double mu = ma * mb / (ma + mb);
    CollConst &C = A.coll[k];
    C.a = a;
    C.b = b;
    // Eq. (12) without the per-pair factors f, w_max, N_min, dV and |u|^3;
    // for hard spheres s = sigma n_eff |u| dt without f, w_max, N_min, dV, |u|
    const double base = qa * qa * qb * qb * lnL * dt / (4.0 * pi * p->eps0 * p->eps0);
    C.coef = p->method == MCC_HARD_SPHERE ? coll[k].cross_section * dt
             : p->relativistic            ? base
                                          : base / (mu * mu);
    C.fa = mb / (ma + mb);
    C.fb = ma / (ma + mb);
  }
  A.stats = stats;
  A.cell_corr = cell_corr;
  A.err = ctx->err;
  A.n97 = ctx->n97.as<double2>();
  A.n97seg = ctx->n97seg;
}

bool ensure_lists(mcc_ctx *ctx, DevBuf &lists, DevBuf &counts, int32_t n_cells) {
  return lists.ensure(sizeof(int32_t) * (size_t)NBUCKET * (size_t)std::max(n_cells, 1)) &&
         counts.ensure(sizeof(uint32_t) * 16);
}

// global-layout variants: persistent grid and per-workgroup scratch
int grid_of(mcc_ctx *ctx, int mode, int v) {
  const Variant V = variant_of(mode, v);
  if (V.layout == 2) return ctx->n_cu;
  return ctx->grid[mode][v];
}

// The scratch's size does not depend on the call, so the first allocation also
// serves a call that is being captured (whose graph then holds it): in relaxed
// mode for this thread, as a malloc would otherwise end the capture.  A capture
// must not need larger-celled eager calls before it.
bool ensure_big(mcc_ctx *ctx, BigScratch &B, int mode, int v) {
  const Variant V = variant_of(mode, v);
  if (V.layout != 2) return true;
  const uint64_t bytes = big_stride_bytes(V.cap, mode == MODE_TAN) * (uint64_t)ctx->n_cu;
  DevBuf &buf = B.of(V, mode == MODE_TAN);
  if (buf.p) return true;
  hipStreamCaptureMode m = hipStreamCaptureModeRelaxed;
  if (hipThreadExchangeStreamCaptureMode(&m) != hipSuccess) return buf.ensure(bytes);
  const bool ok = buf.ensure(bytes);
  (void)hipThreadExchangeStreamCaptureMode(&m);
  return ok;
}

void set_big_args(const BigScratch &B, CollideArgs &A, int mode, int v) {
  const Variant V = variant_of(mode, v);
  if (V.layout != 2) return;
  A.big_scratch = B.of(V, mode == MODE_TAN).as<char>();
  A.big_stride = big_stride_bytes(V.cap, mode == MODE_TAN);
}

#ifdef MCC_PHASE_TIMING
// profiling build: clock ticks per kernel phase, 16 counters per size bucket
unsigned long long *g_phase = nullptr;
#endif

// The caller's variants (mcc_set_variant) or the defaults, which depend on
// n_cells alone, so a plan and a call of the same cells take the same ones (or
// one whose sums are the same) and give the same bits.
Variants pick_variants(const mcc_ctx *ctx, int mode, int32_t n_cells) {
  Variants r;
  const bool few = n_cells <= ctx->n_cu;
  bool merge = few;
  for (int b = 0; b < NBUCKET; ++b) {
    r.v[b] = ctx->variant[b] >= 0 ? ctx->variant[b] : default_variant(mode, b, few);
    if (b <= kFewBucket && ctx->variant[b] >= 0) merge = false;
  }
  r.first = merge ? kFewBucket : 0;
  return r;
}

// enqueue the collide kernel of one bucket, reading its device work list;
// most: no more workgroups than this (cells known or bounded on the host)
mcc_status launch_bucket(mcc_ctx *ctx, BigScratch &big, const CollideArgs &base, int mode,
                         int32_t n_cells, const int32_t *lists, const uint32_t *counts, int b,
                         int v, int64_t most, hipStream_t stream) {
  const void *const *tab = kernel_table(mode);
  if (!ensure_big(ctx, big, mode, v)) return MCC_ERR_OOM;
  CollideArgs A = base;
#ifdef MCC_PHASE_TIMING
  A.phase = g_phase ? g_phase + 16 * b : nullptr;
#endif
  A.cell_list = lists + (int64_t)b * std::max(n_cells, 1);
  A.cell_count = counts + b;
  A.work = ctx->work.as<uint32_t>() + WORK_QUEUES * WORK_STRIDE * b;
  set_big_args(big, A, mode, v);
  void *kargs[] = {&A};
  const int64_t grid = std::max<int64_t>(1, std::min<int64_t>(grid_of(ctx, mode, v), most));
  HIP_TRY(hipLaunchKernel(tab[v], dim3((unsigned)grid), dim3(variant_of(mode, v).tpc), kargs, 0,
                          stream));
  return MCC_OK;
}

// How many streams a plan's bucket kernels are dealt to, in turn.  A bucket's
// persistent grid drains unevenly at its end and, in a small population, never
// fills the GPU; another bucket's cells then take the room.  The fork and join
// cost about 10 us in a graph, which one shared tail does not pay for (4000
// cells of 225-275 in two buckets, FP32: 109 against 98 us), so a plan forks
// from three buckets up, and for the 2048 and 4096 buckets alone, whose cells
// take a CU's LDS or half of it each and last long (cells of 1100-4000 on one
// and two streams, FP32: 300 of them 133 and 112 us, 1500 322 and 291; FP64
// 161 and 135, 402 and 356).  Three streams up to 2^21 particles, two above, where
// two grids fill the GPU and a third only mixes cells of mismatched footprints
// on the CUs.  Lognormal cells, FP64, one, two and three streams: 200 cells of
// 330 272, 170 and 134 us; 4000 351, 243 and 209; 8000 456, 334 and 349;
// 16 411 773, 558 and 633; FP32, 65 536: 1640, 1594 and 1702.
constexpr int64_t kThreeStreams = 1 << 21;
constexpr unsigned kLargePair = (1u << 4) | (1u << 5);
static_assert(kBucketCap[4] == 2048 && kBucketCap[5] == 4096, "the pair that forks alone");

// filled: the buckets that hold cells (bit b)
int plan_streams(int64_t n, unsigned filled) {
  if (filled == kLargePair) return 2;
  return __builtin_popcount(filled) < 3 ? 1 : n <= kThreeStreams ? 3 : 2;
}

// A call, whose counts are on the device, deals its buckets to two streams in
// turn, except where that costs more than it gives: with one bucket holding the
// cells, and as many as keep the GPU full, another stream's tail has nothing to
// fill, and the empty kernels launched beside the loaded one slow it (FP64
// cells of 4, 1e6 of them: 7680 us without, 8830 with one beside it) or, where
// it is the side stream's, delay the next call (16 000 cells of 700, FP32, back
// to back: 885 and 1178).  So the side stream takes the 2048 and 4096 buckets
// alone where the mean cell is in the 1024 bucket and there are more than 8
// cells per compute unit (4000 Poisson cells of 700, FP32: 268 against 362; 1000
// of 700 115 and 122, but 1000 of 550, in two buckets, 153 and 120), and where
// it has at most 128 particles and there are more than 160 (45 000 cells of
// 100, FP64: 465 against 524; 32 000 lognormal cells of 20 488 and 463).
bool call_large_aside(int64_t n, int32_t n_cells, int n_cu) {
  if (n <= (int64_t)n_cells * kBucketCap[0]) return n_cells > 160 * n_cu;
  return n > (int64_t)n_cells * kBucketCap[2] && n <= (int64_t)n_cells * kBucketCap[3] &&
         n_cells > 8 * n_cu;
}

// enqueue the collide kernels of all buckets, largest cells first
// (host_counts: the buckets' cell counts when known on the host; empty
// buckets are then not launched), with br dealt to its streams and this one.
// The global-scratch kernels share one scratch, so they stay on this stream.
mcc_status launch_buckets(mcc_ctx *ctx, BigScratch &big, const CollideArgs &base, int mode,
                          int32_t n_cells, const int32_t *lists, const uint32_t *counts,
                          const Variants &pick, hipStream_t stream,
                          const uint32_t *host_counts = nullptr, const Branches *br = nullptr) {
  auto most = [&](int b) {
    return host_counts ? (int64_t)host_counts[b] : pick.most_cells(base.n, n_cells, b);
  };
  unsigned filled = 0;
  for (int b = 0; b < NBUCKET; ++b) {
    if (most(b) == 0) continue;
    filled |= 1u << b;
    // (scratch before the first launch: an allocation that fails leaves nothing done)
    if (!ensure_big(ctx, big, mode, pick.v[b])) return MCC_ERR_OOM;
  }
  const bool large_aside = br && !host_counts && call_large_aside(base.n, n_cells, ctx->n_cu);
  int K = !br ? 1 : host_counts ? plan_streams(base.n, filled) : 2;
  if (K > 1) K = std::min(K, std::min(__builtin_popcount(filled), 1 + br->ready));
  if (K > 1) {
    HIP_TRY(hipEventRecord(br->fork, stream));
    for (int i = 0; i < K - 1; ++i) HIP_TRY(hipStreamWaitEvent(br->side[i], br->fork, 0));
  }
  int turn = 0;
  mcc_status st = MCC_OK;
  for (int b = NBUCKET - 1; b >= 0 && st == MCC_OK; --b) {
    if (most(b) == 0) continue;
    const int on = variant_of(mode, pick.v[b]).layout == 2 ? 0
                   : large_aside ? (K > 1 ? (kLargePair >> b) & 1u : 0)
                                 : turn % K;
    ++turn;
    st = launch_bucket(ctx, big, base, mode, n_cells, lists, counts, b, pick.v[b], most(b),
                       on ? br->side[on - 1] : stream);
  }
  // (after an error too: what already runs on the side streams stays ordered
  // before the caller's next work, and a capture's branches are closed)
  for (int i = 0; i < K - 1; ++i) {
    HIP_TRY(hipEventRecord(br->join[i], br->side[i]));
    HIP_TRY(hipStreamWaitEvent(stream, br->join[i], 0));
  }
  return st;
}

mcc_status finish(mcc_ctx *ctx) {
  if (!ctx->validate) return MCC_OK;
  HIP_TRY(hipStreamSynchronize(ctx->stream));
  int32_t code = 0;
  HIP_TRY(hipMemcpy(&code, ctx->err, sizeof(code), hipMemcpyDeviceToHost));
  return code ? MCC_ERR_DATA : MCC_OK;
}

}  // namespace

extern "C" {

#ifdef MCC_PHASE_TIMING
// profiling build only (not part of the public header): copy out and
// optionally clear the per-bucket phase counters
int mcc_debug_phase_read(unsigned long long *out, int reset) {
  if (!g_phase) return -1;
  if (hipDeviceSynchronize() != hipSuccess) return -3;
  const size_t bytes = sizeof(unsigned long long) * 16 * NBUCKET;
  if (hipMemcpy(out, g_phase, bytes, hipMemcpyDeviceToHost) != hipSuccess) return -3;
  if (reset && hipMemset(g_phase, 0, bytes) != hipSuccess) return -3;
  return 0;
}
#endif

void mcc_default_params(mcc_params *p) {
  if (!p) return;
  std::memset(p, 0, sizeof(*p));
  p->method = MCC_N97;
  p->precision = MCC_FP64;
  p->relativistic = 0;
  p->moment_correction = 1;
  p->sort_by_weight = 1;
  p->max_passes = 1;
  p->on_failure = MCC_FAIL_RESET;
  p->diagnostics = 0;
  p->pairing = MCC_PAIRING_ORDER_N;
  p->f_E = 0.05;
  p->eps0 = 1.0;
  p->c = 0.0;
}

const char *mcc_status_string(mcc_status s) {
  switch (s) {
    case MCC_OK: return "ok";
    case MCC_ERR_INVALID: return "invalid argument";
    case MCC_ERR_OOM: return "device out of memory";
    case MCC_ERR_DEVICE: return "HIP runtime error";
    case MCC_ERR_UNSUPPORTED: return "unsupported combination";
    case MCC_ERR_DATA: return "device-side data check failed";
  }
  return "unknown status";
}

// ---------------------------------------------------------------------------
// Fixed device scratch of the allocation-free step: the size-bucket counters
// (256 B) and the cell work lists of up to NOALLOC_MAX_CELLS cells.  Each
// device holds its own copy at its own address; host code reaches it only
// through the address hipGetSymbolAddress returns for that device.
// ---------------------------------------------------------------------------
constexpr int32_t NOALLOC_MAX_CELLS = 1 << 18;
constexpr size_t NOALLOC_BYTES = 256 + sizeof(int32_t) * (size_t)NBUCKET * NOALLOC_MAX_CELLS;
static __device__ __align__(256) unsigned char scratch[NOALLOC_BYTES];

// The FP64 form's N97 table, constant once written: filled once per device by
// the first context there (a copy per context would cost each creation a
// device allocation and a host copy).
static __device__ __align__(128) double n97_segments[N97_SEGMENTS * N97_SEG_DOUBLES];

namespace {
constexpr int NOALLOC_MAX_DEVICES = 1024;
std::mutex g_noalloc_mu;
void *g_noalloc_ptr[NOALLOC_MAX_DEVICES] = {};
hipError_t g_noalloc_rc[NOALLOC_MAX_DEVICES] = {};
bool g_noalloc_done[NOALLOC_MAX_DEVICES] = {};
const double *g_n97seg_ptr[NOALLOC_MAX_DEVICES] = {};

// once per device, with that device current
void noalloc_setup(int device) {
  if (device < 0 || device >= NOALLOC_MAX_DEVICES) return;
  std::lock_guard<std::mutex> lock(g_noalloc_mu);
  if (g_noalloc_done[device]) return;
  void *p = nullptr;
  g_noalloc_rc[device] = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
  g_noalloc_ptr[device] = g_noalloc_rc[device] == hipSuccess ? p : nullptr;
  g_noalloc_done[device] = true;
}

// the device's N97 table, filled on the first call (nullptr: the runtime
// refused, and the next call tries again)
const double *n97seg_setup(int device) {
  if (device < 0 || device >= NOALLOC_MAX_DEVICES) return nullptr;
  std::lock_guard<std::mutex> lock(g_noalloc_mu);
  if (!g_n97seg_ptr[device]) {
    void *p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(n97_segments)) == hipSuccess &&
        hipMemcpy(p, n97_segments_host(), sizeof(n97_segments), hipMemcpyHostToDevice) ==
            hipSuccess)
      g_n97seg_ptr[device] = static_cast<const double *>(p);
  }
  return g_n97seg_ptr[device];
}

void *noalloc_ptr(int device) {
  if (device < 0 || device >= NOALLOC_MAX_DEVICES) return nullptr;
  std::lock_guard<std::mutex> lock(g_noalloc_mu);
  return g_noalloc_done[device] ? g_noalloc_ptr[device] : nullptr;
}
}  // namespace

mcc_status mcc_create(mcc_ctx **out, int device, void *hip_stream) {
  if (!out) return MCC_ERR_INVALID;
  *out = nullptr;
  int ndev = 0;
  HIP_TRY(hipGetDeviceCount(&ndev));
  if (device < 0 || device >= ndev) return MCC_ERR_INVALID;
  HIP_TRY(hipSetDevice(device));
  mcc_ctx *ctx = new mcc_ctx();
  ctx->device = device;
  ctx->stream = reinterpret_cast<hipStream_t>(hip_stream);
  hipDeviceProp_t prop;
  hipError_t e = hipGetDeviceProperties(&prop, device);
  if (e != hipSuccess) {
    delete ctx;
    return from_hip(e);
  }
  ctx->n_cu = prop.multiProcessorCount;
  noalloc_setup(device);  // (the device is current)
  for (int b = 0; b < NBUCKET; ++b) ctx->variant[b] = -1;  // the mode's default
  const char *val = std::getenv("MCC_VALIDATE");
  ctx->validate = val && val[0] == '1';
  e = hipMalloc(&ctx->err, sizeof(int32_t));
  if (e == hipSuccess) e = hipMemset(ctx->err, 0, sizeof(int32_t));
  if (e == hipSuccess)
    e = ctx->n97.ensure(sizeof(double2) * N97_TABLE_SIZE) ? hipSuccess : hipErrorOutOfMemory;
  if (e == hipSuccess) e = launch_n97_table(ctx->n97.as<double2>(), nullptr);
  ctx->n97seg = n97seg_setup(device);
  if (e == hipSuccess && !ctx->n97seg) e = hipErrorUnknown;
  if (e == hipSuccess)
    e = ctx->work.ensure(sizeof(uint32_t) * WORK_QUEUES * WORK_STRIDE * NBUCKET)
            ? hipSuccess
            : hipErrorOutOfMemory;
  if (e == hipSuccess && !ctx->branches.create(1)) e = hipErrorUnknown;
  if (e == hipSuccess)
    e = hipMemset(ctx->work.p, 0, sizeof(uint32_t) * WORK_QUEUES * WORK_STRIDE * NBUCKET);
  if (e == hipSuccess) e = hipDeviceSynchronize();
  if (e != hipSuccess) {
    mcc_destroy(ctx);  // (releases what was created)
    return from_hip(e);
  }
#ifdef MCC_PHASE_TIMING
  if (!g_phase && hipMalloc(&g_phase, sizeof(unsigned long long) * 16 * NBUCKET) == hipSuccess)
    (void)hipMemset(g_phase, 0, sizeof(unsigned long long) * 16 * NBUCKET);
#endif
  for (int m = 0; m < NMODE; ++m) {
    const void *const *tab = kernel_table(m);
    for (int v = 0; v < NVARIANT; ++v) {
      int nb = 0;
      e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, tab[v], variant_of(m, v).tpc, 0);
      if (e != hipSuccess || nb < 1) nb = 1;
      ctx->grid[m][v] = nb * ctx->n_cu;
    }
  }
  *out = ctx;
  return MCC_OK;
}

mcc_status mcc_set_stream(mcc_ctx *ctx, void *hip_stream) {
  if (!ctx) return MCC_ERR_INVALID;
  ctx->stream = reinterpret_cast<hipStream_t>(hip_stream);
  return MCC_OK;
}

void mcc_destroy(mcc_ctx *ctx) {
  if (!ctx) return;
  (void)hipSetDevice(ctx->device);
  (void)hipStreamSynchronize(ctx->stream);
  ctx->big.release();
  for (DevBuf *b : {&ctx->lists, &ctx->counts, &ctx->tiles, &ctx->off, &ctx->rec,
                    &ctx->place[0], &ctx->place[1], &ctx->local, &ctx->word,
                    &ctx->bin_k0, &ctx->bin_k1, &ctx->bin_v0, &ctx->bin_v1, &ctx->bin_hist,
                    &ctx->bin_pos, &ctx->grouped, &ctx->n97,
                    &ctx->work, &ctx->rb, &ctx->adj_small, &ctx->adj_big,
                    &ctx->adj_part})
    b->release();
  if (ctx->err) (void)hipFree(ctx->err);
  for (hipStream_t side : ctx->branches.side)
    if (side) (void)hipStreamSynchronize(side);
  ctx->branches.release();
  delete ctx;
}

mcc_status mcc_set_variant(mcc_ctx *ctx, int32_t bucket, int32_t variant) {
  if (!ctx || bucket < 0 || bucket >= NBUCKET || variant < -1 || variant >= NVARIANT)
    return MCC_ERR_INVALID;
  if (variant == -1) {
    ctx->variant[bucket] = -1;
    return MCC_OK;
  }
  if (kVariants[variant].cap < kBucketCap[bucket]) return MCC_ERR_INVALID;
  ctx->variant[bucket] = variant;
  return MCC_OK;
}

mcc_status mcc_sample_angles(mcc_ctx *ctx, int32_t method, int32_t precision, int64_t n,
                             const double *s, const uint32_t *a0, const uint32_t *a1, double *oc,
                             double *st, double *A) {
  if (!ctx || n < 0 || (method != MCC_TA77 && method != MCC_N97) ||
      (precision != MCC_FP64 && precision != MCC_FP32_KINEMATICS))
    return MCC_ERR_INVALID;
  if (n > 0 && (!s || !a0 || !a1 || !oc || !st)) return MCC_ERR_INVALID;
  HIP_TRY(hipSetDevice(ctx->device));
  HIP_TRY(launch_sample_angles(method, precision, n, s, a0, a1, oc, st, A,
                               ctx->n97.as<double2>(), ctx->n97seg,
                               ctx->stream));
  return finish(ctx);
}

mcc_status mcc_device_error(mcc_ctx *ctx, int32_t *code) {
  if (!ctx || !code) return MCC_ERR_INVALID;
  HIP_TRY(hipSetDevice(ctx->device));
  HIP_TRY(hipStreamSynchronize(ctx->stream));
  HIP_TRY(hipMemcpy(code, ctx->err, sizeof(int32_t), hipMemcpyDeviceToHost));
  HIP_TRY(hipMemset(ctx->err, 0, sizeof(int32_t)));
  return MCC_OK;
}

mcc_status mcc_collide_sorted(mcc_ctx *ctx, int64_t n, int32_t n_cells, int32_t n_species,
                              const int64_t *offsets, const double *weights, double *vx,
                              double *vy, double *vz, const double *cell_volume,
                              double cell_volume_scalar, const mcc_species *species,
                              int32_t n_coll, const mcc_collision *coll, double dt,
                              double coulomb_log, uint64_t seed, uint64_t step,
                              const mcc_params *p, mcc_stats *stats, int32_t *cell_corr_pairs) {
  if (!ctx || !offsets) return MCC_ERR_INVALID;
  mcc_status st = check_step(n, n_cells, n_species, weights, vx, vy, vz, cell_volume,
                             cell_volume_scalar, species, n_coll, coll, dt, coulomb_log, p);
  if (st != MCC_OK) return st;
  HIP_TRY(hipSetDevice(ctx->device));
  if (!ensure_lists(ctx, ctx->lists, ctx->counts, n_cells)) return MCC_ERR_OOM;
  CollideArgs A;
  fill_args(A, n, n_cells, n_species, offsets, weights, vx, vy, vz, cell_volume,
            cell_volume_scalar, species, n_coll, coll, dt, coulomb_log, seed, step, p, stats,
            cell_corr_pairs, ctx);
  hipStream_t s = ctx->stream;
  if (n_cells == 0) {
    if (stats) HIP_TRY(launch_zero_stats(stats, s));
    return finish(ctx);
  }
  const int mode = mode_of(p, A);
  const Variants pick = pick_variants(ctx, mode, n_cells);
  // Room for the weight order of cells above 1024 particles, whose kernels
  // have none in LDS and without it sort in every collision, gathering weights
  // from HBM (65 536 lognormal cells in random order, FP32: 3807 us without,
  // 3734 with).  The result is the same: without memory, or in a capture
  // (whose graph must not hold a buffer that a later call may move), they sort.
  if (A.corr && A.sortw &&
      (pick.most_cells(n, n_cells, 4) > 0 || pick.most_cells(n, n_cells, 5) > 0)) {
    hipStreamCaptureStatus cap = hipStreamCaptureStatusActive;
    if (hipStreamIsCapturing(s, &cap) == hipSuccess && cap == hipStreamCaptureStatusNone &&
        ctx->word.ensure(sizeof(uint16_t) * (size_t)n)) {
      A.prep_mode = PREP_KEEP;
      A.prep_word = ctx->word.as<uint16_t>();
    } else {
      (void)hipGetLastError();
    }
  }
  HIP_TRY(launch_front(offsets, n_cells, n_species, n, weights, ctx->lists.as<int32_t>(),
                       ctx->counts.as<uint32_t>(), cell_corr_pairs, stats, nullptr, 0, pick.first,
                       ctx->err, s));
  // (the event calls of more streams cost the host more than the overlap gains when
  // every cell has a CU to itself)
  st = launch_buckets(ctx, ctx->big, A, mode, n_cells, ctx->lists.as<int32_t>(),
                      ctx->counts.as<uint32_t>(), pick, s, nullptr,
                      n_cells > ctx->n_cu ? &ctx->branches : nullptr);
  if (st != MCC_OK) return st;
  return finish(ctx);
}

mcc_status mcc_collide_sorted_noalloc(mcc_ctx *ctx, int64_t n, int32_t n_cells,
                                      int32_t n_species, const int64_t *offsets,
                                      const double *weights, double *vx, double *vy, double *vz,
                                      const double *cell_volume, double cell_volume_scalar,
                                      const mcc_species *species, int32_t n_coll,
                                      const mcc_collision *coll, double dt, double coulomb_log,
                                      uint64_t seed, uint64_t step, const mcc_params *p,
                                      mcc_stats *stats, int32_t *cell_corr_pairs) {
  if (!ctx || !offsets) return MCC_ERR_INVALID;
  mcc_status st = check_step(n, n_cells, n_species, weights, vx, vy, vz, cell_volume,
                             cell_volume_scalar, species, n_coll, coll, dt, coulomb_log, p);
  if (st != MCC_OK) return st;
  if (n_cells > NOALLOC_MAX_CELLS) return MCC_ERR_INVALID;
  if (p->relativistic) return MCC_ERR_UNSUPPORTED;
  HIP_TRY(hipSetDevice(ctx->device));
  char *base = static_cast<char *>(noalloc_ptr(ctx->device));
  if (!base) return MCC_ERR_DEVICE;
  uint32_t *counts = reinterpret_cast<uint32_t *>(base);
  int32_t *lists = reinterpret_cast<int32_t *>(base + 256);
  CollideArgs A;
  fill_args(A, n, n_cells, n_species, offsets, weights, vx, vy, vz, cell_volume,
            cell_volume_scalar, species, n_coll, coll, dt, coulomb_log, seed, step, p, stats,
            cell_corr_pairs, ctx);
  const int mode = mode_of(p, A);
  hipStream_t s = ctx->stream;
  if (n_cells == 0) {
    if (stats) HIP_TRY(launch_zero_stats(stats, s));
    return finish(ctx);
  }
  Variants pick = pick_variants(ctx, mode, n_cells);
  HIP_TRY(launch_front(offsets, n_cells, n_species, n, weights, lists, counts, cell_corr_pairs,
                       stats, nullptr, 0, pick.first, ctx->err, s));
  // cells above 4096 particles need the global-scratch kernels: not stepped
  if (pick.most_cells(n, n_cells, NBUCKET - 1) > 0)
    HIP_TRY(launch_flag_nonzero(counts + (NBUCKET - 1), 2, ctx->err, s));
  BigScratch none;  // (the variants below never use it)
  for (int b = NBUCKET - 2; b >= 0; --b) {
    int v = pick.v[b];
    if (variant_of(mode, v).layout == 2) v = default_variant(mode, b, n_cells <= ctx->n_cu);
    if (variant_of(mode, v).layout == 2) return MCC_ERR_UNSUPPORTED;
    const int64_t most = pick.most_cells(n, n_cells, b);
    if (most == 0) continue;
    st = launch_bucket(ctx, none, A, mode, n_cells, lists, counts, b, v, most, s);
    if (st != MCC_OK) return st;
  }
  return finish(ctx);
}

mcc_status mcc_collide_sorted_jvp(mcc_ctx *ctx, int64_t n, int32_t n_cells, int32_t n_species,
                                  const int64_t *offsets, const double *weights, double *vx,
                                  double *vy, double *vz, double *tx, double *ty, double *tz,
                                  const double *cell_volume, double cell_volume_scalar,
                                  const mcc_species *species, int32_t n_coll,
                                  const mcc_collision *coll, double dt, double coulomb_log,
                                  double coulomb_log_tangent, uint64_t seed, uint64_t step,
                                  const mcc_params *p, int32_t update_primal,
                                  mcc_stats *stats) {
  if (!ctx || !offsets) return MCC_ERR_INVALID;
  mcc_status st = check_step(n, n_cells, n_species, weights, vx, vy, vz, cell_volume,
                             cell_volume_scalar, species, n_coll, coll, dt, coulomb_log, p);
  if (st != MCC_OK) return st;
  if (n > 0 && (!tx || !ty || !tz)) return MCC_ERR_INVALID;
  if (!std::isfinite(coulomb_log_tangent)) return MCC_ERR_INVALID;
  if (coulomb_log_tangent != 0.0 && !(coulomb_log > 0.0)) return MCC_ERR_INVALID;
  if (p->relativistic || p->precision != MCC_FP64 || p->pairing != MCC_PAIRING_ORDER_N ||
      p->method == MCC_HARD_SPHERE)
    return MCC_ERR_UNSUPPORTED;
  HIP_TRY(hipSetDevice(ctx->device));
  if (!ensure_lists(ctx, ctx->lists, ctx->counts, n_cells)) return MCC_ERR_OOM;
  CollideArgs A;
  mcc_params q = *p;
  q.diagnostics = 0;
  fill_args(A, n, n_cells, n_species, offsets, weights, vx, vy, vz, cell_volume,
            cell_volume_scalar, species, n_coll, coll, dt, coulomb_log, seed, step, &q, stats,
            nullptr, ctx);
  A.tx = tx;
  A.ty = ty;
  A.tz = tz;
  A.dlnl = coulomb_log_tangent != 0.0 ? coulomb_log_tangent / coulomb_log : 0.0;
  A.write_primal = update_primal ? 1 : 0;
  hipStream_t s = ctx->stream;
  const Variants pick = pick_variants(ctx, MODE_TAN, n_cells);
  HIP_TRY(launch_front(offsets, n_cells, n_species, n, weights, ctx->lists.as<int32_t>(),
                       ctx->counts.as<uint32_t>(), nullptr, stats, nullptr, 0, pick.first,
                       ctx->err, s));
  if (n_cells == 0) return finish(ctx);
  // (one stream: 1024 cells of 512 in one bucket 96 us, 135 on two)
  st = launch_buckets(ctx, ctx->big, A, MODE_TAN, n_cells, ctx->lists.as<int32_t>(),
                      ctx->counts.as<uint32_t>(), pick, s);
  if (st != MCC_OK) return st;
  return finish(ctx);
}

mcc_status mcc_collide_adjoint(mcc_ctx *ctx, int64_t n, int32_t n_cells, int32_t n_species,
                               const int64_t *offsets, const double *weights, const double *vx,
                               const double *vy, const double *vz, double *gx, double *gy,
                               double *gz, const double *cell_volume,
                               double cell_volume_scalar, const mcc_species *species,
                               int32_t n_coll, const mcc_collision *coll, double dt,
                               double coulomb_log, uint64_t seed, uint64_t step,
                               const mcc_params *p, double *g_coulomb_log) {
  if (!ctx || !offsets) return MCC_ERR_INVALID;
  mcc_status st = check_step(n, n_cells, n_species, weights, vx, vy, vz, cell_volume,
                             cell_volume_scalar, species, n_coll, coll, dt, coulomb_log, p);
  if (st != MCC_OK) return st;
  if (n > 0 && (!gx || !gy || !gz)) return MCC_ERR_INVALID;
  if (p->relativistic || p->pairing != MCC_PAIRING_ORDER_N || p->method == MCC_HARD_SPHERE ||
      p->max_passes != 1)
    return MCC_ERR_UNSUPPORTED;
  HIP_TRY(hipSetDevice(ctx->device));
  if (!ensure_lists(ctx, ctx->lists, ctx->counts, n_cells) ||
      !ctx->adj_part.ensure(sizeof(double) * (size_t)std::max(n_cells, 1)))
    return MCC_ERR_OOM;
  CollideArgs F;
  fill_args(F, n, n_cells, n_species, offsets, weights, const_cast<double *>(vx),
            const_cast<double *>(vy), const_cast<double *>(vz), cell_volume, cell_volume_scalar,
            species, n_coll, coll, dt, coulomb_log, seed, step, p, nullptr, nullptr, ctx);
  AdjointArgs A;
  std::memset(&A, 0, sizeof(A));
  A.offsets = offsets;
  A.w = weights;
  A.vx = vx;
  A.vy = vy;
  A.vz = vz;
  A.gx = gx;
  A.gy = gy;
  A.gz = gz;
  A.cell_volume = cell_volume;
  A.dV = cell_volume_scalar;
  A.n = n;
  A.n_cells = n_cells;
  A.S = n_species;
  A.n_coll = n_coll;
  A.method = p->method;
  A.corr = F.corr;
  A.sortw = F.sortw;
  A.keep = F.keep;
  A.fE = F.fE;
  A.inv_lnl = coulomb_log > 0.0 ? 1.0 / coulomb_log : 0.0;
  A.seed = seed;
  A.step = step;
  for (int s = 0; s < n_species; ++s) A.mass[s] = F.mass[s];
  for (int k = 0; k < n_coll; ++k) A.coll[k] = F.coll[k];
  A.lnl_part = ctx->adj_part.as<double>();
  A.err = ctx->err;
  A.n97 = ctx->n97.as<double2>();
  A.n97seg = ctx->n97seg;
  hipStream_t s = ctx->stream;
  const Variants pick = pick_variants(ctx, MODE_TAN, n_cells);
  HIP_TRY(launch_front(offsets, n_cells, n_species, n, weights, ctx->lists.as<int32_t>(),
                       ctx->counts.as<uint32_t>(), nullptr, nullptr, ctx->adj_part.as<double>(),
                       n_cells, pick.first, ctx->err, s));
  if (n_cells > 0) {
    // the cell counts per size bucket size the scratch (one wait on the stream)
    uint32_t hc[NBUCKET];
    HIP_TRY(hipMemcpyAsync(hc, ctx->counts.p, sizeof(hc), hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
    const bool fp32 = p->precision == MCC_FP32_KINEMATICS;
    for (int b = 0; b < NBUCKET; ++b) {
      if (hc[b] == 0) continue;
      // (threads per cell of the forward-mode variant of the bucket)
      const AdjointKernel K =
          adjoint_kernel_for(fp32, variant_of(MODE_TAN, pick.v[b]).tpc, kBucketCap[b]);
      const bool big = K.form.cap > 4096, global = K.form.global;
      int occ = 0;
      if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, K.fn, K.form.tpc, 0) != hipSuccess ||
          occ < 1)
        occ = 1;
      // (as many workgroups of the global form as before the records of a
      // whole step were kept: its scratch is 1.3 MB and 10 MB each)
      if (global) occ = big ? 1 : 2;
      const int grid = (int)std::min<uint32_t>(hc[b], (uint32_t)(ctx->n_cu * occ));
      DevBuf &buf = big ? ctx->adj_big : ctx->adj_small;
      // (without memory for a step's records, fewer at a time: with one slot
      // less than the 228 B per particle that a fixed record took)
      A.slots = std::min(std::max(n_coll, 1), global ? ADJ_BIG_SLOTS : ADJ_MAX_SLOTS);
      for (;; --A.slots) {
        A.stride = adj_stride_bytes(K.form.cap, A.slots, global);
        if (buf.ensure(A.stride * (uint64_t)grid)) break;
        (void)hipGetLastError();
        if (A.slots == 1) return MCC_ERR_OOM;
      }
      A.scratch = buf.as<char>();
      HIP_TRY(launch_adjoint(K, A, ctx->lists.as<int32_t>(), ctx->counts.as<uint32_t>(), n_cells,
                             b, grid, s));
    }
  }
  if (g_coulomb_log)
    HIP_TRY(launch_sum_f64(ctx->adj_part.as<double>(), n_cells, g_coulomb_log, s));
  return finish(ctx);
}

// scratch of the radix passes: two key buffers, the tiles' digit histograms
// and their scan
static bool ensure_passes(mcc_ctx *ctx, int64_t n) {
  const size_t nn = (size_t)std::max<int64_t>(n, 1);
  const int64_t hb = bin_hist_entries(n);
  return ctx->bin_k0.ensure(4 * nn) && ctx->bin_k1.ensure(4 * nn) &&
         ctx->bin_hist.ensure(sizeof(uint32_t) * (size_t)hb) &&
         ctx->bin_pos.ensure(sizeof(uint32_t) * (size_t)hb) &&
         ctx->tiles.ensure(sizeof(int64_t) * (size_t)scan_tiles_needed(hb));
}

// w, vx, vy, vz in grouped order: four arrays, each starting on a memory line
static int64_t grouped_pad(int64_t n) { return (std::max<int64_t>(n, 1) + 31) / 32 * 32; }
static size_t grouped_bytes(int64_t n) { return 4 * sizeof(double) * (size_t)grouped_pad(n); }
static void grouped_arrays(mcc_ctx *ctx, int64_t n, double *g[4]) {
  for (int i = 0; i < 4; ++i) g[i] = ctx->grouped.as<double>() + i * grouped_pad(n);
}

static mcc_status bin_into(mcc_ctx *ctx, int64_t n, const int32_t *cells,
                           const int32_t *species_id, int32_t n_cells, int32_t n_species,
                           int64_t *offsets, int32_t *perm) {
  const size_t nn = (size_t)std::max<int64_t>(n, 1);
  if (!ensure_passes(ctx, n) || !ctx->bin_v0.ensure(4 * nn) || !ctx->bin_v1.ensure(4 * nn))
    return MCC_ERR_OOM;
  return from_hip(launch_bin(n, cells, species_id, n_cells, n_species,
                             ctx->bin_k0.as<uint32_t>(), ctx->bin_k1.as<uint32_t>(),
                             ctx->bin_v0.as<int32_t>(), ctx->bin_v1.as<int32_t>(),
                             ctx->bin_hist.as<uint32_t>(), ctx->bin_pos.as<uint32_t>(),
                             ctx->tiles.as<int64_t>(), offsets, perm, ctx->err, ctx->stream));
}

mcc_status mcc_bin(mcc_ctx *ctx, int64_t n, const int32_t *cells, const int32_t *species_id,
                   int32_t n_cells, int32_t n_species, int64_t *offsets_out, int32_t *perm_out) {
  if (!ctx || n < 0 || n_cells < 0 || n_species < 1 || n_species > MCC_MAX_SPECIES ||
      !offsets_out || (n > 0 && (!cells || !species_id || !perm_out)))
    return MCC_ERR_INVALID;
  if (n > (int64_t)INT32_MAX || (int64_t)n_cells * n_species > (int64_t)INT32_MAX)
    return MCC_ERR_UNSUPPORTED;
  HIP_TRY(hipSetDevice(ctx->device));
  mcc_status st = bin_into(ctx, n, cells, species_id, n_cells, n_species, offsets_out, perm_out);
  if (st != MCC_OK) return st;
  return finish(ctx);
}

namespace {
// the regrouping of mcc_rebin and mcc_rebin_out: offsets_out and perm_out
mcc_status rebin_keys(mcc_ctx *ctx, int64_t n, int32_t n_cells, int32_t n_species,
                      const int64_t *offsets, const int32_t *cells_new, int64_t *offsets_out,
                      int32_t *perm_out) {
  if (!ctx || n < 0 || n_cells < 0 || n_species < 1 || n_species > MCC_MAX_SPECIES ||
      !offsets || !offsets_out || (n > 0 && (!cells_new || !perm_out)))
    return MCC_ERR_INVALID;
  const int64_t m = (int64_t)n_cells * n_species;
  if (n > (int64_t)INT32_MAX || m > (int64_t)INT32_MAX) return MCC_ERR_UNSUPPORTED;
  if (m == 0 && n > 0) return MCC_ERR_INVALID;
  HIP_TRY(hipSetDevice(ctx->device));
  if (!ctx->rb.ensure(rebin_scratch_bytes(n, m)) ||
      !ctx->tiles.ensure(sizeof(int64_t) * (size_t)rebin_tiles_needed(n, m)))
    return MCC_ERR_OOM;
  if (m == 0) {
    HIP_TRY(launch_set_u64(reinterpret_cast<uint64_t *>(offsets_out), 0ull, ctx->stream));
    return MCC_OK;
  }
  HIP_TRY(launch_rebin(n, m, n_species, n_cells, offsets, cells_new, offsets_out, perm_out,
                       ctx->rb.p, ctx->tiles.as<int64_t>(), ctx->err, ctx->stream));
  return MCC_OK;
}
}  // namespace

mcc_status mcc_rebin(mcc_ctx *ctx, int64_t n, int32_t n_cells, int32_t n_species,
                     const int64_t *offsets, const int32_t *cells_new, int64_t *offsets_out,
                     int32_t *perm_out, double *weights, double *vx, double *vy, double *vz) {
  const int any = (weights != nullptr) + (vx != nullptr) + (vy != nullptr) + (vz != nullptr);
  if (any != 0 && any != 4) return MCC_ERR_INVALID;
  const mcc_status st =
      rebin_keys(ctx, n, n_cells, n_species, offsets, cells_new, offsets_out, perm_out);
  if (st != MCC_OK) return st;
  const size_t nn = (size_t)std::max<int64_t>(n, 1);
  if (any && n > 0 && (int64_t)n_cells * n_species > 0) {
    if (!ctx->grouped.ensure(grouped_bytes(n))) return MCC_ERR_OOM;
    double *g[4];
    grouped_arrays(ctx, n, g);
    HIP_TRY(launch_gather(n, perm_out, weights, vx, vy, vz, g[0], g[1], g[2], g[3], ctx->stream));
    const size_t b = sizeof(double) * (size_t)n;
    HIP_TRY(hipMemcpyAsync(weights, g[0], b, hipMemcpyDeviceToDevice, ctx->stream));
    HIP_TRY(hipMemcpyAsync(vx, g[1], b, hipMemcpyDeviceToDevice, ctx->stream));
    HIP_TRY(hipMemcpyAsync(vy, g[2], b, hipMemcpyDeviceToDevice, ctx->stream));
    HIP_TRY(hipMemcpyAsync(vz, g[3], b, hipMemcpyDeviceToDevice, ctx->stream));
  }
  return finish(ctx);
}

mcc_status mcc_rebin_out(mcc_ctx *ctx, int64_t n, int32_t n_cells, int32_t n_species,
                         const int64_t *offsets, const int32_t *cells_new, int64_t *offsets_out,
                         int32_t *perm_out, const double *weights, const double *vx,
                         const double *vy, const double *vz, double *weights_out,
                         double *vx_out, double *vy_out, double *vz_out) {
  if (n > 0 && (!weights || !vx || !vy || !vz || !weights_out || !vx_out || !vy_out || !vz_out))
    return MCC_ERR_INVALID;
  const double *in[4] = {weights, vx, vy, vz};
  const double *out[4] = {weights_out, vx_out, vy_out, vz_out};
  for (int i = 0; i < 4 && n > 0; ++i)
    for (int j = 0; j < 4; ++j)
      if (in[i] == out[j]) return MCC_ERR_INVALID;  // a gather cannot run in place
  const mcc_status st =
      rebin_keys(ctx, n, n_cells, n_species, offsets, cells_new, offsets_out, perm_out);
  if (st != MCC_OK) return st;
  if (n > 0 && (int64_t)n_cells * n_species > 0)
    HIP_TRY(launch_gather(n, perm_out, weights, vx, vy, vz, weights_out, vx_out, vy_out, vz_out,
                          ctx->stream));
  return finish(ctx);
}

// How the unsorted entry's payload comes into grouped order and back: moved
// with the keys by every radix pass, or gathered and scattered as 32-byte
// records by the permutation.  A pass moves the payload twice over, whatever
// the order; the records cost two random accesses a particle, cheap while they
// fit the 256 MB cache.  Whole steps, FP32 without correction, records against
// moves: two passes, 3e6 particles 433 and 387 us, 1.2e7 1739 and 1401; three,
// 1.2e6 705 and 718, 4e6 4898 and 5293, 6e6 1591 and 1637, 1.5e7 2485 and 2502,
// 1.8e7 3232 and 3190; four, 6e6 10 568 and 10 771, 1.8e7 12 422 and 12 738.
static bool payload_by_record(int64_t n, int passes) {
  return passes == 3 ? n < (int64_t)1 << 24 : passes > 3;
}

mcc_status mcc_collide(mcc_ctx *ctx, int64_t n, const int32_t *cells, const int32_t *species_id,
                       int32_t n_cells, int32_t n_species, const double *weights, double *vx,
                       double *vy, double *vz, const double *cell_volume,
                       double cell_volume_scalar, const mcc_species *species, int32_t n_coll,
                       const mcc_collision *coll, double dt, double coulomb_log, uint64_t seed,
                       uint64_t step, const mcc_params *p, mcc_stats *stats,
                       int32_t *cell_corr_pairs) {
  if (!ctx || (n > 0 && (!cells || !species_id))) return MCC_ERR_INVALID;
  mcc_status st = check_step(n, n_cells, n_species, weights, vx, vy, vz, cell_volume,
                             cell_volume_scalar, species, n_coll, coll, dt, coulomb_log, p);
  if (st != MCC_OK) return st;
  HIP_TRY(hipSetDevice(ctx->device));
  const int64_t m = (int64_t)n_cells * n_species;
  if (m > (int64_t)INT32_MAX) return MCC_ERR_UNSUPPORTED;
  const size_t nn = (size_t)std::max<int64_t>(n, 1);
  const int passes = bin_passes(m);
  const bool records = payload_by_record(n, passes);
  bool ok = ctx->off.ensure(sizeof(int64_t) * (size_t)(m + 1)) &&
            ctx->grouped.ensure(grouped_bytes(n)) && ensure_passes(ctx, n) &&
            (passes == 1 || ctx->rec.ensure(grouped_bytes(n)));  // (one pass: no records)
  uint32_t *place[3] = {};  // (four passes take the records)
  uint16_t *local[3] = {};
  if (records) {
    ok = ok && ctx->place[0].ensure(4 * nn);  // the permutation
  } else {
    ok = ok && ctx->local.ensure(2 * nn * (size_t)passes);
    for (int p = 0; ok && p < passes; ++p) {
      local[p] = ctx->local.as<uint16_t>() + (size_t)p * nn;
      if (p > 0 && p == passes - 1) {  // over the pass's input keys
        place[p] = ((p - 1) & 1 ? ctx->bin_k1 : ctx->bin_k0).as<uint32_t>();
      } else {
        ok = ctx->place[p].ensure(4 * nn);
        place[p] = ctx->place[p].as<uint32_t>();
      }
    }
  }
  if (!ok) return MCC_ERR_OOM;
  double *g[4];
  grouped_arrays(ctx, n, g);
  const double *const payload[4] = {weights, vx, vy, vz};
  double *const v_out[3] = {vx, vy, vz};
  int32_t *const perm = ctx->place[0].as<int32_t>();
  if (records) {
    st = bin_into(ctx, n, cells, species_id, n_cells, n_species, ctx->off.as<int64_t>(), perm);
    if (st != MCC_OK) return st;
    HIP_TRY(launch_gather_rec(n, perm, payload, ctx->rec.as<double>(), g, ctx->stream));
  } else {
    HIP_TRY(launch_bin_move(n, cells, species_id, n_cells, n_species, ctx->bin_k0.as<uint32_t>(),
                            ctx->bin_k1.as<uint32_t>(), place, local,
                            ctx->bin_hist.as<uint32_t>(), ctx->bin_pos.as<uint32_t>(),
                            ctx->tiles.as<int64_t>(), ctx->off.as<int64_t>(), payload, g[0],
                            ctx->rec.as<double>(), grouped_pad(n), ctx->err, ctx->stream));
  }
  const bool v = ctx->validate;
  ctx->validate = false;
  st = mcc_collide_sorted(ctx, n, n_cells, n_species, ctx->off.as<int64_t>(), g[0], g[1], g[2],
                          g[3], cell_volume, cell_volume_scalar, species, n_coll, coll, dt,
                          coulomb_log, seed, step, p, stats, cell_corr_pairs);
  ctx->validate = v;
  if (st != MCC_OK) return st;
  if (records)
    HIP_TRY(launch_scatter_back_rec(n, perm, g, ctx->rec.as<double>(), v_out, ctx->stream));
  else
    HIP_TRY(launch_move_back(n, m, place, local, g[0], ctx->rec.as<double>(), grouped_pad(n),
                             v_out, ctx->stream));
  return finish(ctx);
}

// ---------------------------------------------------------------------------
// Batched plan
// ---------------------------------------------------------------------------
// One step into the graph being captured on s (with launch_buckets' other
// streams, which only carry its branches)
static mcc_status plan_enqueue_step(mcc_plan *pl, hipStream_t s) {
  // counters are reset by kernels (no memset nodes in the graph)
  if (pl->stats) HIP_TRY(launch_zero_stats(pl->stats, s));
  const mcc_status st =
      launch_buckets(pl->ctx, pl->big, pl->args, pl->mode, pl->n_cells, pl->lists.as<int32_t>(),
                     pl->counts.as<uint32_t>(), pl->pick, s, pl->hcount,
                     &pl->ctx->branches);
  if (st != MCC_OK) return st;
  HIP_TRY(launch_inc_u64(pl->step.as<uint64_t>(), s));
  return MCC_OK;
}

// A plan's bucket work lists, largest cell first (ties by cell index), once
// at plan creation.  A persistent bucket kernel claims its cells in list
// order, so the last cells claimed are then the smallest and the grid drains
// evenly.  Cells are independent (their random numbers are keyed by cell),
// so the order changes no result.
// largest0: the particles of bucket 0's largest cell.
static hipError_t order_largest_first(mcc_plan *pl, const int64_t *offsets, int32_t n_cells,
                                      int32_t S, int64_t &largest0) {
  std::vector<int64_t> off((size_t)n_cells * S + 1);
  hipError_t e = hipMemcpy(off.data(), offsets, sizeof(int64_t) * off.size(),
                           hipMemcpyDeviceToHost);
  std::vector<int32_t> list;
  for (int b = 0; b < NBUCKET && e == hipSuccess; ++b) {
    const uint32_t k = pl->hcount[b];
    if (k < (b == 0 ? 1u : 2u)) continue;
    int32_t *dl = pl->lists.as<int32_t>() + (int64_t)b * n_cells;
    list.resize(k);
    e = hipMemcpy(list.data(), dl, sizeof(int32_t) * k, hipMemcpyDeviceToHost);
    if (e != hipSuccess) break;
    auto size = [&](int32_t c) {
      return off[(size_t)(c + 1) * S] - off[(size_t)c * S];
    };
    std::sort(list.begin(), list.end(), [&](int32_t x, int32_t y) {
      const int64_t sx = size(x), sy = size(y);
      return sx > sy || (sx == sy && x < y);
    });
    if (b == 0) largest0 = size(list[0]);
    e = hipMemcpy(dl, list.data(), sizeof(int32_t) * k, hipMemcpyHostToDevice);
  }
  return e;
}

mcc_status mcc_plan_create(mcc_ctx *ctx, mcc_plan **plan, int64_t n, int32_t n_cells,
                           int32_t n_species, const int64_t *offsets, const double *weights,
                           double *vx, double *vy, double *vz, const double *cell_volume,
                           double cell_volume_scalar, const mcc_species *species, int32_t n_coll,
                           const mcc_collision *coll, double dt, double coulomb_log, uint64_t seed,
                           const mcc_params *p, mcc_stats *stats, int32_t *cell_corr_pairs,
                           int32_t autotune) {
  if (!ctx || !plan || !offsets) return MCC_ERR_INVALID;
  *plan = nullptr;
  mcc_status st = check_step(n, n_cells, n_species, weights, vx, vy, vz, cell_volume,
                             cell_volume_scalar, species, n_coll, coll, dt, coulomb_log, p);
  if (st != MCC_OK) return st;
  HIP_TRY(hipSetDevice(ctx->device));
  mcc_plan *pl = new mcc_plan();
  pl->ctx = ctx;
  pl->n_cells = n_cells;
  pl->stats = stats;
  pl->cell_corr = cell_corr_pairs;
  if (!ensure_lists(ctx, pl->lists, pl->counts, n_cells) || !pl->step.ensure(64)) {
    mcc_plan_destroy(pl);
    return MCC_ERR_OOM;
  }
  fill_args(pl->args, n, n_cells, n_species, offsets, weights, vx, vy, vz, cell_volume,
            cell_volume_scalar, species, n_coll, coll, dt, coulomb_log, seed, 0, p, stats,
            cell_corr_pairs, ctx);
  pl->mode = mode_of(p, pl->args);
  for (int b = 0; b < NBUCKET; ++b)  // (a plan keeps every bucket's own list)
    pl->pick.v[b] = default_variant(pl->mode, b, n_cells <= ctx->n_cu);
  pl->args.step_dev = pl->step.as<uint64_t>();
  hipStream_t s = ctx->stream;
  // device work lists, built once (offsets are fixed for the plan); the
  // weights are bound to the plan too: checked here (positive and finite; a
  // violation is latched as data error 4) and never again per step
  hipError_t e = launch_front(offsets, n_cells, n_species, n, weights, pl->lists.as<int32_t>(),
                              pl->counts.as<uint32_t>(), cell_corr_pairs, nullptr, nullptr, 0,
                              pl->pick.first, ctx->err, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (e == hipSuccess)
    e = hipMemcpy(pl->hcount, pl->counts.p, sizeof(pl->hcount), hipMemcpyDeviceToHost);
  int64_t largest0 = 0;
  if (e == hipSuccess && n_cells > 0)
    e = order_largest_first(pl, offsets, n_cells, n_species, largest0);
  // Few cells, none of the smallest bucket above one wave's lanes: one wave per
  // cell, whose sums are bit for bit those of the four waves that a call runs
  // (three of them add zeros).  A call saves launches with the four-wave kernel;
  // a plan has none to save (200 cells of 60, one wave and four: FP64 34.1 and
  // 36.7 us, FP32 31.7 and 33.3, TA77 33.4 and 35.9, relativistic 45.4 and 47.7;
  // N x N FP32 112 and 109, so that form keeps the four).
  if (n_cells <= ctx->n_cu && largest0 > 0 && largest0 <= 64 && pl->mode != MODE_FP32_NXN)
    pl->pick.v[0] = kDefaultVariant[0];
  if (e != hipSuccess) {
    mcc_plan_destroy(pl);
    return from_hip(e);
  }
  if (autotune && n_cells > 0) {
    // time every candidate variant of every non-empty bucket on this
    // population; the trial steps use a scratch copy of the velocities so the
    // caller's state is untouched
    uint32_t hcounts[NBUCKET];
    e = hipMemcpy(hcounts, pl->counts.p, sizeof(hcounts), hipMemcpyDeviceToHost);
    DevBuf tv;
    const size_t nb = sizeof(double) * (size_t)std::max<int64_t>(n, 1);
    if (e != hipSuccess || !tv.ensure(3 * nb)) {
      mcc_plan_destroy(pl);
      return e != hipSuccess ? from_hip(e) : MCC_ERR_OOM;
    }
    CollideArgs T = pl->args;
    T.vx = tv.as<double>();
    T.vy = T.vx + std::max<int64_t>(n, 1);
    T.vz = T.vy + std::max<int64_t>(n, 1);
    T.stats = nullptr;
    T.cell_corr = nullptr;
    T.step_dev = nullptr;
    T.step = 0x7FFFFFFFull;
    hipEvent_t e0, e1;
    (void)hipEventCreate(&e0);
    (void)hipEventCreate(&e1);
    const void *const *tab = kernel_table(pl->mode);
    for (int b = 0; b < NBUCKET && e == hipSuccess; ++b) {
      if (hcounts[b] == 0) continue;
      double best = 1e300;
      for (int ci = 0; ci < 5 && kCandidates[b][ci] >= 0; ++ci) {
        const int v = kCandidates[b][ci];
        if (!ensure_big(ctx, pl->big, pl->mode, v)) continue;
        CollideArgs A = T;
        A.cell_list = pl->lists.as<int32_t>() + (int64_t)b * std::max(n_cells, 1);
        A.cell_count = pl->counts.as<uint32_t>() + b;
        A.work = ctx->work.as<uint32_t>() + WORK_QUEUES * WORK_STRIDE * b;
        set_big_args(pl->big, A, pl->mode, v);
        void *kargs[] = {&A};
        float ms_best = 1e30f;
        for (int rep = 0; rep < 3 && e == hipSuccess; ++rep) {
          e = hipMemcpyAsync(T.vx, vx, nb, hipMemcpyDeviceToDevice, s);
          if (e == hipSuccess) e = hipMemcpyAsync(T.vy, vy, nb, hipMemcpyDeviceToDevice, s);
          if (e == hipSuccess) e = hipMemcpyAsync(T.vz, vz, nb, hipMemcpyDeviceToDevice, s);
          if (e == hipSuccess) e = hipEventRecord(e0, s);
          if (e == hipSuccess)
            e = hipLaunchKernel(tab[v], dim3(grid_of(ctx, pl->mode, v)),
                                dim3(variant_of(pl->mode, v).tpc), kargs, 0, s);
          if (e == hipSuccess) e = hipEventRecord(e1, s);
          if (e == hipSuccess) e = hipEventSynchronize(e1);
          float ms = 0.f;
          if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
          if (rep > 0) ms_best = std::min(ms_best, ms);  // first run warms up
        }
        pl->tuned_ms[b][v] = ms_best;
        if (ms_best < best) {
          best = ms_best;
          pl->pick.v[b] = v;
        }
      }
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    tv.release();
    if (e != hipSuccess) {
      mcc_plan_destroy(pl);
      return from_hip(e);
    }
  }
  // workspace of every chosen variant exists before capture (no allocation
  // while capturing)
  for (int b = 0; b < NBUCKET; ++b)
    if (!ensure_big(ctx, pl->big, pl->mode, pl->pick.v[b])) {
      mcc_plan_destroy(pl);
      return MCC_ERR_OOM;
    }
  // the weights are bound to the plan: their per-(cell, species) sums, range
  // and class, and the descending-weight order, are computed once here (with
  // the chosen variants, so the sums round as in a step) and read by every
  // step
  if (p->moment_correction && n_cells > 0) {
    if (!pl->prep.ensure(sizeof(SpeciesPrep) * (size_t)n_cells * n_species) ||
        // (+4: the kernel reads a cell's entries in whole dwords)
        !pl->prep_word.ensure(sizeof(uint16_t) * (size_t)(std::max<int64_t>(n, 1) + 4))) {
      mcc_plan_destroy(pl);
      return MCC_ERR_OOM;
    }
    CollideArgs W = pl->args;
    W.prep_mode = PREP_WRITE;
    W.n_coll = 0;  // weight data only: no collision is applied (velocities unchanged)
    W.prep = pl->prep.as<SpeciesPrep>();
    W.prep_word = pl->prep_word.as<uint16_t>();
    W.stats = nullptr;
    W.cell_corr = nullptr;
    st = launch_buckets(ctx, pl->big, W, pl->mode, n_cells, pl->lists.as<int32_t>(),
                        pl->counts.as<uint32_t>(), pl->pick, s, pl->hcount);
    if (st == MCC_OK) st = from_hip(hipStreamSynchronize(s));
    if (st != MCC_OK) {
      mcc_plan_destroy(pl);
      return st;
    }
    pl->args.prep_mode = PREP_READ;
    pl->args.prep = W.prep;
    pl->args.prep_word = W.prep_word;
  }
  // capture one step into a graph: stats reset, bucket kernels, step += 1
  // (a default-priority stream)
  unsigned filled = 0;
  for (int b = 0; b < NBUCKET; ++b) filled |= pl->hcount[b] > 0 ? 1u << b : 0u;
  // (without another stream the plan takes those there are)
  (void)ctx->branches.create(plan_streams(n, filled) - 1);
  hipStream_t cs = nullptr;
  e = hipStreamCreateWithFlags(&cs, hipStreamNonBlocking);
  if (e == hipSuccess) e = hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal);
  if (e == hipSuccess) {
    st = plan_enqueue_step(pl, cs);
    hipError_t e2 = hipStreamEndCapture(cs, &pl->graph);
    if (st == MCC_OK && e2 != hipSuccess) st = from_hip(e2);
    if (st == MCC_OK) e = hipGraphInstantiate(&pl->exec, pl->graph, nullptr, nullptr, 0);
  }
  if (cs) (void)hipStreamDestroy(cs);
  if (e != hipSuccess || st != MCC_OK) {
    mcc_plan_destroy(pl);
    return st != MCC_OK ? st : from_hip(e);
  }
  *plan = pl;
  return MCC_OK;
}

mcc_status mcc_plan_run(mcc_plan *pl, uint64_t first_step, int32_t n_steps) {
  if (!pl || n_steps < 0) return MCC_ERR_INVALID;
  HIP_TRY(hipSetDevice(pl->ctx->device));
  hipStream_t s = pl->ctx->stream;
  HIP_TRY(launch_set_u64(pl->step.as<uint64_t>(), first_step, s));
  for (int i = 0; i < n_steps; ++i) HIP_TRY(hipGraphLaunch(pl->exec, s));
  return finish(pl->ctx);
}

mcc_status mcc_plan_run_bucket(mcc_plan *pl, int32_t bucket, uint64_t step) {
  if (!pl || bucket < 0 || bucket >= NBUCKET) return MCC_ERR_INVALID;
  HIP_TRY(hipSetDevice(pl->ctx->device));
  CollideArgs A = pl->args;
  A.step_dev = nullptr;
  A.step = step;
  const mcc_status st = launch_bucket(pl->ctx, pl->big, A, pl->mode, pl->n_cells, pl->lists.as<int32_t>(),
                                      pl->counts.as<uint32_t>(), bucket, pl->pick.v[bucket],
                                      pl->hcount[bucket], pl->ctx->stream);
  if (st != MCC_OK) return st;
  return finish(pl->ctx);
}

mcc_status mcc_plan_describe(mcc_plan *pl, char *buf, size_t len) {
  if (!pl || !buf || len == 0) return MCC_ERR_INVALID;
  uint32_t hc[NBUCKET] = {};
  HIP_TRY(hipStreamSynchronize(pl->ctx->stream));
  HIP_TRY(hipMemcpy(hc, pl->counts.p, sizeof(hc), hipMemcpyDeviceToHost));
  std::string out = "{\"buckets\": [";
  for (int b = 0; b < NBUCKET; ++b) {
    const Variant V = variant_of(pl->mode, pl->pick.v[b]);
    char tmp[512];
    std::snprintf(tmp, sizeof(tmp),
                  "%s{\"max_cell\": %d, \"cells\": %u, \"tpc\": %d, \"cap\": %d, \"layout\": %d, "
                  "\"grid\": %d, \"timed_ms\": {",
                  b ? ", " : "", kBucketCap[b], hc[b], V.tpc, V.cap, V.layout,
                  grid_of(pl->ctx, pl->mode, pl->pick.v[b]));
    out += tmp;
    bool first = true;
    for (int u = 0; u < NVARIANT; ++u) {
      if (pl->tuned_ms[b][u] <= 0.0) continue;
      const Variant U = variant_of(pl->mode, u);
      std::snprintf(tmp, sizeof(tmp), "%s\"%dx%d\": %.4f", first ? "" : ", ", U.tpc, U.cap,
                    pl->tuned_ms[b][u]);
      out += tmp;
      first = false;
    }
    out += "}}";
  }
  out += "]}";
  std::snprintf(buf, len, "%s", out.c_str());
  return MCC_OK;
}

void mcc_plan_destroy(mcc_plan *pl) {
  if (!pl) return;
  (void)hipSetDevice(pl->ctx->device);
  (void)hipStreamSynchronize(pl->ctx->stream);
  if (pl->exec) (void)hipGraphExecDestroy(pl->exec);
  if (pl->graph) (void)hipGraphDestroy(pl->graph);
  pl->lists.release();
  pl->counts.release();
  pl->step.release();
  pl->prep.release();
  pl->prep_word.release();
  pl->big.release();
  delete pl;
}

}  // extern "C"
