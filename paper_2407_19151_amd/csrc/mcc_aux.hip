// mcc_aux.hip -- small kernels around the collide kernels: cell-size
// bucketing of the work list, cell binning for the unsorted entry (count,
// scan, scatter, per-group canonical order, gather/scatter of the payload),
// and counter resets.  Every kernel bounds-checks its indices.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/mcc.h"
#include "mcc_device.hpp"
#include "mcc_variants.hpp"

namespace mcc {

__global__ void k_zero_stats(mcc_stats *s) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    s->pairs = s->corr_pairs = s->failed = s->collisions = 0ull;
    s->max_rel_dP = 0.0;
    s->max_rel_dE = 0.0;
  }
}

__global__ void k_set_u64(uint64_t *p, uint64_t v) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *p = v;
}

// data error `code` when the count of a size bucket is not zero (cells the
// caller's entry point does not step)
__global__ void k_flag_nonzero(const uint32_t *count, int32_t code, int32_t *err) {
  if (threadIdx.x == 0 && *count != 0u) atomicCAS(err, 0, code);
}

__global__ void k_inc_u64(uint64_t *p) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *p += 1ull;
}

// Work lists: cell c of size n goes to the first bucket whose capacity holds
// it.  lists[b * n_cells + i], counts[b].  Empty cells get cell_corr = 0.
// The bucket of cell c (none below `first`), or -1 where it takes no list entry.
__device__ __forceinline__ int bucket_of_cell(const int64_t *offsets, int64_t c, int32_t S,
                                              int64_t n, int first, int32_t *cell_corr,
                                              int32_t *err) {
  const int64_t b0 = offsets[c * S], b1 = offsets[(c + 1) * S];
  const int64_t sz = b1 - b0;
  if (b0 < 0 || b1 < b0 || b1 > n) {
    atomicCAS(err, 0, 1);
    return -1;
  }
  if (sz == 0) {
    if (cell_corr) cell_corr[c] = 0;
    return -1;
  }
  int b = first;
  while (b < NBUCKET && sz > kBucketCap[b]) ++b;
  if (b == NBUCKET) {
    atomicCAS(err, 0, 2);
    if (cell_corr) cell_corr[c] = 0;
    return -1;
  }
  return b;
}

// the lane's slot among its workgroup's cells of bucket b: one LDS atomic per
// wave and bucket, the lanes of a wave in order
__device__ __forceinline__ uint32_t bucket_slot(int b, uint32_t *lcount) {
  const int lane = threadIdx.x & (WAVE - 1);
  const uint64_t below = (1ull << lane) - 1ull;
  uint32_t slot = 0;
  for (int k = 0; k < NBUCKET; ++k) {
    const uint64_t m = __ballot(b == k);
    if (m == 0) continue;  // (uniform over the wave)
    const int leader = __ffsll((unsigned long long)m) - 1;
    uint32_t base = 0;
    if (lane == leader) base = atomicAdd(&lcount[k], (uint32_t)__popcll(m));
    base = __shfl(base, leader);
    if (b == k) slot = base + (uint32_t)__popcll(m & below);
  }
  return slot;
}

// whether any of the weights w[i], i = i0, i0 + stride, ... < n is not
// positive and finite: eight loads in flight per thread
__device__ __forceinline__ bool bad_weights(int64_t n, const double *w, int64_t i0,
                                            int64_t stride) {
  bool bad = false;
  int64_t i = i0;
  for (; i + 7 * stride < n; i += 8 * stride) {
    double x[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) x[j] = w[i + j * stride];
#pragma unroll
    for (int j = 0; j < 8; ++j) bad |= !(x[j] > 0.0) || x[j] == __builtin_inf();
  }
  for (; i < n; i += stride) {
    const double x = w[i];
    bad |= !(x > 0.0) || x == __builtin_inf();
  }
  return bad;
}

// What every call without a plan does before its collide kernels: the
// caller's statistics and `zero` cleared, the weights checked, and the cells
// put on the work lists.  Three forms of the same work:
//  - k_front_one: all of it in one workgroup, which needs no cleared counters
//    and so no launch before it (a launch costs the host 4-5 us; this kernel
//    takes 3 us at 3 200 particles, the four it replaces 12);
//  - k_front_clear, then k_front over the grid, where one workgroup would
//    take longer than the launch it saves.  The first cell_blocks workgroups
//    of k_front list the cells (each counts its cells per bucket in LDS and
//    reserves its slots with one global atomic per bucket), the others read
//    the weights (HBM bound: 8 B per particle).
constexpr int FRONT_TPB = 1024;
__global__ void __launch_bounds__(FRONT_TPB)
    k_front_one(const int64_t *offsets, int32_t n_cells, int32_t S, int64_t n, const double *w,
                int32_t *lists, uint32_t *counts, int32_t *cell_corr, mcc_stats *stats,
                double *zero, int64_t nzero, int first, int32_t *err) {
  __shared__ uint32_t lcount[NBUCKET];
  const int t = threadIdx.x;
  if (t < NBUCKET) lcount[t] = 0u;
  if (stats && t < (int)(sizeof(mcc_stats) / 8)) reinterpret_cast<uint64_t *>(stats)[t] = 0ull;
  for (int64_t i = t; i < nzero; i += FRONT_TPB) zero[i] = 0.0;
  __syncthreads();
  for (int64_t c0 = 0; c0 < n_cells; c0 += FRONT_TPB) {
    const int64_t c = c0 + t;
    const int b = c < n_cells ? bucket_of_cell(offsets, c, S, n, first, cell_corr, err) : -1;
    const uint32_t slot = bucket_slot(b, lcount);
    if (b >= 0) lists[(int64_t)b * n_cells + slot] = (int32_t)c;
  }
  if (bad_weights(n, w, t, FRONT_TPB)) atomicCAS(err, 0, 4);
  __syncthreads();
  if (t < NBUCKET) counts[t] = lcount[t];
}

__global__ void k_front_clear(uint32_t *counts, mcc_stats *stats, double *zero, int64_t nzero) {
  const int64_t i0 = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i0 < NBUCKET) counts[i0] = 0u;
  if (stats && i0 < (int64_t)(sizeof(mcc_stats) / 8))
    reinterpret_cast<uint64_t *>(stats)[i0] = 0ull;
  for (int64_t i = i0; i < nzero; i += (int64_t)gridDim.x * blockDim.x) zero[i] = 0.0;
}

__global__ void __launch_bounds__(256)
    k_front(const int64_t *offsets, int32_t n_cells, int32_t S, int64_t n, const double *w,
            int cell_blocks, int32_t *lists, uint32_t *counts, int32_t *cell_corr, int first,
            int32_t *err) {
  if ((int)blockIdx.x >= cell_blocks) {
    const int64_t wb = blockIdx.x - cell_blocks, nb = gridDim.x - cell_blocks;
    if (bad_weights(n, w, wb * 256 + threadIdx.x, nb * 256)) atomicCAS(err, 0, 4);
    return;
  }
  __shared__ uint32_t lcount[NBUCKET], lbase[NBUCKET];
  for (int64_t c0 = blockIdx.x * 256ll; c0 < n_cells; c0 += (int64_t)cell_blocks * 256) {
    if (threadIdx.x < NBUCKET) lcount[threadIdx.x] = 0u;
    __syncthreads();
    const int64_t c = c0 + threadIdx.x;
    const int b = c < n_cells ? bucket_of_cell(offsets, c, S, n, first, cell_corr, err) : -1;
    const uint32_t slot = bucket_slot(b, lcount);
    __syncthreads();
    if (threadIdx.x < NBUCKET)
      lbase[threadIdx.x] =
          lcount[threadIdx.x] ? atomicAdd(&counts[threadIdx.x], lcount[threadIdx.x]) : 0u;
    __syncthreads();
    if (b >= 0) lists[(int64_t)b * n_cells + lbase[b] + slot] = (int32_t)c;
    __syncthreads();  // (lcount and lbase are reused by the next chunk)
  }
}

// three-phase exclusive scan of u32 counts (totals below 2^32)
constexpr int SCAN_TPB = 256, SCAN_PPT = 8, SCAN_TILE = SCAN_TPB * SCAN_PPT;

__global__ void k_scan_tiles(const uint32_t *in, int64_t m, int64_t *tile_sums) {
  const int64_t base = (int64_t)blockIdx.x * SCAN_TILE;
  int64_t acc = 0;
  for (int j = threadIdx.x; j < SCAN_TILE; j += SCAN_TPB)
    if (base + j < m) acc += in[base + j];
  __shared__ int64_t red[SCAN_TPB];
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int s = SCAN_TPB / 2; s > 0; s >>= 1) {
    if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) tile_sums[blockIdx.x] = red[0];
}

// exclusive scan of the tile sums in one workgroup: serial chunks per
// thread, the chunk sums scanned by shuffles in each wave and across waves
__global__ void k_scan_tile_sums(int64_t *tile_sums, int64_t ntiles) {
  __shared__ int64_t wtot[SCAN_TPB / WAVE];
  const int t = threadIdx.x;
  const int64_t per = (ntiles + SCAN_TPB - 1) / SCAN_TPB;
  const int64_t lo = t * per, hi = lo + per < ntiles ? lo + per : ntiles;
  int64_t acc = 0;
  for (int64_t i = lo; i < hi; ++i) acc += tile_sums[i];
  int64_t incl = acc;
#pragma unroll
  for (int d = 1; d < WAVE; d <<= 1) {
    const int64_t y = __shfl_up(incl, d);
    if ((t & (WAVE - 1)) >= d) incl += y;
  }
  if ((t & (WAVE - 1)) == WAVE - 1) wtot[t / WAVE] = incl;
  __syncthreads();
  int64_t run = incl - acc;
#pragma unroll
  for (int k = 0; k < SCAN_TPB / WAVE; ++k)
    if (k < t / WAVE) run += wtot[k];
  for (int64_t i = lo; i < hi; ++i) {
    const int64_t x = tile_sums[i];
    tile_sums[i] = run;
    run += x;
  }
}

// a tile's prefix sums: each thread sums its SCAN_PPT consecutive entries,
// the thread sums are scanned by shuffles in each wave and across waves, and
// each thread writes its entries' offsets
__global__ void k_scan_apply(const uint32_t *in, int64_t m, const int64_t *tile_off,
                             uint32_t *out) {
  __shared__ int64_t wtot[SCAN_TPB / WAVE];
  const int t = threadIdx.x;
  const int64_t base = (int64_t)blockIdx.x * SCAN_TILE + (int64_t)t * SCAN_PPT;
  uint32_t v[SCAN_PPT];
  int64_t sum = 0;
#pragma unroll
  for (int j = 0; j < SCAN_PPT; ++j) {
    v[j] = base + j < m ? in[base + j] : 0u;
    sum += v[j];
  }
  int64_t incl = sum;
#pragma unroll
  for (int d = 1; d < WAVE; d <<= 1) {
    const int64_t y = __shfl_up(incl, d);
    if ((t & (WAVE - 1)) >= d) incl += y;
  }
  if ((t & (WAVE - 1)) == WAVE - 1) wtot[t / WAVE] = incl;
  __syncthreads();
  int64_t run = tile_off[blockIdx.x] + incl - sum;
#pragma unroll
  for (int k = 0; k < SCAN_TPB / WAVE; ++k)
    if (k < t / WAVE) run += wtot[k];
#pragma unroll
  for (int j = 0; j < SCAN_PPT; ++j) {
    if (base + j < m) out[base + j] = (uint32_t)run;
    run += v[j];
  }
}

// ----------------------------------------------------------------------------
// Binning (unsorted entry): a stable LSD radix sort of the group keys
// g = cell * S + species, 9 bits per pass (two passes up to 2^18 groups).  Each wave owns a tile of
// RADIX_ROWS rows of 64 consecutive particles.  Per pass: the tiles' digit
// histograms (digit-major, so one scan gives every (digit, tile) its first
// output position), the scan, and a scatter in which a particle's rank
// among the equal digits of its row comes from ballots over the digit bits,
// rows taken in order: the pass is stable, and no global atomics are used.
// A particle with an id out of range takes the key m (after every group),
// so it sorts to the end; the group offsets then come from the boundaries
// of the sorted keys.
// ----------------------------------------------------------------------------
constexpr int RADIX_BITS = 9, RADIX_BINS = 1 << RADIX_BITS;
constexpr int RADIX_WPB = 4;                      // waves per workgroup (one tile)
constexpr int RADIX_ROWS = 16;                    // rows of 64 particles per wave
constexpr int RADIX_TILE = RADIX_WPB * RADIX_ROWS * WAVE;  // 4096 particles
static_assert(RADIX_BINS % (RADIX_WPB * WAVE) == 0, "digits per thread");

// The tile of a workgroup.  Consecutive workgroups go to the eight XCDs in
// turn; each XCD takes a range of consecutive tiles, so that what neighbouring
// tiles share -- lines of the digit-major histograms, and the output lines in
// which one tile's run of a digit ends and the next one's begins -- meets in
// one L2.  Launched with xcd_grid(T) workgroups; at least T: no tile.
constexpr int XCDS = 8;
__device__ __forceinline__ int64_t xcd_tile(int64_t T) {
  const int64_t per = (T + XCDS - 1) / XCDS, k = blockIdx.x / XCDS;
  const int64_t tile = (blockIdx.x % XCDS) * per + k;
  return k < per && tile < T ? tile : T;
}
static inline unsigned xcd_grid(int64_t T) { return (unsigned)((T + XCDS - 1) / XCDS * XCDS); }

// The keys of a thread's RADIX_ROWS items, row by row of its wave, every load
// in flight before the first is used (n > 0; a row past the end reads the last
// item, and its key is not used).  FIRST: the group keys, m for an id out of
// range.
template <bool FIRST>
__device__ __forceinline__ void load_keys(int64_t i0, int64_t n, const int32_t *cells,
                                          const int32_t *species, int32_t n_cells, int32_t S,
                                          uint32_t m, const uint32_t *keys,
                                          uint32_t ky[RADIX_ROWS]) {
  int32_t sp[FIRST ? RADIX_ROWS : 1];
#pragma unroll
  for (int r = 0; r < RADIX_ROWS; ++r) {
    const int64_t i = i0 + r * WAVE, ic = i < n ? i : n - 1;
    if constexpr (FIRST) {
      ky[r] = (uint32_t)cells[ic];
      sp[r] = species[ic];
    } else {
      ky[r] = keys[ic];
    }
  }
  if constexpr (FIRST) {
#pragma unroll
    for (int r = 0; r < RADIX_ROWS; ++r) {
      const bool bad = ky[r] >= (uint32_t)n_cells || (uint32_t)sp[r] >= (uint32_t)S;
      ky[r] = bad ? m : ky[r] * (uint32_t)S + (uint32_t)sp[r];
    }
  }
}

// digit histogram of every tile: hist[d * T + tile]
template <bool FIRST>
__global__ void __launch_bounds__(RADIX_WPB * WAVE)
    k_radix_hist(int64_t n, const int32_t *cells, const int32_t *species, int32_t n_cells,
                 int32_t S, uint32_t m, const uint32_t *keys, int shift, int64_t T,
                 uint32_t *hist, int32_t *err) {
  constexpr int TPB = RADIX_WPB * WAVE, DPT = RADIX_BINS / TPB;  // digits per thread
  __shared__ uint32_t h[RADIX_BINS];
  const int t = threadIdx.x, wv = t / WAVE, lane = t & (WAVE - 1);
  const int64_t tile = xcd_tile(T);
  if (tile >= T) return;
#pragma unroll
  for (int j = 0; j < DPT; ++j) h[t + j * TPB] = 0u;
  const int64_t i0 = tile * RADIX_TILE + (int64_t)wv * RADIX_ROWS * WAVE + lane;
  uint32_t ky[RADIX_ROWS];
  load_keys<FIRST>(i0, n, cells, species, n_cells, S, m, keys, ky);
  __syncthreads();
  bool bad = false;
#pragma unroll
  for (int r = 0; r < RADIX_ROWS; ++r)
    if (i0 + r * WAVE < n) {
      bad |= FIRST && ky[r] == m;
      atomicAdd(&h[(ky[r] >> shift) & (RADIX_BINS - 1)], 1u);
    }
  if (FIRST && bad) atomicCAS(err, 0, 3);
  __syncthreads();
#pragma unroll
  for (int j = 0; j < DPT; ++j) hist[(int64_t)(t + j * TPB) * T + tile] = h[t + j * TPB];
}

// Stable ranks of a tile's items by the digit.  On return slot[r] is the
// item's place in the tile sorted by digit, and gbase[d] + slot its output
// position (pos[d * T + tile]: the first output position of the tile's digit
// d, from the scan of the histograms).  Wave w ranks its rows in order:
// ballots over the digit bits give an item's rank among the equal digits of
// its row, the wave's counts those of the rows before, and the scan of the
// per-(digit, wave) counts the rest.
template <class Cnt>
__device__ __forceinline__ void radix_ranks(int64_t i0, int64_t n, const uint32_t ky[RADIX_ROWS],
                                            int shift, int64_t T, int64_t tile,
                                            const uint32_t *pos, Cnt cnt, uint32_t *gbase,
                                            uint32_t *gsum, uint32_t slot[RADIX_ROWS]) {
  const int t = threadIdx.x, wv = t / WAVE, lane = t & (WAVE - 1);
  constexpr int TPB = RADIX_WPB * WAVE, DPT = RADIX_BINS / TPB;
  const uint64_t lt = (1ull << lane) - 1ull;
  uint32_t gp[DPT];  // (in flight during the ranking)
#pragma unroll
  for (int j = 0; j < DPT; ++j) gp[j] = pos[(int64_t)(DPT * t + j) * T + tile];
  for (int d = lane; d < RADIX_BINS; d += WAVE) cnt[wv][d] = 0u;
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int r = 0; r < RADIX_ROWS; ++r) {
    const bool act = i0 + r * WAVE < n;
    const uint32_t d = (ky[r] >> shift) & (RADIX_BINS - 1);
    uint64_t eq = __ballot(act);
#pragma unroll
    for (int b = 0; b < RADIX_BITS; ++b) {
      const uint64_t bb = __ballot((d >> b) & 1u);
      eq &= ((d >> b) & 1u) ? bb : ~bb;
    }
    slot[r] = act ? cnt[wv][d] + (uint32_t)__popcll(eq & lt) : 0u;
    // (every lane has read the count before the leader of its digit advances it)
    __builtin_amdgcn_wave_barrier();
    if (act && (eq & lt) == 0ull) cnt[wv][d] += (uint32_t)__popcll(eq);
    __builtin_amdgcn_wave_barrier();
  }
  __syncthreads();
  // digit totals of the tile and their exclusive scan (thread t owns the DPT
  // consecutive digits from DPT t)
  uint32_t sum = 0;
#pragma unroll
  for (int j = 0; j < DPT; ++j)
#pragma unroll
    for (int w = 0; w < RADIX_WPB; ++w) sum += cnt[w][DPT * t + j];
  uint32_t gt;
  uint32_t run = block_excl_scan1<TPB, false>(sum, gsum, gt);
#pragma unroll
  for (int j = 0; j < DPT; ++j) {
    const int d = DPT * t + j;
    gbase[d] = gp[j] - run;  // (mod 2^32: a slot added gives the position)
    // each wave's first slot within the digit
#pragma unroll
    for (int w = 0; w < RADIX_WPB; ++w) {
      const uint32_t c = cnt[w][d];
      cnt[w][d] = run;
      run += c;
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < RADIX_ROWS; ++r)
    slot[r] += cnt[wv][(ky[r] >> shift) & (RADIX_BINS - 1)];
}

// Stable scatter of (key, value) by the digit: the tile goes through LDS in
// digit order, so that every digit's run is written to consecutive addresses.
// Bound by LDS and latency (6e6 particles: 35 and 30 us for the two passes,
// 2.8 TB/s; 63 and 51 when each row's loads waited for the row before).
template <bool FIRST>
__global__ void __launch_bounds__(RADIX_WPB * WAVE)
    k_radix_scatter(int64_t n, const int32_t *cells, const int32_t *species, int32_t n_cells,
                    int32_t S, uint32_t m, const uint32_t *keys_in, const int32_t *vals_in,
                    int shift, int64_t T, const uint32_t *pos, uint32_t *keys_out,
                    int32_t *vals_out) {
  __shared__ uint32_t cnt[RADIX_WPB][RADIX_BINS];  // per wave: its digit counts
  __shared__ uint32_t gbase[RADIX_BINS];
  __shared__ uint32_t gsum[RADIX_WPB];
  __shared__ uint32_t lk[RADIX_TILE];
  __shared__ int32_t lv[RADIX_TILE];
  const int t = threadIdx.x, wv = t / WAVE, lane = t & (WAVE - 1);
  const int64_t tile = xcd_tile(T);
  if (tile >= T) return;
  const int64_t base = tile * RADIX_TILE;
  const int64_t i0 = base + (int64_t)wv * RADIX_ROWS * WAVE + lane;
  uint32_t ky[RADIX_ROWS], slot[RADIX_ROWS];
  int32_t vl[RADIX_ROWS];
  load_keys<FIRST>(i0, n, cells, species, n_cells, S, m, keys_in, ky);
#pragma unroll
  for (int r = 0; r < RADIX_ROWS; ++r) {
    const int64_t i = i0 + r * WAVE;
    vl[r] = FIRST ? (int32_t)i : vals_in[i < n ? i : n - 1];
  }
  radix_ranks(i0, n, ky, shift, T, tile, pos, cnt, gbase, gsum, slot);
#pragma unroll
  for (int r = 0; r < RADIX_ROWS; ++r)
    if (i0 + r * WAVE < n) {
      lk[slot[r]] = ky[r];
      lv[slot[r]] = vl[r];
    }
  __syncthreads();
  const int64_t tn = n - base < RADIX_TILE ? n - base : RADIX_TILE;
  for (int j = t; j < tn; j += RADIX_WPB * WAVE) {
    const uint32_t k = lk[j];
    const uint32_t g = gbase[(k >> shift) & (RADIX_BINS - 1)] + (uint32_t)j;
    keys_out[g] = k;
    vals_out[g] = lv[j];
  }
}

// group offsets from the sorted keys: offsets[g] = first position whose key
// is >= g (keys above m - 1 mark particles with bad ids, at the end).  Each
// thread takes BOUNDS_PT keys in a row (HBM bound: 4 B per particle).
constexpr int BOUNDS_PT = 8;
__global__ void __launch_bounds__(256)
    k_bin_bounds(int64_t n, const uint32_t *keys, uint32_t m, int64_t *offsets) {
  const int64_t i0 = (blockIdx.x * 256ll + threadIdx.x) * BOUNDS_PT;
  if (i0 > n) return;
  uint32_t k[BOUNDS_PT];
  if (i0 + BOUNDS_PT <= n) {  // (the key buffers are 256-byte aligned)
    const uint4 *p = reinterpret_cast<const uint4 *>(keys + i0);
#pragma unroll
    for (int j = 0; j < BOUNDS_PT / 4; ++j) {
      const uint4 q = p[j];
      k[4 * j] = q.x;
      k[4 * j + 1] = q.y;
      k[4 * j + 2] = q.z;
      k[4 * j + 3] = q.w;
    }
  } else {
#pragma unroll
    for (int j = 0; j < BOUNDS_PT; ++j) k[j] = i0 + j < n ? keys[i0 + j] : m;
  }
  int64_t prev = i0 == 0 ? -1 : (int64_t)keys[i0 - 1];
#pragma unroll
  for (int j = 0; j < BOUNDS_PT; ++j) {
    if (i0 + j > n) break;
    const int64_t kk = k[j] < m ? (int64_t)k[j] : (int64_t)m;  // (at n: m)
    for (int64_t g = prev + 1; g <= kk; ++g) offsets[g] = i0 + j;
    prev = k[j];
  }
}

__global__ void k_gather(int64_t n, const int32_t *perm, const double *w, const double *vx,
                         const double *vy, const double *vz, double *gw, double *gx, double *gy,
                         double *gz) {
  for (int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; j < n;
       j += (int64_t)gridDim.x * blockDim.x) {
    const int64_t i = perm[j];
    if (i < 0 || i >= n) continue;
    gw[j] = w[i];
    gx[j] = vx[i];
    gy[j] = vy[i];
    gz[j] = vz[i];
  }
}

// The unsorted entry's payload through 32-byte records (w, vx, vy, vz) of a
// context-owned array in the caller's order, after a binning that gave the
// permutation: a particle's random access is one aligned record, one memory
// segment, instead of an 8-byte word in each of four arrays.  Packing and
// unpacking stream.
struct alignas(32) Rec4 {
  double w, x, y, z;
};

__global__ void k_pack_rec(int64_t n, const double *w, const double *vx, const double *vy,
                           const double *vz, Rec4 *rec) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    rec[i] = Rec4{w[i], vx[i], vy[i], vz[i]};
}

__global__ void k_gather_rec(int64_t n, const int32_t *perm, const Rec4 *rec, double *gw,
                             double *gx, double *gy, double *gz) {
  for (int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; j < n;
       j += (int64_t)gridDim.x * blockDim.x) {
    const int64_t i = perm[j];
    if (i < 0 || i >= n) continue;
    const Rec4 r = rec[i];
    gw[j] = r.w;
    gx[j] = r.x;
    gy[j] = r.y;
    gz[j] = r.z;
  }
}

// whole records back (the weight unchanged), then the velocities out
__global__ void k_scatter_rec(int64_t n, const int32_t *perm, const double *gw, const double *gx,
                              const double *gy, const double *gz, Rec4 *rec) {
  for (int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; j < n;
       j += (int64_t)gridDim.x * blockDim.x) {
    const int64_t i = perm[j];
    if (i < 0 || i >= n) continue;
    rec[i] = Rec4{gw[j], gx[j], gy[j], gz[j]};
  }
}

__global__ void k_unpack_v(int64_t n, const Rec4 *rec, double *vx, double *vy, double *vz) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const Rec4 r = rec[i];
    vx[i] = r.x;
    vy[i] = r.y;
    vz[i] = r.z;
  }
}

// The unsorted entry's payload travels with the keys through the radix passes,
// each of its four arrays staged in LDS in digit order and written as runs of
// a digit (8 particles at 512 digits and tiles of 4096): neighbouring tiles
// continue each other's runs, so memory lines are used whole, where one random
// access per particle over the whole population costs a line each.  `place` and
// `local` keep, in a tile's digit order, where its items went and which of the
// tile's they are; the way back follows them, pass by pass.
struct Payload {
  const double *in[4];  // w, vx, vy, vz
  double *out[4];
};

template <bool FIRST>
__global__ void __launch_bounds__(RADIX_WPB * WAVE)
    k_radix_move(int64_t n, const int32_t *cells, const int32_t *species, int32_t n_cells,
                 int32_t S, uint32_t m, const uint32_t *keys_in, int shift, int64_t T,
                 const uint32_t *pos, uint32_t *keys_out, uint32_t *place, uint16_t *local,
                 Payload P) {
  constexpr int TPB = RADIX_WPB * WAVE;
  __shared__ uint32_t cnt[RADIX_WPB][RADIX_BINS];
  __shared__ uint32_t gbase[RADIX_BINS];
  __shared__ uint32_t gsum[RADIX_WPB];
  __shared__ double stage[RADIX_TILE];
  uint32_t *lk = reinterpret_cast<uint32_t *>(stage);  // keys and indices, before the payload
  uint16_t *li = reinterpret_cast<uint16_t *>(lk + RADIX_TILE);
  const int t = threadIdx.x, wv = t / WAVE, lane = t & (WAVE - 1);
  const int64_t tile = xcd_tile(T);
  if (tile >= T) return;
  const int64_t base = tile * RADIX_TILE;
  const int64_t i0 = base + (int64_t)wv * RADIX_ROWS * WAVE + lane;
  const int tn = (int)(n - base < RADIX_TILE ? n - base : RADIX_TILE);
  uint32_t ky[RADIX_ROWS], slot[RADIX_ROWS];
  load_keys<FIRST>(i0, n, cells, species, n_cells, S, m, keys_in, ky);
  double q[RADIX_ROWS];  // one array's rows, in flight
#pragma unroll
  for (int r = 0; r < RADIX_ROWS; ++r) {
    const int64_t i = i0 + r * WAVE;
    q[r] = P.in[0][i < n ? i : n - 1];
  }
  radix_ranks(i0, n, ky, shift, T, tile, pos, cnt, gbase, gsum, slot);
#pragma unroll
  for (int r = 0; r < RADIX_ROWS; ++r)
    if (i0 + r * WAVE < n) {
      lk[slot[r]] = ky[r];
      li[slot[r]] = (uint16_t)(i0 + r * WAVE - base);
    }
  __syncthreads();
  uint32_t g[RADIX_ROWS];  // output positions of the slots this thread writes
#pragma unroll
  for (int r = 0; r < RADIX_ROWS; ++r) {
    const int j = t + r * TPB;
    if (j < tn) {
      const uint32_t k = lk[j];
      g[r] = gbase[(k >> shift) & (RADIX_BINS - 1)] + (uint32_t)j;
      keys_out[g[r]] = k;
      place[base + j] = g[r];
      local[base + j] = li[j];
    }
  }
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    __syncthreads();
#pragma unroll
    for (int r = 0; r < RADIX_ROWS; ++r)
      if (i0 + r * WAVE < n) stage[slot[r]] = q[r];
    if (c < 3) {
#pragma unroll
      for (int r = 0; r < RADIX_ROWS; ++r) {
        const int64_t i = i0 + r * WAVE;
        q[r] = P.in[c + 1][i < n ? i : n - 1];
      }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < RADIX_ROWS; ++r)
      if (t + r * TPB < tn) P.out[c][g[r]] = stage[t + r * TPB];
  }
}

// the way back through one pass: the velocities of its output (in) to its
// input.  Read in runs and put in order in LDS: gathered by each item instead,
// with 8 B of a line per request, the two passes took 0.74 ms at 2.15e7.
__global__ void __launch_bounds__(RADIX_WPB * WAVE)
    k_move_back(int64_t n, int64_t T, const uint32_t *place, const uint16_t *local, Payload P) {
  constexpr int TPB = RADIX_WPB * WAVE;
  __shared__ double stage[RADIX_TILE];
  const int t = threadIdx.x;
  const int64_t tile = xcd_tile(T);
  if (tile >= T) return;
  const int64_t base = tile * RADIX_TILE;
  const int tn = (int)(n - base < RADIX_TILE ? n - base : RADIX_TILE);
  uint32_t g[RADIX_ROWS], li[RADIX_ROWS];
#pragma unroll
  for (int r = 0; r < RADIX_ROWS; ++r) {
    const int j = t + r * TPB, jc = j < tn ? j : tn - 1;
    g[r] = place[base + jc];
    li[r] = local[base + jc];
  }
  double q[RADIX_ROWS];  // one array's rows, in flight
#pragma unroll
  for (int r = 0; r < RADIX_ROWS; ++r) q[r] = P.in[1][g[r]];
#pragma unroll
  for (int c = 1; c < 4; ++c) {
#pragma unroll
    for (int r = 0; r < RADIX_ROWS; ++r)
      if (t + r * TPB < tn) stage[li[r]] = q[r];
    if (c < 3) {
#pragma unroll
      for (int r = 0; r < RADIX_ROWS; ++r) q[r] = P.in[c + 1][g[r]];
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < RADIX_ROWS; ++r)
      if (t + r * TPB < tn) P.out[c][base + t + r * TPB] = stage[t + r * TPB];
    __syncthreads();
  }
}

}  // namespace mcc

namespace mcc {
// the angle sampler of the collision step, evaluated alone
template <typename T>
__global__ void k_sample_angles(int method, int64_t n, const double *s, const uint32_t *a0,
                                const uint32_t *a1, double *oc, double *st, double *A,
                                const double2 *tab, const double *seg) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    T o, t;
    const T si = (T)s[i];
    double a = 0.0;
    if constexpr (sizeof(T) == 8) {
      if (method == 1 && !(si > 0.0)) {  // (no pair: the segments take s > 0)
        o = t = 0.0;
        a = __builtin_inf();
      } else {
        sample_angle(method, si, a0[i], a1[i], o, t, seg);
        if (method == 1 && !(si > KMath<double>::S_ISO)) a = 1.0 / n97_root(si, seg).R();
      }
    } else {
      sample_angle(method, si, a0[i], a1[i], o, t, tab);
      if (method == 1) a = (double)n97_A_fast(si, tab);
    }
    oc[i] = (double)o;
    st[i] = (double)t;
    if (A) A[i] = a;
  }
}

// the N97 table: A at the knots t_i = T0 + i h (s = e^t) from the bracketed
// solver, and h dA/dt = -h s exp(-s) / L'(A) from differentiating L(A) = exp(-s)
__global__ void k_n97_table(double2 *tab) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= N97_TN) return;
  const double s = exp(N97_T0 + i * N97_H);
  const double A = n97_A<double>(s);
  const double dAdt = -s * exp(-s) / langevin_deriv<double>(A);
  tab[i] = make_double2(A, N97_H * dAdt);
}
}  // namespace mcc

// ----------------------------------------------------------------------------
// Host-side launchers (called by the runtime in mcc_api.hip)
// ----------------------------------------------------------------------------
namespace mcc {

static inline int grid_for(int64_t n, int tpb) {
  int64_t g = (n + tpb - 1) / tpb;
  if (g < 1) g = 1;
  if (g > 65536) g = 65536;
  return (int)g;
}

hipError_t launch_zero_stats(mcc_stats *st, hipStream_t s) {
  hipLaunchKernelGGL(k_zero_stats, dim3(1), dim3(64), 0, s, st);
  return hipGetLastError();
}

hipError_t launch_set_u64(uint64_t *p, uint64_t v, hipStream_t s) {
  hipLaunchKernelGGL(k_set_u64, dim3(1), dim3(64), 0, s, p, v);
  return hipGetLastError();
}

hipError_t launch_flag_nonzero(const uint32_t *count, int32_t code, int32_t *err,
                               hipStream_t s) {
  hipLaunchKernelGGL(k_flag_nonzero, dim3(1), dim3(64), 0, s, count, code, err);
  return hipGetLastError();
}

hipError_t launch_inc_u64(uint64_t *p, hipStream_t s) {
  hipLaunchKernelGGL(k_inc_u64, dim3(1), dim3(64), 0, s, p);
  return hipGetLastError();
}

// one workgroup up to these sizes: 16 cells or 16 weights per thread, the
// most whose passes stay under the cost of a second launch
constexpr int64_t FRONT_ONE_CELLS = 16 * FRONT_TPB, FRONT_ONE_WEIGHTS = 16 * FRONT_TPB;

hipError_t launch_front(const int64_t *offsets, int32_t n_cells, int32_t S, int64_t n,
                        const double *w, int32_t *lists, uint32_t *counts, int32_t *cell_corr,
                        mcc_stats *stats, double *zero, int64_t nzero, int first,
                        int32_t *err, hipStream_t s) {
  if (n_cells <= FRONT_ONE_CELLS && n <= FRONT_ONE_WEIGHTS) {
    hipLaunchKernelGGL(k_front_one, dim3(1), dim3(FRONT_TPB), 0, s, offsets, n_cells, S, n, w,
                       lists, counts, cell_corr, stats, zero, nzero, first, err);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(k_front_clear, dim3(grid_for(nzero / 4 + 1, 256)), dim3(256), 0, s, counts,
                     stats, zero, nzero);
  const int cb = n_cells > 0 ? grid_for(n_cells, 256) : 0;
  const int wb = n > 0 ? (int)(n / 2048 + 1 < 8192 ? n / 2048 + 1 : 8192) : 0;
  if (cb + wb > 0)
    hipLaunchKernelGGL(k_front, dim3(cb + wb), dim3(256), 0, s, offsets, n_cells, S, n, w, cb,
                       lists, counts, cell_corr, first, err);
  return hipGetLastError();
}

// exclusive scan of counts[m] (m > 0); tiles: scratch of ceil(m / SCAN_TILE) int64
static hipError_t launch_scan(const uint32_t *counts, int64_t m, int64_t *tiles,
                              uint32_t *offsets, hipStream_t s) {
  const int64_t nt = (m + SCAN_TILE - 1) / SCAN_TILE;
  hipLaunchKernelGGL(k_scan_tiles, dim3((unsigned)nt), dim3(SCAN_TPB), 0, s, counts, m, tiles);
  hipLaunchKernelGGL(k_scan_tile_sums, dim3(1), dim3(SCAN_TPB), 0, s, tiles, nt);
  hipLaunchKernelGGL(k_scan_apply, dim3((unsigned)nt), dim3(SCAN_TPB), 0, s, counts, m, tiles,
                     offsets);
  return hipGetLastError();
}

int64_t scan_tiles_needed(int64_t m) { return (m + SCAN_TILE - 1) / SCAN_TILE + 1; }

// scratch of launch_bin: two key and two value buffers of n u32, the tiles'
// digit histograms and their scanned positions
int64_t bin_tiles(int64_t n) { return (n + RADIX_TILE - 1) / RADIX_TILE; }
// entries of the digit histograms (and of their scanned positions, + 1)
int64_t bin_hist_entries(int64_t n) {
  const int64_t T = bin_tiles(n);
  return (int64_t)RADIX_BINS * (T > 0 ? T : 1);
}

// radix passes of the group keys (which run up to m, the bad-id key)
int bin_passes(int64_t m) {
  int bits = 1;
  while (bits < 32 && ((uint32_t)m >> bits) != 0u) ++bits;
  return (bits + RADIX_BITS - 1) / RADIX_BITS;
}

// the tiles' digit histograms of one pass and their scan into pos
template <bool FIRST>
static hipError_t launch_pass_positions(int64_t n, const int32_t *cells, const int32_t *species,
                                        int32_t n_cells, int32_t S, uint32_t m,
                                        const uint32_t *keys, int shift, uint32_t *hist,
                                        uint32_t *pos, int64_t *tiles, int32_t *err,
                                        hipStream_t s) {
  const int64_t T = bin_tiles(n);
  hipLaunchKernelGGL(k_radix_hist<FIRST>, dim3(xcd_grid(T)), dim3(RADIX_WPB * WAVE), 0, s, n,
                     cells, species, n_cells, S, m, keys, shift, T, hist, err);
  return launch_scan(hist, (int64_t)RADIX_BINS * T, tiles, pos, s);
}

static hipError_t launch_bounds(int64_t n, const uint32_t *keys, uint32_t m, int64_t *offsets,
                                hipStream_t s) {
  hipLaunchKernelGGL(k_bin_bounds, dim3((unsigned)(n / (256 * BOUNDS_PT) + 1)), dim3(256), 0, s,
                     n, keys, m, offsets);
  return hipGetLastError();
}

hipError_t launch_bin(int64_t n, const int32_t *cells, const int32_t *species, int32_t n_cells,
                      int32_t S, uint32_t *keys0, uint32_t *keys1, int32_t *vals0,
                      int32_t *vals1, uint32_t *hist, uint32_t *pos, int64_t *tiles,
                      int64_t *offsets, int32_t *perm, int32_t *err, hipStream_t s) {
  const uint32_t m = (uint32_t)((int64_t)n_cells * S);
  const int passes = bin_passes(m);
  const int64_t T = bin_tiles(n);
  uint32_t *kb[2] = {keys0, keys1};
  int32_t *vb[2] = {vals0, vals1};
  for (int p = 0; n > 0 && p < passes; ++p) {
    const int shift = p * RADIX_BITS;
    const uint32_t *kin = p ? kb[(p - 1) & 1] : nullptr;
    const int32_t *vin = p ? vb[(p - 1) & 1] : nullptr;
    int32_t *vout = p == passes - 1 ? perm : vb[p & 1];
    auto positions = p ? launch_pass_positions<false> : launch_pass_positions<true>;
    const hipError_t e = positions(n, cells, species, n_cells, S, m, kin, shift, hist, pos,
                                   tiles, err, s);
    if (e != hipSuccess) return e;
    auto scatter = p ? k_radix_scatter<false> : k_radix_scatter<true>;
    hipLaunchKernelGGL(scatter, dim3(xcd_grid(T)), dim3(RADIX_WPB * WAVE), 0, s, n, cells,
                       species, n_cells, S, m, kin, vin, shift, T, pos, kb[p & 1], vout);
  }
  return launch_bounds(n, kb[(passes - 1) & 1], m, offsets, s);
}

// where the payload is after pass p: the last pass leaves it in g, the ones
// before take turns, so that more passes need no more memory (g and rec are
// four arrays of n_pad >= n doubles each; a single pass uses no rec)
static double *payload_buffer(int passes, int p, double *g, double *rec) {
  return (passes - 1 - p) & 1 ? rec : g;
}

// The grouping of launch_bin with the payload moved through the passes: g
// receives w, vx, vy, vz in grouped order.  place, local: one array of n
// each per pass; the last of two or more passes may put its places over its
// input keys, keys0 or keys1 (a tile's keys are read before they are written).
hipError_t launch_bin_move(int64_t n, const int32_t *cells, const int32_t *species,
                           int32_t n_cells, int32_t S, uint32_t *keys0, uint32_t *keys1,
                           uint32_t *const *place, uint16_t *const *local, uint32_t *hist,
                           uint32_t *pos, int64_t *tiles, int64_t *offsets,
                           const double *const *payload, double *g, double *rec, int64_t n_pad,
                           int32_t *err, hipStream_t s) {
  const uint32_t m = (uint32_t)((int64_t)n_cells * S);
  const int passes = bin_passes(m);
  const int64_t T = bin_tiles(n);
  uint32_t *kb[2] = {keys0, keys1};
  for (int p = 0; n > 0 && p < passes; ++p) {
    const int shift = p * RADIX_BITS;
    const uint32_t *kin = p ? kb[(p - 1) & 1] : nullptr;
    auto positions = p ? launch_pass_positions<false> : launch_pass_positions<true>;
    const hipError_t e = positions(n, cells, species, n_cells, S, m, kin, shift, hist, pos,
                                   tiles, err, s);
    if (e != hipSuccess) return e;
    Payload P;
    for (int c = 0; c < 4; ++c) {
      P.in[c] = p ? payload_buffer(passes, p - 1, g, rec) + c * n_pad : payload[c];
      P.out[c] = payload_buffer(passes, p, g, rec) + c * n_pad;
    }
    auto move = p ? k_radix_move<false> : k_radix_move<true>;
    hipLaunchKernelGGL(move, dim3(xcd_grid(T)), dim3(RADIX_WPB * WAVE), 0, s, n, cells, species,
                       n_cells, S, m, kin, shift, T, pos, kb[p & 1], place[p], local[p],
                       P);
  }
  return launch_bounds(n, kb[(passes - 1) & 1], m, offsets, s);
}

// the velocities back to the caller's order, through the passes in reverse
hipError_t launch_move_back(int64_t n, int64_t m, uint32_t *const *place, uint16_t *const *local,
                            double *g, double *rec, int64_t n_pad, double *const *v,
                            hipStream_t s) {
  const int passes = bin_passes(m);
  const int64_t T = bin_tiles(n);
  for (int p = passes - 1; n > 0 && p >= 0; --p) {
    Payload P;
    for (int c = 1; c < 4; ++c) {
      P.in[c] = payload_buffer(passes, p, g, rec) + c * n_pad;
      P.out[c] = p ? payload_buffer(passes, p - 1, g, rec) + c * n_pad : v[c - 1];
    }
    hipLaunchKernelGGL(k_move_back, dim3(xcd_grid(T)), dim3(RADIX_WPB * WAVE), 0, s, n, T,
                       place[p], local[p], P);
  }
  return hipGetLastError();
}

// the payload into grouped order and the velocities back by perm, through
// records (rec: 32 n bytes, 32-byte aligned)
hipError_t launch_gather_rec(int64_t n, const int32_t *perm, const double *const *payload,
                             double *rec, double *const *g, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  Rec4 *r = reinterpret_cast<Rec4 *>(rec);
  hipLaunchKernelGGL(k_pack_rec, dim3(grid_for(n, 256)), dim3(256), 0, s, n, payload[0],
                     payload[1], payload[2], payload[3], r);
  hipLaunchKernelGGL(k_gather_rec, dim3(grid_for(n, 256)), dim3(256), 0, s, n, perm, r, g[0],
                     g[1], g[2], g[3]);
  return hipGetLastError();
}

hipError_t launch_scatter_back_rec(int64_t n, const int32_t *perm, double *const *g, double *rec,
                                   double *const *v, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  Rec4 *r = reinterpret_cast<Rec4 *>(rec);
  hipLaunchKernelGGL(k_scatter_rec, dim3(grid_for(n, 256)), dim3(256), 0, s, n, perm, g[0], g[1],
                     g[2], g[3], r);
  hipLaunchKernelGGL(k_unpack_v, dim3(grid_for(n, 256)), dim3(256), 0, s, n, r, v[0], v[1], v[2]);
  return hipGetLastError();
}

// ----------------------------------------------------------------------------
// The FP64 form's N97 table (N97_SEGMENTS polynomials), computed once per
// process in extended precision: on each segment the root A of Nanbu's
// equation at the Chebyshev nodes, the polynomial through 1/A and exp(-2A) or
// expm1(-2A) there by divided differences.  The truncation error is below
// 2 (1/128)^8 = 3e-17 relative, and below 1e-18 on the finer segments.
// ----------------------------------------------------------------------------
static long double n97_root_l(long double s) {
  // Newton on 1 - L(A) = -expm1(-s) (A > 1.6) or L(A) = exp(-s), from the
  // leading terms of either end
  const bool useM = s <= 0.6931471805599453L;
  const long double y = expl(-s), target = useM ? -expm1l(-s) : y;
  long double A = y < 0.5L ? 3.0L * y * (1.0L + 0.6L * y * y) : 1.0L / -expm1l(-s);
  for (int it = 0; it < 60; ++it) {
    long double g, d;
    if (A < 0.5L) {  // Lambert's continued fraction of coth A - 1/A
      const long double x2 = A * A;
      long double cf = 43.0L;
      for (int k = 20; k >= 1; --k) cf = (2.0L * k + 1.0L) + x2 / cf;
      const long double L = A / cf;
      g = useM ? target - (1.0L - L) : L - target;
      d = 1.0L / 3.0L - x2 / 15.0L + 2.0L * x2 * x2 / 189.0L - x2 * x2 * x2 / 675.0L;
    } else {
      const long double e = 2.0L / expm1l(2.0L * A), sh = sinhl(A);
      g = useM ? target - (1.0L / A - e) : (1.0L + e - 1.0L / A) - target;
      d = 1.0L / (A * A) - 1.0L / (sh * sh);
    }
    long double An = A - g / d;
    if (!(An > 0.0L)) An = 0.5L * A;
    const bool done = fabsl(An - A) <= 2e-19L * A;
    A = An;
    if (done) break;
  }
  return A;
}

struct N97Segments {
  double v[N97_SEGMENTS * N97_SEG_DOUBLES];
  N97Segments() {
    constexpr int N = N97_SEG_DEG + 1;
    // segment 0: A > 64, so 1/A = -expm1(-s) and exp(-2A) = 0
    long double fact = 1.0L;
    for (int k = 0; k < N; ++k) {
      if (k) fact *= k;
      v[k] = k == 0 ? 0.0 : (double)((k & 1 ? 1.0L : -1.0L) / fact);
      v[N + k] = 0.0;
    }
    for (int i = 1; i < N97_SEGMENTS; ++i) {
      const bool fine = i >= N97_FINE0;
      const int bits = fine ? N97_FINE_BITS : N97_SEG_BITS, k0 = i - (fine ? N97_FINE0 : 1);
      const int e = (fine ? N97_SEG_E1 : N97_SEG_E0) + (k0 >> bits);
      const int m = k0 & ((1 << bits) - 1);
      const int M = fine ? N - 1 : N;  // coefficients
      const long double c = ldexpl(1.0L + (m + 0.5L) / (1 << bits), e);
      const long double h = ldexpl(0.5L / (1 << bits), e);
      long double z[N], w[2][N];
      for (int q = 0; q < M; ++q) {
        z[q] = cosl((2 * q + 1) * 3.14159265358979323846264338L / (2 * M));
        const long double A = n97_root_l(c + h * z[q]);
        w[0][q] = 1.0L / A;
        w[1][q] = fine ? expm1l(-2.0L * A) : expl(-2.0L * A);
      }
      for (int f = 0; f < 2; ++f) {
        long double *d = w[f], p[N] = {};
        for (int o = 1; o < M; ++o)
          for (int q = M - 1; q >= o; --q) d[q] = (d[q] - d[q - 1]) / (z[q] - z[q - o]);
        for (int q = M - 1; q >= 0; --q) {  // Newton form to powers of z
          for (int k = M - 1; k > 0; --k) p[k] = p[k - 1] - z[q] * p[k];
          p[0] = d[q] - z[q] * p[0];
        }
        double *out = v + i * N97_SEG_DOUBLES + f * N;
        long double hk = 1.0L;
        for (int k = 0; k < M; ++k, hk *= h) out[k] = (double)(p[k] / hk);
        if (fine) out[M] = (double)(p[0] - (long double)out[0]);
      }
    }
  }
};

// the table on the host (built on first use; safe from several threads)
const double *n97_segments_host() {
  static const N97Segments t;
  return t.v;
}

hipError_t launch_n97_table(double2 *tab, hipStream_t s) {
  hipLaunchKernelGGL(k_n97_table, dim3((N97_TN + 63) / 64), dim3(64), 0, s, tab);
  return hipGetLastError();
}

hipError_t launch_sample_angles(int method, int precision, int64_t n, const double *s,
                                const uint32_t *a0, const uint32_t *a1, double *oc, double *st,
                                double *A, const double2 *tab, const double *seg,
                                hipStream_t st_) {
  if (n <= 0) return hipSuccess;
  if (precision == 1)
    hipLaunchKernelGGL(k_sample_angles<float>, dim3(grid_for(n, 256)), dim3(256), 0, st_, method,
                       n, s, a0, a1, oc, st, A, tab, seg);
  else
    hipLaunchKernelGGL(k_sample_angles<double>, dim3(grid_for(n, 256)), dim3(256), 0, st_,
                       method, n, s, a0, a1, oc, st, A, tab, seg);
  return hipGetLastError();
}

hipError_t launch_gather(int64_t n, const int32_t *perm, const double *w, const double *vx,
                         const double *vy, const double *vz, double *gw, double *gx, double *gy,
                         double *gz, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_gather, dim3(grid_for(n, 256)), dim3(256), 0, s, n, perm, w, vx, vy, vz,
                     gw, gx, gy, gz);
  return hipGetLastError();
}

}  // namespace mcc
