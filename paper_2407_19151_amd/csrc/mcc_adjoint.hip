// mcc_adjoint.hip -- reverse-mode derivative of one collision step: the
// vector-Jacobian product behind mcc_collide_adjoint.
//
// The step (Algorithm 1: pairing, weighted scatter with the TA77/N97 angle of
// Eq. (12), momentum restore of Eq. (17), energy violation and partition of
// Eqs. (18), (24), zero-angle pair correction of Eqs. (19)-(23), failure
// fallback of Sec. 6.2) is a smooth map of the velocities and of lnL once
// every random number and every discrete choice is fixed: the pairs, the
// acceptances, the correction order, the cut pair and the failure decision.
// For an adjoint g of the step's output, this kernel returns g J (the
// adjoint of the step's input) and g dv'/dlnL, cell by cell:
//
//   run the collisions forward, recording of each: the state at its start,
//     after its momentum restore, and (where a chain changes it) before each
//     scatter pair; its pairing; its correction pairs, their energies and the
//     cut pair; and its failure decision;
//   sweep back, last collision first: the pair corrections (disjoint pairs;
//     the cut pair's U depends on Delta E_s and on the K of the pairs before
//     it), the energy partition, the momentum restore, then the scatter
//     chains in reverse.
//
// A workgroup holds the records of up to `slots` collisions; a longer list is
// taken in groups from its end, each group's start recomputed from the
// step's input.  The forward runs in the step's own precision form (FP32
// kinematics or FP64) so that it takes the same discrete choices; the pair
// adjoints are evaluated in FP64 with that form's uniforms.  One workgroup
// per cell, with the threads per cell of the forward-mode kernels, so the
// per-cell sums are split as there (adjoint_form).
//
// Bound by the latency of the cell's phases.  Cells of up to 2048 particles
// keep what is accessed through the lists (velocities, weights, adjoints) in
// LDS, 70 B per particle of capacity, so that eight waves are resident per CU
// (the registers allow no more), and only stream the records through the
// per-workgroup global scratch: 1024 cells of 256 + 256, FP64, 136 us, against
// 478 us with everything in global scratch, 512 two-wave workgroups, and the
// collisions before k recomputed for each k.
#include "mcc_adjoint_args.hpp"
#include "mcc_collide.hpp"

namespace mcc {

// Adjoint of a scatter pair: with u = v_I - v_J, the pair's update is
// v_I += fa du (if accepted), v_J -= fb du (if accepted), du = du(u, s) the
// rotation of u by the sampled angle and s = cf w_max / |u|^3.  Given the
// adjoints (gI, gJ) of its output, returns the adjoint of u through du: the
// input's adjoints are gI + it and gJ - it.  lbar gains the pair's part of
// the lnL adjoint (s is proportional to lnL).
struct PairBar {
  double x, y, z;
};
template <typename KR>
__device__ __forceinline__ PairBar pair_adjoint(
    double ux, double uy, double uz, double wi, double wj, uint32_t kp, double cf, double fa,
    double fb, int method, uint32_t cell, uint32_t step_lo, uint32_t c3, uint32_t k0, uint32_t k1,
    const double *n97tab, double inv_lnl, double gIx, double gIy, double gIz, double gJx,
    double gJy, double gJz, double &lbar) {
  using K = KMath<double>;
  const double wmax = wi > wj ? wi : wj;
  // the primal's skips, in its own precision
  {
    const KR fx = (KR)ux, fy = (KR)uy, fz = (KR)uz;
    const KR f2 = fx * fx + fy * fy + fz * fz;
    if (f2 == KR(0)) return PairBar{0.0, 0.0, 0.0};
    const KR fs = KMath<KR>::div((KR)(cf * wmax), f2 * KMath<KR>::sqrt_(f2));
    if (!(fs > KR(0))) return PairBar{0.0, 0.0, 0.0};
  }
  const U4 r = philox(kp, cell, step_lo, c3, k0, k1);
  const double u3 = unif64(r.w);
  const bool take = u3 * wmax <= (wi < wj ? wi : wj);
  const bool ai = take || wi <= wj, aj = take || wj <= wi;
  // adjoint of du
  const double bx = (ai ? fa * gIx : 0.0) - (aj ? fb * gJx : 0.0);
  const double by = (ai ? fa * gIy : 0.0) - (aj ? fb * gJy : 0.0);
  const double bz = (ai ? fa * gIz : 0.0) - (aj ? fb * gJz : 0.0);
  if (bx == 0.0 && by == 0.0 && bz == 0.0) return PairBar{0.0, 0.0, 0.0};
  const double up2 = ux * ux + uy * uy;
  const double um2 = up2 + uz * uz;
  const double um = K::sqrt_(um2);
  const double s = (cf * wmax) / (um2 * um);
  // the form's uniforms (the FP32 form draws 23-bit ones)
  const double u0 = (double)KMath<KR>::u(r.x), u1 = (double)KMath<KR>::u(r.y);
  const double u2 = (double)KMath<KR>::u(r.z);
  // the angle and d(1 - cos)/ds
  double oc, st, ocs = 0.0;
  if (method == 0) {  // TA77: delta = tan(theta/2) scales as sqrt(s)
    const double z = sqrt(-2.0 * log(u0)) * cospi(2.0 * u1);
    const double delta = sqrt(0.5 * s) * z;
    const double d2 = delta * delta;
    if (__builtin_isinf(d2)) {
      oc = 2.0;
      st = 0.0;
    } else {
      const double q = 1.0 / (1.0 + d2);
      st = 2.0 * delta * q;
      oc = 2.0 * d2 * q;
      ocs = oc * q / s;  // 2 q^2 d(delta^2)/ds, d(delta^2)/ds = delta^2 / s
    }
  } else {
    const N97Root root = n97_root(s, n97tab);
    n97_angle(s, u0, root, oc, st);
    ocs = n97_oc_s(s, u0, oc, root);
  }
  double sp, cp;
  sincospi(2.0 * u2, &sp, &cp);
  // du (rotate_delta) in reverse: adjoints of 1 - cos, sin, |u| and u
  const double stc = st * cp, sts = st * sp;
  double ocb, stb, umb, vx, vy, vz;
  if (up2 > 0.0) {
    const double up = K::sqrt_(up2), iup = 1.0 / up;
    const double ax = ux * iup, ay = uy * iup;
    const double al = ax * bx + ay * by, cr = ax * by - ay * bx;
    ocb = -(ux * bx + uy * by + uz * bz);
    stb = cp * (uz * al - up * bz) + sp * um * cr;
    umb = sts * cr;
    const double axb = uz * stc * bx + um * sts * by, ayb = uz * stc * by - um * sts * bx;
    const double upb = -stc * bz - (axb * ax + ayb * ay) * iup;
    vx = axb * iup - oc * bx + upb * ax;
    vy = ayb * iup - oc * by + upb * ay;
    vz = stc * al - oc * bz;
  } else {
    const double al = cp * bx + sp * by;
    ocb = -uz * bz;
    stb = um * al;
    umb = st * al;
    vx = 0.0;
    vy = 0.0;
    vz = -oc * bz;
  }
  if (st != 0.0) ocb += stb * (1.0 - oc) / st;  // st^2 = oc (2 - oc), either sign of st
  // adjoint of ln s (0 where the angle does not depend on s, also where s has
  // overflowed)
  const double sb = ocs != 0.0 ? ocb * ocs * s : 0.0;
  lbar += sb * inv_lnl;
  // |u| through the rotation and through s: ds = -3 s (u . du) / |u|^2
  const double c = umb / um - 3.0 * sb / um2;
  return PairBar{vx + c * ux, vy + c * uy, vz + c * uz};
}

// What a recorded collision leaves for its reverse sweep beside its slot's
// arrays
struct AdjRec {
  double dE, ea, eb, D, res0, res1;
  int nc0, nc1, fail;
};

// GLOB: the cell lives in the per-workgroup global scratch, else in LDS.
// Cells of 2048 fill a CU's LDS: its one workgroup may take every register.
template <int TPC, int CAP, typename KR, bool GLOB>
__global__ void __launch_bounds__(TPC, GLOB || CAP * 2 / TPC > 8 ? 1 : 2) adjoint_kernel(AdjointArgs A) {
  constexpr int PPT = CAP / TPC;
  constexpr int NW = TPC / WAVE;
  constexpr int VS = GLOB ? SPACE_GLOBAL : SPACE_LDS;  // where the cell lives
  static_assert(CAP % TPC == 0 && TPC % WAVE == 0, "bad variant");
  __shared__ double red[2 * 6 * NW];
  uint64_t *redu = reinterpret_cast<uint64_t *>(red);
  __shared__ uint32_t wsum[NW];
  __shared__ uint32_t maxocc;
  __shared__ int s_so[MCC_MAX_SPECIES + 1];
  __shared__ int s_bad;
  __shared__ long long s_cb;
  __shared__ unsigned long long s_wlo[MCC_MAX_SPECIES], s_whi[MCC_MAX_SPECIES];
  __shared__ double s_sw[MCC_MAX_SPECIES], s_sw2[MCC_MAX_SPECIES];
  __shared__ int s_wflag[MCC_MAX_SPECIES];
  __shared__ int s_ncut[2];
  __shared__ double s_res[2];
  __shared__ double s_ubar[2];
  __shared__ AdjRec s_rec[ADJ_MAX_SLOTS];
  __shared__ __attribute__((aligned(16))) uint32_t lcnt[CAP + 2];

  char *const base = A.scratch + (uint64_t)blockIdx.x * A.stride;
  // record slots: 9 arrays of CAP doubles (state at the collision's start,
  // after its momentum restore, and the shared particle's before each pair),
  // the odd triple's pairs, the correction pairs (energies and members), and
  // the shuffled lists
  struct Slot {
    double *b, *q, *p, *odd, *kb;
    uint32_t *pq;
    uint16_t *list;
  };
  auto slot_of = [&](int i) -> Slot {
    double *d = reinterpret_cast<double *>(base + (uint64_t)i * adj_slot_bytes(CAP));
    Slot s;
    s.b = d;
    s.q = d + 3 * CAP;
    s.p = d + 6 * CAP;
    s.odd = d + 9 * CAP;
    s.kb = s.odd + 32;
    s.pq = reinterpret_cast<uint32_t *>(s.kb + CAP / 2);
    s.list = reinterpret_cast<uint16_t *>(s.pq + CAP / 2);
    return s;
  };
  CellMem M;
  double *W, *GX, *GY, *GZ;  // weights, and the adjoint being swept back
  if constexpr (!GLOB) {
    __shared__ double lv[7 * CAP];
    __shared__ __attribute__((aligned(16))) uint16_t lidx[5 * CAP + 4];
    M.vx = lv;
    W = lv + 3 * CAP;
    GX = lv + 4 * CAP;
    M.list0 = lidx;
    M.ord0 = lidx + CAP;
    M.ord1 = lidx + 2 * CAP;
    M.mem = lidx + 3 * CAP;
    M.word = lidx + 4 * CAP;
    // shuffle keys in the orders (dead until the weight order), pair energies
    // in the bucket counters (dead after it)
    M.key = reinterpret_cast<uint32_t *>(lidx + CAP);
    M.kbuf = reinterpret_cast<double *>(lcnt);
    M.slotbuf = nullptr;
  } else {
    double *dv = reinterpret_cast<double *>(base + (uint64_t)A.slots * adj_slot_bytes(CAP));
    M.vx = dv;
    W = dv + 3 * CAP;
    GX = dv + 4 * CAP;
    M.kbuf = dv + 7 * CAP;  // CAP / 2 doubles
    M.key = reinterpret_cast<uint32_t *>(M.kbuf + CAP / 2);
    M.slotbuf = M.key + CAP;
    uint16_t *ix = reinterpret_cast<uint16_t *>(M.slotbuf + CAP);
    M.list0 = ix;
    M.ord0 = ix + CAP;
    M.ord1 = ix + 2 * CAP;
    M.mem = ix + 3 * CAP;
    M.word = ix + 4 * CAP;
  }
  M.vy = M.vx + CAP;
  M.vz = M.vx + 2 * CAP;
  M.w = W;
  GY = GX + CAP;
  GZ = GX + 2 * CAP;
  M.cnt = lcnt;
  M.list1 = nullptr;
  M.bx = M.by = M.bz = nullptr;
  M.tx = M.ty = M.tz = M.btx = M.bty = M.btz = M.kdot = nullptr;

  const int t = threadIdx.x;
  const int lane = t & (WAVE - 1);
  const int S = A.S;
  const uint32_t step_lo = (uint32_t)A.step;
  const uint32_t k0 = (uint32_t)A.seed, k1 = (uint32_t)(A.seed >> 32);
  const uint32_t count = *A.cell_count;

  for (uint32_t li = blockIdx.x; li < count; li += gridDim.x) {
    const int cell = A.cell_list[li];
    if (t < WAVE) {
      const int64_t o = t <= S ? A.offsets[(int64_t)cell * S + t] : 0;
      const int64_t cb = __shfl(o, 0), ce = __shfl(o, S);
      const int64_t o1 = __shfl_down(o, 1);
      int bad = (t == 0 && !(cb >= 0 && ce >= cb && ce <= A.n)) ||
                (t < S && (o < cb || o1 < o || o1 > ce));
      bad = __ballot(bad) ? 1 : 0;
      if (!bad && ce - cb > CAP) bad = 2;
      if (t <= S) s_so[t] = (int)(o - cb);
      if (t == 0) {
        if (bad) atomicCAS(A.err, 0, bad);
        s_bad = bad;
        s_cb = cb;
      }
    }
    __syncthreads();
    if (s_bad) {  // skipped by the step too: its derivative is the identity
      __syncthreads();
      continue;
    }
    const int64_t cb = uni(s_cb);
    const int n = uni(s_so[S]);
    const double dV = A.cell_volume ? A.cell_volume[cell] : A.dV;
    auto load_state = [&]() {
      for (int e = t; e < n; e += TPC) {
        M.vx[e] = A.vx[cb + e];
        M.vy[e] = A.vy[cb + e];
        M.vz[e] = A.vz[cb + e];
      }
    };
    for (int e = t; e < n; e += TPC) {
      W[e] = A.w[cb + e];
      GX[e] = A.gx[cb + e];
      GY[e] = A.gy[cb + e];
      GZ[e] = A.gz[cb + e];
    }
    __syncthreads();
    if (A.corr) {
      // per species: sum w, sum w^2, the weight range and class, and the
      // descending-weight order (as the step computes them per cell)
      for (int sp = 0; sp < S; ++sp) {
        const int o = s_so[sp], ns = s_so[sp + 1] - o;
        CSum<2> acc;  // compensated, as the step sums them
        acc.zero();
        uint64_t lo[1] = {~0ull}, hi[1] = {0ull};
        for (int e = o + t; e < o + ns; e += TPC) {
          const double we = W[e];
          acc.add(0, we);
          acc.add(1, we * we);
          const uint64_t bits = (uint64_t)__double_as_longlong(we);
          lo[0] = bits < lo[0] ? bits : lo[0];
          hi[0] = bits > hi[0] ? bits : hi[0];
        }
        double tot[2];
        block_csum<TPC, 2>(acc, red, tot);
        block_minmax_u64<TPC, 1>(lo, hi, redu);
        int flag = WORDER_EQUAL;
        if (A.sortw && ns >= 2 && lo[0] != hi[0]) {
          weight_sort<TPC, PPT, GLOB>(M, ns, nullptr, o, M.word + o, lo[0], hi[0], wsum,
                                      &maxocc);
          int tie = 0;
          for (int q = t; q + 1 < ns; q += TPC)
            if (W[M.word[o + q]] == W[M.word[o + q + 1]]) tie = 1;
          flag = __syncthreads_or(tie) ? WORDER_TIES : WORDER_DISTINCT;
        }
        if (t == 0) {
          s_sw[sp] = tot[0];
          s_sw2[sp] = tot[1];
          s_wlo[sp] = lo[0];
          s_whi[sp] = hi[0];
          s_wflag[sp] = flag;
        }
      }
      __syncthreads();
    }

    // one collision of the step on M.vx/vy/vz (the step's arithmetic, the
    // choices it takes included); rec: keep in slot sl what the reverse sweep
    // needs
    auto fwd = [&](int k, bool rec, int sl) {
      const Slot R = slot_of(sl);
      const int a = A.coll[k].a, b = A.coll[k].b;
      const bool intra = a == b;
      const int oa = uni(s_so[a]), na = uni(s_so[a + 1]) - oa;
      const int ob = uni(s_so[b]), nb = uni(s_so[b + 1]) - ob;
      const CollConst &C = A.coll[k];
      const double ma = A.mass[a], mb = A.mass[b];
      auto in_a = [&](int e) { return (unsigned)(e - oa) < (unsigned)na; };
      auto part = [&](int e) { return in_a(e) || (!intra && (unsigned)(e - ob) < (unsigned)nb); };
      // the state at the collision's start goes to the slot in every case; the
      // sums below read it from there
      for (int e = t; e < n; e += TPC) {
        R.b[e] = M.vx[e];
        R.b[CAP + e] = M.vy[e];
        R.b[2 * CAP + e] = M.vz[e];
      }
      if (intra)
        shuffle_species<TPC, PPT, GLOB>(M, na, oa, (uint32_t)cell, step_lo,
                                        ctr3(A.step, k, PURPOSE_SHUFFLE0 + 0), k0, k1, M.list0,
                                        wsum, &maxocc);
      else
        shuffle_two<TPC, PPT, GLOB>(M, na, oa, nb, ob, (uint32_t)cell, step_lo,
                                    ctr3(A.step, k, PURPOSE_SHUFFLE0 + 0),
                                    ctr3(A.step, k, PURPOSE_SHUFFLE0 + 1), k0, k1, M.list0,
                                    wsum, &maxocc);
      if (rec)
        for (int i = t; i < na + (intra ? 0 : nb); i += TPC) R.list[i] = M.list0[i];
      const uint16_t *L0 = M.list0, *L1 = M.list0 + na;
      const uint32_t c3p = ctr3(A.step, k, PURPOSE_PAIR);
      const bool abig = na >= nb;
      const int Nmax = abig ? na : nb, Nmin = abig ? nb : na;
      const double nmin_dv = (intra ? (double)(na - 1) : (double)Nmin) / dV;
      const bool odd = intra && (na & 1);
      const int nch = intra ? (odd ? 1 + (na - 3) / 2 : na / 2) : Nmin;
      for (int ch = t; ch < nch; ch += TPC) {
        const int len = intra ? ((odd && ch == 0) ? 3 : 1) : (Nmax - ch + Nmin - 1) / Nmin;
        for (int r = 0; r < len; ++r) {
          int I, J;
          uint32_t kp;
          double f = 1.0;
          if (intra) {
            if (odd && ch == 0) {
              I = L0[r];
              J = L0[r == 2 ? 0 : r + 1];
              kp = (uint32_t)r;
              f = 0.5;
              if (rec) {
                R.odd[6 * r] = M.vx[I];
                R.odd[6 * r + 1] = M.vy[I];
                R.odd[6 * r + 2] = M.vz[I];
                R.odd[6 * r + 3] = M.vx[J];
                R.odd[6 * r + 4] = M.vy[J];
                R.odd[6 * r + 5] = M.vz[J];
              }
            } else if (odd) {
              I = L0[3 + 2 * (ch - 1)];
              J = L0[4 + 2 * (ch - 1)];
              kp = (uint32_t)(3 + ch - 1);
            } else {
              I = L0[2 * ch];
              J = L0[2 * ch + 1];
              kp = (uint32_t)ch;
            }
          } else {
            const int kk = r * Nmin + ch;
            I = abig ? L0[kk] : L0[ch];
            J = abig ? L1[ch] : L1[kk];
            kp = (uint32_t)kk;
            if (rec && r > 0) {  // (before a chain's first pair: the start state)
              const int sh = abig ? J : I;
              R.p[kk] = M.vx[sh];
              R.p[CAP + kk] = M.vy[sh];
              R.p[2 * CAP + kk] = M.vz[sh];
            }
          }
          const double cf = C.coef * f * nmin_dv;
          if constexpr (sizeof(KR) == 8)
            scatter_pair_nr_f64<VS, VS, CAP>(in_space<VS>(M.vx), nullptr, I, J, kp, cf, C.fa,
                                             C.fb, A.method, (uint32_t)cell, step_lo, c3p, k0,
                                             k1, A.n97seg);
          else
            scatter_pair_nr<KR>(M.vx, M.vy, M.vz, M.w, I, J, kp, cf, C.fa, C.fb, A.method,
                                (uint32_t)cell, step_lo, c3p, k0, k1, A.n97);
        }
      }
      __syncthreads();
      if (!A.corr) return;  // (no correction, no record of one: rev reads none)
      // momentum restore, Eq. (17)
      double P[3] = {0.0, 0.0, 0.0};
      for_owned<TPC, PPT, !GLOB>(n, [&](int j, int e) {
        if (part(e)) {
          const double mp = (in_a(e) ? ma : mb) * W[e];
          P[0] += mp * (M.vx[e] - R.b[e]);
          P[1] += mp * (M.vy[e] - R.b[CAP + e]);
          P[2] += mp * (M.vz[e] - R.b[2 * CAP + e]);
        }
      });
      double tot[3];
      block_sum<TPC, 3>(P, red, tot);
      const double D = ma * s_sw2[a] + (intra ? 0.0 : mb * s_sw2[b]);
      const double Bx = tot[0] / D, By = tot[1] / D, Bz = tot[2] / D;
      // energy violation, Eq. (18), and the species energies of Eq. (24)
      double es = 0.0, ec = 0.0;
      double Ev[2] = {0.0, 0.0};
      for_owned<TPC, PPT, !GLOB>(n, [&](int j, int e) {
        if (part(e)) {
          const bool isa = in_a(e);
          const double we = W[e];
          const double mp = (isa ? ma : mb) * we;
          const double vx = M.vx[e] - Bx * we, vy = M.vy[e] - By * we, vz = M.vz[e] - Bz * we;
          M.vx[e] = vx;
          M.vy[e] = vy;
          M.vz[e] = vz;
          if (rec) {
            R.q[e] = vx;
            R.q[CAP + e] = vy;
            R.q[2 * CAP + e] = vz;
          }
          const double ox = R.b[e], oy = R.b[CAP + e], oz = R.b[2 * CAP + e];
          const double dd = (vx - ox) * (vx + ox) + (vy - oy) * (vy + oy) + (vz - oz) * (vz + oz);
          csum_add(es, ec, 0.5 * mp * dd);
          const double ke = 0.5 * mp * (vx * vx + vy * vy + vz * vz);
          Ev[0] += isa ? ke : 0.0;
          Ev[1] += isa ? 0.0 : ke;
        }
      });
      double dE, et[2];
      block_sum_c1<TPC, 2>(es, ec, Ev, red, dE, et);
      double dEs0 = dE, dEs1 = 0.0, ea = 0.0, eb = 0.0;
      if (!intra && dE != 0.0) {
        ea = s_sw[a] / na * et[0];
        eb = s_sw[b] / nb * et[1];
        dEs0 = ea / (ea + eb) * dE;
        dEs1 = eb / (ea + eb) * dE;
      }
      // correction order (Alg. 1, optional sort)
      const int nsl = intra ? 1 : 2;
      const uint16_t *O0 = L0, *O1 = L1;
      if (A.sortw) {
        auto order = [&](int sp, int o, int ns, const uint16_t *L, uint16_t *ord) {
          const int f = s_wflag[sp];
          if (f == WORDER_EQUAL) return L;
          if (f == WORDER_DISTINCT) return (const uint16_t *)(M.word + o);
          weight_sort<TPC, PPT, GLOB>(M, ns, L, 0, ord, s_wlo[sp], s_whi[sp], wsum, &maxocc);
          return (const uint16_t *)ord;
        };
        O0 = order(a, oa, na, L0, M.ord0);
        if (!intra) O1 = order(b, ob, nb, L1, M.ord1);
      }
      // cut-off, Eq. (23): the first pair whose prefix sum of f_E K reaches
      // |Delta E_s| takes the remainder (one wave per species, 64 pairs at
      // a time, as the step)
      double *Kb = M.kbuf;
      const int base1 = na / 2;
      auto cutoff = [&](int s2) {
        const double E0 = s2 == 0 ? dEs0 : dEs1;
        const double sgn = E0 < 0.0 ? -1.0 : 1.0;
        const int np = (s2 == 0 ? na : nb) / 2, kb = s2 == 0 ? 0 : base1;
        double absE = fabs(E0);
        int ncut = 0;
        for (int m0 = 0; m0 < np && absE != 0.0; m0 += WAVE) {
          const int m = m0 + lane;
          double lim = 0.0;
          if (m < np) {
            const uint16_t *O = s2 ? O1 : O0;
            const double ms = s2 ? mb : ma;
            const int p = O[2 * m], q = O[2 * m + 1];
            lim = A.fE * pair_K_nr(ms * W[p], ms * W[q], M.vx[p], M.vy[p], M.vz[p], M.vx[q],
                                   M.vy[q], M.vz[q]);
          }
          const double Pi = wave_incl_scan(lim);
          const double Pprev = wave_shr1(Pi);
          const unsigned long long hit = __ballot(m < np && Pi >= absE);
          if (hit) {
            const int kc = __builtin_ctzll(hit);
            const double U = lane < kc ? lim : absE - Pprev;
            if (lane <= kc) Kb[kb + m] = sgn * U;
            ncut = m0 + kc + 1;
            absE = 0.0;
          } else {
            if (m < np) Kb[kb + m] = sgn * lim;
            const int last = (np - m0 < WAVE ? np - m0 : WAVE) - 1;
            absE -= wave_bcast(Pi, last);
            ncut = m0 + last + 1;
          }
        }
        if (lane == 0) {
          s_ncut[s2] = ncut;
          s_res[s2] = sgn * absE;
        }
      };
      if constexpr (NW > 1) {
        if (t / WAVE < nsl) cutoff(t / WAVE);
      } else {
        cutoff(0);
        if (nsl == 2) cutoff(1);
      }
      if (nsl == 1 && t == 0) {
        s_ncut[1] = 0;
        s_res[1] = 0.0;
      }
      __syncthreads();
      const int nc0 = s_ncut[0], nc1 = s_ncut[1];
      for (int m = t; m < nc0 + nc1; m += TPC) {
        const bool s1 = m >= nc0;
        const int mm = s1 ? m - nc0 : m;
        const int at = (s1 ? base1 : 0) + mm;
        const double U = Kb[at];
        const uint16_t *O = s1 ? O1 : O0;
        const int p = O[2 * mm], q = O[2 * mm + 1];
        if (rec) {
          R.kb[at] = U;
          R.pq[at] = (uint32_t)p | ((uint32_t)q << 16);
        }
        if (U == 0.0) continue;
        const double ms = s1 ? mb : ma;
        const double m1 = ms * W[p], m2 = ms * W[q];
        const double mu = m1 * m2 / (m1 + m2);
        const double rx = M.vx[p] - M.vx[q], ry = M.vy[p] - M.vy[q], rz = M.vz[p] - M.vz[q];
        const double K = 0.5 * mu * (rx * rx + ry * ry + rz * rz);
        const double x = U / K;
        const double g = -x / (1.0 + sqrt(1.0 - x));
        const double f1 = mu / m1 * g, f2 = mu / m2 * g;
        M.vx[p] += f1 * rx;
        M.vy[p] += f1 * ry;
        M.vz[p] += f1 * rz;
        M.vx[q] -= f2 * rx;
        M.vy[q] -= f2 * ry;
        M.vz[q] -= f2 * rz;
      }
      const double res0 = s_res[0], res1 = s_res[1];
      __syncthreads();
      const bool fail = res0 != 0.0 || res1 != 0.0;
      if (fail && !A.keep)
        for_owned<TPC, PPT, !GLOB>(n, [&](int j, int e) {
          if (part(e)) {
            M.vx[e] = R.b[e];
            M.vy[e] = R.b[CAP + e];
            M.vz[e] = R.b[2 * CAP + e];
          }
        });
      if (rec && t == 0) s_rec[sl] = AdjRec{dE, ea, eb, D, res0, res1, nc0, nc1, fail ? 1 : 0};
      __syncthreads();
    };

    // the reverse sweep of collision k (recorded by fwd in slot sl): GX/GY/GZ,
    // the adjoint of the collision's output, becomes that of its input; the
    // velocities are overwritten with the collision's start state
    auto rev = [&](int k, int sl, double &lbar) {
      const Slot R = slot_of(sl);
      const AdjRec &Z = s_rec[sl];
      const int a = A.coll[k].a, b = A.coll[k].b;
      const bool intra = a == b;
      const int oa = uni(s_so[a]), na = uni(s_so[a + 1]) - oa;
      const int ob = uni(s_so[b]), nb = uni(s_so[b + 1]) - ob;
      const CollConst &C = A.coll[k];
      const double ma = A.mass[a], mb = A.mass[b];
      auto in_a = [&](int e) { return (unsigned)(e - oa) < (unsigned)na; };
      auto part = [&](int e) { return in_a(e) || (!intra && (unsigned)(e - ob) < (unsigned)nb); };
      // Sec. 6.2 reset: the output is the input (Z is set only with the correction)
      if (A.corr && Z.fail && !A.keep) return;
      const double *QX = R.q, *QY = R.q + CAP, *QZ = R.q + 2 * CAP;
      for (int e = t; e < n; e += TPC) {
        M.vx[e] = R.b[e];
        M.vy[e] = R.b[CAP + e];
        M.vz[e] = R.b[2 * CAP + e];
      }
      double dEbar = 0.0, Bb[3] = {0.0, 0.0, 0.0};
      if (A.corr) {
        const int nsl = intra ? 1 : 2;
        const int base1 = na / 2;
        // the cut pair of each species: adjoint of its U (before any pair's
        // adjoint changes GX/GY/GZ)
        if (t < 2) {
          double ub = 0.0;
          const double res = t == 0 ? Z.res0 : Z.res1;
          const int nc = t == 0 ? Z.nc0 : Z.nc1;
          if (t < nsl && res == 0.0 && nc > 0) {
            const int at = (t ? base1 : 0) + nc - 1;
            const double U = R.kb[at];
            if (U != 0.0) {
              const uint32_t pq = R.pq[at];
              const int p = pq & 0xFFFFu, q = pq >> 16;
              const double ms = t ? mb : ma;
              const double m1 = ms * W[p], m2 = ms * W[q];
              const double mu = m1 * m2 / (m1 + m2);
              const double rx = QX[p] - QX[q], ry = QY[p] - QY[q], rz = QZ[p] - QZ[q];
              const double K = 0.5 * mu * (rx * rx + ry * ry + rz * rz);
              const double sq = sqrt(1.0 - U / K);
              const double a1 = mu / m1, a2 = mu / m2;
              const double gb = (a1 * GX[p] - a2 * GX[q]) * rx + (a1 * GY[p] - a2 * GY[q]) * ry +
                                (a1 * GZ[p] - a2 * GZ[q]) * rz;
              ub = -gb / (2.0 * K * sq);  // dg/dU = -1 / (2 K sqrt(1 - U/K))
            }
          }
          s_ubar[t] = ub;
        }
        __syncthreads();
        // every correction pair (disjoint): v1' = v1 + (mu/m1) g r,
        // v2' = v2 - (mu/m2) g r, r = v1 - v2, g = sqrt(1 - U/K) - 1.  A pair
        // before the cut has U/K = +-f_E (g fixed); the cut pair's g moves
        // with its K and with U = Delta E_s - sum over earlier pairs of
        // +-f_E K, whose K then carry -+f_E times the adjoint of U.
        const int nc0 = Z.nc0, nc1 = Z.nc1;
        for (int m = t; m < nc0 + nc1; m += TPC) {
          const bool s1 = m >= nc0;
          const int mm = s1 ? m - nc0 : m;
          const int at = (s1 ? base1 : 0) + mm;
          const double U = R.kb[at];
          if (U == 0.0) continue;
          const uint32_t pq = R.pq[at];
          const int p = pq & 0xFFFFu, q = pq >> 16;
          const double ms = s1 ? mb : ma;
          const double m1 = ms * W[p], m2 = ms * W[q];
          const double mu = m1 * m2 / (m1 + m2);
          const double rx = QX[p] - QX[q], ry = QY[p] - QY[q], rz = QZ[p] - QZ[q];
          const double K = 0.5 * mu * (rx * rx + ry * ry + rz * rz);
          const double x = U / K;
          const double sq = sqrt(1.0 - x);
          const double g = -x / (1.0 + sq);
          const double a1 = mu / m1, a2 = mu / m2;
          const double dx = a1 * GX[p] - a2 * GX[q], dy = a1 * GY[p] - a2 * GY[q],
                       dz = a1 * GZ[p] - a2 * GZ[q];
          const double res = s1 ? Z.res1 : Z.res0;
          const int nc = s1 ? nc1 : nc0;
          double Kbar = 0.0;
          if (res == 0.0) {
            if (mm == nc - 1) {
              const double gb = dx * rx + dy * ry + dz * rz;
              Kbar = gb * x / (2.0 * K * sq);  // dg/dK = x / (2 K sqrt(1 - x))
            } else {
              Kbar = -(U < 0.0 ? -1.0 : 1.0) * A.fE * s_ubar[s1 ? 1 : 0];
            }
          }
          // r's adjoint: g (d) + Kbar dK/dr, dK/dr = mu r
          const double rbx = g * dx + Kbar * mu * rx, rby = g * dy + Kbar * mu * ry,
                       rbz = g * dz + Kbar * mu * rz;
          GX[p] += rbx;
          GY[p] += rby;
          GZ[p] += rbz;
          GX[q] -= rbx;
          GY[q] -= rby;
          GZ[q] -= rbz;
        }
        __syncthreads();
        // energy violation (difference form of Eq. (18)) and partition
        // (Eq. (24)): the cut pairs' U adjoints are those of Delta E_s
        const double ua = s_ubar[0], ubb = nsl == 2 ? s_ubar[1] : 0.0;
        double kina = 0.0, kinb = 0.0;
        if (intra) {
          dEbar = ua;
        } else if (Z.dE != 0.0) {
          const double Ssum = Z.ea + Z.eb;
          dEbar = ua * (Z.ea / Ssum) + ubb * (Z.eb / Ssum);
          const double eabar = Z.dE * (ua - ubb) * Z.eb / (Ssum * Ssum);
          const double ebbar = -Z.dE * (ua - ubb) * Z.ea / (Ssum * Ssum);
          kina = eabar * (s_sw[a] / na);
          kinb = ebbar * (s_sw[b] / nb);
        }
        // Delta E = sum 1/2 m (|q|^2 - |b|^2), E_s = sum over s of 1/2 m |q|^2:
        // q (after the restore) takes (dEbar + kin_s) m q, b takes -dEbar m b
        // (at the end)
        double P[3] = {0.0, 0.0, 0.0};
        for (int e = t; e < n; e += TPC)
          if (part(e)) {
            const bool isa = in_a(e);
            const double mp = (isa ? ma : mb) * W[e];
            const double cq = (dEbar + (isa ? kina : kinb)) * mp;
            const double gx = GX[e] + cq * QX[e], gy = GY[e] + cq * QY[e],
                         gz = GZ[e] + cq * QZ[e];
            GX[e] = gx;
            GY[e] = gy;
            GZ[e] = gz;
            // momentum restore, q = v_ps - B w: adjoint of B is -sum w g_q
            P[0] -= W[e] * gx;
            P[1] -= W[e] * gy;
            P[2] -= W[e] * gz;
          }
        block_sum<TPC, 3>(P, red, Bb);
        // B = sum m (v_ps - b) / D: v_ps takes Bbar m / D, b takes -Bbar m / D
        for (int e = t; e < n; e += TPC)
          if (part(e)) {
            const double c = (in_a(e) ? ma : mb) * W[e] / Z.D;
            GX[e] += Bb[0] * c;
            GY[e] += Bb[1] * c;
            GZ[e] += Bb[2] * c;
          }
      }
      __syncthreads();
      // the scatter: chains of pairs (one lane each), last pair first
      const uint16_t *L0 = R.list, *L1 = R.list + na;
      const uint32_t c3p = ctr3(A.step, k, PURPOSE_PAIR);
      const bool abig = na >= nb;
      const int Nmax = abig ? na : nb, Nmin = abig ? nb : na;
      const double nmin_dv = (intra ? (double)(na - 1) : (double)Nmin) / dV;
      const bool odd = intra && (na & 1);
      const int nch = intra ? (odd ? 1 + (na - 3) / 2 : na / 2) : Nmin;
      for (int ch = t; ch < nch; ch += TPC) {
        const int len = intra ? ((odd && ch == 0) ? 3 : 1) : (Nmax - ch + Nmin - 1) / Nmin;
        for (int r = len - 1; r >= 0; --r) {
          int I, J;
          uint32_t kp;
          double f = 1.0;
          double ux, uy, uz;
          if (odd && ch == 0) {
            I = L0[r];
            J = L0[r == 2 ? 0 : r + 1];
            kp = (uint32_t)r;
            f = 0.5;
            ux = R.odd[6 * r] - R.odd[6 * r + 3];
            uy = R.odd[6 * r + 1] - R.odd[6 * r + 4];
            uz = R.odd[6 * r + 2] - R.odd[6 * r + 5];
          } else {
            if (intra) {
              const int m = odd ? 3 + 2 * (ch - 1) : 2 * ch;
              I = L0[m];
              J = L0[m + 1];
              kp = (uint32_t)(odd ? 2 + ch : ch);
            } else {
              const int kk = r * Nmin + ch;
              I = abig ? L0[kk] : L0[ch];
              J = abig ? L1[ch] : L1[kk];
              kp = (uint32_t)kk;
            }
            double ix = M.vx[I], iy = M.vy[I], iz = M.vz[I];
            double jx = M.vx[J], jy = M.vy[J], jz = M.vz[J];
            if (!intra && r > 0) {
              const double px = R.p[kp], py = R.p[CAP + kp], pz = R.p[2 * CAP + kp];
              if (abig) {
                jx = px;
                jy = py;
                jz = pz;
              } else {
                ix = px;
                iy = py;
                iz = pz;
              }
            }
            ux = ix - jx;
            uy = iy - jy;
            uz = iz - jz;
          }
          const PairBar u = pair_adjoint<KR>(ux, uy, uz, W[I], W[J], kp, C.coef * f * nmin_dv,
                                             C.fa, C.fb, A.method, (uint32_t)cell, step_lo, c3p,
                                             k0, k1, A.n97seg, A.inv_lnl, GX[I], GY[I], GZ[I],
                                             GX[J], GY[J], GZ[J], lbar);
          GX[I] += u.x;
          GY[I] += u.y;
          GZ[I] += u.z;
          GX[J] -= u.x;
          GY[J] -= u.y;
          GZ[J] -= u.z;
        }
      }
      __syncthreads();
      // the start state's adjoint through the energy and momentum sums
      if (A.corr)
        for (int e = t; e < n; e += TPC)
          if (part(e)) {
            const double mp = (in_a(e) ? ma : mb) * W[e], c = mp / Z.D;
            GX[e] += -dEbar * mp * M.vx[e] - Bb[0] * c;
            GY[e] += -dEbar * mp * M.vy[e] - Bb[1] * c;
            GZ[e] += -dEbar * mp * M.vz[e] - Bb[2] * c;
          }
      __syncthreads();
    };

    auto has_pairs = [&](int k) {
      const int a = A.coll[k].a, b = A.coll[k].b;
      const int na = uni(s_so[a + 1]) - uni(s_so[a]), nb = uni(s_so[b + 1]) - uni(s_so[b]);
      return a == b ? na >= 2 : (na > 0 && nb > 0);
    };
    double lbar = 0.0;
    for (int k1_ = A.n_coll; k1_ > 0;) {
      const int kg = k1_ > A.slots ? k1_ - A.slots : 0;  // the group [kg, k1_)
      load_state();
      __syncthreads();
      for (int k = 0; k < k1_; ++k)
        if (has_pairs(k)) fwd(k, k >= kg, k >= kg ? k - kg : 0);
      for (int k = k1_ - 1; k >= kg; --k)
        if (has_pairs(k)) rev(k, k - kg, lbar);
      k1_ = kg;
    }
    double acc[1] = {lbar}, tot[1];
    block_sum<TPC, 1>(acc, red, tot);
    if (t == 0) A.lnl_part[cell] = tot[0];
    for (int e = t; e < n; e += TPC) {
      A.gx[cb + e] = GX[e];
      A.gy[cb + e] = GY[e];
      A.gz[cb + e] = GZ[e];
    }
    __syncthreads();
  }
}

// deterministic sum of x[0..n) into out[0] (one workgroup, fixed order)
__global__ void __launch_bounds__(1024) k_sum_f64(const double *x, int64_t n, double *out) {
  __shared__ double red[2 * 6 * 16];
  double acc[1] = {0.0};
  for (int64_t i = threadIdx.x; i < n; i += 1024) acc[0] += x[i];
  double tot[1];
  block_sum<1024, 1>(acc, red, tot);
  if (threadIdx.x == 0) out[0] = tot[0];
}

template <typename KR, int TPC, int CAP, bool GLOB>
const void *adjoint_fn() {
  return reinterpret_cast<const void *>(&adjoint_kernel<TPC, CAP, KR, GLOB>);
}
template <typename KR>
const void *adjoint_kernel_of(const AdjointForm &f) {
  switch (f.cap) {
    case 128: return adjoint_fn<KR, 64, 128, false>();
    case 256: return adjoint_fn<KR, 64, 256, false>();
    case 512: return adjoint_fn<KR, 128, 512, false>();
    case 1024: return adjoint_fn<KR, 256, 1024, false>();
    case 2048:
      return f.tpc == 512 ? adjoint_fn<KR, 512, 2048, false>() : adjoint_fn<KR, 256, 2048, false>();
    case 4096: return adjoint_fn<KR, 64, 4096, true>();
    default: return adjoint_fn<KR, 64, 32768, true>();
  }
}

// the kernel of a bucket (largest cell `most`) beside the tangent's of tpc threads
AdjointKernel adjoint_kernel_for(bool fp32, int tpc, int most) {
  AdjointKernel k;
  k.form = adjoint_form(tpc, most);
  k.fn = fp32 ? adjoint_kernel_of<float>(k.form) : adjoint_kernel_of<double>(k.form);
  return k;
}

hipError_t launch_adjoint(const AdjointKernel &k, const AdjointArgs &base, const int32_t *lists,
                          const uint32_t *counts, int32_t n_cells, int b, int grid,
                          hipStream_t s) {
  AdjointArgs A = base;
  A.cell_list = lists + (int64_t)b * (n_cells > 0 ? n_cells : 1);
  A.cell_count = counts + b;
  void *kargs[] = {&A};
  return hipLaunchKernel(k.fn, dim3(grid), dim3(k.form.tpc), kargs, 0, s);
}

hipError_t launch_sum_f64(const double *x, int64_t n, double *out, hipStream_t s) {
  hipLaunchKernelGGL(k_sum_f64, dim3(1), dim3(1024), 0, s, x, n, out);
  return hipGetLastError();
}

}  // namespace mcc
