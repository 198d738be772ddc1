// The plain gradient of deep stacks: the scan kernel of nr_kernels_scan.hip (one
// workgroup of NW waves per data point, lane l owning the levels
// [l CH, (l + 1) CH), the same tape, units and records), with less work per
// node:
//  * No prefix scan of 2x2 matrices.  The cotangent of the state leaving a
//    chunk is Lambda (-Q, P) with (P, Q) that state: (p, q) (P, Q)^T = 0 at the
//    top, since r = Q / P does not change with the state's scale, and a level's
//    matrix keeps the form, with Lambda times its determinant e (1 - r'^2).  So
//    Lambda is 1 / P_0^2 times the product of the determinants above the
//    chunk: a scan of one complex number instead of four, and no cancellation
//    in (p, q) below a thick evanescent slab.
//  * The node forms, s^2 and exponent factors of nr_select.hpp, tested per node
//    for the whole workgroup (one data point, one item), and the phase
//    cotangent from the state leaving the level.
//  * Records in the order that the lanes read them (LaneRecords).
// Two waves per SIMD as there; what bounds it is the FP64 VALU (active 0.42 of each
// wave's cycles in both) with the waits of the scans' shuffles and barriers (0.19
// before, 0.23 now): 4175 VALU instructions per node and wave at 1000 slabs before,
// 3547 now.  Measured
// on MI355X, us a call (5 % dQ/Q): 64 x 1000 slabs x 200 points 4290 -> 3640;
// x 150 points: 16 x 50 slabs 163 -> 129, 16 x 100 187 -> 158, 16 x 200 290 ->
// 239, 16 x 450 503 -> 445, 8 x 800 492 -> 435, 4 x 1500 526 -> 445.
#include <type_traits>

#include "nr_scan.hpp"
#include "nr_select.hpp"

namespace nr {

namespace {

// A level's record as the lanes load it: the other factors are multiples of pd
// (0 at level 0) and lc.
struct ScanRec {
  double A, B, Nr, Ni, pd, lc;
};
// The records in the scan's own order (scan_slot): row j of lane j / CH at slot
// (j % CH) LN + j / CH, LN = ceil(rows / CH), as three planes of pairs (A, B),
// (Nr, Ni), (pd, lc), so that the lanes' loads of one level are contiguous.
// With the rows in item order each lane's 16 bytes came from a cache line of
// their own and the waves waited on the L1 (64 lines a load): the 1000-slab
// batch 4.28 ms, as with the prefix scan.  Up to two
// rows past a lane's last are read ahead of their use; they lie in the item's
// part of the workspace and are not used.
// (the workspace is only known to be aligned for doubles)
typedef double Pair __attribute__((ext_vector_type(2), aligned(8)));
struct LaneRecords {
  const Pair* ab;
  const Pair* nn;
  const Pair* pl;
  uint32_t gl;
  int CH, LN;
  // row t of this lane, t the same for every lane: a scalar base and the
  // lane's offset, so that no address stays in vector registers
  __device__ __forceinline__ ScanRec at(int t) const {
    const int q = (t >= CH) + (t >= 2 * CH);
    return get(__builtin_amdgcn_readfirstlane((t - q * CH) * LN + q), gl);
  }
  // (t differs between lanes)
  __device__ __forceinline__ ScanRec at_lane(int t) const {
    const int q = t >= CH;
    return get(0, gl + (uint32_t)((t - q * CH) * LN + q));
  }
  __device__ __forceinline__ ScanRec get(int base, uint32_t lane) const {
    const Pair x = (ab + base)[lane], y = (nn + base)[lane], z = (pl + base)[lane];
    return {x.x, x.y, y.x, y.y, z.x, z.y};
  }
};
__device__ __forceinline__ LevelRecords::Rec full_rec(const ScanRec& s) {
  constexpr double kLn2OverPi = 0.22063560015265158, kPiOverLn2 = 4.5323601418271938;
  LevelRecords::Rec r;
  r.A = s.A;
  r.B = s.B;
  r.Nr = s.Nr;
  r.Ni = s.Ni;
  r.pd = s.pd;
  r.lc = s.lc;
  r.C = s.lc * kLn264;
  r.D = s.pd * kPi64;
  r.pc = s.lc * kLn2OverPi;
  r.ld = s.pd * kPiOverLn2;
  return r;
}

struct ScanLevel {
  cd kk, g, rp, e;
};
// level jj from its medium c and the one below, n (Bn its absorption); e = 1
// at level 0, whose pd is 0
template <bool ABOVE>
__device__ __forceinline__ ScanLevel scan_level(const MathTables& T, const LevelRecords::Rec& r,
                                                const Medium& c, const Medium& n, double Bn) {
  ScanLevel o;
  o.kk = c.kz * n.kz;
  const RoughPart<ABOVE> f = rough_issue<ABOVE>(T, r, o.kk);
  const PhasePart<ABOVE> p = phase_issue<ABOVE>(T, r, c.kz);
  o.g = inv_sum_sq(c.x, n.x, r.B, Bn, o.kk) * rough_finish<ABOVE>(f);
  o.rp = mk(r.Nr, r.Ni) * o.g;
  o.e = phase_finish<ABOVE>(p);
  return o;
}

__device__ __forceinline__ cd one_minus_sq(cd z) {
  return mk(fma(z.im, z.im, fma(-z.re, z.re, 1.0)), -2.0 * (z.re * z.im));
}

}  // namespace

template <int CHT, int NW>
__global__ __launch_bounds__(64 * NW, 2) void k_grad_scan_select(KernelArgs a) {
  constexpr int NT = 64 * NW;
  constexpr bool kTapeLds = CHT >= 8;
  __shared__ Shared s;
  __shared__ double tape_lds[kTapeLds ? CHT * 4 * NT : 1];
  // per wave: the product of its lanes' chunks and of their determinants, its
  // last lane's boundary slot
  __shared__ cd xt[NW][5];
  __shared__ double xb[NW][4];
  LaneTape<CHT, kTapeLds, NT> tape;
  LaneTape<CHT + 1, false, NT> accs;
  const int gl = threadIdx.x;  // lane of the data point
  const int lane = gl & 63;    // lane of the wave
  const int wv = gl >> 6;      // wave of the data point
  auto TP = [&](int t, int f) -> double& { return tape.at(tape_lds, gl, t, f); };
  auto AC = [&](int t, int f) -> double& { return accs.at(nullptr, gl, t, f); };

  const int w = blockIdx.x;
  const int item = a.wu_item[w];
  const int ds = a.dataset_of_item[item];
  const int64_t qoff = a.q_off[ds];
  const int i = a.wu_p0[w];
  const int64_t roff = a.row_off[item];
  const int N = (int)(a.row_off[item + 1] - roff) - 2;
  const int NL = N + 1;  // levels 0..N
  const int CH = (NL + NT - 1) / NT;
  const int lo = min(gl * CH, NL), hi = min(lo + CH, NL);
  const int n = hi - lo;  // levels of this lane (0 .. CH <= CHT)
  const bool own = n > 0;
  stage_shared(s, lane, a.rule, wv == 0);
#pragma unroll
  for (int t = 0; t <= CHT; ++t)
#pragma unroll
    for (int f = 0; f < 4; ++f) AC(t, f) = 0.0;

  const double Q = a.q[qoff + i];
  const bool smeared = a.dq_over_q[ds] > 0.0;
  const double dqq = a.dqq_item ? a.dqq_item[item] : a.dq_over_q[ds];
  const double sig = a.dq != nullptr ? smear_sigma_abs(a.dq[qoff + i]) : smear_sigma_rel(Q, dqq);
  const int K = smeared ? kSmearNodes : 1;
  const int LN = (N + 2 + CH - 1) / CH;
  const double* rec0 = a.consts + roff * kRecDoubles;
  const double* ext0 = reinterpret_cast<const double*>(a.constsf) + roff * kExtDoubles;
  const LaneRecords R{reinterpret_cast<const Pair*>(rec0),
                      reinterpret_cast<const Pair*>(rec0) + CH * LN,
                      reinterpret_cast<const Pair*>(ext0), (uint32_t)gl, CH, LN};

  double Rsm = 0.0;
  bool badq = !(Q > 0.0);
  double edge = 0.0;
  uint32_t above = 0;
  {
    const double qlo = ext0[4 * (N + 2) - 2], qhi = ext0[4 * (N + 2) - 1];
    for (int k = 0; k < K; ++k) {
      const double q = (K == 1) ? Q : smear_at(Q, sig, a.rule[k]);
      const double kz0sq = kz0_squared(q);
      badq |= !(q > 0.0);
      if (__ballot(!((kz0sq >= qlo) & (kz0sq <= qhi) & (q > 0.0))) == 0) above |= 1u << k;
    }
  }

  auto node = [&](int k, auto form) {
    constexpr bool ABOVE = decltype(form)::value;
    const double q = (K == 1) ? Q : smear_at(Q, sig, ld(s.t[k]));
    const double wk = (K == 1) ? 1.0 : ld(s.w[k]);
    const double kz0sq = kz0_squared(q);
    auto med = [&](bool front, const ScanRec& r) {
      Medium o = medium<ABOVE>(kz0sq, r.A, r.B);
      if (front) {
        o.kz = mk(0.5 * q, 0.0);
        o.inv_abs2 = 0.0;
      }
      return o;
    };

    // 1. the chunk product, applied to both columns bottom-up, and its
    //    determinant; each level's r' and e are kept in its tape slot
    M2 X = m2_identity();
    cd det = mk(1.0, 0.0);
    if (own) {
      // each level's record is loaded a level ahead
      const ScanRec rb = R.at_lane(n);
      Medium mn = med(false, rb);
      double Bn = rb.B;
      if constexpr (!ABOVE) edge = fmax(edge, mn.inv_abs2);
      ScanRec rnx = R.at_lane(n - 1);
#pragma unroll
      for (int t = CHT - 1; t >= 0; --t) {
        if (t < n) {
          const ScanRec rc = rnx;
          if (t >= 1) rnx = R.at(t - 1);
          const Medium mc = med(t == 0 && gl == 0, rc);
          if constexpr (!ABOVE) edge = fmax(edge, mc.inv_abs2);
          const ScanLevel lv = scan_level<ABOVE>(s.tab, full_rec(rc), mc, mn, Bn);
          TP(t, 0) = lv.rp.re;
          TP(t, 1) = lv.rp.im;
          TP(t, 2) = lv.e.re;
          TP(t, 3) = lv.e.im;
          const cd a0 = cmul_add(lv.rp, X.c, X.a), b0 = cmul_add(lv.rp, X.d, X.b);
          X.c = lv.e * cmul_add(lv.rp, X.a, X.c);
          X.d = lv.e * cmul_add(lv.rp, X.b, X.d);
          X.a = a0;
          X.b = b0;
          det = (lv.e * det) * one_minus_sq(lv.rp);
          mn = mc;
          Bn = rc.B;
        }
      }
    }
    // 2. the suffix scan of the chunk products and the prefix scan of the
    //    determinants across the wave's lanes ...
    M2 U = X;
    cd W = det;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const M2 Yu = shfl_m2(U, lane + off < 64 ? lane + off : 63);
      const cd Yw = shfl_cd(W, lane >= off ? lane - off : 0);
      if (lane + off < 64) U = m2_mul(U, Yu);
      if (lane >= off) W = Yw * W;
    }
    // ... and across the waves
    M2 Ub;
    cd V = shfl_cd(W, lane > 0 ? lane - 1 : 0);  // determinants above the chunk
    if (lane == 0) V = mk(1.0, 0.0);
    cd P0, Q0;
    if constexpr (NW == 1) {
      Ub = shfl_m2(U, lane < 63 ? lane + 1 : 63);
      P0 = shfl_cd(U.a, 0);
      Q0 = shfl_cd(U.c, 0);
    } else {
      if (lane == 0) {
        xt[wv][0] = U.a;
        xt[wv][1] = U.b;
        xt[wv][2] = U.c;
        xt[wv][3] = U.d;
      }
      if (lane == 63) xt[wv][4] = W;
      __syncthreads();
      M2 S = m2_identity(), F = load_m2(xt[0]);
#pragma unroll
      for (int v = NW - 1; v >= 1; --v)
        if (v > wv) S = m2_mul(load_m2(xt[v]), S);
#pragma unroll
      for (int v = 0; v < NW - 1; ++v)
        if (v < wv) V = xt[v][4] * V;
      // the top state, formed in the same order by every lane
#pragma unroll
      for (int v = 1; v < NW; ++v) F = m2_mul(F, load_m2(xt[v]));
      __syncthreads();  // xt is written again at the next node
      U = m2_mul(U, S);
      Ub = shfl_m2(U, lane < 63 ? lane + 1 : 63);
      if (lane == 63) Ub = S;  // the next wave's first lane
      P0 = F.a;
      Q0 = F.c;
    }
    const cd iP = crecip(P0);
    const cd r = Q0 * iP;
    Rsm += wk * cabs2(r);
    if (!own) return;
    // conj(Lambda) rbar of this chunk's top, rbar = 2 w_k r
    const cd mu = cmulc((iP * iP) * V, (2.0 * wk) * r);
    cd Pv = mk(1.0, 0.0), Qv = mk(0.0, 0.0);
    if (gl < NT - 1) {
      Pv = Ub.a;
      Qv = Ub.c;
    }

    // 3. the lane's forward sweep from its entering state with the r' and e
    //    of step 1; each slot then holds the state entering its level
    {
      // (each slot's r' and e are read a level ahead of their use; slot n - 1
      // found by a compile-time loop: the register tape takes no runtime index)
      cd rpn = mk(0.0, 0.0), en = mk(0.0, 0.0);
#pragma unroll
      for (int t = 0; t < CHT; ++t) {
        if (t == n - 1) {
          rpn = mk(TP(t, 0), TP(t, 1));
          en = mk(TP(t, 2), TP(t, 3));
        }
      }
#pragma unroll
      for (int t = CHT - 1; t >= 0; --t) {
        if (t < n) {
          const cd rp = rpn;
          const cd e = en;
          if (t >= 1) {
            rpn = mk(TP(t - 1, 0), TP(t - 1, 1));
            en = mk(TP(t - 1, 2), TP(t - 1, 3));
          }
          TP(t, 0) = Pv.re;
          TP(t, 1) = Pv.im;
          TP(t, 2) = Qv.re;
          TP(t, 3) = Qv.im;
          const cd Pn = cmul_add(rp, Qv, Pv);
          Qv = e * cmul_add(rp, Pv, Qv);  // e = 1 at level 0
          Pv = Pn;
        }
      }
    }
    // the cotangent of the state leaving the chunk, conj(Lambda (-Q, P)) rbar
    cd Pb = -cmulc(Qv, mu), Qb = cmulc(Pv, mu);
    cd Qo = Qv;  // second component of the state leaving the level
    // records a level ahead: ri of level jj, rm of medium jj + 1
    ScanRec ri = R.at(0), rm = R.at(1);
    Medium c = med(gl == 0, ri);
    cd kzbc = mk(0.0, 0.0);
#pragma unroll
    for (int t = 0; t < CHT; ++t) {
      if (t < n) {
        const ScanRec rnext = R.at(t + 2);
        const Medium mn = med(false, rm);
        const LevelRecords::Rec rec = full_rec(ri);
        const ScanLevel lv = scan_level<ABOVE>(s.tab, rec, c, mn, rm.B);
        ri = rm;
        rm = rnext;
        const cd Ps = mk(TP(t, 0), TP(t, 1));
        const cd Qs = mk(TP(t, 2), TP(t, 3));
        const cd tb = cmulc(lv.e, Qb);
        const cd wp = cmulc(Qo, Qb);
        const cd rpb = cmulc_add(Ps, tb, cmulc(Qs, Pb));
        const cd Pi = cmulc_add(lv.rp, tb, Pb);
        Qb = cmulc_add(lv.rp, Pb, tb);
        Pb = Pi;
        Qo = Qs;
        const cd ub = cmulc(lv.rp, rpb);
        const cd Xc = rec.C * ub;
        const cd Y = cmulc(lv.g, rpb);
        const cd Zc = mk(fma(2.0, Y.re, Xc.re), fma(2.0, Y.im, Xc.im));
        const cd Zn = mk(fma(-2.0, Y.re, Xc.re), fma(-2.0, Y.im, Xc.im));
        {
          double hs = AC(t + 1, 3);
          acc_re_dot(hs, ub, lv.kk);
          AC(t + 1, 3) = hs;
        }
        kzbc = cmulc_add(mn.kz, Zc, kzbc);
        kzbc.re = fma(-rec.D, wp.im, kzbc.re);
        kzbc.im = fma(rec.D, wp.re, kzbc.im);
        {
          // (the fronting's slots are not read: the reduction takes neither
          // its thickness nor its wavevector)
          double hd = AC(t, 2);
          acc_dd(hd, c.kz, wp);
          AC(t, 2) = hd;
          cd hw = mk(AC(t, 0), AC(t, 1));
          acc_wbar(hw, c.kz, c.inv_abs2, kzbc);
          AC(t, 0) = hw.re;
          AC(t, 1) = hw.im;
        }
        kzbc = cmulc(c.kz, Zn);
        c = mn;
        if (t == n - 1) {
          // this lane's part of its lower boundary medium (hi), from level hi - 1
          cd hw = mk(AC(t + 1, 0), AC(t + 1, 1));
          acc_wbar(hw, c.kz, c.inv_abs2, kzbc);
          AC(t + 1, 0) = hw.re;
          AC(t + 1, 1) = hw.im;
        }
      }
    }
  };
  // one loop per form (see k_grad_select)
  for (int k = 0; k < K; ++k)
    if ((above >> k & 1u) == 0) node(k, std::false_type{});
  for (int k = 0; k < K; ++k)
    if ((above >> k & 1u) != 0) node(k, std::true_type{});

  // w_m = 0 exactly: tested only where 1/|w| hit the root's guard
  bool singular = false;
  if (edge >= 1e140)
    for (int k = 0; k < K; ++k) {
      const double kz0sq = kz0_squared((K == 1) ? Q : smear_at(Q, sig, a.rule[k]));
      for (int t = (gl == 0) ? 1 : 0; t <= n; ++t) {
        const ScanRec r = R.at_lane(t);
        singular |= (kz_real_part(kz0sq, r.A) == 0.0) & (r.B == 0.0);
      }
    }

  // ---- the point's likelihood and seed (uniform over the lanes) ----
  const int NR = N + 2;
  const double sc = a.scale[item];
  const double Rhat = sc * Rsm + a.bkg[item];
  uint32_t bits = 0;
  double ll, ghat;
  if (a.seed != nullptr) {
    ghat = a.seed[a.out_off[item] + i];
    ll = badq ? __builtin_nan("") : ghat * Rhat;
    if (badq) bits |= kItemBadQ;
    if (!isfinite(ll)) bits |= kItemNonfinite;
  } else {
    const double e = a.r_err[qoff + i];
    ll = point_loglik(Rhat, a.r_obs[qoff + i], e, badq, bits);
    ghat = -(Rhat - a.r_obs[qoff + i]) / (e * e);
  }
  const double fac = ghat * sc;
  const double fw = kHwScale * fac, fd = kHdScale * fac;
  if (__ballot(singular) != 0) bits |= kItemEdgeSingular;
  if (lane == 0) flag(a.item_status, item, bits);

  // ---- the record: boundary slots join the next lane's first medium ----
  double* rec = a.rec + a.wu_rec[w];
  double bnd[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int t = 1; t <= CHT; ++t)
    if (t == n)
#pragma unroll
      for (int f = 0; f < 4; ++f) bnd[f] = AC(t, f);
  double from_above[4];
#pragma unroll
  for (int f = 0; f < 4; ++f) from_above[f] = __shfl(bnd[f], lane > 0 ? lane - 1 : 0, 64);
  if constexpr (NW > 1) {
    if (lane == 63)
#pragma unroll
      for (int f = 0; f < 4; ++f) xb[wv][f] = bnd[f];
    __syncthreads();
    if (lane == 0 && wv > 0)
#pragma unroll
      for (int f = 0; f < 4; ++f) from_above[f] = xb[wv - 1][f];
  }
#pragma unroll
  for (int f = 0; f < 4; ++f)
    if (own && gl > 0) AC(0, f) += from_above[f];
  if (own) {
#pragma unroll
    for (int t = 0; t < CHT; ++t) {
      if (t < n) {
        const int m = lo + t;
        rec[3 + m] = fw * AC(t, 0);
        rec[3 + NR + m] = fw * AC(t, 1);
        rec[3 + 2 * NR + m] = fd * AC(t, 2);
        rec[3 + 3 * NR + m] = fac * AC(t, 3);
      }
    }
    if (hi == NL) {  // the backing medium N + 1
      rec[3 + NL] = fw * bnd[0];
      rec[3 + NR + NL] = fw * bnd[1];
      rec[3 + 2 * NR + NL] = fd * bnd[2];
      rec[3 + 3 * NR + NL] = fac * bnd[3];
    }
  }
  if (gl == 0) {
    rec[0] = ll;
    rec[1] = ghat * Rsm;
    rec[2] = ghat;
  }
}

template <int CHT, int NW>
static void launch_cht(const KernelArgs& a, int n_wu, hipStream_t st) {
  hipLaunchKernelGGL((k_grad_scan_select<CHT, NW>), dim3(n_wu), dim3(64 * NW), 0, st, a);
}

hipError_t launch_grad_scan_select(int ch_max, const KernelArgs& a, int n_wu, hipStream_t st) {
  if (n_wu <= 0) return hipSuccess;
  if (ch_max < 1 || ch_max > kScanMaxChunk) return hipErrorInvalidValue;
  switch (scan_nw(ch_max) * 100 + scan_cht(ch_max)) {
    case 101: launch_cht<1, 1>(a, n_wu, st); break;
    case 102: launch_cht<2, 1>(a, n_wu, st); break;
    case 104: launch_cht<4, 1>(a, n_wu, st); break;
    case 108: launch_cht<8, 1>(a, n_wu, st); break;
    case 208: launch_cht<8, 2>(a, n_wu, st); break;
    case 408: launch_cht<8, 4>(a, n_wu, st); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace nr
