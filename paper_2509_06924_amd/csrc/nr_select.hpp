// FP64 gradient kernels that choose, node by node, between two forms of the
// layer product and its adjoint:
//
//   above    every medium propagates well above its critical edge and absorbs
//            little (the item's range of kz0^2 from k_item_consts, tested over
//            the wave): each wavevector is real up to a small imaginary part.
//            Its root takes one reciprocal square root instead of two, the
//            phase exp(-2 i kz d) is a sine and cosine times an exponential
//            of a small argument, the Nevot-Croce factor an exponential times
//            the sine and cosine of a small argument: short polynomials stand
//            in for half of the table-driven functions, with no clamps.
//   general  any stack at any q.
//
// Both give the function to rounding; the choice follows from the values of a
// node alone.  What bounds these kernels is the FP64 VALU: it is active for 0.47
// of each wave's cycles at two waves per SIMD (10 layers), and v_rsq_f64 and
// v_rcp_f64 hold it for four instructions (16 cycles measured on MI355X at one to
// eight waves per SIMD, against 4 for an FMA).  So the forms differ in instructions
// per level: at 10 layers, epilogue and all, 244 VALU instructions per level and
// node where every node is general and 214 where every node is above, 5.4 and 3.4
// of them transcendental, against 254 and 5.4 in k_loglik_grad (counters of 2048
// items x 448 points at q below 0.009 and above 0.25, 1580 and 1430 us).
//
// Measured on MI355X against k_loglik_grad (2048 draws x 448 points, 5 %
// dQ/Q, about 0.6 of the nodes above; one box, us):
//   layers   6     8     10    12    14    16    18    20    24    28    32    36
//   before   790   1033  1340  1680  1987  2381  2666  3061  3790  4567  5416  6625
//   after    724   946   1238  1531  1886  2196  2509  2865  3528  4246  5075  6373
// 4096 draws x 10 layers x 400 points 2.42 -> 2.25 ms.  The two bodies (100 KB
// and more from 24 layers on) crowd the instruction cache that two compute
// units share, so units in flight together should run the same form: ordered
// by their place in the data set instead of item by item, 16-20 layers gained
// 4-5 %.  40 layers run 10 % slower (464 B of spill beside 200 KB of
// code).  Packed tail units spilled up to 1 KB here and stay with
// k_loglik_grad, and so do the resolution form and FP32 (whose exponentials
// are hardware functions).
#pragma once

#include "nr_kernels.hpp"

namespace nr {

// The records of one item.  Beside the six doubles of Layers (A, B, Nr, Ni, C,
// D) four per row in the second array:
//   pd = D 64/pi, ld = D 64/ln 2, pc = C 64/pi, lc = C 64/ln 2
// (the factors of sincos_issue_scaled and exp_issue_scaled).  The fronting
// medium has no phase; its pd and ld hold the item's range [lo, hi] of kz0^2
// for the above form.
struct LevelRecords {
  const double* rec;
  const double* ext;
  int z;   // an opaque zero (see Layers)
  int nb;  // the backing medium, N + 1
  struct Rec {
    double A, B, Nr, Ni, C, D, pd, ld, pc, lc;
  };
  __device__ __forceinline__ Rec of(int m) const {
    const int i = (m < nb ? m : nb) + z;
    const double* r = rec + i * kRecDoubles;
    const double* x = ext + i * kExtDoubles;
    Rec o;
    o.A = r[0];
    o.B = r[1];
    o.Nr = r[2];
    o.Ni = r[3];
    o.C = r[4];
    o.D = r[5];
    o.pd = x[0];
    o.ld = x[1];
    o.pc = x[2];
    o.lc = x[3];
    return o;
  }
};

__device__ __forceinline__ LevelRecords level_records(const KernelArgs& a, int64_t roff, int N,
                                                      int k) {
  LevelRecords L;
  L.rec = a.consts + roff * kRecDoubles;
  L.ext = reinterpret_cast<const double*>(a.constsf) + roff * kExtDoubles;
  L.z = k & a.zero_mask;
  L.nb = N + 1;
  return L;
}

// A medium at one node: kz, the real part x of w = x - i B, 1/|w|.
struct Medium {
  cd kz;
  double x, inv_abs2;
};
template <bool ABOVE>
__device__ __forceinline__ Medium medium(double kz0sq, double A, double B) {
  Medium o;
  o.x = kz_real_part(kz0sq, A);
  const Root r = ABOVE ? kz_root_above(o.x, B) : kz_root(o.x, -B);
  o.kz = r.kz;
  o.inv_abs2 = r.inv_abs2;
  return o;
}

// s^2 = 1/(kz_c + kz_n)^2 from (kz_c + kz_n)^2 = w_c + w_n + 2 kz_c kz_n.
// No cancellation: both wavevectors lie in one quadrant, so the modulus is at
// least |w_c| + |w_n|.
__device__ __forceinline__ cd inv_sum_sq(double xc, double xn, double Bc, double Bn, cd kk) {
  const double re = fma(2.0, kk.re, xc + xn);
  const double im = fma(2.0, kk.im, -Bc) - Bn;
  const double inv = rcp(fma(re, re, im * im));
  return mk(re * inv, -im * inv);
}

// exp(C kk) and exp(-2 i kz d) in halves (reads issued, then combined).
template <bool ABOVE>
struct RoughPart;
template <>
struct RoughPart<true> {
  ExpPart ex;
  double sn, cs;
};
template <>
struct RoughPart<false> {
  ExpPart ex;
  SinCosPart sc;
};
template <bool ABOVE>
struct PhasePart;
template <>
struct PhasePart<true> {
  SinCosPart sc;
  double e;
};
template <>
struct PhasePart<false> {
  SinCosPart sc;
  ExpPart ex;
};
template <bool ABOVE>
__device__ __forceinline__ RoughPart<ABOVE> rough_issue(const MathTables& T,
                                                        const LevelRecords::Rec& r, cd kk) {
  RoughPart<ABOVE> o;
  if constexpr (ABOVE) {
    o.ex = exp_issue_bounded(T, r.lc, kk.re);
    sincos_small(r.C * kk.im, &o.sn, &o.cs);
  } else {
    o.ex = exp_issue_scaled(T, r.lc, kk.re);
    o.sc = sincos_issue_scaled(T, r.pc, kk.im);
  }
  return o;
}
template <bool ABOVE>
__device__ __forceinline__ cd rough_finish(const RoughPart<ABOVE>& p) {
  const double e = exp_finish(p.ex);
  if constexpr (ABOVE) {
    return mk(e * p.cs, e * p.sn);
  } else {
    double s, c;
    sincos_finish(p.sc, &s, &c);
    return mk(e * c, e * s);
  }
}
template <bool ABOVE>
__device__ __forceinline__ PhasePart<ABOVE> phase_issue(const MathTables& T,
                                                        const LevelRecords::Rec& r, cd kz) {
  PhasePart<ABOVE> o;
  o.sc = sincos_issue_scaled(T, r.pd, -kz.re);
  if constexpr (ABOVE)
    o.e = exp_small(r.D * kz.im);
  else
    o.ex = exp_issue_scaled(T, r.ld, kz.im);
  return o;
}
template <bool ABOVE>
__device__ __forceinline__ cd phase_finish(const PhasePart<ABOVE>& p) {
  double s, c;
  sincos_finish(p.sc, &s, &c);
  double e;
  if constexpr (ABOVE)
    e = p.e;
  else
    e = exp_finish(p.ex);
  return mk(e * c, e * s);
}

// ---------------------------------------------------------------------------
// One node: forward sweep, adjoint, w_k dR/d(.) added to the accumulators;
// returns R(q).  The recompute form of node_grad_recompute (state tape in
// registers, every second level with CK; e and g of KS levels and e of KE more
// in LDS), with PIPE its software pipeline.  Two things are cheaper than
// there: s^2 from w_c + w_n + 2 kk (inv_sum_sq), and the phase cotangent
// w = conj(e) ebar = conj(Q+) Qbar with Q+ = e t the state leaving the level,
// which the tape holds as the state entering the level above.
// ---------------------------------------------------------------------------
template <int LMAX, int KS, int KE, bool CK, bool PIPE, bool ABOVE>
__device__ __forceinline__ double node_grad_select(const MathTables& T, const LevelRecords& L,
                                                   EfCache<double, KS, KE>& ef, Accum<LMAX>& acc,
                                                   int lane, double q, double wk, double& edge) {
  static_assert(!CK || LMAX % 2 == 0, "checkpointed tape needs an even depth");
  using Rec = LevelRecords::Rec;
  const double kz0sq = kz0_squared(q);
  const double k0 = 0.5 * q;
  constexpr int NT = CK ? LMAX / 2 + 1 : LMAX + 1;
  cd tapeP[NT], tapeQ[NT];
  cd Pv = mk(1.0, 0.0), Qv = mk(0.0, 0.0);
  auto kz_prod = [&](int jj, cd kc, cd kn) {
    return jj == 0 ? mk(k0 * kn.re, k0 * kn.im) : kc * kn;
  };

  // ---- forward ----
  struct FwdPre {
    Medium me;  // medium jj
    cd s2;
    RoughPart<ABOVE> f;
    PhasePart<ABOVE> e;
  };
  auto fwd_pre = [&](int jj, const Medium& below, double Bbelow, const Rec& r) {
    FwdPre o;
    if (jj == 0) {
      o.me.kz = mk(k0, 0.0);
      o.me.x = kz0sq;
    } else {
      o.me = medium<ABOVE>(kz0sq, r.A, r.B);
      if constexpr (!ABOVE) edge = fmax(edge, o.me.inv_abs2);
    }
    const cd kk = kz_prod(jj, o.me.kz, below.kz);
    o.s2 = inv_sum_sq(o.me.x, below.x, jj == 0 ? 0.0 : r.B, Bbelow, kk);
    o.f = rough_issue<ABOVE>(T, r, kk);
    if (jj >= 1) o.e = phase_issue<ABOVE>(T, r, o.me.kz);
    return o;
  };
  {
    Rec R[LMAX + 2];
    R[LMAX + 1] = L.of(LMAX + 1);
    R[LMAX] = L.of(LMAX);
    if (PIPE && LMAX >= 1) R[LMAX - 1] = L.of(LMAX - 1);
    Medium below = medium<ABOVE>(kz0sq, R[LMAX + 1].A, R[LMAX + 1].B);
    if constexpr (!ABOVE) edge = fmax(edge, below.inv_abs2);
    FwdPre cur;
    if constexpr (PIPE) cur = fwd_pre(LMAX, below, R[LMAX + 1].B, R[LMAX]);
#pragma unroll
    for (int jj = LMAX; jj >= 0; --jj) {
      FwdPre nxt;
      if constexpr (PIPE) {
        if (jj >= 2) R[jj - 2] = L.of(jj - 2);
        if (jj >= 1) nxt = fwd_pre(jj - 1, cur.me, R[jj].B, R[jj - 1]);
      } else {
        if (jj < LMAX) R[jj] = L.of(jj);
        cur = fwd_pre(jj, below, R[jj + 1].B, R[jj]);
      }
      if (!CK || jj % 2 == 0) {
        tapeP[CK ? jj / 2 : jj] = Pv;
        tapeQ[CK ? jj / 2 : jj] = Qv;
      }
      const cd g = cur.s2 * rough_finish<ABOVE>(cur.f);
      const cd rp = mk(R[jj].Nr, R[jj].Ni) * g;
      const cd Pn = cmul_add(rp, Qv, Pv);
      const cd t = cmul_add(rp, Pv, Qv);
      const cd e = (jj >= 1) ? phase_finish<ABOVE>(cur.e) : mk(1.0, 0.0);
      if (jj < KS) {
        ef.v[jj][0][lane] = e.re;
        ef.v[jj][1][lane] = e.im;
        ef.v[jj][2][lane] = g.re;
        ef.v[jj][3][lane] = g.im;
      } else if (jj < KS + KE) {
        ef.put_e_extra(jj, lane, e);
      }
      Qv = (jj >= 1) ? e * t : t;
      Pv = Pn;
      if constexpr (PIPE) {
        if (jj >= 1) cur = nxt;
        __builtin_amdgcn_sched_barrier(0);
      } else {
        below = cur.me;
        __builtin_amdgcn_sched_barrier(0x0100);  // only LDS reads may move across
      }
    }
  }
  const cd iP = crecip(Pv);
  const cd r = Qv * iP;
  const cd rbar = (2.0 * wk) * r;
  cd Pb = cmulc(-(r * iP), rbar);
  cd Qb = cmulc(iP, rbar);
  cd kzbc = mk(0.0, 0.0);

  // ---- adjoint ----
  struct AdjPre {
    Medium rn;     // medium jj + 1
    cd s2, kk;     // s^2 (below the cache), kz_jj kz_jj+1
    cd gv, ev;     // g (jj < KS) and e (jj < KS + KE) from the LDS cache
    RoughPart<ABOVE> f;
    PhasePart<ABOVE> e;
    double C, D, Nr, Ni;
  };
  // (c: medium jj; ri, rn: the records of media jj and jj + 1)
  auto adj_pre = [&](int jj, const Medium& c, const Rec& ri, const Rec& rn) {
    AdjPre o;
    o.rn = medium<ABOVE>(kz0sq, rn.A, rn.B);
    o.C = ri.C;
    o.D = ri.D;
    o.Nr = ri.Nr;
    o.Ni = ri.Ni;
    o.kk = kz_prod(jj, c.kz, o.rn.kz);
    if (jj < KS) {
      o.gv = mk(ef.v[jj][2][lane], ef.v[jj][3][lane]);
      if (jj >= 1) o.ev = mk(ef.v[jj][0][lane], ef.v[jj][1][lane]);
    } else {
      o.s2 = inv_sum_sq(c.x, o.rn.x, jj == 0 ? 0.0 : ri.B, rn.B, o.kk);
      o.f = rough_issue<ABOVE>(T, ri, o.kk);
      if (jj >= 1) {
        if (jj < KS + KE)
          o.ev = ef.e_extra(jj, lane);
        else
          o.e = phase_issue<ABOVE>(T, ri, c.kz);
      }
    }
    return o;
  };
  struct Lev {
    Medium rn;
    cd kk, g, rp, e;
    double C, D;
  };
  auto adj_level = [&](int jj, const AdjPre& p) {
    Lev o;
    o.rn = p.rn;
    o.kk = p.kk;
    o.C = p.C;
    o.D = p.D;
    if (jj < KS)
      o.g = p.gv;
    else
      o.g = p.s2 * rough_finish<ABOVE>(p.f);
    o.rp = mk(p.Nr, p.Ni) * o.g;
    if (jj < 1)
      o.e = mk(1.0, 0.0);
    else if (jj < KS + KE)
      o.e = p.ev;
    else
      o.e = phase_finish<ABOVE>(p.e);
    return o;
  };
  // the adjoint of level jj (see adjoint_step): (Ps, Qs) enters it, Qo is the
  // second component of the state leaving it
  auto step = [&](int jj, const Lev& lv, cd Ps, cd Qs, cd Qo, const Medium& c) {
    const bool ph = jj >= 1;
    const cd tb = ph ? cmulc(lv.e, Qb) : Qb;
    const cd w = ph ? cmulc(Qo, Qb) : mk(0.0, 0.0);
    const cd rpb = cmulc_add(Ps, tb, cmulc(Qs, Pb));
    const cd Pi = cmulc_add(lv.rp, tb, Pb);
    Qb = cmulc_add(lv.rp, Pb, tb);
    Pb = Pi;
    const cd ub = cmulc(lv.rp, rpb);
    const cd X = lv.C * ub;
    const cd Y = cmulc(lv.g, rpb);
    const cd Zn = mk(fma(-2.0, Y.re, X.re), fma(-2.0, Y.im, X.im));
    acc_re_dot(acc.Hs[jj + 1], ub, lv.kk);
    if (ph) {
      const cd Zc = mk(fma(2.0, Y.re, X.re), fma(2.0, Y.im, X.im));
      kzbc = cmulc_add(lv.rn.kz, Zc, kzbc);
      kzbc.re = fma(-lv.D, w.im, kzbc.re);
      kzbc.im = fma(lv.D, w.re, kzbc.im);
      acc_dd(acc.Hd[jj], c.kz, w);
      acc_wbar(acc.Hw[jj], c.kz, c.inv_abs2, kzbc);
      kzbc = cmulc(c.kz, Zn);
    } else {
      kzbc = k0 * Zn;
    }
    if (jj == LMAX) acc_wbar(acc.Hw[jj + 1], lv.rn.kz, lv.rn.inv_abs2, kzbc);
  };

  Medium c;
  c.kz = mk(k0, 0.0);
  c.x = kz0sq;
  c.inv_abs2 = 0.0;
  // records of media 0 .. LMAX + 1, each loaded a region before its use
  Rec RA[LMAX + 2];
  auto load_rec = [&](int m) {
    if (m <= LMAX + 1) RA[m] = L.of(m);
  };
  constexpr int kAhead = PIPE ? 1 : 0;
  load_rec(0);
  load_rec(1);
  if (PIPE) load_rec(2);
  if constexpr (CK) {
    // level 0, then pairs of levels (jj, jj + 1), jj odd: the state entering
    // level jj is re-formed from the one below
    AdjPre cur = adj_pre(0, c, RA[0], RA[1]);
    {
      load_rec(2 + kAhead);
      AdjPre nxt;
      if (PIPE) nxt = adj_pre(1, cur.rn, RA[1], RA[2]);
      const Lev l0 = adj_level(0, cur);
      step(0, l0, tapeP[0], tapeQ[0], mk(0.0, 0.0), c);
      c = l0.rn;
      if (PIPE) cur = nxt;
    }
    __builtin_amdgcn_sched_barrier(PIPE ? 0 : 0x0100);
#pragma unroll
    for (int jj = 1; jj <= LMAX; jj += 2) {
      if (!PIPE) {
        load_rec(jj + 2);
        cur = adj_pre(jj, c, RA[jj], RA[jj + 1]);
      } else {
        load_rec(jj + 3);
      }
      const AdjPre pb = adj_pre(jj + 1, cur.rn, RA[jj + 1], RA[jj + 2]);
      const Lev la = adj_level(jj, cur);
      if (PIPE) {
        __builtin_amdgcn_sched_barrier(0);
        load_rec(jj + 4);
      } else {
        load_rec(jj + 3);
      }
      AdjPre nxt;
      if (PIPE && jj + 1 < LMAX) nxt = adj_pre(jj + 2, pb.rn, RA[jj + 2], RA[jj + 3]);
      const Lev lb = adj_level(jj + 1, pb);
      const cd P1 = tapeP[(jj + 1) / 2], Q1 = tapeQ[(jj + 1) / 2];
      const cd P0 = cmul_add(lb.rp, Q1, P1);
      const cd Q0 = lb.e * cmul_add(lb.rp, P1, Q1);
      step(jj, la, P0, Q0, tapeQ[(jj - 1) / 2], c);
      step(jj + 1, lb, P1, Q1, Q0, la.rn);
      c = lb.rn;
      if (PIPE && jj + 1 < LMAX) cur = nxt;
      __builtin_amdgcn_sched_barrier(PIPE ? 0 : 0x0100);
    }
  } else {
    AdjPre cur;
    if (PIPE) cur = adj_pre(0, c, RA[0], RA[1]);
#pragma unroll
    for (int jj = 0; jj <= LMAX; ++jj) {
      load_rec(jj + 2 + kAhead);
      AdjPre nxt;
      if (PIPE) {
        if (jj < LMAX) nxt = adj_pre(jj + 1, cur.rn, RA[jj + 1], RA[jj + 2]);
      } else {
        cur = adj_pre(jj, c, RA[jj], RA[jj + 1]);
      }
      const Lev lv = adj_level(jj, cur);
      step(jj, lv, tapeP[jj], tapeQ[jj], jj >= 1 ? tapeQ[jj - 1] : mk(0.0, 0.0), c);
      c = lv.rn;
      if (PIPE && jj < LMAX) cur = nxt;
      __builtin_amdgcn_sched_barrier(PIPE ? 0 : 0x0100);
    }
  }
  return cabs2(r);
}

// ---------------------------------------------------------------------------
// logL + gradient partials per work unit, the records of k_loglik_grad.
// ---------------------------------------------------------------------------
template <int LMAX, bool SPLIT>
__global__ __launch_bounds__(64, F64::min_waves(LMAX, false)) void k_grad_select(KernelArgs a) {
  __shared__ Shared s;
  constexpr int KS = F64::ef_levels(LMAX), KE = F64::e_levels(LMAX);
  constexpr bool CK = F64::checkpoint(LMAX), PIPE = F64::pipelined(LMAX, SPLIT);
  using Ef = EfCache<double, KS, KE>;
  __shared__ Ef efc;
  const int lane = threadIdx.x;
  const int w = blockIdx.x;
  SplitInfo sp{0, 1, 64};
  const WuInfo u = SPLIT ? split_setup(a, w, lane, sp) : wu_setup(a, w, lane);
  stage_shared(s, lane, a.rule);
  const int K = u.smeared ? kSmearNodes : 1;

  Accum<LMAX> acc;
#pragma unroll
  for (int m = 0; m < LMAX + 2; ++m) {
    acc.Hw[m] = mk(0.0, 0.0);
    acc.Hd[m] = 0.0;
    acc.Hs[m] = 0.0;
  }
  double Rsm = 0.0;
  bool badq = !(u.Q > 0.0);
  double edge = 0.0;
  // A split unit's lane takes every G-th node from its group's first; the
  // counter is the wave's, so that the layer records stay scalar loads.
  auto node_q = [&](int k) { return (K == 1) ? u.Q : smear_at(u.Q, u.sig, ld(s.t[k])); };
  // The nodes of each form, then one loop per form: both forms in one loop
  // body share their registers' live ranges and spill hundreds of bytes.
  // (The rule is read from memory here: the LDS reads are volatile, and behind
  // a loop of them the compiler reads the layer records with vector loads.)
  uint32_t above = 0;
  {
    const LevelRecords L = level_records(a, u.roff, u.N, 0);
    const double lo = L.ext[0], hi = L.ext[1];
    for (int k0 = 0; k0 < K; k0 += sp.G) {
      const int k = k0 + sp.g;
      bool out = false;
      if (!SPLIT || (u.active && k < K)) {
        const double q = (K == 1) ? u.Q : smear_at(u.Q, u.sig, a.rule[k]);
        const double kz0sq = kz0_squared(q);
        out = !((kz0sq >= lo) & (kz0sq <= hi) & (q > 0.0));
        badq |= !(q > 0.0);
      }
      if (__ballot(out) == 0) above |= 1u << k0;
    }
  }
#define NR_SELECT_NODES(ABOVE, TODO)                                                          \
  for (int k0 = 0; k0 < K; k0 += sp.G) {                                                      \
    if (((TODO) >> k0 & 1u) == 0) continue;                                                   \
    const int k = k0 + sp.g;                                                                  \
    if (SPLIT && !(u.active && k < K)) continue;                                              \
    const double wk = (K == 1) ? 1.0 : ld(s.w[k]);                                            \
    Rsm += wk * node_grad_select<LMAX, KS, KE, CK, PIPE, ABOVE>(                              \
                    s.tab, level_records(a, u.roff, u.N, k0), efc, acc, lane, node_q(k), wk,  \
                    edge);                                                                    \
  }
  NR_SELECT_NODES(false, ~above)
  NR_SELECT_NODES(true, above)
#undef NR_SELECT_NODES
  // w_m = 0 exactly gives 1/|w_m| = 1e150 (the root's guard): only then are
  // the lane's nodes and media tested one by one
  bool singular = false;
  if (edge >= 1e140) {
    const LevelRecords L = level_records(a, u.roff, u.N, 0);
    for (int k = sp.g; k < K; k += sp.G) {
      const double kz0sq = kz0_squared((K == 1) ? u.Q : smear_at(u.Q, u.sig, a.rule[k]));
      for (int m = 1; m <= u.N + 1; ++m)
        singular |= (kz_real_part(kz0sq, L.rec[m * kRecDoubles]) == 0.0) &
                    (L.rec[m * kRecDoubles + 1] == 0.0);
    }
  }
  // the item was evaluated at depth LMAX: the copies of the backing below it
  // (media N + 2 .. LMAX + 1) are the backing's parameters
  {
    cd back = mk(0.0, 0.0);
#pragma unroll
    for (int m = 1; m < LMAX + 2; ++m)
      if (m >= u.N + 1) back += acc.Hw[m];
#pragma unroll
    for (int m = 1; m < LMAX + 2; ++m)
      if (m == u.N + 1) acc.Hw[m] = back;
  }

  write_grad_record<LMAX, false, SPLIT, false>(a, u, sp, w, lane, acc, Rsm, 0.0, badq, singular,
                                               reinterpret_cast<double*>(&efc));
}

#define NR_SELECT_LAUNCH(LM)                                                           \
  if (mode == kModeSplit)                                                              \
    hipLaunchKernelGGL((k_grad_select<LM, true>), dim3(n_wu), dim3(64), 0, st, a);     \
  else                                                                                 \
    hipLaunchKernelGGL((k_grad_select<LM, false>), dim3(n_wu), dim3(64), 0, st, a);

}  // namespace nr
