// Value kernels (nr_reflectivity, nr_loglik): R_hat per point, or logL partials
// per work unit.  Runtime layer loops, so one kernel serves every depth and
// the units of all items form one launch, longest first.
#pragma once

#include "nr_kernels.hpp"
#include "nr_select.hpp"

namespace nr {

// ---------------------------------------------------------------------------
// R of one node (no state kept): the FP32 variant.
// ---------------------------------------------------------------------------
template <class P>
__device__ __forceinline__ double node_reflectivity(const MathTables& T, const Layers<P>& L, int N,
                                                    double q) {
  using Re = typename P::real;
  using Cx = cx<Re>;
  const double kz0sq = kz0_squared(q);
  Cx kzn = medium_root(L, kz0sq, N + 1).kz;
  Cx Pv = mk(Re(1), Re(0)), Qv = mk(Re(0), Re(0));
  for (int jj = N; jj >= 1; --jj) {
    const Cx kzc = medium_root(L, kz0sq, jj).kz;
    const Iface<Re> it = interface_coeffs(T, kzc, kzn, L.Nr(jj), L.Ni(jj), L.C(jj));
    const Cx Pn = cmul_add(it.rp, Qv, Pv);
    const Cx t = cmul_add(it.rp, Pv, Qv);
    Qv = layer_phase(T, kzc, L.D(jj)) * t;
    Pv = Pn;
    kzn = kzc;
  }
  {
    const Iface<Re> it = interface_coeffs(T, fronting_kz<P>(q), kzn, L.Nr(0), L.Ni(0), L.C(0));
    const Cx Pn = cmul_add(it.rp, Qv, Pv);
    Qv = cmul_add(it.rp, Pv, Qv);
    Pv = Pn;
  }
  return (double)cabs2(Qv * crecip(Pv));
}

// The same in FP64, in the node form that the caller tested (nr_select.hpp).
// Bound by the FP64 VALU like the gradient kernels: at 10 layers 129 VALU
// instructions per level and node, 3.1 of them transcendental, where every node is
// general, 105 and 2.1 where every node is above (778 and 644 us for 2048 items x
// 448 points under the counters).  4096 draws x 10 layers x 400
// points: 1.40 ms with one kernel per depth bucket and whole waves for partial
// groups, 1.15 with these units and node forms, 1.09 with levels in pairs (no
// register moves from one level to the next); four waves per SIMD (100 VGPRs)
// run 1-3 % faster than five or six.  1024 ragged items: 1.89 -> 0.79 ms, the
// sixteen launches of under one round each being one.
template <bool ABOVE>
__device__ __forceinline__ double node_value(const MathTables& T, const LevelRecords& L, int N,
                                             double q) {
  const double kz0sq = kz0_squared(q);
  cd Pv = mk(1.0, 0.0), Qv = mk(0.0, 0.0);
  struct Below {
    Medium me;
    double B;
  };
  // one level: below its upper interface b, above it the medium returned
  auto level = [&](int jj, const Below& b) {
    const LevelRecords::Rec r = L.of(jj);
    Below c;
    c.B = r.B;
    c.me = medium<ABOVE>(kz0sq, r.A, r.B);
    const PhasePart<ABOVE> ep = phase_issue<ABOVE>(T, r, c.me.kz);
    const cd kk = c.me.kz * b.me.kz;
    const RoughPart<ABOVE> fp = rough_issue<ABOVE>(T, r, kk);
    const cd s2 = inv_sum_sq(c.me.x, b.me.x, r.B, b.B, kk);
    const cd rp = mk(r.Nr, r.Ni) * (s2 * rough_finish<ABOVE>(fp));
    const cd Pn = cmul_add(rp, Qv, Pv);
    const cd t = cmul_add(rp, Pv, Qv);
    Qv = phase_finish<ABOVE>(ep) * t;
    Pv = Pn;
    return c;
  };
  Below b;
  {
    const LevelRecords::Rec r = L.of(N + 1);
    b.me = medium<ABOVE>(kz0sq, r.A, r.B);
    b.B = r.B;
  }
  int jj = N;
  for (; jj >= 2; jj -= 2) b = level(jj - 1, level(jj, b));
  if (jj == 1) b = level(1, b);
  {
    const LevelRecords::Rec r = L.of(0);
    const double k0 = 0.5 * q;
    const cd kk = mk(k0 * b.me.kz.re, k0 * b.me.kz.im);
    const cd s2 = inv_sum_sq(kz0sq, b.me.x, 0.0, b.B, kk);
    const cd rp = mk(r.Nr, r.Ni) * (s2 * rough_finish<ABOVE>(rough_issue<ABOVE>(T, r, kk)));
    const cd Pn = cmul_add(rp, Qv, Pv);
    Qv = cmul_add(rp, Pv, Qv);
    Pv = Pn;
  }
  return cabs2(Qv * crecip(Pv));
}

// Touches the item's record lines, one per lane and all in flight at once: the
// sweep's first reads would each wait for a line that the constants kernel left
// in another die's cache.  (The gradient kernels do not take it: 1400 split units
// of 10 layers 153 -> 161 us, 2000 of 26 layers in FP32 529 -> 595.)
__device__ __forceinline__ void warm_records(const KernelArgs& a, int64_t roff, int N, int lane) {
  const int n = (N + 2) * (lane < 32 ? kRecDoubles : kExtDoubles);
  const double* r = lane < 32 ? a.consts + roff * kRecDoubles
                              : reinterpret_cast<const double*>(a.constsf) + roff * kExtDoubles;
  const int i = (lane & 31) * 8;
  const double x = r[i < n ? i : n - 1];
  asm volatile("" ::"v"(x));
}

// A unit holds npts points of one item; lane g npts + p evaluates point p on
// the nodes g, g + G, g + 2G, ... (split_setup; G = 1: 64 points, all nodes),
// and the point's G lanes add their partial sums.  OP: kOpReflectivity writes
// R_hat, kOpLoglik one logL partial per unit.
// FEW: launches of so few waves that each waits for its own record loads.  FP64,
// up to two waves per SIMD: the item's record lines are touched first (589 units
// of 12 layers 18.5 -> 16.1 us a call, 528 of 18 layers 23.6 -> 21.8).  FP32, up to
// one: nodes counted per lane, whose record loads are vector loads and run ahead
// (45 units of 64 points in 17 groups, 20 layers 20.1 -> 18.2 us, 40 layers 28.5 ->
// 26.0).  Of many waves the others cover the wait, and either costs more: 4096
// items of 10 layers FP64 1040 -> 1092 us, 64 units of 20 layers in 17 groups FP32
// 20.1 -> 20.4, 700 in 9 groups 52.8 -> 56.5.
// SPLIT: whether any unit of the launch has node groups.  Without, the divisions
// of split_setup go and the counter is uniform anyway (28000 units of one node and
// one layer FP64 41.7 -> 38.0 us a call).
// FORMS (FP64): the node forms of nr_select.hpp, or the one form on plain records
// (28000 units of one node and one layer 38.3 -> 33.9 us a call; the rule in
// nr_plan_create_ex).
template <class P, int OP, bool SPLIT, bool FEW, bool FORMS>
__global__ __launch_bounds__(64) void k_value(KernelArgs a) {
  __shared__ Shared s;
  const int lane = threadIdx.x;
  const int w = blockIdx.x;
  SplitInfo sp{0, 1, 64};
  const WuInfo u = SPLIT ? split_setup(a, w, lane, sp) : wu_setup(a, w, lane);
  if constexpr (FEW && FORMS) warm_records(a, u.roff, u.N, lane);
  stage_shared(s, lane, a.rule);
  const int K = u.smeared ? kSmearNodes : 1;
  bool badq = !(u.Q > 0.0);
  double Rsm = 0.0;
  for (int k0 = 0; k0 < K; k0 += sp.G) {
    const int k = k0 + sp.g;
    if (SPLIT && !(u.active && k < K)) continue;
    const double q = (K == 1) ? u.Q : smear_at(u.Q, u.sig, ld(s.t[k]));
    badq |= !(q > 0.0);
    const double wk = (K == 1) ? 1.0 : ld(s.w[k]);
    double R;
    if constexpr (FORMS) {
      // (the counter is the wave's: the records stay scalar loads)
      const LevelRecords L = level_records(a, u.roff, u.N, k0);
      const double kz0sq = kz0_squared(q);
      const bool out = !((kz0sq >= L.ext[0]) & (kz0sq <= L.ext[1]) & (q > 0.0));
      R = __ballot(out) == 0 ? node_value<true>(s.tab, L, u.N, q)
                             : node_value<false>(s.tab, L, u.N, q);
    } else {
      R = node_reflectivity(s.tab, item_layers<P>(a, u.roff, u.N, SPLIT && FEW ? k : k0), u.N,
                            q);
    }
    Rsm += wk * R;
  }
  if (SPLIT && sp.G > 1) {
    double tot = 0.0;
    int bq = 0;
    for (int gg = 0; gg < sp.G; ++gg) {
      const int src = gg * sp.npts + lane % sp.npts;
      tot += __shfl(Rsm, src, 64);
      bq |= __shfl(badq ? 1 : 0, src, 64);
    }
    Rsm = tot;
    badq = bq != 0;
  }
  const bool mine = u.active && sp.g == 0;
  if constexpr (OP == kOpReflectivity) {
    if (!mine) return;
    double Rhat = a.scale[u.item] * Rsm + a.bkg[u.item];
    uint32_t bits = 0;
    if (badq) {
      Rhat = __builtin_nan("");
      bits |= kItemBadQ;
    }
    if (!isfinite(Rhat)) bits |= kItemNonfinite;
    flag(a.item_status, u.item, bits);
    a.out[a.out_off[u.item] + u.i] = Rhat;
  } else {
    double ll = 0.0;
    uint32_t bits = 0;
    if (mine) {
      const double Rhat = a.scale[u.item] * Rsm + a.bkg[u.item];
      ll = point_loglik(Rhat, a.r_obs[u.qoff + u.i], a.r_err[u.qoff + u.i], badq, bits);
    }
    flag(a.item_status, u.item, bits);
    ll = wave_sum(ll);
    if (lane == 0) a.rec[a.wu_rec[w]] = ll;
  }
}

template <class P, int OP>
static void launch_value_op(bool split, bool few, bool forms, const KernelArgs& a, int n_wu,
                            hipStream_t st) {
  constexpr bool kF64 = std::is_same<P, F64>::value;
  if (kF64 && !forms)
    hipLaunchKernelGGL((k_value<P, OP, false, false, false>), dim3(n_wu), dim3(64), 0, st, a);
  else if (split && few)
    hipLaunchKernelGGL((k_value<P, OP, true, true, kF64>), dim3(n_wu), dim3(64), 0, st, a);
  else if (split)
    hipLaunchKernelGGL((k_value<P, OP, true, false, kF64>), dim3(n_wu), dim3(64), 0, st, a);
  else if (kF64 && few)
    hipLaunchKernelGGL((k_value<P, OP, false, kF64, kF64>), dim3(n_wu), dim3(64), 0, st, a);
  else
    hipLaunchKernelGGL((k_value<P, OP, false, false, kF64>), dim3(n_wu), dim3(64), 0, st, a);
}

// (forms: FP64, the scaled constants were made; without them no unit is split)
template <class P>
hipError_t launch_value(int op, bool split, bool forms, const KernelArgs& a, int n_wu,
                        hipStream_t st) {
  if (n_wu <= 0) return hipSuccess;
  const bool few = n_wu <= (std::is_same<P, F64>::value ? 2048 : 1024);
  if (op == kOpReflectivity)
    launch_value_op<P, kOpReflectivity>(split, few, forms, a, n_wu, st);
  else
    launch_value_op<P, kOpLoglik>(split, few, forms, a, n_wu, st);
  return hipGetLastError();
}

}  // namespace nr
