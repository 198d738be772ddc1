// What the two scan kernels for deep stacks share (nr_kernels_scan.hip,
// nr_scan_select.hip): 2x2 complex matrices, the per-lane tape, the launch
// configurations.
#pragma once

#include "nr_kernels.hpp"

namespace nr {

struct M2 {
  cd a, b, c, d;  // [[a, b], [c, d]]
};

__device__ __forceinline__ M2 m2_mul(const M2& x, const M2& y) {
  M2 z;
  z.a = x.a * y.a + x.b * y.c;
  z.b = x.a * y.b + x.b * y.d;
  z.c = x.c * y.a + x.d * y.c;
  z.d = x.c * y.b + x.d * y.d;
  return z;
}

__device__ __forceinline__ M2 m2_identity() {
  M2 z;
  z.a = mk(1.0, 0.0);
  z.b = mk(0.0, 0.0);
  z.c = mk(0.0, 0.0);
  z.d = mk(1.0, 0.0);
  return z;
}

__device__ __forceinline__ cd shfl_cd(cd v, int src) {
  return mk(__shfl(v.re, src, 64), __shfl(v.im, src, 64));
}

__device__ __forceinline__ M2 shfl_m2(const M2& m, int src) {
  M2 z;
  z.a = shfl_cd(m.a, src);
  z.b = shfl_cd(m.b, src);
  z.c = shfl_cd(m.c, src);
  z.d = shfl_cd(m.d, src);
  return z;
}

__device__ __forceinline__ M2 load_m2(const cd* x) {
  M2 z;
  z.a = x[0];
  z.b = x[1];
  z.c = x[2];
  z.d = x[3];
  return z;
}

// Per-lane storage of the state tape (the state entering each of the lane's
// levels; between steps 1 and 3, the level's r' and e) and of the
// accumulators (Hw re, Hw im, Hd, Hs per medium slot; slot t is medium lo + t,
// slot n = hi - lo the lane's lower boundary medium): registers, or LDS in
// planes interleaved over the NT lanes of a data point.
template <int CHT, bool IN_LDS, int NT>
struct LaneTape {
  double r[IN_LDS ? 1 : CHT][4];
  __device__ __forceinline__ double& at(double* lds, int gl, int t, int f) {
    if constexpr (IN_LDS)
      return lds[(t * 4 + f) * NT + gl];
    else
      return r[t][f];
  }
};

// (the constants kernel lays deep items' records out by the same rule)
// The configuration of a launch whose deepest item needs ch64 levels per
// lane at 64 lanes: one wave per data point up to 8 levels per lane, else two
// or four waves, so that no lane holds more than 8 levels (the tape then fits
// 2 KB of LDS per level and wave, and the kernel two waves per SIMD); the
// levels per lane round up to a power of two.
inline int scan_nw(int ch64) { return ch64 <= 8 ? 1 : ch64 <= 16 ? 2 : 4; }

inline int scan_cht(int ch64) {
  const int nw = scan_nw(ch64);
  const int ch = (ch64 + nw - 1) / nw;
  int c = 1;
  while (c < ch) c <<= 1;
  return c;
}

}  // namespace nr
