// Device code shared by the forward passes that start an operator product:
// the Krylov update fused into them.
#pragma once

#include "fft_common.h"
#include "kernels.h"

namespace vie {

__device__ __forceinline__ c64 kcdiv(c64 a, c64 b) {
  const double d = b.re * b.re + b.im * b.im;
  return mk((a.re * b.re + a.im * b.im) / d, (a.im * b.re - a.re * b.im) / d);
}
__device__ __forceinline__ double kcabs2(c64 a) { return a.re * a.re + a.im * a.im; }

// Sum of n pairs of partials, to every thread, in the order of a 256-thread
// workgroup (thread t takes pairs t, t + 256, ...; a butterfly per 64 threads;
// the four wave sums in order) whatever the workgroup's size NT, so that every
// kernel that folds the same partials gets the same bits.  red: 16 doubles of
// LDS, free on entry; ends with a barrier after the last read of it.
template <int NT>
__device__ __forceinline__ void fold_pairs(const c64* __restrict__ part, int n, double* red,
                                           c64& a, c64& b) {
  constexpr int V = 256 / (NT < 256 ? NT : 256);  // virtual threads per thread
#pragma unroll
  for (int v = 0; v < V; ++v) {
    const int t = threadIdx.x + v * NT;
    if (t >= 256) break;  // whole waves
    c64 s0 = mk(0.0, 0.0), s1 = mk(0.0, 0.0);
    for (int k = t; k < n; k += 256) {
      s0 = s0 + part[2 * k];
      s1 = s1 + part[2 * k + 1];
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) {
      s0.re += __shfl_xor(s0.re, m, 64);
      s0.im += __shfl_xor(s0.im, m, 64);
      s1.re += __shfl_xor(s1.re, m, 64);
      s1.im += __shfl_xor(s1.im, m, 64);
    }
    if ((t & 63) == 0) {
      double* r = red + (t >> 6) * 4;
      r[0] = s0.re;
      r[1] = s0.im;
      r[2] = s1.re;
      r[3] = s1.im;
    }
  }
  __syncthreads();
  a = b = mk(0.0, 0.0);
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    a = a + mk(red[4 * w], red[4 * w + 1]);
    b = b + mk(red[4 * w + 2], red[4 * w + 3]);
  }
  __syncthreads();
}

// The decision that ends or continues a cycle after a residual update, on a =
// (rhat, r) and b = |r|^2: 0 continue, else stop with `breakdown` (0: target
// or iteration cap reached).
__device__ __forceinline__ int rho_decision(c64 a, double rr, c64 omega, int iters,
                                            double target2, int max_iter, int& breakdown) {
  breakdown = 0;
  if (!(rr <= 1e300)) {  // NaN / overflow: end the cycle, restart from x
    breakdown = 4;
    return 1;
  }
  if (rr <= target2 || iters >= max_iter) return 1;
  if (kcabs2(a) == 0.0 || kcabs2(omega) == 0.0) {
    breakdown = kcabs2(omega) == 0.0 ? 3 : 2;  // omega = 0 / rhat . r vanished
    return 1;
  }
  return 0;
}

// Scalars of the fused update of right-hand side rhs.  With u.npart the
// workgroup folds the partials itself (and, as `lead`, records the outcome);
// otherwise they are in the state.  Returns false when the right-hand side
// stopped.  The state's fields written here are not read here; the activity
// flag is, before (group_flag), and every workgroup comes to the same decision.
struct UpdScal {
  c64 beta, om, al;
  bool first;
};
template <int NT>
__device__ __forceinline__ bool upd_scalars(const UpdArgs& u, int rhs, bool lead, double* red,
                                            UpdScal& s) {
  KState& S = u.st[rhs];
  s.first = S.it_cycle == 0;
  if (u.mode == UPD_P) {
    s.om = S.omega;
    if (s.first) {  // p = r
      s.beta = mk(0.0, 0.0);
      return true;
    }
    if (!u.npart) {
      s.beta = S.beta;
      return true;
    }
    const c64 rho = S.rho, al = S.alpha;
    const int iters = S.iters;
    const double target2 = S.target2;
    c64 a, b;
    fold_pairs<NT>(u.part + (int64_t)rhs * u.npart * 2, u.npart, red, a, b);
    int bd;
    const int stop = rho_decision(a, b.re, s.om, iters, target2, u.max_iter, bd);
    if (lead && threadIdx.x == 0) {
      S.rho1 = a;
      S.rnorm2 = b.re;
      if (stop) {
        if (bd) S.breakdown = bd;
        S.active = 0;
        u.flags[rhs] = 0;
        u.flags[2 * u.nrhs + rhs] = 1;
      }
    }
    if (stop) return false;
    s.beta = kcdiv(a, rho) * kcdiv(al, s.om);
    return true;
  }
  if (!u.npart) {
    s.al = S.alpha;
    return true;
  }
  const c64 rho1 = S.rho1;
  c64 a, b;
  fold_pairs<NT>(u.part + (int64_t)rhs * u.npart * 2, u.npart, red, a, b);
  // only an exact zero (or overflow) is a breakdown, see k_finalize
  const bool stop = kcabs2(a) == 0.0 || !(kcabs2(a) < 1e300);
  s.al = stop ? mk(0.0, 0.0) : kcdiv(rho1, a);
  if (lead && threadIdx.x == 0) {
    if (stop) {
      S.breakdown = 1;  // rhat . A p vanished
      S.active = 0;
      u.flags[rhs] = 0;
      u.flags[2 * u.nrhs + rhs] = 1;
    } else {
      S.alpha = s.al;
    }
  }
  return !stop;
}

// The updated vector's element k (offset of the right-hand side included):
// p = r + beta (p - omega v), p = r at the start of a cycle; s = r - alpha v.
__device__ __forceinline__ c64 upd_value(const UpdArgs& u, const UpdScal& s, c64 r, c64 p, c64 v) {
  if (u.mode == UPD_P) return s.first ? r : r + s.beta * (p - s.om * v);
  return r - s.al * v;
}

}  // namespace vie
