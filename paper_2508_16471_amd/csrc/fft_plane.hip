// Fused x and y passes of the operator product for short lines: one workgroup
// per (right-hand side, component, z) plane keeps the plane's x-transformed
// lines in LDS, so the x-y scratch never leaves the CU and a product takes
// three launches (x-y, z, y-x) instead of five.  On the 16^3 grid (FFT 32^3)
// each separate pass is 4 to 5 us of launch and latency with a few hundred
// bytes per thread.  The grids that take it: plane_ok below.
//
// Forward: the x lines of the plane, a batch at a time, are loaded (from a box
// vector, or scattered from a body-compressed one, with the Krylov update of
// that vector fused in), transformed in their own LDS row and left there; then
// the columns, a batch at a time, are transformed along y and written to the y/z
// scratch.  Inverse: the reverse, ending in the product's epilogue and dot
// partials (one pair per plane).
#include "fft_plane.h"

namespace vie {

// Threads: short planes do not fill four waves, and their batch of lines
// would take the LDS of other workgroups.
constexpr int plane_threads(int P1) { return P1 <= 32 ? 128 : 256; }

template <int P, int NT>
struct PlaneLine {
  static constexpr int E = P % 3 == 0 ? 12 : 8, TT = P / E;  // points per thread, threads
  static constexpr int L = NT / TT;                          // lines (columns) per batch
  static constexpr int S = P + P / 16 + 1;                   // padded line
  // a line's threads are neighbouring lanes of one wave
  static_assert(64 % TT == 0, "plane line");
};

template <typename T, int P, bool INV, bool HIN, bool HOUT, int E>
__device__ __forceinline__ void plane_fft(cpx<T> (&v)[E], cpx<T>* line, int t,
                                          const TwReg<T, P, E>& tr) {
  fft_stages_p<T, P, E, 1, INV, 0, HIN, HOUT>(v, LdsLine<T>{line}, t, tr.w);
}

template <typename T, int P2, int NT>
__device__ __forceinline__ void plane_y_fwd(const cpx<T>* plane, int RS, cpx<T>* ubuf,
                                            cpx<T>* __restrict__ out, int64_t row,
                                            const cpx<T>* __restrict__ tw2, int N2, int P1) {
  using Y = PlaneLine<P2, NT>;
  const int cw = threadIdx.x % Y::L, t = threadIdx.x / Y::L;
  TwReg<T, P2, Y::E> tr;
  tr.load(t, tw2);
  for (int p0 = 0; p0 < P1; p0 += Y::L) {
    const int col = p0 + cw;
    const bool valid = col < P1;
    cpx<T> v[Y::E];
#pragma unroll
    for (int q = 0; q < Y::E; ++q) {
      const int r = t + q * Y::TT;
      v[q] = (q < Y::E / 2 && valid && r < N2) ? plane[r * RS + pidx(col)] : mk<T>(0, 0);
    }
    plane_fft<T, P2, false, true, false>(v, ubuf + cw * Y::S, t, tr);
    if (valid) {
#pragma unroll
      for (int q = 0; q < Y::E; ++q) out[(int64_t)(t + q * Y::TT) * row + col] = v[q];
    }
  }
}

template <typename T, int P2, int NT>
__device__ __forceinline__ void plane_y_inv(cpx<T>* plane, int RS, cpx<T>* ubuf,
                                            const cpx<T>* __restrict__ in, int64_t row,
                                            const cpx<T>* __restrict__ tw2, int N2, int P1) {
  using Y = PlaneLine<P2, NT>;
  const int cw = threadIdx.x % Y::L, t = threadIdx.x / Y::L;
  TwReg<T, P2, Y::E> tr;
  tr.load(t, tw2);
  for (int p0 = 0; p0 < P1; p0 += Y::L) {
    const int col = p0 + cw;
    const bool valid = col < P1;
    cpx<T> v[Y::E];
#pragma unroll
    for (int q = 0; q < Y::E; ++q)
      v[q] = valid ? in[(int64_t)(t + q * Y::TT) * row + col] : mk<T>(0, 0);
    plane_fft<T, P2, true, false, true>(v, ubuf + cw * Y::S, t, tr);
    if (valid) {
#pragma unroll
      for (int q = 0; q < Y::E / 2; ++q) {
        const int r = t + q * Y::TT;
        if (r < N2) plane[r * RS + pidx(col)] = v[q];
      }
    }
  }
}

#define VIE_PLANE_Y(P2_, CALL)                       \
  switch (P2_) {                                     \
    case 24: { constexpr int PP = 24; CALL; break; } \
    case 32: { constexpr int PP = 32; CALL; break; } \
    case 48: { constexpr int PP = 48; CALL; break; } \
    default: { constexpr int PP = 64; CALL; break; } \
  }

struct PlaneArgs {
  int N1, N2, N3, P2, nrhs, zl;
  int64_t zhs, zls, cs, rs, row;  // y/z scratch (see StridedArgs)
  int64_t n;                      // voxels of the box
  int ubuf;                       // elements of the plane rows in front of the line buffer
};

template <typename T, int P1, bool COMP, int NT = plane_threads(P1)>
__global__ __launch_bounds__(NT) void k_plane_fwd(
    const c64* __restrict__ x, cpx<T>* __restrict__ B, const cpx<T>* __restrict__ tw1,
    const cpx<T>* __restrict__ tw2, BodyIdx bi, PlaneArgs a, const int* active, UpdArgs u) {
  using X = PlaneLine<P1, NT>;
  extern __shared__ __align__(16) char smem[];
  __shared__ double red[16];
  cpx<T>* plane = reinterpret_cast<cpx<T>*>(smem);
  cpx<T>* ubuf = plane + a.ubuf;
  const int rhs = blockIdx.x % a.nrhs, cz = blockIdx.x / a.nrhs;
  if (active && !group_flag(active + rhs)) return;
  const int comp = cz / a.N3, z = cz % a.N3;
  UpdScal us;
  if (COMP && u.mode != UPD_NONE) {
    if (!upd_scalars<NT>(u, rhs, cz == 0, red, us)) return;
  }
  const int li = threadIdx.x / X::TT, t = threadIdx.x % X::TT;
  TwReg<T, P1, X::E> tr;
  tr.load(t, tw1);
  for (int n = 0; n * X::L < a.N2; ++n) {
    const int y = n * X::L + li;
    const bool valid = y < a.N2;
    // lines past the plane exchange in the (still unused) line buffer
    cpx<T>* line = valid ? plane + y * X::S : ubuf + li * X::S;
    cpx<T> v[X::E];
    if constexpr (COMP) {
      const int body = bi.rhs_body[rhs];
      const int nb = bi.nb[body];
      const int* vox = bi.vox + bi.voff[body];
      const int* lp = bi.line_ptr + (int64_t)body * (a.N2 * a.N3 + 1) + z * a.N2;
      const int64_t vb = bi.roff[rhs] + (int64_t)comp * nb;
#pragma unroll
      for (int q = 0; q < X::E / 2; ++q) line[pidx(t + q * X::TT)] = mk<T>(0, 0);
      lds_barrier();
      if (valid) {
        const int k0 = lp[y] + t, k1 = lp[y + 1], base = (z * a.N2 + y) * a.N1;
        // a line holds at most P1 / 2 voxels: every load before the first use
        int kv[X::E / 2];
        c64 xr[X::E / 2], pr[X::E / 2], vr[X::E / 2];
        const bool upd = u.mode != UPD_NONE, needv = upd && !(u.mode == UPD_P && us.first);
        const c64* src = upd ? u.r : x;
#pragma unroll
        for (int i = 0; i < X::E / 2; ++i) {
          const int k = k0 + i * X::TT;
          pr[i] = vr[i] = mk(0.0, 0.0);
          if (k < k1) {
            kv[i] = vox[k];
            xr[i] = src[vb + k];
            if (needv) {
              vr[i] = u.v[vb + k];
              if (u.mode == UPD_P) pr[i] = u.out[vb + k];
            }
          }
        }
#pragma unroll
        for (int i = 0; i < X::E / 2; ++i) {
          const int k = k0 + i * X::TT;
          if (k >= k1) continue;
          c64 w = xr[i];
          if (upd) {
            w = upd_value(u, us, w, pr[i], vr[i]);
            u.out[vb + k] = w;
          }
          line[pidx(kv[i] - base)] = cvt<T>(w);
        }
      }
      lds_barrier();
#pragma unroll
      for (int q = 0; q < X::E; ++q)
        v[q] = q < X::E / 2 ? line[pidx(t + q * X::TT)] : mk<T>(0, 0);
    } else {
      const c64* xin = x + (((int64_t)rhs * 3 + comp) * a.N3 + z) * a.N2 * a.N1 + (int64_t)y * a.N1;
#pragma unroll
      for (int q = 0; q < X::E; ++q) {
        const int i = t + q * X::TT;
        v[q] = q < X::E / 2 && valid && i < a.N1 ? cvt<T>(xin[i]) : mk<T>(0, 0);
      }
    }
    plane_fft<T, P1, false, true, false>(v, line, t, tr);
    wave_fence();  // the line's own threads (one wave) have done its last reads
    if (valid) {
#pragma unroll
      for (int q = 0; q < X::E; ++q) line[pidx(t + q * X::TT)] = v[q];
    }
  }
  lds_barrier();
  cpx<T>* out = B + rhs * a.rs + comp * a.cs + (z / a.zl) * a.zhs + (z % a.zl) * a.zls;
  VIE_PLANE_Y(a.P2, (plane_y_fwd<T, PP, NT>(plane, X::S, ubuf, out, a.row, tw2, a.N2, P1)));
}

template <typename T, int P1, bool COMP, int NT = plane_threads(P1)>
__global__ __launch_bounds__(NT) void k_plane_inv(
    const cpx<T>* __restrict__ B, const c64* __restrict__ xin, c64* __restrict__ yout,
    const double* __restrict__ chi, const cpx<T>* __restrict__ tw1,
    const cpx<T>* __restrict__ tw2, BodyIdx bi, PlaneArgs a, int mode, c64* __restrict__ aux,
    c64* __restrict__ partials, const c64* __restrict__ pol, const c64* __restrict__ ph,
    const int* __restrict__ active) {
  using X = PlaneLine<P1, NT>;
  extern __shared__ __align__(16) char smem[];
  __shared__ double red[4 * (NT / 64)];
  cpx<T>* plane = reinterpret_cast<cpx<T>*>(smem);
  cpx<T>* ubuf = plane + a.ubuf;
  const int rhs = blockIdx.x % a.nrhs, cz = blockIdx.x / a.nrhs;
  if (active && !active[rhs]) return;
  const int comp = cz / a.N3, z = cz % a.N3;
  const cpx<T>* in = B + rhs * a.rs + comp * a.cs + (z / a.zl) * a.zhs + (z % a.zl) * a.zls;
  VIE_PLANE_Y(a.P2, (plane_y_inv<T, PP, NT>(plane, X::S, ubuf, in, a.row, tw2, a.N2, P1)));
  lds_barrier();
  const int li = threadIdx.x / X::TT, t = threadIdx.x % X::TT;
  TwReg<T, P1, X::E> tr;
  tr.load(t, tw1);
  c64 s0 = mk(0.0, 0.0), s1 = mk(0.0, 0.0);
  for (int n = 0; n * X::L < a.N2; ++n) {
    const int y = n * X::L + li;
    const bool valid = y < a.N2;
    cpx<T>* line = valid ? plane + y * X::S : ubuf + li * X::S;
    cpx<T> v[X::E];
#pragma unroll
    for (int q = 0; q < X::E; ++q) v[q] = valid ? line[pidx(t + q * X::TT)] : mk<T>(0, 0);
    plane_fft<T, P1, true, false, true>(v, line, t, tr);  // only x < N1 is used
    if constexpr (COMP) {
      wave_fence();          // as in the forward pass
      if (!valid) continue;  // no barrier below
      // the line's own threads (one wave) exchange the result
#pragma unroll
      for (int q = 0; q < X::E / 2; ++q) line[pidx(t + q * X::TT)] = v[q];
      const int body = bi.rhs_body[rhs];
      const int nb = bi.nb[body];
      const int* vox = bi.vox + bi.voff[body];
      const double* chic = bi.chic + bi.voff[body];
      const int* lp = bi.line_ptr + (int64_t)body * (a.N2 * a.N3 + 1) + z * a.N2;
      const int64_t vb = bi.roff[rhs] + (int64_t)comp * nb;
      const int k0 = lp[y] + t, k1 = lp[y + 1], base = (z * a.N2 + y) * a.N1;
      c64 phyz = mk(0.0, 0.0), pc = mk(0.0, 0.0);
      const c64* phr = ph + (int64_t)rhs * (a.N1 + a.N2 + a.N3);
      if (mode == EPI_RESID) {
        phyz = phr[a.N1 + y] * phr[a.N1 + a.N2 + z];
        pc = pol[rhs * 3 + comp];
      }
      int kv[X::E / 2];
      double cv[X::E / 2];
      c64 xr[X::E / 2], ar[X::E / 2];
#pragma unroll
      for (int i = 0; i < X::E / 2; ++i) {
        const int k = k0 + i * X::TT;
        ar[i] = mk(0.0, 0.0);
        if (k < k1) {
          kv[i] = vox[k];
          cv[i] = chic[k];
          xr[i] = xin[vb + k];
          if (mode == EPI_RHV) ar[i] = aux[vb + k];
        }
      }
      wave_fence();
#pragma unroll
      for (int i = 0; i < X::E / 2; ++i) {
        const int k = k0 + i * X::TT;
        if (k >= k1) continue;
        const int xi = kv[i] - base;
        const double c = cv[i];
        const c64 yv = xr[i] - c * cvt<double>(line[pidx(xi)]);
        const int64_t gi = vb + k;
        if (mode == EPI_RESID) {
          const c64 e = pc * (phyz * phr[xi]);
          const c64 r = c * e - yv;
          yout[gi] = r;
          aux[gi] = r;
          s1.re += r.re * r.re + r.im * r.im;
        } else {
          yout[gi] = yv;
          if (mode == EPI_RHV) {
            s0 = s0 + cmulc(ar[i], yv);
          } else if (mode == EPI_TS) {
            s0 = s0 + cmulc(yv, xr[i]);
            s1.re += yv.re * yv.re + yv.im * yv.im;
          }
        }
      }
    } else {
      if (!valid) continue;
      const int64_t sp = ((int64_t)z * a.N2 + y) * a.N1;
      const int64_t gi = ((int64_t)rhs * 3 + comp) * a.n + sp;
#pragma unroll
      for (int q = 0; q < X::E / 2; ++q) {
        const int i = t + q * X::TT;
        if (i < a.N1) yout[gi + i] = xin[gi + i] - chi[sp + i] * cvt<double>(v[q]);
      }
    }
  }
  if (COMP && mode != EPI_PLAIN) {
    block_sum2(s0, s1, red);
    if (threadIdx.x == 0) {
      c64* pp = partials + ((int64_t)rhs * 3 * a.N3 + cz) * 2;
      pp[0] = s0;
      pp[1] = s1;
    }
  }
}

// Line lengths along x and y that take the fused passes.  Products of n^3
// boxes, microseconds separate / fused: FP64 16^3 x 1, 8, 32 vectors 22.9 / 15.5,
// 32.5 / 23.5, 51.7 / 41.4; 32^3 33.6 / 27.0, 83.0 / 66.3, 285.6 / 212.0; FP32 32^3
// 29.5 / 19.2, 50.3 / 35.7, 137.1 / 104.1.  At 96 points a plane's lines pass in
// three to five batches and one workgroup (FP32 two) fills a CU's LDS: 48^3 x 1,
// 8, 32 vectors FP64 70 / 73, 349 / 335, 1397 / 1418, FP32 45 / 48, 142 / 152, 651 /
// 653; 40 x 35 x 44 FP64 62 / 66, 273 / 293, 1126 / 1197, FP32 45 / 47, 128 / 146, 567 /
// 593.
static bool plane_len(int p) { return p == 24 || p == 32 || p == 48 || p == 64; }
bool plane_ok(const GroupGeom& g) {
  return plane_len(g.P[0]) && plane_len(g.P[1]);
}

static int plane_stride(int p) { return p + p / 16 + 1; }
static int plane_lines(int p, int nt) { return nt / (p / (p % 3 == 0 ? 12 : 8)); }

static PlaneArgs plane_args(const GroupGeom& g, size_t elem, size_t& lds) {
  PlaneArgs a;
  a.N1 = g.N[0];
  a.N2 = g.N[1];
  a.N3 = g.N[2];
  a.P2 = g.P[1];
  a.nrhs = g.nrhs;
  a.n = g.n;
  a.zl = z_block(g);
  const int nzh = (g.N[2] + a.zl - 1) / a.zl;
  a.row = (int64_t)a.zl * g.P[0];
  a.zls = g.P[0];
  a.zhs = (int64_t)g.P[1] * a.zl * g.P[0];
  a.cs = a.zhs * nzh;
  a.rs = a.cs * 3;
  a.ubuf = g.N[1] * plane_stride(g.P[0]);
  int u = 0;
  for (int k = 0; k < 2; ++k) {
    const int e = plane_lines(g.P[k], plane_threads(g.P[0])) * plane_stride(g.P[k]);
    u = u > e ? u : e;
  }
  lds = (a.ubuf + u) * elem;
  return a;
}

#define VIE_PLANE_X(P1_, CALL)                       \
  switch (P1_) {                                     \
    case 24: { constexpr int PP = 24; CALL; break; } \
    case 32: { constexpr int PP = 32; CALL; break; } \
    case 48: { constexpr int PP = 48; CALL; break; } \
    case 64: { constexpr int PP = 64; CALL; break; } \
    default: return hipErrorInvalidValue;            \
  }

template <typename T>
hipError_t plane_fwd(const GroupGeom& g, const c64* x, cpx<T>* B, const cpx<T>* tw1,
                     const cpx<T>* tw2, const BodyIdx* bi, const int* active, const UpdArgs* upd,
                     hipStream_t s) {
  if (!plane_ok(g) || (upd && !bi)) return hipErrorInvalidValue;
  size_t lds;
  const PlaneArgs a = plane_args(g, sizeof(cpx<T>), lds);
  const UpdArgs u = upd ? *upd : UpdArgs();
  const int grid = 3 * g.N[2] * g.nrhs;
  VIE_PLANE_X(g.P[0], ({
                if (bi)
                  k_plane_fwd<T, PP, true>
                      <<<grid, plane_threads(PP), lds, s>>>(x, B, tw1, tw2, *bi, a, active, u);
                else
                  k_plane_fwd<T, PP, false>
                      <<<grid, plane_threads(PP), lds, s>>>(x, B, tw1, tw2, BodyIdx(), a, active, u);
              }));
  return hipGetLastError();
}

// chi: the body's box (box vectors only; all right-hand sides of one body)
template <typename T>
hipError_t plane_inv(const GroupGeom& g, const cpx<T>* B, const c64* x, c64* y, const double* chi,
                     const cpx<T>* tw1, const cpx<T>* tw2, const BodyIdx* bi, EpiArgs& e,
                     const int* active, hipStream_t s) {
  if (!plane_ok(g) || (!bi && e.mode != EPI_PLAIN))
    return hipErrorInvalidValue;
  size_t lds;
  const PlaneArgs a = plane_args(g, sizeof(cpx<T>), lds);
  e.part_blocks = 3 * g.N[2];
  const int grid = 3 * g.N[2] * g.nrhs;
  VIE_PLANE_X(g.P[0], ({
                if (bi)
                  k_plane_inv<T, PP, true><<<grid, plane_threads(PP), lds, s>>>(
                      B, x, y, chi, tw1, tw2, *bi, a, e.mode, e.aux, e.partials, e.pol, e.ph,
                      active);
                else
                  k_plane_inv<T, PP, false><<<grid, plane_threads(PP), lds, s>>>(
                      B, x, y, chi, tw1, tw2, BodyIdx(), a, e.mode, e.aux, e.partials, e.pol,
                      e.ph, active);
              }));
  return hipGetLastError();
}

#define VIE_PLANE_INST(T)                                                                       \
  template hipError_t plane_fwd<T>(const GroupGeom&, const c64*, cpx<T>*, const cpx<T>*,        \
                                   const cpx<T>*, const BodyIdx*, const int*, const UpdArgs*,   \
                                   hipStream_t);                                                \
  template hipError_t plane_inv<T>(const GroupGeom&, const cpx<T>*, const c64*, c64*,           \
                                   const double*, const cpx<T>*, const cpx<T>*, const BodyIdx*, \
                                   EpiArgs&, const int*, hipStream_t);
VIE_PLANE_INST(double)
VIE_PLANE_INST(float)

}  // namespace vie
