// Rooftop basis with pulse testing (Sec. II-C, eq. Js_expand): FP64 products,
// or FP32 products inside FP64 refinement.
//
// The paper expands the current in rooftops along x, y and z on the uniform
// grid and tests with pulses.  Reading taken (entries and the body surface
// are not given): the contrast current w = chi E, component i carried by
// rooftops on the faces normal to i, a full rooftop between two body cells,
// the inside half on the body surface (alpha = 1 or 1/2); the charge
// rho = div w is constant per cell, a surface face's sheet charge carried by
// its outside cell; E_sca = k0^2 A + grad phi with A = g * w, phi = g * rho,
// both collocated at face centres, midpoint weights h^3 alpha (a rooftop) and
// h^3 (a cell) off the diagonal and the cube-cell integral of g on it; grad
// phi across a face is the difference of its two cells' potentials over h;
// at a face E = W / chi_f with 1/chi_f the mean of its body sides' 1/chi.
//
// The grid is the body grid padded by one cell on every side, so every
// active face has both of its cells on the grid.  A and phi are four scalar
// convolutions with the same kernel h^3 g (self: the cube integral) over the
// padded grid: its circulant (length P >= 2 E - 1 per axis) is transformed
// once at setup, each product transforms alpha W_x, alpha W_y, alpha W_z and
// rho forward, multiplies by the spectrum and transforms back (the inverse as
// the conjugate of the forward transform of the conjugate).  The transforms
// are pruned: the forward one skips the zero padding, the inverse one
// computes only the padded grid's outputs.  The solver is
// BiCGSTAB (the paper's method) with the true residual deciding convergence.
#include <math.h>
#include <string.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <memory>
#include <new>
#include <type_traits>
#include <vector>

#include "../../include/vie.h"
#include "entry.h"
#include "fft_plane.h"
#include "green.h"
#include "kernels.h"
#include "trace.h"

namespace vie {

// Circulant length of an axis of n cells: the smallest supported transform
// length (2^k >= 8 or 3 * 2^k >= 12) with P >= 2 n - 1.
static int rt_fft_length(int n) {
  const int need = std::max(8, 2 * n - 1);
  int p2 = 8, p3 = 12;
  while (p2 < need) p2 <<= 1;
  while (p3 < need) p3 <<= 1;
  return std::min(p2, p3);
}

struct RtGeom {
  int E[3];   // padded grid (body grid + 2)
  int P[3];   // circulant lengths
  int64_t m;  // E1 E2 E3
  int64_t M;  // P1 P2 P3
};

// Circulant samples of h^3 e^{i k0 r} / (4 pi r) over displacements
// [-(E-1), E-1] per axis at index d mod P, zero elsewhere; the cube integral
// at d = 0.
__global__ void k_rt_green(c64* __restrict__ work, RtGeom q, double h, double k0, double s_re,
                           double s_im) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < q.M;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int idx[3] = {(int)(e % q.P[0]), (int)((e / q.P[0]) % q.P[1]),
                        (int)(e / ((int64_t)q.P[0] * q.P[1]))};
    int d[3];
    bool ok = true;
    for (int a = 0; a < 3; ++a) {
      if (idx[a] <= q.E[a] - 1)
        d[a] = idx[a];
      else if (idx[a] >= q.P[a] - (q.E[a] - 1))
        d[a] = idx[a] - q.P[a];
      else
        ok = false;
    }
    c64 v = mk(0.0, 0.0);
    if (ok) {
      if (d[0] == 0 && d[1] == 0 && d[2] == 0) {
        v = mk(s_re, s_im);
      } else {
        const double r = h * sqrt((double)d[0] * d[0] + (double)d[1] * d[1] + (double)d[2] * d[2]);
        double sn, cs;
        sincos(k0 * r, &sn, &cs);
        const double f = h * h * h / (4.0 * M_PI * r);
        v = mk(f * cs, f * sn);
      }
    }
    work[e] = v;
  }
}

// The kernel samples are even along every axis (they depend on |d| per
// axis), so is their transform: only the octant [0, P/2]^3 is kept,
// [z][y][x] with extents Q = P/2 + 1, scaled by s (= 1/M), with an FP32 copy.
__global__ void k_rt_octant(const c64* __restrict__ in, c64* __restrict__ out,
                            c32* __restrict__ out32, RtGeom q, double s) {
  const int Q0 = q.P[0] / 2 + 1, Q1 = q.P[1] / 2 + 1, Q2 = q.P[2] / 2 + 1;
  const int64_t n = (int64_t)Q0 * Q1 * Q2;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int x = (int)(e % Q0), y = (int)((e / Q0) % Q1), z = (int)(e / ((int64_t)Q0 * Q1));
    const c64 v = s * in[((int64_t)z * q.P[1] + y) * q.P[0] + x];
    out[e] = v;
    out32[e] = cvt<float>(v);
  }
}

// ------------------------------------------------------- product passes
// Fields f = 0..2: the weighted currents alpha W_f, f = 3: the cell charge.
constexpr int kRtFields = 4;

// Value of field f at cell c = (cx, cy, cz) of the vector x [3][m].  Inactive
// faces (alpha = 0) contribute nothing, whatever x holds there.  Every load is
// issued before the first is used (neighbours off the grid read the cell
// itself): loading x only behind a test of alpha made the pass wait twice per
// face.
__device__ __forceinline__ c64 rt_field(const c64* __restrict__ x, const double* __restrict__ alpha,
                                        const RtGeom& q, int f, int cx, int cy, int cz, int64_t c,
                                        double inv_h) {
  const c64 zero = mk(0.0, 0.0);
  if (f < 3) {
    const double a = alpha[f * q.m + c];
    const c64 v = x[f * q.m + c];
    return a != 0.0 ? a * v : zero;
  }
  const int64_t step[3] = {1, q.E[0], (int64_t)q.E[0] * q.E[1]};
  const int pc[3] = {cx, cy, cz};
  double a[6];
  c64 xv[6];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const int64_t o = i * q.m + c, lo = pc[i] > 0 ? o - step[i] : o;
    a[2 * i] = alpha[o];
    xv[2 * i] = x[o];
    a[2 * i + 1] = alpha[lo];
    xv[2 * i + 1] = x[lo];
  }
  c64 v = zero;
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    v = v + (a[2 * i] != 0.0 ? xv[2 * i] : zero);                                   // + face
    v = v - (pc[i] > 0 && a[2 * i + 1] != 0.0 ? xv[2 * i + 1] : zero);  // - face
  }
  return inv_h * v;
}

// x pass with the gather, over the lines (field, z, y) of every vector of a
// batch: E1 gathered values -> P1 points of t1 [vector][field][z][y][P1].
// HBM/L2 bound (one thread group per line, unit-stride reads and writes).
template <typename T, int P>
__global__ __launch_bounds__(nt_lines_p<T>(P)) void k_rt_xfwd(
    const c64* __restrict__ x, const double* __restrict__ alpha, cpx<T>* __restrict__ t1,
    const cpx<T>* __restrict__ tw, RtGeom q, double inv_h, int blocks_per_vec,
    const int* __restrict__ active) {
  constexpr int E = fft_e<P>(), TT = P / E, NT = nt_lines_p<T>(P), L = NT / TT,
                LS = PadX<P, TT>::LSTR;
  __shared__ cpx<T> lds[L * LS];
  const int vec = blockIdx.x / blocks_per_vec, blk = blockIdx.x % blocks_per_vec;
  if (active && !active[vec]) return;
  const int li = threadIdx.x / TT, t = threadIdx.x % TT;
  const int zy = q.E[1] * q.E[2], lines = kRtFields * zy;
  const int line = blk * L + li;
  const bool valid = line < lines;
  const int f = valid ? line / zy : 0, yz = valid ? line % zy : 0;
  const int cy = yz % q.E[1], cz = yz / q.E[1];
  const c64* xv = x + (int64_t)vec * 3 * q.m;
  TwReg<T, P, E> tr;
  tr.load(t, tw);
  cpx<T> v[E];
#pragma unroll
  for (int k = 0; k < E; ++k) {
    const int cx = t + k * TT;
    if (k < E / 2 && valid && cx < q.E[0])
      v[k] = cvt<T>(rt_field(xv, alpha, q, f, cx, cy, cz, (int64_t)yz * q.E[0] + cx, inv_h));
    else
      v[k] = mk<T>(0, 0);
  }
  line_fft<T, P, false, true>(v, lds + li * LS, t, tr);
  if (valid) {
    cpx<T>* o = t1 + ((int64_t)vec * lines + line) * P;
#pragma unroll
    for (int k = 0; k < E; ++k) o[t + k * TT] = v[k];
  }
}

// The z stage, in place on t2 [vector][field][z < E3][P2][P1]: forward z
// transforms of the four fields of a column (zero half skipped), the three
// components g (k0^2 F_i + D_i F_3) per point (1/M folded in g), inverse
// transforms keeping z < E3, into fields 0..2.  Only the charge's transform
// stays in registers; the components pass one by one, each one's points
// requested while the one before is transformed, and the twiddles come from an
// LDS table, so two waves share a SIMD.  Latency of the FP64 transforms' LDS
// exchanges bounds it.  Microseconds per BiCGSTAB iteration of two channels on
// 40^3 / 64^3 cells: 193 / 1077; four fields and register twiddles in one
// wave's registers 217 / 1150; a launch per field, channel and pass 600 / 1430.
template <int P>
constexpr int rz_e() {
  return P % 3 == 0 ? 12 : 8;
}
template <typename T, int P>
constexpr int rz_threads() {
  constexpr int n = (int)(128 / sizeof(cpx<T>)) * (P / rz_e<P>());  // 128-byte rows
  return n < 64 ? 64 : n;
}
template <typename T, int P, int NT = rz_threads<T, P>()>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(2))) void k_rt_z(
    cpx<T>* __restrict__ t2, const cpx<T>* __restrict__ ghat, const cpx<T>* __restrict__ tw,
    const cpx<T>* __restrict__ dx, const cpx<T>* __restrict__ dy, const cpx<T>* __restrict__ dz,
    int E3, int P1, int P2, int tiles, int nvec, T k0sq, const int* __restrict__ active) {
  constexpr int E = rz_e<P>(), TT = P / E, W = NT / TT, LS = Pad<P>::LSTR;
  __shared__ cpx<T> lds[W * LS];
  // vectors innermost: they share the spectrum
  const int b = xcd_remap(blockIdx.x, gridDim.x);
  const int vec = b % nvec, rest = b / nvec;
  if (active && !active[vec]) return;
  const int tile = rest % tiles, y = rest / tiles;
  const int cw = threadIdx.x % W, t = threadIdx.x / W;
  const int col = tile * W + cw;
  const bool valid = col < P1;
  const int xc = valid ? col : 0;
  const int64_t plane = (int64_t)P2 * P1, cs = plane * E3;
  cpx<T>* base = t2 + (int64_t)vec * kRtFields * cs + (int64_t)y * P1 + xc;
  __shared__ cpx<T> stw[P];
  for (int k = threadIdx.x; k < P; k += NT) stw[k] = tw[k];
  lds_barrier();
  const LdsLine<T> ll{lds + cw * LS};
  auto load = [&](int f, cpx<T> (&v)[E / 2]) {
#pragma unroll
    for (int k = 0; k < E / 2; ++k) {
      const int z = t + k * TT;
      v[k] = valid && z < E3 ? base[f * cs + z * plane] : mk<T>(0, 0);
    }
  };
  // the spectrum's octant record of this column (mirrored x and y)
  const int Q0 = P1 / 2 + 1, Q1 = P2 / 2 + 1;
  const int xo = xc <= P1 / 2 ? xc : P1 - xc, yo = y <= P2 / 2 ? y : P2 - y;
  const cpx<T>* gcol = ghat + (int64_t)yo * Q0 + xo;
  const int64_t gplane = (int64_t)Q0 * Q1;
  const cpx<T> fxy[2] = {dx[xc], dy[y]};
  cpx<T> rho[E], v[E], nx[E / 2];
  load(3, nx);
#pragma unroll
  for (int k = 0; k < E; ++k) rho[k] = k < E / 2 ? nx[k < E / 2 ? k : 0] : mk<T>(0, 0);
  load(0, nx);
  fft_stages_p<T, P, E, 1, false, 0, true, false, true>(rho, ll, t, stw);
#pragma unroll
  for (int i = 0; i < 3; ++i) {
#pragma unroll
    for (int k = 0; k < E; ++k) v[k] = k < E / 2 ? nx[k < E / 2 ? k : 0] : mk<T>(0, 0);
    if (i < 2) load(i + 1, nx);
    fft_stages_p<T, P, E, 1, false, 0, true, false, true>(v, ll, t, stw);
#pragma unroll
    for (int k = 0; k < E; ++k) {
      const int z = t + k * TT;
      const cpx<T> g = gcol[(int64_t)(z <= P / 2 ? z : P - z) * gplane];
      const cpx<T> d = i < 2 ? fxy[i < 2 ? i : 0] : dz[z];
      v[k] = g * cfma(d, rho[k], k0sq * v[k]);
    }
    fft_stages_p<T, P, E, 1, true, 0, false, true, true>(v, ll, t, stw);
    if (valid) {
#pragma unroll
      for (int k = 0; k < E / 2; ++k) {
        const int z = t + k * TT;
        if (z < E3) base[i * cs + z * plane] = v[k];
      }
    }
  }
}

// Last pass: inverse x transform of the lines (component, z, y), keeping
// x < E1, then y = x - chi_f E (y = x on inactive faces) and the product's dot
// partials, one pair per workgroup (fixed order):
//   kEpiRhv: (aux, y);  kEpiTs: (y, x) and |y|^2;
//   kEpiRes: out = aux - y, |out|^2
enum { kEpiPlain = 0, kEpiRhv = 1, kEpiTs = 2, kEpiRes = 3 };
template <typename T, int P, int MODE>
__global__ __launch_bounds__(nt_lines_p<T>(P)) void k_rt_xinv(
    const cpx<T>* __restrict__ t1, const c64* __restrict__ x, const double* __restrict__ chif,
    const c64* __restrict__ aux, c64* __restrict__ out, c64* __restrict__ part,
    const cpx<T>* __restrict__ tw, RtGeom q, int blocks_per_vec, const int* __restrict__ active) {
  constexpr int E = fft_e<P>(), TT = P / E, NT = nt_lines_p<T>(P), L = NT / TT,
                LS = PadX<P, TT>::LSTR;
  __shared__ cpx<T> lds[L * LS];
  __shared__ double red[4 * (NT / 64 + 1)];
  const int vec = blockIdx.x / blocks_per_vec, blk = blockIdx.x % blocks_per_vec;
  if (active && !active[vec]) return;
  const int li = threadIdx.x / TT, t = threadIdx.x % TT;
  const int lines = 3 * q.E[1] * q.E[2];
  const int line = blk * L + li;
  const bool valid = line < lines;
  const cpx<T>* src = t1 + ((int64_t)vec * lines + (valid ? line : 0)) * P;
  TwReg<T, P, E> tr;
  tr.load(t, tw);
  cpx<T> v[E];
#pragma unroll
  for (int k = 0; k < E; ++k) v[k] = valid ? src[t + k * TT] : mk<T>(0, 0);
  line_fft<T, P, true, false, true>(v, lds + li * LS, t, tr);
  c64 s0 = mk(0.0, 0.0), s1 = mk(0.0, 0.0);
  if (valid) {
#pragma unroll
    for (int k = 0; k < E / 2; ++k) {
      const int cx = t + k * TT;
      if (cx >= q.E[0]) continue;
      const int64_t e = (int64_t)line * q.E[0] + cx;  // within the vector
      const int64_t g = (int64_t)vec * 3 * q.m + e;
      const double cf = chif[e];
      const c64 xv = x[g];
      const c64 y = cf != 0.0 ? xv - cf * cvt<double>(v[k]) : xv;
      if (MODE == kEpiRes) {
        const c64 r = aux[g] - y;
        out[g] = r;
        s1.re += r.re * r.re + r.im * r.im;
      } else {
        out[g] = y;
        if (MODE == kEpiRhv) s0 = s0 + cmulc(aux[g], y);
        if (MODE == kEpiTs) {
          s0 = s0 + cmulc(y, xv);
          s1.re += y.re * y.re + y.im * y.im;
        }
      }
    }
  }
  if (MODE != kEpiPlain) {
    block_sum2(s0, s1, red);
    if (threadIdx.x == 0) {
      c64* pp = part + ((int64_t)vec * blocks_per_vec + blk) * 2;
      pp[0] = s0;
      pp[1] = s1;
    }
  }
}

// Incident channel of a batch.
struct RtWave {
  double k[3];
  c64 p[3];
};

constexpr int kRtThreads = 256;
constexpr int kRtFold = 64;  // partial pairs per vector that a vector kernel sums itself

// Sum of n pairs of partials in a fixed order, to every thread.
__device__ __forceinline__ void rt_sum(const c64* __restrict__ part, int n, c64& a, c64& b) {
  __shared__ double red[16];
  fold_pairs<kRtThreads>(part, n, red, a, b);
}

// This thread's sums into the workgroup's partial pair.
__device__ __forceinline__ void rt_partial(c64 s0, c64 s1, c64* __restrict__ out) {
  __shared__ double red[4 * (kRtThreads / 64)];
  block_sum2(s0, s1, red);
  if (threadIdx.x == 0) {
    out[0] = s0;
    out[1] = s1;
  }
}

// Many partials (one per workgroup of a large grid's last pass) folded to
// kRtFold per vector.
__global__ void __launch_bounds__(64) k_rt_fold(const c64* __restrict__ part, int n,
                                                c64* __restrict__ out,
                                                const int* __restrict__ active) {
  const int vec = blockIdx.x / kRtFold, j = blockIdx.x % kRtFold;
  if (!active[vec]) return;
  const int k0 = (int)((int64_t)n * j / kRtFold), k1 = (int)((int64_t)n * (j + 1) / kRtFold);
  const c64* p = part + (int64_t)vec * n * 2;
  double v[4] = {0, 0, 0, 0};
  for (int k = k0 + threadIdx.x; k < k1; k += 64) {
    v[0] += p[2 * k].re;
    v[1] += p[2 * k].im;
    v[2] += p[2 * k + 1].re;
    v[3] += p[2 * k + 1].im;
  }
  for (int m = 32; m >= 1; m >>= 1)
    for (int c = 0; c < 4; ++c) v[c] += __shfl_xor(v[c], m, 64);
  if (threadIdx.x == 0) {
    c64* o = out + ((int64_t)vec * kRtFold + j) * 2;
    o[0] = mk(v[0], v[1]);
    o[1] = mk(v[2], v[3]);
  }
}

// BiCGSTAB scalars of one vector, on the device between host checks.  A
// vector kernel sums the partials it needs in every workgroup and one
// workgroup per vector stores the results; no kernel stores a value that
// another workgroup of the same launch reads (except `active`, cleared by the
// same decision that every workgroup takes for itself, see group_flag).
struct RtScal {
  c64 rho, rho1, alpha, omega;
  double tol2;      // tol^2 ||b||^2 (recursive residual threshold)
  int it, max_it;   // iterations done (all cycles), cap
  int stop;         // 0 running, 1 recursive residual reached, 2 breakdown, 3 cap
};

__device__ __forceinline__ bool rt_zero(c64 a) { return a.re == 0.0 && a.im == 0.0; }

// b = chi_f pol_i e^{i k0 khat . r_f}, face i of padded cell c at
// origin + h (c - 1) + (h/2) e_i; x = p = v = 0, r = rh = b, partials |b|^2.
__global__ void __launch_bounds__(kRtThreads) k_rt_rhs(
    c64* __restrict__ b, c64* __restrict__ x, c64* __restrict__ r, c64* __restrict__ rh,
    c64* __restrict__ p, c64* __restrict__ v, const double* __restrict__ chif, RtGeom q, double h,
    double o0, double o1, double o2, double k0, const RtWave* __restrict__ wave, int vb,
    c64* __restrict__ part) {
  const int vec = blockIdx.x / vb, blk = blockIdx.x % vb;
  const RtWave w = wave[vec];
  const int64_t n = 3 * q.m;
  c64 s = mk(0.0, 0.0);
  for (int64_t e = (int64_t)blk * kRtThreads + threadIdx.x; e < n; e += (int64_t)vb * kRtThreads) {
    const double cf = chif[e];
    c64 val = mk(0.0, 0.0);
    if (cf != 0.0) {
      const int i = (int)(e / q.m);
      const int64_t c = e - i * q.m;
      double rr[3] = {o0 + h * ((int)(c % q.E[0]) - 1),
                      o1 + h * ((int)((c / q.E[0]) % q.E[1]) - 1),
                      o2 + h * ((int)(c / ((int64_t)q.E[0] * q.E[1])) - 1)};
      rr[i] += 0.5 * h;
      double sn, cs;
      sincos(k0 * (w.k[0] * rr[0] + w.k[1] * rr[1] + w.k[2] * rr[2]), &sn, &cs);
      val = cf * (w.p[i] * mk(cs, sn));
    }
    const int64_t g = vec * n + e;
    b[g] = r[g] = rh[g] = val;
    x[g] = p[g] = v[g] = mk(0.0, 0.0);
    s.re += val.re * val.re + val.im * val.im;
  }
  rt_partial(s, s, part + ((int64_t)vec * vb + blk) * 2);
}

// Restart of the marked vectors from their true residual t: r = rh = t,
// p = v = 0, partials |t|^2.
__global__ void __launch_bounds__(kRtThreads) k_rt_restart(
    const c64* __restrict__ t, c64* __restrict__ r, c64* __restrict__ rh, c64* __restrict__ p,
    c64* __restrict__ v, int64_t n, int vb, c64* __restrict__ part, const int* __restrict__ mark) {
  const int vec = blockIdx.x / vb, blk = blockIdx.x % vb;
  if (!mark[vec]) return;
  c64 s = mk(0.0, 0.0);
  for (int64_t e = (int64_t)blk * kRtThreads + threadIdx.x; e < n; e += (int64_t)vb * kRtThreads) {
    const int64_t g = vec * n + e;
    const c64 val = t[g];
    r[g] = rh[g] = val;
    p[g] = v[g] = mk(0.0, 0.0);
    s.re += val.re * val.re + val.im * val.im;
  }
  rt_partial(s, s, part + ((int64_t)vec * vb + blk) * 2);
}

// Ends or continues the iteration on the partials ((rh, r), (r, r)) of the
// last residual update, then p = r + beta (p - omega v),
// beta = (rho1 / rho)(alpha / omega).  A zero denominator stops the cycle
// (breakdown); so does the iteration cap.
__global__ void __launch_bounds__(kRtThreads) k_rt_pupd(
    c64* __restrict__ p, const c64* __restrict__ r, const c64* __restrict__ v,
    RtScal* __restrict__ scal, int* active, int64_t n, int vb,
    const c64* __restrict__ part, int npart) {
  const int vec = blockIdx.x / vb, blk = blockIdx.x % vb;
  if (!group_flag(active + vec)) return;
  RtScal* S = scal + vec;
  const c64 rho = S->rho, alpha = S->alpha, om = S->omega;
  const double tol2 = S->tol2;
  const int it = S->it, max_it = S->max_it;
  c64 rho1, rr;
  rt_sum(part + (int64_t)vec * npart * 2, npart, rho1, rr);
  int stop = 0;
  if (rr.re <= tol2)
    stop = 1;
  else if (rt_zero(om))
    stop = 2;
  else if (it >= max_it)
    stop = 3;
  else if (rt_zero(rho1))
    stop = 2;
  if (blk == 0 && threadIdx.x == 0) {
    S->rho1 = rho1;
    S->stop = stop;
    if (stop) active[vec] = 0;
  }
  if (stop) return;
  const c64 beta = kcdiv(rho1, rho) * kcdiv(alpha, om);
  for (int64_t e = (int64_t)blk * kRtThreads + threadIdx.x; e < n; e += (int64_t)vb * kRtThreads) {
    const int64_t g = vec * n + e;
    p[g] = r[g] + beta * (p[g] - om * v[g]);
  }
}

// alpha = rho1 / (rh, v); s = r - alpha v
__global__ void __launch_bounds__(kRtThreads) k_rt_supd(
    c64* __restrict__ s, const c64* __restrict__ r, const c64* __restrict__ v,
    RtScal* __restrict__ scal, int* active, int64_t n, int vb,
    const c64* __restrict__ part, int npart) {
  const int vec = blockIdx.x / vb, blk = blockIdx.x % vb;
  if (!group_flag(active + vec)) return;
  RtScal* S = scal + vec;
  const c64 rho1 = S->rho1;
  c64 rhv, none;
  rt_sum(part + (int64_t)vec * npart * 2, npart, rhv, none);
  const bool stop = rt_zero(rhv);
  const c64 al = stop ? mk(0.0, 0.0) : kcdiv(rho1, rhv);
  if (blk == 0 && threadIdx.x == 0) {
    if (stop) {
      S->stop = 2;
      active[vec] = 0;
    } else {
      S->alpha = al;
    }
  }
  if (stop) return;
  for (int64_t e = (int64_t)blk * kRtThreads + threadIdx.x; e < n; e += (int64_t)vb * kRtThreads) {
    const int64_t g = vec * n + e;
    s[g] = r[g] - al * v[g];
  }
}

// omega = (t, s) / (t, t); x += alpha p + omega s; r = s - omega t; one
// iteration done; partials (rh, r), |r|^2.
__global__ void __launch_bounds__(kRtThreads) k_rt_xrupd(
    c64* __restrict__ x, c64* __restrict__ r, const c64* __restrict__ p,
    const c64* __restrict__ s, const c64* __restrict__ t, const c64* __restrict__ rh,
    RtScal* __restrict__ scal, const int* __restrict__ active, int64_t n, int vb,
    const c64* __restrict__ part, int npart, c64* __restrict__ out) {
  const int vec = blockIdx.x / vb, blk = blockIdx.x % vb;
  if (!active[vec]) return;
  RtScal* S = scal + vec;
  const c64 al = S->alpha;
  c64 ts, tt;
  rt_sum(part + (int64_t)vec * npart * 2, npart, ts, tt);
  const c64 om = tt.re > 0 ? mk(ts.re / tt.re, ts.im / tt.re) : mk(0.0, 0.0);
  if (blk == 0 && threadIdx.x == 0) {
    S->omega = om;
    S->rho = S->rho1;
    S->it += 1;
  }
  c64 s0 = mk(0.0, 0.0), s1 = mk(0.0, 0.0);
  for (int64_t e = (int64_t)blk * kRtThreads + threadIdx.x; e < n; e += (int64_t)vb * kRtThreads) {
    const int64_t g = vec * n + e;
    const c64 se = s[g];
    x[g] = x[g] + al * p[g] + om * se;
    const c64 rn = se - om * t[g];
    r[g] = rn;
    s0 = s0 + cmulc(rh[g], rn);
    s1.re += rn.re * rn.re + rn.im * rn.im;
  }
  rt_partial(s0, s1, out + ((int64_t)vec * vb + blk) * 2);
}

// The sums of one pair of partials per marked vector, for the host.
__global__ void __launch_bounds__(kRtThreads) k_rt_total(const c64* __restrict__ part, int npart,
                                                         double* __restrict__ out,
                                                         const int* __restrict__ mark) {
  if (mark && !mark[blockIdx.x]) return;
  c64 a, b;
  rt_sum(part + (int64_t)blockIdx.x * npart * 2, npart, a, b);
  if (threadIdx.x == 0) out[blockIdx.x] = b.re;
}

}  // namespace vie

using namespace vie;

namespace {
// Grow-only device buffer (contents not preserved).
struct RtBuf {
  void* p = nullptr;
  size_t bytes = 0;
  RtBuf() = default;
  RtBuf(const RtBuf&) = delete;
  RtBuf& operator=(const RtBuf&) = delete;
  ~RtBuf() {
    if (p) (void)hipFree(p);
  }
  hipError_t reserve(size_t b) {
    if (b <= bytes) return hipSuccess;
    if (p) (void)hipFree(p);
    p = nullptr;
    bytes = 0;
    const hipError_t e = dev_malloc(&p, b);
    if (e == hipSuccess) bytes = b;
    return e;
  }
  template <typename T>
  T* as() const {
    return (T*)p;
  }
};
}  // namespace

// Pinned pieces between the device and the caller's pageable arrays.  For the
// 13.8 MB of a 64^3 body's vector the runtime's own copy back takes 940 us; a
// pinned copy takes 256 us and one core reads what the device has just written
// in 530 us, so with four pieces of 1 MB in turn the two overlap: 537 us (256
// KB: 994, 512 KB: 628, 2 MB: 543 us).  The other way staging is no faster (475
// us against 342 us for 12.4 MB).  Kept by the handle, made by its first large
// copy (300 us).
struct RtStage {
  static constexpr int kPieces = 4;
  static constexpr size_t kPiece = (size_t)1 << 20;
  static constexpr size_t kLeast = kPieces * kPiece;  // 4 MB: 150 us against 240 us
  char* p = nullptr;
  hipEvent_t ev[kPieces] = {};
  ~RtStage() {
    for (auto e : ev)
      if (e) (void)hipEventDestroy(e);
    if (p) (void)hipHostFree(p);
  }
  bool ready() {
    if (p) return true;
    for (auto& e : ev)
      if (!e && hipEventCreateWithFlags(&e, hipEventDisableTiming) != hipSuccess) {
        e = nullptr;
        (void)hipGetLastError();
        return false;
      }
    if (hipHostMalloc((void**)&p, kPieces * kPiece) == hipSuccess) return true;
    p = nullptr;
    (void)hipGetLastError();
    return false;
  }
  // Copies to `host`; it and all queued before it are done on return.  Memory
  // that the runtime knows (pinned, managed) needs no staging, and without
  // staging memory the copy is the runtime's.
  hipError_t to_host(void* host, const void* dev, size_t bytes, hipStream_t s) {
    bool plain = bytes < kLeast;
    if (!plain) {
      hipPointerAttribute_t a;
      if (hipPointerGetAttributes(&a, host) != hipSuccess)
        (void)hipGetLastError();
      else
        plain = a.type != hipMemoryTypeUnregistered;
    }
    if (plain || !ready()) {
      const hipError_t e = hipMemcpyAsync(host, dev, bytes, hipMemcpyDeviceToHost, s);
      return e == hipSuccess ? hipStreamSynchronize(s) : e;
    }
    const size_t np = (bytes + kPiece - 1) / kPiece;
    for (size_t i = 0; i < np + kPieces; ++i) {
      const int k = (int)(i % kPieces);
      hipError_t e = hipSuccess;
      if (i >= kPieces && i - kPieces < np) {
        const size_t at = (i - kPieces) * kPiece;
        if ((e = hipEventSynchronize(ev[k])) != hipSuccess) return e;
        memcpy((char*)host + at, p + k * kPiece, std::min(kPiece, bytes - at));
      }
      if (i < np) {
        e = hipMemcpyAsync(p + k * kPiece, (const char*)dev + i * kPiece,
                           std::min(kPiece, bytes - i * kPiece), hipMemcpyDeviceToHost, s);
        if (e == hipSuccess) e = hipEventRecord(ev[k], s);
        if (e != hipSuccess) return e;
      }
    }
    return hipSuccess;
  }
};

// Workspace of `cap` vectors, one allocation: transform scratch
// [vec][4][E3][E2][P1] and [vec][4][E3][P2][P1], eight solver vectors, dot
// partials, the solver's scalars and flags.
struct RtWork {
  char* base = nullptr;
  int cap = 0;
  c64 *t1, *t2, *vecs, *part[3], *fold;
  RtScal* scal;
  RtWave* wave;
  double* total;
  int *active, *mark;
};

struct vie_rt {
  int N[3] = {0, 0, 0};
  double h = 0, k0 = 0, origin[3] = {0, 0, 0};
  RtGeom q{};
  GroupGeom g{};
  hipStream_t stream = nullptr;
  bool poisoned = false;
  // one allocation each: the faces, the spectrum, the tables
  double* alpha = nullptr;  // [3][m]
  double* chif = nullptr;   // [3][m]
  c64* ghat = nullptr;      // spectrum / M on the octant [0, P/2]^3
  c32* ghat32 = nullptr;    // its FP32 copy
  c64* tables = nullptr;    // per axis tw, df, then their FP32 copies
  c64* tw[3] = {nullptr, nullptr, nullptr};
  c32* tw32[3] = {nullptr, nullptr, nullptr};
  c64* df[3] = {nullptr, nullptr, nullptr};    // D_a(k) = (e^{2 pi i k / P_a} - 1) / h
  c32* df32[3] = {nullptr, nullptr, nullptr};
  int dev = 0;  // HIP device current at setup
  RtWork w;     // of the largest batch of vectors so far, one from setup on
  // far field: the cells with an active face (ascending), their blocks and
  // columns (built on first use), scratch
  std::vector<int> cells;
  bool far_blocks = false, far_columns = false;
  FarBlocks fb;
  FarColumns fc;
  RtBuf fvi, forg, cptr, corg, cent, fw, fin, fidx, fdirs, fwd, fpart, fF;
  RtStage stage;
};

namespace {

constexpr int kRtMaxN = 128;

int blocks_for(int64_t n) {
  int64_t b = (n + kRtThreads - 1) / kRtThreads;
  return (int)std::min<int64_t>(std::max<int64_t>(b, 1), 4096);
}

template <typename T>
hipError_t dalloc(T** p, size_t count) {
  return dev_malloc(p, count * sizeof(T));
}

void rt_free(vie_rt* r) {
  auto f = [](void* p) {
    if (p) (void)hipFree(p);
  };
  f(r->alpha);
  f(r->ghat);
  f(r->tables);
  f(r->w.base);
  if (r->stream) (void)hipStreamDestroy(r->stream);
}

#define RT_HIP(call)                 \
  do {                               \
    hipError_t e_ = (call);          \
    if (e_ != hipSuccess) {          \
      r->poisoned = true;            \
      return VIE_EDEVICE;            \
    }                                \
  } while (0)

// Launch shapes of a vector kernel and of the last product pass: workgroups
// (partial pairs) per vector.
int vec_blocks(int64_t n) {
  return (int)std::min<int64_t>(512, std::max<int64_t>(1, (n + 4 * kRtThreads - 1) /
                                                              (4 * kRtThreads)));
}
template <typename T>
int xinv_blocks(const RtGeom& q) {
  const int L = lines_per_block<T>(q.P[0]);
  return (3 * q.E[1] * q.E[2] + L - 1) / L;
}

// Makes the handle's device the current one for a call: the calls allocate.
struct RtDevice {
  int prev = -1;
  explicit RtDevice(int dev) {
    int cur = dev;
    if (hipGetDevice(&cur) == hipSuccess && cur != dev && hipSetDevice(dev) == hipSuccess)
      prev = cur;
  }
  ~RtDevice() {
    if (prev >= 0) (void)hipSetDevice(prev);
  }
};

// Workspace for nvec vectors at once.  Where it cannot grow the old one stays
// in place (setup makes one for a single vector), so a product always runs and
// a solve always fits one channel.  least: bytes wanted for another use.
hipError_t rt_reserve(vie_rt* r, int nvec, size_t least = 0) {
  if (nvec <= r->w.cap) return hipSuccess;
  const RtGeom& q = r->q;
  RtWork w;
  size_t bytes = 0;
  auto lay = [&](auto*& p, size_t count) {  // the first pass counts, the second places
    using T = std::remove_reference_t<decltype(*p)>;
    p = w.base ? (T*)(w.base + bytes) : nullptr;
    bytes += (nvec * count * sizeof(T) + 255) / 256 * 256;
  };
  const size_t row = (size_t)kRtFields * q.E[2] * q.P[0];
  const size_t np = std::max(std::max(xinv_blocks<double>(q), xinv_blocks<float>(q)),
                             vec_blocks(3 * q.m));
  for (int pass = 0; pass < 2; ++pass) {
    bytes = 0;
    lay(w.t1, row * q.E[1]);
    lay(w.t2, row * q.P[1]);
    lay(w.vecs, (size_t)8 * 3 * q.m);
    for (auto& p : w.part) lay(p, np * 2);
    lay(w.fold, (size_t)kRtFold * 2);
    lay(w.scal, 1);
    lay(w.wave, 1);
    lay(w.total, 1);
    lay(w.active, 1);
    lay(w.mark, 1);
    if (pass == 0) {
      const hipError_t e = dev_malloc(&w.base, std::max(bytes, least));
      if (e != hipSuccess) return e;
    }
  }
  w.cap = nvec;
  if (r->w.base) (void)hipFree(r->w.base);
  r->w = w;
  return hipSuccess;
}

// out = A x (kEpiRes: aux - A x) of nvec vectors [nvec][3][m] (device), with
// the dot partials of `mode` in part.  The transforms run in T (FP64, or FP32
// for the inner products of a mixed solve); gather, epilogue and out stay
// FP64.  active (nullable): only the vectors with a non-zero flag.
template <typename T>
int rt_apply_t(vie_rt* r, const c64* x, c64* out, int nvec, int mode, const c64* aux, c64* part,
               const int* active) {
  const RtGeom& q = r->q;
  const bool f64 = sizeof(T) == 8;
  auto pick = [&](const void* a, const void* b) { return (const cpx<T>*)(f64 ? a : b); };
  const cpx<T>* tw[3];
  const cpx<T>* df[3];
  for (int a = 0; a < 3; ++a) {
    tw[a] = pick(r->tw[a], r->tw32[a]);
    df[a] = pick(r->df[a], r->df32[a]);
  }
  const cpx<T>* ghat = pick(r->ghat, r->ghat32);
  cpx<T>* t1 = (cpx<T>*)r->w.t1;
  cpx<T>* t2 = (cpx<T>*)r->w.t2;
  const double inv_h = 1.0 / r->h;
  const int L = lines_per_block<T>(q.P[0]);
  const int bf = (kRtFields * q.E[1] * q.E[2] + L - 1) / L, bi = xinv_blocks<T>(q);
  auto xf = [&]() -> hipError_t {
    VIE_DISPATCH_P(q.P[0], (k_rt_xfwd<T, PP><<<bf * nvec, nt_lines_p<T>(PP), 0, r->stream>>>(
                               x, r->alpha, t1, tw[0], q, inv_h, bf, active)));
    return hipGetLastError();
  };
  auto zc = [&]() -> hipError_t {
    VIE_DISPATCH_PZ(q.P[2], ({
                      constexpr int NT = rz_threads<T, PP>();
                      constexpr int W = NT / (PP / rz_e<PP>());
                      const int tiles = (q.P[0] + W - 1) / W;
                      k_rt_z<T, PP><<<tiles * q.P[1] * nvec, NT, 0, r->stream>>>(
                          t2, ghat, tw[2], df[0], df[1], df[2], q.E[2], q.P[0], q.P[1], tiles,
                          nvec, (T)(r->k0 * r->k0), active);
                    }));
    return hipGetLastError();
  };
#define RT_XINV(MODE_)                                                                     \
  VIE_DISPATCH_P(q.P[0], (k_rt_xinv<T, PP, MODE_><<<bi * nvec, nt_lines_p<T>(PP), 0,         \
                                                    r->stream>>>(t1, x, r->chif, aux, out, \
                                                                 part, tw[0], q, bi, active)))
  auto xi = [&]() -> hipError_t {
    switch (mode) {
      case kEpiPlain: RT_XINV(kEpiPlain); break;
      case kEpiRhv: RT_XINV(kEpiRhv); break;
      case kEpiTs: RT_XINV(kEpiTs); break;
      default: RT_XINV(kEpiRes); break;
    }
    return hipGetLastError();
  };
#undef RT_XINV
  RT_HIP(xf());
  RT_HIP(launch_fft_y_fields(t1, t2, q.E, q.P, tw[1], nvec, kRtFields, kRtFields, false, active,
                             r->stream));
  RT_HIP(zc());
  RT_HIP(launch_fft_y_fields(t2, t1, q.E, q.P, tw[1], nvec, 3, kRtFields, true, active,
                             r->stream));
  RT_HIP(xi());
  return VIE_OK;
}

int rt_apply(vie_rt* r, const c64* x, c64* out, int nvec, bool fp32, int mode = kEpiPlain,
             const c64* aux = nullptr, c64* part = nullptr, const int* active = nullptr) {
  return fp32 ? rt_apply_t<float>(r, x, out, nvec, mode, aux, part, active)
              : rt_apply_t<double>(r, x, out, nvec, mode, aux, part, active);
}

#define RT_TRY(call)          \
  do {                        \
    int rc_ = (call);         \
    if (rc_ != VIE_OK) return rc_; \
  } while (0)

}  // namespace

extern "C" int vie_rt_setup(const vie_body* body, double k0, vie_rt** out) try {
  TraceRange trace_("vie_rt_setup");
  if (!out) return VIE_EINVAL;
  *out = nullptr;
  if (!body || !body->eps_r || !(body->h > 0) || !std::isfinite(body->h) || !(k0 > 0) ||
      !std::isfinite(k0))
    return VIE_EINVAL;
  for (int a = 0; a < 3; ++a) {
    if (body->n[a] < 1) return VIE_EINVAL;
    if (!std::isfinite(body->origin[a])) return VIE_EINVAL;
  }
  for (int a = 0; a < 3; ++a)
    if (body->n[a] > kRtMaxN) return VIE_ENOTSUP;
  const int64_t nvox = (int64_t)body->n[0] * body->n[1] * body->n[2];
  for (int64_t v = 0; v < nvox; ++v)
    if (!std::isfinite(body->eps_r[v]) || body->eps_r[v] < 1.0) return VIE_EINVAL;

  vie_rt* r = new (std::nothrow) vie_rt();
  if (!r) return VIE_ENOMEM;
  std::unique_ptr<vie_rt, void (*)(vie_rt*)> hold(r, vie_rt_destroy);  // until it is complete
  for (int a = 0; a < 3; ++a) {
    r->N[a] = body->n[a];
    r->origin[a] = body->origin[a];
    r->q.E[a] = body->n[a] + 2;
    r->q.P[a] = rt_fft_length(r->q.E[a]);
    r->g.N[a] = r->q.E[a];
    r->g.P[a] = r->q.P[a];
    r->g.Q[a] = r->q.P[a] / 2 + 1;
  }
  r->h = body->h;
  r->k0 = k0;
  const RtGeom& q = r->q;
  r->q.m = (int64_t)q.E[0] * q.E[1] * q.E[2];
  r->q.M = (int64_t)q.P[0] * q.P[1] * q.P[2];
  r->g.n = r->q.m;
  r->g.nrhs = 1;
  const int64_t m = r->q.m, M = r->q.M;

  // face data: chi on the padded grid, then alpha and chi_f per face
  std::vector<double> chi(m, 0.0), faces(6 * m, 0.0);
  double *alpha = faces.data(), *chif = alpha + 3 * m;
  for (int z = 0; z < r->N[2]; ++z)
    for (int y = 0; y < r->N[1]; ++y)
      for (int x = 0; x < r->N[0]; ++x)
        chi[((int64_t)(z + 1) * q.E[1] + (y + 1)) * q.E[0] + (x + 1)] =
            body->eps_r[((int64_t)z * r->N[1] + y) * r->N[0] + x] - 1.0;
  const int64_t step[3] = {1, q.E[0], (int64_t)q.E[0] * q.E[1]};
  for (int i = 0; i < 3; ++i)
    for (int z = 0; z < q.E[2]; ++z)
      for (int y = 0; y < q.E[1]; ++y)
        for (int x = 0; x < q.E[0]; ++x) {
          const int pc[3] = {x, y, z};
          const int64_t c = ((int64_t)z * q.E[1] + y) * q.E[0] + x;
          const double ca = chi[c];
          const double cb = pc[i] + 1 < q.E[i] ? chi[c + step[i]] : 0.0;
          double a = 0.0, cf = 0.0;
          if (ca != 0.0 && cb != 0.0) {
            a = 1.0;
            cf = 1.0 / (0.5 * (1.0 / ca + 1.0 / cb));
          } else if (ca != 0.0) {
            a = 0.5;
            cf = ca;
          } else if (cb != 0.0) {
            a = 0.5;
            cf = cb;
          }
          alpha[i * m + c] = a;
          chif[i * m + c] = cf;
        }
  for (int64_t c = 0; c < m; ++c)
    if (alpha[c] != 0.0 || alpha[m + c] != 0.0 || alpha[2 * m + c] != 0.0) r->cells.push_back((int)c);

  hipError_t e = hipSuccess;
  auto chk = [&](hipError_t x) {
    if (e == hipSuccess) e = x;
  };
  chk(hipGetDevice(&r->dev));
  chk(hipStreamCreate(&r->stream));
  chk(dalloc(&r->alpha, 6 * m));
  r->chif = r->alpha + 3 * m;
  const int64_t noct = (int64_t)(q.P[0] / 2 + 1) * (q.P[1] / 2 + 1) * (q.P[2] / 2 + 1);
  chk(dalloc(&r->ghat, noct + (noct + 1) / 2));
  r->ghat32 = (c32*)(r->ghat + noct);
  const int sum = q.P[0] + q.P[1] + q.P[2];
  chk(dalloc(&r->tables, 3 * sum));
  for (int a = 0, at = 0; a < 3; at += q.P[a++]) {
    r->tw[a] = r->tables + at;
    r->df[a] = r->tables + sum + at;
    r->tw32[a] = (c32*)(r->tables + 2 * sum) + at;
    r->df32[a] = (c32*)(r->tables + 2 * sum) + sum + at;
  }
  // the circulant and its transform, for the spectrum only, then the workspace:
  // whichever is larger is the one allocation
  chk(rt_reserve(r, 1, 2 * M * sizeof(c64)));
  if (e != hipSuccess) return e == hipErrorOutOfMemory ? VIE_ENOMEM : VIE_EDEVICE;
  c64 *work = (c64*)r->w.base, *tmp = work + M;
  std::vector<c64> tab(3 * sum);
  c32* tab32 = (c32*)(tab.data() + 2 * sum);
  for (int a = 0, at = 0; a < 3; at += q.P[a++])
    for (int k = 0; k < q.P[a]; ++k) {
      const long double pi = 3.14159265358979323846264338327950288L;
      const long double ang = -2.0L * pi * k / q.P[a], cs = cosl(ang), sn = sinl(ang);
      tab[at + k] = mk((double)cs, (double)sn);
      tab32[at + k] = mk((float)cs, (float)sn);
      // e^{i a} - 1 = -2 sin(a/2)^2 + i sin a: no cancellation at small k
      const long double sh = sinl(pi * k / q.P[a]);
      const long double dr = -2.0L * sh * sh / r->h, di = -sn / r->h;
      tab[sum + at + k] = mk((double)dr, (double)di);
      tab32[sum + at + k] = mk((float)dr, (float)di);
    }
  chk(hipMemcpy(r->tables, tab.data(), tab.size() * sizeof(c64), hipMemcpyHostToDevice));
  chk(hipMemcpy(r->alpha, faces.data(), faces.size() * sizeof(double), hipMemcpyHostToDevice));
  double s_re, s_im;
  cube_green_integral(k0, r->h, &s_re, &s_im);
  const void* tw[3] = {r->tw[0], r->tw[1], r->tw[2]};
  if (e == hipSuccess) {
    k_rt_green<<<blocks_for(M), kRtThreads, 0, r->stream>>>(work, q, r->h, k0, s_re, s_im);
    chk(hipGetLastError());
  }
  if (e == hipSuccess) chk(launch_fft3d_full(work, tmp, r->g, tw, r->stream));
  if (e == hipSuccess) {
    k_rt_octant<<<blocks_for(noct), kRtThreads, 0, r->stream>>>(tmp, r->ghat, r->ghat32, q,
                                                                1.0 / (double)M);
    chk(hipGetLastError());
  }
  if (e == hipSuccess) chk(hipStreamSynchronize(r->stream));
  if (e != hipSuccess) return VIE_EDEVICE;
  *out = hold.release();
  return VIE_OK;
} VIE_CATCH

extern "C" int vie_rt_grid(const vie_rt* r, int32_t* ext, int32_t* fft) {
  if (!r) return VIE_EINVAL;
  for (int a = 0; a < 3; ++a) {
    if (ext) ext[a] = r->q.E[a];
    if (fft) fft[a] = r->q.P[a];
  }
  return VIE_OK;
}

extern "C" int vie_rt_matvec(vie_rt* r, const vie_c64* x, vie_c64* y, int32_t nvec,
                             int32_t precision) try {
  if (!r || !x || !y || nvec < 1 || (precision != VIE_FP64 && precision != VIE_MIXED))
    return VIE_EINVAL;
  if (r->poisoned) return VIE_ESTATE;
  const RtDevice on(r->dev);
  const int64_t n = 3 * r->q.m;
  c64 *dx = r->w.vecs, *dy = dx + n;
  for (int v = 0; v < nvec; ++v) {
    RT_HIP(hipMemcpyAsync(dx, x + v * n, n * sizeof(c64), hipMemcpyHostToDevice, r->stream));
    RT_TRY(rt_apply(r, dx, dy, 1, precision == VIE_MIXED));
    RT_HIP(r->stage.to_host(y + v * n, dy, n * sizeof(c64), r->stream));
  }
  return VIE_OK;
} VIE_CATCH

// Solves nc channels as one batch (host driver of the iteration): chunks of
// iterations run on the device, the host looks at the scalars once per chunk
// and, for every vector whose cycle ended, takes the true residual and
// restarts it from there unless it converged, hit the cap or took no step.
static int rt_solve_batch(vie_rt* r, const vie_planewave* inc, int nc, double tol, int max_iter,
                          bool mixed, vie_c64* w, vie_stats* stats, bool* all) {
  constexpr double kInnerTol = 1e-3;  // residual reduction per refinement cycle (mixed)
  constexpr int kChunk = 8;
  const RtGeom& q = r->q;
  const int64_t n = 3 * q.m;
  const auto t0 = std::chrono::steady_clock::now();
  c64* vec[8];
  for (int k = 0; k < 8; ++k) vec[k] = r->w.vecs + (int64_t)k * nc * n;
  c64 *x = vec[0], *b = vec[1], *rr = vec[2], *rh = vec[3], *p = vec[4], *v = vec[5], *s = vec[6],
      *t = vec[7];
  RtScal* sc = r->w.scal;
  int* active = r->w.active;
  int* mark = r->w.mark;
  c64 *pr = r->w.part[0], *pv = r->w.part[1], *pt = r->w.part[2];
  const int vb = vec_blocks(n);
  const int bi64 = xinv_blocks<double>(q), bi = mixed ? xinv_blocks<float>(q) : bi64;
  // a product's partials: folded first when every consumer would sum many
  auto fold = [&](c64* part, int& np, const int* act) -> c64* {
    if (np <= 512) return part;
    k_rt_fold<<<kRtFold * nc, 64, 0, r->stream>>>(part, np, r->w.fold, act);
    np = kRtFold;
    return r->w.fold;
  };
  std::vector<RtWave> hw(nc);
  for (int k = 0; k < nc; ++k)
    for (int a = 0; a < 3; ++a) {
      hw[k].k[a] = inc[k].khat[a];
      hw[k].p[a] = mk(inc[k].pol[a].re, inc[k].pol[a].im);
    }
  RT_HIP(hipMemcpyAsync(r->w.wave, hw.data(), nc * sizeof(RtWave), hipMemcpyHostToDevice,
                        r->stream));
  k_rt_rhs<<<vb * nc, kRtThreads, 0, r->stream>>>(b, x, rr, rh, p, v, r->chif, q, r->h,
                                                  r->origin[0], r->origin[1], r->origin[2], r->k0,
                                                  r->w.wave, vb, pr);
  k_rt_total<<<nc, kRtThreads, 0, r->stream>>>(pr, vb, r->w.total, nullptr);
  RT_HIP(hipGetLastError());
  std::vector<double> bb(nc), r2(nc);
  RT_HIP(hipMemcpyAsync(bb.data(), r->w.total, nc * sizeof(double), hipMemcpyDeviceToHost,
                        r->stream));
  RT_HIP(hipStreamSynchronize(r->stream));
  std::vector<RtScal> hs(nc);
  std::vector<int> run(nc), mk_(nc), it0(nc, 0);
  std::vector<vie_stats> st(nc);
  // the cycle's target: tol ||b||, and for a mixed solve no deeper than
  // kInnerTol times its starting residual (the FP32 products' accuracy)
  auto start_cycle = [&](int k, double r0, int it) {
    RtScal S;
    S.rho = S.rho1 = S.alpha = S.omega = mk(1.0, 0.0);
    S.tol2 = tol * tol * bb[k];
    if (mixed) S.tol2 = std::max(S.tol2, kInnerTol * kInnerTol * r0);
    S.it = it0[k] = it;
    S.max_it = max_iter;
    S.stop = 0;
    hs[k] = S;
    run[k] = 1;
    ++st[k].cycles;
  };
  for (int k = 0; k < nc; ++k) {
    st[k] = vie_stats{};
    st[k].rel_res_x0 = 1.0;
    st[k].rel_res = bb[k] > 0 ? 1.0 : 0.0;
    run[k] = 0;
    if (bb[k] > 0)
      start_cycle(k, bb[k], 0);
    else
      st[k].converged = 1;
  }
  auto any = [&]() { return std::find(run.begin(), run.end(), 1) != run.end(); };
  bool fresh = true;  // hs and run are newer than the device's copies
  while (any()) {
    if (fresh) {
      RT_HIP(hipMemcpyAsync(sc, hs.data(), nc * sizeof(RtScal), hipMemcpyHostToDevice, r->stream));
      RT_HIP(hipMemcpyAsync(active, run.data(), nc * sizeof(int), hipMemcpyHostToDevice,
                            r->stream));
      fresh = false;
    }
    for (int j = 0; j < kChunk; ++j) {
      k_rt_pupd<<<vb * nc, kRtThreads, 0, r->stream>>>(p, rr, v, sc, active, n, vb, pr, vb);
      RT_TRY(rt_apply(r, p, v, nc, mixed, kEpiRhv, rh, pv, active));
      int np = bi;
      const c64* fv = fold(pv, np, active);
      k_rt_supd<<<vb * nc, kRtThreads, 0, r->stream>>>(s, rr, v, sc, active, n, vb, fv, np);
      RT_TRY(rt_apply(r, s, t, nc, mixed, kEpiTs, nullptr, pt, active));
      np = bi;
      const c64* ft = fold(pt, np, active);
      k_rt_xrupd<<<vb * nc, kRtThreads, 0, r->stream>>>(x, rr, p, s, t, rh, sc, active, n, vb, ft,
                                                        np, pr);
      RT_HIP(hipGetLastError());
    }
    RT_HIP(hipMemcpyAsync(hs.data(), sc, nc * sizeof(RtScal), hipMemcpyDeviceToHost, r->stream));
    RT_HIP(hipStreamSynchronize(r->stream));
    bool ended = false;
    for (int k = 0; k < nc; ++k) {
      mk_[k] = run[k] && hs[k].stop != 0;
      ended |= mk_[k] != 0;
    }
    if (!ended) continue;
    // the true residual decides
    RT_HIP(hipMemcpyAsync(mark, mk_.data(), nc * sizeof(int), hipMemcpyHostToDevice, r->stream));
    RT_TRY(rt_apply(r, x, t, nc, false, kEpiRes, b, pt, mark));
    int np = bi64;
    const c64* ft = fold(pt, np, mark);
    k_rt_total<<<nc, kRtThreads, 0, r->stream>>>(ft, np, r->w.total, mark);
    RT_HIP(hipGetLastError());
    RT_HIP(hipMemcpyAsync(r2.data(), r->w.total, nc * sizeof(double), hipMemcpyDeviceToHost,
                          r->stream));
    RT_HIP(hipStreamSynchronize(r->stream));
    bool again = false;
    for (int k = 0; k < nc; ++k) {
      if (!mk_[k]) continue;
      const int it = hs[k].it;
      st[k].iters = it;
      st[k].matvecs += 2 * (it - it0[k]) + 1;
      st[k].rel_res = sqrt(r2[k]) / sqrt(bb[k]);
      st[k].converged = st[k].rel_res <= tol ? 1 : 0;
      run[k] = 0;
      if (st[k].converged)
        st[k].seconds =
            std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
      // the cap, or a cycle that could not take a single step, ends the solve
      if (st[k].converged || hs[k].stop == 3 || it == it0[k] || it >= max_iter) {
        mk_[k] = 0;
      } else {
        start_cycle(k, r2[k], it);
        again = true;
      }
    }
    if (again) {
      // the running vectors' scalars go back as they came
      RT_HIP(hipMemcpyAsync(mark, mk_.data(), nc * sizeof(int), hipMemcpyHostToDevice, r->stream));
      k_rt_restart<<<vb * nc, kRtThreads, 0, r->stream>>>(t, rr, rh, p, v, n, vb, pr, mark);
      RT_HIP(hipGetLastError());
      RT_HIP(hipStreamSynchronize(r->stream));  // mk_ is reused
      fresh = true;
    }
  }
  RT_HIP(r->stage.to_host(w, x, (size_t)nc * n * sizeof(c64), r->stream));
  for (int k = 0; k < nc; ++k) {
    if (stats) stats[k] = st[k];
    *all &= st[k].converged != 0;
  }
  return VIE_OK;
}

extern "C" int vie_rt_solve(vie_rt* r, const vie_planewave* inc, int32_t nrhs, double tol,
                            int32_t max_iter, int32_t precision, vie_c64* w, vie_stats* stats) try {
  TraceRange trace_("vie_rt_solve");
  if (!r || !inc || !w || nrhs < 1 || !(tol > 0) || !(tol < 1) || max_iter < 1 ||
      (precision != VIE_FP64 && precision != VIE_MIXED))
    return VIE_EINVAL;
  if (r->poisoned) return VIE_ESTATE;
  for (int k = 0; k < nrhs; ++k)
    for (int a = 0; a < 3; ++a)
      if (!std::isfinite(inc[k].khat[a]) || !std::isfinite(inc[k].pol[a].re) ||
          !std::isfinite(inc[k].pol[a].im))
        return VIE_EINVAL;
  const RtDevice on(r->dev);
  // channels per batch: 1 GB of y/z scratch, fewer where their workspace does
  // not fit (the iterates are the same)
  const RtGeom& q = r->q;
  const int64_t one = (int64_t)kRtFields * q.E[2] * q.P[1] * q.P[0] * sizeof(c64);
  int nb = (int)std::max<int64_t>(1, std::min<int64_t>(nrhs, ((int64_t)1 << 30) / one));
  while (nb > r->w.cap) {
    const hipError_t e = rt_reserve(r, nb);
    if (e == hipSuccess) break;
    if (e != hipErrorOutOfMemory) RT_HIP(e);
    nb = std::max(r->w.cap, nb / 2);
  }
  bool all = true;
  for (int k = 0; k < nrhs; k += nb)
    RT_TRY(rt_solve_batch(r, inc + k, std::min(nb, nrhs - k), tol, max_iter,
                          precision == VIE_MIXED, w + k * 3 * q.m, stats ? stats + k : nullptr,
                          &all));
  return all ? VIE_OK : VIE_ENOCONV;
} VIE_CATCH

extern "C" int vie_rt_farfield(vie_rt* r, const vie_c64* w, int32_t nrhs, const double* theta,
                               const double* phi, int32_t ndir, vie_c64* F) try {
  TraceRange trace_("vie_rt_farfield");
  if (!r || !w || !theta || !phi || !F || nrhs < 1 || ndir < 1) return VIE_EINVAL;
  if (r->poisoned) return VIE_ESTATE;
  for (int d = 0; d < ndir; ++d)
    if (!std::isfinite(theta[d]) || !std::isfinite(phi[d])) return VIE_EINVAL;
  if ((int64_t)nrhs * ndir > (int64_t)1 << 30) return VIE_EINVAL;
  const RtDevice on(r->dev);
  // Component i of cell c is its face c + e_i / 2: the voxel contraction over
  // the cells with an active face, weights alpha, and one half-cell phase per
  // component and direction at the end (a direct sum over the faces took
  // 71 ms for a 180 x 360 sweep of two channels on the 64^3 sphere).
  const int64_t n = 3 * r->q.m;
  const int nc = (int)r->cells.size();
  if (nc == 0) {
    memset(F, 0, (size_t)nrhs * ndir * 2 * sizeof(vie_c64));
    return VIE_OK;
  }
  hipError_t e = hipSuccess;
  auto chk = [&](hipError_t x) {
    if (e == hipSuccess) e = x;
    return e == hipSuccess;
  };
  auto up = [&](RtBuf& d, const std::vector<int>& v) {
    if (chk(d.reserve(std::max<size_t>(v.size(), 1) * sizeof(int))) && !v.empty())
      chk(hipMemcpyAsync(d.p, v.data(), v.size() * sizeof(int), hipMemcpyHostToDevice, r->stream));
  };
  FarGroups gr;
  bool sweep = 1.25 * ndir * (double)nc > 3e7 && far_groups(theta, ndir, gr);
  if (sweep) {
    if (!r->far_columns) {
      far_columns_build(r->cells.data(), nc, r->q.E, r->fc);
      for (size_t k = 0; k < r->fc.ent.size(); k += 2) r->fc.ent[k] = r->cells[r->fc.ent[k]];
      up(r->cptr, r->fc.ptr);
      up(r->corg, r->fc.org);
      up(r->cent, r->fc.ent);
      r->far_columns = e == hipSuccess;
    }
    sweep = far_by_columns(gr, ndir, r->fc, nc);
  }
  if (!sweep && !r->far_blocks) {
    far_blocks_build(r->cells.data(), nc, r->q.E, r->fb);
    for (int& v : r->fb.vi) v = v < 0 ? v : r->cells[v];
    up(r->fvi, r->fb.vi);
    up(r->forg, r->fb.org);
    r->far_blocks = e == hipSuccess;
  }
  // right-hand sides per upload: 256 MB of currents and of results
  const int64_t each = std::max<int64_t>(n, (int64_t)ndir * 2) * (int64_t)sizeof(c64);
  const int per =
      (int)std::max<int64_t>(1, std::min<int64_t>(nrhs, ((int64_t)256 << 20) / each));
  FarPlan pl;
  FarSweepPlan sp;
  std::vector<int> idx;
  if (sweep) {
    sp = far_sweep_plan(gr, r->fc, per, ndir);
    idx = gr.tile;
    idx.insert(idx.end(), gr.perm.begin(), gr.perm.end());
    idx.insert(idx.end(), gr.first.begin(), gr.first.end());
    up(r->fidx, idx);
  } else {
    pl = far_plan(r->fb, per, ndir);
  }
  std::vector<double> in((size_t)2 * ndir + per);
  memcpy(in.data(), theta, ndir * sizeof(double));
  memcpy(in.data() + ndir, phi, ndir * sizeof(double));
  for (int q = 0; q < per; ++q) {
    const int64_t off = q * n;
    memcpy(&in[(size_t)2 * ndir + q], &off, sizeof(off));
  }
  const int* perm = nullptr;
  if (chk(r->fin.reserve(in.size() * sizeof(double))) &&
      chk(r->fdirs.reserve((size_t)ndir * 9 * sizeof(double))) &&
      chk(r->fw.reserve((size_t)per * n * sizeof(c64))) &&
      chk(r->fwd.reserve((sweep ? sp.wd : pl.wd) * sizeof(c64))) &&
      chk(r->fpart.reserve((sweep ? sp.part : pl.part) * sizeof(c64))) &&
      chk(r->fF.reserve((size_t)per * ndir * 2 * sizeof(c64))) &&
      chk(hipMemcpyAsync(r->fin.p, in.data(), in.size() * sizeof(double), hipMemcpyHostToDevice,
                         r->stream))) {
    if (sweep) perm = r->fidx.as<int>() + gr.tile.size();
    chk(launch_far_frames(r->fin.as<double>(), perm, ndir, r->fdirs.as<double>(), r->stream));
  }
  const FarSrc src = {r->fw.as<c64>(), (const int64_t*)(r->fin.as<double>() + 2 * (size_t)ndir),
                      r->q.m, r->alpha};
  const FarGeom geo = far_geom(r->k0, r->h, r->origin, 1, r->q.E, 0.5 * r->h);
  for (int q0 = 0; q0 < nrhs && e == hipSuccess; q0 += per) {
    const int nq = std::min(per, nrhs - q0);
    chk(hipMemcpyAsync(r->fw.p, w + q0 * n, (size_t)nq * n * sizeof(c64), hipMemcpyHostToDevice,
                       r->stream));
    if (e == hipSuccess) {
      if (sweep)
        chk(launch_farfield_sweep(src, nq, r->fc, r->cptr.as<int>(), r->corg.as<int>(),
                                  r->cent.as<int>(), gr, perm, perm + gr.perm.size(),
                                  r->fidx.as<int>(), sp, r->fdirs.as<double>(), ndir, r->q.E[2],
                                  geo, r->fwd.as<c64>(), r->fpart.as<c64>(), r->fF.as<c64>(),
                                  r->stream));
      else
        chk(launch_farfield_mfma(src, nq, r->fb, r->fvi.as<int>(), r->forg.as<int>(), pl,
                                 r->fdirs.as<double>(), ndir, geo, r->fwd.as<c64>(),
                                 r->fpart.as<c64>(), r->fF.as<c64>(), r->stream));
    }
    if (e == hipSuccess)
      chk(r->stage.to_host(F + (int64_t)q0 * ndir * 2, r->fF.p,
                           (size_t)nq * ndir * 2 * sizeof(c64), r->stream));
  }
  if (e != hipSuccess) {
    if (e == hipErrorOutOfMemory) return VIE_ENOMEM;
    r->poisoned = true;
    return VIE_EDEVICE;
  }
  return VIE_OK;
} VIE_CATCH

extern "C" void vie_rt_destroy(vie_rt* r) {
  if (!r) return;
  if (r->stream) (void)hipStreamSynchronize(r->stream);
  rt_free(r);
  delete r;
}
