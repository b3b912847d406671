// Fused x and y passes of the packed-FP16 products (see "approximate
// products" in fft_passes.hip) on the matrix cores: one workgroup per
// (right-hand side, component, z) plane.
//
// Both transforms of a plane are small dense products with the DFT matrix,
// the zero half of each line left out and the mirror pairs k, -k sharing
// their sums:
//
//   forward  P = C re, Q = S im, R = C im, T = S re  over n < H = P / 2, then
//            X[j] = (P + Q) + i (R - T), X[-j] = (P - Q) + i (R + T), j < H
//   inverse  E = X[j] + X[-j], O = X[j] - X[-j]  over j < H, then
//            x[n] = C E + i S O, n < H
//
// with C, S = cos, sin(2 pi j n / P).  S row 0 is zero: the slot carries
// X[H] = sum (-1)^n x[n] instead.
//
// The x transforms are FP32 transforms of values with at most 11 significant
// bits (a bfloat16 vector times 2^14, or the FP16 plane): the products with
// C and S split into two halves each (hi + lo, 2^-25 off) are exact and are
// summed in FP32.  The y transforms are FP16 transforms: FP16 operands, FP32
// sums, one rounding at the end.
//
// A plane is a scatter, 64 matrix instructions a wave and one store (the
// inverse: loads, 128 and the compressed epilogue); what bounds it is the
// y/z scratch in HBM.  The Stockham transforms of the same passes spent twice
// that on LDS exchanges and vector arithmetic.
#include "fft_common.h"

namespace vie {

typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

// Operand tables.  Set of length P: planes C hi, C lo, S hi, S lo, S hi with
// the X[H] row, each [tile of 32][step of 16 k][lane][8]: row (column) tile
// 32 + lane % 32, k = 16 step + 8 (lane / 32) + e, zero beyond H.  Then the
// set of the inverse y transform: planes C, S with the X[H] column, each
// [tile of 16][step of 32 k][lane][8].
template <int P>
struct Dft16 {
  static constexpr int H = P / 2;
  static constexpr int T = (H + 31) / 32, K = H / 16;
  static constexpr int PLANE = T * K * 64;  // half8 entries
  static constexpr int SET = 5 * PLANE;
  static constexpr int TI = H / 16, KI = (H + 31) / 32;
  static constexpr int PLANE_I = TI * KI * 64;
};
enum { kChi = 0, kClo = 1, kShi = 2, kSlo = 3, kSx = 4 };

size_t xy16_table_bytes(const GroupGeom& g) {
  auto set = [](int P) { return (size_t)5 * ((P / 2 + 31) / 32) * (P / 32) * 64; };
  const int H2 = g.P[1] / 2;
  return (set(g.P[0]) + set(g.P[1]) + (size_t)2 * (H2 / 16) * ((H2 + 31) / 32) * 64) *
         sizeof(half8);
}

__device__ static double dft_entry(int sin_, int j, int n, int P) {
  double s, c;
  sincospi(2.0 * ((j * n) % P) / P, &s, &c);
  return sin_ ? s : c;
}

// set of length P (inv: the inverse y set), one value per thread
__global__ void k_dft16_table(_Float16* out, int P, int inv) {
  const int H = P / 2;
  const int tile = inv ? 16 : 32, step = inv ? 32 : 16;
  const int T = (H + tile - 1) / tile, K = (H + step - 1) / step;
  const int plane = T * K * 512, total = (inv ? 2 : 5) * plane;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < total; i += gridDim.x * blockDim.x) {
    const int pl = i / plane, r = i % plane;
    const int e = r & 7, lane = (r >> 3) & 63, ks = (r >> 9) % K, t = (r >> 9) / K;
    const int row = t * tile + lane % tile, k = ks * step + 8 * (lane / tile) + e;
    double v = 0.0;
    if (row < H && k < H) {
      if (inv)
        v = pl == 0 ? dft_entry(0, row, k, P)
                    : (k == 0 ? (row & 1 ? -1.0 : 1.0) : dft_entry(1, row, k, P));
      else if (pl == kSx && row == 0)
        v = k & 1 ? -1.0 : 1.0;
      else
        v = dft_entry(pl >= kShi, row, k, P);
    }
    const _Float16 hi = (_Float16)v;
    out[i] = !inv && (pl == kClo || pl == kSlo) ? (_Float16)(v - (double)hi) : hi;
  }
}

hipError_t launch_xy16_tables(void* tab, const GroupGeom& g, hipStream_t s) {
  auto set = [](int P) { return (size_t)5 * ((P / 2 + 31) / 32) * (P / 32) * 512; };
  _Float16* t = (_Float16*)tab;
  k_dft16_table<<<32, 256, 0, s>>>(t, g.P[0], 0);
  t += set(g.P[0]);
  k_dft16_table<<<32, 256, 0, s>>>(t, g.P[1], 0);
  t += set(g.P[1]);
  k_dft16_table<<<32, 256, 0, s>>>(t, g.P[1], 1);
  return hipGetLastError();
}

struct Xy16Args {
  int N1, N2, N3, zl;
  int row, zls;       // y/z scratch strides in packed pairs
  int64_t zhs, cs, rs;
  const half8* tab;
};

__device__ __forceinline__ f32x16 mma32(half8 a, half8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 mma16(half8 a, half8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ unsigned pack_c(float re, float im) {
  return __builtin_bit_cast(unsigned, h2{(_Float16)re, (_Float16)im});
}
// voxel v < 64 N1 of a plane: its row (inv = ceil(2^20 / N1))
__device__ __forceinline__ int plane_row(int v, unsigned inv) {
  return (int)(((unsigned)v * inv) >> 20);
}

// NRM: the input is an FP32 work vector, normalised per right-hand side
// (see MatvecArgs::npart) into the bfloat16 vector vout on the way in.
template <int P1, int P2, bool NRM>
__global__ __launch_bounds__(256, 3) void k_fft_xy_fwd_h2(
    const void* __restrict__ xcv, cpx<h2>* __restrict__ B, BodyIdx bi, Xy16Args a, float hs1,
    float hs2, const int* __restrict__ active, const double* __restrict__ npart, int nblk,
    double* __restrict__ nrm, int ldn, cb16* __restrict__ vout) {
  using TXI = typename std::conditional<NRM, c32, cb16>::type;
  using D1 = Dft16<P1>;
  using D2 = Dft16<P2>;
  constexpr int H1 = D1::H, H2 = D2::H;
  constexpr int XS = H1 + 8, FS = H2 + 8;  // rows 16 bytes apart in the banks
  constexpr int XP = D2::T * 32 * XS, FP = P1 * FS;
  static_assert(XP <= FP, "the input plane lies inside the transformed one");
  // [re, im][y][x] of the input, then [re, im][x frequency][y]
  __shared__ __align__(16) _Float16 buf[2 * FP];
  const int nrhs = gridDim.x / (3 * a.N3);
  const int rhs = blockIdx.x % nrhs, cz = blockIdx.x / nrhs;
  if (active && !active[rhs]) return;
  const int comp = cz / a.N3, z = cz % a.N3;
  const int body = bi.rhs_body[rhs];
  const int nb = bi.nb[body];
  const int* vox = bi.vox + bi.voff[body];
  const int* lp = bi.line_ptr + (int64_t)body * (a.N2 * a.N3 + 1) + z * a.N2;
  const int k0 = lp[0], k1 = lp[a.N2];  // the plane's voxels
  const TXI* xv = reinterpret_cast<const TXI*>(xcv) + bi.roff[rhs] + (int64_t)comp * nb;
  cb16* vo = NRM ? vout + bi.roff[rhs] + (int64_t)comp * nb : nullptr;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l32 = lane & 31, half = lane >> 5;
  {
    // at most H1 H2 voxels, NB a thread per round
    constexpr int NB = H1 * H2 / 256 < 8 ? H1 * H2 / 256 : 8;
    int kv[NB];
    TXI xr[NB];
    auto fetch = [&](int kb) {
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        const int k = kb + i * 256;
        if (k < k1) {
          kv[i] = vox[k];
          xr[i] = xv[k];
        }
      }
    };
    fetch(k0 + tid);
    for (int i = tid; i < 2 * XP / 8; i += 256)
      reinterpret_cast<u32x4*>(buf)[i] = u32x4{0, 0, 0, 0};
    double sc = 1.0;
    if constexpr (NRM) {
      // ||w||^2 of this right-hand side: every wave sums the partials in the
      // order of the separate reduction (lane-strided, then a fixed butterfly)
      double t2 = 0.0;
      for (int k = lane; k < nblk; k += 64) t2 += npart[(int64_t)rhs * nblk + k];
      for (int mk = 32; mk >= 1; mk >>= 1) t2 += __shfl_xor(t2, mk);
      sc = t2 > 0.0 ? 1.0 / sqrt(t2) : 0.0;
      if (comp == 0 && z == 0 && tid == 0) nrm[(int64_t)rhs * ldn] = t2;
    }
    const unsigned inv = ((1u << 20) + a.N1 - 1) / a.N1;
    const int base = z * a.N2 * a.N1;
    lds_barrier();
    for (int kb = k0 + tid; kb < k1; kb += NB * 256) {
      if (kb != k0 + tid) fetch(kb);
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        const int k = kb + i * 256;
        if (k >= k1) continue;
        c32 v;
        if constexpr (NRM) {
          // the basis vector as stored (bfloat16 through FP32) is what is multiplied
          const c64 wn = sc * cvt<double>(xr[i]);
          cb16 b16;
          b16.re = (__bf16)(float)wn.re;
          b16.im = (__bf16)(float)wn.im;
          vo[k] = b16;
          v = cvt<float>(b16);
        } else {
          v = cvt<float>(xr[i]);
        }
        // |v| <= 1: times 2^14 the 8 bits of every |v| >= 2^-31 fit FP16
        const int vx = kv[i] - base, y = plane_row(vx, inv), x = vx - y * a.N1;
        buf[y * XS + x] = (_Float16)(v.re * 16384.f);
        buf[XP + y * XS + x] = (_Float16)(v.im * 16384.f);
      }
    }
  }
  lds_barrier();
  {  // x: wave = (32 rows, 32 frequency pairs)
    const int mt = wave % D2::T, nt = wave / D2::T;
    f32x16 p = 0.f, q = 0.f, r = 0.f, t = 0.f;
    if (nt < D1::T) {
      const half8* tb = a.tab + nt * D1::K * 64 + lane;
      const _Float16* ar = buf + (mt * 32 + l32) * XS + 8 * half;
#pragma unroll
      for (int ks = 0; ks < D1::K; ++ks) {
        const half8 re = *reinterpret_cast<const half8*>(ar + ks * 16);
        const half8 im = *reinterpret_cast<const half8*>(ar + XP + ks * 16);
        const half8 ch = tb[kChi * D1::PLANE + ks * 64], cl = tb[kClo * D1::PLANE + ks * 64];
        const half8 sh = tb[kSx * D1::PLANE + ks * 64], sl = tb[kSlo * D1::PLANE + ks * 64];
        p = mma32(re, ch, p);
        q = mma32(im, sh, q);
        r = mma32(im, ch, r);
        t = mma32(re, sh, t);
        p = mma32(re, cl, p);
        q = mma32(im, sl, q);
        r = mma32(im, cl, r);
        t = mma32(re, sl, t);
      }
    }
    lds_barrier();  // every wave has read the input plane
    const int j = nt * 32 + l32;
    if (nt < D1::T && j < H1) {
      const float sc = hs1 * (1.f / 16384.f);
      _Float16* lo = buf + j * FS;
      _Float16* hi = buf + (j ? P1 - j : H1) * FS;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int y = mt * 32 + 8 * g + 4 * half;
        if (y >= H2) continue;
        half4 lr, li, hr, hi4;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float P = p[4 * g + i], Q = q[4 * g + i], R = r[4 * g + i], T = t[4 * g + i];
          lr[i] = (_Float16)(sc * (j ? P + Q : P));
          li[i] = (_Float16)(sc * (j ? R - T : R));
          hr[i] = (_Float16)(sc * (j ? P - Q : T));
          hi4[i] = (_Float16)(sc * (j ? R + T : Q));
        }
        *reinterpret_cast<half4*>(lo + y) = lr;
        *reinterpret_cast<half4*>(lo + FP + y) = li;
        *reinterpret_cast<half4*>(hi + y) = hr;
        *reinterpret_cast<half4*>(hi + FP + y) = hi4;
      }
    }
  }
  lds_barrier();
  // y: an item is 32 columns and 32 row pairs; neighbouring lanes hold
  // neighbouring columns, one exchange packs them (the even lane stores the
  // first of two rows, the odd lane the second)
  constexpr int NT = P1 / 32;
  const half8* ty = a.tab + D1::SET + lane;
  cpx<h2>* po = B + rhs * a.rs + comp * a.cs + (z / a.zl) * a.zhs + (z % a.zl) * a.zls;
  const int odd = lane & 1;
  for (int it = wave; it < NT * D2::T; it += 4) {
    const int nt = it % NT, mt = it / NT;
    f32x16 p = 0.f, q = 0.f, r = 0.f, t = 0.f;
    const _Float16* br = buf + (nt * 32 + l32) * FS + 8 * half;
    const half8* tb = ty + mt * D2::K * 64;
#pragma unroll
    for (int ks = 0; ks < D2::K; ++ks) {
      const half8 re = *reinterpret_cast<const half8*>(br + ks * 16);
      const half8 im = *reinterpret_cast<const half8*>(br + FP + ks * 16);
      const half8 c = tb[kChi * D2::PLANE + ks * 64], s = tb[kSx * D2::PLANE + ks * 64];
      p = mma32(c, re, p);
      q = mma32(s, im, q);
      r = mma32(c, im, r);
      t = mma32(s, re, t);
    }
    cpx<h2>* pc = po + ((nt * 32 + l32) >> 1);
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int j0 = mt * 32 + 8 * g + 4 * half;
      if (j0 >= H2) continue;
      unsigned lo[4], hi[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float P = p[4 * g + i], Q = q[4 * g + i], R = r[4 * g + i], T = t[4 * g + i];
        float lr = P + Q, li = R - T, hr = P - Q, hm = R + T;
        if (g == 0 && i == 0 && j0 == 0) {
          lr = P;
          li = R;
          hr = T;
          hm = Q;
        }
        lo[i] = pack_c(hs2 * lr, hs2 * li);
        hi[i] = pack_c(hs2 * hr, hs2 * hm);
      }
#pragma unroll
      for (int i = 0; i < 4; i += 2) {
        auto pair = [&](unsigned a0, unsigned a1) {
          const unsigned rc = (unsigned)__builtin_amdgcn_update_dpp(
              0, (int)(odd ? a0 : a1), 0xB1, 0xF, 0xF, false);  // lanes 2i <-> 2i + 1
          const unsigned L = odd ? rc : a0, R = odd ? a1 : rc;
          return u32x2{__builtin_amdgcn_perm(R, L, 0x05040100u),
                       __builtin_amdgcn_perm(R, L, 0x07060302u)};
        };
        const int j = j0 + i + odd;
        *reinterpret_cast<u32x2*>(pc + (int64_t)j * a.row) = pair(lo[i], lo[i + 1]);
        *reinterpret_cast<u32x2*>(pc + (int64_t)(j ? P2 - j : H2) * a.row) =
            pair(hi[i], hi[i + 1]);
      }
    }
  }
}

template <int P1, int P2>
__global__ __launch_bounds__(256, 3) void k_fft_yx_inv_h2(
    const cpx<h2>* __restrict__ B, const cb16* __restrict__ xin, c32* __restrict__ yout,
    BodyIdx bi, Xy16Args a, float hs, const int* __restrict__ active) {
  using D1 = Dft16<P1>;
  using D2 = Dft16<P2>;
  constexpr int H1 = D1::H, H2 = D2::H;
  constexpr int GS = P1 + 8, GP = D2::T * 32 * GS;
  constexpr int RS = H1 + 1;
  constexpr int BYTES = 2 * GP * 2 > H2 * RS * 8 ? 2 * GP * 2 : H2 * RS * 8;
  // [re, im][y][x frequency], then the plane's values [y][x] in FP32
  __shared__ __align__(16) char ubuf[BYTES];
  _Float16* buf = reinterpret_cast<_Float16*>(ubuf);
  c32* res = reinterpret_cast<c32*>(ubuf);
  const int nrhs = gridDim.x / (3 * a.N3);
  const int rhs = blockIdx.x % nrhs, cz = blockIdx.x / nrhs;
  if (active && !active[rhs]) return;
  const int comp = cz / a.N3, z = cz % a.N3;
  const int body = bi.rhs_body[rhs];
  const int nb = bi.nb[body];
  const int* vox = bi.vox + bi.voff[body];
  const double* chic = bi.chic + bi.voff[body];
  const int* lp = bi.line_ptr + (int64_t)body * (a.N2 * a.N3 + 1) + z * a.N2;
  const int k0 = lp[0], k1 = lp[a.N2];
  const int64_t vb = bi.roff[rhs] + (int64_t)comp * nb;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l32 = lane & 31, half = lane >> 5;
  const int l16 = lane & 15, quad = lane >> 4;
  if (wave < P1 / 32) {  // inverse y: a wave takes 16 column pairs, all rows
    const cpx<h2>* pin = B + rhs * a.rs + comp * a.cs + (z / a.zl) * a.zhs +
                         (z % a.zl) * a.zls + wave * 16 + l16;
    const half8* ti = a.tab + D1::SET + D2::SET + lane;
    f32x4 er[D2::TI], ei[D2::TI], dr[D2::TI], di[D2::TI];  // even, odd columns
#pragma unroll
    for (int t = 0; t < D2::TI; ++t) er[t] = ei[t] = dr[t] = di[t] = 0.f;
#pragma unroll
    for (int ks = 0; ks < D2::KI; ++ks) {
      const int jb = ks * 32 + 8 * quad;
      cpx<h2> lo[8], hi[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        // past H2 the table is zero: any row will do
        const int j = (H2 % 32 == 0 || jb < H2) ? jb + e : 0;
        lo[e] = pin[(int64_t)j * a.row];
        hi[e] = pin[(int64_t)(j ? P2 - j : H2) * a.row];
      }
      unsigned ere[8], eim[8], ore[8], oim[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        h2 sr = lo[e].re + hi[e].re, si = lo[e].im + hi[e].im;
        h2 dre = lo[e].re - hi[e].re, dim = hi[e].im - lo[e].im;
        if (ks == 0 && e == 0 && quad == 0) {
          sr = lo[e].re;
          si = lo[e].im;
          dre = hi[e].im;
          dim = hi[e].re;
        }
        ere[e] = __builtin_bit_cast(unsigned, sr);
        eim[e] = __builtin_bit_cast(unsigned, si);
        ore[e] = __builtin_bit_cast(unsigned, dre);
        oim[e] = __builtin_bit_cast(unsigned, dim);
      }
      auto column = [](const unsigned (&v)[8], unsigned sel) {
        u32x4 o;
#pragma unroll
        for (int d = 0; d < 4; ++d) o[d] = __builtin_amdgcn_perm(v[2 * d + 1], v[2 * d], sel);
        return __builtin_bit_cast(half8, o);
      };
      const half8 ere0 = column(ere, 0x05040100u), ere1 = column(ere, 0x07060302u);
      const half8 eim0 = column(eim, 0x05040100u), eim1 = column(eim, 0x07060302u);
      const half8 ore0 = column(ore, 0x05040100u), ore1 = column(ore, 0x07060302u);
      const half8 oim0 = column(oim, 0x05040100u), oim1 = column(oim, 0x07060302u);
#pragma unroll
      for (int t = 0; t < D2::TI; ++t) {
        const half8 c = ti[(t * D2::KI + ks) * 64], s = ti[D2::PLANE_I + (t * D2::KI + ks) * 64];
        er[t] = mma16(ere0, c, er[t]);
        ei[t] = mma16(eim0, c, ei[t]);
        dr[t] = mma16(ere1, c, dr[t]);
        di[t] = mma16(eim1, c, di[t]);
        er[t] = mma16(oim0, s, er[t]);
        ei[t] = mma16(ore0, s, ei[t]);
        dr[t] = mma16(oim1, s, dr[t]);
        di[t] = mma16(ore1, s, di[t]);
      }
    }
#pragma unroll
    for (int t = 0; t < D2::TI; ++t) {
      half8 re, im;  // four neighbouring pairs of row 16 t + l16
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        re[2 * i] = (_Float16)er[t][i];
        re[2 * i + 1] = (_Float16)dr[t][i];
        im[2 * i] = (_Float16)ei[t][i];
        im[2 * i + 1] = (_Float16)di[t][i];
      }
      _Float16* o = buf + (t * 16 + l16) * GS + 2 * (wave * 16 + 4 * quad);
      *reinterpret_cast<half8*>(o) = re;
      *reinterpret_cast<half8*>(o + GP) = im;
    }
  }
  lds_barrier();
  {  // inverse x in FP32: wave = (32 rows, 32 points)
    const int mt = wave % D2::T, nt = wave / D2::T;
    f32x16 r1 = 0.f, r2 = 0.f, im = 0.f;
    if (nt < D1::T) {
      const half8* tb = a.tab + nt * D1::K * 64 + lane;
      const _Float16* ar = buf + (mt * 32 + l32) * GS + 8 * half;
      const unsigned flip = lane & 1 ? 0x80008000u : 0u;  // e^{i pi x} of frequencies >= H1
      auto flipped = [&](half8 v) {
        return __builtin_bit_cast(half8, __builtin_bit_cast(u32x4, v) ^ u32x4{flip, flip, flip, flip});
      };
#pragma unroll
      for (int ks = 0; ks < D1::K; ++ks) {
        half8 ch = tb[kChi * D1::PLANE + ks * 64], cl = tb[kClo * D1::PLANE + ks * 64];
        half8 sh = tb[kShi * D1::PLANE + ks * 64], sl = tb[kSlo * D1::PLANE + ks * 64];
#pragma unroll
        for (int up = 0; up < 2; ++up) {
          const half8 gr = *reinterpret_cast<const half8*>(ar + up * H1 + ks * 16);
          const half8 gi = *reinterpret_cast<const half8*>(ar + GP + up * H1 + ks * 16);
          if (up) {
            ch = flipped(ch);
            cl = flipped(cl);
            sh = flipped(sh);
            sl = flipped(sl);
          }
          r1 = mma32(gr, ch, r1);
          r2 = mma32(gi, sh, r2);
          im = mma32(gi, ch, im);
          r1 = mma32(gr, cl, r1);
          r2 = mma32(gi, sl, r2);
          im = mma32(gr, sh, im);
          im = mma32(gi, cl, im);
          im = mma32(gr, sl, im);
        }
      }
    }
    lds_barrier();  // every wave has read the plane
    const int x = nt * 32 + l32;
    if (nt < D1::T && x < H1) {
#pragma unroll
      for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int y = mt * 32 + 8 * g + 4 * half + i;
          if (y < H2) res[y * RS + x] = mk<float>(r1[4 * g + i] - r2[4 * g + i], im[4 * g + i]);
        }
    }
  }
  lds_barrier();
  // the compressed epilogue
  const unsigned inv = ((1u << 20) + a.N1 - 1) / a.N1;
  const int base = z * a.N2 * a.N1;
#pragma unroll 4
  for (int k = k0 + tid; k < k1; k += 256) {
    const int vx = vox[k] - base, y = plane_row(vx, inv), x = vx - y * a.N1;
    const c64 conv = (double)hs * cvt<double>(res[y * RS + x]);
    const c64 r = cvt<double>(xin[vb + k]) - chic[k] * conv;
    yout[vb + k] = cvt<float>(r);
  }
}

// The fused x-y passes take FFT lengths 64, 96 and 128 along x and y.
static bool xy_len_ok(int p) { return p == 64 || p == 96 || p == 128; }
bool xy_fused_ok(const GroupGeom& g) { return xy_len_ok(g.P[0]) && xy_len_ok(g.P[1]); }

#define VIE_DISPATCH_XY(P_, CALL)                    \
  switch (P_) {                                      \
    case 64: { constexpr int PP = 64; CALL; break; } \
    case 96: { constexpr int PP = 96; CALL; break; } \
    case 128: { constexpr int PP = 128; CALL; break; } \
    default: return hipErrorInvalidValue;            \
  }

static bool xy16_args(const MatvecArgs& m, Xy16Args* a) {
  const GroupGeom& g = *m.g;
  if (!xy_fused_ok(g) || !m.dft16 || !m.bi) return false;
  for (int d = 0; d < 2; ++d)
    if (g.N[d] < 1 || 2 * g.N[d] > g.P[d]) return false;
  a->N1 = g.N[0];
  a->N2 = g.N[1];
  a->N3 = g.N[2];
  a->zl = z_block(g);
  a->row = a->zl * g.P[0] / 2;
  a->zls = g.P[0] / 2;
  a->zhs = (int64_t)g.P[1] * a->row;
  a->cs = a->zhs * ((g.N[2] + a->zl - 1) / a->zl);
  a->rs = 3 * a->cs;
  a->tab = (const half8*)m.dft16;
  return true;
}

// m.npart set: normalising FP32 input (see MatvecArgs), else bfloat16 input
hipError_t xy_fwd_h2(const MatvecArgs& m, const void* xc, void* B, hipStream_t s) {
  const GroupGeom& g = *m.g;
  Xy16Args a;
  if (!xy16_args(m, &a)) return hipErrorInvalidValue;
  const dim3 grid(g.nrhs * 3 * g.N[2]);
  VIE_DISPATCH_XY(g.P[0], ({
                    constexpr int Q1 = PP;
                    VIE_DISPATCH_XY(g.P[1], ({
                                      if (m.npart)
                                        k_fft_xy_fwd_h2<Q1, PP, true><<<grid, 256, 0, s>>>(
                                            xc, (cpx<h2>*)B, *m.bi, a, m.hs[0], m.hs[1], m.active,
                                            m.npart, m.nblk, m.nrm, m.ldn, (cb16*)m.vout);
                                      else
                                        k_fft_xy_fwd_h2<Q1, PP, false><<<grid, 256, 0, s>>>(
                                            xc, (cpx<h2>*)B, *m.bi, a, m.hs[0], m.hs[1], m.active,
                                            nullptr, 0, nullptr, 0, nullptr);
                                    }));
                  }));
  return hipGetLastError();
}

hipError_t yx_inv_h2(const MatvecArgs& m, const void* B, const void* x, void* y, hipStream_t s) {
  const GroupGeom& g = *m.g;
  Xy16Args a;
  if (!xy16_args(m, &a)) return hipErrorInvalidValue;
  const dim3 grid(g.nrhs * 3 * g.N[2]);
  VIE_DISPATCH_XY(g.P[0], ({
                    constexpr int Q1 = PP;
                    VIE_DISPATCH_XY(g.P[1], (k_fft_yx_inv_h2<Q1, PP><<<grid, 256, 0, s>>>(
                                                (const cpx<h2>*)B, (const cb16*)x, (c32*)y, *m.bi,
                                                a, m.hout, m.active)));
                  }));
  return hipGetLastError();
}
#undef VIE_DISPATCH_XY

}  // namespace vie
