// Packed-FP16 products (see "approximate products" in fft_passes.hip) of short
// lines on the matrix cores, in three passes over an FP16 scratch of the
// x-transformed field, [rhs][component][z][x frequency][re, im][y] (one row of
// padding per plane: without it a column's rows are 32 KB apart and share one
// memory channel):
//
//   x      one (right-hand side, component, z) plane per workgroup: scatter,
//          x transform, store
//   y-z    one (right-hand side, x frequency) column of all three components:
//          y and z transforms, the spectrum, the inverse z and y transforms,
//          in place; the doubled y and z lines live in LDS and registers only
//   x      back, and the compressed epilogue y = x - chi conv
//
// Every transform is a small dense product with the DFT matrix, the zero half
// of a line left out and the mirror pairs k, -k sharing their sums:
//
//   forward  P = C re, Q = S im, R = C im, T = S re  over n < H = P / 2, then
//            X[j] = (P + Q) + i (R - T), X[-j] = (P - Q) + i (R + T), j < H
//   inverse  E = X[j] + X[-j], O = X[j] - X[-j]  over j < H, then
//            x[n] = C E + i S O, n < H
//
// with C, S = cos, sin(2 pi j n / P).  S row 0 is zero: the slot carries
// X[H] = sum (-1)^n x[n] instead.  (Where the two halves of a line would have
// to be brought together first -- the inverse x and y -- the sum runs over
// all P frequencies.)
//
// The x transforms are FP32 transforms of values with at most 11 significant
// bits (a bfloat16 vector times 2^14, or the FP16 plane): the products with
// C and S split into two halves each (hi + lo, 2^-25 off) are exact and are
// summed in FP32, 6e-8 to 7e-8 off the 64-bit transform for P = 64 to 128
// (FP32 Stockham stages: 6e-8 to 8e-8).  The input is a vector of the block
// solves' basis, of norm 1 in whichever form it comes: no entry reaches the 4
// at which 2^14 times it overflows (the forward scales rest on the norm as
// well).  Entries below 2^-31 keep 2^-39 instead of their 8 bits, at most 2^-33 in
// a sum of 64, whose result is rounded to FP16 at the scale 1/8: 2^-36 against
// half of that format's smallest step, 2^-25.  The y and z transforms are FP16
// transforms: FP16 operands, FP32 sums, one rounding per transform.
#include "fft_common.h"

namespace vie {

typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

// Operand tables.  x: planes C hi, C lo, S hi, S lo, S hi with the X[H] row,
// each [tile of 32][step of 16 k][lane][8]: row (column) tile 32 + lane % 32,
// k = 16 step + 8 (lane / 32) + e, zero beyond H.
template <int P>
struct Dft16 {
  static constexpr int H = P / 2;
  static constexpr int T = (H + 31) / 32, K = H / 16;
  static constexpr int PLANE = T * K * 64;  // half8 entries
};
enum { kChi = 0, kClo = 1, kShi = 2, kSlo = 3, kSx = 4 };

// y and z: planes C, S each [tile of 16][step of 32 k][lane][8], row tile 16 +
// lane % 16, k = 32 step + 8 (lane / 16) + e:
//   y forward, z forward  row = frequency (S row 0: the X[H] row), k = point,
//                         times the pass's scale (a power of two), zero beyond
//                         the grid's points: what the operand holds there
//                         need only be finite
//   z inverse             row = point, k = frequency (S column 0: X[H]) in the
//                         order the spectrum stage leaves them: 4 (lane / 16)
//                         + e, e < 4, of the step's first 16, then the next
//                         16; pairs count twice
//   y inverse             row = point, k = slot of the y frequencies: j, then H
//                         + j for -j, with P / 2 in the slot of -0
struct Yz16Tab {
  int yf, zf, zi, yi, end;  // first half8 entry of each set
};
__host__ __device__ constexpr Yz16Tab yz16_tab(int P2, int P3) {
  const int H2 = P2 / 2, H3 = P3 / 2;
  const int z = 2 * (H3 / 16) * ((H3 + 31) / 32) * 64;
  Yz16Tab t{0, 0, 0, 0, 0};
  t.zf = t.yf + 2 * (H2 / 16) * ((H2 + 31) / 32) * 64;
  t.zi = t.zf + z;
  t.yi = t.zi + z;
  t.end = t.yi + 2 * (H2 / 16) * (P2 / 32) * 64;
  return t;
}
static size_t x16_entries(int P) { return (size_t)5 * ((P / 2 + 31) / 32) * (P / 32) * 64; }

size_t dft16_table_bytes(const GroupGeom& g) {
  return (x16_entries(g.P[0]) + yz16_tab(g.P[1], g.P[2]).end) * sizeof(half8);
}

__device__ static double dft_entry(int sin_, int j, int n, int P) {
  double s, c;
  sincospi(2.0 * ((j * n) % P) / P, &s, &c);
  return sin_ ? s : c;
}

__global__ void k_dft16_x(_Float16* out, int P) {
  const int H = P / 2, T = (H + 31) / 32, K = H / 16;
  const int plane = T * K * 512, total = 5 * plane;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < total; i += gridDim.x * blockDim.x) {
    const int pl = i / plane, r = i % plane;
    const int e = r & 7, lane = (r >> 3) & 63, ks = (r >> 9) % K, t = (r >> 9) / K;
    const int row = t * 32 + lane % 32, k = ks * 16 + 8 * (lane / 32) + e;
    double v = 0.0;
    if (row < H && k < H)
      v = pl == kSx && row == 0 ? (k & 1 ? -1.0 : 1.0) : dft_entry(pl >= kShi, row, k, P);
    const _Float16 hi = (_Float16)v;
    out[i] = pl == kClo || pl == kSlo ? (_Float16)(v - (double)hi) : hi;
  }
}

enum { kFwd = 0, kInvPairs = 1, kInvAll = 2 };
__global__ void k_dft16_yz(_Float16* out, int P, int kind, int kmax, float scale) {
  const int H = P / 2;
  const int K = ((kind == kInvAll ? P : H) + 31) / 32, plane = H / 16 * K * 512;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < 2 * plane;
       i += gridDim.x * blockDim.x) {
    const int pl = i / plane, r = i % plane;
    const int e = r & 7, lane = (r >> 3) & 63, ks = (r >> 9) % K, t = (r >> 9) / K;
    const int row = t * 16 + lane % 16, q = lane / 16;
    const int k = ks * 32 + (kind == kInvPairs ? 4 * q + e % 4 + 16 * (e / 4) : 8 * q + e);
    double v = 0.0;
    if (k < kmax) {
      const int f = kind == kInvAll && k >= H ? (k == H ? H : P - (k - H)) : k;
      v = dft_entry(pl, row, f, P);
      if (pl && kind == kFwd && row == 0) v = k & 1 ? -1.0 : 1.0;
      if (pl && kind == kInvPairs && k == 0) v = row & 1 ? -1.0 : 1.0;
      if (kind == kInvPairs && k > 0) v *= 2.0;
    }
    out[i] = (_Float16)(v * scale);
  }
}

hipError_t launch_dft16_tables(void* tab, const GroupGeom& g, const float hs[3], hipStream_t s) {
  half8* t = (half8*)tab;
  k_dft16_x<<<32, 256, 0, s>>>((_Float16*)t, g.P[0]);
  t += x16_entries(g.P[0]);
  const Yz16Tab o = yz16_tab(g.P[1], g.P[2]);
  auto set = [&](int at, int d, int kind, int kmax, float scale) {
    k_dft16_yz<<<32, 256, 0, s>>>((_Float16*)(t + at), g.P[d], kind, kmax, scale);
  };
  set(o.yf, 1, kFwd, g.N[1], hs[1]);
  set(o.zf, 2, kFwd, g.N[2], hs[2]);
  set(o.zi, 2, kInvPairs, g.P[2] / 2, 1.f);
  set(o.yi, 1, kInvAll, g.P[1], 1.f);
  return hipGetLastError();
}

// The spectrum copy: [x octant][z octant / 4][entry][y octant] with the four z
// of one entry together (FP16 re, -im each), scaled by gs.
size_t spec_cols_bytes(const GroupGeom& g) {
  return (size_t)g.Q[0] * (g.P[2] / 8 + 1) * 6 * g.Q[1] * 16;
}
__global__ void k_spec_cols(const c32* __restrict__ in, unsigned* __restrict__ out, int Q1, int Q2,
                            int Q3, float gs) {
  const int Z4 = (Q3 - 1) / 4 + 1;
  const int64_t n = (int64_t)Q1 * Z4 * 6 * Q2 * 4;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int zi = (int)(i & 3), yo = (int)((i >> 2) % Q2);
    const int64_t r = (i >> 2) / Q2;
    const int ab = (int)(r % 6), zo = (int)((r / 6) % Z4) * 4 + zi, xo = (int)(r / 6 / Z4);
    c32 v = mk<float>(0, 0);
    if (zo < Q3) v = in[(((int64_t)yo * Q3 + zo) * Q1 + xo) * 6 + ab];
    out[i] = __builtin_bit_cast(unsigned, h2{(_Float16)(v.re * gs), (_Float16)(-v.im * gs)});
  }
}
hipError_t launch_spec_cols(const void* spec32, void* out, const GroupGeom& g, float gs,
                            hipStream_t s) {
  k_spec_cols<<<1024, 256, 0, s>>>((const c32*)spec32, (unsigned*)out, g.Q[0], g.Q[1], g.Q[2], gs);
  return hipGetLastError();
}

struct X16Args {
  int N1, N2, N3;
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
__global__ __launch_bounds__(256, 4) void k_x16_fwd(
    const void* __restrict__ xcv, _Float16* __restrict__ A, BodyIdx bi, X16Args a, float hs1,
    const int* __restrict__ active, const double* __restrict__ npart, int nblk,
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
  half8* out = reinterpret_cast<half8*>(
      A + (((int64_t)rhs * 3 + comp) * a.N3 + z) * ((P1 + 1) * 2 * H2));
  for (int i = tid; i < P1 * 2 * H2 / 8; i += 256) {
    const int yc = i % (H2 / 8), pt = i / (H2 / 8) % 2, k = i / (H2 / 4);
    out[i] = *reinterpret_cast<const half8*>(buf + pt * FP + k * FS + yc * 8);
  }
}

// y and z transforms, spectrum and back of one x frequency's column of three
// components, in place.  A wave takes 16 pairs of y frequencies j, -j (slots j
// and H + j; P / 2 sits in the slot of -0) through the z stage: their z lines
// come from LDS, and the four points of +-ky, +-kz read one octant record (a
// mirrored axis only flips the signs of the two entries odd along it).  The
// products stay in registers, and the layout of a matrix product's sums is the
// next one's operand layout with its k permuted, so nothing is exchanged but
// the y-z transpositions.
//
// What bounds it is instruction issue: vector instructions (the spectrum's 18
// dot products a point, conversions) take 64 % of its cycles, the matrix cores
// 30 %, and the two add up.  Wide waves load each table and record for twice
// the points (narrow ones, each with one of j, -j, were bound by the vector
// cache); the two of a pair go through the spectrum one after the other and
// rows are not padded, so that three workgroups of four waves share a CU (49 KB
// of LDS, 168 registers, for 128 x 64).  128 x 128 x 64, 29 planes, 32 right-
// hand sides: 116 us (153 with narrow waves; 137 with the pairs kz, -kz formed
// before the spectrum, 126 without; two workgroups until here), x passes 50 and
// 52 us.  Before, with the y lines in HBM: packed Stockham passes x-y 102, z
// 137, y-x 101 us; the same with x and y on the matrix cores 82, 139, 82 us.
template <int P2, int P3>
struct Yz16 {
  static constexpr int H2 = P2 / 2, H3 = P3 / 2;
  static constexpr int TY = H2 / 16, TZ = H3 / 16;
  static constexpr int NW = TY, NT = 64 * NW;
  static constexpr int KY = (H2 + 31) / 32, KZ = (H3 + 31) / 32, KI = P2 / 32;
  // the column as loaded, the z lines, the y lines.  16-byte pieces of a row are
  // rotated by the row where its length is a power of two, else rows are padded
  // by one piece: neighbouring rows' pieces lie in different banks
  static constexpr bool YR = P2 != 96, ZR = H3 != 48;
  static constexpr int CS = YR ? P2 : P2 + 8, ZS = ZR ? H3 : H3 + 8;
  static constexpr int L0 = 3 * H3 * CS, L1 = 6 * P2 * ZS, L2 = 6 * H3 * CS;
  static __device__ __forceinline__ int ypos(int row, int y) {  // of L0, L2
    return row * CS + (YR ? y ^ ((row & 7) << 3) : y);
  }
  static __device__ __forceinline__ int zpos(int row, int z) {
    constexpr int M = H3 / 8 - 1;  // pieces of a row - 1
    return row * ZS + (ZR ? z ^ (((row / (8 / (M < 7 ? M + 1 : 8))) & M) << 3) : z);
  }
  static constexpr int LDS = L1 > L2 ? (L1 > L0 ? L1 : L0) : (L2 > L0 ? L2 : L0);
  static constexpr int FIT = 160 * 1024 / (2 * LDS) * NW / 4;  // waves per SIMD the LDS holds
  static constexpr int CAP = TZ > 2 ? 1 : 3;                   // and the registers
  static constexpr int WPE = FIT > CAP ? CAP : FIT < 1 ? 1 : FIT;
};

// o += g v in FP32, from g' = (g.re, -g.im): v = (re, im) gives the real part,
// w = (im, -re) the imaginary one
struct PairOp {
  h2 v, w;
};
__device__ __forceinline__ PairOp pair_op(unsigned u, h2 sign) {  // sign = (1, -1)
  PairOp p;
  p.v = __builtin_bit_cast(h2, u);
  p.w = h2{p.v.y, p.v.x} * sign;
  return p;
}
__device__ __forceinline__ c32 cdot(unsigned g, PairOp p, c32 c) {
  const h2 a = __builtin_bit_cast(h2, g);
  return mk<float>(__builtin_amdgcn_fdot2(a, p.v, c.re, false),
                   __builtin_amdgcn_fdot2(a, p.w, c.im, false));
}
// v: the three components of the part the entries even in z multiply, o: of the
// part the odd ones do
__device__ __forceinline__ void green3(const unsigned (&g)[6], const PairOp (&v)[3],
                                       const PairOp (&o)[3], c32 (&r)[3]) {
  const c32 zero = mk<float>(0, 0);
  r[0] = cdot(g[2], o[2], cdot(g[1], v[1], cdot(g[0], v[0], zero)));
  r[1] = cdot(g[4], o[2], cdot(g[3], v[1], cdot(g[1], v[0], zero)));
  r[2] = cdot(g[5], v[2], cdot(g[4], o[1], cdot(g[2], o[0], zero)));
}
__device__ __forceinline__ half4 round4(f32x4 v) {
  return half4{(_Float16)v[0], (_Float16)v[1], (_Float16)v[2], (_Float16)v[3]};
}

struct Yz16Args {
  int P1, N3, nrhs;
  const half8* tab;  // of the y-z sets
  const u32x4* spec;
};

template <int P2, int P3, int NT = Yz16<P2, P3>::NT, int WPE = Yz16<P2, P3>::WPE>
__global__ __launch_bounds__(NT, WPE) void k_yz16_green(
    _Float16* __restrict__ A, Yz16Args a, const int* __restrict__ active) {
  using S = Yz16<P2, P3>;
  constexpr int H2 = S::H2, H3 = S::H3, TZ = S::TZ, KZ = S::KZ;
  constexpr Yz16Tab off = yz16_tab(P2, P3);
  __shared__ __align__(16) _Float16 buf[S::LDS];
  // right-hand side innermost, mirror columns in pairs: a spectrum column is
  // read by neighbouring workgroups of one XCD
  const int b = xcd_remap(blockIdx.x, gridDim.x);
  const int rhs = b % a.nrhs, u = b / a.nrhs;
  if (active && !active[rhs]) return;
  int kx = 0;
  if (u == a.P1 - 1)
    kx = a.P1 / 2;
  else if (u > 0)
    kx = (u & 1) ? (u + 1) / 2 : a.P1 - u / 2;
  const bool xm = kx > a.P1 / 2;
  const int kxo = xm ? a.P1 - kx : kx;
  constexpr unsigned kNeg = 0x80008000u;  // both signs of a packed (re, im)
  unsigned one_m1 = 0xBC003C00u;  // FP16 (1, -1), opaque so that the swap folds into the product
  asm volatile("" : "+v"(one_m1));
  const h2 sign = __builtin_bit_cast(h2, one_m1);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l16 = lane & 15, quad = lane >> 4;
  auto column = [&](int comp, int z) {
    return A + ((((int64_t)rhs * 3 + comp) * a.N3 + z) * (a.P1 + 1) + kx) * 2 * H2;
  };
  {  // the column into LDS, [component][z][re, im][y]
    constexpr int C = P2 / 8, N = 3 * H3 * C;  // 16-byte pieces
    half8 v[(N + S::NT - 1) / S::NT];
#pragma unroll
    for (int n = 0; n < (N + S::NT - 1) / S::NT; ++n) {
      const int i = min(tid + n * S::NT, N - 1), zc = i / C;
      // rows past the grid repeat the last one: the z table is zero there
      v[n] = reinterpret_cast<const half8*>(column(zc / H3, min(zc % H3, a.N3 - 1)))[i % C];
    }
#pragma unroll
    for (int n = 0; n < (N + S::NT - 1) / S::NT; ++n) {
      const int i = min(tid + n * S::NT, N - 1);
      *reinterpret_cast<half8*>(buf + S::ypos(i / C, i % C * 8)) = v[n];
    }
  }
  lds_barrier();
  {  // y forward: the wave's 16 frequency pairs
    half8 re[3 * TZ][S::KY], im[3 * TZ][S::KY];
#pragma unroll
    for (int t = 0; t < 3 * TZ; ++t)
#pragma unroll
      for (int ks = 0; ks < S::KY; ++ks) {
        const int y = min(ks * 32 + 8 * quad, H2 - 8);
        re[t][ks] = *reinterpret_cast<const half8*>(buf + S::ypos(t * 16 + l16, y));
        im[t][ks] = *reinterpret_cast<const half8*>(buf + S::ypos(t * 16 + l16, H2 + y));
      }
    const half8* tb = a.tab + off.yf + wave * S::KY * 64 + lane;
    half8 c[S::KY], sn[S::KY];
#pragma unroll
    for (int ks = 0; ks < S::KY; ++ks) {
      c[ks] = tb[ks * 64];
      sn[ks] = tb[(S::TY * S::KY + ks) * 64];
    }
    lds_barrier();  // every wave has read the column
    const int j = wave * 16 + l16;
#pragma unroll
    for (int t = 0; t < 3 * TZ; ++t) {
      f32x4 p = 0.f, q = 0.f, r = 0.f, u = 0.f;
#pragma unroll
      for (int ks = 0; ks < S::KY; ++ks) {
        p = mma16(re[t][ks], c[ks], p);
        q = mma16(im[t][ks], sn[ks], q);
        r = mma16(im[t][ks], c[ks], r);
        u = mma16(re[t][ks], sn[ks], u);
      }
      half4 lr = round4(p + q), li = round4(r - u), hr = round4(p - q), hi = round4(r + u);
      if (wave == 0 && l16 == 0) {
        lr = round4(p);
        li = round4(r);
        hr = round4(u);
        hi = round4(q);
      }
      // (H2 and P2 rows further the rotation is the same)
      _Float16* o = buf + S::zpos(t / TZ * 2 * P2 + j, t % TZ * 16 + 8 * (quad / 2)) + 4 * (quad & 1);
      *reinterpret_cast<half4*>(o) = lr;
      *reinterpret_cast<half4*>(o + H2 * S::ZS) = hr;
      *reinterpret_cast<half4*>(o + P2 * S::ZS) = li;
      *reinterpret_cast<half4*>(o + (P2 + H2) * S::ZS) = hi;
    }
  }
  // octant records of the wave's y frequencies, and of P / 2 for the slot of -0
  const int Q2 = H2 + 1, yo = wave * 16 + l16;
  const u32x4* sp = a.spec + (int64_t)kxo * (H3 / 4 + 1) * 6 * Q2 + yo;
  const int skip = yo == 0 ? H2 : 0;
  u32x4 rec[6];
#pragma unroll
  for (int c = 0; c < 6; ++c) rec[c] = sp[(quad * 6 + c) * Q2];
  lds_barrier();
  // The wave's z lines into registers, then 16 pairs kz = j, -j at a time
  // through the z transform and the spectrum.  With a = C re + i C im, b = S im
  // - i S re the pair is a + b, a - b, and entries odd in z change sign between
  // the two: a takes b where they act and the other way round, so neither the
  // pair nor, for the inverse, its sum and difference is ever formed.
  half8 vr[2][3][KZ], vi[2][3][KZ];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int comp = 0; comp < 3; ++comp) {
#pragma unroll
      for (int ks = 0; ks < KZ; ++ks) {
        const _Float16* row =
            buf + S::zpos(comp * 2 * P2 + h * H2 + yo, min(ks * 32 + 8 * quad, H3 - 8));
        vr[h][comp][ks] = *reinterpret_cast<const half8*>(row);
        vi[h][comp][ks] = *reinterpret_cast<const half8*>(row + P2 * S::ZS);
      }
    }
  lds_barrier();  // every wave has read its lines
  // half the sum (re, im) and half the difference (re, -im) of each component's
  // pair, two points a register; X[0] and X[P3 / 2] (im, re) in the first
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    unsigned op[3][4][4 * KZ];
    if constexpr (TZ & 1) {
#pragma unroll
      for (int c = 0; c < 12; ++c) op[c / 4][c % 4][4 * KZ - 2] = op[c / 4][c % 4][4 * KZ - 1] = 0;
    }
#pragma unroll
    for (int zt = 0; zt < TZ; ++zt) {
      const half8* tb = a.tab + off.zf + zt * KZ * 64 + lane;
      half8 tc[KZ], ts[KZ];
#pragma unroll
      for (int ks = 0; ks < KZ; ++ks) {
        tc[ks] = tb[ks * 64];
        ts[ks] = tb[(TZ * KZ + ks) * 64];
      }
      unsigned lo[3][4], hi[3][4];
#pragma unroll
      for (int comp = 0; comp < 3; ++comp) {
        f32x4 p = 0.f, q = 0.f, r = 0.f, t = 0.f;
#pragma unroll
        for (int ks = 0; ks < KZ; ++ks) {
          p = mma16(tc[ks], vr[h][comp][ks], p);
          q = mma16(ts[ks], vi[h][comp][ks], q);
          r = mma16(tc[ks], vi[h][comp][ks], r);
          t = mma16(ts[ks], vr[h][comp][ks], t);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          unsigned l = pack_c(p[i], r[i]);
          unsigned u = pack_c(q[i], -t[i]);
          if (zt == 0 && i == 0 && quad == 0) u = pack_c(t[i], q[i]);  // P3 / 2
          lo[comp][i] = l;
          hi[comp][i] = u;
        }
      }
      // (the empty asm statements keep the compiler from spreading the stages
      // over each other, whose registers do not fit together)
#pragma unroll
      for (int c = 0; c < 12; ++c)
        asm volatile("" : "+v"(lo[c / 4][c % 4]), "+v"(hi[c / 4][c % 4]));
      unsigned gn[6];
      if (zt == 0) {
#pragma unroll
        for (int c = 0; c < 6; ++c)  // kz = P3 / 2
          gn[c] = sp[((quad == 0 ? H3 / 4 : quad) * 6 + c) * Q2 + (h ? skip : 0)][0];
      }
      // G_ab is odd along an axis iff exactly one of a, b is that axis
      const bool ym = h && yo;
      const unsigned sxy = xm != ym ? kNeg : 0u, sxz = xm ? kNeg : 0u, syz = ym ? kNeg : 0u;
#pragma unroll
      for (int i = 0; i < 4; i += 2) {
        float o[2][3][4];
#pragma unroll
        for (int d = 0; d < 2; ++d) {
          const bool first = zt == 0 && i + d == 0;
          unsigned g[6];
          auto mirror = [&] {
            g[1] ^= sxy;
            g[2] ^= sxz;
            g[4] ^= syz;
          };
#pragma unroll
          for (int c = 0; c < 6; ++c) g[c] = rec[c][i + d];
          mirror();
          PairOp va[3], vb[3];
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            va[c] = pair_op(lo[c][i + d], sign);
            vb[c] = pair_op(hi[c][i + d], sign);
          }
          c32 e[3], u[3];
          if (first) {  // kz = 0 and P3 / 2 share the lanes of quad 0, uncoupled
            PairOp oa[3], ob[3];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
              oa[c].v = quad == 0 ? va[c].v : vb[c].v;
              oa[c].w = quad == 0 ? va[c].w : vb[c].w;
              ob[c].v = quad == 0 ? vb[c].v : va[c].v;
              ob[c].w = quad == 0 ? vb[c].w : va[c].w;
            }
            green3(g, va, oa, e);
#pragma unroll
            for (int c = 0; c < 6; ++c) g[c] = gn[c];
            mirror();
            green3(g, vb, ob, u);
          } else {
            green3(g, va, vb, e);
            green3(g, vb, va, u);
          }
          const bool nyq = first && quad == 0;
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            o[d][c][0] = e[c].re;
            o[d][c][1] = e[c].im;
            o[d][c][2] = nyq ? u[c].im : u[c].re;
            o[d][c][3] = nyq ? u[c].re : -u[c].im;
          }
        }
#pragma unroll
        for (int c = 0; c < 12; ++c) {
          unsigned& w = op[c / 4][c % 4][2 * zt + i / 2];
          w = pack_c(o[0][c / 4][c % 4], o[1][c / 4][c % 4]);
          asm volatile("" : "+v"(w));
        }
      }
      // the next records; P2 / 2's in lane 0's slot of -0
      if (zt + 1 < TZ || h == 0) {
        const int zn = zt + 1 < TZ ? zt + 1 : 0, at = h == 1 || zt + 1 == TZ ? skip : 0;
#pragma unroll
        for (int c = 0; c < 6; ++c) rec[c] = sp[((zn * 4 + quad) * 6 + c) * Q2 + at];
      }
    }
    // z inverse, into [component][re, im][z][y slot]
#pragma unroll
    for (int zt = 0; zt < TZ; ++zt) {
      const half8* tb = a.tab + off.zi + zt * KZ * 64 + lane;
      half8 tc[KZ], ts[KZ];
#pragma unroll
      for (int ks = 0; ks < KZ; ++ks) {
        tc[ks] = tb[ks * 64];
        ts[ks] = tb[(TZ * KZ + ks) * 64];
      }
#pragma unroll
      for (int comp = 0; comp < 3; ++comp) {
        f32x4 re = 0.f, im = 0.f;
        auto frag = [&](int k, int ks) {
          const unsigned* o = op[comp][k] + 4 * ks;
          return __builtin_bit_cast(half8, u32x4{o[0], o[1], o[2], o[3]});
        };
#pragma unroll
        for (int ks = 0; ks < KZ; ++ks) {
          re = mma16(frag(0, ks), tc[ks], re);
          im = mma16(frag(1, ks), tc[ks], im);
          re = mma16(frag(3, ks), ts[ks], re);
          im = mma16(frag(2, ks), ts[ks], im);
        }
        const int z = comp * 2 * H3 + zt * 16 + l16, k = h * H2 + wave * 16 + 8 * (quad / 2);
        *reinterpret_cast<half4*>(buf + S::ypos(z, k) + 4 * (quad & 1)) = round4(re);
        *reinterpret_cast<half4*>(buf + S::ypos(z + H3, k) + 4 * (quad & 1)) = round4(im);
      }
    }
  }
  {  // y inverse: the wave's 16 points
    const half8* tb = a.tab + off.yi + wave * S::KI * 64 + lane;
    half8 c[S::KI], sn[S::KI];
#pragma unroll
    for (int ks = 0; ks < S::KI; ++ks) {
      c[ks] = tb[ks * 64];
      sn[ks] = tb[(S::TY * S::KI + ks) * 64];
    }
    lds_barrier();
#pragma unroll
    for (int t = 0; t < 3 * TZ; ++t) {
      const int comp = t / TZ, z = t % TZ * 16 + l16;
      f32x4 r1 = 0.f, r2 = 0.f, i1 = 0.f, i2 = 0.f;
#pragma unroll
      for (int ks = 0; ks < S::KI; ++ks) {
        const int k = ks * 32 + 8 * quad;
        const half8 gr = *reinterpret_cast<const half8*>(buf + S::ypos(comp * 2 * H3 + z, k));
        const half8 gi = *reinterpret_cast<const half8*>(buf + S::ypos(comp * 2 * H3 + H3 + z, k));
        r1 = mma16(c[ks], gr, r1);
        r2 = mma16(sn[ks], gi, r2);
        i1 = mma16(c[ks], gi, i1);
        i2 = mma16(sn[ks], gr, i2);
      }
      if (z < a.N3) {
        _Float16* o = column(comp, z) + wave * 16 + 4 * quad;
        *reinterpret_cast<half4*>(o) = round4(r1 - r2);
        *reinterpret_cast<half4*>(o + H2) = round4(i1 + i2);
      }
    }
  }
}

template <int P1, int P2>
__global__ __launch_bounds__(256, 4) void k_x16_inv(
    const _Float16* __restrict__ A, const cb16* __restrict__ xin, c32* __restrict__ yout,
    BodyIdx bi, X16Args a, float hs, const int* __restrict__ active) {
  using D1 = Dft16<P1>;
  constexpr int H1 = D1::H, H2 = P2 / 2;
  constexpr int GP = P1 * H2;  // a part's halves; rows of 32 y pairs may read past the last
  constexpr int RS = H1 + 1;
  constexpr int BYTES = (2 * GP + 64) * 2 > H2 * RS * 8 ? (2 * GP + 64) * 2 : H2 * RS * 8;
  // [re, im][x frequency][y], then the plane's values [y][x] in FP32
  __shared__ __align__(16) char ubuf[BYTES];
  _Float16* buf = reinterpret_cast<_Float16*>(ubuf);
  c32* res = reinterpret_cast<c32*>(ubuf);
  const int nrhs = gridDim.x / (3 * a.N3);
  const int rhs = blockIdx.x % nrhs, cz = blockIdx.x / nrhs;
  if (active && !active[rhs]) return;
  const int comp = cz / a.N3, z = cz % a.N3;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l32 = lane & 31, half = lane >> 5;
  const half8* in = reinterpret_cast<const half8*>(
      A + (((int64_t)rhs * 3 + comp) * a.N3 + z) * ((P1 + 1) * 2 * H2));
#pragma unroll
  for (int n = 0; n < (P1 * H2 / 4 + 255) / 256; ++n) {
    const int i = tid + n * 256;
    if (P1 * H2 / 4 % 256 && i >= P1 * H2 / 4) break;
    const int yc = i % (H2 / 8), pt = i / (H2 / 8) % 2, k = i / (H2 / 4);
    *reinterpret_cast<half8*>(buf + pt * GP + k * H2 + yc * 8) = in[i];
  }
  const int body = bi.rhs_body[rhs];
  const int nb = bi.nb[body];
  const int* vox = bi.vox + bi.voff[body];
  const double* chic = bi.chic + bi.voff[body];
  const int* lp = bi.line_ptr + (int64_t)body * (a.N2 * a.N3 + 1) + z * a.N2;
  const int k0 = lp[0], k1 = lp[a.N2];
  const int64_t vb = bi.roff[rhs] + (int64_t)comp * nb;
  lds_barrier();
  {  // inverse x in FP32: wave = (32 points, the even or the odd rows)
    const int nt = wave % D1::T, odd = wave / D1::T;
    f32x16 r1 = 0.f, r2 = 0.f, im = 0.f;
    if (odd < 2) {
      const half8* tb = a.tab + nt * D1::K * 64 + lane;
      const unsigned* br = reinterpret_cast<const unsigned*>(buf) + 8 * half * (H2 / 2) + l32;
      const unsigned sel = odd ? 0x07060302u : 0x05040100u;
      auto rows = [&](const unsigned* p) {  // 8 frequencies of this lane's row
        u32x4 o;
#pragma unroll
        for (int d = 0; d < 4; ++d)
          o[d] = __builtin_amdgcn_perm(p[(2 * d + 1) * (H2 / 2)], p[2 * d * (H2 / 2)], sel);
        return __builtin_bit_cast(half8, o);
      };
      const unsigned flip = lane & 1 ? 0x80008000u : 0u;  // e^{i pi x} of frequencies >= H1
      auto flipped = [&](half8 v) {
        return __builtin_bit_cast(half8,
                                  __builtin_bit_cast(u32x4, v) ^ u32x4{flip, flip, flip, flip});
      };
#pragma unroll
      for (int ks = 0; ks < D1::K; ++ks) {
        half8 ch = tb[kChi * D1::PLANE + ks * 64], cl = tb[kClo * D1::PLANE + ks * 64];
        half8 sh = tb[kShi * D1::PLANE + ks * 64], sl = tb[kSlo * D1::PLANE + ks * 64];
#pragma unroll
        for (int up = 0; up < 2; ++up) {
          const half8 gr = rows(br + (up * H1 + ks * 16) * (H2 / 2));
          const half8 gi = rows(br + GP / 2 + (up * H1 + ks * 16) * (H2 / 2));
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
    if (odd < 2 && x < H1) {
#pragma unroll
      for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int y = 2 * (8 * g + 4 * half + i) + odd;
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

// FFT lengths 64, 96 and 128 along x and y (the z lengths are h16_ok's).
static bool xy_len_ok(int p) { return p == 64 || p == 96 || p == 128; }
bool xy_fused_ok(const GroupGeom& g) {
  return xy_len_ok(g.P[0]) && xy_len_ok(g.P[1]) && 4 * g.N[1] >= g.P[1] &&  // bufA holds it
         (g.P[2] == 32 || g.P[2] == 64 || g.P[2] == 96 || g.P[2] == 128);
}

#define VIE_DISPATCH_XY(P_, CALL)                    \
  switch (P_) {                                      \
    case 64: { constexpr int PP = 64; CALL; break; } \
    case 96: { constexpr int PP = 96; CALL; break; } \
    case 128: { constexpr int PP = 128; CALL; break; } \
    default: return hipErrorInvalidValue;            \
  }

// The lengths divide into the products' tiles, and a plane and a column fit the
// LDS.  (Three passes, us, before and after, FFT lengths x, y, z with 32
// right-hand sides: 64 96 96: 234, 180; 96 64 96: 241, 178; 96 128 96: 415, 300;
// 128 64 64: 160, 125; 128 128 64: 340, 218; 64 64 64 with 8: 51, 35.)
static bool x16_args(const MatvecArgs& m, X16Args* a) {
  const GroupGeom& g = *m.g;
  if (!xy_fused_ok(g) || !m.dft16 || !m.bi) return false;
  for (int d = 0; d < 3; ++d)
    if (g.N[d] < 1 || 2 * g.N[d] > g.P[d]) return false;
  a->N1 = g.N[0];
  a->N2 = g.N[1];
  a->N3 = g.N[2];
  a->tab = (const half8*)m.dft16;
  return true;
}

// m.npart set: normalising FP32 input (see MatvecArgs), else bfloat16 input
hipError_t x16_fwd(const MatvecArgs& m, const void* xc, void* A, hipStream_t s) {
  const GroupGeom& g = *m.g;
  X16Args a;
  if (!x16_args(m, &a)) return hipErrorInvalidValue;
  const dim3 grid(g.nrhs * 3 * g.N[2]);
  VIE_DISPATCH_XY(g.P[0], ({
                    constexpr int Q1 = PP;
                    VIE_DISPATCH_XY(g.P[1], ({
                                      if (m.npart)
                                        k_x16_fwd<Q1, PP, true><<<grid, 256, 0, s>>>(
                                            xc, (_Float16*)A, *m.bi, a, m.hs[0], m.active,
                                            m.npart, m.nblk, m.nrm, m.ldn, (cb16*)m.vout);
                                      else
                                        k_x16_fwd<Q1, PP, false><<<grid, 256, 0, s>>>(
                                            xc, (_Float16*)A, *m.bi, a, m.hs[0], m.active,
                                            nullptr, 0, nullptr, 0, nullptr);
                                    }));
                  }));
  return hipGetLastError();
}

template <int P2>
static hipError_t yz16_p2(const MatvecArgs& m, _Float16* A, const Yz16Args& a, hipStream_t s) {
  const dim3 grid(a.P1 * a.nrhs);
#define VIE_YZ16(P3_)                                                              \
  case P3_:                                                                        \
    k_yz16_green<P2, P3_><<<grid, Yz16<P2, P3_>::NT, 0, s>>>(A, a, m.active); \
    break;
  switch (m.g->P[2]) {
    VIE_YZ16(32)
    VIE_YZ16(64)
    VIE_YZ16(96)
    VIE_YZ16(128)
    default: return hipErrorInvalidValue;
  }
#undef VIE_YZ16
  return hipGetLastError();
}

hipError_t yz16_green(const MatvecArgs& m, void* A, hipStream_t s) {
  const GroupGeom& g = *m.g;
  X16Args x;
  if (!x16_args(m, &x)) return hipErrorInvalidValue;
  const Yz16Args a{g.P[0], g.N[2], g.nrhs, x.tab + x16_entries(g.P[0]), (const u32x4*)m.spec16};
  switch (g.P[1]) {
    case 64: return yz16_p2<64>(m, (_Float16*)A, a, s);
    case 96: return yz16_p2<96>(m, (_Float16*)A, a, s);
    case 128: return yz16_p2<128>(m, (_Float16*)A, a, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t x16_inv(const MatvecArgs& m, const void* A, const void* x, void* y, hipStream_t s) {
  const GroupGeom& g = *m.g;
  X16Args a;
  if (!x16_args(m, &a)) return hipErrorInvalidValue;
  const dim3 grid(g.nrhs * 3 * g.N[2]);
  VIE_DISPATCH_XY(g.P[0], ({
                    constexpr int Q1 = PP;
                    VIE_DISPATCH_XY(g.P[1], (k_x16_inv<Q1, PP><<<grid, 256, 0, s>>>(
                                                (const _Float16*)A, (const cb16*)x, (c32*)y,
                                                *m.bi, a, m.hout, m.active)));
                  }));
  return hipGetLastError();
}
#undef VIE_DISPATCH_XY

}  // namespace vie
