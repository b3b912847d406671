// Learned warm start: 3x3x3 convolutions as implicit GEMMs on bf16 MFMA
// (gfx950's v_mfma_f32_16x16x32_bf16, fp32 accumulation; the 16-deep
// v_mfma_f32_16x16x16_bf16 where a reduction step has only 16 channels), with
// training kernels.
//
// Convolution (forward and backward-data): a workgroup marches a 16 x 16
// lateral tile through its z layers, the layer's halo and the whole weight
// tensor in LDS; every layer read feeds the three output layers it touches
// (see k_conv3d).
// Weight gradient: rows = Cout, columns = (tap, Cin), reduction over the
// tile voxels; activations and gradients are staged channels-first in LDS,
// the activations in three copies shifted along x, so that every operand is
// one aligned 16-byte read.  Per-block partials are summed in fixed order by a
// second kernel (deterministic).
#include <math.h>
#include <string.h>

#include <algorithm>
#include <type_traits>

#include "cnn.h"

namespace vie {

typedef short v4s __attribute__((ext_vector_type(4)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));

// A caller's tensor may start anywhere its elements may (a view into a larger
// one): 16- and 8-byte accesses to it claim no more.  The memory unit takes
// them so; on aligned tensors they are the same instructions.
typedef uint32_t u4any __attribute__((ext_vector_type(4), aligned(2)));
typedef uint32_t u2any __attribute__((ext_vector_type(2), aligned(2)));
typedef float f4any __attribute__((ext_vector_type(4), aligned(4)));

// One 16x16 output tile += A (16 x K) B (K x 16) over K = 32 (or 16): lane l
// holds row / column l % 16 and the K slice 8 (l / 16) .. + 7 (4 (l / 16) .. +
// 3) of its operands, and receives D[4 (l / 16) + i][l % 16], i = 0..3.  Only
// the pairing of A and B slices matters for the sum, so any fixed K order
// that both operands share gives the same product.
__device__ __forceinline__ v4f mfma32(v8bf a, v8bf b, v4f c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ v4f mfma16(v4s a, v4s b, v4f c) {
  return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ bf16raw f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);  // round to nearest even
  return (bf16raw)(u >> 16);
}
__device__ __forceinline__ float bf2f(bf16raw h) { return __uint_as_float(((uint32_t)h) << 16); }

CnnLayerOffsets cnn_offsets() {
  CnnLayerOffsets o;
  int64_t at = 0;
  for (int l = 0; l < kCnnLayers; ++l) {
    o.w[l] = at;
    at += 27 * (int64_t)kCnnCh[l] * kCnnCh[l + 1];
    o.b[l] = at;
    at += kCnnCh[l + 1];
  }
  o.total = at;
  return o;
}

// ------------------------------------------------------------ convolution
constexpr int CT = 16;                 // lateral tile edge
constexpr int CH = CT + 2;             // with its halo
constexpr int CNT = 256;               // threads: four waves

struct ConvDims {
  int d0, d1, d2, tx, ty, zc;  // box, lateral tiles, z layers per workgroup
};

// MODE 0: + bias, ReLU -> bf16; MODE 1: + bias -> fp32; MODE 2: * (ref > 0) -> bf16
//
// One workgroup: outputs z0 .. z0 + zc - 1 of a 16 x 16 lateral tile.  It
// walks the input layers z0 - 1 .. z0 + zc; layer p feeds output p + 1 with the
// nine dz = -1 taps, p with dz = 0 and p - 1 with dz = +1, so each output sums
// its taps in the order dz, dy, dx.  A wave holds four rows of 16 voxels and
// every output channel: with four activation operands and 3 x 2 weight
// operands a tap reads 10 operands from LDS for 24 MFMAs (0.42 per MFMA; one
// layer per wave took 0.75, eight rows and one channel tile 0.46).  LDS holds
// the weights and one layer (76 KB for 32 -> 32), the next layer waits in
// registers: two workgroups share a CU, so one's staging and stores run under
// the other's MFMAs.  Rows of 64 bytes are stored with their 16-byte slots
// rotated by the voxel (row) index so that neighbouring lanes hit different
// banks.  The voxels are the MFMA's columns: each lane ends with four
// neighbouring channels of one voxel, one packed store.  41 us per 32 -> 32
// layer on 128 x 128 x 37, where one layer per wave with 2-byte stores took 79;
// the matrix cores are busy for 41 % of the CUs' busy cycles, the LDS for 22 %
// (no bank conflicts): the waits between reads, products and staging bound it.
template <int CIN, int COUT, int MODE>
__global__ __launch_bounds__(CNT) __attribute__((amdgpu_waves_per_eu(2))) void k_conv3d(
    const bf16raw* __restrict__ in, const bf16raw* __restrict__ w, const float* __restrict__ bias,
    bf16raw* __restrict__ outb, float* __restrict__ outf, const bf16raw* __restrict__ ref,
    ConvDims cd) {
  constexpr bool X32 = CIN == 32;
  static_assert(CIN == 32 || CIN == 16, "channels");
  constexpr int RB = 2 * CIN;       // bytes per voxel (weight row)
  constexpr int SL = RB / 16;       // 16-byte slots per row
  constexpr int NCT = COUT / 16;    // channel tiles
  constexpr int NS = 4;             // 16-voxel rows per wave
  constexpr int NP = CH * CH * SL;  // 16-byte items of a layer
  constexpr int PF = (NP + CNT - 1) / CNT;
  constexpr int NW = 27 * COUT * SL;
  __shared__ __align__(16) char s_w[NW * 16];
  __shared__ __align__(16) char s_p[NP * 16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r = lane & 15, kq = lane >> 4;
  const int row0 = wave * NS;
  const int ntile = cd.tx * cd.ty;
  const int tile = blockIdx.x % ntile, z0 = (blockIdx.x / ntile) * cd.zc;
  const int z1 = min(cd.d2, z0 + cd.zc);
  const int x0 = (tile % cd.tx) * CT, y0 = (tile / cd.tx) * CT;
  auto swz = [](int v) { return X32 ? (v >> 1) & 3 : 0; };
  for (int i = tid; i < NW; i += CNT) {
    const int row = i / SL, sl = i % SL;
    *(uint4*)&s_w[row * RB + ((sl ^ swz(row)) << 4)] = *(const uint4*)&w[(size_t)i * 8];
  }
  // this thread's items of every layer: offset inside the layer (-1: outside the box)
  int goff[PF];
#pragma unroll
  for (int p = 0; p < PF; ++p) {
    const int i = tid + p * CNT, v = i / SL;
    const int gx = x0 + v % CH - 1, gy = y0 + v / CH - 1;
    const bool ok = i < NP && gx >= 0 && gx < cd.d0 && gy >= 0 && gy < cd.d1;
    goff[p] = ok ? (gy * cd.d0 + gx) * CIN + (i % SL) * 8 : -1;
  }
  const size_t layer = (size_t)cd.d0 * cd.d1;
  u4any pre[PF];
  auto fetch = [&](int z) {
    const bf16raw* src = in + (size_t)z * layer * CIN;
#pragma unroll
    for (int p = 0; p < PF; ++p) {
      pre[p] = u4any{0u, 0u, 0u, 0u};
      if (goff[p] >= 0) pre[p] = *(const u4any*)&src[goff[p]];
    }
  };
  // operand addresses: activations of voxel (row0 + s + dy', r + dx'), dy', dx' = 0..2,
  // = abase[c % 8] + c RB with c = (s + dy') CH + dx' known at compile time (row0 CH
  // is a multiple of 8); weights likewise
  int abase[8];
#pragma unroll
  for (int c = 0; c < 8; ++c)
    abase[c] = (row0 * CH + r) * RB + (X32 ? (kq ^ swz(r + c)) << 4 : kq << 3);
  const int wbase = r * RB + (X32 ? (kq ^ swz(r)) << 4 : kq << 3);
  using frag = typename std::conditional<X32, v8bf, v4s>::type;
  auto mma = [](frag a, frag b, v4f c) {
    if constexpr (X32)
      return mfma32(a, b, c);
    else
      return mfma16(a, b, c);
  };
  float4 bv[NCT];
#pragma unroll
  for (int ct = 0; ct < NCT; ++ct)
    bv[ct] = MODE == 2 ? make_float4(0.f, 0.f, 0.f, 0.f)
                       : *(const float4*)&bias[ct * 16 + 4 * kq];
  auto emit = [&](const v4f (&acc)[NS][NCT], int z) {
    const int gx = x0 + r;
    if (gx >= cd.d0) return;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const int gy = y0 + row0 + s;
      if (gy >= cd.d1) break;
#pragma unroll
      for (int ct = 0; ct < NCT; ++ct) {
        const size_t at = ((size_t)z * layer + (size_t)gy * cd.d0 + gx) * COUT + ct * 16 + 4 * kq;
        const v4f c = acc[s][ct];
        const float v[4] = {c[0] + bv[ct].x, c[1] + bv[ct].y, c[2] + bv[ct].z, c[3] + bv[ct].w};
        if (MODE == 1) {
          *(f4any*)&outf[at] = f4any{v[0], v[1], v[2], v[3]};
        } else {
          bf16raw h[4];
          if (MODE == 0) {
#pragma unroll
            for (int i = 0; i < 4; ++i) h[i] = f2bf(v[i] > 0.f ? v[i] : 0.f);
          } else {
            const uint2 m = *(const uint2*)&ref[at];
            const uint32_t mw[2] = {m.x, m.y};
#pragma unroll
            for (int i = 0; i < 4; ++i)
              h[i] = f2bf(bf2f((bf16raw)(mw[i / 2] >> (16 * (i & 1)))) > 0.f ? c[i] : 0.f);
          }
          *(uint2*)&outb[at] = make_uint2((uint32_t)h[0] | (uint32_t)h[1] << 16,
                                          (uint32_t)h[2] | (uint32_t)h[3] << 16);
        }
      }
    }
  };
  const int p0 = max(0, z0 - 1), p1 = min(cd.d2 - 1, z1);
  const v4f zero = {0.f, 0.f, 0.f, 0.f};
  v4f am[NS][NCT], a0[NS][NCT], ap[NS][NCT];  // outputs p - 1, p, p + 1
#pragma unroll
  for (int s = 0; s < NS; ++s)
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct) am[s][ct] = a0[s][ct] = ap[s][ct] = zero;
  fetch(p0);
  for (int p = p0; p <= p1; ++p) {
    lds_barrier();  // the previous layer's operand reads are done
#pragma unroll
    for (int q = 0; q < PF; ++q) {
      const int i = tid + q * CNT, v = i / SL;
      if (i < NP)
        *(uint4*)&s_p[v * RB + (((i % SL) ^ swz(v)) << 4)] =
            make_uint4(pre[q].x, pre[q].y, pre[q].z, pre[q].w);
    }
    if (p < p1) fetch(p + 1);
    lds_barrier();
    const bool up = p + 1 < z1, mid = p >= z0 && p < z1, dn = p > z0;
#pragma unroll
    for (int t = 0; t < 9; ++t) {
      frag b[NS], k[3][NCT];
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const int c = (s + t / 3) * CH + t % 3;
        b[s] = *(const frag*)&s_p[abase[c % 8] + c * RB];
      }
#pragma unroll
      for (int dz = 0; dz < 3; ++dz)
#pragma unroll
        for (int ct = 0; ct < NCT; ++ct)
          k[dz][ct] = *(const frag*)&s_w[wbase + ((9 * dz + t) * COUT + ct * 16) * RB];
      if (up) {
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
          for (int ct = 0; ct < NCT; ++ct) ap[s][ct] = mma(k[0][ct], b[s], ap[s][ct]);
      }
      if (mid) {
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
          for (int ct = 0; ct < NCT; ++ct) a0[s][ct] = mma(k[1][ct], b[s], a0[s][ct]);
      }
      if (dn) {
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
          for (int ct = 0; ct < NCT; ++ct) am[s][ct] = mma(k[2][ct], b[s], am[s][ct]);
      }
    }
    // output p - 1 is complete, and output p too at the top of the box
    if (dn) emit(am, p - 1);
    if (p + 1 == cd.d2 && mid) emit(a0, p);
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
      for (int ct = 0; ct < NCT; ++ct) {
        am[s][ct] = a0[s][ct];
        a0[s][ct] = ap[s][ct];
        ap[s][ct] = zero;
      }
  }
}

// -------------------------------------------------------- weight gradient
constexpr int TX = 8, TY = 8, TZ = 4;  // tile (256 voxels)
constexpr int GNT = 768;               // threads: twelve waves

struct GradDims {
  int d0, d1, d2, tx, ty, tz, ntiles;
};

// dW[tap][co][ci] = sum_m in[m + tap][ci] g[m][co];  db[co] = sum_m g[m][co]
//
// A reduction step is four x-rows of eight voxels.  An activation operand
// (halo layer hz, rows shifted by dy, copy shifted by dx, 16 channels) meets
// the gradient operands of layers hz - dz for the three dz and every
// 16-channel tile of Cout: 3 COUT / 16 MFMAs per LDS read, the tile's
// gradient operands kept in registers.  Wave (u, yg): units 3 u .. 3 u + 2 of the 18
// (dy, dx, channel tile) combinations, rows 4 yg .. 4 yg + 3 of every layer; the
// two halves are added through LDS at the end.  The next tile's voxels
// wait in registers while this one's MFMAs run; a thread holds ten (eight)
// neighbouring voxels of four channels and writes them transposed.  Channel
// c of quad q is stored at index c (channels / 4) + q, which spreads the
// writes over the banks; partials are written in operand order and
// k_reduce_parts puts them in place.  With 8 two-byte LDS reads per operand and
// one thread per channel summing the bias, 32 x 32 channels on 121 x 107 x 37
// took 160 us, plus 121 us for the sum of 512 partials.
template <int COUT>
__global__ __launch_bounds__(GNT) void k_conv3d_wgrad(const bf16raw* __restrict__ in,
                                                      const bf16raw* __restrict__ g,
                                                      float* __restrict__ part, GradDims cd) {
  constexpr int CIN = 32, NRT = COUT / 16;
  constexpr int HR = (TY + 2) * (TZ + 2);  // halo rows
  constexpr int HP = HR + 1;               // padded rows per channel (odd)
  constexpr int MR = TY * TZ, MP = MR + 1;
  constexpr int IN_B = 3 * CIN * HP * 16, G_B = COUT * MP * 16;
  constexpr int NI = HR * (CIN / 4), NG = MR * (COUT / 4);
  constexpr int NT = 27 * CIN * COUT;
  static_assert(NI + NG <= GNT && HP % 2 == 1 && MP % 2 == 1, "staging");
  constexpr int RED_B = 6 * 9 * NRT * 64 * 16;
  constexpr int LDS_B = IN_B + G_B > RED_B ? IN_B + G_B : RED_B;
  __shared__ __align__(16) char lds[LDS_B];
  char* s_g = lds + IN_B;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r = lane & 15, kq = lane >> 4;
  const int yg = wave & 1, u0 = (wave >> 1) * 3;
  // staging item: row and channel quad
  const bool is_in = tid < NI, is_g = !is_in && tid < NI + NG;
  const int it = is_in ? tid : tid - NI;
  const int quad = is_in ? it % (CIN / 4) : it % (COUT / 4);
  const int row = is_in ? it / (CIN / 4) : it / (COUT / 4);
  uint2 pre[TX + 2];
  auto fetch = [&](int tile) {
    const int tx = tile % cd.tx, ty = (tile / cd.tx) % cd.ty, tz = tile / (cd.tx * cd.ty);
    const int x0 = tx * TX, y0 = ty * TY, z0 = tz * TZ;
#pragma unroll
    for (int v = 0; v < TX + 2; ++v) pre[v] = make_uint2(0u, 0u);
    if (is_in) {
      const int gy = y0 + row % (TY + 2) - 1, gz = z0 + row / (TY + 2) - 1;
      if (gy < 0 || gy >= cd.d1 || gz < 0 || gz >= cd.d2) return;
      const bf16raw* src = in + ((size_t)gz * cd.d1 + gy) * cd.d0 * CIN + 4 * quad;
#pragma unroll
      for (int v = 0; v < TX + 2; ++v) {
        const int gx = x0 + v - 1;
        if (gx >= 0 && gx < cd.d0) {
          const u2any t = *(const u2any*)&src[(size_t)gx * CIN];
          pre[v] = make_uint2(t.x, t.y);
        }
      }
    } else if (is_g) {
      const int gy = y0 + row % TY, gz = z0 + row / TY;
      if (gy >= cd.d1 || gz >= cd.d2) return;
      const bf16raw* src = g + ((size_t)gz * cd.d1 + gy) * cd.d0 * COUT + 4 * quad;
#pragma unroll
      for (int v = 0; v < TX; ++v)
        if (x0 + v < cd.d0) pre[v] = *(const uint2*)&src[(size_t)(x0 + v) * COUT];
    }
  };
  // channel c (of the quad) of voxels a .. a + 7, packed
  auto pack8 = [&](int a, int c) {
    uint32_t o[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint32_t lo = c < 2 ? pre[a + 2 * k].x : pre[a + 2 * k].y;
      const uint32_t hi = c < 2 ? pre[a + 2 * k + 1].x : pre[a + 2 * k + 1].y;
      o[k] = (c & 1) ? (lo >> 16) | (hi & 0xFFFF0000u) : (lo & 0xFFFFu) | (hi << 16);
    }
    return make_uint4(o[0], o[1], o[2], o[3]);
  };
  v4f acc[3][3][NRT];
#pragma unroll
  for (int j = 0; j < 3; ++j)
#pragma unroll
    for (int dz = 0; dz < 3; ++dz)
#pragma unroll
      for (int rt = 0; rt < NRT; ++rt) acc[j][dz][rt] = v4f{0.f, 0.f, 0.f, 0.f};
  float bs[4] = {0.f, 0.f, 0.f, 0.f};
  const char* bp[3];  // this lane's activation operands of its units (layer hz: + 160 hz)
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    const int u = u0 + j, cit = u & 1, dy = (u >> 1) / 3, dx = (u >> 1) % 3;
    bp[j] = lds + ((dx * CIN + cit * 16 + r) * HP + 4 * yg + kq + dy) * 16;
  }
  const char* ga = s_g + (r * MP + 4 * yg + kq) * 16;
  if ((int)blockIdx.x < cd.ntiles) fetch(blockIdx.x);
  for (int tile = blockIdx.x; tile < cd.ntiles; tile += gridDim.x) {
    lds_barrier();  // the previous tile's operand reads are done
    if (is_in) {
#pragma unroll
      for (int dx = 0; dx < 3; ++dx)
#pragma unroll
        for (int c = 0; c < 4; ++c)
          *(uint4*)&lds[((dx * CIN + c * (CIN / 4) + quad) * HP + row) * 16] = pack8(dx, c);
    } else if (is_g) {
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const uint4 v = pack8(0, c);
        *(uint4*)&s_g[((c * (COUT / 4) + quad) * MP + row) * 16] = v;
        const uint32_t wv[4] = {v.x, v.y, v.z, v.w};
        float t = 0.f;
#pragma unroll
        for (int k = 0; k < 4; ++k)
          t += bf2f((bf16raw)(wv[k] & 0xFFFFu)) + bf2f((bf16raw)(wv[k] >> 16));
        bs[c] += t;
      }
    }
    if (tile + (int)gridDim.x < cd.ntiles) fetch(tile + gridDim.x);
    lds_barrier();
    v8bf a[TZ][NRT];
#pragma unroll
    for (int lz = 0; lz < TZ; ++lz)
#pragma unroll
      for (int rt = 0; rt < NRT; ++rt)
        a[lz][rt] = *(const v8bf*)(ga + (rt * 16 * MP + lz * TY) * 16);
#pragma unroll
    for (int j = 0; j < 3; ++j)
#pragma unroll
      for (int hz = 0; hz < TZ + 2; ++hz) {
        const v8bf b = *(const v8bf*)(bp[j] + hz * (TY + 2) * 16);
#pragma unroll
        for (int dz = 0; dz < 3; ++dz)
          if (hz - dz >= 0 && hz - dz < TZ) {
#pragma unroll
            for (int rt = 0; rt < NRT; ++rt)
              acc[j][dz][rt] = mfma32(a[hz - dz][rt], b, acc[j][dz][rt]);
          }
      }
  }
  // the two row halves of every unit, then the partial in operand order
  // [unit][dz][rt][lane][4]
  __syncthreads();
  v4f* red = (v4f*)lds;
  if (yg) {
#pragma unroll
    for (int j = 0; j < 3; ++j)
#pragma unroll
      for (int dz = 0; dz < 3; ++dz)
#pragma unroll
        for (int rt = 0; rt < NRT; ++rt)
          red[((wave >> 1) * 9 * NRT + (j * 3 + dz) * NRT + rt) * 64 + lane] = acc[j][dz][rt];
  }
  __syncthreads();
  float* pb = part + (size_t)blockIdx.x * (NT + COUT);
  if (!yg) {
#pragma unroll
    for (int j = 0; j < 3; ++j)
#pragma unroll
      for (int dz = 0; dz < 3; ++dz)
#pragma unroll
        for (int rt = 0; rt < NRT; ++rt)
          *(v4f*)&pb[((((u0 + j) * 3 + dz) * NRT + rt) * 64 + lane) * 4] =
              acc[j][dz][rt] +
              red[((wave >> 1) * 9 * NRT + (j * 3 + dz) * NRT + rt) * 64 + lane];
  }
  __syncthreads();
  float* sb = (float*)lds;  // [row][quad][4]
  if (is_g)
#pragma unroll
    for (int c = 0; c < 4; ++c) sb[it * 4 + c] = bs[c];
  __syncthreads();
  if (tid < COUT) {
    float t = 0.f;
    for (int k = 0; k < MR; ++k) t += sb[(k * (COUT / 4) + tid / 4) * 4 + tid % 4];
    pb[NT + tid] = t;
  }
}

// Sum of the weight-gradient partials, in fixed order, put in parameter order
// ([tap][co][ci], then the biases): four waves take a quarter of the blocks
// each for 64 neighbouring elements.  Chains of 64 partials after a block's own:
// 2.1e-7, 1.7e-7 and 1.0e-7 off the 64-bit sums on boxes of 121 x 107 x 37, 64 x 64 x
// 37 and 30 x 25 x 16 (512 partials in one chain: 4.1e-7, 4.6e-7, 1.6e-7).
template <int COUT>
__global__ __launch_bounds__(256) void k_reduce_parts(const float* __restrict__ part, int nblk,
                                                      float* __restrict__ out) {
  constexpr int CIN = 32, NRT = COUT / 16, NT = 27 * CIN * COUT, N = NT + COUT;
  __shared__ float red[4][64];
  const int l = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int e = blockIdx.x * 64 + l;
  const int b0 = (int)((int64_t)nblk * wv / 4), b1 = (int)((int64_t)nblk * (wv + 1) / 4);
  float s = 0.f;
  if (e < N) {
#pragma unroll 8
    for (int b = b0; b < b1; ++b) s += part[(size_t)b * N + e];
  }
  red[wv][l] = s;
  __syncthreads();
  if (wv != 0 || e >= N) return;
  s = (red[0][l] + red[1][l]) + (red[2][l] + red[3][l]);
  if (e >= NT) {
    out[e] = s;
    return;
  }
  // e = (((unit * 3 + dz) * NRT + rt) * 64 + lane) * 4 + i: D[co index][ci index]
  const int i = e & 3, lane = (e >> 2) & 63, f = e >> 8;
  const int rt = f % NRT, dz = (f / NRT) % 3, u = f / (3 * NRT);
  const int cit = u & 1, dy = (u >> 1) / 3, dx = (u >> 1) % 3;
  const int coi = rt * 16 + 4 * (lane >> 4) + i, cii = cit * 16 + (lane & 15);
  const int co = coi % (COUT / 4) * 4 + coi / (COUT / 4), ci = cii % (CIN / 4) * 4 + cii / (CIN / 4);
  out[((size_t)(dz * 9 + dy * 3 + dx) * COUT + co) * CIN + ci] = s;
}

// masked relative L2 loss over outputs 0..5; mask = feature channel 0 > 0
__global__ __launch_bounds__(256) void k_loss_partial(const float* __restrict__ out,
                                                      const float* __restrict__ tgt,
                                                      const bf16raw* __restrict__ feat,
                                                      size_t nvox, float* __restrict__ part) {
  __shared__ float sn[256], sd[256];
  float num = 0.f, den = 0.f;
  for (size_t v = (size_t)blockIdx.x * 256 + threadIdx.x; v < nvox; v += (size_t)gridDim.x * 256) {
    if (bf2f(feat[v * kCnnIn]) > 0.f) {
#pragma unroll
      for (int c = 0; c < kCnnOut; ++c) {
        const float t = tgt[v * kCnnOut + c], d = out[v * 16 + c] - t;
        num += d * d;
        den += t * t;
      }
    }
  }
  sn[threadIdx.x] = num;
  sd[threadIdx.x] = den;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o) {
      sn[threadIdx.x] += sn[threadIdx.x + o];
      sd[threadIdx.x] += sd[threadIdx.x + o];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    part[blockIdx.x * 2] = sn[0];
    part[blockIdx.x * 2 + 1] = sd[0];
  }
}

// The block sums in block order, one chain each (the order fixes the bits of
// the loss, which scales a bfloat16 gradient), staged in LDS: read one by one
// from memory the chain took 53 us.
constexpr int kLossBlocks = 1024;
__global__ __launch_bounds__(256) void k_loss_final(const float* __restrict__ part, int nblk,
                                                    float* __restrict__ loss) {
  __shared__ float s[2 * kLossBlocks];
  for (int i = threadIdx.x; i < 2 * nblk; i += 256) s[i] = part[i];
  __syncthreads();
  if (threadIdx.x >= 2) return;
  float t = 0.f;
#pragma unroll 16
  for (int b = 0; b < nblk; ++b) t += s[2 * b + threadIdx.x];
  loss[threadIdx.x] = t;
}

__global__ __launch_bounds__(256) void k_loss_grad(const float* __restrict__ out,
                                                   const float* __restrict__ tgt,
                                                   const bf16raw* __restrict__ feat,
                                                   const float* __restrict__ loss, size_t nvox,
                                                   bf16raw* __restrict__ g) {
  const float inv = loss[1] > 0.f ? 2.f / loss[1] : 0.f;
  for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < nvox * 16;
       e += (size_t)gridDim.x * 256) {
    const size_t v = e / 16;
    const int c = (int)(e % 16);
    float val = 0.f;
    if (c < kCnnOut && bf2f(feat[v * kCnnIn]) > 0.f) val = inv * (out[e] - tgt[v * kCnnOut + c]);
    g[e] = f2bf(val);
  }
}

__global__ void k_adam(float* __restrict__ p, float* __restrict__ m, float* __restrict__ v,
                       const float* __restrict__ g, int64_t n, float lr, float c1, float c2) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const float gi = g[i];
    const float mi = 0.9f * m[i] + 0.1f * gi;
    const float vi = 0.999f * v[i] + 0.001f * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + 1e-8f);
  }
}

// bf16 weight copies: forward [27][Cout][Cin]; backward-data [27][Cin][Cout]
// with tap t' = 26 - t (the adjoint of a same-padded convolution).
__global__ void k_refresh_bf16(const float* __restrict__ p, bf16raw* __restrict__ wf,
                               bf16raw* __restrict__ wb, CnnLayerOffsets off) {
  for (int l = 0; l < kCnnLayers; ++l) {
    const int ci_n = kCnnCh[l], co_n = kCnnCh[l + 1];
    const int64_t n = 27 * (int64_t)ci_n * co_n;
    const float* W = p + off.w[l];
    // bf16 weights are packed without the biases: layer offset in bf16 arrays
    int64_t wo = 0;
    for (int q = 0; q < l; ++q) wo += 27 * (int64_t)kCnnCh[q] * kCnnCh[q + 1];
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
      const int tap = (int)(i / ((int64_t)co_n * ci_n));
      const int co = (int)((i / ci_n) % co_n), ci = (int)(i % ci_n);
      const bf16raw h = f2bf(W[i]);
      wf[wo + i] = h;
      wb[wo + ((int64_t)(26 - tap) * ci_n + ci) * co_n + co] = h;
    }
  }
}

// ------------------------------------------------- features / target / gather
__device__ __forceinline__ size_t box_index(int lin, const int N[3], const int lo[3],
                                            const int d[3]) {
  const int i = lin % N[0], j = (lin / N[0]) % N[1], l = lin / (N[0] * N[1]);
  return ((size_t)(l - lo[2]) * d[1] + (j - lo[1])) * d[0] + (i - lo[0]);
}

struct Box {
  int d[3], lo[3], N[3];
};

struct KrylovIn {
  const c64* v[kCnnKrylov];
  double inv[kCnnKrylov];
};

__global__ void k_cnn_features(bf16raw* __restrict__ feat, Box bx, const int* __restrict__ vox,
                               const double* __restrict__ chic, int nb, KrylovIn kin) {
  for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < nb; k += gridDim.x * blockDim.x) {
    const size_t v = box_index(vox[k], bx.N, bx.lo, bx.d);
    bf16raw* f = feat + v * kCnnIn;
    f[0] = f2bf((float)(chic[k] * 0.25));
#pragma unroll
    for (int q = 0; q < kCnnKrylov; ++q)
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const c64 bv = kin.v[q][(size_t)c * nb + k];
        f[1 + 6 * q + 2 * c] = f2bf((float)(bv.re * kin.inv[q]));
        f[2 + 6 * q + 2 * c] = f2bf((float)(bv.im * kin.inv[q]));
      }
  }
}

__global__ void k_cnn_target(float* __restrict__ tgt, Box bx, const int* __restrict__ vox, int nb,
                             const c64* __restrict__ w, double inv_s) {
  for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < nb; k += gridDim.x * blockDim.x) {
    const size_t v = box_index(vox[k], bx.N, bx.lo, bx.d);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const c64 wv = w[(size_t)c * nb + k];
      tgt[v * kCnnOut + 2 * c] = (float)(wv.re * inv_s);
      tgt[v * kCnnOut + 2 * c + 1] = (float)(wv.im * inv_s);
    }
  }
}

__global__ void k_cnn_gather(c64* __restrict__ x, const float* __restrict__ out, Box bx,
                             const int* __restrict__ vox, int nb, double s) {
  for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < nb; k += gridDim.x * blockDim.x) {
    const size_t v = box_index(vox[k], bx.N, bx.lo, bx.d);
#pragma unroll
    for (int c = 0; c < 3; ++c)
      x[(size_t)c * nb + k] = mk(s * out[v * 16 + 2 * c], s * out[v * 16 + 2 * c + 1]);
  }
}

static Box mkbox(const int d[3], const int lo[3], const int N[3]) {
  Box b;
  for (int a = 0; a < 3; ++a) {
    b.d[a] = d[a];
    b.lo[a] = lo[a];
    b.N[a] = N[a];
  }
  return b;
}

static int grid_for(int64_t n, int per = 256) {
  int64_t b = (n + per - 1) / per;
  if (b > 4096) b = 4096;
  if (b < 1) b = 1;
  return (int)b;
}

hipError_t launch_cnn_features(bf16raw* feat, const int d[3], const int lo[3], const int N[3],
                               const int* vox, const double* chic, int nb,
                               const c64* const vec[kCnnKrylov], const double inv[kCnnKrylov],
                               hipStream_t st) {
  const size_t nv = (size_t)d[0] * d[1] * d[2];
  hipError_t e = hipMemsetAsync(feat, 0, nv * kCnnIn * sizeof(bf16raw), st);
  if (e != hipSuccess || nb == 0) return e;
  KrylovIn kin;
  for (int q = 0; q < kCnnKrylov; ++q) {
    kin.v[q] = vec[q];
    kin.inv[q] = inv[q];
  }
  k_cnn_features<<<grid_for(nb), 256, 0, st>>>(feat, mkbox(d, lo, N), vox, chic, nb, kin);
  return hipGetLastError();
}

hipError_t launch_cnn_target(float* tgt, const int d[3], const int lo[3], const int N[3],
                             const int* vox, int nb, const c64* w, double s, hipStream_t st) {
  const size_t nv = (size_t)d[0] * d[1] * d[2];
  hipError_t e = hipMemsetAsync(tgt, 0, nv * kCnnOut * sizeof(float), st);
  if (e != hipSuccess || nb == 0) return e;
  k_cnn_target<<<grid_for(nb), 256, 0, st>>>(tgt, mkbox(d, lo, N), vox, nb, w,
                                             s > 0 ? 1.0 / s : 0.0);
  return hipGetLastError();
}

hipError_t launch_cnn_gather(c64* x, const float* out, const int d[3], const int lo[3],
                             const int N[3], const int* vox, int nb, double s, hipStream_t st) {
  if (nb == 0) return hipSuccess;
  k_cnn_gather<<<grid_for(nb), 256, 0, st>>>(x, out, mkbox(d, lo, N), vox, nb, s);
  return hipGetLastError();
}

// ------------------------------------------------------------------ host
static int64_t bf16_weights_total() {
  int64_t n = 0;
  for (int l = 0; l < kCnnLayers; ++l) n += 27 * (int64_t)kCnnCh[l] * kCnnCh[l + 1];
  return n;
}
static int64_t bf16_weight_offset(int l) {
  int64_t n = 0;
  for (int q = 0; q < l; ++q) n += 27 * (int64_t)kCnnCh[q] * kCnnCh[q + 1];
  return n;
}

hipError_t cnn_alloc(Cnn& c) {
  c.off = cnn_offsets();
  const size_t np = (size_t)c.off.total;
  hipError_t e;
  if ((e = dev_malloc(&c.p, np * 4)) != hipSuccess) return e;
  if ((e = dev_malloc(&c.m, np * 4)) != hipSuccess) return e;
  if ((e = dev_malloc(&c.v, np * 4)) != hipSuccess) return e;
  if ((e = dev_malloc(&c.g, np * 4)) != hipSuccess) return e;
  if ((e = hipMemset(c.m, 0, np * 4)) != hipSuccess) return e;
  if ((e = hipMemset(c.v, 0, np * 4)) != hipSuccess) return e;
  const size_t nw = (size_t)bf16_weights_total();
  if ((e = dev_malloc(&c.wf, nw * 2)) != hipSuccess) return e;
  if ((e = dev_malloc(&c.wb, nw * 2)) != hipSuccess) return e;
  if ((e = dev_malloc(&c.loss, 4 * 4096 * 2)) != hipSuccess) return e;
  if ((e = hipHostMalloc(&c.hostloss, 2 * sizeof(float))) != hipSuccess) return e;
  return hipSuccess;
}

void cnn_free(Cnn& c) {
  void* ps[] = {c.p, c.m, c.v, c.g, c.wf, c.wb, c.out, c.wpart, c.loss, c.gbuf[0], c.gbuf[1],
                c.act[1], c.act[2], c.act[3]};
  for (void* q : ps)
    if (q) (void)hipFree(q);
  if (c.hostloss) (void)hipHostFree(c.hostloss);
  c = Cnn();
}

// Weight gradient: one persistent 12-wave workgroup per CU.
static constexpr int kGradBlocks = 256;
// Convolution: z layers per workgroup so that about two workgroups per CU
// exist (each takes two more layers than it writes).
static constexpr int kConvBlocks = 512;

hipError_t cnn_ensure_ws(Cnn& c, size_t vox) {
  if (vox <= c.ws_vox) return hipSuccess;
  void* old[] = {c.out, c.gbuf[0], c.gbuf[1], c.act[1], c.act[2], c.act[3], c.wpart};
  for (void* q : old)
    if (q) (void)hipFree(q);
  c.out = nullptr;
  c.gbuf[0] = c.gbuf[1] = c.act[1] = c.act[2] = c.act[3] = nullptr;
  c.wpart = nullptr;
  c.ws_vox = 0;
  hipError_t e;
  if ((e = dev_malloc(&c.out, vox * 16 * 4)) != hipSuccess) return e;
  for (int k = 0; k < 2; ++k)
    if ((e = dev_malloc(&c.gbuf[k], vox * 32 * 2)) != hipSuccess) return e;
  for (int l = 1; l < kCnnLayers; ++l)
    if ((e = dev_malloc(&c.act[l], vox * kCnnCh[l] * 2)) != hipSuccess) return e;
  const size_t maxlayer = 27 * 32 * 32 + 32;
  if ((e = dev_malloc(&c.wpart, (size_t)kGradBlocks * maxlayer * 4)) != hipSuccess) return e;
  c.ws_vox = vox;
  return hipSuccess;
}

hipError_t cnn_refresh_bf16(Cnn& c, hipStream_t s) {
  k_refresh_bf16<<<256, 256, 0, s>>>(c.p, c.wf, c.wb, c.off);
  return hipGetLastError();
}

static ConvDims conv_dims(const int d[3]) {
  ConvDims c;
  c.d0 = d[0];
  c.d1 = d[1];
  c.d2 = d[2];
  c.tx = (d[0] + CT - 1) / CT;
  c.ty = (d[1] + CT - 1) / CT;
  const int64_t nt = (int64_t)c.tx * c.ty;
  c.zc = (int)std::min<int64_t>(d[2], (nt * d[2] + kConvBlocks - 1) / kConvBlocks);
  return c;
}

static GradDims grad_dims(const int d[3]) {
  GradDims c;
  c.d0 = d[0];
  c.d1 = d[1];
  c.d2 = d[2];
  c.tx = (d[0] + TX - 1) / TX;
  c.ty = (d[1] + TY - 1) / TY;
  c.tz = (d[2] + TZ - 1) / TZ;
  c.ntiles = c.tx * c.ty * c.tz;
  return c;
}

template <int CIN, int COUT, int MODE>
static void conv(const ConvDims& cd, const bf16raw* in, const bf16raw* w, const float* bias,
                 bf16raw* ob, float* of, const bf16raw* ref, hipStream_t s) {
  const int grid = cd.tx * cd.ty * ((cd.d2 + cd.zc - 1) / cd.zc);
  k_conv3d<CIN, COUT, MODE><<<grid, CNT, 0, s>>>(in, w, bias, ob, of, ref, cd);
}

template <int COUT>
static void wgrad(const GradDims& cd, const bf16raw* in, const bf16raw* g, float* part,
                  float* out, hipStream_t s) {
  const int grid = cd.ntiles < kGradBlocks ? cd.ntiles : kGradBlocks;
  k_conv3d_wgrad<COUT><<<grid, GNT, 0, s>>>(in, g, part, cd);
  const int n = 27 * 32 * COUT + COUT;
  k_reduce_parts<COUT><<<(n + 63) / 64, 256, 0, s>>>(part, grid, out);
}

hipError_t cnn_forward(Cnn& c, const int d[3], const bf16raw* feat, float* out, hipStream_t s) {
  const ConvDims cd = conv_dims(d);
  hipError_t e = cnn_ensure_ws(c, (size_t)d[0] * d[1] * d[2]);
  if (e != hipSuccess) return e;
  c.act[0] = const_cast<bf16raw*>(feat);
  conv<32, 32, 0>(cd, feat, c.wf + bf16_weight_offset(0), c.p + c.off.b[0], c.act[1], nullptr,
                  nullptr, s);
  conv<32, 32, 0>(cd, c.act[1], c.wf + bf16_weight_offset(1), c.p + c.off.b[1], c.act[2],
                  nullptr, nullptr, s);
  conv<32, 32, 0>(cd, c.act[2], c.wf + bf16_weight_offset(2), c.p + c.off.b[2], c.act[3],
                  nullptr, nullptr, s);
  conv<32, 16, 1>(cd, c.act[3], c.wf + bf16_weight_offset(3), c.p + c.off.b[3], nullptr,
                  out ? out : c.out, nullptr, s);
  return hipGetLastError();
}

hipError_t cnn_backward(Cnn& c, const int d[3], const float* target, float* loss_host,
                        hipStream_t s) {
  const ConvDims cd = conv_dims(d);
  const GradDims cw = grad_dims(d);
  const size_t nv = (size_t)d[0] * d[1] * d[2];
  const int lb = std::min(grid_for((int64_t)nv, 256), kLossBlocks);
  k_loss_partial<<<lb, 256, 0, s>>>(c.out, target, c.act[0], nv, c.loss + 2);
  k_loss_final<<<1, 256, 0, s>>>(c.loss + 2, lb, c.loss);
  k_loss_grad<<<grid_for((int64_t)nv * 16), 256, 0, s>>>(c.out, target, c.act[0], c.loss, nv,
                                                         c.gbuf[0]);
  // layer 4 (32 -> 16): weight gradient, then data gradient masked by ReLU'
  wgrad<16>(cw, c.act[3], c.gbuf[0], c.wpart, c.g + c.off.w[3], s);
  conv<16, 32, 2>(cd, c.gbuf[0], c.wb + bf16_weight_offset(3), nullptr, c.gbuf[1], nullptr,
                  c.act[3], s);
  wgrad<32>(cw, c.act[2], c.gbuf[1], c.wpart, c.g + c.off.w[2], s);
  conv<32, 32, 2>(cd, c.gbuf[1], c.wb + bf16_weight_offset(2), nullptr, c.gbuf[0], nullptr,
                  c.act[2], s);
  wgrad<32>(cw, c.act[1], c.gbuf[0], c.wpart, c.g + c.off.w[1], s);
  conv<32, 32, 2>(cd, c.gbuf[0], c.wb + bf16_weight_offset(1), nullptr, c.gbuf[1], nullptr,
                  c.act[1], s);
  wgrad<32>(cw, c.act[0], c.gbuf[1], c.wpart, c.g + c.off.w[0], s);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (loss_host) {
    if ((e = hipMemcpyAsync(c.hostloss, c.loss, 2 * sizeof(float), hipMemcpyDeviceToHost, s)) !=
        hipSuccess)
      return e;
    if ((e = hipStreamSynchronize(s)) != hipSuccess) return e;
    *loss_host = c.hostloss[1] > 0 ? c.hostloss[0] / c.hostloss[1] : 0.f;
  }
  return hipSuccess;
}

hipError_t cnn_adam(Cnn& c, float lr, hipStream_t s) {
  c.step += 1;
  const float c1 = 1.f - powf(0.9f, (float)c.step), c2 = 1.f - powf(0.999f, (float)c.step);
  k_adam<<<grid_for(c.off.total), 256, 0, s>>>(c.p, c.m, c.v, c.g, c.off.total, lr, c1, c2);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return cnn_refresh_bf16(c, s);
}

}  // namespace vie
