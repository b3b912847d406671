// Far-field amplitude (eq. 25 with the radiation-zone Green's function):
//   F(r) = k0^2 h^3 / (4 pi) (I - r r) sum_n w_n exp(-i k0 r . r_n),
// reported as (F_theta, F_phi) = (theta-hat . F, phi-hat . F).
//
// The sum over voxels is a dense complex contraction [directions x voxels] x
// [voxels x 3R] run on FP64 MFMA (v_mfma_f64_16x16x4f64).  The phase matrix is
// never stored: the body voxels are grouped into aligned blocks of 16 voxels
// (shape bx x by x bz, chosen per body to minimise padding), and for a voxel
// at block origin o_b plus offset u the phase factors as
//   exp(-i k0 r.(o + h(o_b + u - c))) = P(r) S(r, b) A(r, u),
// P(r) = exp(-i k0 r.o),  S(r, b) = exp(-i k0 h r.(o_b - c)),  A(r, u) = exp(-i k0 h r.u)
// (c the reference point, see FarGeom).
// A is the same for every block, so it stays in registers as the MFMA's left
// operand for the whole kernel; each block contributes
//   G(r, b, qc) = sum_u A(r, u) W(b, u, qc)   (16x16x16 complex tiles on MFMA)
// and is scaled by S(r, b) (one sincos per direction and block) and summed.
// The accumulation over blocks is split across workgroups (K-split) and
// reduced in fixed order by a second kernel that projects onto theta-hat /
// phi-hat and applies P and the constant.
//
// Directions that share theta share the phase's z factor exp(-i k0 h cos(theta) z),
// so a sweep on a (theta, phi) grid needs the voxels only once per theta:
//   U(theta, x, y) = sum_z w(x, y, z) exp(-i k0 h cos(theta) (z - c_z))   (k_ff_columns)
//   F(theta, phi)  = sum_xy U(theta, x, y) exp(-i k0 (r_x x + r_y y))
// and the second sum is the same contraction over blocks of 16 columns.  On
// the 128-cell metasurface (193,248 voxels in 16,384 columns) a 180 x 360
// sweep of two channels does a twelfth of the contraction.
#include <string.h>

#include <algorithm>
#include <vector>

#include "kernels.h"

namespace vie {

typedef double d4 __attribute__((ext_vector_type(4)));

static constexpr int FF_QC = 3;          // complex columns per block (components)
static constexpr int FF_BS = 16;         // voxels per block (MFMA K = 4 per step, 4 steps)
static constexpr int FF_TB = 16;         // blocks per tile (MFMA N)
static constexpr int FF_WAVES = 4;       // waves per workgroup, 16 directions each
static constexpr int FF_DIRS = 16 * FF_WAVES;
static constexpr int FF_TILE = FF_QC * FF_BS * FF_TB;  // c64 per packed tile

// ------------------------------------------------------------ host: blocks
namespace {
const int kShapes[][3] = {{16, 1, 1}, {8, 2, 1}, {4, 4, 1}, {4, 2, 2}, {2, 4, 2},
                          {2, 2, 4}, {1, 4, 4}, {2, 8, 1}, {1, 16, 1}, {1, 1, 16}};
constexpr int kNumShapes = sizeof(kShapes) / sizeof(kShapes[0]);

struct VoxIJK {
  int i, j, z;
};
}  // namespace

void far_blocks_build(const int* vox, int nb, const int N[3], FarBlocks& fb) {
  std::vector<VoxIJK> p(nb);
  for (int k = 0; k < nb; ++k) {
    const int lin = vox[k];
    p[k] = {lin % N[0], (lin / N[0]) % N[1], lin / (N[0] * N[1])};
  }
  // blocks per band of H z layers for every shape with bz dividing H
  // (aligned blocks of such shapes never cross a band boundary)
  auto count_bands = [&](int H, std::vector<std::vector<int64_t>>& cnt) {
    const int nbands = (N[2] + H - 1) / H;
    cnt.assign(kNumShapes, std::vector<int64_t>(nbands, -1));
    std::vector<uint8_t> mark;
    for (int s = 0; s < kNumShapes; ++s) {
      const int bx = kShapes[s][0], by = kShapes[s][1], bz = kShapes[s][2];
      if (H % bz) continue;
      const int gx = (N[0] + bx - 1) / bx, gy = (N[1] + by - 1) / by, gz = (N[2] + bz - 1) / bz;
      mark.assign((size_t)gx * gy * gz, 0);
      std::fill(cnt[s].begin(), cnt[s].end(), 0);
      for (const VoxIJK& v : p) {
        const size_t key = ((size_t)(v.z / bz) * gy + v.j / by) * gx + v.i / bx;
        if (!mark[key]) {
          mark[key] = 1;
          ++cnt[s][v.z / H];
        }
      }
    }
    return nbands;
  };
  // pick the band height (4 or 16 layers) and per-band shape with the fewest blocks
  int bestH = 16;
  std::vector<int> best_choice;
  int64_t best_total = -1;
  for (int H : {4, 16}) {
    std::vector<std::vector<int64_t>> cnt;
    const int nbands = count_bands(H, cnt);
    std::vector<int> choice(nbands, 0);
    int64_t total = 0;
    for (int band = 0; band < nbands; ++band) {
      int64_t bc = -1;
      for (int s = 0; s < kNumShapes; ++s)
        if (cnt[s][band] >= 0 && (bc < 0 || cnt[s][band] < bc)) {
          bc = cnt[s][band];
          choice[band] = s;
        }
      total += bc;
    }
    if (best_total < 0 || total < best_total) {
      best_total = total;
      bestH = H;
      best_choice = choice;
    }
  }
  // one group per shape in use; blocks numbered in (z, y, x) block order
  fb.groups.clear();
  fb.org.clear();
  fb.vi.clear();
  fb.nblk = 0;
  int tiles = 0;
  for (int s = 0; s < kNumShapes; ++s) {
    bool used = false;
    for (int c : best_choice) used |= (c == s);
    if (!used) continue;
    const int bx = kShapes[s][0], by = kShapes[s][1], bz = kShapes[s][2];
    const int gx = (N[0] + bx - 1) / bx, gy = (N[1] + by - 1) / by, gz = (N[2] + bz - 1) / bz;
    std::vector<int> id((size_t)gx * gy * gz, -1);
    for (const VoxIJK& v : p)
      if (best_choice[v.z / bestH] == s) id[((size_t)(v.z / bz) * gy + v.j / by) * gx + v.i / bx] = 0;
    const size_t base = fb.org.size() / 4;
    int nblk = 0;
    for (int zb = 0; zb < gz; ++zb)
      for (int yb = 0; yb < gy; ++yb)
        for (int xb = 0; xb < gx; ++xb) {
          int& e = id[((size_t)zb * gy + yb) * gx + xb];
          if (e < 0) continue;
          e = nblk++;
          fb.org.insert(fb.org.end(), {xb * bx, yb * by, zb * bz, 0});
        }
    if (nblk == 0) continue;  // a shape chosen only for empty bands
    const int padded = (nblk + FF_TB - 1) / FF_TB * FF_TB;
    fb.org.resize((base + padded) * 4, 0);
    fb.vi.resize((base + padded) * FF_BS, -1);
    for (int k = 0; k < nb; ++k) {
      const VoxIJK& v = p[k];
      if (best_choice[v.z / bestH] != s) continue;
      const int b = id[((size_t)(v.z / bz) * gy + v.j / by) * gx + v.i / bx];
      const int u = v.i % bx + bx * (v.j % by + by * (v.z % bz));
      fb.vi[(base + b) * FF_BS + u] = k;
    }
    FarGroup gr;
    gr.shape[0] = bx;
    gr.shape[1] = by;
    gr.shape[2] = bz;
    gr.tile0 = tiles;
    gr.ntiles = padded / FF_TB;
    fb.groups.push_back(gr);
    tiles += gr.ntiles;
    fb.nblk += nblk;
  }
  fb.ntiles = tiles;
}

void far_columns_build(const int* vox, int nb, const int N[3], FarColumns& fc) {
  const int plane = N[0] * N[1];
  std::vector<int> cnt(plane, 0);
  for (int k = 0; k < nb; ++k) ++cnt[vox[k] % plane];
  // the lateral block shape that covers the columns with the fewest blocks
  const int shapes[][2] = {{16, 1}, {8, 2}, {4, 4}, {2, 8}, {1, 16}};
  int best = -1, nblk = 0;
  for (int s = 0; s < 5; ++s) {
    const int bx = shapes[s][0], by = shapes[s][1];
    int n = 0;
    for (int y0 = 0; y0 < N[1]; y0 += by)
      for (int x0 = 0; x0 < N[0]; x0 += bx) {
        bool any = false;
        for (int y = y0; y < std::min(N[1], y0 + by) && !any; ++y)
          for (int x = x0; x < std::min(N[0], x0 + bx) && !any; ++x) any = cnt[y * N[0] + x] > 0;
        n += any;
      }
    if (best < 0 || n < nblk) {
      best = s;
      nblk = n;
    }
  }
  fc.bx = shapes[best][0];
  fc.by = shapes[best][1];
  fc.ntiles = (nblk + FF_TB - 1) / FF_TB;
  const size_t nslot = (size_t)fc.ntiles * FF_TB * FF_BS;
  fc.org.assign((size_t)fc.ntiles * FF_TB * 4, 0);
  fc.ptr.assign(nslot + 1, 0);
  std::vector<int> slot(plane, -1);
  int b = 0;
  for (int y0 = 0; y0 < N[1]; y0 += fc.by)
    for (int x0 = 0; x0 < N[0]; x0 += fc.bx) {
      bool any = false;
      for (int v = 0; v < fc.by; ++v)
        for (int u = 0; u < fc.bx; ++u) {
          const int x = x0 + u, y = y0 + v;
          if (x >= N[0] || y >= N[1] || cnt[y * N[0] + x] == 0) continue;
          any = true;
          slot[y * N[0] + x] = b * FF_BS + v * fc.bx + u;
        }
      if (!any) continue;
      fc.org[(size_t)b * 4 + 0] = x0;
      fc.org[(size_t)b * 4 + 1] = y0;
      ++b;
    }
  for (int c = 0; c < plane; ++c)
    if (slot[c] >= 0) fc.ptr[slot[c] + 1] = cnt[c];
  for (size_t k = 0; k < nslot; ++k) fc.ptr[k + 1] += fc.ptr[k];
  fc.ent.resize((size_t)nb * 2);
  std::vector<int> at(fc.ptr.begin(), fc.ptr.end() - 1);
  for (int k = 0; k < nb; ++k) {  // ascending voxels: each column's entries ascend in z
    const int e = at[slot[vox[k] % plane]]++;
    fc.ent[(size_t)e * 2] = k;
    fc.ent[(size_t)e * 2 + 1] = vox[k] / plane;
  }
}

FarGeom far_geom(double k0, double h, const double o[3], int pad, const int N[3], double half) {
  FarGeom g = {k0, h, {0, 0, 0}, half, {0, 0, 0}, 16};
  for (int a = 0; a < 3; ++a) {
    g.nmax = std::max(g.nmax, N[a]);
    const double near = rint(pad - o[a] / h);
    g.c[a] = near > 0.0 ? (near < N[a] - 1 ? (int)near : N[a] - 1) : 0;
    g.o[a] = fma(h, (double)(g.c[a] - pad), o[a]);
  }
  return g;
}

bool far_groups(const double* theta, int nd, FarGroups& fg) {
  // open-addressed table of the distinct angles (by their bits), at most half
  // as many as directions: beyond that nothing is shared
  const int most = nd / 2;
  if (most < 1) return false;
  int cap = 16;
  while (cap < 2 * most) cap <<= 1;
  std::vector<uint64_t> key(cap);
  std::vector<int> val(cap, -1), id(nd);
  fg.first.assign(1, 0);
  std::vector<int> cnt;
  int last = -1;
  uint64_t lastbits = 0;
  for (int d = 0; d < nd; ++d) {
    uint64_t b;
    memcpy(&b, &theta[d], sizeof(b));
    if (last < 0 || b != lastbits) {
      uint64_t hsh = b * 0x9E3779B97F4A7C15ull;
      int i = (int)((hsh >> 32) & (uint64_t)(cap - 1));
      while (val[i] >= 0 && key[i] != b) i = (i + 1) & (cap - 1);
      if (val[i] < 0) {
        if ((int)cnt.size() >= most) return false;
        key[i] = b;
        val[i] = (int)cnt.size();
        cnt.push_back(0);
      }
      last = val[i];
      lastbits = b;
    }
    id[d] = last;
    ++cnt[last];
  }
  const int ng = (int)cnt.size();
  fg.first.resize(ng + 1);
  for (int g = 0; g < ng; ++g) fg.first[g + 1] = fg.first[g] + cnt[g];
  std::vector<int> at(fg.first.begin(), fg.first.end() - 1);
  fg.perm.resize(nd);
  for (int d = 0; d < nd; ++d) fg.perm[at[id[d]]++] = d;
  // direction tiles: up to 64 directions of one group each
  fg.tile.clear();
  fg.tile0.assign(1, 0);
  fg.rows = 0;
  for (int g = 0; g < ng; ++g) {
    for (int k = 0; k < cnt[g]; k += FF_DIRS) {
      const int n = std::min(FF_DIRS, cnt[g] - k);
      fg.tile.insert(fg.tile.end(), {fg.first[g] + k, n, g, 0});
      fg.rows += (n + 15) / 16 * 16;
    }
    fg.tile0.push_back((int)(fg.tile.size() / 4));
  }
  return true;
}

// ------------------------------------------------------------ kernels
// Wd[q][tile][c][u][s] = w of right-hand side q (blockIdx.y), component c at
// offset u of block tile*16 + s (zero where the block has no body voxel).
__global__ void k_ff_pack(FarSrc f, const int* __restrict__ blk_vi, int ntiles,
                          c64* __restrict__ Wd) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (int64_t)ntiles * FF_TILE) return;
  const int s = (int)(e % FF_TB);
  const int u = (int)((e / FF_TB) % FF_BS);
  const int c = (int)((e / (FF_TB * FF_BS)) % FF_QC);
  const int64_t tile = e / FF_TILE;
  const int vi = blk_vi[(tile * FF_TB + s) * FF_BS + u];
  c64 v = mk(0.0, 0.0);
  if (vi >= 0) v = f.at(f.roff[blockIdx.y], c, vi);
  Wd[(int64_t)blockIdx.y * ntiles * FF_TILE + e] = v;
}

// dirs[p] = (r-hat, theta-hat, phi-hat) of the angles ang[d] = theta,
// ang[nd + d] = phi of direction d = perm[p] (p itself without perm).  On the device because the host's trigonometry and a
// 72-byte upload per direction cost more than the sweep's copies otherwise.
__global__ void k_far_frames(const double* __restrict__ ang, const int* __restrict__ perm, int nd,
                             double* __restrict__ dirs) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= nd) return;
  const int d = perm ? perm[p] : p;
  double st, ct, sp, cp;
  sincos(ang[d], &st, &ct);
  sincos(ang[nd + d], &sp, &cp);
  double* D = dirs + (int64_t)p * 9;
  D[0] = st * cp;
  D[1] = st * sp;
  D[2] = ct;
  D[3] = ct * cp;
  D[4] = ct * sp;
  D[5] = -st;
  D[6] = -sp;
  D[7] = cp;
  D[8] = 0.0;
}

struct FfGeom {
  double kh, khl;  // -k0 h to twice the precision
  double split;    // see FfAxes
  int c[3];
};

// Phases per voxel along the axes, -k0 h r, each split in two parts: whole
// multiples of a quantum (adding and taking away `split` = 3/2 of 2^52 quanta
// leaves them) and the rest.  The quantum is such that products with voxel
// offsets and their sums are exact in the first parts, so a block's phase and
// an offset's inside it have no error of their own: where one takes back what
// the other has put on (a body near the reference point) nothing is left.
struct FfAxes {
  double x, y, z, xl, yl, zl;
  __device__ __forceinline__ void set(const FfGeom& g, double rx, double ry, double rz) {
    part(g, rx, x, xl);
    part(g, ry, y, yl);
    part(g, rz, z, zl);
  }
  // (written out with fma: the same bits wherever it is inlined)
  static __device__ __forceinline__ void part(const FfGeom& g, double r, double& hi, double& lo) {
    hi = fma(g.kh, r, g.split) - g.split;
    lo = fma(g.khl, r, fma(g.kh, r, -hi));
  }
  __device__ __forceinline__ double hi(double i, double j, double l) const {
    return fma(z, l, fma(y, j, x * i));
  }
  __device__ __forceinline__ double lo(double i, double j, double l) const {
    return fma(zl, l, fma(yl, j, xl * i));
  }
};
static FfGeom ff_geom(const FarGeom& g) {
  FfGeom f;
  const double kh = g.k0 * g.h;
  f.kh = -kh;
  f.khl = -fma(g.k0, g.h, -kh);
  int e;
  frexp(3.0 * kh * g.nmax, &e);  // every sum is below 2^e
  f.split = ldexp(1.5, e);
  for (int a = 0; a < 3; ++a) f.c[a] = g.c[a];
  return f;
}

// The tile groups of one launch: group g's K-splits start at ks0[g] and end at
// the next group's, its tiles are tile0[g] .. + ntiles[g] - 1, its blocks bx[g] x by[g] x (16 / bx / by).
struct FfGroups {
  int n;
  int ks0[kNumShapes], tile0[kNumShapes], ntiles[kNumShapes], bx[kNumShapes], by[kNumShapes];
};

// The integer nearest x s, as a double and its low bits: adding 3/2 2^52 leaves
// it in the low mantissa bits for |x s| < 2^51 (a conversion to int would end
// at 2^31).
__device__ __forceinline__ double ff_round(double x, double s, int& low) {
  const double t = fma(x, s, 6755399441055744.0);
  low = (int)(unsigned)__double_as_longlong(t);
  return t - 6755399441055744.0;
}

// sin and cos of q pi/2 + r, |r| <= pi/4: Taylor polynomials through r^17 (sin)
// and r^16 (cos); absolute error about 2e-16.
__device__ __forceinline__ void ff_quadrant(double r, int q, double& sn, double& cs) {
  const double r2 = r * r;
  double ps = 2.8114572543455207632e-15;    // 1/17!
  ps = fma(ps, r2, -7.6471637318198164759e-13);  // -1/15!
  ps = fma(ps, r2, 1.6059043836821614599e-10);   // 1/13!
  ps = fma(ps, r2, -2.5052108385441718775e-08);  // -1/11!
  ps = fma(ps, r2, 2.7557319223985890653e-06);   // 1/9!
  ps = fma(ps, r2, -1.9841269841269841270e-04);  // -1/7!
  ps = fma(ps, r2, 8.3333333333333333333e-03);   // 1/5!
  ps = fma(ps, r2, -1.6666666666666666667e-01);  // -1/3!
  const double s0 = fma(r * r2, ps, r);
  double pc = 4.7794773323873852974e-14;    // 1/16!
  pc = fma(pc, r2, -1.1470745597729724714e-11);  // -1/14!
  pc = fma(pc, r2, 2.0876756987868098979e-09);   // 1/12!
  pc = fma(pc, r2, -2.7557319223985890653e-07);  // -1/10!
  pc = fma(pc, r2, 2.4801587301587301587e-05);   // 1/8!
  pc = fma(pc, r2, -1.3888888888888888889e-03);  // -1/6!
  pc = fma(pc, r2, 4.1666666666666666667e-02);   // 1/4!
  pc = fma(pc, r2, -0.5);
  const double c0 = fma(r2, pc, 1.0);
  const bool swap = q & 1;
  const double s1 = swap ? c0 : s0, c1 = swap ? s0 : c0;
  sn = (q & 2) ? -s1 : s1;
  cs = ((q + 1) & 2) ? -c1 : c1;
}

// sin and cos of x + lo for |x| < 1e15, tiny lo: Cody-Waite reduction by pi/2 with
// a two-part constant (FMA).  Branch-free, so it schedules between the matrix
// instructions.
__device__ __forceinline__ void ff_sincos(double x, double lo, double& sn, double& cs) {
  int q;
  const double n = ff_round(x, 0.63661977236758134308, q);  // 2 / pi
  double r = fma(-n, 1.5707963267948966192, x);
  r = fma(-n, 6.123233995736766036e-17, r) + lo;
  ff_quadrant(r, q, sn, cs);
}

// exp(i (x + lo)), |x| < 1e13, from a 256-entry table of exp(2 pi i k / 256) in LDS:
// x = k pi/128 + e with |e| <= pi/256 (two-part FMA reduction), then Taylor
// polynomials of cos e through e^6 and sin e through e^7 (truncation below
// 1e-19) and one complex product with the table entry.
constexpr int FF_NT = 256;
__device__ __forceinline__ c64 ff_table(int k) {  // the angle within pi/4 of its quadrant's
  const int q = (k + FF_NT / 8) / (FF_NT / 4);
  double sn, cs;
  ff_quadrant((k - q * (FF_NT / 4)) * (2.0 * M_PI / FF_NT), q, sn, cs);
  return mk(cs, sn);
}
__device__ __forceinline__ c64 ff_expi(double x, double lo, const c64* sT) {
  int k;
  const double kf = ff_round(x, 40.743665431525205957, k);  // 128 / pi
  double e = fma(-kf, 2.4543692606170259375e-02, x);  // fl(pi) / 128
  e = fma(-kf, 9.5675531183386971e-19, e) + lo;       // (pi - fl(pi)) / 128
  const c64 t = sT[k & (FF_NT - 1)];
  const double e2 = e * e;
  double pc = fma(e2, -1.3888888888888888889e-03, 4.1666666666666666667e-02);
  pc = fma(e2, pc, -0.5);
  const double c = fma(e2, pc, 1.0);
  double ps = fma(e2, -1.9841269841269841270e-04, 8.3333333333333333333e-03);
  ps = fma(e2, ps, -1.6666666666666666667e-01);
  const double sn = fma(e * e2, ps, e);
  return mk(t.re * c - t.im * sn, fma(t.re, sn, t.im * c));
}

// packed tile t -> registers (FF_TILE / 256 c64 and one block origin per thread)
constexpr int FF_PER = FF_TILE / (FF_DIRS * 4);
struct FfPre {
  c64 v[FF_PER];
  int4 o;
};

__device__ __forceinline__ FfPre ff_fetch(const c64* __restrict__ Wd,
                                          const int4* __restrict__ org, int t) {
  FfPre p;
  const c64* src = Wd + (int64_t)t * FF_TILE;
#pragma unroll
  for (int k = 0; k < FF_PER; ++k) p.v[k] = src[k * FF_DIRS * 4 + threadIdx.x];
  p.o = threadIdx.x < FF_TB ? org[(int64_t)t * FF_TB + threadIdx.x] : make_int4(0, 0, 0, 0);
  return p;
}

__device__ __forceinline__ void ff_store(c64* sW, int4* sOrg, const FfPre& p) {
#pragma unroll
  for (int k = 0; k < FF_PER; ++k) sW[k * FF_DIRS * 4 + threadIdx.x] = p.v[k];
  if (threadIdx.x < FF_TB) sOrg[threadIdx.x] = p.o;
}

// G(r, b, qc) = sum_u A(r, u) W(b, u, qc) for one staged tile (complex as
// four real products), and the block scale S(r, b) of this lane's column.
__device__ __forceinline__ void ff_tile(const c64* sW, const int4* sOrg, const c64* sT,
                                        const double (&aR)[4],
                                        const double (&aI)[4], const double (&aIn)[4],
                                        const FfAxes (&rw)[4], const int (&ref)[3], int lane,
                                        d4 (&gR)[FF_QC],
                                        d4 (&gI)[FF_QC], c64 (&S)[4]) {
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) {
    c64 b[FF_QC];
#pragma unroll
    for (int qc = 0; qc < FF_QC; ++qc)
      b[qc] = sW[(qc * FF_BS + 4 * ks + (lane >> 4)) * FF_TB + (lane & 15)];
    if (ks == 0) {
#pragma unroll
      for (int qc = 0; qc < FF_QC; ++qc) {
        gR[qc] = __builtin_amdgcn_mfma_f64_16x16x4f64(aR[ks], b[qc].re, d4{0.0, 0.0, 0.0, 0.0},
                                                      0, 0, 0);
        gI[qc] = __builtin_amdgcn_mfma_f64_16x16x4f64(aR[ks], b[qc].im, d4{0.0, 0.0, 0.0, 0.0},
                                                      0, 0, 0);
      }
    } else {
#pragma unroll
      for (int qc = 0; qc < FF_QC; ++qc) {
        gR[qc] = __builtin_amdgcn_mfma_f64_16x16x4f64(aR[ks], b[qc].re, gR[qc], 0, 0, 0);
        gI[qc] = __builtin_amdgcn_mfma_f64_16x16x4f64(aR[ks], b[qc].im, gI[qc], 0, 0, 0);
      }
    }
#pragma unroll
    for (int qc = 0; qc < FF_QC; ++qc) {
      gR[qc] = __builtin_amdgcn_mfma_f64_16x16x4f64(aIn[ks], b[qc].im, gR[qc], 0, 0, 0);
      gI[qc] = __builtin_amdgcn_mfma_f64_16x16x4f64(aI[ks], b[qc].re, gI[qc], 0, 0, 0);
    }
  }
  const int4 ob = sOrg[lane & 15];
  const double ox = ob.x - ref[0], oy = ob.y - ref[1], oz = ob.z - ref[2];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    S[r] = ff_expi(rw[r].hi(ox, oy, oz), rw[r].lo(ox, oy, oz), sT);
  }
}

__device__ __forceinline__ void ff_accum(const d4 (&gR)[FF_QC], const d4 (&gI)[FF_QC],
                                         const c64 (&S)[4], c64 (&acc)[4][FF_QC]) {
#pragma unroll
  for (int qc = 0; qc < FF_QC; ++qc)
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[r][qc] = cfma(S[r], mk(gR[qc][r], gI[qc][r]), acc[r][qc]);
}

// Sums over columns of z: U of theta group g0 + g (g < ng) and right-hand
// side q, written as the packed operand Wd[q][g][tile] of the lateral
// contraction.  One thread per column slot (16 of a block are neighbouring
// lanes, so a block's loads are contiguous), FF_CG groups per pass over the
// column's voxels, whose z factors sit in LDS; FP64 VALU bound (24 complex
// multiply-adds per voxel and pass against 56 bytes read).
constexpr int FF_CG = 8;
constexpr int FF_NZ = 256;  // most z layers of a grid
__global__ __launch_bounds__(256) void k_ff_columns(FarSrc f, const int* __restrict__ ptr,
                                                    const int2* __restrict__ ent, int ntiles,
                                                    const int* __restrict__ gfirst, int g0, int ng,
                                                    const double* __restrict__ dirs, FfGeom fg,
                                                    int nz, c64* __restrict__ Wd) {
  __shared__ c64 sT[FF_CG][FF_NZ];
  const int gb = blockIdx.y * FF_CG;
  for (int k = threadIdx.x; k < FF_CG * nz; k += 256) {
    const int g = k / nz, z = k % nz;
    double sn = 0.0, cs = 0.0;
    if (gb + g < ng) {
      double hi, lo;
      FfAxes::part(fg, dirs[(int64_t)gfirst[g0 + gb + g] * 9 + 2], hi, lo);
      ff_sincos(hi * (z - fg.c[2]), lo * (z - fg.c[2]), sn, cs);
    }
    sT[g][z] = mk(cs, sn);
  }
  __syncthreads();
  const int p = blockIdx.x * 256 + threadIdx.x;
  const int64_t off = f.roff[blockIdx.z];
  c64 acc[FF_CG][FF_QC];
#pragma unroll
  for (int g = 0; g < FF_CG; ++g)
#pragma unroll
    for (int c = 0; c < FF_QC; ++c) acc[g][c] = mk(0.0, 0.0);
  const int k1 = ptr[p + 1];
  for (int k = ptr[p]; k < k1; ++k) {
    const int2 e = ent[k];
    c64 wv[FF_QC];
#pragma unroll
    for (int c = 0; c < FF_QC; ++c) wv[c] = f.at(off, c, e.x);
#pragma unroll
    for (int g = 0; g < FF_CG; ++g) {
      const c64 t = sT[g][e.y];
#pragma unroll
      for (int c = 0; c < FF_QC; ++c) acc[g][c] = cfma(t, wv[c], acc[g][c]);
    }
  }
  const int u = threadIdx.x & 15, s = threadIdx.x >> 4;
#pragma unroll
  for (int g = 0; g < FF_CG; ++g) {
    if (gb + g >= ng) break;
    c64* o = Wd + (((int64_t)blockIdx.z * ng + gb + g) * ntiles + blockIdx.x) * FF_TILE;
#pragma unroll
    for (int c = 0; c < FF_QC; ++c) o[(c * FF_BS + u) * FF_TB + s] = acc[g][c];
  }
}

// One workgroup: 64 directions (16 per wave) of right-hand side blockIdx.z
// against the blocks of tiles [t0, t1); with a tile table dt (first direction,
// count, theta group - g0) the directions of one theta group against that
// group's packed columns.  Tiles are double-buffered in LDS (one barrier per
// tile) with a register prefetch; two waves per SIMD so that one wave's scale-
// and-accumulate and phase work runs while the other's matrix products execute.
__global__ __launch_bounds__(FF_DIRS * 4) __attribute__((amdgpu_waves_per_eu(2))) void k_ff_mfma(
    const c64* __restrict__ Wd, int64_t wq, const int4* __restrict__ org, FfGroups gs,
    int tiles_per_split, const double* __restrict__ dirs, const int4* __restrict__ dt, int g0,
    int npos, FfGeom fg, c64* __restrict__ part, int kst) {
  int ks0 = 0, ntiles = gs.ntiles[0], bx = gs.bx[0], by = gs.by[0], tile0 = gs.tile0[0];
#pragma unroll
  for (int g = 1; g < kNumShapes; ++g)
    if (g < gs.n && (int)blockIdx.y >= gs.ks0[g]) {
      ks0 = gs.ks0[g];
      ntiles = gs.ntiles[g];
      bx = gs.bx[g];
      by = gs.by[g];
      tile0 = gs.tile0[g];
    }
  Wd += blockIdx.z * wq + (int64_t)tile0 * FF_TILE;
  org += (int64_t)tile0 * FF_TB;
  int first = blockIdx.x * FF_DIRS, nd = npos;
  if (dt) {
    const int4 t = dt[blockIdx.x];
    first = t.x;
    nd = t.x + t.y;  // positions past the group's last one are idle
    Wd += (int64_t)(t.z - g0) * ntiles * FF_TILE;
  }
  __shared__ c64 sW[2][FF_TILE];
  __shared__ int4 sOrg[2][FF_TB];
  __shared__ c64 sT[FF_NT];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int k = threadIdx.x; k < FF_NT; k += FF_DIRS * 4) sT[k] = ff_table(k);  // visible after the first barrier of the tile loop
  const int dbase = first + wave * 16;
  const int t0 = ((int)blockIdx.y - ks0) * tiles_per_split;
  const int t1 = min(ntiles, t0 + tiles_per_split);

  // left operand A(r, u): direction dbase + lane%16, offsets u = 4 ks + lane/16
  double aR[4], aI[4], aIn[4];
  {
    const int d = dbase + (lane & 15);
    double rx = 0, ry = 0, rz = 0;
    if (d < nd) {
      rx = dirs[d * 9 + 0];
      ry = dirs[d * 9 + 1];
      rz = dirs[d * 9 + 2];
    }
    FfAxes ax;
    ax.set(fg, rx, ry, rz);
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      const int u = 4 * ks + (lane >> 4);
      const int du = u % bx, dv = (u / bx) % by, dw = u / (bx * by);
      double sn, cs;
      ff_sincos(ax.hi(du, dv, dw), ax.lo(du, dv, dw), sn, cs);
      aR[ks] = cs;
      aI[ks] = sn;
      aIn[ks] = -sn;
    }
  }
  // output rows of this lane (FP64 16x16x4 result layout: row lane/16 + 4 r,
  // column lane % 16): directions dbase + lane/16 + 4 r
  FfAxes rw[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int d = dbase + (lane >> 4) + 4 * r;
    double rx = 0, ry = 0, rz = 0;
    if (d < nd) {
      rx = dirs[d * 9 + 0];
      ry = dirs[d * 9 + 1];
      rz = dirs[d * 9 + 2];
    }
    rw[r].set(fg, rx, ry, rz);
  }
  c64 acc[4][FF_QC];
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int qc = 0; qc < FF_QC; ++qc) acc[r][qc] = mk(0.0, 0.0);

  d4 gR[FF_QC], gI[FF_QC];
  c64 S[4];
  FfPre pre;
  if (t0 < t1) pre = ff_fetch(Wd, org, t0);
  for (int t = t0; t < t1; ++t) {
    const int cb = (t - t0) & 1;
    ff_store(sW[cb], sOrg[cb], pre);
    if (t + 1 < t1) pre = ff_fetch(Wd, org, t + 1);
    __syncthreads();
    if (dbase < nd) {
      ff_tile(sW[cb], sOrg[cb], sT, aR, aI, aIn, rw, fg.c, lane, gR, gI, S);
      ff_accum(gR, gI, S, acc);
    }
  }
  // sum over the 16 column blocks (lanes sharing lane / 16), fixed pattern
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int qc = 0; qc < FF_QC; ++qc) {
      double re = acc[r][qc].re, im = acc[r][qc].im;
#pragma unroll
      for (int m = 8; m >= 1; m >>= 1) {
        re += __shfl_xor(re, m, 64);
        im += __shfl_xor(im, m, 64);
      }
      acc[r][qc] = mk(re, im);
    }
  if ((lane & 15) == 0) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int d = dbase + (lane >> 4) + 4 * r;
      if (d >= nd) continue;
#pragma unroll
      for (int qc = 0; qc < FF_QC; ++qc)
        part[(((int64_t)blockIdx.z * npos + d) * FF_QC + qc) * kst + blockIdx.y] = acc[r][qc];
    }
  }
}

// hi + lo += a b to twice the precision.
__device__ __forceinline__ void ff_dot(double& hi, double& lo, double a, double b) {
  const double p = a * b, s = hi + p, t = s - hi;
  lo += ((hi - (s - t)) + (p - t)) + fma(a, b, -p);
  hi = s;
}
// v exp(i (x + lo)) as v + v (exp - 1): a small phase's rounding stays as small as
// the phase.
__device__ __forceinline__ c64 ff_turn(c64 v, double x, double lo) {
  double s, c;
  ff_sincos(0.5 * x, 0.5 * lo, s, c);
  const double im = 2.0 * s * c, re = -2.0 * s * s;
  return mk(v.re + fma(re, v.re, -(im * v.im)), v.im + fma(re, v.im, im * v.re));
}

// F = scale (theta-hat . S, phi-hat . S), S = the sum of the kst partials
// of a (right-hand side, direction position) pair, which are contiguous per
// component; the reference point's phase -k0 r.o enters here, and component c's
// points sit g.half off the grid points along axis c (rooftop faces; 0 for
// voxels).  What is done once per direction is not averaged over the points, so
// its roundings would be most of the error: the phases are kept to twice the
// precision and applied as small corrections.  Position p is direction
// perm[p].  L lanes share a pair: 64 where there are many partials (a
// detector scan splits the voxels into hundreds; one thread walking them took
// 190 us at 181 directions and 341 partials), 1 where a sweep leaves a few.
// Fixed order either way.
template <int L>
__global__ __launch_bounds__(256) void k_farfield_project(const c64* __restrict__ part, int kst,
                                                          int npair, int nd,
                                                          const double* __restrict__ dirs,
                                                          const int* __restrict__ perm,
                                                          double scale, FarGeom g,
                                                          c64* __restrict__ F) {
  const int e = (blockIdx.x * 256 + threadIdx.x) / L, lane = threadIdx.x % L;
  if (e >= npair) return;
  const int pos = e % nd, q = e / nd;
  double D[9];  // requested before the partials
#pragma unroll
  for (int k = 0; k < 9; ++k) D[k] = dirs[(int64_t)pos * 9 + k];
  c64 v[3];
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const c64* p = part + ((int64_t)e * 3 + c) * kst;
    v[c] = mk(0.0, 0.0);
    for (int k = lane; k < kst; k += L) v[c] = v[c] + p[k];
  }
#pragma unroll
  for (int m = L / 2; m >= 1; m >>= 1)
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      v[c].re += __shfl_xor(v[c].re, m, 64);
      v[c].im += __shfl_xor(v[c].im, m, 64);
    }
  double at = 0.0, atl = 0.0;
#pragma unroll
  for (int a = 0; a < 3; ++a) ff_dot(at, atl, D[a], g.o[a]);
  auto turned = [&](double r, c64 w) {
    double x = at, xl = atl;
    ff_dot(x, xl, r, g.half);
    const double ang = -g.k0 * x;
    return ff_turn(w, ang, fma(-g.k0, xl, fma(-g.k0, x, -ang)));
  };
  if constexpr (L > 1) {  // the components side by side in the first lanes
    auto mine = [&](double a, double b, double c) { return lane == 1 ? b : lane == 2 ? c : a; };
    const c64 t = turned(mine(D[0], D[1], D[2]), mk(mine(v[0].re, v[1].re, v[2].re),
                                                    mine(v[0].im, v[1].im, v[2].im)));
#pragma unroll
    for (int c = 0; c < 3; ++c) v[c] = mk(__shfl(t.re, c, 64), __shfl(t.im, c, 64));
    if (lane != 0) return;
  } else {
#pragma unroll
    for (int c = 0; c < 3; ++c) v[c] = turned(D[c], v[c]);
  }
  c64 ft = mk(0.0, 0.0), fp = mk(0.0, 0.0);
  for (int c = 0; c < 3; ++c) {
    ft = ft + D[3 + c] * v[c];
    fp = fp + D[6 + c] * v[c];
  }
  c64* o = F + ((int64_t)q * nd + (perm ? perm[pos] : pos)) * 2;
  o[0] = scale * ft;
  o[1] = scale * fp;
}

static hipError_t far_project_sums(const c64* part, int kst, int npair, int nd,
                                   const double* dirs, const int* perm, const FarGeom& fg, c64* F,
                                   hipStream_t s) {
  const double scale = fg.k0 * fg.k0 * fg.h * fg.h * fg.h / (4.0 * M_PI);
  if (kst > 8)
    k_farfield_project<64><<<(npair + 3) / 4, 256, 0, s>>>(part, kst, npair, nd, dirs, perm, scale,
                                                           fg, F);
  else
    k_farfield_project<1><<<(npair + 255) / 256, 256, 0, s>>>(part, kst, npair, nd, dirs, perm,
                                                              scale, fg, F);
  return hipGetLastError();
}

// Workgroups wanted in one launch: the chip holds 512 (two per CU), and a
// workgroup's own tables cost about as much as three tiles.  181 directions of
// two channels of the 128-cell metasurface: 94 us a call with 512, 104 with
// 1024, 107 with 2048.
static constexpr int kFarBlocks = 512;

// K-splits of `ntiles` tiles when `blocks` workgroups exist without a split.
static int far_split(int ntiles, int blocks) {
  if (ntiles <= 0) return 0;
  const int want = std::max(1, kFarBlocks / std::max(1, blocks));
  const int ks = std::min(ntiles, want);
  const int tps = (ntiles + ks - 1) / ks;
  return (ntiles + tps - 1) / tps;
}

// Tiles per split of a launch over every group of `fb`.
static int far_tps(const FarBlocks& fb, int blocks) {
  int nt = 0;
  for (const FarGroup& gr : fb.groups) nt += gr.ntiles;
  const int want = std::max(1, kFarBlocks / std::max(1, blocks));
  return std::max(1, (nt + want - 1) / want);
}

FarPlan far_plan(const FarBlocks& fb, int nr, int nd) {
  // right-hand sides per launch: as many as keep the packed operand and the
  // partials within 64 MB each
  constexpr int64_t kCap = (int64_t)64 << 20;
  FarPlan p;
  const int64_t wb = (int64_t)std::max(1, fb.ntiles) * FF_TILE * sizeof(c64);
  const int db = (nd + FF_DIRS - 1) / FF_DIRS;
  p.nq = (int)std::max<int64_t>(1, std::min<int64_t>(nr, kCap / wb));
  for (;;) {
    p.tps = far_tps(fb, db * p.nq);
    p.kst = 0;
    for (const FarGroup& gr : fb.groups) p.kst += (gr.ntiles + p.tps - 1) / p.tps;
    if (p.nq == 1 || (int64_t)p.nq * nd * FF_QC * p.kst * (int64_t)sizeof(c64) <= kCap) break;
    p.nq = (p.nq + 1) / 2;
  }
  p.wd = (size_t)p.nq * fb.ntiles * FF_TILE;
  p.part = (size_t)p.nq * nd * FF_QC * p.kst;
  return p;
}

// Whether a sweep goes by theta groups: complex multiply-adds of the lateral
// contraction (whole 16-direction rows x column slots) plus the column sums,
// which run on the VALU at about a quarter of the rate, against the direct
// contraction of every voxel (1.25 slots per voxel).  Below about 3e7 direct
// multiply-adds both are a few launches of latency, and the direct path has
// two fewer.
bool far_by_columns(const FarGroups& fg, int nd, const FarColumns& fc, int nb) {
  const double direct = 1.25 * nd * (double)nb;
  const double cols = (double)fg.rows * fc.ntiles * FF_TB * FF_BS +
                      4.0 * (double)(fg.first.size() - 1) * nb;
  return direct > 3e7 && cols < 0.8 * direct;
}

FarSweepPlan far_sweep_plan(const FarGroups& fg, const FarColumns& fc, int nr, int nd) {
  constexpr int64_t kCap = (int64_t)64 << 20;  // packed operand and partials, as far_plan
  FarSweepPlan p;
  const int ng = (int)fg.first.size() - 1;
  const int64_t gb = (int64_t)fc.ntiles * FF_TILE * sizeof(c64);
  p.nq = (int)std::max<int64_t>(1, std::min<int64_t>(nr, kCap / std::max<int64_t>(gb, 1)));
  for (;;) {
    p.ngc = (int)std::max<int64_t>(1, std::min<int64_t>(ng, kCap / (gb * p.nq)));
    const int64_t blocks = (int64_t)(fg.tile.size() / 4) * p.ngc / ng * p.nq;
    p.kst = far_split(fc.ntiles, (int)std::min<int64_t>(blocks, kFarBlocks));
    if (p.nq == 1 || (int64_t)p.nq * nd * FF_QC * p.kst * (int64_t)sizeof(c64) <= kCap) break;
    p.nq = (p.nq + 1) / 2;
  }
  p.wd = (size_t)p.nq * p.ngc * fc.ntiles * FF_TILE;
  p.part = (size_t)p.nq * nd * FF_QC * p.kst;
  return p;
}

hipError_t launch_far_frames(const double* ang, const int* perm, int nd, double* dirs,
                             hipStream_t s) {
  k_far_frames<<<(nd + 255) / 256, 256, 0, s>>>(ang, perm, nd, dirs);
  return hipGetLastError();
}

hipError_t launch_farfield_sweep(const FarSrc& src, int nr, const FarColumns& fc, const int* ptr,
                                 const int* org, const int* ent, const FarGroups& gr,
                                 const int* perm, const int* first, const int* tile,
                                 const FarSweepPlan& pl, const double* dirs, int nd, int nz,
                                 const FarGeom& geo, c64* Wd, c64* part, c64* F, hipStream_t s) {
  if (nz > FF_NZ) return hipErrorInvalidValue;
  const int ng = (int)gr.first.size() - 1;
  const int tps = (fc.ntiles + pl.kst - 1) / pl.kst;
  const FfGeom fz = ff_geom(geo);
  FfGeom fg = fz;
  fg.c[2] = 0;  // z is in the columns' sums
  FfGroups gs = {};
  gs.n = 1;
  gs.ntiles[0] = fc.ntiles;
  gs.bx[0] = fc.bx;
  gs.by[0] = fc.by;
  for (int q0 = 0; q0 < nr; q0 += pl.nq) {
    const int nq = std::min(pl.nq, nr - q0);
    FarSrc f = src;
    f.roff += q0;
    for (int g0 = 0; g0 < ng; g0 += pl.ngc) {
      const int n = std::min(pl.ngc, ng - g0);
      k_ff_columns<<<dim3(fc.ntiles, (n + FF_CG - 1) / FF_CG, nq), 256, 0, s>>>(
          f, ptr, (const int2*)ent, fc.ntiles, first, g0, n, dirs, fz, nz, Wd);
      hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
      const int d0 = gr.tile0[g0], d1 = gr.tile0[g0 + n];
      k_ff_mfma<<<dim3(d1 - d0, pl.kst, nq), FF_DIRS * 4, 0, s>>>(
          Wd, (int64_t)n * fc.ntiles * FF_TILE, (const int4*)org, gs, tps, dirs,
          (const int4*)tile + d0, g0, nd, fg, part, pl.kst);
      e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
    const hipError_t e = far_project_sums(part, pl.kst, nq * nd, nd, dirs, perm, geo,
                                          F + (int64_t)q0 * nd * 2, s);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_farfield_mfma(const FarSrc& src, int nr, const FarBlocks& fb, const int* blk_vi,
                                const int* blk_org, const FarPlan& pl, const double* dirs, int nd,
                                const FarGeom& geo, c64* Wd, c64* part, c64* F, hipStream_t s) {
  const int ntiles = fb.ntiles;
  const FfGeom fg = ff_geom(geo);
  const int db = (nd + FF_DIRS - 1) / FF_DIRS;
  const int64_t tot = (int64_t)ntiles * FF_TILE;
  // every block shape in one launch, all splits equally long: launched one
  // after the other, each split to fill the chip, the three shapes of the
  // 128-cell metasurface took 85 us of a 146 us call (181 directions, two
  // channels), mostly the workgroups' own tables for 2 tiles each; 94 us a call now
  FfGroups gs = {};
  int ks = 0;
  for (const FarGroup& gr : fb.groups) {
    if (gr.ntiles < 1) continue;
    if (gs.n == kNumShapes) return hipErrorInvalidValue;
    gs.ks0[gs.n] = ks;
    gs.tile0[gs.n] = gr.tile0;
    gs.ntiles[gs.n] = gr.ntiles;
    gs.bx[gs.n] = gr.shape[0];
    gs.by[gs.n++] = gr.shape[1];
    ks += (gr.ntiles + pl.tps - 1) / pl.tps;
  }
  if (ks != pl.kst) return hipErrorInvalidValue;
  for (int q0 = 0; q0 < nr; q0 += pl.nq) {
    const int nq = std::min(pl.nq, nr - q0);
    FarSrc f = src;
    f.roff += q0;
    k_ff_pack<<<dim3((unsigned)((tot + 255) / 256), nq), 256, 0, s>>>(f, blk_vi, ntiles, Wd);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (pl.kst > 0) {
      k_ff_mfma<<<dim3(db, pl.kst, nq), FF_DIRS * 4, 0, s>>>(Wd, tot, (const int4*)blk_org, gs,
                                                             pl.tps, dirs, nullptr, 0, nd, fg, part,
                                                             pl.kst);
      e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
    e = far_project_sums(part, pl.kst, nq * nd, nd, dirs, nullptr, geo, F + (int64_t)q0 * nd * 2,
                         s);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace vie
