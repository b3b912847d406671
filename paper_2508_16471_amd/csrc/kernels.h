// Internal launcher interface between the host runtime and the HIP kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <vector>

#include "common.h"

namespace vie {

// Per-right-hand-side BiCGSTAB state, resident in device memory.
struct KState {
  c64 rho, alpha, omega, beta;
  c64 rho1;        // (rhat, r) of the current residual; rho: of the one before (the
                   // residual update makes it rho)
  double bnorm2;   // ||b||^2
  double rnorm2;   // ||r||^2 (recursive inside a cycle, true after a restart)
  double target2;  // stop the current cycle when rnorm2 <= target2
  int active;      // 1 while this right-hand side iterates
  int it_cycle;    // iterations in the current cycle
  int iters;       // total iterations
  int breakdown;   // why the last cycle broke down: 0 no, 1 rhat.Ap, 2 rhat.r, 3 omega, 4 overflow
  int notdone;     // 1 while the true residual is above tol
  double rh2;      // ||rhat||^2 (shadow residual of the current cycle)
  int cycles;      // FP64 true-residual products (restarts) so far
  int pad_;
  unsigned long long t_done;  // device wall clock when the true residual first met tol (0: not)
};

// Epilogue of the inverse-x pass (y = x - chi * conv, then):
enum EpiMode {
  EPI_PLAIN = 0,  // y only
  EPI_RHV = 1,    // partial sum conj(rhat) . y          (v = A p)
  EPI_TS = 2,     // partial sums conj(y) . x, |y|^2       (t = A s)
  EPI_RESID = 3   // r = b - y, rhat = r, partial |r|^2    (restart)
};

// Geometry of one group of right-hand sides sharing a grid and spectrum.
struct GroupGeom {
  int N[3];     // grid
  int P[3];     // FFT lengths (powers of two >= 2N - 1)
  int Q[3];     // octant extents P/2 + 1
  int64_t n;    // N1 N2 N3
  int nrhs;     // right-hand sides in the group
};

// Body-compressed vectors: the solver stores each right-hand side's vectors
// over its body's voxels only, v[rhs][comp][k] at roff[rhs] + comp nb + k.
struct BodyIdx {
  const int* vox;        // concatenated body-voxel linear indices (ascending per body)
  const int* line_ptr;   // [body][N2 N3 + 1] start of each x-line in the body's list
  const double* chic;    // chi at the body voxels (same order as vox)
  const int* nb;         // [body] body voxels
  const int* voff;       // [body] offset of the body's lists in vox / chic
  const int64_t* roff;   // [rhs] offset of the right-hand side's vector
  const int* rhs_body;   // [rhs] body of each right-hand side
};

// Krylov update fused into the pass that starts a product of body-compressed
// FP64 vectors: the multiplied vector is p = r + beta (p - omega v) or s = r -
// alpha v, stored in `out` on the way.  With npart > 0 the pass folds the
// partials [nrhs][npart][2] that the scalars need (FIN_RHO's, FIN_ALPHA's) and
// takes the decisions of k_finalize; with npart = 0 they are in the state.
enum UpdMode { UPD_NONE = 0, UPD_P = 1, UPD_S = 2 };
struct UpdArgs {
  int mode = UPD_NONE;
  KState* st = nullptr;
  int* flags = nullptr;  // as k_finalize's
  int nrhs = 0, max_iter = 0;
  const c64* part = nullptr;
  int npart = 0;
  const c64* r = nullptr;
  const c64* v = nullptr;
  c64* out = nullptr;  // p (read and written) or s
};
// Partials a fused update may fold itself: beyond, every workgroup reading
// them all costs more than the launch of k_finalize it saves.
static constexpr int kFoldMax = 512;

// Device pointers used by one operator product of a group.
struct MatvecArgs {
  const GroupGeom* g;
  const double* chi;       // [n] of the body, for box vectors (all of one body)
  const void* spec;        // octant spectrum, c64 or c32 per precision
  const void* tw[3];       // twiddle tables per axis (c64 or c32)
  void* bufA;              // x-transformed scratch [nrhs][3][N3][N2][P1]
  void* bufB;              // y-transformed scratch [nrhs][3][N3/zl][P2][zl][P1]
  const int* active;       // [nrhs] or nullptr
  int zvar = 0;            // launch shape of the z pass (autotuned per group/precision)
  const BodyIdx* bi = nullptr;  // non-null: x and y are body-compressed
  const UpdArgs* upd = nullptr;  // update that makes x (then x itself is not read)
  int io32 = 0;  // compressed x and y stored in FP32 (FP32 passes, plain epilogue only);
                 // 2: x stored in bfloat16, y in FP32
  // Approximate products (FP32, bfloat16 x, FP32 y, plain epilogue): with
  // spec16 set the y and z transforms are FP16 transforms on FP16 scratch (see
  // h16_ok for the grids this takes): spec16 the scaled FP16 spectrum, hs the
  // forward scales along x, y, z, hout the inverse x pass's scale back.  Grids
  // of short lines (xy_fused_ok) run three passes on the matrix cores with the
  // operand tables dft16, others five with the splatted twiddles tw16.
  const void* spec16 = nullptr;
  const void* tw16[2] = {nullptr, nullptr};
  const void* dft16 = nullptr;
  float hs[3] = {0.f, 0.f, 0.f};
  float hout = 0.f;
  // Three-pass products only (xy_fused_ok), with npart set: x is an FP32 work
  // vector w; right-hand side q of it is scaled by 1 / ||w_q|| (||w_q||^2
  // summed from the nblk partials npart[q nblk ..] in a fixed order and
  // stored at nrm[q ldn]) and rounded to bfloat16, that vector is stored at
  // vout (bfloat16) and multiplied: the normalisation of an Arnoldi step
  // done inside the next product
  const double* npart = nullptr;
  int nblk = 0;
  double* nrm = nullptr;
  int ldn = 0;
  void* vout = nullptr;
};

// precision 0: FP64 passes, 1: FP32 passes (input/output vectors are FP64)
// epilogue extras: aux (rhat for EPI_RHV, rhat output for EPI_RESID),
// partials [nrhs][blocks][2] (c64), pol/phase tables for EPI_RESID.
struct EpiArgs {
  int mode;
  c64* aux;
  c64* partials;
  int part_blocks;  // filled by the launcher: blocks per right-hand side
  const c64* pol;   // [nrhs][3]
  const c64* ph;    // [nrhs][N1 + N2 + N3]  exp(i k0 khat_a (o_a + h idx))
};

// Dot partials (pairs per right-hand side) of a product's last pass.
int part_blocks_product(const GroupGeom& g, int precision);
// Whether a grid takes the fused x-y passes of short lines (fft_plane.hip).
bool plane_ok(const GroupGeom& g);
int z_block(const GroupGeom& g);        // z planes kept adjacent in the y/z scratch
int64_t bufB_elems(const GroupGeom& g);  // y/z scratch elements per right-hand side
int vec_blocks(const GroupGeom& g);

// x, y: c64 vectors, or c32 when a.io32.
hipError_t launch_matvec(const MatvecArgs& a, int precision, const void* x, void* y, EpiArgs& epi,
                         hipStream_t s, void (*ev_cb)(int kind, bool begin, void* u), void* u);
int z_variants(int precision);  // z-pass launch shapes (0 = FP64, 1 = FP32)
// z pass alone on bufB (autotuning; contents are scratch)
hipError_t launch_z_only(const MatvecArgs& a, int precision, hipStream_t s);
// Packed-FP16 transforms of approximate FP32 products: whether the grid takes
// them, and whether in three passes on the matrix cores (fft_mm16.hip).
bool h16_ok(const GroupGeom& g);
bool xy_fused_ok(const GroupGeom& g);
// timing kinds: the five separate passes (26..30); the three passes are z (28)
// between xy_fwd and yx_inv (31, 32), the x passes before and after it
static constexpr int kH16Kind0 = 26;
// max |re|, |im| of an FP32 octant spectrum (n complex values) as float bits
// atomically maxed into *dmax (zeroed by the caller)
hipError_t launch_spec_absmax(const void* spec32, int64_t n, unsigned* dmax, hipStream_t s);
// Tables of the five passes: the pair-packed FP16 spectrum scaled by gs (Q2 Q3
// P1/2 6 packed pairs, 8 bytes each), the splatted FP16 twiddles of n points.
hipError_t launch_spec_pairs(const void* spec32, void* spec16, const GroupGeom& g, float gs,
                             hipStream_t s);
hipError_t launch_tw_h2(const void* tw32, void* tw16, int n, hipStream_t s);
// Tables of the three passes: DFT operands (with the forward scales) and the
// FP16 spectrum scaled by gs, four z of an entry together.
size_t dft16_table_bytes(const GroupGeom& g);
hipError_t launch_dft16_tables(void* tab, const GroupGeom& g, const float hs[3], hipStream_t s);
size_t spec_cols_bytes(const GroupGeom& g);
hipError_t launch_spec_cols(const void* spec32, void* out, const GroupGeom& g, float gs,
                            hipStream_t s);

// Green spectrum: sample the circulant kernel of component ab into
// work[P3][P2][P1] (c64).
hipError_t launch_green_sample(c64* work, const GroupGeom& g, int ab, double h, double k0,
                               hipStream_t s);
// In-place unpadded 3-D FFT of one P3 x P2 x P1 c64 array (forward).
hipError_t launch_fft3d_full(c64* work, c64* tmp, const GroupGeom& g, const void* tw[3],
                             hipStream_t s);
// y stage of scalar fields, nvec vectors at once (FP64 or FP32; E[a] <= P[a] /
// 2).  Forward: in [vec][fs][E3][E2][P1] -> out [vec][fs][E3][P2][P1], the first
// nf fields; inverse: in [vec][fs][E3][P2][P1] -> out [vec][nf][E3][E2][P1].
hipError_t launch_fft_y_fields(const c64* in, c64* out, const int E[3], const int P[3],
                               const c64* tw1, int nvec, int nf, int fs, bool inverse,
                               const int* active, hipStream_t s);
hipError_t launch_fft_y_fields(const c32* in, c32* out, const int E[3], const int P[3],
                               const c32* tw1, int nvec, int nf, int fs, bool inverse,
                               const int* active, hipStream_t s);
// Octant compression with 1/M scaling into spec64 (and spec32 if non-null).
hipError_t launch_octant(const c64* work, c64* spec64, c32* spec32, const GroupGeom& g, int ab,
                         hipStream_t s);

// Krylov vector kernels on body-compressed FP64 vectors (3 nb per rhs).
// vb = vec_blocks(max 3 nb) workgroups per right-hand side.
int vec_blocks_n(int64_t max_len);
// b = chi pol e^{i k0 khat.r}; r = rhat = b; x = 0 unless keep_x; partials |b|^2.
// mask (nullable): only right-hand sides with mask[rhs] != 0.
hipError_t launch_init_zero_guess(const GroupGeom& g, const BodyIdx& bi, int vb,
                                  const c64* pol, const c64* ph, c64* x, c64* r, c64* rh,
                                  c64* partials, int keep_x, const int* mask, hipStream_t s);
// x += alpha p + omega s, r = s - omega t, one iteration done, partials
// ((rhat, r), |r|^2); omega from the product's partials tpart (ntpart pairs per
// right-hand side) or, with ntpart = 0, from the state.
hipError_t launch_update_xr(const GroupGeom& g, const BodyIdx& bi, int vb, KState* st,
                            const int* active, c64* x, c64* r, const c64* p, const c64* sv,
                            const c64* t, const c64* rh, const c64* tpart, int ntpart,
                            c64* partials, hipStream_t s);
// Finalize reductions (one workgroup per right-hand side, fixed order):
// FIN_RESTART acts on the right-hand sides not done; FIN_PENDING (the same
// restart) on those whose cycle has ended and waits for its true residual.
enum FinWhich {
  FIN_ALPHA = 0,
  FIN_OMEGA = 1,
  FIN_RHO = 2,
  FIN_INIT = 3,
  FIN_RESTART = 4,
  FIN_PENDING = 5
};
struct FinParams {
  double tol2_done;   // converged when ||r_true||^2 <= tol2_done ||b||^2
  double tol2_inner;  // a cycle may stop at ||r||^2 <= tol2_inner ||b||^2 ...
  double eta2;        // ... or at ||r||^2 <= eta2 ||r_cycle_start||^2 (larger of the two)
  int max_iter;
};
hipError_t launch_finalize(int which, int nrhs, int nblk, const c64* partials, KState* st,
                           int* active, const FinParams& fp, hipStream_t s);
hipError_t launch_axpy_real(int64_t n, double a, const c64* x, c64* y, hipStream_t s);

// Far field (eq. 25) on FP64 MFMA.  The body voxels are grouped into aligned
// blocks of 16 voxels.  The block shape (bx x by x bz) is chosen per band of
// z layers to minimise empty slots (a slab and the fins on it want different
// shapes); bands with the same shape form one group of whole tiles of 16.
struct FarGroup {
  int shape[3];
  int tile0, ntiles;
};
struct FarBlocks {
  std::vector<FarGroup> groups;
  int nblk = 0, ntiles = 0;
  std::vector<int> org;  // [ntiles*16][4] block origin (i, j, k, 0) in voxels
  std::vector<int> vi;   // [ntiles*16][16] compressed voxel index at offset u, -1 empty
};
void far_blocks_build(const int* vox, int nb, const int N[3], FarBlocks& fb);
// Launch plan of nr right-hand sides at nd directions: right-hand sides per
// launch, K-split partials per (right-hand side, direction, component), and
// the scratch it needs (c64 counts of the packed operand and the partials).
struct FarPlan {
  int nq = 1, kst = 0, tps = 1;  // tps: tiles per split
  size_t wd = 0, part = 0;
};
FarPlan far_plan(const FarBlocks& fb, int nr, int nd);
// The currents: component c of point k of right-hand side q is
// w[roff[q] + c cs + k], times scale[c cs + k] if given (0 where that is 0,
// whatever w holds).  roff on the device.
struct FarSrc {
  const c64* w;
  const int64_t* roff;
  int64_t cs;
  const double* scale;
  __device__ __forceinline__ c64 at(int64_t off, int c, int k) const {
    if (!scale) return w[off + c * cs + k];
    const double a = scale[c * cs + k];
    return a != 0.0 ? a * w[off + c * cs + k] : mk(0.0, 0.0);
  }
};
// Point (i, j, l) at o + h ((i, j, l) - c), component c's moved by `half` along
// axis c.  Phases are taken relative to the reference point c, the grid point
// nearest the coordinate origin, and its own once per direction at the end: the
// error of a phase grows with its size, and relative to the grid's corner every
// phase of a body about the origin would be large, alike for all its points.
// Against extended precision, 24 rooftop bodies of 10 to 64 cells an axis: 4.5e-16
// (rms 4.9e-16) from the corner, 2.3e-16 (2.6e-16) now, 2.4e-16 (3.2e-16) for a
// direct sum over the faces.
struct FarGeom {
  double k0, h, o[3], half;
  int c[3];
  int nmax;  // largest extent (at least a block's)
};
// Point (0, 0, 0) at o - h pad of a grid of N points.
FarGeom far_geom(double k0, double h, const double o[3], int pad, const int N[3], double half);
// dirs[p][9] = (r, theta-hat, phi-hat) of direction perm[p] (nullable: p) of
// device angles ang = theta[nd], phi[nd].
hipError_t launch_far_frames(const double* ang, const int* perm, int nd, double* dirs,
                             hipStream_t s);
// F[rhs][dir][2] = (F_theta, F_phi) for nr right-hand sides of one body;
// blk_vi / blk_org the device copies of fb.vi / fb.org; dirs[nd][9] = (r,
// theta-hat, phi-hat).  Scratch: Wd pl.wd c64, part pl.part c64.
hipError_t launch_farfield_mfma(const FarSrc& src, int nr, const FarBlocks& fb, const int* blk_vi,
                                const int* blk_org, const FarPlan& pl, const double* dirs, int nd,
                                const FarGeom& geo, c64* Wd, c64* part, c64* F, hipStream_t s);

// Sweeps: the body's voxel columns along z in lateral blocks of 16 (bx by =
// 16), blocks in tiles of 16; slot p = 16 block + offset holds entries
// ptr[p] .. ptr[p + 1] of ent = (voxel, z).
struct FarColumns {
  int bx = 16, by = 1, ntiles = 0;
  std::vector<int> org;  // [ntiles*16][4] block origin (i, j, 0, 0)
  std::vector<int> ptr;  // [ntiles*256 + 1]
  std::vector<int> ent;  // [nb][2]
};
void far_columns_build(const int* vox, int nb, const int N[3], FarColumns& fc);
// Directions grouped by equal theta: group g is positions first[g] ..
// first[g + 1] of perm; tile = (first position, count <= 64, g, 0), those of
// group g from tile0[g]; rows = directions rounded up to 16 per tile.  False
// when more than half of the angles differ.
struct FarGroups {
  std::vector<int> perm, first, tile, tile0;
  int64_t rows = 0;
};
bool far_groups(const double* theta, int nd, FarGroups& fg);
bool far_by_columns(const FarGroups& fg, int nd, const FarColumns& fc, int nb);
// Right-hand sides and theta groups per launch, K-splits, scratch (c64).
struct FarSweepPlan {
  int nq = 1, ngc = 1, kst = 1;
  size_t wd = 0, part = 0;
};
FarSweepPlan far_sweep_plan(const FarGroups& fg, const FarColumns& fc, int nr, int nd);
// As launch_farfield_mfma by theta groups: ptr, org, ent the device copies of
// fc's, perm, first, tile those of gr's, dirs in perm order, nz <= 256 layers.
hipError_t launch_farfield_sweep(const FarSrc& src, int nr, const FarColumns& fc, const int* ptr,
                                 const int* org, const int* ent, const FarGroups& gr,
                                 const int* perm, const int* first, const int* tile,
                                 const FarSweepPlan& pl, const double* dirs, int nd, int nz,
                                 const FarGeom& geo, c64* Wd, c64* part, c64* F, hipStream_t s);
// ||v_rhs||^2 of body-compressed vectors into out[nrhs] (device).
hipError_t launch_vec_norm2(int nrhs, const BodyIdx& bi, const c64* v, double* out,
                            hipStream_t s);
// p[i] = v for i < n (device ints), by a kernel (no memset node when captured).
hipError_t launch_fill_int(int* p, int n, int v, hipStream_t s);
// *out = the device wall clock (constant rate, hipDeviceAttributeWallClockRate
// kHz) when the stream reaches this launch
hipError_t launch_stamp(unsigned long long* out, hipStream_t s);
// Gather a box-layout vector [3][n] into body-compressed storage [3][nb].
hipError_t launch_compress(const c64* box, c64* comp, const int* vox, int nb, int64_t n,
                           hipStream_t s);

}  // namespace vie
