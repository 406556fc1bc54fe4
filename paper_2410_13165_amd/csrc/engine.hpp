// Device-side parameter block and kernel launchers shared by the C ABI layer
// (capi.hip) and the kernels (kernels.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <cstdint>

#include "lattice.hpp"

namespace lbm {

constexpr int kMaxModes = 16;
constexpr int kNumAcc = 6;        // accumulators of the moment reduction
constexpr int kRedBlocks = 1024;  // fixed grid of the deterministic reductions
constexpr int kRedThreads = 256;

enum Scheme : int { kNoWall = 0, kFullWay = 1, kHalfWay = 2 };
// work selected by the `what` mask of lbm_moments (the LBM_MOM_* bits)
enum MomentBits : unsigned { kMomPhi = 1, kMomSums = 2, kMomRmse = 4, kMomEntropy = 8 };
// Storage modes (the values of lbm_precision).  kSplit and kHiLo share the
// layout: float32 g_k = f_k - omega_k phi plus 8 bytes of phi per node
// (float64, or an unevaluated float32 pair hi + lo).
enum Mode : int { kFP64 = 0, kFP32 = 1, kSplit = 2, kHiLo = 3 };
constexpr bool split_layout(int mode) { return mode == kSplit || mode == kHiLo; }
enum FieldKind : int { kFieldNone = 0, kFieldCos = 1, kFieldExp = 2, kFieldTanh = 3 };

// Analytic solution phi*(x, t) = F(x - u t) + R t (see include/lbm.h).
struct FieldDev {
  int kind;
  int nmodes;
  double amp[kMaxModes];
  double phase[kMaxModes];
  double ku[kMaxModes];                 // kappa_j . u
  double kvec[kMaxModes][kMaxDim];
  // half-cell shifts of the half-way wall points, h = dx / 2, per axis a:
  // cos sums (cos(h kappa_ja), sin(h kappa_ja)); exp sums
  // (exp(-h kappa_ja), exp(h kappa_ja))
  double rot[kMaxModes][kMaxDim][2];
  double Rr, W;
  double center[kMaxDim];
};

// Everything a kernel needs about one lattice, passed by value.
struct KParams {
  int d, q;
  int n[kMaxDim];          // nodes per axis, n[0] fastest in memory
  int stride[kMaxDim];     // node strides
  int nodes;
  int rows;                // nodes / n[0]
  long long pstride;       // elements between two population planes
  int bc[kMaxDim];         // 0 periodic, 1 full-way, 2 half-way
  int scheme;              // Scheme of the Dirichlet axes
  int P;                   // wall scheme order
  int K;                   // initialisation order
  double omega[kMaxQ];
  float omega_f[kMaxQ];
  float omega_lo[kMaxQ];    // omega - omega_f, rounded (hi/lo mode)
  signed char cv[kMaxQ][kMaxDim];  // velocities (Sec. 2.3 order)
  int kbar[kMaxQ];                 // c_kbar = -c_k
  double s, tau, dt, dx, R;
  double dtR;              // dt R, the source term of one step (split modes)
  float dtR_hi, dtR_lo;    // dt R as a float32 pair (hi/lo mode)
  float oms_f;             // 1 - s in float32 (hi/lo mode)
  float s_f;
  double origin[kMaxDim];
  double shift[kMaxDim];   // 1/2 on half-way axes, else 0
  double u[kMaxDim];
  double inv_u[kMaxDim];   // 1 / u_j on Dirichlet axes (tangential wall data)
  int wall_data;           // 0: jets of the exact solution; 1: Remark-1 construction
  double phi_ref;          // FP32 mode: mean of phi0
  // rows on a wall of an axis >= 2, listed face by face (see k_wall)
  int nwfaces;
  int wface_axis[2 * kMaxDim];
  int wface_side[2 * kMaxDim];
  int wface_count[2 * kMaxDim];
  int wall_rows;
  // analytic wall data of the x_1 faces: element xoff + row of each
  // population plane (float64 / float32 modes); split mode:
  // xdata[(side * (2d - 1) + slot) * rows + row]
  int xoff;
  double* xdata;
  FieldDev field;
};

// What the marching passes of d = 2 (march.hpp) need of a lattice, by value: a
// tenth of KParams, whose field table they do not read.
struct MarchParams {
  int n0, n1, bc0, bc1;
  long long ps;              // elements between two population planes
  double omega[9];
  float omega_f[9];
  float s_f;
  double s, dt, R, dtR, phi_ref;
  // wall data of the steps of a pass (l = 0, 1, ...):
  // wx[((l * 2 + side) * 3 + slot) * n1 + row], wy[((l * 2 + side) * 3 + slot) * n0 + x]
  const double* wx;
  const double* wy;
};
struct MarchBufs {
  const void* src;
  void* dst;
  const double* phi_src;     // split mode
  double* phi_dst;
};
MarchParams march_params(const KParams& p);

// Output columns of one wavefront's tile in a pass of nl steps: 64 lanes less a
// halo of nl on either side, in whole 64-byte pieces of float64 rows.
__host__ __device__ constexpr int march_width(int nl) { return (64 - 2 * nl) / 8 * 8; }
constexpr int kMarchMaxSteps = 8, kMarchMaxWallSteps = 4;

// Steps (nl: 1 for none, 2, 4 or 8) and rows per tile (yc) of a pass.  block: two
// steps with one tile per block and the state between them in LDS (periodic
// lattices) instead of one per wavefront.
struct MarchPlan {
  int nl, yc;
  bool block;
};
void march_plans(const KParams& p, int mode, MarchPlan (&plans)[4]);
// plan.nl steps of a d = 2 lattice (float64, float32 or split mode) in one
// pass; p.wx / p.wy hold the wall data of those steps.
hipError_t launch_march2(const MarchParams& p, int scheme, int mode, const MarchPlan& plan,
                         const MarchBufs& b, long long n, hipStream_t stream);
// nsteps (at most line_steps) steps of a d = 1 lattice in one launch; p.wx holds the
// wall data of those steps (launch_wall_data1).  A lattice of at most kLineNodes
// nodes is held by one block; longer ones take windows of kLineNodes nodes,
// kLineCut per thread, whose halo is nsteps wide: 64 steps recompute an eighth of
// the nodes.
constexpr int kLineNodes = 1024, kLineCut = 4;
constexpr int line_steps(int n0) { return n0 <= kLineNodes ? 1024 : 64; }
hipError_t launch_line(const MarchParams& p, int scheme, int mode, int nsteps, const MarchBufs& b,
                       long long n, hipStream_t stream);
hipError_t launch_wall_data1(const KParams& p, double* wx, long long n, int nsteps,
                             hipStream_t stream);
// d = 2: doubles of wall data per step (x_1 faces, then x_2 faces), and the wall data of
// steps n .. n + nsteps - 1 into wx / wy in the layout of MarchParams.
long long wall_data2_x(const KParams& p);
long long wall_data2_y(const KParams& p);
hipError_t launch_wall_data2(const KParams& p, double* wx, double* wy, long long n, int nsteps,
                             hipStream_t stream);

// One block of a batched reduction or initialisation: block `block` of the
// kRedBlocks that cover instance inst.
struct BatchBlock {
  int inst;
  int block;
};

// One block of a batched launch: rows row0 .. row0 + blockDim.y - 1 of an
// instance.
struct BatchTile {
  int inst;
  int row0;
};

// Tile of a batched marching pass (d = 2): instance, first x_1 node, output
// rows y0 .. y1 - 1.
struct BatchTile2 {
  int inst;
  int x0, y0, y1;
};

struct LaunchShape {
  int tx, ty;
  unsigned blocks;
};

LaunchShape step_shape(const KParams& p);

// One time step t_n -> t_{n+1}.  Non-split modes read/write post-collision
// populations; split mode reads/writes (phi, g) pre-collision.
// ev (nullable): three events recorded before the bulk kernel, between the
// bulk and the wall kernel, and after the wall kernel.
hipError_t launch_step(const KParams& p, int mode, const void* src, void* dst,
                       const double* phi_src, double* phi_dst, long long n,
                       hipStream_t stream, hipEvent_t* ev = nullptr);

// Buffers of a two-step pass: A holds the state at t_n, B receives t_{n+2},
// C is a scratch state of the same layout for the rows on and next to the
// walls of x_2 / x_3.  Split mode adds the phi planes and a second x_1-face
// array (the step-2 data; p.xdata holds step 1's).
struct FusedBufs {
  const void* A;
  void* B;
  void* C;
  const double* phiA;
  double* phiB;
  double* phiC;
  double* xdata2;
};

// The x_1-face data of up to three steps, one launch of k_xface (blockIdx.y = step):
// step i's go to the row slots of buf[i] or (split layout) to xdata[i], for the step
// that starts at t[i].
struct XfaceSteps {
  int count = 1;
  void* buf[3] = {};
  double* xdata[3] = {};
  double t[3] = {};
};

// Two steps t_n -> t_{n+2} of a lattice with d = 3 (any mode) in one pass of
// the bulk kernel (k_fused2, k_fused2_split).  Bitwise equal to two
// launch_step calls.  ev (nullable): three events around the fused kernel and
// after the step-2 wall kernel.
hipError_t launch_fused_pair(const KParams& p, int mode, const FusedBufs& fb, long long n,
                             hipStream_t stream, hipEvent_t* ev = nullptr);

// Buffers of a three-step pass: A at t_n, B at t_{n+3}, and with wall rows the
// scratch states C1 and C2 for the rows on and next to the walls of x_2 / x_3 after
// one and two steps (C1 also holds the second step's x_1-face data).
struct TriBufs {
  const void* A;
  void* B;
  void* C1;
  void* C2;
};
// Three steps of a d = 3 lattice in one pass (tri.hpp); bitwise three
// launch_step calls.  tri_applies: whether the pass takes the lattice and pays on it (a
// plane of x_3 under 4 GiB; x_1 walls only together with wall rows, whose scratch state
// holds their data); tri_last: whether also for the last three or five steps of a call.
bool tri_applies(const KParams& p, int mode);
bool tri_last(const KParams& p, int mode);
hipError_t launch_tri(const KParams& p, int mode, const TriBufs& tb, long long n,
                      hipStream_t stream, hipEvent_t* ev = nullptr);

// Initial state from the analytic field (phi0 == nullptr) or from device
// arrays (grad0 == nullptr: fourth-order central differences).
hipError_t launch_init(const KParams& p, int mode, void* dst, double* phi_dst,
                       const double* phi0, const double* grad0, hipStream_t stream);

// Moments of the state at step n selected by `what` (MomentBits); with any
// scalar bit, writes kRedBlocks x kNumAcc partials, then the final kNumAcc
// values into out.
hipError_t launch_moments(const KParams& p, int mode, const void* f, const double* phi,
                          long long n, double* phi_out, double* partial, double* out,
                          unsigned what, hipStream_t stream);

// Count the non-finite values among n float64 (dbl) or float32 values at
// `vals` into *count (added); zero_count sets *count = 0 with a kernel (no
// memset node in a captured graph).
hipError_t launch_count_nonfinite(const void* vals, bool dbl, long long n, unsigned* count,
                                  hipStream_t stream);
hipError_t launch_zero_count(unsigned* count, hipStream_t stream);

// Sum over the nodes of phi0 (analytic when arr == nullptr), into out[0].
hipError_t launch_sum_phi0(const KParams& p, const double* arr, double* partial,
                           double* out, hipStream_t stream);

// Whole-batch forms of launch_moments (scalars only), launch_sum_phi0 and
// launch_init: nblocks BatchBlocks, instance i's at first[i] .. first[i + 1); its
// kNumAcc results go to out[i * kNumAcc ..].  offset[i]: instance i's first
// element of the concatenated phi0 (d offset[i] of the gradients).
hipError_t launch_batch_moments(int d, const KParams* kps, void* const* bufs,
                                const BatchBlock* blocks, int nblocks, const int* first,
                                int count, int mode, int cur, long long n, double* partial,
                                double* out, unsigned what, hipStream_t stream);
hipError_t launch_batch_sum_phi0(int d, const KParams* kps, const BatchBlock* blocks, int nblocks,
                                 const int* first, int count, const long long* offset,
                                 const double* phi0, double* partial, double* out,
                                 hipStream_t stream);
// launch_batch_init leaves out float64 instances of more than kBatchInitNodes nodes (one per
// thread of their blocks), which a launch of their own initialises faster: two of 2048^2 231
// against 379 us, three of 100^3 183 against 290 (float32: 221 against 199, 191 and 152).
constexpr int kBatchInitNodes = kRedBlocks * 256;
hipError_t launch_batch_init(int d, const KParams* kps, void* const* bufs,
                             const BatchBlock* blocks, int nblocks, const long long* offset,
                             int mode, const double* phi0, const double* grad0,
                             hipStream_t stream);

// nsteps steps of every instance of a batch (periodic lattices of one d and
// precision), one launch per step over the tile table.
hipError_t launch_batch(int d, const KParams* kps, void* const* bufs, const BatchTile* tiles,
                        int ntiles, int tx, int ty, int mode, int cur, int nsteps,
                        hipStream_t stream);

// One marching pass of nl (2, 4 or 8) steps of every instance of a d = 2 batch
// (float32 or float64) over the BatchTile2 table, whose tiles are kBatchTileWidth
// wide (march_width(2) for two steps).
constexpr int kBatchTileWidth = march_width(kMarchMaxSteps);
hipError_t launch_batch_march(const MarchParams* mps, void* const* bufs, const BatchTile2* tiles,
                              int ntiles, int mode, int nl, int cur, hipStream_t stream);

// nsteps (even) steps of every instance of a d = 2 batch in one launch: block b
// advances instance order[b] (largest first) through all the passes, its
// wavefronts sharing the instance's tiles tiles[first[i] .. first[i + 1]); the
// instances never share a block, so no block waits for another.
hipError_t launch_batch_resident(const MarchParams* mps, void* const* bufs,
                                 const BatchTile2* tiles, const int* first, const int* order,
                                 int count, int mode, int cur, int nsteps, hipStream_t stream);
// Parity of the number of passes of nsteps (even) steps: as many of 8 as fit,
// then one of 4 and one of 2.
inline int march_pass_parity(long long nsteps) {
  return static_cast<int>((nsteps / 8 + nsteps % 8 / 4 + nsteps % 4 / 2) & 1);
}

// Adjoint step lambda^{n+1} -> lambda^n (adjoint.hip).  g: forward state at
// step n (nullable); when given, per-block partial sums of
// <nu^n, (omega 1^T - I) f^n> (without the 1/(1-s) factor of the
// post-collision modes) go to partial[0 .. step_shape(p).blocks).
hipError_t launch_adjoint_step(const KParams& p, int mode, const void* lsrc, void* ldst,
                               const void* g, const double* gphi, double* partial,
                               hipStream_t stream);
// Two adjoint steps lambda^{n+1} -> lambda^{n-1} in one pass (d = 3; the
// layout of the forward two-step pass).  g1, g2: forward states at steps n and
// n - 1 (both nullable); their contractions are added to
// partial[0 .. adjoint_pair_blocks(p, mode)).
hipError_t launch_adjoint_pair(const KParams& p, int mode, const void* lsrc, void* ldst,
                               const void* g1, const void* g2, double* partial,
                               hipStream_t stream);
long long adjoint_pair_blocks(const KParams& p, int mode);
hipError_t launch_adjoint_seed(const KParams& p, int mode, const double* dldphi, void* lam,
                               hipStream_t stream);
// Transpose of the initialisation; partial[0 .. *nblocks) receives the
// contraction of lambda^0 with d f^0 / d tau.
hipError_t launch_adjoint_init(const KParams& p, int mode, const void* lam, const void* g0,
                               const double* g0phi, double* dphi, double* dgrad, bool fd,
                               double* partial, unsigned* nblocks, hipStream_t stream);
hipError_t launch_sum_partials(const double* partial, long long n, double* out,
                               hipStream_t stream);
// Wall-data sensitivities of the adjoint step that consumes lambda^{n+1}
// (lam): adds its contractions with dW/da_j and dW/dtheta_j of the analytic
// field to partial[0 .. wall_grad_partials()); launch_sum_wall_grad reduces
// them to out[0 .. 2 kMaxModes) (d/da_j at j, d/dtheta_j at kMaxModes + j).
long long wall_grad_partials();
hipError_t launch_wall_grad(const KParams& p, int mode, const void* lam, long long n,
                            double* partial, hipStream_t stream);
hipError_t launch_sum_wall_grad(const double* partial, double* out, hipStream_t stream);

// Spectral radius of the amplification matrix over the wave-number grid
// xi = 2 pi j / m, j in [0, m)^d (nxi = m^d points), for count parameter
// points (sigma[pt*d .. pt*d+d), s[pt]); one block per point
// (stability.hip).  min_omega and unconverged are nullable.
hipError_t launch_stability(int d, long long count, const double* sigma, const double* s,
                            double g, int m, long long nxi, double* rho, double* min_omega,
                            int32_t* unconverged, hipStream_t stream);

}  // namespace lbm
