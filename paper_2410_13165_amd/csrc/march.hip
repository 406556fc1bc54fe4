// Launches of the d = 2 marching passes (march.hpp) and of their wall data.
#include <algorithm>

#include "march.hpp"

namespace lbm {

// One tile per wavefront; kMarchWaves of them share a block, tiles next to each
// other in x_1, whose halos read the same lines.  Walls take two per block, to
// keep its wall data within 64 KB of LDS.
template <int WALL>
constexpr int kMarchWaves = WALL ? 2 : 4;

template <int MODE, int NL, int WALL, int D>
__global__ void __launch_bounds__(64 * kMarchWaves<WALL>)
    k_march2(const MarchParams p, const MarchBufs b, const int yc, const int gx, const int ntiles,
             const long long n) {
  extern __shared__ __align__(16) unsigned char march_mem[];
  const int wave = static_cast<int>(threadIdx.x) / 64;
  const int w = static_cast<int>(blockIdx.x) * kMarchWaves<WALL> + wave;
  if (w >= ntiles) return;
  constexpr int W = march_width(NL);
  const int y0 = (w / gx) * yc;
  march2_tile<MODE, NL, WALL, D>(
      p, b, (w % gx) * W, W, y0, min(y0 + yc, p.n1), n,
      reinterpret_cast<double*>(march_mem + (WALL ? wave * march_lds(NL, yc) : 0)));
}

// Tiles next to each other go to one XCD in turn (as fuse_tile orders them), so that
// the rows they share are read through one L2.
template <class T>
__global__ void __launch_bounds__(kPairWidth)
    k_pair2(const MarchParams p, const T* __restrict__ src, T* __restrict__ dst, const int yc,
            const int gx) {
  __shared__ T lds[kPairSlots * (kPairWidth + 2)];
  const int nb = static_cast<int>(gridDim.x), per = nb / 8, b = static_cast<int>(blockIdx.x);
  const int t = b < 8 * per ? (b % 8) * per + b / 8 : b;
  const int y0 = t / gx * yc;
  pair2_tile<T>(p, src, dst, lds, t % gx * kPairWidth, y0, min(y0 + yc, p.n1));
}

template <class T>
static hipError_t pair2_t(const MarchParams& p, const MarchBufs& b, int yc, hipStream_t stream) {
  const int gx = (p.n0 + kPairWidth - 1) / kPairWidth;
  const dim3 grid(static_cast<unsigned>(gx * ((p.n1 + yc - 1) / yc)));
  hipLaunchKernelGGL((k_pair2<T>), grid, dim3(kPairWidth), 0, stream, p,
                     static_cast<const T*>(b.src), static_cast<T*>(b.dst), yc, gx);
  return hipGetLastError();
}

MarchParams march_params(const KParams& p) {
  MarchParams m{};
  m.n0 = p.n[0];
  m.n1 = p.n[1];
  m.bc0 = p.bc[0];
  m.bc1 = p.bc[1];
  m.ps = p.pstride;
  for (int k = 0; k < 9; ++k) {  // d = 1 uses the first three
    m.omega[k] = p.omega[k];
    m.omega_f[k] = p.omega_f[k];
  }
  m.s_f = p.s_f;
  m.s = p.s;
  m.dt = p.dt;
  m.R = p.R;
  m.dtR = p.dtR;
  m.phi_ref = p.phi_ref;
  return m;
}

template <int MODE, int NL, int WALL, int D>
static hipError_t march2_l(const MarchParams& p, const MarchBufs& b, long long n, int yc,
                           hipStream_t stream) {
  constexpr int W = march_width(NL), NW = kMarchWaves<WALL>;
  const int gx = (p.n0 + W - 1) / W;
  const int ntiles = gx * ((p.n1 + yc - 1) / yc);
  const size_t lds = WALL ? NW * march_lds(NL, yc) : 0;
  hipLaunchKernelGGL((k_march2<MODE, NL, WALL, D>), dim3((ntiles + NW - 1) / NW), dim3(64 * NW),
                     lds, stream, p, b, yc, gx, ntiles, n);
  return hipGetLastError();
}

// Source rows in flight: two hide more of the load latency than one (512^2,
// 8 steps per pass, float64: 22 against 25 us); four cost registers (and are
// slower on large lattices).  With walls one, beside the wall data.
template <int MODE, int NL>
static hipError_t march2_w(const MarchParams& p, int scheme, const MarchBufs& b, long long n,
                           int yc, hipStream_t stream) {
  if (scheme == kNoWall) return march2_l<MODE, NL, 0, 2>(p, b, n, yc, stream);
  if constexpr (NL <= kMarchMaxWallSteps)
    return scheme == kFullWay ? march2_l<MODE, NL, kFullWay, 1>(p, b, n, yc, stream)
                              : march2_l<MODE, NL, kHalfWay, 1>(p, b, n, yc, stream);
  return hipErrorInvalidValue;
}

// Steps and rows per tile of passes of at most 1, 2, 4 and 8 steps, by a model of its
// time fitted to measured passes (64^2 to 2048^2, us): 4 for the launch, then
// the largest of
//   * one tile alone: c per row and stage (its instructions at one wavefront per
//     SIMD: 0.115 in float64, 0.172 in float32 with its compensated sum, 0.177
//     split) and 0.35 per source row (its load);
//   * a SIMD's tiles one after another: c per row and stage of each;
//   * the traffic at 5.2 TB/s, halo columns and rows read again.
// The minimum is over time per step.  Large lattices are bound by the third (2048^2
// float64: 8 steps, 106 rows, 157 us) or, in float32, nearly as much by the second (4
// steps, 46 rows, 89 us), small ones by the first and the launch (64^2 float64: 8 steps of
// one row per tile, 16 us).  The second term charges every tile a lone wavefront's time,
// which several on one SIMD hide in part: 8 steps of 44 rows, which it rules out for
// float32, take 140 us at 2048^2 against the 178 of twice 4.
// 16 wall rows and columns per wavefront are more registers and instructions:
// passes over walls stop at 4 steps and 32 rows.  Two-step passes that the third binds
// stop at 8 rows: the traffic of their halo rows, which the model charges to memory,
// stays in the caches, and more tiles hide more of the loads (8 rows against the 32 to
// 128 that the model would take: 4096^2 with full-way walls float32 316 and 428 us, 1024^2
// periodic float64 47 and 66; 3 x 100000, bound by the second, 48 and 44).
void march_plans(const KParams& p, int mode, MarchPlan (&plans)[4]) {
  const bool walls = p.scheme != kNoWall;
  const double c = mode == kFP64 ? 0.115 : mode == kFP32 ? 0.172 : 0.177;
  const double node_bytes = mode == kFP64 ? 72.0 : mode == kFP32 ? 36.0 : 44.0;
  const int simds = 4 * device_cus();
  MarchPlan best{1, 0, false};
  double best_t = 0.0;
  plans[0] = best;
  for (int i = 1; i < 4; ++i, plans[i - 1] = best) {
    const int nl = 1 << i;
    if (nl > (walls ? kMarchMaxWallSteps : kMarchMaxSteps)) continue;
    const int w = march_width(nl);
    const long long gx = (p.n[0] + w - 1) / w;
    for (int yc = 1; yc <= (walls ? 32 : 128); ++yc) {
      const long long tiles = gx * ((p.n[1] + yc - 1) / yc);
      if (tiles > (1LL << 28)) continue;
      const double rows = nl * yc + nl * (nl - 1);
      const double alone = rows * c + (yc + 2 * nl) * 0.35;
      const double issue = static_cast<double>((tiles + simds - 1) / simds) * rows * c;
      const double bytes = p.nodes * node_bytes * ((1.0 + 2.0 * nl / yc) * 64.0 / w + 1.0);
      const double work = std::max(alone, issue), traffic = bytes / 5.2e6;
      const double t = (4.0 + std::max(work, traffic)) / nl;
      if (best.nl == 1 || t < best_t) {
        best_t = t;
        best = MarchPlan{nl, yc, false};
        if (nl == 2 && traffic > work) best.yc = std::min(yc, 8);
      }
      if (yc >= p.n[1]) break;
    }
  }
  // Two steps of a large periodic lattice whose blocks of columns are at least four
  // fifths full: us of one call, in blocks and in wavefront tiles, 1000^2 float64 35 and
  // 41, 700^2 31 and 24; float32 2048^2 67 and 85, 1280^2 36 and 32; 300 x 14000 float64
  // 161 and 147.  The rows per block: 64, halved (down to 8) while the grid has fewer
  // than four blocks per CU.
  const long long gx = (p.n[0] + kPairWidth - 1) / kPairWidth;
  const long long full = mode == kFP64 ? 900000 : 1900000;
  if (!walls && mode != kSplit && p.nodes >= full && 5LL * p.n[0] >= 4 * gx * kPairWidth) {
    int yc = 64;
    while (yc > 8 && gx * ((p.n[1] + yc - 1) / yc) < 4 * device_cus()) yc /= 2;
    plans[1] = MarchPlan{2, yc, true};
  }
}

template <int MODE>
static hipError_t march2_m(const MarchParams& p, int scheme, int nl, const MarchBufs& b,
                           long long n, int yc, hipStream_t stream) {
  switch (nl) {
    case 2: return march2_w<MODE, 2>(p, scheme, b, n, yc, stream);
    case 4: return march2_w<MODE, 4>(p, scheme, b, n, yc, stream);
    case 8: return march2_w<MODE, 8>(p, scheme, b, n, yc, stream);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_march2(const MarchParams& p, int scheme, int mode, const MarchPlan& plan,
                         const MarchBufs& b, long long n, hipStream_t stream) {
  if (plan.yc < 1) return hipErrorInvalidValue;
  if (plan.block) {
    if (scheme != kNoWall || plan.nl != 2) return hipErrorInvalidValue;
    if (mode == kFP64) return pair2_t<double>(p, b, plan.yc, stream);
    if (mode == kFP32) return pair2_t<float>(p, b, plan.yc, stream);
    return hipErrorInvalidValue;
  }
  switch (mode) {
    case kFP64: return march2_m<kFP64>(p, scheme, plan.nl, b, n, plan.yc, stream);
    case kFP32: return march2_m<kFP32>(p, scheme, plan.nl, b, n, plan.yc, stream);
    case kSplit: return march2_m<kSplit>(p, scheme, plan.nl, b, n, plan.yc, stream);
    default: return hipErrorInvalidValue;
  }
}

// ---- batches of periodic lattices: one tile of the table per wavefront
template <int MODE, int NL>
__global__ void __launch_bounds__(256)
    k_march2_batch(const MarchParams* __restrict__ mps, void* const* __restrict__ bufs,
                   const BatchTile2* __restrict__ tiles, const int ntiles, const int cur) {
  const int w = static_cast<int>(blockIdx.x) * 4 + static_cast<int>(threadIdx.x) / 64;
  if (w >= ntiles) return;
  const BatchTile2 t = tiles[__builtin_amdgcn_readfirstlane(w)];
  const MarchBufs b{bufs[2 * t.inst + cur], bufs[2 * t.inst + 1 - cur], nullptr, nullptr};
  constexpr int W = NL == 2 ? march_width(2) : kBatchTileWidth;
  march2_tile<MODE, NL, 0, 2>(mps[t.inst], b, t.x0, W, t.y0, t.y1, 0, nullptr);
}

template <int MODE>
static hipError_t batch_march_m(const MarchParams* mps, void* const* bufs,
                                const BatchTile2* tiles, int ntiles, int nl, int cur,
                                hipStream_t stream) {
  const dim3 g((ntiles + 3) / 4), b(256);
  switch (nl) {
    case 2: hipLaunchKernelGGL((k_march2_batch<MODE, 2>), g, b, 0, stream, mps, bufs, tiles, ntiles, cur); break;
    case 4: hipLaunchKernelGGL((k_march2_batch<MODE, 4>), g, b, 0, stream, mps, bufs, tiles, ntiles, cur); break;
    case 8: hipLaunchKernelGGL((k_march2_batch<MODE, 8>), g, b, 0, stream, mps, bufs, tiles, ntiles, cur); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_batch_march(const MarchParams* mps, void* const* bufs, const BatchTile2* tiles,
                              int ntiles, int mode, int nl, int cur, hipStream_t stream) {
  if (mode == kFP64) return batch_march_m<kFP64>(mps, bufs, tiles, ntiles, nl, cur, stream);
  if (mode == kFP32) return batch_march_m<kFP32>(mps, bufs, tiles, ntiles, nl, cur, stream);
  return hipErrorInvalidValue;
}

// Every pass of a call for one instance per block: its wavefronts take the
// instance's tiles in turn, and the block's barrier ends each pass (the state
// never leaves the block, so no block waits for another).  Bitwise the result of
// the launches per pass: the same tile body on the same tiles.
template <int MODE>
__global__ void __launch_bounds__(256)
    k_march2_resident(const MarchParams* __restrict__ mps, void* const* __restrict__ bufs,
                      const BatchTile2* __restrict__ tiles, const int* __restrict__ first,
                      const int* __restrict__ order, const int nsteps, const int cur) {
  const int inst = order[blockIdx.x];
  const int t0 = first[inst], t1 = first[inst + 1];
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / 64);
  int c = cur;
  auto pass = [&](auto Nl) {
    constexpr int NL = decltype(Nl)::value;
    const MarchBufs b{bufs[2 * inst + c], bufs[2 * inst + 1 - c], nullptr, nullptr};
    for (int i = t0 + wave; i < t1; i += 4) {
      const BatchTile2 t = tiles[i];
      march2_tile<MODE, NL, 0, 2>(mps[inst], b, t.x0, kBatchTileWidth, t.y0, t.y1, 0, nullptr);
    }
    // this pass's output is read by the next: the block's global stores must
    // be visible to all of its threads
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __syncthreads();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    c = 1 - c;
  };
  for (int s = 0; s < nsteps / 8; ++s) pass(std::integral_constant<int, 8>{});
  if (nsteps & 4) pass(std::integral_constant<int, 4>{});
  if (nsteps & 2) pass(std::integral_constant<int, 2>{});
}

hipError_t launch_batch_resident(const MarchParams* mps, void* const* bufs,
                                 const BatchTile2* tiles, const int* first, const int* order,
                                 int count, int mode, int cur, int nsteps, hipStream_t stream) {
  if (nsteps <= 0 || count <= 0) return hipSuccess;
  const dim3 g(static_cast<unsigned>(count)), b(256);
  if (mode == kFP64)
    hipLaunchKernelGGL((k_march2_resident<kFP64>), g, b, 0, stream, mps, bufs, tiles, first, order,
                       nsteps, cur);
  else if (mode == kFP32)
    hipLaunchKernelGGL((k_march2_resident<kFP32>), g, b, 0, stream, mps, bufs, tiles, first, order,
                       nsteps, cur);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

// ---- d = 1
template <int MODE, int WALL, int M>
__global__ void __launch_bounds__(M == 1 ? kLineNodes : kLineNodes / kLineCut)
    k_line(const MarchParams p, const MarchBufs b, const int nsteps, const long long n) {
  extern __shared__ __align__(16) unsigned char march_mem[];
  if constexpr (M == 1) {
    line_block<MODE, WALL, 1>(p, b, 0, p.n0, 0, p.n0, nsteps, n, march_mem);
  } else {
    const int out = kLineNodes - 2 * nsteps;
    const long long o0 = static_cast<long long>(blockIdx.x) * out;
    line_block<MODE, WALL, M>(p, b, static_cast<int>(o0) - nsteps, kLineNodes,
                              static_cast<int>(o0),
                              static_cast<int>(min(o0 + out, static_cast<long long>(p.n0))), nsteps,
                              n, march_mem);
  }
}

template <int MODE, int WALL, int M>
static hipError_t line_m(const MarchParams& p, const MarchBufs& b, int nsteps, long long n,
                         hipStream_t stream) {
  constexpr size_t as = MODE == kFP32 ? sizeof(float) : sizeof(double);
  const int nt = M == 1 ? (p.n0 + 63) / 64 * 64 : kLineNodes / kLineCut;
  const int out = kLineNodes - 2 * nsteps;
  const unsigned blocks = M == 1 ? 1 : static_cast<unsigned>((p.n0 + out - 1) / out);
  const size_t lds = (WALL ? sizeof(double) * 2 * nsteps : 0) + as * 4 * nt;
  hipLaunchKernelGGL((k_line<MODE, WALL, M>), dim3(blocks), dim3(nt), lds, stream, p, b, nsteps, n);
  return hipGetLastError();
}

template <int MODE>
static hipError_t line_w(const MarchParams& p, int scheme, const MarchBufs& b, int nsteps,
                         long long n, hipStream_t stream) {
  if (p.n0 <= kLineNodes) {
    if (scheme == kFullWay) return line_m<MODE, kFullWay, 1>(p, b, nsteps, n, stream);
    if (scheme == kHalfWay) return line_m<MODE, kHalfWay, 1>(p, b, nsteps, n, stream);
    return line_m<MODE, 0, 1>(p, b, nsteps, n, stream);
  }
  if (scheme == kFullWay) return line_m<MODE, kFullWay, kLineCut>(p, b, nsteps, n, stream);
  if (scheme == kHalfWay) return line_m<MODE, kHalfWay, kLineCut>(p, b, nsteps, n, stream);
  return line_m<MODE, 0, kLineCut>(p, b, nsteps, n, stream);
}

hipError_t launch_line(const MarchParams& p, int scheme, int mode, int nsteps, const MarchBufs& b,
                       long long n, hipStream_t stream) {
  if (nsteps < 1 || nsteps > line_steps(p.n0)) return hipErrorInvalidValue;
  switch (mode) {
    case kFP64: return line_w<kFP64>(p, scheme, b, nsteps, n, stream);
    case kFP32: return line_w<kFP32>(p, scheme, b, nsteps, n, stream);
    case kSplit: return line_w<kSplit>(p, scheme, b, nsteps, n, stream);
    default: return hipErrorInvalidValue;
  }
}

// one thread per (step, face): k_xface's values before their rounding
template <bool TAN>
__global__ void __launch_bounds__(256)
    k_wall_data1(double* __restrict__ wx, const KParams p, const long long n, const int nsteps) {
  const int idx = blockIdx.x * 256 + threadIdx.x;
  if (idx >= 2 * nsteps) return;
  const int side = idx & 1;
  const double t_n = step_time(n + (idx >> 1), p.dt);
  double x[kMaxDim] = {0.0, 0.0, 0.0, 0.0};
  x[0] = wall_coord<1>(p, 0, side ? p.n[0] - 1 : 0);
  const int want = side ? 2 : 1;
  double val[3];
  wall_analytic<1, TAN, -1>(p, x, t_n, [&](int k) { return k == want; }, [](int) { return 0; }, val);
  wx[idx] = side ? val[2] : val[1];
}

hipError_t launch_wall_data1(const KParams& p, double* wx, long long n, int nsteps,
                             hipStream_t stream) {
  const dim3 g(static_cast<unsigned>((2 * nsteps + 255) / 256)), b(256);
  if (p.wall_data)
    hipLaunchKernelGGL((k_wall_data1<true>), g, b, 0, stream, wx, p, n, nsteps);
  else
    hipLaunchKernelGGL((k_wall_data1<false>), g, b, 0, stream, wx, p, n, nsteps);
  return hipGetLastError();
}

// ---- wall data of several steps of d = 2: one thread per step and face node (of the step
// blockIdx.y where all of them are too many for one index); the
// values k_xface and k_wall compute, before their rounding to the storage type.
template <bool TAN, int V>
__global__ void __launch_bounds__(256)
    k_wall_data2(double* __restrict__ wx, double* __restrict__ wy, const KParams p,
                 const long long n, const int nsteps) {
  const unsigned fx = p.bc[0] != 0 ? 2u * p.n[1] : 0, fy = p.bc[1] != 0 ? 2u * p.n[0] : 0;
  unsigned idx = blockIdx.x * 256 + threadIdx.x;
  int l = blockIdx.y;
  if (gridDim.y == 1) {
    l = static_cast<int>(idx / (fx + fy));
    idx -= l * (fx + fy);
  }
  if (l >= nsteps || idx >= fx + fy) return;
  const double t_n = step_time(n + l, p.dt);
  const bool onx = idx < fx;
  const int e = onx ? idx : idx - fx;
  const int len = onx ? p.n[1] : p.n[0];
  const int side = e / len, pos = e - side * len;
  const int ax = onx ? 0 : 1;
  const int i0 = onx ? (side ? p.n[0] - 1 : 0) : pos;
  const int i1 = onx ? pos : (side ? p.n[1] - 1 : 0);
  double x[kMaxDim] = {0.0, 0.0, 0.0, 0.0};
  x[0] = wall_coord<2>(p, 0, i0);
  x[1] = wall_coord<2>(p, 1, i1);
  const int want = side ? -1 : 1;
  double val[q_of(2)];
  wall_analytic<2, TAN, V>(p, x, t_n, [&](int k) { return p.cv[k][ax] == want; },
                           [&](int) { return ax; }, val);
  double* out = (onx ? wx : wy) + static_cast<long long>((l * 2 + side) * 3) * len + pos;
  static_for<0, q_of(2)>([&](auto K) {
    constexpr int k = decltype(K)::value;
    constexpr int cx = vel_comp(2, k, 0), cy = vel_comp(2, k, 1);
    if (onx) {
      if (cx == want) out[static_cast<long long>(xface_slot(2, k)) * len] = val[k];
    } else {
      if (cy == want) out[static_cast<long long>(march_slot(k)) * len] = val[k];
    }
  });
}

long long wall_data2_x(const KParams& p) { return p.bc[0] != 0 ? 6LL * p.n[1] : 0; }
long long wall_data2_y(const KParams& p) { return p.bc[1] != 0 ? 6LL * p.n[0] : 0; }

template <bool TAN>
static void wall_data2_t(dim3 g, const KParams& p, double* wx, double* wy, long long n,
                         int nsteps, hipStream_t stream) {
  const dim3 b(256);
  switch (wall_variant(p)) {
    case 0: hipLaunchKernelGGL((k_wall_data2<TAN, 0>), g, b, 0, stream, wx, wy, p, n, nsteps); break;
    case 1: hipLaunchKernelGGL((k_wall_data2<TAN, 1>), g, b, 0, stream, wx, wy, p, n, nsteps); break;
    case 2: hipLaunchKernelGGL((k_wall_data2<TAN, 2>), g, b, 0, stream, wx, wy, p, n, nsteps); break;
    default: hipLaunchKernelGGL((k_wall_data2<TAN, 3>), g, b, 0, stream, wx, wy, p, n, nsteps);
  }
}

hipError_t launch_wall_data2(const KParams& p, double* wx, double* wy, long long n, int nsteps,
                             hipStream_t stream) {
  const long long per = (wall_data2_x(p) + wall_data2_y(p)) / 3;
  if (per <= 0 || nsteps <= 0) return hipSuccess;
  const bool flat = per * nsteps <= 1LL << 30;
  const dim3 grid(static_cast<unsigned>(((flat ? per * nsteps : per) + 255) / 256),
                  static_cast<unsigned>(flat ? 1 : nsteps));
  if (p.wall_data) wall_data2_t<true>(grid, p, wx, wy, n, nsteps, stream);
  else wall_data2_t<false>(grid, p, wx, wy, n, nsteps, stream);
  return hipGetLastError();
}

}  // namespace lbm
