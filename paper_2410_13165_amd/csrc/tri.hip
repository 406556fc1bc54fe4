// Launches of the three-step passes of d = 3 (tri.hpp).
#include "tri.hpp"

#include <mutex>

namespace lbm {

// wall-row and x_1-face launches (walls.hpp, instantiated in walls_d*.hip)
template <int D, class T, bool TAN>
void launch_xface(hipStream_t stream, const XfaceSteps& xs, const KParams& p, int mode);
template <int D, class T, bool TAN>
void launch_wall(dim3 g, dim3 b, hipStream_t stream, const T* src, T* dst, const KParams& p,
                 double t);

// One step of the rows next to a Dirichlet wall of x_2 or x_3 (k_step's rows): the
// two-step values of the wall rows are formed from them before the pass.  Rows
// near walls of both axes are taken with x_2's.
template <class T>
__global__ void __launch_bounds__(256)
    k_step_near(const T* __restrict__ src, T* __restrict__ dst, const KParams p) {
  int i = blockIdx.x * blockDim.y + threadIdx.y;
  const int n1 = p.n[1], n2 = p.n[2];
  const int c1 = p.bc[1] != 0 ? 2 * n2 : 0, c2 = p.bc[2] != 0 ? 2 * n1 : 0;
  int iy, iz;
  if (i < c1) {
    const int side = i >= n2;
    iz = i - side * n2;
    iy = side ? n1 - 2 : 1;
    if (n1 < 3 || (side && n1 == 3)) return;
  } else {
    i -= c1;
    if (i >= c2) return;
    const int side = i >= n1;
    iy = i - side * n1;
    iz = side ? n2 - 2 : 1;
    if (n2 < 3 || (side && n2 == 3)) return;
    if (p.bc[1] != 0 && (iy == 1 || iy == n1 - 2)) return;
  }
  step_row<3, T>(src, dst, p, iz * n1 + iy);
}

// x_3 planes per block, as fuse_zchunk chooses them: a block of zc planes takes
// zc + 4 iterations, one block per CU at a time.
static int tri_zchunk(int tiles_xy, int n2) {
  const long long cus = device_cus();
  int best = 64;
  long long best_cost = -1;
  for (int zc = 128; zc >= 4; --zc) {
    const long long blocks = static_cast<long long>(tiles_xy) * ((n2 + zc - 1) / zc);
    const long long cost = (blocks + cus - 1) / cus * ((zc < n2 ? zc : n2) + 4);
    if (best_cost < 0 || cost < best_cost) {
      best_cost = cost;
      best = zc;
    }
  }
  return best;
}

template <class T, bool TAN, bool HALF>
static hipError_t tri_t(const KParams& p, const TriBufs& tb, long long n, hipStream_t stream,
                        hipEvent_t* ev) {
  using S = TriShape<T, HALF>;
  constexpr size_t lds =
      sizeof(T) * (16 * (S::TX + 4) * (2 * S::TY + 6) + 2 * 2 * 3 * 5 * (S::TY + 4));
  static_assert(lds <= 160 * 1024, "tile exceeds the LDS of a CU");
  constexpr int mode = std::is_same<T, float>::value ? kFP32 : kFP64;
  static std::once_flag once;
  static hipError_t attr = hipSuccess;
  std::call_once(once, [] {
    attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_tri<T, HALF>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
  });
  if (attr != hipSuccess) return attr;
  auto* A = static_cast<T*>(const_cast<void*>(tb.A));
  auto* B = static_cast<T*>(tb.B);
  auto* C1 = static_cast<T*>(tb.C1);
  auto* C2 = static_cast<T*>(tb.C2);
  const LaunchShape s = step_shape(p);
  const dim3 block(s.tx, s.ty);
  const dim3 wgrid(static_cast<unsigned>((p.wall_rows + s.ty - 1) / s.ty));
  auto t = [&](int i) { return static_cast<double>(n + i) * p.dt; };
  if (p.bc[0] != 0)
    launch_xface<3, T, TAN>(stream, XfaceSteps{3, {A, C1, B}, {}, {t(0), t(1), t(2)}}, p, mode);
  if (p.wall_rows > 0) {
    launch_wall<3, T, TAN>(wgrid, block, stream, A, C1, p, t(0));
    const int near = (p.bc[1] != 0 ? 2 * p.n[2] : 0) + (p.bc[2] != 0 ? 2 * p.n[1] : 0);
    hipLaunchKernelGGL((k_step_near<T>), dim3((near + s.ty - 1) / s.ty), block, 0, stream, A, C1,
                       p);
    launch_wall<3, T, TAN>(wgrid, block, stream, C1, C2, p, t(1));
  }
  const int tiles_xy = ((p.n[0] + S::TX - 1) / S::TX) * ((p.n[1] + S::TY - 1) / S::TY);
  const int zc = tri_zchunk(tiles_xy, p.n[2]);
  const dim3 grid(static_cast<unsigned>(tiles_xy * ((p.n[2] + zc - 1) / zc)));
  if (ev) (void)hipEventRecord(ev[0], stream);
  hipLaunchKernelGGL((k_tri<T, HALF>), grid, dim3(S::NT), lds, stream, A, B, C1, C2, p, zc);
  if (ev) (void)hipEventRecord(ev[1], stream);
  if (p.wall_rows > 0) launch_wall<3, T, TAN>(wgrid, block, stream, C2, B, p, t(2));
  if (ev) (void)hipEventRecord(ev[2], stream);
  return hipGetLastError();
}

template <class T>
static hipError_t tri_m(const KParams& p, const TriBufs& tb, long long n, hipStream_t stream,
                        hipEvent_t* ev) {
  const bool half = p.scheme == kHalfWay;
  if (p.wall_data)
    return half ? tri_t<T, true, true>(p, tb, n, stream, ev)
                : tri_t<T, true, false>(p, tb, n, stream, ev);
  return half ? tri_t<T, false, true>(p, tb, n, stream, ev)
              : tri_t<T, false, false>(p, tb, n, stream, ev);
}

// Periodic lattices gain at every size (24^3: 11.7 against 12.7 us per step in
// float32, 160^3: 72 against 92).  With wall rows the pass has six launches for
// three steps against four for two, and small lattices are bound by those: 64^3
// full-way 27.9 against 27.4 us, 112^3 45.8 against 45.6 (float64 71.9 against 79.2);
// with the x_1-face data in a launch per step, 128^3 61.6 against 65.2 (109 against 126).
//
// The split mode keeps its two-step pass: in this layout (32 x 14 columns, rings of
// three planes of t in LDS) three steps of 512^3 took 9.2 ms full-way and 8.4 ms periodic,
// against 5.95 ms for two.
bool tri_applies(const KParams& p, int mode) {
  if (p.d != 3 || (mode != kFP64 && mode != kFP32)) return false;
  if (p.wall_rows > 0 && p.nodes < 1400000) return false;
  const long long plane = static_cast<long long>(p.n[0]) * p.n[1];
  if (plane * 8 >= (1LL << 32)) return false;
  return p.bc[0] == 0 || p.wall_rows > 0;
}

hipError_t launch_tri(const KParams& p, int mode, const TriBufs& tb, long long n,
                      hipStream_t stream, hipEvent_t* ev) {
  if (!tri_applies(p, mode)) return hipErrorInvalidValue;
  if (p.wall_rows > 0 && (!tb.C1 || !tb.C2)) return hipErrorInvalidValue;
  return mode == kFP64 ? tri_m<double>(p, tb, n, stream, ev) : tri_m<float>(p, tb, n, stream, ev);
}

}  // namespace lbm
