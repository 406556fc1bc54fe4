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

template <class S>
static int tiles_of(const KParams& p) {
  return ((p.n[0] + S::TX - 1) / S::TX) * ((p.n[1] + S::TY - 1) / S::TY);
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
  const int tiles_xy = tiles_of<S>(p);
  const int zc = pass_zchunk(tiles_xy, p.n[2], 128, 4).zc;
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

// Three steps in one pass or 3/2 passes of two, by the iterations that either takes
// (pass_zchunk) and what one of three steps takes of one of two (`weight`, hundredths,
// fitted to the passes of 200 lattices): float64 0.80, float32 0.87, its half-way
// tiles, which are smaller, 0.65, and 0.84 below 3 million nodes without x_1 walls,
// where the wall launches weigh more.  So lattices that fill their tiles or the last
// round of blocks worse go on in pairs: us for two and three steps, 300 x 300 x 8
// periodic float64 66 and 119, 130 x 120 x 110 with half-way x_2 walls float32 125 and
// 205; 160^3 full-way 205 and 277.
//
// Thin lattices go in pairs too: the pass recomputes four planes, keeps the rows next to
// walls, and has three wall launches (1000 x 700 x 16 full-way float64 1115 and 1691,
// x 24 1701 and 2302), as do lattices with wall rows below 1.4 million nodes, which are
// bound by its launches (64^3 full-way 27.9 us per step in threes, 27.4 in pairs; 112^3
// 45.8 and 45.6).
//
// The split mode keeps its two-step pass: in this layout (32 x 14 columns, rings of
// three planes of t in LDS) three steps of 512^3 took 9.2 ms full-way and 8.4 ms periodic,
// against 5.95 ms for two.
template <class T, bool HALF>
static bool tri_pays(const KParams& p, int weight) {
  const long long three = pass_zchunk(tiles_of<TriShape<T, HALF>>(p), p.n[2], 128, 4).cost;
  const long long two = pass_zchunk(tiles_of<FuseFwdShape<T, HALF>>(p), p.n[2], 64, 2).cost;
  return 2 * weight * three < 300 * two;
}

bool tri_applies(const KParams& p, int mode) {
  if (p.d != 3 || (mode != kFP64 && mode != kFP32)) return false;
  const long long plane = static_cast<long long>(p.n[0]) * p.n[1];
  if (plane * 8 >= (1LL << 32)) return false;
  if (p.bc[0] != 0 && p.wall_rows == 0) return false;
  const bool dbl = mode == kFP64, half = p.scheme == kHalfWay;
  if (p.wall_rows > 0) {
    if (p.nodes < 1400000 || p.n[2] < 8) return false;
    if (static_cast<long long>(p.wall_rows) * (dbl ? 8 : 5) > p.rows) return false;
  } else if (p.n[2] < (dbl ? (p.nodes < 100000 ? 16 : 4) : 3)) {
    return false;
  }
  if (dbl) return half ? tri_pays<double, true>(p, 80) : tri_pays<double, false>(p, 80);
  if (!half) return tri_pays<float, false>(p, 87);
  return tri_pays<float, true>(p, p.bc[0] == 0 && p.nodes < 3000000 ? 84 : 65);
}

// A pass of three steps for the last three or five of a call: on small lattices two steps
// and one are faster (48^3 float32 32 against 36 us, 64^3 39 and 37; 40^3 float64 32 and
// 33, 16 x 16 x 300, whose single step takes a wavefront per row, 35 and 30).
bool tri_last(const KParams& p, int mode) {
  if (mode != kFP64) return p.nodes >= 200000;
  return static_cast<long long>(p.rows) * ((p.n[0] + 63) / 64 * 64) >= 120000;
}

hipError_t launch_tri(const KParams& p, int mode, const TriBufs& tb, long long n,
                      hipStream_t stream, hipEvent_t* ev) {
  if (p.d != 3 || (mode != kFP64 && mode != kFP32)) return hipErrorInvalidValue;
  if (p.wall_rows > 0 && (!tb.C1 || !tb.C2)) return hipErrorInvalidValue;
  return mode == kFP64 ? tri_m<double>(p, tb, n, stream, ev) : tri_m<float>(p, tb, n, stream, ev);
}

}  // namespace lbm
