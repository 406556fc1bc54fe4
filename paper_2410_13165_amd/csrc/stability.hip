// Batched von Neumann analysis of the periodic scheme (Sec. 4.2, eq. (G)):
// the spectral radius of the amplification matrix over a grid of wave
// numbers, for many parameter points (sigma = u, s) at once, and the
// smallest equilibrium weight (the entropy criterion of Sec. 4.1, Prop. 1).
//
// In population space the Fourier symbol of one step is
//     G(xi) = T(xi) [(1 - s) I + s omega 1^T],   T(xi) = diag(exp(-i c_k . xi)),
// which is similar to the moment-space matrix of eq. (G) (M is invertible;
// s = 2 gives eq. (G) itself).  G is a diagonal matrix plus a rank-one term,
// so its spectrum has a closed structure.  Let the velocities be grouped by
// equal tau_k = exp(-i c_k . xi) (groups g with tau_g, W_g = sum of their
// omega_k, n_g members).  Then
//   * every vector supported on one group with zero sum is an eigenvector
//     with eigenvalue (1 - s) tau_g (n_g - 1 of them per group), and
//   * the other eigenvalues are the roots of the secular equation
//         1 = s sum_g W_g tau_g / (lambda - (1 - s) tau_g)
//     (the matrix determinant lemma), i.e. of a polynomial of degree equal
//     to the number of groups with W_g != 0.
// On the grid xi = 2 pi j / m the phase c_k . xi is 2 pi (c_k . j) / m, so the
// grouping is exact integer arithmetic on (c_k . j) mod m.
//
// The roots come from the Aberth-Ehrlich simultaneous iteration (Aberth,
// Math. Comp. 27 (1973); Ehrlich, Comm. ACM 10 (1967)).  With a = 1 - s,
// v_g = s W_g tau_g and poles a tau_g, the polynomial is
//     p(lambda) = prod_g (lambda - a tau_g) - sum_g v_g prod_{g' != g} (lambda - a tau_g'),
// and its Newton ratio p / p' is evaluated in secular form with the pole h
// nearest to lambda factored out, which stays accurate when a root sits next
// to a pole (a weight near 0):
//     p / prod_{g != h} = e f_h - v_h,   e = lambda - a tau_h,
//     f_h = 1 - sum_{g != h} v_g / (lambda - a tau_g).
// All but one root sit near the poles a tau_g (exactly so for s -> 1, where
// they collapse to 0); the remaining one carries the conserved mode (1 at
// xi = 0) and starts from sum_g v_g + a mean(tau).
//
// One thread takes one wave number.  G(-xi) is the complex conjugate of G(xi), so
// only the wave numbers with j_d <= m / 2 are visited, those strictly inside
// standing for two.  A block is one wavefront; stab_split deals the wave numbers to
// blocks.
//
// The kernel is bound by float64 arithmetic: per sweep two complex reciprocals for
// each pair of groups.  No array that a run-time index walks is private: the roots
// lie in LDS, and the groups in registers or LDS (kStabListed), where the scratch
// traffic of private arrays bound the kernel before.  The divisions share a refined
// reciprocal (cinv).  Calls at s = 2, with private arrays and divisions, and now: 61^2
// points of D2Q9, m = 16, 5.9 and 1.4 ms; 9^2, m = 8, 366 and 206 us; 13^3 of D3Q19, m =
// 12, 56 and 22 ms; 300000 of D1Q3, m = 16, 10.3 and 0.67 ms; 1 point of D2Q9, m = 256,
// 130 and 0.24 ms (there for the split over blocks).
#include <hip/hip_runtime.h>

#include <cstdint>
#include <utility>

#include "engine.hpp"
#include "lattice.hpp"
#include "meta.hpp"

namespace lbm {
namespace {

struct cplx {
  double re, im;
};
__device__ __forceinline__ cplx cadd(cplx a, cplx b) { return {a.re + b.re, a.im + b.im}; }
__device__ __forceinline__ cplx csub(cplx a, cplx b) { return {a.re - b.re, a.im - b.im}; }
__device__ __forceinline__ cplx cmul(cplx a, cplx b) {
  return {a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re};
}
__device__ __forceinline__ cplx cscale(cplx a, double r) { return {a.re * r, a.im * r}; }
// 1 / a = conj(a) / |a|^2.  The two quotients share the reciprocal of |a|^2, the hardware's
// estimate after two Newton steps, and each is corrected by its remainder (Markstein, IBM
// J. Res. Dev. 34 (1990)), which rounds as a division does; div_fixup gives a division's
// results for zero, infinite and undefined |a|^2.
__device__ __forceinline__ cplx cinv(cplx a) {
  const double n = a.re * a.re + a.im * a.im;
  double r = __builtin_amdgcn_rcp(n);
  r = fma(r, fma(-n, r, 1.0), r);
  r = fma(r, fma(-n, r, 1.0), r);
  const auto quotient = [&](double x) {
    const double q = x * r;
    return __builtin_amdgcn_div_fixup(fma(fma(-n, q, x), r, q), n, x);
  };
  return {quotient(a.re), quotient(-a.im)};
}
__device__ __forceinline__ cplx cdiv(cplx a, cplx b) { return cmul(a, cinv(b)); }
__device__ __forceinline__ double cabs2(cplx a) { return a.re * a.re + a.im * a.im; }
__device__ __forceinline__ bool cfinite(cplx a) { return isfinite(a.re) && isfinite(a.im); }

constexpr int kAberthSweeps = 200;
constexpr double kAberthTol = 1e-14;
constexpr double kAberthFloor = 1e-12;

// Where the groups live.  d <= 2: at the velocity that leads them, in registers; the
// places of velocities that lead none are computed and masked off.  d >= 3: listed in
// LDS, since most of the q places would be empty (m = 8 has at most 8 groups of
// D3Q19's 19 or D4Q33's 33 velocities): at 300 points of D3Q19, m = 8, the registers'
// form took 3759 us.
template <int D>
constexpr bool kStabListed = D >= 3;
// Bytes of LDS per lane and group
template <int D>
constexpr int kStabBytes = kStabListed<D> ? 40 : 16;

// rho(G(xi)) at xi = 2 pi j / m; *converged is false when the iteration did
// not settle within kAberthSweeps sweeps.  roots: this lane's LDS column, root i
// at roots[64 i]; taus and sws, used if kStabListed<D>, likewise.
template <int D>
__device__ double rho_at(const double (&w)[q_of(D)], double s, const int (&j)[kMaxDim], int m,
                         cplx* roots, cplx* taus, double* sws, bool* converged) {
  constexpr int Q = q_of(D);
  constexpr bool LISTED = kStabListed<D>;
  const double a = 1.0 - s;
  double rho = 0.0;
  // group of velocity k: led by the first velocity with its phase
  int key[Q];
  static_for<0, Q>([&](auto K) {
    constexpr int k = decltype(K)::value;
    int ph = 0;
#pragma unroll
    for (int b = 0; b < D; ++b) ph += vel_comp(D, k, b) * j[b];
    ph %= m;
    key[k] = ph < 0 ? ph + m : ph;
  });
  cplx pole_r[Q], v_r[Q];
  unsigned long long active = 0;
  int ng = 0;
  static_for<0, Q>([&](auto K) {
    constexpr int k = decltype(K)::value;
    bool lead = true;
#pragma unroll
    for (int e = 0; e < k; ++e) lead = lead && key[e] != key[k];
    double W = 0.0;
    int cnt = 0;
#pragma unroll
    for (int e = k; e < Q; ++e) {
      const bool same = key[e] == key[k];
      W += same ? w[e] : 0.0;
      cnt += same ? 1 : 0;
    }
    // (1 - s) tau_g from the zero-sum vectors of a group, and from a group
    // whose weights cancel (its pole is then a root)
    if (lead && (cnt > 1 || W == 0.0)) rho = fmax(rho, fabs(a));
    const bool on = lead && W != 0.0;
    double sn, cs;
    sincospi(2.0 * key[k] / m, &sn, &cs);
    const cplx tau{cs, -sn};
    if constexpr (LISTED) {
      if (on) {
        taus[64 * ng] = tau;
        sws[64 * ng] = s * W;
      }
    } else {
      pole_r[k] = cscale(tau, a);
      v_r[k] = on ? cscale(tau, s * W) : cplx{0.0, 0.0};
      active |= on ? 1ull << k : 0ull;
    }
    ng += on ? 1 : 0;
  });
  const int places = LISTED ? ng : Q;
  const auto is_on = [&](int k) { return LISTED || ((active >> k) & 1); };
  const auto pole = [&](int k) {
    if constexpr (LISTED) return cscale(taus[64 * k], a);
    else return pole_r[k];
  };
  const auto v = [&](int k) {
    if constexpr (LISTED) return cscale(taus[64 * k], sws[64 * k]);
    else return v_r[k];
  };
  const auto each = [&](auto body) {
    if constexpr (LISTED) {
#pragma unroll 2
      for (int k = 0; k < ng; ++k) body(k);
    } else {
      static_for<0, Q>([&](auto K) { body(K); });
    }
  };
  *converged = true;
  if (ng == 0) return rho;
  cplx vsum{0.0, 0.0}, psum{0.0, 0.0};
  int big = 0;
  double vbig = -1.0;
  each([&](auto k_) {
      const int k = k_;
    const bool on = is_on(k);
    vsum = cadd(vsum, v(k));
    psum.re += on ? pole(k).re : 0.0;
    psum.im += on ? pole(k).im : 0.0;
    const double vg = cabs2(v(k));
    if (on && vg > vbig) {
      vbig = vg;
      big = k;
    }
  });
  // all poles at 0: p(lambda) = lambda^(ng-1) (lambda - sum_g v_g)
  if (a == 0.0) return fmax(rho, sqrt(cabs2(vsum)));
  // Start: ng - 1 roots just beside the poles (scaled by 1.01, turned by
  // pi / (4 ng)); the one of the largest |v_g| is replaced by the estimate of
  // the root that carries the conserved mode, sum_g v_g + a mean(tau).
  {
    double sn, cs;
    sincospi(0.25 / ng, &sn, &cs);
    const cplx turn{1.01 * cs, 1.01 * sn};
    each([&](auto k_) {
      const int k = k_;
      roots[64 * k] = cmul(pole(k), turn);
    });
    roots[64 * big] = cadd(cadd(vsum, cscale(psum, 1.0 / ng)), cplx{0.0, 1e-3});
  }
  bool done = false;
  double prev = INFINITY;
  for (int it = 0; it < kAberthSweeps && !done; ++it) {
    double worst = 0.0;
    for (int i = 0; i < places; ++i) {
      if (!is_on(i)) continue;
      const cplx z = roots[64 * i];
      // nearest pole h, kept out of the sums so that nothing blows up near it
      int h = -1;
      double dh = INFINITY;
      cplx ph{0.0, 0.0}, vh{0.0, 0.0};
      each([&](auto g_) {
      const int g = g_;
        const double dg = cabs2(csub(z, pole(g)));
        const bool nearer = is_on(g) && (dg < dh || h < 0);
        dh = nearer ? dg : dh;
        h = nearer ? g : h;
        ph.re = nearer ? pole(g).re : ph.re;
        ph.im = nearer ? pole(g).im : ph.im;
        vh.re = nearer ? v(g).re : vh.re;
        vh.im = nearer ? v(g).im : vh.im;
      });
      cplx f{1.0, 0.0}, fp{0.0, 0.0}, S{0.0, 0.0}, ab{0.0, 0.0};
      each([&](auto g_) {
      const int g = g_;
        const bool on = is_on(g);
        const bool keep = on && g != h;
        cplx inv = cinv(csub(z, pole(g)));
        inv.re = keep ? inv.re : 0.0;
        inv.im = keep ? inv.im : 0.0;
        const cplx vi = cmul(v(g), inv);
        f = csub(f, vi);
        fp = cadd(fp, cmul(vi, inv));
        S = cadd(S, inv);
        const bool other = on && g != i;
        const cplx il = cinv(csub(z, roots[64 * g]));
        ab.re += other ? il.re : 0.0;
        ab.im += other ? il.im : 0.0;
      });
      // p / p' with p = prod_{g != h} (z - pole_g) [(z - pole_h) f_h - v_h]
      const cplx e = csub(z, ph);
      const cplx num = csub(cmul(e, f), vh);
      const cplx den = csub(cadd(f, cmul(e, cadd(cmul(S, f), fp))), cmul(vh, S));
      const cplx N = cdiv(num, den);
      cplx corr = cdiv(N, csub(cplx{1.0, 0.0}, cmul(N, ab)));
      if (!cfinite(corr)) corr = cplx{1e-8, 1e-8};  // landed on a pole or a root
      const cplx next = csub(z, corr);
      roots[64 * i] = next;
      const double rel = sqrt(cabs2(corr)) / fmax(1.0, sqrt(cabs2(next)));
      worst = fmax(worst, rel);
    }
    // settled: corrections below the tolerance, or at the rounding floor
    // (small and no longer shrinking the way a converging iteration does)
    done = worst < kAberthTol || (worst < kAberthFloor && worst > 0.5 * prev);
    prev = worst;
  }
  *converged = done;
  for (int g = 0; g < places; ++g) {
    if (!is_on(g)) continue;
    const cplx l = roots[64 * g];
    if (!cfinite(l)) {
      *converged = false;
      return INFINITY;
    }
    rho = fmax(rho, sqrt(cabs2(l)));
  }
  return rho;
}

// How the wave numbers (nh per point) are dealt to blocks of one wavefront: `points` whole
// points to a block, or, if the call is too small to fill the chip so, one point to `parts`
// blocks.  81 points of D2Q9, m = 8, and 343 of D3Q19, m = 8, take 206 and 521 us in parts.
struct StabSplit {
  int points, parts;
};
// Two wavefronts per SIMD; four rounds of a block leave at most a fifth of its last one
// idle.
constexpr long long kStabFill = 2048;
constexpr int kStabRounds = 4, kStabMaxPoints = 64;
StabSplit stab_split(long long nh, long long count) {
  const long long rounds = (nh + 63) / 64;
  if (rounds > 1 && count < kStabFill) {
    const long long parts = (kStabFill + count - 1) / count;
    return {1, static_cast<int>(parts < rounds ? parts : rounds)};
  }
  int p = 1;
  while (p < kStabMaxPoints && p * nh < 64 * kStabRounds && (p + 1) * kStabFill / 2 <= count) ++p;
  return {p, 1};
}

// The outputs of a call whose points are split over blocks, which accumulate them.
__global__ void k_stability_clear(long long count, double* __restrict__ rho_out,
                                  int32_t* __restrict__ unconv_out) {
  const long long i = static_cast<long long>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= count) return;
  rho_out[i] = 0.0;
  if (unconv_out) unconv_out[i] = 0;
}

template <int D>
__global__ void __launch_bounds__(64)
    k_stability(const double* sigma, const double* s_arr, double gm4, int m, long long nh,
                long long count, StabSplit split, int groups, double* rho_out,
                double* min_omega_out, int32_t* unconv_out) {
  constexpr int Q = q_of(D);
  extern __shared__ __align__(16) unsigned char stab_lds[];  // kStabBytes<D> x 64 x groups
  cplx* const roots = reinterpret_cast<cplx*>(stab_lds);
  cplx* const taus = roots + 64 * groups;
  double* const sws = reinterpret_cast<double*>(taus + 64 * groups);
  __shared__ unsigned long long best[kStabMaxPoints];  // rho as its bits: rho >= 0
  __shared__ int bad[kStabMaxPoints];
  const int lane = threadIdx.x;
  const long long p0 = blockIdx.x / split.parts * static_cast<long long>(split.points);
  const int part = blockIdx.x % split.parts;
  const int here = static_cast<int>(min(static_cast<long long>(split.points), count - p0));
  if (lane < here) {
    best[lane] = 0ull;
    bad[lane] = 0;
  }
  __syncthreads();
  const int half = m / 2 + 1;
  for (long long e = part * 64 + lane; e < here * nh; e += 64 * split.parts) {
    const int pl = static_cast<int>(e / nh);
    const long long pt = p0 + pl;
    double u[kMaxDim] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int a = 0; a < D; ++a) u[a] = sigma[pt * D + a];
    const double m4 = (D >= 2) ? m4_interpolated(D, u, gm4) : 0.0;
    double w[Q];
    omega_closed_form(D, u, m4, w);
    long long r = e - pl * nh;
    int j[kMaxDim] = {0, 0, 0, 0};
    j[D - 1] = static_cast<int>(r % half);
    r /= half;
#pragma unroll
    for (int a = 0; a < D - 1; ++a) {
      j[a] = static_cast<int>(r % m);
      r /= m;
    }
    bool ok = true;
    const double rho = rho_at<D>(w, s_arr[pt], j, m, roots + lane, taus + lane, sws + lane, &ok);
    atomicMax(&best[pl], static_cast<unsigned long long>(__double_as_longlong(rho)));
    // a wave number strictly inside stands for its mirror image too
    if (!ok) atomicAdd(&bad[pl], j[D - 1] == 0 || 2 * j[D - 1] == m ? 1 : 2);
  }
  __syncthreads();
  if (lane < here) {
    const long long pt = p0 + lane;
    // from the inputs before an output is written: they may share memory
    double mw = 0.0;
    if (min_omega_out && part == 0) {
      double u[kMaxDim] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int a = 0; a < D; ++a) u[a] = sigma[pt * D + a];
      double w[Q];
      omega_closed_form(D, u, (D >= 2) ? m4_interpolated(D, u, gm4) : 0.0, w);
      mw = w[0];
#pragma unroll
      for (int k = 1; k < Q; ++k) mw = fmin(mw, w[k]);
    }
    if (split.parts > 1) {
      atomicMax(reinterpret_cast<unsigned long long*>(rho_out) + pt, best[lane]);
      if (unconv_out && bad[lane]) atomicAdd(unconv_out + pt, bad[lane]);
    } else {
      rho_out[pt] = __longlong_as_double(static_cast<long long>(best[lane]));
      if (unconv_out) unconv_out[pt] = bad[lane];
    }
    if (min_omega_out && part == 0) min_omega_out[pt] = mw;
  }
}

template <int D>
hipError_t stability_pass(long long count, const double* sigma, const double* s, double g, int m,
                          long long nxi, double* rho, double* min_omega, int32_t* unconverged,
                          hipStream_t stream) {
  const long long nh = nxi / m * (m / 2 + 1);
  StabSplit split = stab_split(nh, count);
  // outputs in the memory of s (or, d = 1, of sigma): one block reads a point's inputs
  // before it writes them
  for (const double* out : {rho, min_omega})
    if (out && (out == s || out == sigma)) split = StabSplit{1, 1};
  // no wave number has more groups than phases or velocities
  const int groups = kStabListed<D> && m < q_of(D) ? m : q_of(D);
  constexpr int most = kStabBytes<D> * 64 * q_of(D);
  if constexpr (most > 65536) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_stability<D>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, most);
    if (e != hipSuccess) return e;
  }
  const unsigned blocks =
      static_cast<unsigned>((count + split.points - 1) / split.points * split.parts);
  if (split.parts > 1)
    hipLaunchKernelGGL(k_stability_clear, dim3(static_cast<unsigned>((count + 255) / 256)),
                       dim3(256), 0, stream, count, rho, unconverged);
  hipLaunchKernelGGL(k_stability<D>, dim3(blocks), dim3(64), kStabBytes<D> * 64 * groups, stream,
                     sigma, s, g, m, nh, count, split, groups, rho, min_omega, unconverged);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_stability(int d, long long count, const double* sigma, const double* s,
                            double g, int m, long long nxi, double* rho, double* min_omega,
                            int32_t* unconverged, hipStream_t stream) {
  switch (d) {
    case 1:
      return stability_pass<1>(count, sigma, s, g, m, nxi, rho, min_omega, unconverged, stream);
    case 2:
      return stability_pass<2>(count, sigma, s, g, m, nxi, rho, min_omega, unconverged, stream);
    case 3:
      return stability_pass<3>(count, sigma, s, g, m, nxi, rho, min_omega, unconverged, stream);
    case 4:
      return stability_pass<4>(count, sigma, s, g, m, nxi, rho, min_omega, unconverged, stream);
    default:
      return hipErrorInvalidValue;
  }
}

}  // namespace lbm
