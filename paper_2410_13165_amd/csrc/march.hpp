// Several time steps of a d = 2 lattice in one pass (k_march2, and k_pair2 for two steps
// of large periodic lattices) and of a d = 1 lattice (k_line), with the data of the
// Dirichlet walls for the steps of a pass formed beforehand (k_wall_data2, k_wall_data1).
//
// d = 2.
// One wavefront owns 64 consecutive columns of x_1 and marches along x_2.  Per
// source row it loads the post-collision populations of its columns (stage 0)
// and pushes them into stage 1, which thereby completes its row one behind,
// collides it and pushes it into stage 2, and so on: stage L holds the state
// after L steps, one row behind stage L - 1, and the last stage stores.  A
// population moves along x_1 by a one-lane shift of the wavefront (a DPP move),
// along x_2 by waiting in a register: c_2 = -1 values complete the row behind
// at once, c_2 = 0 values wait one row and c_2 = +1 values two.  Nothing is
// exchanged between wavefronts, so there is no LDS and no barrier; the price is
// a halo of NL columns on either side and NL rows above and below a tile, computed twice.
//
// Every node goes through the arithmetic of k_step (k_step_split, k_wall and
// k_wall_split on the walls), so a pass is bitwise NL single steps.
#pragma once

#include <hip/hip_runtime.h>

#include "kernels.hpp"

namespace lbm {

// value of the lane below (l - 1) or above (l + 1); the first (last) lane
// keeps its own
__device__ __forceinline__ int lane_below(int v) {
  return __builtin_amdgcn_update_dpp(v, v, 0x138, 0xf, 0xf, false);  // wave_shr:1
}
__device__ __forceinline__ int lane_above(int v) {
  return __builtin_amdgcn_update_dpp(v, v, 0x130, 0xf, 0xf, false);  // wave_shl:1
}
__device__ __forceinline__ float lane_below(float v) {
  return __int_as_float(lane_below(__float_as_int(v)));
}
__device__ __forceinline__ float lane_above(float v) {
  return __int_as_float(lane_above(__float_as_int(v)));
}
__device__ __forceinline__ double lane_below(double v) {
  return __hiloint2double(lane_below(__double2hiint(v)), lane_below(__double2loint(v)));
}
__device__ __forceinline__ double lane_above(double v) {
  return __hiloint2double(lane_above(__double2hiint(v)), lane_above(__double2loint(v)));
}

// The populations of D2Q9 by their c_2: march_pop(cy, j) is the j-th
// (j = 0..2) with c_2 = cy; march_slot(k) its j.
constexpr int march_pop(int cy, int j) {
  int n = 0;
  for (int k = 0; k < q_of(2); ++k) {
    if (vel_comp(2, k, 1) != cy) continue;
    if (n == j) return k;
    ++n;
  }
  return -1;
}
constexpr int march_slot(int k) {
  const int cy = vel_comp(2, k, 1);
  int idx = 0;
  for (int m = 0; m < k; ++m)
    if (vel_comp(2, m, 1) == cy) ++idx;
  return idx;
}

// Value of population k that enters a wall node from outside: v the analytic
// wall value (wall_close included), own the node's own post-collision kbar
// value (half-way walls), ref the float32 reference of the step.  The rows on
// a wall of x_2 round as k_wall does, the x_1 faces of the other rows as
// k_xface and k_step do (the two differ in float32 half-way lattices only).
template <int MODE, bool HALF, int k, class A, int D = 2>
__device__ __forceinline__ A march_wall_value(double v, A own, bool rowwall, double ref,
                                              const MarchParams& p) {
  constexpr int kb = opp_index(D, k);
  if constexpr (MODE == kFP32) {
    if constexpr (!HALF) return static_cast<A>(wall_deviation<2>(v, p.omega[k], ref));
    const double fs = wall_absolute<2>(static_cast<double>(own), p.omega[kb], ref);
    const A row = static_cast<A>(wall_deviation<2>(v - fs, p.omega[k], ref));
    const A face = static_cast<A>(wall_deviation<2>(v, p.omega[k] + p.omega[kb], ref)) - own;
    return rowwall ? row : face;
  } else {
    return HALF ? v - own : v;
  }
}

// Bytes of LDS one wavefront of a pass over walls takes: the data of both x_1
// faces for its rows, and of both x_2 faces for its columns.
__host__ __device__ constexpr int march_lds(int nl, int yc) {
  return static_cast<int>(sizeof(double)) * nl * 6 * ((yc + 2 * nl) + 64);
}

// One wavefront's tile: NL steps of output columns x0 .. x0 + width - 1 and rows
// y0 .. y1 - 1 (width <= march_width(NL)).  The next D source rows are kept in
// flight.  WALL: 0 periodic lattice, kFullWay or kHalfWay with either axis
// Dirichlet (lds: march_lds bytes of this wavefront's own).  step: index n of
// the source state.
template <int MODE, int NL, int WALL, int D>
__device__ __forceinline__ void march2_tile(const MarchParams& p, const MarchBufs& b, const int x0,
                                            const int width, const int y0, const int y1,
                                            const long long step, double* lds) {
  using T = std::conditional_t<MODE == kFP64, double, float>;   // stored populations
  using A = std::conditional_t<MODE == kFP32, float, double>;   // arithmetic
  constexpr int Q = q_of(2);
  constexpr bool HALF = WALL == kHalfWay;
  const int n0 = p.n0, n1 = p.n1;
  const long long ps = p.ps;
  const T* __restrict__ src = static_cast<const T*>(b.src);
  T* __restrict__ dst = static_cast<T*>(b.dst);
  const int lane = static_cast<int>(threadIdx.x) & 63;
  const int x = x0 - NL + lane;
  const bool wallx = WALL != 0 && p.bc0 != 0, wally = WALL != 0 && p.bc1 != 0;
  const int xc = wallx ? min(max(x, 0), n0 - 1) : fuse_wrap(x, n0);
  const bool store_lane = lane >= NL && lane < NL + width && x < n0;
  const bool lo = wallx && x == 0, hi = wallx && x == n0 - 1;
  const bool edge = wallx && (x0 - NL <= 0 || x0 - NL + 63 >= n0 - 1);  // wave-uniform
  auto row_in = [&](int r) { return wally ? min(max(r, 0), n1 - 1) : fuse_wrap(r, n1); };

  // wall data of the pass: wfx[((l * 2 + side) * 3 + j) * rows + y - ybase] and
  // wfy[((l * 2 + side) * 3 + j) * 64 + lane], read back by this wavefront only
  const int ybase = y0 - NL, rows = (y1 - y0) + 2 * NL;
  double* wfx = lds;
  double* wfy = lds + NL * 6 * rows;
  if constexpr (WALL != 0) {
    // groups of loads in flight together: one at a time, their latencies alone
    // took as long as the pass of a small lattice
    if (edge) {
      const int total = NL * 6 * rows;
      for (int i0 = lane; i0 < total; i0 += 64 * 8) {
        double v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int i = min(i0 + 64 * u, total - 1), e = i / rows;
          v[u] = p.wx[static_cast<long long>(e) * n1 + row_in(ybase + i - e * rows)];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) wfx[min(i0 + 64 * u, total - 1)] = v[u];
      }
    }
    if (wally && (ybase <= 0 || ybase + rows >= n1)) {
      double v[NL * 6];
#pragma unroll
      for (int e = 0; e < NL * 6; ++e) v[e] = p.wy[static_cast<long long>(e) * n0 + xc];
#pragma unroll
      for (int e = 0; e < NL * 6; ++e) wfy[e * 64 + lane] = v[e];
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
  // source rows in flight
  T raw[D][Q];
  double phr[D];
  auto load_row = [&](int r, auto Slot) {
    constexpr int s = decltype(Slot)::value;
    const long long node = static_cast<long long>(row_in(r)) * n0 + xc;
#pragma unroll
    for (int k = 0; k < Q; ++k) raw[s][k] = src[k * ps + node];
    if constexpr (MODE == kSplit) phr[s] = b.phi_src[node];
  };
  // stage l + 1: c_2 = +1 values waiting for the next row (up) and the one
  // after it (up2), c_2 = 0 for the next row (mid); half-way: the values that
  // replace c_2 = -1 ones of the next row (over)
  A up[NL][3] = {}, up2[NL][3] = {}, mid[NL][3] = {};
  A over[HALF ? NL : 1][3] = {};
  const int iters = (y1 - y0) + 2 * NL;
  static_for<0, D>([&](auto S) {
    if (decltype(S)::value < iters) load_row(y0 - NL + decltype(S)::value, S);
  });
  auto iteration = [&](const int i, auto Slot) {
    constexpr int slot = decltype(Slot)::value;
    const int r = y0 - NL + i;  // source row of this iteration
    A g[Q];
    if constexpr (MODE == kSplit) {
      const double t = phr[slot] + p.dtR;
#pragma unroll
      for (int k = 0; k < Q; ++k) g[k] = split_fstar_t(p.omega[k], t, raw[slot][k], p);
    } else {
#pragma unroll
      for (int k = 0; k < Q; ++k) g[k] = raw[slot][k];
    }
    if (i + D < iters) load_row(r + D, Slot);
    // x_1-face data of the row whose wall values each stage forms: the one it
    // completes (full-way) or the one pushed into it, whose own values it needs
    // (half-way); read together, so that the stages wait for LDS once
    double wx[WALL ? NL : 1][3] = {};
    if constexpr (WALL != 0) {
      if (edge) {
#pragma unroll
        for (int l = 0; l < NL; ++l) {
          const int yi = max(r - l - (HALF ? 0 : 1) - ybase, 0);
#pragma unroll
          for (int j = 0; j < 3; ++j) wx[l][j] = wfx[((l * 2 + (hi ? 1 : 0)) * 3 + j) * rows + yi];
        }
      }
    }
    static_for<0, NL>([&](auto Lx) {
      constexpr int l = decltype(Lx)::value;
      if (i < 2 * l) return;    // nothing complete below yet
      const int rho = r - l;    // row of g
      const int y = rho - 1;    // row this stage completes
      A f[Q], sh[Q];
      static_for<0, Q>([&](auto K) {
        constexpr int k = decltype(K)::value;
        constexpr int cx = vel_comp(2, k, 0);
        if constexpr (cx == 1) sh[k] = lane_below(g[k]);
        else if constexpr (cx == -1) sh[k] = lane_above(g[k]);
        else sh[k] = g[k];
      });
      static_for<0, Q>([&](auto K) {
        constexpr int k = decltype(K)::value;
        constexpr int cy = vel_comp(2, k, 1);
        if constexpr (cy == 1) f[k] = up[l][march_slot(k)];
        else if constexpr (cy == 0) f[k] = mid[l][march_slot(k)];
        else f[k] = sh[k];
      });
      if constexpr (WALL != 0) {
        const bool rowlo = wally && y == 0, rowhi = wally && y == n1 - 1;
        if constexpr (!HALF) {
          const double ref =
              MODE == kFP32 ? p.phi_ref + p.R * (step_time(step + l, p.dt) + p.dt) : 0.0;
          if (rowlo || rowhi) {
            double wy[3];
#pragma unroll
            for (int j = 0; j < 3; ++j) wy[j] = wfy[((l * 2 + (rowhi ? 1 : 0)) * 3 + j) * 64 + lane];
            static_for<1, Q>([&](auto K) {
              constexpr int k = decltype(K)::value;
              constexpr int cy = vel_comp(2, k, 1);
              if constexpr (cy != 0) {
                const A val =
                    march_wall_value<MODE, false, k>(wy[march_slot(k)], A(0), true, ref, p);
                f[k] = (cy == 1 ? rowlo : rowhi) ? val : f[k];
              }
            });
          }
          if (edge) {
            static_for<1, Q>([&](auto K) {
              constexpr int k = decltype(K)::value;
              constexpr int cx = vel_comp(2, k, 0);
              if constexpr (cx != 0) {
                const A val = march_wall_value<MODE, false, k>(wx[l][xface_slot(2, k)], A(0),
                                                               rowlo || rowhi, ref, p);
                f[k] = (cx == 1 ? lo : hi) ? val : f[k];
              }
            });
          }
        } else {
          static_for<0, 3>([&](auto J) {
            constexpr int j = decltype(J)::value;
            constexpr int k = march_pop(-1, j);
            constexpr int cx = vel_comp(2, k, 0);
            const bool in = rowhi || (cx == 1 ? lo : (cx == -1 ? hi : false));
            f[k] = in ? over[l][j] : f[k];
          });
        }
      }
#pragma unroll
      for (int m = 0; m < 3; ++m) up[l][m] = up2[l][m];
      static_for<0, Q>([&](auto K) {
        constexpr int k = decltype(K)::value;
        constexpr int cy = vel_comp(2, k, 1);
        if constexpr (cy == 1) up2[l][march_slot(k)] = sh[k];
        else if constexpr (cy == 0) mid[l][march_slot(k)] = sh[k];
      });
      if constexpr (HALF) {
        // what enters row rho from outside, formed from its own post-collision
        // values g, which are here now
        const bool rowlo = wally && rho == 0, rowhi = wally && rho == n1 - 1;
        const bool rw = rowlo || rowhi;
        if (edge || rw) {
          const double ref =
              MODE == kFP32 ? p.phi_ref + p.R * (step_time(step + l, p.dt) + p.dt) : 0.0;
          double wy[3] = {};
          if (rw) {
#pragma unroll
            for (int j = 0; j < 3; ++j) wy[j] = wfy[((l * 2 + (rowhi ? 1 : 0)) * 3 + j) * 64 + lane];
          }
          static_for<1, Q>([&](auto K) {
            constexpr int k = decltype(K)::value;
            constexpr int cx = vel_comp(2, k, 0), cy = vel_comp(2, k, 1);
            constexpr int kb = opp_index(2, k), m = march_slot(k);
            const bool inx = (cx == 1 && lo) || (cx == -1 && hi);
            const bool in = inx || (cy == 1 && rowlo) || (cy == -1 && rowhi);
            double w = wy[m];
            if constexpr (cx != 0) {
              const double fx = wx[l][xface_slot(2, k)];
              if (inx) w = fx;
            }
            const A val = march_wall_value<MODE, true, k>(w, g[kb], rw, ref, p);
            if constexpr (cy == 1) up[l][m] = in ? val : up[l][m];
            else if constexpr (cy == 0) mid[l][m] = in ? val : mid[l][m];
            else over[l][m] = in ? val : over[l][m];
          });
        }
      }
      const long long node = static_cast<long long>(y) * n0 + x;
      if constexpr (MODE == kSplit) {
        double phi = 0.0;
#pragma unroll
        for (int k = 0; k < Q; ++k) phi += f[k];
        float gk[Q];
#pragma unroll
        for (int k = 0; k < Q; ++k) gk[k] = static_cast<float>(f[k] - p.omega[k] * phi);
        if constexpr (l == NL - 1) {
          if (store_lane && i >= 2 * NL) {
            phi_put(b.phi_dst, node, phi);
#pragma unroll
            for (int k = 0; k < Q; ++k) __builtin_nontemporal_store(gk[k], dst + k * ps + node);
          }
        } else {
          const double t = phi + p.dtR;
#pragma unroll
          for (int k = 0; k < Q; ++k) g[k] = split_fstar_t(p.omega[k], t, gk[k], p);
        }
      } else {
        collide_vals<2, A>(f, p);
        if constexpr (l == NL - 1) {
          if (store_lane && i >= 2 * NL) {
#pragma unroll
            for (int k = 0; k < Q; ++k)
              __builtin_nontemporal_store(static_cast<T>(f[k]), dst + k * ps + node);
          }
        } else {
#pragma unroll
          for (int k = 0; k < Q; ++k) g[k] = f[k];
        }
      }
    });
  };
  for (int i = 0; i < iters; i += D)
    static_for<0, D>([&](auto S) {
      if (i + decltype(S)::value < iters) iteration(i + decltype(S)::value, S);
    });
}

// Two steps of a periodic d = 2 lattice, one tile of kPairWidth columns per block.
// The block marches along x_2; the state after the first step of a row lies in LDS
// until the second has read it: c_2 = +1 values for three rows, c_2 = 0 values two,
// c_2 = -1 values one.  Loads and stores are whole aligned lines and the halo is two
// columns of 258, where a wavefront's tile recomputes 8 of 64: large lattices, bound by
// their traffic, gain (two steps of 4096^2: float32 238 against 327 us, float64 465
// against 498).
constexpr int kPairWidth = 256, kPairSlots = 18;

template <int k>
__device__ __forceinline__ int pair_slot(int it) {
  constexpr int cy = vel_comp(2, k, 1), i = march_slot(k);
  if constexpr (cy == 0) return 2 * i + (it & 1);
  else if constexpr (cy == 1) return 6 + 3 * i + it % 3;
  else return 15 + i;
}

template <class T>
__device__ __forceinline__ void pair2_tile(const MarchParams& p, const T* __restrict__ src,
                                           T* __restrict__ dst, T* lds, const int x0, const int y0,
                                           const int y1) {
  constexpr int Q = q_of(2), R = kPairWidth + 2;
  const long long ps = p.ps;
  const int n0 = p.n0, n1 = p.n1;
  const int r = static_cast<int>(threadIdx.x);
  const int iters = y1 - y0 + 2;
  for (int it = 0; it < iters; ++it) {
    // step 1 on the tile and its halo of row y0 - 1 + it
    const int y = fuse_wrap(y0 - 1 + it, n1);
    const int ym = y == 0 ? n1 - 1 : y - 1, yp = y == n1 - 1 ? 0 : y + 1;
    for (int rr = r; rr < R; rr += kPairWidth) {
      const int x = fuse_wrap(x0 - 1 + rr, n0);
      const int xm = x == 0 ? n0 - 1 : x - 1, xp = x == n0 - 1 ? 0 : x + 1;
      T f[Q];
      static_for<0, Q>([&](auto K) {
        constexpr int k = decltype(K)::value;
        constexpr int cx = vel_comp(2, k, 0), cy = vel_comp(2, k, 1);
        const int ys = cy == 1 ? ym : (cy == -1 ? yp : y), xs = cx == 1 ? xm : (cx == -1 ? xp : x);
        f[k] = src[k * ps + static_cast<long long>(ys) * n0 + xs];
      });
      collide_vals<2, T>(f, p);
      static_for<0, Q>([&](auto K) {
        constexpr int k = decltype(K)::value;
        lds[pair_slot<k>(it) * R + rr] = f[k];
      });
    }
    __syncthreads();
    // step 2 on the row before it
    const int x = x0 + r;
    if (it >= 2 && x < n0) {
      T f[Q];
      static_for<0, Q>([&](auto K) {
        constexpr int k = decltype(K)::value;
        constexpr int cx = vel_comp(2, k, 0), cy = vel_comp(2, k, 1);
        constexpr int back = cy == 0 ? 1 : (cy == 1 ? 2 : 0);
        f[k] = lds[pair_slot<k>(it - back) * R + (r + 1 - cx)];
      });
      collide_vals<2, T>(f, p);
      const long long node = static_cast<long long>(y0 - 2 + it) * n0 + x;
#pragma unroll
      for (int k = 0; k < Q; ++k) __builtin_nontemporal_store(f[k], dst + k * ps + node);
    }
    __syncthreads();
  }
}

// nsteps steps of a d = 1 lattice in one launch.  A block keeps a window of nodes
// in registers, M adjacent ones per thread, and only the two populations that
// cross to a neighbouring thread go through LDS, double-buffered: one barrier per
// step.  A lattice of at most kLineNodes nodes is one window (M = 1, nothing
// computed twice, any number of steps); longer ones are cut into windows with a
// halo of nsteps nodes on either side.  wx[l * 2 + side]: the wall data of step l.
// Per node the arithmetic of k_step (k_step_split) with k_xface's data.
template <int MODE, int WALL, int M>
__device__ __forceinline__ void line_block(const MarchParams& p, const MarchBufs& b,
                                           const int first, const int used, const int out0,
                                           const int out1, const int nsteps,
                                           const long long step, unsigned char* mem) {
  using T = std::conditional_t<MODE == kFP64, double, float>;
  using A = std::conditional_t<MODE == kFP32, float, double>;
  constexpr bool HALF = WALL == kHalfWay;
  const int tid = static_cast<int>(threadIdx.x), nt = static_cast<int>(blockDim.x);
  double* wx = reinterpret_cast<double*>(mem);
  A* edge = reinterpret_cast<A*>(mem + (WALL ? sizeof(double) * 2 * nsteps : 0));
  const int n0 = p.n0;
  const long long ps = p.ps;
  const T* __restrict__ src = static_cast<const T*>(b.src);
  T* __restrict__ dst = static_cast<T*>(b.dst);
  if constexpr (WALL != 0)
    for (int i = tid; i < 2 * nsteps; i += nt) wx[i] = p.wx[i];  // seen after the first barrier
  // the window's nodes first .. first + used - 1; a window that is the whole
  // periodic lattice closes on itself
  const int left = tid == 0 ? (used - 1) / M : tid - 1;
  const int right = (tid + 1) * M >= used ? 0 : tid + 1;
  A g[M][3];
  float gs[M][3];
  double phi[M];
#pragma unroll
  for (int j = 0; j < M; ++j) {
    int x = first + tid * M + j;
    x = WALL != 0 ? min(max(x, 0), n0 - 1) : fuse_wrap(x, n0);
    if constexpr (MODE == kSplit) {
      phi[j] = b.phi_src[x];
#pragma unroll
      for (int k = 0; k < 3; ++k) gs[j][k] = src[k * ps + x];
#pragma unroll
      for (int k = 0; k < 3; ++k)
        g[j][k] = split_fstar_t(p.omega[k], phi[j] + p.dtR, gs[j][k], p);
    } else {
#pragma unroll
      for (int k = 0; k < 3; ++k) g[j][k] = src[k * ps + x];
    }
  }
  for (int l = 0; l < nsteps; ++l) {
    A* e = edge + (l & 1) * 2 * nt;
    e[tid] = g[M - 1][1];
    e[nt + tid] = g[0][2];
    __syncthreads();
    const A from_left = e[left], from_right = e[nt + right];
    A f[M][3];
#pragma unroll
    for (int j = 0; j < M; ++j) {
      f[j][0] = g[j][0];
      f[j][1] = j == 0 ? from_left : g[j - 1][1];
      f[j][2] = j == M - 1 ? from_right : g[j + 1][2];
    }
    if constexpr (WALL != 0) {
      const double ref =
          MODE == kFP32 ? p.phi_ref + p.R * (step_time(step + l, p.dt) + p.dt) : 0.0;
#pragma unroll
      for (int j = 0; j < M; ++j) {
        const int x = first + tid * M + j;
        if (x == 0)
          f[j][1] = march_wall_value<MODE, HALF, 1, A, 1>(wx[2 * l], g[j][2], false, ref, p);
        if (x == n0 - 1)
          f[j][2] = march_wall_value<MODE, HALF, 2, A, 1>(wx[2 * l + 1], g[j][1], false, ref, p);
      }
    }
#pragma unroll
    for (int j = 0; j < M; ++j) {
      if constexpr (MODE == kSplit) {
        double s = 0.0;
#pragma unroll
        for (int k = 0; k < 3; ++k) s += f[j][k];
        phi[j] = s;
#pragma unroll
        for (int k = 0; k < 3; ++k) gs[j][k] = static_cast<float>(f[j][k] - p.omega[k] * s);
        const double t = s + p.dtR;
#pragma unroll
        for (int k = 0; k < 3; ++k) g[j][k] = split_fstar_t(p.omega[k], t, gs[j][k], p);
      } else {
        collide_vals<1, A>(f[j], p);
#pragma unroll
        for (int k = 0; k < 3; ++k) g[j][k] = f[j][k];
      }
    }
  }
#pragma unroll
  for (int j = 0; j < M; ++j) {
    const int x = first + tid * M + j;
    if (x < out0 || x >= out1) continue;
    if constexpr (MODE == kSplit) b.phi_dst[x] = phi[j];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      if constexpr (MODE == kSplit) dst[k * ps + x] = gs[j][k];
      else dst[k * ps + x] = static_cast<T>(g[j][k]);
    }
  }
}

}  // namespace lbm
