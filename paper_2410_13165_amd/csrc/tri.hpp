// Three time steps of a d = 3 lattice in one pass (k_tri).
//
// A block owns an x_1-x_2 tile and marches along x_3.  Each thread owns one
// column of the tile and its halo of two, for all three steps: per source plane it
// pulls 19 values (step 1), collides and writes what leaves its column to LDS;
// after a barrier the columns inside the halo of one read their neighbours' values
// and push them into step 2, and after a second barrier the tile's columns do the
// same for step 3 and store.  As in the d = 2 passes (march.hpp) a step's values
// wait in registers along the marching direction: c_3 = -1 values complete the
// plane behind at once, c_3 = 0 values wait one plane, c_3 = +1 values two.  So LDS
// holds one plane of 16 populations per step (the three that stay in their column
// never go there), where the two-step passes hold two planes on average, and the
// next source plane's pulls are in flight while steps 2 and 3 compute.
//
// Rows on a Dirichlet wall of x_2 or x_3 are not updated here.  Their values after
// one step come from C1 (k_wall on A), after two from C2 (k_wall on C1, whose rows
// next to a wall k_step_near has updated), and k_wall on C2 updates them for step
// 3 afterwards; for that launch this kernel stores its two-step values of the rows
// next to those walls in C2.  The x_1-face data of the three steps lie in the row
// slots of A, C1 and B.  Every node goes through the arithmetic of k_step,
// so a pass is bitwise three single steps.
#pragma once

#include <hip/hip_runtime.h>

#include "kernels.hpp"

namespace lbm {

// Tiles: TX output columns by TY rows, one thread per column of the tile and its
// halo of two, PX = TX + 4 by PY = TY + 4 (threads come in whole wavefronts of 64
// interior columns, or two rows of 32).  Float32 takes the largest tile that 1024
// threads cover (its 128 registers hold the waiting values of both steps and the
// plane in flight); with half-way walls that many spilled 21 registers (2600 us
// per 512^3 step), so it takes 768 threads (2350). Float64 needs twice the
// registers: 512 threads.
template <class T, bool HALF>
struct TriShape;
template <>
struct TriShape<float, false> {
  static constexpr int TX = 64, TY = 11, NT = 1024;
  static constexpr bool AHEAD = false;
};
template <>
struct TriShape<float, true> {
  static constexpr int TX = 64, TY = 7, NT = 768;
  static constexpr bool AHEAD = true;
};
template <bool HALF>
struct TriShape<double, HALF> {
  static constexpr int TX = 32, TY = 10, NT = 512;
  static constexpr bool AHEAD = false;
};

// LDS slot of population k among the 16 that leave their column (-1: the others)
constexpr int tri_slot(int k) {
  if (vel_comp(3, k, 0) == 0 && vel_comp(3, k, 1) == 0) return -1;
  int n = 0;
  for (int m = 0; m < k; ++m)
    if (vel_comp(3, m, 0) != 0 || vel_comp(3, m, 1) != 0) ++n;
  return n;
}

// thread t's column (px, py) in the tile and its halo: the TX interior columns of
// every row first (aligned loads), then the four halo columns
template <int TX, int PY>
__device__ __forceinline__ void tri_column(int t, int& px, int& py) {
  if (t < TX * PY) {
    py = t / TX;
    px = 2 + t % TX;
  } else {
    const int h = t - TX * PY;
    py = h >> 2;
    px = (h & 3) < 2 ? (h & 3) : TX + (h & 3);
  }
}

// Address at a uniform base and a 32-bit byte offset of the lane (a plane is under
// 4 GiB).  The empty asm keeps the offset from being added to the base outside the
// loop: the load then takes the base as a scalar pair and the offset as one
// register, where 19 hoisted 64-bit addresses would fill 38 of the 128 there are.
template <class T>
__device__ __forceinline__ T* lane_ptr(T* base, unsigned bytes) {
  asm volatile("" : "+v"(bytes));
  return reinterpret_cast<T*>(reinterpret_cast<std::conditional_t<std::is_const<T>::value, const char, char>*>(base) + bytes);
}
template <class T>
__device__ __forceinline__ T lane_at(T* base, unsigned bytes) {
  return *lane_ptr(base, bytes);
}

template <class T, bool HALF>
__global__ void __launch_bounds__((TriShape<T, HALF>::NT))
    k_tri(const T* __restrict__ A, T* __restrict__ B, const T* __restrict__ C1,
          T* __restrict__ C2, const KParams p, const int zc) {
  using S = TriShape<T, HALF>;
  constexpr int D = 3, Q = q_of(3), TX = S::TX, TY = S::TY;
  constexpr int PX = TX + 4, PY = TY + 4, R1 = PX * PY, R2 = PX * (PY - 2);
  static_assert(R1 <= S::NT, "one thread per column");
  extern __shared__ __align__(16) unsigned char tri_lds[];
  T* P1 = reinterpret_cast<T*>(tri_lds);  // P1[slot * R1 + py * PX + px]
  T* P2 = P1 + 16 * R1;                   // the same less the first row
  // x_1-face values of two iterations: F[parity][((side * 3 + step) * 5 + slot) * PY + py]
  constexpr int SX = 2 * D - 1, FN = 2 * 3 * SX * PY;
  static_assert(FN <= S::NT, "one thread per x_1-face value");
  T* F = P2 + 16 * R2;
  const long long ps = p.pstride;
  const int n0 = p.n[0], n1 = p.n[1], n2 = p.n[2];
  const unsigned plane = static_cast<unsigned>(n0) * n1;
  int tx_, ty_, tz_;
  fuse_tile(p, TX, TY, tx_, ty_, tz_);
  const int x0 = tx_ * TX, y0 = ty_ * TY, zc0 = tz_ * zc;
  const int zend = min(zc0 + zc, n2);
  const int iters = zend - zc0 + 4;
  const bool w0 = p.bc[0] != 0, w1 = p.bc[1] != 0, w2 = p.bc[2] != 0;

  // the thread's column
  int px, py;
  tri_column<TX, PY>(threadIdx.x, px, py);
  int gx = x0 - 2 + px, gy = y0 - 2 + py;
  bool in1 = static_cast<int>(threadIdx.x) < R1;
  if (gx < 0 || gx >= n0) {
    in1 = in1 && !w0;
    gx = fuse_wrap(gx, n0);
  }
  if (gy < 0 || gy >= n1) {
    in1 = in1 && !w1;
    gy = fuse_wrap(gy, n1);
  }
  const bool in2 = in1 && px >= 1 && px <= TX + 2 && py >= 1 && py <= TY + 2;
  const bool own = px >= 2 && px <= TX + 1 && py >= 2 && py <= TY + 1 && x0 - 2 + px < n0 &&
                   y0 - 2 + py < n1;
  const bool in3 = in1 && own;
  const bool lo = w0 && gx == 0, hi = w0 && gx == n0 - 1;
  const bool ywall = w1 && (gy == 0 || gy == n1 - 1);
  const bool ynear = w1 && (gy == 1 || gy == n1 - 2);
  // byte offsets within a plane: the column, and the upwind columns x - cx, y - cy
  constexpr unsigned sz = sizeof(T);
  const unsigned xc = gx * sz, yc = static_cast<unsigned>(gy) * n0 * sz, node2 = xc + yc;
  const unsigned xm = (gx == 0 ? n0 - 1 : gx - 1) * sz, xp = (gx == n0 - 1 ? 0 : gx + 1) * sz;
  const unsigned ym = static_cast<unsigned>(gy == 0 ? n1 - 1 : gy - 1) * n0 * sz;
  const unsigned yp = static_cast<unsigned>(gy == n1 - 1 ? 0 : gy + 1) * n0 * sz;
  const int pos = py * PX + px;

  auto wrap_z = [&](int z) { return fuse_wrap(z, n2); };
  // The x_1-face values that iteration i uses: step 1's for plane zc0 - 2 + i, those
  // of steps 2 and 3 for the planes they complete (full-way) or absorb
  // (half-way), one value per thread.  They are loaded two iterations ahead and go
  // to F one iteration ahead: read by the face columns themselves when they are
  // needed, their latency came twice per plane (6.49 against 5.61 ms per 512^3
  // float32 launch without walls).
  const int fe = static_cast<int>(threadIdx.x);
  const int fside = fe / (3 * SX * PY), fstep = fe / (SX * PY) % 3, fslot = fe / PY % SX;
  const bool fhere = w0 && fe < FN && (fside == 0 ? x0 - 2 <= 0 : x0 + TX + 1 >= n0 - 1);
  int fgy = y0 - 2 + fe % PY;
  fgy = w1 ? min(max(fgy, 0), n1 - 1) : fuse_wrap(fgy, n1);
  int fk = 0, fkb = 0;
  static_for<0, SX>([&](auto Sl) {
    constexpr int sl = decltype(Sl)::value;
    constexpr int kl = face_pop(D, 1, sl), kh = face_pop(D, -1, sl);
    if (fslot == sl) {
      fk = fside ? kh : kl;
      fkb = fside ? opp_index(D, kh) : opp_index(D, kl);
    }
  });
  const T* fsrc = (fstep == 0 ? A : (fstep == 1 ? C1 : B)) + (fk * ps + p.xoff + fgy);
  T fx = T(0), fsb = T(0);
  auto face_load = [&](int i) {
    if (!fhere) return;
    int z = zc0 - 2 + i - (HALF ? (fstep == 2 ? 1 : 0) : fstep);
    z = w2 ? min(max(z, 0), n2 - 1) : wrap_z(z);
    fx = fsrc[static_cast<long long>(z) * n1];
    if constexpr (HALF) {
      // step 1's unknowns less the node's own opposite population
      if (fstep == 0)
        fsb = A[fkb * ps + static_cast<long long>(z) * plane + static_cast<long long>(fgy) * n0 +
                (fside ? n0 - 1 : 0)];
    }
  };
  auto face_put = [&](int i) {
    if (fhere) F[(i & 1) * FN + fe] = HALF && fstep == 0 ? fx - fsb : fx;
  };
  // value of slot sl for this column's face in step s of iteration i
  auto face_at = [&](int i, int s, int sl) {
    return F[(i & 1) * FN + (((hi ? 1 : 0) * 3 + s) * SX + sl) * PY + py];
  };
  // the 19 values step 1 of plane z starts from
  // Every thread loads, from a wrapped column and plane where it owns none, and
  // wall rows are loaded when they are used: a branch around the loads may join
  // their registers and wait for them there.  Float32 with half-way walls takes
  // the branch (S::AHEAD: its registers do join without a wait, and the wall rows
  // come ahead; 2350 against 2550 us per 512^3 step).
  auto load = [&](int z, T (&g)[Q]) {
    const int zw = z < 0 || z >= n2 ? wrap_z(z) : z;
    if constexpr (S::AHEAD) {
      if ((w2 && zw != z) || !in1) return;
      if (ywall || (w2 && (zw == 0 || zw == n2 - 1))) {
        const T* c = C1 + static_cast<long long>(zw) * plane;
#pragma unroll
        for (int k = 0; k < Q; ++k) g[k] = lane_at(c + k * ps, node2);
        return;
      }
    }
    const int zm = zw == 0 ? n2 - 1 : zw - 1, zq = zw == n2 - 1 ? 0 : zw + 1;
    static_for<0, Q>([&](auto K) {
      constexpr int k = decltype(K)::value;
      constexpr Vec4i c = vel_vec(D, k);
      const int zk = c.v[2] == 1 ? zm : (c.v[2] == -1 ? zq : zw);
      const T* a = A + (k * ps + static_cast<long long>(zk) * plane);
      const unsigned off = (c.v[1] == 1 ? ym : (c.v[1] == -1 ? yp : yc)) +
                           (c.v[0] == 1 ? xm : (c.v[0] == -1 ? xp : xc));
      g[k] = lane_at(a, off);
    });
  };
  // the values of a wall row from a scratch state, waited for here (at the join
  // with the updated rows the wait would fall on those too)
  auto load_wall = [&](const T* c, T (&g)[Q]) {
#pragma unroll
    for (int k = 0; k < Q; ++k) g[k] = lane_at(c + k * ps, node2);
#pragma unroll
    for (int k = 0; k < Q; ++k) asm volatile("" : "+v"(g[k]));
  };

  // waiting values of steps 2 and 3 (index by population): up / up2 for the next
  // two planes, mid for the next one
  T up[2][5] = {}, up2[2][5] = {}, mid[2][9] = {};
  T over[HALF ? 2 : 1] = {};  // half-way: the entering c_3 = -1 value of the next plane
  T g[Q] = {}, next[Q] = {};
  load(zc0 - 2, next);
  face_load(0);
  face_put(0);
  face_load(1);
#pragma unroll
  for (int k = 0; k < Q; ++k) asm volatile("" : "+v"(next[k]));
  asm volatile("" : "+v"(fx), "+v"(fsb));
  if (w0) __syncthreads();
  // value of population k at (column - c_k) in the plane of the step below
  auto pulled = [&](auto K, auto Rc, const T* P) -> T {
    constexpr int k = decltype(K)::value, R = decltype(Rc)::value;
    constexpr Vec4i c = vel_vec(D, k);
    return P[tri_slot(k) * R + pos - c.v[1] * PX - c.v[0]];
  };
  // Step s + 2 from plane zeta of the step below (its own-column values rest, +z
  // and -z in o): complete gives its pulled values for plane zeta - 1; absorb_own
  // and absorb keep those of plane zeta that complete later planes (absorb after
  // the values of zeta - 1 are used up, to bound the registers).
  auto complete = [&](auto Sx, auto Rc, const T* P, const T (&o)[3], const int it, T (&f)[Q]) {
    constexpr int s = decltype(Sx)::value;
    static_for<0, Q>([&](auto K) {
      constexpr int k = decltype(K)::value;
      constexpr int cz = vel_comp(3, k, 2), i = cz_index(k);
      if constexpr (cz == 1) f[k] = up[s][i];
      else if constexpr (cz == 0) f[k] = mid[s][i];
      else if constexpr (tri_slot(k) < 0) f[k] = o[2];
      else f[k] = pulled(K, Rc, P);
    });
    if constexpr (!HALF) {
      if (lo || hi) {
        static_for<0, SX>([&](auto Sl) {
          constexpr int sl = decltype(Sl)::value;
          const T v = face_at(it, s + 1, sl);
          constexpr int kl = face_pop(D, 1, sl), kh = face_pop(D, -1, sl);
          f[kl] = lo ? v : f[kl];
          f[kh] = lo ? f[kh] : v;
        });
      }
    } else {
      static_for<0, Q>([&](auto K) {
        constexpr int k = decltype(K)::value;
        constexpr int cx = vel_comp(3, k, 0), cz = vel_comp(3, k, 2);
        if constexpr (cz == -1 && cx != 0) f[k] = (cx == 1 ? lo : hi) ? over[s] : f[k];
      });
    }
  };
  auto absorb_own = [&](auto Sx, const T (&o)[3]) {
    constexpr int s = decltype(Sx)::value;
    up[s][cz_index(3)] = up2[s][cz_index(3)];
    up2[s][cz_index(3)] = o[1];
    mid[s][cz_index(0)] = o[0];
  };
  auto absorb = [&](auto Sx, auto Rc, const T* P, const int it) {
    constexpr int s = decltype(Sx)::value, R = decltype(Rc)::value;
    asm volatile("" ::: "memory");
    static_for<0, Q>([&](auto K) {
      constexpr int k = decltype(K)::value;
      constexpr int cz = vel_comp(3, k, 2), i = cz_index(k);
      if constexpr (tri_slot(k) >= 0) {
        if constexpr (cz == 1) {
          up[s][i] = up2[s][i];
          up2[s][i] = pulled(K, Rc, P);
        } else if constexpr (cz == 0) {
          mid[s][i] = pulled(K, Rc, P);
        }
      }
    });
    if constexpr (HALF) {
      if (lo || hi) {
        // what enters the absorbed plane through the x_1 faces: the data minus
        // the node's own value of the opposite population, at hand now
        static_for<0, SX>([&](auto Sl) {
          constexpr int sl = decltype(Sl)::value;
          constexpr int kl = face_pop(D, 1, sl), kh = face_pop(D, -1, sl);
          const T sb =
              P[(lo ? tri_slot(opp_index(D, kl)) : tri_slot(opp_index(D, kh))) * R + pos];
          const T v = face_at(it, s + 1, sl) - sb;
          auto put = [&](auto K, bool here) {
            constexpr int k = decltype(K)::value;
            constexpr int cz = vel_comp(3, k, 2), i = cz_index(k);
            if constexpr (cz == 1) up[s][i] = here ? v : up[s][i];
            else if constexpr (cz == 0) mid[s][i] = here ? v : mid[s][i];
            else over[s] = here ? v : over[s];
          };
          put(std::integral_constant<int, kl>{}, lo);
          put(std::integral_constant<int, kh>{}, !lo);
        });
      }
    }
  };
  auto put_plane = [&](T* P, auto Rc, const T (&f)[Q]) {
    constexpr int R = decltype(Rc)::value;
    static_for<0, Q>([&](auto K) {
      constexpr int k = decltype(K)::value;
      if constexpr (tri_slot(k) >= 0) P[tri_slot(k) * R + pos] = f[k];
    });
  };

  for (int it = 0; it < iters; ++it) {
    const int zp = zc0 - 2 + it;  // plane of step 1
    const int z1 = (zp < 0 || zp >= n2) && !w2 ? wrap_z(zp) : zp;
    const bool zin = z1 >= 0 && z1 < n2;
    // ---- step 1
    T o1[3] = {};
    {
#pragma unroll
      for (int k = 0; k < Q; ++k) g[k] = next[k];
      if (in1 && zin) {
        const bool rowwall = ywall || (w2 && (z1 == 0 || z1 == n2 - 1));
        if (rowwall) {
          if constexpr (!S::AHEAD) load_wall(C1 + static_cast<long long>(z1) * plane, g);
        } else {
          if (lo || hi)
            static_for<0, SX>([&](auto Sl) {
              constexpr int sl = decltype(Sl)::value;
              const T v = face_at(it, 0, sl);
              constexpr int kl = face_pop(D, 1, sl), kh = face_pop(D, -1, sl);
              g[kl] = lo ? v : g[kl];
              g[kh] = lo ? g[kh] : v;
            });
          collide_vals<D, T>(g, p);
        }
        put_plane(P1, std::integral_constant<int, R1>{}, g);
      }
      o1[0] = g[0];
      o1[1] = g[3];
      o1[2] = g[6];
    }
    __syncthreads();
    face_put(it + 1);
    face_load(it + 2);
    // ---- step 2 on plane zp - 1
    T o2[3] = {};
    T h[Q] = {};
    if (in2) {
      complete(std::integral_constant<int, 0>{}, std::integral_constant<int, R1>{}, P1, o1, it, h);
      absorb_own(std::integral_constant<int, 0>{}, o1);
      const int zq = zp - 1;
      const int z2 = (zq < 0 || zq >= n2) && !w2 ? wrap_z(zq) : zq;
      if (z2 >= 0 && z2 < n2) {
        const bool zwall = w2 && (z2 == 0 || z2 == n2 - 1);
        T* c = C2 + static_cast<long long>(z2) * plane;
        if (ywall || zwall) {
          load_wall(c, h);
        } else {
          collide_vals<D, T>(h, p);
          const bool near = ynear || (w2 && (z2 == 1 || z2 == n2 - 2));
          if (near && own && zq >= zc0 && zq < zend) {
            // (keeps the allocator from moving the registers of the plane in flight
            // across this branch: 5.78 against 6.07 ms per 512^3 float32 launch)
            if constexpr (!S::AHEAD) {
#pragma unroll
              for (int k = 0; k < Q; ++k) asm volatile("" : "+v"(next[k]));
            }
#pragma unroll
            for (int k = 0; k < Q; ++k)
              __builtin_nontemporal_store(h[k], lane_ptr(c + k * ps, node2));
          }
        }
        put_plane(P2 - PX, std::integral_constant<int, R2>{}, h);
      }
      o2[0] = h[0];
      o2[1] = h[3];
      o2[2] = h[6];
      absorb(std::integral_constant<int, 0>{}, std::integral_constant<int, R1>{}, P1, it);
    }
    // the next source plane, in flight through step 3
    load(zp + 1, next);
    __syncthreads();
    // ---- step 3 on plane zp - 2
    T f[Q] = {};
    const int z3 = zp - 2;
    const bool store = in3 && it >= 4 && !ywall && !(w2 && (z3 == 0 || z3 == n2 - 1));
    if (in3) {
      complete(std::integral_constant<int, 1>{}, std::integral_constant<int, R2>{}, P2 - PX, o2,
               it, f);
      if (store) collide_vals<D, T>(f, p);
    }
    // The loads in flight are waited for here, before the stores are issued: the
    // vector-memory counter of this chip covers stores too, so a wait at the loop
    // head would last until they had reached memory (6.24 against 5.59 ms per 512^3
    // float32 launch).
#pragma unroll
    for (int k = 0; k < Q; ++k) asm volatile("" : "+v"(next[k]));
    if (store) {
      T* b = B + static_cast<long long>(z3) * plane;
#pragma unroll
      for (int k = 0; k < Q; ++k) __builtin_nontemporal_store(f[k], lane_ptr(b + k * ps, node2));
    }
    if (in3) {
      absorb_own(std::integral_constant<int, 1>{}, o2);
      absorb(std::integral_constant<int, 1>{}, std::integral_constant<int, R2>{}, P2 - PX, it);
    }
  }
}

}  // namespace lbm
