// march.hpp -- two time steps per pass over a large enthalpy lattice.
//
// A step of a large enthalpy lattice streams its seven populations through HBM.
// k_march2 takes two steps per pass, from one buffer to another (both in the
// natural layout, kernels.hpp).  A block owns a column of 64 V x nodes by R - 2
// rows and marches along z: step 1 on plane c for its rows and one row on each
// side, step 2 on plane c - 1.  A wavefront is a row, a lane V neighbouring nodes
// (one vector access); what moves along x passes between
// lanes, along y through LDS, along z stays in registers.  The nodes just
// beyond both ends of the rows are computed by the block's last wavefront.
// Every node goes through the functions of k_step_enthalpy, so the states are
// bit for bit those of two single steps.
#pragma once

#include "enthalpy.hpp"

namespace lbm {

constexpr int march_threads(int rows) { return 64 * (rows + 1); }
// Rows of step 1 in a box of one plane.
constexpr int kFlatRows = 7;

// How a pass is cut: columns of tiles_x by tiles_y, each in `chunks` ranges of
// planes; every XCD takes a contiguous run of items.
struct MarchGrid {
  int tiles_x, tiles_y, chunks, items, per_xcd;
};

template <class C, int V>
__device__ __forceinline__ void march_load(const C* base, uint32_t e, C (&v)[V]) {
  typedef C Vec __attribute__((ext_vector_type(V)));
  const Vec x = *(const LBM_GLOBAL Vec*)((const LBM_GLOBAL char*)base + e * (uint32_t)sizeof(C));
#pragma unroll
  for (int j = 0; j < V; ++j) v[j] = x[j];
}
// STREAM: past the caches (states that do not stay in the last-level cache).
template <bool STREAM, class C, int V>
__device__ __forceinline__ void march_store(C* base, uint32_t e, const C (&v)[V]) {
  typedef C Vec __attribute__((ext_vector_type(V)));
  Vec x;
#pragma unroll
  for (int j = 0; j < V; ++j) x[j] = v[j];
  LBM_GLOBAL Vec* const to = (LBM_GLOBAL Vec*)((LBM_GLOBAL char*)base + e * (uint32_t)sizeof(C));
  if constexpr (STREAM) __builtin_nontemporal_store(x, to);
  else *to = x;
}

// V, R: nodes per lane and rows of step 1.  Registers bound them: with 16-byte
// vectors (V = 4 FP32, 2 FP64) and R = 11, three wavefronts per SIMD at 158-165
// registers; R = 15 would spill 35-53.  Measured (us per step at default load
// priority, cached stores): FP32 1024x128x128 V = 4 R = 11 109, V = 2 R = 15 113, V = 2
// R = 11 123, V = 4 R = 7 143, k_step_enthalpy 136; 1024x64x64 26.5, 25.9, 27.1, 36.3, 36.5;
// FP64 1024x128x128 V = 2 R = 11 194, V = 1 R = 15 221, k_step_enthalpy 302.  With load
// priority 106 / 25.0 / 187, with streaming stores too 100 / 33 / 178 (so only for
// states past the last-level cache; streaming loads lost 7-12 %).  What bounds it:
// 56 B (112 FP64) per node and pass, and again the rows that two columns read
// (R / (R - 2)), at the 5 TB/s that marching columns of 1 KB rows reach.
// FLAT: boxes of one plane, which is its own neighbour or lies between two walls.
// Marched like others it went through step 1 three times (us per step, 4096x257x1:
// FP64 18.8 single, 22.9 marched, 12.7 FLAT; FP32 12.3, 14.0, 7.6); without the march
// there is nothing to keep from plane to plane, so all items are launched at once,
// and of R = 7, 11 and 15 the smallest blocks do best or within 3 % (1024x1024x1 FP64
// 12.5, 14.4, 13.4, FP32 7.5, 7.7, 9.0).
template <class C, int V, int R, bool STREAM, bool FLAT>
__global__ void __launch_bounds__(march_threads(R)) k_march2(const KParams<C> kp, const EnthalpyConsts<C> ec,
                                                             const Store<C, C, C> src, const Store<C, C, C> dst,
                                                             const MarchGrid mg) {
  using S = Store<C, C, C>;
  constexpr int NX = 64 * V;
  __shared__ C ys[2][2][R][NX];   // populations 3 and 4 of each row after step 1
  __shared__ C ends[2][2][R];     // population 1 of the node before each row, 2 of the one after it
  const int lane = (int)threadIdx.x & 63, r = (int)threadIdx.x >> 6;
  const int stride = (int)gridDim.x / 8;
  const bool perx = kp.per[0], pery = kp.per[1], perz = kp.per[2];
  auto wall = [&](int f, C v) { return kp.heat_a[f] * v + kp.heat_b[f]; };
  int buf = 0;
  for (int it = (int)blockIdx.x / 8; it < mg.per_xcd; it += stride) {
    const int item = ((int)blockIdx.x & 7) * mg.per_xcd + it;
    if (item >= mg.items) break;
    const int tiles = mg.tiles_x * mg.tiles_y;
    const int chunk = item / tiles, tile = item % tiles;
    const int x0 = tile % mg.tiles_x * NX, y0 = tile / mg.tiles_x * (R - 2);
    const int z0 = (int)((long long)kp.nz * chunk / mg.chunks), z1 = (int)((long long)kp.nz * (chunk + 1) / mg.chunks);
    const int xn = min(x0 + NX, kp.nx);  // end of the rows
    // the row this thread works on: its wavefront's, or for the ends its lane's
    const bool ends_wave = r == R;
    const int row = ends_wave ? lane >> 1 : r;
    int y = y0 - 1 + row;
    const bool inner = !ends_wave && row >= 1 && row <= R - 2 && y < kp.ny;
    bool live = row < R && (pery ? y <= kp.ny : (y >= 0 && y < kp.ny));
    y = y < 0 ? kp.ny - 1 : (y >= kp.ny ? 0 : y);
    int x;
    if (ends_wave) {
      x = (lane & 1) ? xn : x0 - 1;
      live = live && (perx || (x >= 0 && x < kp.nx));
      x = x < 0 ? kp.nx - 1 : (x >= kp.nx ? 0 : x);
    } else {
      x = x0 + lane * V;
      live = live && x < kp.nx;
    }
    const int m = x + kp.nx * y;
    const bool first = x == x0, last = x + V == xn;  // ends of the row
    const int c0 = FLAT || (z0 == 0 && !perz) ? 0 : z0 - 1;

    C h[7][V];                      // plane c: loaded, then after step 1
    C RA[6][V], RB[6][V];           // populations 0 to 5 entering planes c - 1 and c, in turn
    C U[V];                         // population 5 of plane c after step 1
    auto load = [&](int c) {
      const int zc = c < 0 ? kp.nz - 1 : (c >= kp.nz ? 0 : c);
      const uint32_t n = (uint32_t)(zc * kp.nxy + m);
      if (ends_wave) {
        C g[7];
        const Nbr none{};
        gather_g<false, S, C>(kp, src, (int)n, none, g);
#pragma unroll
        for (int k = 0; k < 7; ++k) h[k][0] = g[k];
      } else {
        march_load(src.rs, g0slot<S>(n), h[0]);
        static_for<1, 7>([&](auto K) { march_load(src.mg, gslot(decltype(K)::value, n), h[decltype(K)::value]); });
      }
    };
    auto collide = [&](C (&a)[7][V], int j) {
      C g[7];
#pragma unroll
      for (int k = 0; k < 7; ++k) g[k] = a[k][j];
      collide_enthalpy<C>(ec, g);
#pragma unroll
      for (int k = 0; k < 7; ++k) a[k][j] = g[k];
    };
    if (live) load(c0);
    auto plane = [&](int c, C (&F)[6][V], C (&G)[6][V]) {
      const bool here = FLAT || perz || c < kp.nz, below = perz || c > 0;
      C f6[V];  // population 6 entering plane c - 1
      if (here) {
        if (live) {
          collide(h, 0);
          if (ends_wave) {
            ends[buf][lane & 1][row] = (lane & 1) ? h[2][0] : h[1][0];
          } else {
#pragma unroll
            for (int j = 1; j < V; ++j) collide(h, j);
#pragma unroll
            for (int j = 0; j < V; ++j) {
              ys[buf][0][r][lane * V + j] = h[3][j];
              ys[buf][1][r][lane * V + j] = h[4][j];
            }
          }
        }
        __syncthreads();
        const C left = __shfl_up(h[1][V - 1], 1), right = __shfl_down(h[2][0], 1);
        if (inner) {
          // population k entering a node that has no neighbour there: the wall rule on its own
          C before = left, after = right;
          if (first) before = (x > 0 || perx) ? ends[buf][0][r] : wall(0, h[2][0]);
          if (last) after = (xn < kp.nx || perx) ? ends[buf][1][r] : wall(1, h[1][V - 1]);
          const bool south = pery || y > 0, north = pery || y < kp.ny - 1;
#pragma unroll
          for (int j = 0; j < V; ++j) {
            G[0][j] = h[0][j];
            G[1][j] = j > 0 ? h[1][j > 0 ? j - 1 : 0] : before;
            G[2][j] = j < V - 1 ? h[2][j < V - 1 ? j + 1 : 0] : after;
            G[3][j] = south ? ys[buf][0][r - 1][lane * V + j] : wall(2, h[4][j]);
            G[4][j] = north ? ys[buf][1][r + 1][lane * V + j] : wall(3, h[3][j]);
            if constexpr (FLAT) {
              G[5][j] = perz ? h[5][j] : wall(4, h[6][j]);
              f6[j] = perz ? h[6][j] : wall(5, h[5][j]);
            } else {
              G[5][j] = below ? U[j] : wall(4, h[6][j]);
              f6[j] = h[6][j];
            }
          }
        }
#pragma unroll
        for (int j = 0; j < V; ++j) U[j] = h[5][j];
        buf ^= 1;
      } else {
#pragma unroll
        for (int j = 0; j < V; ++j) f6[j] = wall(5, U[j]);
      }
      // loads at raised wavefront priority: 3-4 % in every case measured
      __builtin_amdgcn_s_setprio(1);
      if (!FLAT && c < z1 && (perz || c + 1 < kp.nz) && live) load(c + 1);
      __builtin_amdgcn_s_setprio(0);
      // step 2 of plane c - 1 (every lane of an inner row: the shuffles need them)
      if ((FLAT || c > z0) && !ends_wave && r >= 1 && r <= R - 2) {
        C a[7][V];
#pragma unroll
        for (int j = 0; j < V; ++j) {
#pragma unroll
          for (int k = 0; k < 6; ++k) a[k][j] = F[k][j];
          a[6][j] = f6[j];
          collide(a, j);
        }
        const C left = __shfl_up(a[1][V - 1], 1), right = __shfl_down(a[2][0], 1);
        if (inner && live) {
          const int zn = FLAT ? 0 : c - 1;
          const uint32_t n = (uint32_t)(zn * kp.nxy + m);
          march_store<STREAM>(dst.rs, g0slot<S>(n), a[0]);
          // along z and y whole vectors move, or bounce into the opposite slot
          auto move = [&](int k, int ko, bool in, int off, int face) {
            if (in) {
              march_store<STREAM>(dst.mg, gslot(k, n + (uint32_t)off), a[k]);
            } else {
              C w[V];
#pragma unroll
              for (int j = 0; j < V; ++j) w[j] = wall(face, a[k][j]);
              march_store<STREAM>(dst.mg, gslot(ko, n), w);
            }
          };
          move(5, 6, perz || zn < kp.nz - 1, zn < kp.nz - 1 ? kp.nxy : -(kp.nz - 1) * kp.nxy, 5);
          move(6, 5, perz || zn > 0, zn > 0 ? -kp.nxy : (kp.nz - 1) * kp.nxy, 4);
          move(3, 4, pery || y < kp.ny - 1, y < kp.ny - 1 ? kp.nx : -(kp.ny - 1) * kp.nx, 3);
          move(4, 3, pery || y > 0, y > 0 ? -kp.nx : (kp.ny - 1) * kp.nx, 2);
          // along x the lane stores what its own nodes receive; what crosses the
          // end of the row goes to the next column's first or last node
          C w[V];
          const bool wall_lo = first && x == 0 && !perx, wall_hi = last && xn == kp.nx && !perx;
#pragma unroll
          for (int j = 0; j < V; ++j) w[j] = j > 0 ? a[1][j > 0 ? j - 1 : 0] : (wall_lo ? wall(0, a[2][0]) : left);
          if (!first || wall_lo) {
            march_store<STREAM>(dst.mg, gslot(1, n), w);
          } else {
#pragma unroll
            for (int j = 1; j < V; ++j) st_mg<S, C>(dst, gslot(1, n + (uint32_t)j), w[j]);
          }
          if (last && !wall_hi)
            st_mg<S, C>(dst, gslot(1, xn < kp.nx ? n + (uint32_t)V : n + (uint32_t)V - (uint32_t)kp.nx), a[1][V - 1]);
#pragma unroll
          for (int j = 0; j < V; ++j)
            w[j] = j < V - 1 ? a[2][j < V - 1 ? j + 1 : 0] : (wall_hi ? wall(1, a[1][V - 1]) : right);
          if (!last || wall_hi) {
            march_store<STREAM>(dst.mg, gslot(2, n), w);
          } else {
#pragma unroll
            for (int j = 0; j < V - 1; ++j) st_mg<S, C>(dst, gslot(2, n + (uint32_t)j), w[j]);
          }
          if (first && !wall_lo)
            st_mg<S, C>(dst, gslot(2, x > 0 ? n - 1u : n + (uint32_t)kp.nx - 1u), a[2][0]);
        }
      }
    };
    if constexpr (FLAT) {
      plane(0, RB, RB);
    } else {
      for (int c = c0;;) {
        plane(c, RA, RB);
        if (++c > z1) break;
        plane(c, RB, RA);
        if (++c > z1) break;
      }
    }
    __syncthreads();
  }
}

}  // namespace lbm
