// brick.hpp -- several time steps per launch for lattices whose steps are latency.
//
// A step of a small lattice takes 5-10 us of which the chip works a fraction:
// launch, parameter and first-touch latency, one wavefront's serial arithmetic.
// k_brick2 takes two steps per launch.  The box is cut into bricks; a block
// reads its brick and one layer of nodes around it at time t, computes step 1
// on all of them (the layer is computed by the neighbour bricks too), keeps the
// result in LDS and computes step 2 on the brick alone.  A brick reads nodes
// that other blocks own, so the pass goes from one buffer to another, both in
// the natural layout of even parity (kernels.hpp).  Step 1 stores and step 2
// reads exactly what an even and an odd k_step would, through the same
// functions, so the states are bit for bit those of two single steps.
#pragma once

#include "enthalpy.hpp"
#include "kernels.hpp"

namespace lbm {

// How a box is cut into bricks.
struct BrickGrid {
  int b[3];      // brick edges
  int e[3];      // edges with the layers around it (none along an axis the brick spans)
  int halo[3];   // layers on both sides along this axis
  float inv_b0, inv_b01, inv_e0, inv_e01;  // 1 / b0, 1 / (b0 b1), 1 / e0, 1 / (e0 e1)
};

// i / d for 0 <= i < 2^12, 1 <= d, given 1.0f / d: the half keeps the product
// off the integers by more than its rounding.
__device__ __forceinline__ int small_div(int i, float inv) { return (int)(((float)i + 0.5f) * inv); }

// Local coordinates of thread i in a box of edges d0, d1 (inverses given).
__device__ __forceinline__ void local_coords(int i, int d0, int d1, float inv0, float inv01, int (&c)[3]) {
  c[2] = small_div(i, inv01);
  const int r = i - c[2] * d0 * d1;
  c[1] = small_div(r, inv0);
  c[0] = r - c[1] * d0;
}

// Node of local position c (layer included) of the brick that starts at o:
// false where the position is no node of this pass.
template <class C>
__device__ __forceinline__ bool brick_node(const KParams<C>& kp, const BrickGrid& bg, const int (&o)[3],
                                           const int (&c)[3], int (&x)[3]) {
  const int dim[3] = {kp.nx, kp.ny, kp.nz};
  bool live = true;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    x[a] = o[a] + c[a] - bg.halo[a];
    if (kp.per[a]) {
      live = live && x[a] < dim[a] + bg.halo[a];
      x[a] += x[a] < 0 ? dim[a] : (x[a] >= dim[a] ? -dim[a] : 0);
    } else {
      live = live && x[a] >= 0 && x[a] < dim[a];
    }
  }
  return live;
}

// Offsets inside the block's local box to the neighbour at -1 / +1 along each
// axis; along an axis the brick spans the wrap stays inside.
__device__ __forceinline__ void local_nbr(const BrickGrid& bg, const int (&c)[3], int (&off)[3][2]) {
  const int str[3] = {1, bg.e[0], bg.e[0] * bg.e[1]};
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    off[a][0] = (c[a] > 0 ? -1 : bg.e[a] - 1) * str[a];
    off[a][1] = (c[a] < bg.e[a] - 1 ? 1 : 1 - bg.e[a]) * str[a];
  }
}

template <int EX, int EY, int EZ, int SG>
__device__ __forceinline__ int local_link(const int (&off)[3][2]) {
  int d = 0;
  if constexpr (EX != 0) d += off[0][EX * SG > 0 ? 1 : 0];
  if constexpr (EY != 0) d += off[1][EY * SG > 0 ? 1 : 0];
  if constexpr (EZ != 0) d += off[2][EZ * SG > 0 ? 1 : 0];
  return d;
}

// A second view of uniform parameters: the compiler reads them again instead of
// keeping more of them than the scalar registers hold across the block.
template <class T>
__device__ __forceinline__ const T* again(const T* p) {
  auto c = (const __attribute__((address_space(4))) T*)p;
  asm volatile("" : "+s"(c));
  return (const T*)c;
}

// Stores u and T of node n as a check step's snapshot does.
template <class C>
__device__ __forceinline__ void store_macro(const KParams<C>& kp, const Macro<C>& M, C* out, int n) {
  LBM_GLOBAL C* const o = gbl(out);
  o[n] = M.ux;
  o[n + kp.n] = M.uy;
  o[n + 2 * kp.n] = M.uz;
  o[n + 3 * kp.n] = M.T;
}

// clk, slot: the lattice's step count on the device (drives FP16 rounding), which
// this pass reads in one slot and leaves for the next in the other.  macro1,
// macro2: where u and T of the state before step 1 / step 2 go, or null.
template <class Lat, class S, class C, int NT>
__global__ void __launch_bounds__(NT) k_brick2(const KParams<C>* __restrict__ params, const S src, const S dst, const BrickGrid bg,
                                               uint32_t* clk, int slot, C* macro1, C* macro2) {
  using H = typename S::MoveF;
  constexpr int Q = Lat::Q;
  // state between the steps: flow populations as the step carries them, in
  // their storage type, and temperature populations
  __shared__ C lg[7][NT];
  __shared__ H lf[Q][NT];
  const int tid = (int)threadIdx.x;
  const int o[3] = {(int)blockIdx.x * bg.b[0], (int)blockIdx.y * bg.b[1], (int)blockIdx.z * bg.b[2]};
  uint32_t now = 0u;
  if constexpr (kStochastic<S>) {
    now = clk[slot];
    if ((blockIdx.x | blockIdx.y | blockIdx.z) == 0 && tid == 0) gbl(clk)[slot ^ 1] = now + 2u;
  }
  C h[Q], p[7];
  {
    const KParams<C>& kp = *again(params);
    int c[3], x[3];
    local_coords(tid, bg.e[0], bg.e[1], bg.inv_e0, bg.inv_e01, c);
    if (c[2] < bg.e[2] && brick_node(kp, bg, o, c, x)) {
      const int n = x[0] + kp.nx * (x[1] + kp.ny * x[2]);
      const Nbr nb{};
      gather<Lat, false, false, S, C, true>(kp, src, n, nb, h, p);
      const Pairs<Lat, C> P = make_pairs<Lat, C>(h);
      const Macro<C> M = macro<Lat, kFlowScale<S>, C>(kp, P, p);
      if (macro1) {
        bool mine = true;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          const int at = c[a] - bg.halo[a];
          mine = mine && at >= 0 && at < bg.b[a] && o[a] + at == x[a];
        }
        if (mine) store_macro(kp, M, macro1, n);
      }
      collide_flow<Lat, C>(kp, M, P, h);
      collide_heat<C>(kp, M, p);
      const uint32_t rnd = kStochastic<S> ? mix32(mix32(now) + (uint32_t)n) : 0u;
      static_for<0, Q>([&](auto I) {
        constexpr int i = decltype(I)::value;
        if constexpr (kStochastic<S>) lf[i][tid] = half_sr((float)h[i], (rnd + (uint32_t)i * 0x9E3779B9u) >> 19);
        else lf[i][tid] = h[i];
      });
      static_for<0, 7>([&](auto K) { lg[decltype(K)::value][tid] = p[decltype(K)::value]; });
    }
  }
  __syncthreads();
  const KParams<C>& kp = *again(params);
  int c[3], x[3];
  local_coords(tid, bg.b[0], bg.b[1], bg.inv_b0, bg.inv_b01, c);
  bool mine = c[2] < bg.b[2];
  const int dim[3] = {kp.nx, kp.ny, kp.nz};
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    x[a] = o[a] + c[a];
    mine = mine && x[a] < dim[a];
    c[a] += bg.halo[a];
  }
  if (!mine) return;
  const int n = x[0] + kp.nx * (x[1] + kp.ny * x[2]);
  const Nbr nb = make_nbr(kp, x[0], x[1], x[2]);
  int off[3][2];
  local_nbr(bg, c, off);
  const int q = c[0] + bg.e[0] * (c[1] + bg.e[1] * c[2]);
  h[0] = (C)lf[0][q];
  static_for<1, Q>([&](auto I) {
    constexpr int i = decltype(I)::value;
    int unused;
    bool in;
    link<Lat::e(0, i), Lat::e(1, i), Lat::e(2, i), -1>(nb, unused, in);
    const int d = local_link<Lat::e(0, i), Lat::e(1, i), Lat::e(2, i), -1>(off);
    h[i] = (C)(&lf[0][0])[in ? i * NT + q + d : Lat::opp(i) * NT + q];
  });
  p[0] = lg[0][q];
  static_for<1, 7>([&](auto K) {
    constexpr int k = decltype(K)::value;
    int unused;
    bool in;
    link<D3Q7::e(0, k), D3Q7::e(1, k), D3Q7::e(2, k), -1>(nb, unused, in);
    const int d = local_link<D3Q7::e(0, k), D3Q7::e(1, k), D3Q7::e(2, k), -1>(off);
    C v = (&lg[0][0])[in ? k * NT + q + d : D3Q7::opp(k) * NT + q];
    constexpr int fc = d3q7_face<k, -1>();
    v = in ? v : kp.heat_a[fc] * v + kp.heat_b[fc];
    p[k] = v;
  });
  const Pairs<Lat, C> P = make_pairs<Lat, C>(h);
  const Macro<C> M = macro<Lat, kFlowScale<S>, C>(kp, P, p);
  if (macro2) store_macro(kp, M, macro2, n);
  collide_flow<Lat, C>(kp, M, P, h);
  collide_heat<C>(kp, M, p);
  scatter<Lat, true, false, S, C, true, true>(kp, dst, n, nb, h, p, M, kStochastic<S> ? mix32(now + 1u) : 0u);
}

// The residual of a check whose step ran in a two-step pass: compares the stored
// u and T (cur) with the snapshot, in the blocks and the order of summation of a
// compare step of k_step and k_fold, in one launch.
template <class C>
__global__ void __launch_bounds__(kMaxBlock) k_compare(const KParams<C>* __restrict__ params,
                                                       const C* __restrict__ snap, const C* __restrict__ cur,
                                                       double* part, uint32_t* done, double* res, double* host) {
  const KParams<C>& kp = *again(params);
  const int n = blockIdx.x * blockDim.x + threadIdx.x, N = kp.n;
  double v[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
  if (n < N)
    residual_terms(kp, cur[n], cur[n + N], cur[n + 2 * N], cur[n + 3 * N], snap[n], snap[n + N], snap[n + 2 * N],
                   snap[n + 3 * N], v);
  block_reduce<5>(v, 1u << 4);
  if (threadIdx.x == 0) {
#pragma unroll
    for (int j = 0; j < 5; ++j) st_agent(part + (size_t)blockIdx.x * kPartStride + j, v[j]);
  }
  if (!last_block(done, gridDim.x)) return;
  // the groups of k_fold, one after another (boxes this small have one or two)
  double t[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
  for (int g = 0; g < (int)gridDim.x; g += (int)blockDim.x) {
    const int i = g + (int)threadIdx.x;
#pragma unroll
    for (int j = 0; j < 5; ++j) v[j] = i < (int)gridDim.x ? ld_agent(part + (size_t)i * kPartStride + j) : 0.0;
    __syncthreads();
    block_reduce<5>(v, 1u << 4);
    // the last stage gives each group to a thread of its own
    __shared__ double sums[5];
    if (threadIdx.x == 0) {
#pragma unroll
      for (int j = 0; j < 5; ++j) sums[j] = v[j];
    }
    __syncthreads();
    if ((int)threadIdx.x == g / (int)blockDim.x) {
#pragma unroll
      for (int j = 0; j < 5; ++j) t[j] = sums[j];
    }
  }
  __syncthreads();
  block_reduce<5>(t, 1u << 4);
  if (threadIdx.x == 0) {
    finish_residual(t, res);
#pragma unroll
    for (int j = 0; j < 8; ++j) host[j] = res[j];
  }
}

// T >= 2 steps per launch of an enthalpy lattice (k_step_enthalpy T times): a
// brick with T - 1 layers around it, one node a thread, its seven populations
// in LDS between steps.  After step s the outermost s layers hold nothing of
// use; the brick itself is exact after step T.
template <class S, class C, int NT>
__global__ void __launch_bounds__(NT) k_brick_enthalpy(const KParams<C> kp, const EnthalpyConsts<C> ec, const S src,
                                                       const S dst, const BrickGrid bg, int T) {
  __shared__ C lg[2][7][NT];
  const int tid = (int)threadIdx.x;
  const int o[3] = {(int)blockIdx.x * bg.b[0], (int)blockIdx.y * bg.b[1], (int)blockIdx.z * bg.b[2]};
  int c[3], x[3], off[3][2];
  local_coords(tid, bg.e[0], bg.e[1], bg.inv_e0, bg.inv_e01, c);
  const bool live = c[2] < bg.e[2] && brick_node(kp, bg, o, c, x);
  const int n = live ? x[0] + kp.nx * (x[1] + kp.ny * x[2]) : 0;
  const Nbr nb = make_nbr(kp, x[0], x[1], x[2]);
  local_nbr(bg, c, off);
  C g[7];
  if (live) {
    gather_g<false, S, C>(kp, src, n, nb, g);
    collide_enthalpy<C>(ec, g);
  }
  for (int s = 1; s < T; ++s) {
    C(&l)[7][NT] = lg[s & 1];
    if (live) static_for<1, 7>([&](auto K) { l[decltype(K)::value][tid] = g[decltype(K)::value]; });
    __syncthreads();
    if (live) {
      C v[7];
      static_for<1, 7>([&](auto K) {
        constexpr int k = decltype(K)::value, ko = D3Q7::opp(k);
        int unused;
        bool in;
        link<D3Q7::e(0, k), D3Q7::e(1, k), D3Q7::e(2, k), -1>(nb, unused, in);
        const int d = local_link<D3Q7::e(0, k), D3Q7::e(1, k), D3Q7::e(2, k), -1>(off);
        constexpr int fc = d3q7_face<k, -1>();
        const C r = (&l[0][0])[in ? k * NT + tid + d : ko * NT + tid];
        v[k] = in ? r : kp.heat_a[fc] * r + kp.heat_b[fc];
      });
      static_for<1, 7>([&](auto K) { g[decltype(K)::value] = v[decltype(K)::value]; });
      collide_enthalpy<C>(ec, g);
    }
  }
  bool mine = live;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const int dim[3] = {kp.nx, kp.ny, kp.nz};
    const int at = c[a] - bg.halo[a];
    mine = mine && at >= 0 && at < bg.b[a] && o[a] + at < dim[a];
  }
  if (mine) scatter_g<true, S, C>(kp, dst, n, nb, g);
}

}  // namespace lbm
