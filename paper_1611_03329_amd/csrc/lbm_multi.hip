// lbm_multi.hip -- launches of the kernels that take several steps per launch.
#include "multi.hpp"

#include <algorithm>
#include <cmath>

#include "brick.hpp"
#include "lbm.h"
#include "march.hpp"

namespace lbm {

template <class S>
static S store_of(const StateRegions& r) {
  S s;
  s.mf = static_cast<typename S::MoveF*>(r.mf);
  s.mg = static_cast<typename S::MoveG*>(r.mg);
  s.rs = static_cast<typename S::Rest*>(r.rs);
  s.r0 = static_cast<typename S::MoveF*>(r.r0);
  return s;
}

static int cuts(int n, int b) { return (n + b - 1) / b; }

// Local box of brick b with `layers` around it along the axes it does not span.
static int local_nodes(const int dim[3], const int b[3], int layers) {
  int e = 1;
  for (int a = 0; a < 3; ++a) e *= b[a] + (b[a] < dim[a] ? 2 * layers : 0);
  return e;
}

// Estimated time (us) of a two-step pass: launch and first touch, then per
// filling of the CUs (a block's LDS limits how many share one) a fixed part and
// one that grows with the wavefronts W of step 1 on a CU, and the traffic of
// all local nodes (rows of x that are no multiple of 8 nodes cost more).  Fitted
// to sweeps of bricks on 8^3 to 64^3 boxes, which it meets to
// about 10 %.
static double brick_pass_us(int prec, int nx, long long blocks, int local, int share, int ncu) {
  const long long per_cu = (blocks + ncu - 1) / ncu;
  const long long rounds = (per_cu + share - 1) / share;
  const double W = (double)std::min<long long>(share, per_cu) * ((local + 63) / 64);
  const double all = (double)blocks * local / 131072.0;
  if (prec == LBM_FP64) return 1.2 + rounds * (4.0 + 0.4 * W) + 2.5 * all;
  const bool rows = nx % 8 == 0;
  if (rounds > 1 || W > 12.0)
    return (rows ? 1.0 : 1.2) * (1.5 + rounds * (6.4 + 0.62 * std::max(0.0, W - 12.0)));
  return 5.5 + 0.2 * W + (rows ? 1.0 : 3.0) * all;
}

// Bricks of the two-step pass, chosen by that estimate where it is 10 % below
// two single steps (s0 + s1 nodes each).  Bricks that span x read and write
// whole rows; others pay 1.2x, with short rows 1.5x.  Measured per step (us),
// two-step passes against k_step: FP64 8^3 3.7 / 5.0, 16x12x10 3.9 / 5.0, 24^3 5.3 /
// 6.5, 32^3 5.7 / 8.6, 40^3 8.4 / 12.3, 100x20x20 6.4 / 8.4, but 48^3 12.2 / 11.2 and 64^3
// 25 / 20 at best; FP32 16x12x10 3.4 / 4.0, 32^3 4.0 / 5.5, 40^3 6.5 / 7.7, but 28^3 4.7 /
// 5.0, 100x20x20 5.9 / 5.7, 64^3 13.8 / 10.7; FP16 16x12x10 3.7 / 4.3, 32^3 4.1 / 5.2, but
// 36^3 5.7 / 5.6.  Above the node limits the layers' redundant work costs more
// than the launches saved, or the estimate no longer tells.
BrickShape brick_shape(const int dim[3], int prec, int ncu) {
  const bool fp64 = prec == LBM_FP64, fp16 = prec == LBM_FP16_STORAGE;
  const long long nodes = (long long)dim[0] * dim[1] * dim[2];
  BrickShape best;
  if (nodes > (fp64 ? 90000 : (fp16 ? 40000 : 70000))) return best;
  const double single = fp64 ? 4.7 + 1.1e-4 * nodes : (fp16 ? 4.0 + 3.5e-5 * nodes : 3.7 + 5.5e-5 * nodes);
  double least = 0.9 * single;
  for (int kx = 1; kx <= 16 && (kx == 1 || cuts(dim[0], kx) >= 4); ++kx)
    for (int by = 1; by <= 8; ++by)
      for (int bz = 1; bz <= 8; ++bz) {
        // equal bricks along each axis
        const int b[3] = {cuts(dim[0], kx), cuts(dim[1], cuts(dim[1], by)), cuts(dim[2], cuts(dim[2], bz))};
        const int e = local_nodes(dim, b, 1);
        if (e > 768) continue;
        const int threads = e <= 256 ? 256 : (e <= 512 ? 512 : 768);
        const int share = fp64 ? (threads == 256 ? 3 : 1) : (threads == 256 ? 6 : (threads == 512 ? 3 : 2));
        const long long blocks = (long long)cuts(dim[0], b[0]) * cuts(dim[1], b[1]) * cuts(dim[2], b[2]);
        double t = 0.5 * brick_pass_us(prec, dim[0], blocks, e, share, ncu);
        if (b[0] < dim[0]) t *= b[0] >= (fp64 ? 12 : 24) ? 1.2 : 1.5;
        if (t < least) {
          least = t;
          for (int a = 0; a < 3; ++a) best.b[a] = b[a];
          best.threads = threads;
          best.steps = 2;
        }
      }
  return best;
}

// The same for enthalpy lattices, whose node takes a fraction of the work, so
// that more steps per pass pay: step = 4.5 / T + rounds (c0 + c1 L / 1024) + reads
// of all local nodes at 4.5 TB/s / T, L the local nodes of the blocks that share
// a CU, against s0 + s1 nodes of k_step_enthalpy.  Measured per step (us, 200
// steps; the single step's launch floor differs by 1 us between boxes): 400x6x6
// FP64 1.5 / 2.9-3.8, FP32 1.1 / 2.7-3.9, 1000x6x5 1.6 / 3.3-4.1 and 1.2 / 3.0-3.6, 640x8x8
// 2.5 / 3.2-4.0 and 1.8 / 3.1-3.8, 120x16x15 3.0 / 3.3-4.0 and 2.4 / 2.8-3.8, but 158x21x20
// (66k nodes) 4.3 / 4.2-4.8 and 4.0 / 3.4-4.1, 100x36x36 7.1 / 5.8-6.1 and 5.5 / 4.1-4.8:
// hence the node limit.
BrickShape brick_shape_enthalpy(const int dim[3], int prec, int ncu) {
  const bool fp64 = prec == LBM_FP64;
  const long long nodes = (long long)dim[0] * dim[1] * dim[2];
  BrickShape best;
  if (nodes > 60000) return best;
  const double c0 = fp64 ? 0.35 : 0.3, c1 = fp64 ? 0.9 : 0.45;
  double least = 0.93 * (fp64 ? 2.9 + 2.3e-5 * nodes : 2.65 + 1.15e-5 * nodes);
  const int edges[] = {1, 2, 3, 4, 6, 8, 12, 16, 24, 32, 48, 64, 0};  // 0: the whole axis
  for (int T : {2, 3, 4, 6, 8, 12}) {
    // edge b along axis a and the local edge around it; 0 where it does not fit:
    // a brick that does not span its axis needs T - 1 layers of other nodes
    auto local = [&](int a, int want, int& b) {
      b = want == 0 ? dim[a] : want;
      if (want == 0) return b;
      return b < dim[a] && T - 1 <= dim[a] ? b + 2 * (T - 1) : 0;
    };
    int b[3];
    for (int ex : edges) {
      const int e0 = local(0, ex, b[0]);
      if (e0 == 0 || e0 > 1024) continue;
      for (int ey : edges) {
        const int e1 = local(1, ey, b[1]);
        if (e1 == 0 || e1 > 1024 / e0) continue;
        for (int ez : edges) {
          const int e2 = local(2, ez, b[2]);
          if (e2 == 0 || e2 > 1024 / (e0 * e1)) continue;
          const int e = e0 * e1 * e2;
          const int threads = e <= 256 ? 256 : (e <= 512 ? 512 : 1024);
          const int share = (fp64 ? 1 : 2) * (1024 / threads);
          const long long blocks = (long long)cuts(dim[0], b[0]) * cuts(dim[1], b[1]) * cuts(dim[2], b[2]);
          const long long per_cu = (blocks + ncu - 1) / ncu;
          const long long rounds = (per_cu + share - 1) / share;
          const double local_nodes = (double)std::min<long long>(share, per_cu) * e;
          double t = 4.5 / T + rounds * (c0 + c1 * local_nodes / 1024.0) +
                     (double)blocks * e * (fp64 ? 56.0 : 28.0) / 4.5e6 / T;
          if (rounds > 1) t *= fp64 ? 1.15 : 1.35;
          if (b[0] < dim[0] && b[0] < 8) t *= 1.1;  // short rows
          if (t < least) {
            least = t;
            for (int a = 0; a < 3; ++a) best.b[a] = b[a];
            best.threads = threads;
            best.steps = T;
          }
        }
      }
    }
  }
  return best;
}

static BrickGrid brick_grid(const int dim[3], const BrickShape& s, int layers) {
  BrickGrid g;
  for (int a = 0; a < 3; ++a) {
    g.b[a] = s.b[a];
    g.halo[a] = s.b[a] < dim[a] ? layers : 0;
    g.e[a] = s.b[a] + 2 * g.halo[a];
  }
  g.inv_b0 = 1.0f / (float)g.b[0];
  g.inv_b01 = 1.0f / (float)(g.b[0] * g.b[1]);
  g.inv_e0 = 1.0f / (float)g.e[0];
  g.inv_e01 = 1.0f / (float)(g.e[0] * g.e[1]);
  return g;
}

template <class Lat, class S, class C, int NT>
static void launch_brick2_nt(const void* params, const int dim[3], const BrickShape& s, const StateRegions& src,
                             const StateRegions& dst, uint32_t* clk, int slot, void* macro1,
                             void* macro2, hipStream_t stream) {
  const dim3 grid((dim[0] + s.b[0] - 1) / s.b[0], (dim[1] + s.b[1] - 1) / s.b[1], (dim[2] + s.b[2] - 1) / s.b[2]);
  hipLaunchKernelGGL((k_brick2<Lat, S, C, NT>), grid, dim3(NT), 0, stream, static_cast<const KParams<C>*>(params), store_of<S>(src), store_of<S>(dst),
                     brick_grid(dim, s, 1), clk, slot, static_cast<C*>(macro1), static_cast<C*>(macro2));
}

template <class Lat, class S, class C>
static void launch_brick2_of(const void* params, const int dim[3], const BrickShape& s, const StateRegions& src,
                             const StateRegions& dst, uint32_t* clk, int slot, void* macro1,
                             void* macro2, hipStream_t stream) {
  if (s.threads == 256) launch_brick2_nt<Lat, S, C, 256>(params, dim, s, src, dst, clk, slot, macro1, macro2, stream);
  else if (s.threads == 512) launch_brick2_nt<Lat, S, C, 512>(params, dim, s, src, dst, clk, slot, macro1, macro2, stream);
  else launch_brick2_nt<Lat, S, C, 768>(params, dim, s, src, dst, clk, slot, macro1, macro2, stream);
}

void launch_brick2(int q, int prec, const void* params, const int dim[3], const BrickShape& shape,
                   const StateRegions& src, const StateRegions& dst, uint32_t* clk, int slot, void* macro1,
                             void* macro2, hipStream_t stream) {
  using S64 = Store<double, double, double>;
  using S32 = Store<float, float, float>;
  using S16 = Store<_Float16, float, float>;
  if (q == 19) {
    if (prec == LBM_FP64) launch_brick2_of<D3Q19, S64, double>(params, dim, shape, src, dst, clk, slot, macro1, macro2, stream);
    else if (prec == LBM_FP32) launch_brick2_of<D3Q19, S32, float>(params, dim, shape, src, dst, clk, slot, macro1, macro2, stream);
    else launch_brick2_of<D3Q19, S16, float>(params, dim, shape, src, dst, clk, slot, macro1, macro2, stream);
  } else {
    if (prec == LBM_FP64) launch_brick2_of<D3Q15, S64, double>(params, dim, shape, src, dst, clk, slot, macro1, macro2, stream);
    else if (prec == LBM_FP32) launch_brick2_of<D3Q15, S32, float>(params, dim, shape, src, dst, clk, slot, macro1, macro2, stream);
    else launch_brick2_of<D3Q15, S16, float>(params, dim, shape, src, dst, clk, slot, macro1, macro2, stream);
  }
}

template <class C>
static void launch_compare_of(const void* params, int nodes, const void* snap, const void* cur, double* part,
                              uint32_t* done, double* res, double* host, hipStream_t stream) {
  hipLaunchKernelGGL((k_compare<C>), dim3((nodes + 255) / 256), dim3(256), 0, stream,
                     static_cast<const KParams<C>*>(params), static_cast<const C*>(snap), static_cast<const C*>(cur),
                     part, done, res, host);
}

void launch_compare(int prec, const void* params, int nodes, const void* snap, const void* cur, double* part,
                    uint32_t* done, double* res, double* host, hipStream_t stream) {
  if (prec == LBM_FP64) launch_compare_of<double>(params, nodes, snap, cur, part, done, res, host, stream);
  else launch_compare_of<float>(params, nodes, snap, cur, part, done, res, host, stream);
}

template <class C, int NT>
static void launch_brick_enthalpy_nt(const KParams<C>& kp, const EnthalpyConsts<C>& ec, const BrickShape& s, int steps,
                                     const StateRegions& src, const StateRegions& dst, hipStream_t stream) {
  using S = Store<C, C, C>;
  const int dim[3] = {kp.nx, kp.ny, kp.nz};
  const dim3 grid((dim[0] + s.b[0] - 1) / s.b[0], (dim[1] + s.b[1] - 1) / s.b[1], (dim[2] + s.b[2] - 1) / s.b[2]);
  hipLaunchKernelGGL((k_brick_enthalpy<S, C, NT>), grid, dim3(NT), 0, stream, kp, ec, store_of<S>(src),
                     store_of<S>(dst), brick_grid(dim, s, steps - 1), steps);
}

template <class C>
static void launch_brick_enthalpy_of(const KParams<C>& kp, const EnthalpyConsts<C>& ec, const BrickShape& s, int steps,
                                     const StateRegions& src, const StateRegions& dst, hipStream_t stream) {
  if (s.threads == 256) launch_brick_enthalpy_nt<C, 256>(kp, ec, s, steps, src, dst, stream);
  else if (s.threads == 512) launch_brick_enthalpy_nt<C, 512>(kp, ec, s, steps, src, dst, stream);
  else launch_brick_enthalpy_nt<C, 1024>(kp, ec, s, steps, src, dst, stream);
}

void launch_brick_enthalpy(const KParams<float>& kp, const EnthalpyConsts<float>& ec, const BrickShape& shape,
                           int steps, const StateRegions& src, const StateRegions& dst, hipStream_t stream) {
  launch_brick_enthalpy_of(kp, ec, shape, steps, src, dst, stream);
}
void launch_brick_enthalpy(const KParams<double>& kp, const EnthalpyConsts<double>& ec, const BrickShape& shape,
                           int steps, const StateRegions& src, const StateRegions& dst, hipStream_t stream) {
  launch_brick_enthalpy_of(kp, ec, shape, steps, src, dst, stream);
}

// Columns and the number of z ranges that finishes first when each CU takes one
// item at a time (a range of P planes costs P + 2: step 1 runs on a plane more
// at each end).
static long long march_cost(long long tiles, int nz, int chunks, int ncu) {
  return (tiles * chunks + ncu - 1) / ncu * (cuts(nz, chunks) + 3);
}
static MarchGrid march_grid(const int dim[3], int row, int rows, int ncu) {
  MarchGrid g;
  g.tiles_x = cuts(dim[0], row);
  g.tiles_y = cuts(dim[1], rows - 2);
  const long long tiles = (long long)g.tiles_x * g.tiles_y;
  g.chunks = 1;
  for (int k = 2; k <= dim[2] && k <= 64; ++k)
    if (march_cost(tiles, dim[2], k, ncu) < march_cost(tiles, dim[2], g.chunks, ncu)) g.chunks = k;
  g.items = (int)tiles * g.chunks;
  g.per_xcd = cuts(g.items, 8);
  return g;
}

// The variant of k_march2 an enthalpy lattice takes (0: none; 4: FP32 with four
// nodes per lane, FP64 with two, both with streaming stores; 2: two nodes per
// lane, cached stores).  A lane's vector needs x edges that it divides.
//
// States of 160 MB up, which with the other buffer stay out of the 256 MB last-level
// cache, run better with streaming stores, FP32 ones also in 1 KB rows of four
// nodes per lane if the rows are filled; cached FP32 ones in 512 B rows, of which
// the box makes more.  Measured (us per step, cached -> streaming stores): FP64 128^3
// (117 MB) 25 -> 29, 160x128x128 (147 MB) 44.2 -> 43.7, 200x128x128 (183 MB) 49.7 ->
// 46.9, 356x128x128 (327 MB) 83.1 -> 78.2, 1024x128x128 187 -> 178; FP32 256x128x128
// (117 MB) 23.6 -> 31.6, 2684x168x12 (152 MB) 49.6 -> 50.9, 378x128x123 (167 MB) 46.4 ->
// 44.6, and with four nodes per lane 480x128x100 (172 MB) 47.0 -> 43.3, 1024x128x128 107
// -> 99.
//
// A pass pays where its estimate is below that of two single steps.  An item's
// plane takes the same time however much of its row lies in the box, and less if
// fewer rows do; to that comes the traffic of the state.
// Fitted to 170 boxes of 2^18 to 1.7e7 nodes with edges from 1 to 10^5, which it meets to 6 %
// (rms); of 600 others that it takes, drawn at random, 4 % ran 2 to 9 % slower than single
// steps.  Measured per step (us, k_step_enthalpy / passes): FP64 128^3 35.1 / 23.4,
// 64^3 10.6 / 8.5, 1024x256x4 18.7 / 15.3, 130^3 36.8 / 37.6, 1024x2x512 18.8 / 20.7,
// 16x256x256 18.5 / 62, 2x512x512 10.6 / 223; FP32 128^3 19.5 / 14.8, 130^3 20.6 / 21.1,
// 1024x512x2 11.3 / 13.5, 2048x1x1024 20 / 57, 20x489x271 25 / 69.  FP32 below 2^20 nodes
// loses or is even (320x53x53 10.4 / 11.5).
constexpr long long kMarchStream = 160'000'000;

static double march_pass_us(const int dim[3], bool fp64, bool stream, double state_mb, int ncu) {
  const long long nodes = (long long)dim[0] * dim[1] * dim[2];
  if (dim[2] == 1) {  // one plane: items side by side, several per CU
    const double items = (double)cuts(dim[0], 2 * 64) * cuts(dim[1], kFlatRows - 2) * 256.0 / ncu;
    return fp64 ? 3.5 + 0.0145 * items : 4.0 + 0.0062 * items;
  }
  const int rows = fp64 || stream ? 11 : 15, live = std::min(dim[1] + 2, rows);
  const MarchGrid g = march_grid(dim, 64 * (!fp64 && stream ? 4 : 2), rows, ncu);
  const double cost = (double)march_cost((long long)g.tiles_x * g.tiles_y, dim[2], g.chunks, ncu);
  // us per plane of an item; us per node of traffic, more for stores that pass
  // through a last-level cache which does not hold both buffers
  double plane, node;
  if (fp64) {
    plane = stream ? 3.4 + 0.07 * live : 1.15 + 0.2 * live;
    node = stream ? 1.75e-5 : (state_mb < 128.0 ? 1.7e-5 : 2.5e-5);
  } else {
    plane = stream ? 4.6 : 1.3 + 0.107 * live;
    node = stream ? 0.8e-5 : (state_mb < 128.0 ? 0.65e-5 : 1.4e-5);
  }
  return std::hypot(plane * cost, node * (double)nodes);
}

int march_variant(const int dim[3], int prec, int ncu) {
  const bool fp64 = prec == LBM_FP64;
  const long long nodes = (long long)dim[0] * dim[1] * dim[2], state = nodes * 7 * (fp64 ? 8 : 4);
  if (nodes < (fp64 ? 1 << 18 : 1 << 20) || dim[0] % 2 != 0) return 0;
  const bool wide = dim[0] % 4 == 0 && 4 * dim[0] >= 3 * 256 * cuts(dim[0], 256);
  const bool stream = state >= kMarchStream && (fp64 || wide);
  const double step = fp64 ? std::max(9.2, 2.0 + 1.62e-5 * nodes) : 4.0 + 0.78e-5 * nodes;
  if (march_pass_us(dim, fp64, stream, state * 1e-6, ncu) >= 2.0 * step) return 0;
  return stream ? 4 : 2;
}

// Items beyond one per CU wait in the block that marches; without a march (FLAT)
// every item is a block, and several share a CU.
template <class C, int V, int R, bool STREAM, bool FLAT>
static void launch_march2_of(const KParams<C>& kp, const EnthalpyConsts<C>& ec, const StateRegions& src,
                             const StateRegions& dst, int ncu, hipStream_t stream) {
  const int dim[3] = {kp.nx, kp.ny, kp.nz};
  const MarchGrid g = march_grid(dim, 64 * V, R, ncu);
  const int per = FLAT ? g.per_xcd : std::min(g.per_xcd, std::max(1, ncu / 8));
  using S = Store<C, C, C>;
  hipLaunchKernelGGL((k_march2<C, V, R, STREAM, FLAT>), dim3(8 * per), dim3(march_threads(R)), 0, stream, kp, ec, store_of<S>(src),
                     store_of<S>(dst), g);
}

void launch_march2(const KParams<float>& kp, const EnthalpyConsts<float>& ec, const StateRegions& src,
                   const StateRegions& dst, int variant, int ncu, hipStream_t stream) {
  if (kp.nz == 1) launch_march2_of<float, 2, kFlatRows, false, true>(kp, ec, src, dst, ncu, stream);
  else if (variant == 4) launch_march2_of<float, 4, 11, true, false>(kp, ec, src, dst, ncu, stream);
  else launch_march2_of<float, 2, 15, false, false>(kp, ec, src, dst, ncu, stream);
}
void launch_march2(const KParams<double>& kp, const EnthalpyConsts<double>& ec, const StateRegions& src,
                   const StateRegions& dst, int variant, int ncu, hipStream_t stream) {
  if (kp.nz == 1) launch_march2_of<double, 2, kFlatRows, false, true>(kp, ec, src, dst, ncu, stream);
  else if (variant == 4) launch_march2_of<double, 2, 11, true, false>(kp, ec, src, dst, ncu, stream);
  else launch_march2_of<double, 2, 11, false, false>(kp, ec, src, dst, ncu, stream);
}

}  // namespace lbm
