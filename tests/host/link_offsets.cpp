// The kernels' link offsets (kernels.hpp link_at, link_base) on the host: for nodes of
// small and of the largest boxes, every link of each lattice has to lead to the element
// that link and the tiled slots give.
#include <cstdio>
#include <random>

#include "kernels.hpp"

extern "C" {  // the host half of the header's kernels registers itself; nothing is launched
extern const char __hip_fatbin = 0;
void** __hipRegisterFatBinary(const void*) { static void* module; return &module; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void*, char*, const char*, unsigned, void*, void*, void*, void*, int*) {}
}

using namespace lbm;

static int failures = 0;

// Slots of region population i (from 1) of node n: flow, or temperature (D3Q7).
template <class L>
static uint64_t slot(int i, int n) {
  if constexpr (std::is_same<L, D3Q7>::value) return gslot(i, (uint32_t)n);
  else return fslot<L>(i, (uint32_t)n);
}

template <class L, int Q, class T>
static void check(const KParams<float>& kp, int n) {
  const int x = n % kp.nx, y = n / kp.nx % kp.ny, z = n / kp.nxy;
  const Nbr nb = make_nbr(kp, x, y, z);
  T* const region = reinterpret_cast<T*>(uintptr_t{1} << 40);
  const uint32_t own = (uint32_t)(slot<L>(1, n) * sizeof(T));
  static_for<1, Q>([&](auto I) {
    constexpr int i = decltype(I)::value, io = L::opp(i);
    static_for<0, 2>([&](auto D) {
      constexpr int sg = decltype(D)::value ? 1 : -1;
      int off;
      bool in, at_in;
      link<L::e(0, i), L::e(1, i), L::e(2, i), sg>(nb, off, in);
      const uint64_t want = in ? slot<L>(sg < 0 ? io : i, n + off) : slot<L>(sg < 0 ? i : io, n);
      const uint32_t at = link_at<(uint32_t)(Q - 1), L, i, sg, T>(nb, n, own, at_in);
      const uint64_t got = (uint64_t)(uintptr_t)(link_base<L, i>(region)) + at - (uint64_t)(uintptr_t)region;
      if (at_in != in || got != want * sizeof(T)) {
        if (++failures < 10)
          std::printf("D3Q%d box %dx%dx%d node %d population %d sign %d: %llu, not %llu\n", Q, kp.nx, kp.ny, kp.nz, n, i,
                      sg, (unsigned long long)got, (unsigned long long)(want * sizeof(T)));
      }
    });
  });
}

template <class L, int Q, class T>
static void box(int nx, int ny, int nz, int periodic) {
  if ((long long)nx * ny * nz * (Q - 1) * (long long)sizeof(T) >= (1LL << 32) - (1 << 20)) return;
  KParams<float> kp{};
  kp.nx = nx, kp.ny = ny, kp.nz = nz, kp.nxy = nx * ny, kp.n = nx * ny * nz;
  for (int a = 0; a < 3; ++a) kp.per[a] = (periodic >> a) & 1;
  std::mt19937 rng(nx * 31 + ny * 7 + nz + periodic);
  const int tile = (int)kTile;
  for (int n : {0, 1, nx - 1, nx, kp.nxy - 1, kp.nxy, tile - 1, tile, tile + 1, kp.n / 2, kp.n - tile, kp.n - 2, kp.n - 1})
    if (n >= 0 && n < kp.n) check<L, Q, T>(kp, n);
  for (int k = 0; k < 300; ++k) check<L, Q, T>(kp, (int)(rng() % (unsigned)kp.n));
}

template <class L, int Q>
static void lattice() {
  const int boxes[][3] = {{1, 1, 1},   {2, 1, 3},     {7, 5, 3},      {33, 47, 61},  {64, 64, 64},   {2048, 3, 2},
                          {100, 9, 8}, {125, 125, 9}, {256, 256, 96}, {306, 307, 301}, {480, 500, 493}, {380, 381, 379}};
  for (const auto& b : boxes)
    for (int periodic = 0; periodic < 8; ++periodic) {
      box<L, Q, _Float16>(b[0], b[1], b[2], periodic);
      box<L, Q, float>(b[0], b[1], b[2], periodic);
      box<L, Q, double>(b[0], b[1], b[2], periodic);
    }
}

int main() {
  lattice<D3Q19, 19>();
  lattice<D3Q15, 15>();
  lattice<D3Q7, 7>();
  return failures ? 1 : 0;
}
