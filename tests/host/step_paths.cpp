// The host side of lbm_step_ws without a GPU: this program defines the HIP runtime
// functions that liblbm.so calls (an executable's definitions come before those
// of the runtime library).  Device memory is host memory and launches are recorded
// instead of run; a pass of several steps counts itself up in the first word of
// the populations it writes.  One scenario per call, named in argv[1]; or "kernel" and a
// box, for the kernel that its passes take.
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

#include "lbm.h"
#include "shapes.hpp"

namespace {

std::map<const void*, std::string>& names() {
  static std::map<const void*, std::string> m;
  return m;
}
std::map<char*, size_t> g_device;         // device allocations
std::vector<std::string> g_launched;      // kernels of passes and checks, in order
int g_order = 0;                          // the tile order of the last step, field or totals launch
int g_fail_at = -1;                       // the launch of these that fails
hipError_t g_error = hipSuccess;          // what hipGetLastError returns next
uint32_t* g_home = nullptr;   // first word of the populations that the first pass read
uint32_t* g_clock = nullptr;  // FP16 step count that the first pass read
hipStreamCaptureStatus g_capture = hipStreamCaptureStatusNone;
struct Call { dim3 grid, block; size_t lds; hipStream_t stream; };
std::vector<Call> g_calls;

bool has(const std::string& s, const char* part) { return s.find(part) != std::string::npos; }

struct Regions { uint32_t *mf, *mg, *rs, *r0; };  // a kernel's Store argument

int g_failures = 0;
#define CHECK(cond, ...)                                                       \
  do {                                                                         \
    if (!(cond)) {                                                             \
      std::printf("%s:%d: %s: ", __FILE__, __LINE__, #cond);                   \
      std::printf(__VA_ARGS__);                                                \
      std::printf("\n");                                                       \
      ++g_failures;                                                            \
    }                                                                          \
  } while (0)

}  // namespace

extern "C" {
void** __hipRegisterFatBinary(const void*) { static void* module; return &module; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*,
                           int*) { names()[host] = name; }
void __hipRegisterVar(void**, void*, char*, const char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t stream) {
  g_calls.push_back({grid, block, lds, stream});
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* stream) {
  const Call c = g_calls.back();
  g_calls.pop_back();
  *grid = c.grid, *block = c.block, *lds = c.lds, *stream = c.stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* fn, dim3, dim3, void** args, size_t, hipStream_t) {
  const std::string& name = names()[fn];
  const bool brick = has(name, "k_brick2"), melt = has(name, "k_brick_enthalpy") || has(name, "k_march2");
  if (brick || melt || has(name, "k_compare")) {
    if ((int)g_launched.size() == g_fail_at) {
      g_launched.push_back("failed");
      return g_error = hipErrorLaunchFailure;
    }
    g_launched.push_back(name);
  } else if (has(name, "k_step")) {
    g_launched.push_back("step");
    if (!has(name, "enthalpy")) g_order = *static_cast<int*>(args[3]);
  } else if (has(name, "k_fields") || has(name, "k_totals")) {
    g_order = *static_cast<int*>(args[has(name, "k_fields") ? 9 : 3]);
  }
  if (brick || melt) {
    const Regions src = *static_cast<Regions*>(args[brick ? 1 : 2]), dst = *static_cast<Regions*>(args[brick ? 2 : 3]);
    if (!g_home) g_home = src.mg;
    dst.mg[0] = src.mg[0] + 1;
  }
  if (brick && has(name, "DF16_")) {
    uint32_t* const clk = *static_cast<uint32_t**>(args[4]);
    const int slot = *static_cast<int*>(args[5]);
    if (!g_clock) g_clock = clk + slot;
    clk[slot ^ 1] = clk[slot] + 2;
  }
  return hipSuccess;
}
hipError_t hipGetLastError() {
  const hipError_t e = g_error;
  g_error = hipSuccess;
  return e;
}
const char* hipGetErrorString(hipError_t) { return "an error"; }
hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { return *v = 256, hipSuccess; }
hipError_t hipMalloc(void** p, size_t n) {
  *p = std::aligned_alloc(256, (n + 255) / 256 * 256);
  std::memset(*p, 0, n);
  g_device[static_cast<char*>(*p)] = n;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  g_device.erase(static_cast<char*>(p));
  std::free(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return *p = std::calloc(1, n), hipSuccess; }
hipError_t hipHostFree(void* p) { return std::free(p), hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) { return std::memset(d, v, n), hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) { return *s = g_capture, hipSuccess; }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void* p) {
  for (const auto& [base, size] : g_device)
    if (p >= base && p < base + size) {
      std::memset(a, 0, sizeof *a);
      a->type = hipMemoryTypeDevice;
      a->devicePointer = const_cast<void*>(p);
      return hipSuccess;
    }
  return hipErrorInvalidValue;
}
}

namespace {

enum Kind { kFlow, kMelt, kMarch };

lbm_params params(Kind kind, int precision, int interval) {
  lbm_params p;
  lbm_default_params(&p);
  p.precision = precision;
  p.check_interval = interval;
  p.rayleigh = 1e4;
  p.nx = 16, p.ny = 12, p.nz = 10;
  if (kind != kFlow) {
    p.energy = LBM_ENERGY_ENTHALPY;
    p.nx = 400, p.ny = p.nz = 6;
  }
  if (kind == kMarch) p.nx = 256, p.ny = p.nz = 64;
  return p;
}

struct Run {
  lbm_lattice* h = nullptr;
  char* buf = nullptr;
  char* ws = nullptr;
  size_t ws_bytes = 0;
  explicit Run(const lbm_params& p) {
    size_t need = 0;
    CHECK(lbm_required_bytes(&p, &need) == LBM_OK, "%s", lbm_last_error());
    (void)hipMalloc((void**)&buf, need);
    ws_bytes = need + (size_t)p.nx * p.ny * p.nz * 64;  // more than any pass needs
    (void)hipMalloc((void**)&ws, ws_bytes);
    CHECK(lbm_create(&p, buf, need, reinterpret_cast<void*>(64), &h) == LBM_OK, "%s", lbm_last_error());
    g_launched.clear();
    g_home = g_clock = nullptr;
    g_fail_at = -1;
  }
  ~Run() {
    (void)lbm_destroy(h);
    (void)hipFree(buf);
    (void)hipFree(ws);
  }
  int64_t time() const {
    int64_t t = -1;
    (void)lbm_time(h, &t);
    return t;
  }
  size_t offered(int64_t n) const {
    size_t bytes = 1;
    CHECK(lbm_step_workspace(h, n, &bytes) == LBM_OK, "%s", lbm_last_error());
    return bytes;
  }
};

int passes() {
  int n = 0;
  for (const std::string& s : g_launched) n += has(s, "k_brick") || has(s, "k_march");
  return n;
}

// A captured call would tie its graph to the lent workspace: it takes single steps.
void capture() {
  for (Kind kind : {kFlow, kMelt, kMarch}) {
    Run r(params(kind, LBM_FP64, 0));
    const size_t before = r.offered(8);
    CHECK(before > 0 && before <= r.ws_bytes, "kind %d", kind);
    g_capture = hipStreamCaptureStatusActive;
    CHECK(r.offered(8) == 0, "kind %d", kind);
    CHECK(lbm_step_ws(r.h, 8, r.ws, before) == LBM_OK, "%s", lbm_last_error());
    g_capture = hipStreamCaptureStatusNone;
    CHECK(passes() == 0 && g_launched.size() == 8 && r.time() == 8, "kind %d: %d passes", kind, passes());
  }
}

// A workspace is offered exactly where the call then makes passes with it.
void offered() {
  for (Kind kind : {kFlow, kMelt, kMarch})
    for (int interval : {0, 1, 2, 3, 10})
      for (int parity : {0, 1})
        for (int n : {1, 3, 4, 5, 6, 7, 23}) {
          if (kind != kFlow && interval) continue;
          Run r(params(kind, LBM_FP64, interval));
          CHECK(lbm_step(r.h, parity) == LBM_OK, "%s", lbm_last_error());
          const size_t bytes = r.offered(n);
          CHECK(bytes <= r.ws_bytes, "%zu bytes", bytes);
          CHECK(lbm_step_ws(r.h, n, r.ws, r.ws_bytes) == LBM_OK, "%s", lbm_last_error());
          CHECK((bytes > 0) == (passes() > 0) && passes() % 2 == 0, "kind %d check %d parity %d: %zu bytes, %d passes for %d steps",
                kind, interval, parity, bytes, passes(), n);
          CHECK(r.time() == parity + n, "%d steps", n);
          // a workspace that no pass would use is not looked at
          if (!bytes) CHECK(lbm_step_ws(r.h, 1, r.ws + 16, r.ws_bytes - 16) == LBM_OK, "%s", lbm_last_error());
        }
}

// A launch that fails leaves the lattice with the steps it counts: the populations of
// the last pass in its own buffer (wherever that pass wrote them), its FP16 clock too.
void failed() {
  for (Kind kind : {kFlow, kMelt, kMarch})
    for (int precision : {(int)LBM_FP64, (int)LBM_FP16_STORAGE})
      for (int interval : {0, 4}) {
        if (kind != kFlow && (interval || precision != LBM_FP64)) continue;
        Run all(params(kind, precision, interval));
        CHECK(lbm_step_ws(all.h, 40, all.ws, all.ws_bytes) == LBM_OK, "%s", lbm_last_error());
        const std::vector<std::string> launches = g_launched;
        for (int at = 0; at < (int)launches.size(); ++at) {
          if (launches[at] == "step") continue;
          Run r(params(kind, precision, interval));
          g_fail_at = at;
          CHECK(lbm_step_ws(r.h, 40, r.ws, r.ws_bytes) == LBM_ERR_DEVICE, "launch %d", at);
          const uint32_t done = (uint32_t)passes();
          if (done) CHECK(*g_home == done, "kind %d launch %d: %u passes in the buffer of %u", kind, at, *g_home, done);
          if (kind == kFlow) CHECK(r.time() == 2 * done, "%u passes", done);
          if (done && precision == LBM_FP16_STORAGE) CHECK(*g_clock == 2 * done, "clock %u after %u passes", *g_clock, done);
          int64_t check = 0;
          double res = 0;
          (void)lbm_residual(r.h, &res, &check);
          CHECK(check < r.time(), "check at %lld", (long long)check);
        }
      }
}

struct Box { int dim[3], q, precision; bool general; };
lbm_params box_params(const Box& b) {
  lbm_params p;
  lbm_default_params(&p);
  p.nx = b.dim[0], p.ny = b.dim[1], p.nz = b.dim[2];
  p.lattice = b.q;
  p.precision = b.precision;
  p.rayleigh = 1e4;
  if (b.general) p.face[5].u_wall[0] = 0.01;
  return p;
}

// Tile order of steps: ranges per XCD (8) for states that the last-level cache serves,
// but not where they were slower.
void step_order() {
  const struct { Box box; int even, odd; } cases[] = {
      {{{103, 103, 103}, 19, LBM_FP32, false}, 8, 8},         {{{125, 125, 125}, 19, LBM_FP16_STORAGE, false}, 8, 8},
      {{{155, 155, 155}, 19, LBM_FP32, false}, 8, 8},         {{{160, 160, 168}, 15, LBM_FP32, false}, 0, 0},
      {{{128, 128, 100}, 19, LBM_FP16_STORAGE, true}, 0, 0},  {{{170, 170, 170}, 19, LBM_FP16_STORAGE, false}, 0, 0},
      {{{128, 128, 100}, 19, LBM_FP32, true}, 8, 8},          {{{64, 64, 64}, 15, LBM_FP64, true}, 0, 0},
      {{{80, 80, 80}, 19, LBM_FP16_STORAGE, false}, 0, 0},    {{{1036, 152, 25}, 19, LBM_FP32, false}, 0, 0},
      {{{168, 168, 168}, 19, LBM_FP32, false}, 0, -32},
  };
  for (const auto& c : cases) {
    Run r(box_params(c.box));
    const int* d = c.box.dim;
    CHECK(lbm_step(r.h, 1) == LBM_OK && g_order == c.even, "even %d x %d x %d: %d", d[0], d[1], d[2], g_order);
    CHECK(lbm_step(r.h, 1) == LBM_OK && g_order == c.odd, "odd %d x %d x %d: %d", d[0], d[1], d[2], g_order);
  }
}

// Tile order of queries: by the state and the outputs of the call together.
void query_order() {
  const struct { Box box; int all, one, totals; } cases[] = {
      {{{103, 103, 103}, 19, LBM_FP32, false}, 8, 8, 8},         {{{103, 103, 103}, 19, LBM_FP64, false}, 0, 0, 8},
      {{{125, 125, 125}, 19, LBM_FP16_STORAGE, true}, 8, 8, 8},  {{{126, 126, 126}, 19, LBM_FP32, false}, 0, 8, 8},
      {{{140, 140, 140}, 15, LBM_FP32, false}, 0, 0, 0},         {{{64, 64, 64}, 15, LBM_FP32, false}, 0, 0, 0},
  };
  for (const auto& c : cases) {
    Run r(box_params(c.box));
    const int* d = c.box.dim;
    void* out = nullptr;
    (void)hipMalloc(&out, (size_t)d[0] * d[1] * d[2] * 8);
    double* const o = static_cast<double*>(out);
    CHECK(lbm_fields(r.h, o, o, o, o, o) == LBM_OK && g_order == c.all, "fields %d^3: %d", d[0], g_order);
    CHECK(lbm_fields(r.h, 0, 0, 0, 0, o) == LBM_OK && g_order == c.one, "T %d^3: %d", d[0], g_order);
    CHECK(lbm_fields_noalloc(r.h, 0, 0, 0, 0, o) == LBM_OK && g_order == c.one, "T %d^3: %d", d[0], g_order);
    CHECK(lbm_totals(r.h, nullptr, nullptr) == LBM_OK && g_order == c.totals, "totals %d^3: %d", d[0], g_order);
    (void)hipFree(out);
  }
}

// Marching passes: not where a row fills few lanes or a block few rows, where they
// took up to 20 times the single steps.
void marching() {
  struct { int dim[3], fp64, fp32; } const boxes[] = {
      {{128, 128, 128}, 2, 2},   {{1024, 128, 128}, 4, 4},  {{1024, 8, 128}, 2, 2}, {{4096, 257, 1}, 2, 2},
      {{640, 640, 1}, 2, 0},     {{356, 128, 128}, 4, 2},   {{258, 55, 75}, 2, 2},  {{2, 512, 512}, 0, 0},
      {{4, 400, 400}, 0, 0},     {{16, 256, 256}, 0, 0},    {{36, 240, 449}, 0, 0}, {{1024, 2, 512}, 0, 0},
      {{2048, 1, 1024}, 0, 0},   {{138, 580, 58}, 0, 0},    {{2, 800000, 1}, 0, 0}, {{1000000, 1, 1}, 0, 0},
      {{100000, 4, 4}, 0, 0},    {{129, 128, 128}, 0, 0},   {{60, 60, 60}, 0, 0}};
  for (const auto& b : boxes) {
    const int v[2] = {lbm::march_variant(b.dim, LBM_FP64, 256), lbm::march_variant(b.dim, LBM_FP32, 256)};
    CHECK(v[0] == b.fp64 && v[1] == b.fp32, "%d x %d x %d: %d %d", b.dim[0], b.dim[1], b.dim[2], v[0], v[1]);
  }
}

}  // namespace

int main(int argc, char** argv) {
  if (argc == 7 && std::string(argv[1]) == "kernel") {  // table precision nx ny nz
    const int prec = std::atoi(argv[3]), dim[3] = {std::atoi(argv[4]), std::atoi(argv[5]), std::atoi(argv[6])};
    const std::string table = argv[2];
    const int kernel = table == "FLOW"   ? lbm::brick_shape(dim, prec, 256).threads
                       : table == "MELT" ? lbm::brick_shape_enthalpy(dim, prec, 256).threads
                                         : lbm::march_variant(dim, prec, 256);
    std::printf("%d\n", kernel);
    return 0;
  }
  const std::map<std::string, void (*)()> scenarios = {{"capture", capture}, {"offered", offered}, {"failed", failed}, {"marching", marching},
                                                         {"step_order", step_order}, {"query_order", query_order}};
  const auto it = argc == 2 ? scenarios.find(argv[1]) : scenarios.end();
  if (it == scenarios.end()) return 2;
  it->second();
  return g_failures ? 1 : 0;
}
