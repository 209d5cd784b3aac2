// The host side of the scene upload and of the solve's launch (wob.hip: validation,
// records, trees, guide, launch shapes) on the CPU, under sanitizers: the HIP runtime
// below keeps "device" memory on the heap, checks that every copy lies inside an
// allocation, launches nothing, and can refuse an allocation.  Prints "ok", or the
// first violation.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <random>
#include <vector>

#include "../../include/wob.h"
#include "../../paper_2305_04403_amd/csrc/internal.hpp"

static std::map<char*, size_t> on_device, on_host;
static int asked = 0, refuse = -1;  // allocations so far, and which to refuse
static size_t last_size = 0;
static hipError_t last = hipSuccess;
static struct {
  dim3 grid, block;
  size_t lds;
  hipStream_t stream;
} config;
static int launches = 0;

static hipError_t set(hipError_t e) {
  if (e != hipSuccess) last = e;
  return e;
}
static void fail(const char* what) {
  std::printf("%s\n", what);
  std::exit(1);
}
static bool inside(const void* p, size_t n) {
  for (const auto& a : on_device)
    if ((const char*)p >= a.first && (const char*)p + n <= a.first + a.second) return true;
  return false;
}

extern "C" {
hipError_t hipMalloc(void** p, size_t n) {
  last_size = n;
  if (asked++ == refuse) return set(hipErrorOutOfMemory);
  // 256-byte aligned, as the device's
  *p = std::aligned_alloc(256, (n + 255) / 256 * 256);
  on_device[(char*)*p] = n;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  if (on_device.erase((char*)p) != 1) fail("hipFree of what hipMalloc did not give");
  std::free(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  *p = std::aligned_alloc(256, (n + 255) / 256 * 256);
  on_host[(char*)*p] = n;
  return hipSuccess;
}
hipError_t hipHostFree(void* p) {
  if (on_host.erase((char*)p) != 1) fail("hipHostFree of what hipHostMalloc did not give");
  std::free(p);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* to, const void* from, size_t n, hipMemcpyKind kind, hipStream_t) {
  if (kind == hipMemcpyHostToDevice && !inside(to, n)) fail("copy past an allocation");
  std::memcpy(to, from, n);
  return hipSuccess;
}
hipError_t hipMemsetAsync(void* p, int v, size_t n, hipStream_t) {
  if (!inside(p, n)) fail("fill past an allocation");
  std::memset(p, v, n);
  return hipSuccess;
}
hipError_t hipGetLastError(void) {
  const hipError_t e = last;
  last = hipSuccess;
  return e;
}
hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { return *v = 256, hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t) { return ++launches, hipSuccess; }
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t st) {
  config = {g, b, lds, st};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* lds, hipStream_t* st) {
  *g = config.grid, *b = config.block, *lds = config.lds, *st = config.stream;
  return hipSuccess;
}
void** __hipRegisterFatBinary(const void*) { return nullptr; }
void __hipRegisterFunction(void**, const void*, char*, const char*, unsigned, void*, void*, void*, void*, int*) {}
void __hipUnregisterFatBinary(void**) {}
wob_status wob_mlp_forward(wob_mlp, const float*, int64_t, float*, void*) { return WOB_E_DEVICE; }
}
namespace wobi {
OrderLayout order_layout(int, int, int64_t) { return OrderLayout{}; }
wob_status order_points(int, int, const OrderLayout&, void*, const void*, const int32_t*, int64_t, void*, OrderBuffers*) {
  return WOB_E_DEVICE;
}
wob_status scatter_results(int, const OrderBuffers&, int64_t, void*, void*, void*) { return WOB_E_DEVICE; }
}  // namespace wobi

// A strip of n random primitives (2D: segments; 3D: triangles).
static void mesh(int dim, int n, std::vector<double>& v, std::vector<int32_t>& p) {
  std::mt19937_64 rng(n * 10 + dim);
  std::uniform_real_distribution<double> u(-1.0, 1.0);
  v.resize((size_t)(n + dim - 1) * dim);
  for (double& x : v) x = u(rng);
  p.resize((size_t)n * dim);
  for (int i = 0; i < n; ++i)
    for (int c = 0; c < dim; ++c) p[(size_t)i * dim + c] = i + c;
}

static wob_scene build(int dim, int precision, int n, wob_status* s, bool dirichlet = false) {
  std::vector<double> v;
  std::vector<int32_t> p;
  mesh(dim, n, v, p);
  std::vector<uint8_t> kind(n);
  std::vector<double> alpha(n, 0.5);
  for (int i = 0; i < n; ++i) kind[i] = (uint8_t)(dirichlet ? 0 : i % 3);
  wob_scene sc = nullptr;
  *s = wob_build_bvh(dim, precision, v.data(), (int64_t)v.size() / dim, p.data(), n, kind.data(), alpha.data(), &sc);
  return sc;
}

// Dynamic LDS of a double-layer solve beyond what its stacks take.
static long extra_lds(wob_scene sc, int64_t points, int paths) {
  std::vector<double> buffer(points * 3);
  wob_bc bc;
  std::memset(&bc, 0, sizeof(bc));
  bc.domain = 1;
  bc.formulation = WOB_F_DOUBLE_LAYER;
  if (wob_solve(sc, buffer.data(), nullptr, points, &bc, paths, 4, 0, buffer.data(), nullptr, nullptr) != WOB_OK)
    fail("a solve was refused");
  return (long)config.lds - (long)wob::walk_lds_bytes(sc->stack_cap, (int)config.block.x);
}

// Fewer wavefronts for the double layer: large FP32 scenes of triangles and several
// paths per lane alone.
static void check_lds() {
  struct { int dim, precision, n; int64_t points; int paths; bool more; } const cases[] = {
      {3, WOB_F32, 165000, 100000, 256, true}, {3, WOB_F32, 165000, 100000, 128, false},
      {3, WOB_F32, 165000, 100000, 16, false}, {3, WOB_F32, 125000, 100000, 512, true},
      {3, WOB_F32, 125000, 100000, 256, false}, {3, WOB_F32, 110000, 100000, 512, false},
      {2, WOB_F32, 165000, 100000, 256, false}, {3, WOB_F64, 165000, 100000, 256, false}};
  for (const auto& c : cases) {
    wob_status s;
    wob_scene sc = build(c.dim, c.precision, c.n, &s, true);
    if (s != WOB_OK) fail("a scene was refused");
    if ((extra_lds(sc, c.points, c.paths) > 0) != c.more) {
      std::printf("%dD precision %d, %d primitives, %d paths: ", c.dim, c.precision, c.n, c.paths);
      fail("LDS beyond the stacks");
    }
    wob_free(sc);
  }
}

int main() {
  check_lds();
  for (int dim = 2; dim <= 3; ++dim)
    for (int precision : {WOB_F32, WOB_F64})
      for (int n : {1, 2, 3, 5, 64, 1000, 40001, 60000}) {
        wob_status s;
        asked = 0;
        wob_scene sc = build(dim, precision, n, &s);
        if (s != WOB_OK || last != hipSuccess) fail("a scene was refused");
        wob_scene_info info;
        wob_get_scene_info(sc, &info);
        size_t held = 0;
        for (const auto& a : on_device) held += a.second;
        if ((size_t)info.device_bytes != held) fail("device_bytes is not what the scene holds");
        wob_free(sc);
        if (!on_device.empty() || !on_host.empty()) fail("memory left by a scene");

        // no device memory for the RIS candidates: the scene has them on the host
        const size_t per = precision == WOB_F32 ? 64 : 128;
        if (last_size != per * n) fail("the candidates' table is not the last allocation");
        refuse = asked - 1;
        asked = 0;
        sc = build(dim, precision, n, &s);
        refuse = -1;
        if (s != WOB_OK) fail("a scene without room for its candidates was refused");
        if (hipGetLastError() != hipSuccess) fail("the refused allocation is left as an error");
        if (on_host.size() != 1 || on_host.begin()->second != per * n) fail("no candidates on the host");
        wob_get_scene_info(sc, &info);
        if ((size_t)info.device_bytes != held - per * n) fail("device_bytes counts host memory");
        wob_free(sc);
        if (!on_device.empty() || !on_host.empty()) fail("memory left by a scene with candidates on the host");
      }
  std::printf("ok\n");
}
