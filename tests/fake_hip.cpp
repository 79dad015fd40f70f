// A stand-in for the HIP runtime on the host: a program that defines the runtime's entry points itself and loads the
// library, so that the launch sequence of its calls can be followed without a GPU.  "Device" memory is host memory,
// no kernel runs; the scan of the bins reports the totals that a case asks for, and every launch, copy and wait is
// noted, so that a case can say what is still in flight on a stream when a call returns, which allocations a call
// made, and what a kernel was launched with.  Test infrastructure only.
//
// usage: fake_hip <libapc.so> <case> [arguments]   exit status 0: the case holds
#include <dlfcn.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <hip/hip_runtime_api.h>

#include <functional>
#include <map>
#include <string>
#include <vector>

#include "../include/apc.h"

namespace {

struct Launch {
  std::string name;
  uint64_t grid, block;
  std::vector<uint64_t> arg;  // the first 8 bytes of each argument a case looks at
};
std::vector<Launch> g_launches;
std::map<const void*, std::string> g_kernels;
std::map<void*, size_t> g_mem;
size_t g_fail_above = SIZE_MAX;  // device allocations of more bytes are refused
size_t g_refuse_from = 1, g_refuse_to = 0;  // the next so many device allocations of sizes between these are refused
int g_refusals = 0;
unsigned long long g_records = 0, g_pairs = 0;  // what the scan of the bins reports
uint64_t g_issued = 0, g_done = 0;              // work handed to the device, and waited for (one stream at a time)
bool g_captured = false;                        // the caller captures the stream
hipError_t g_last = hipSuccess;
struct Event {
  uint64_t at = 0;
};

bool in_flight() { return g_done < g_issued; }
size_t device_bytes() {
  size_t n = 0;
  for (auto& m : g_mem) n += m.second;
  return n;
}

}  // namespace

extern "C" {

void** __hipRegisterFatBinary(const void*) {
  static void* h = nullptr;
  return &h;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char* device, const char*, unsigned, void*, void*, void*, void*,
                           int*) {
  g_kernels[host] = device;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
struct Config {
  dim3 grid, block;
  size_t lds;
  hipStream_t s;
};
static thread_local Config g_config;
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t s) {
  g_config = {grid, block, lds, s};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* s) {
  *grid = g_config.grid;
  *block = g_config.block;
  *lds = g_config.lds;
  *s = g_config.s;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t, hipStream_t) {
  Launch l{g_kernels[f], uint64_t(grid.x) * grid.y * grid.z, uint64_t(block.x) * block.y * block.z, {}};
  // the runtime takes fewer than 2^32 threads in each dimension
  if (!l.grid || uint64_t(grid.x) * block.x >= (1ull << 32)) return g_last = hipErrorInvalidConfiguration;
  auto is = [&](const char* k) { return l.name.find(k) != std::string::npos; };
  if (is("k_bin_scan"))
    for (int k = 0; k < 8; ++k) l.arg.push_back(*static_cast<uint64_t*>(args[k]));
  if (is("k_bin_supers"))
    for (int k = 0; k < 3; ++k) l.arg.push_back(*static_cast<uint64_t*>(args[k]));
  if (is("k_pair_list"))
    for (int k = 0; k < 5; ++k) l.arg.push_back(*static_cast<uint64_t*>(args[k]));
  if (is("k_bin_scan") && l.arg[7]) {
    unsigned long long* totals = reinterpret_cast<unsigned long long*>(l.arg[7]);
    totals[0] = g_records;
    totals[1] = g_pairs;
  }
  if (is("k_adjacency")) {  // every face on the hull
    const int64_t n = *static_cast<int64_t*>(args[1]);
    memset(*static_cast<int**>(args[4]), 0xff, size_t(4 * n) * sizeof(int));
  }
  if (is("k_fill") && *static_cast<int*>(args[1]) == 0) {
    int* p = *static_cast<int**>(args[0]);
    const int64_t n = *static_cast<int64_t*>(args[2]);
    if (n < (1 << 20)) memset(p, 0, size_t(n) * sizeof(int));
  }
  g_launches.push_back(l);
  ++g_issued;
  return hipSuccess;
}

hipError_t hipMalloc(void** p, size_t n) {
  const bool refuse = g_refusals > 0 && n >= g_refuse_from && n <= g_refuse_to;
  if (refuse) --g_refusals;
  if (n > g_fail_above || refuse) {
    *p = nullptr;
    return hipErrorOutOfMemory;
  }
  *p = malloc(n);
  memset(*p, 0x5a, n < (1 << 20) ? n : (1 << 20));  // memory comes as somebody left it
  g_mem[*p] = n;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  g_mem.erase(p);
  free(p);
  g_done = g_issued;  // waits for the device
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  *p = calloc(1, n);
  return hipSuccess;
}
hipError_t hipHostFree(void* p) {
  free(p);
  return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
  memcpy(d, s, n);
  g_done = g_issued;
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  memcpy(d, s, n);
  ++g_issued;
  return hipSuccess;
}
hipError_t hipMemset(void* d, int v, size_t n) {
  memset(d, v, n);
  return hipSuccess;
}
hipError_t hipMemGetInfo(size_t* f, size_t* t) {
  *f = *t = size_t(256) << 30;
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void*) {
  static void* mem = calloc(1, size_t(64) << 20);
  *p = mem;
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) {
  *v = 256;
  return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) {
  *n = 4;
  return hipSuccess;
}
hipError_t hipDeviceSynchronize() {
  g_done = g_issued;
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) {
  g_done = g_issued;
  return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* st) {
  *st = g_captured ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) {
  *e = reinterpret_cast<hipEvent_t>(new Event);
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) {
  delete reinterpret_cast<Event*>(e);
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t) {
  reinterpret_cast<Event*>(e)->at = g_issued;
  return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e) {
  const uint64_t at = reinterpret_cast<Event*>(e)->at;
  g_done = at > g_done ? at : g_done;
  return hipSuccess;
}
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  *ms = 0.0f;
  return hipSuccess;
}
hipError_t hipGetDevice(int* d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDeviceCount(int* n) {
  *n = 1;
  return hipSuccess;
}
hipError_t hipGetLastError() {
  const hipError_t e = g_last;
  g_last = hipSuccess;
  return e;
}
const char* hipGetErrorString(hipError_t e) { return e == hipSuccess ? "no error" : "refused"; }

}  // extern "C"

// ------------------------------------------------------------------ cases

namespace {

void* g_lib;
template <class F>
F sym(const char* name) {
  void* p = dlsym(g_lib, name);
  if (!p) {
    printf("no %s\n", name);
    exit(3);
  }
  return reinterpret_cast<F>(p);
}
#define APC(fn) sym<decltype(&fn)>(#fn)

#define CHECK(x)                                                              \
  do {                                                                        \
    if (!(x)) {                                                               \
      printf("line %d: %s\n", __LINE__, #x);                                  \
      return 1;                                                               \
    }                                                                         \
  } while (0)

// `n_sub` subdomains of `tets_each` tets, seen from in front
struct Scene {
  apc_ctx ctx = nullptr;
  apc_mesh mesh = nullptr;
  std::vector<float> xyz, scalar;
  std::vector<int32_t> tet, of, subs;
  apc_tf tf = {};
  apc_mboit mb = {};
  std::vector<float> table;
  float *moments = reinterpret_cast<float*>(0x1000000), *rgba = reinterpret_cast<float*>(0x2000000);  // never read

  explicit Scene(int n_sub, int tets_each = 1) : table(8, 0.5f) {
    if (APC(apc_create)(0, &ctx) != APC_OK) exit(4);
    for (int k = 0; k < n_sub * tets_each; ++k) {
      const float p[4][3] = {{0, 0, 0}, {1, 0, 0}, {0, 1, 0}, {0, 0, 1}};
      for (int q = 0; q < 4; ++q) {
        for (int c = 0; c < 3; ++c) xyz.push_back(p[q][c] + (c == 2 ? 2.0f * float(k) : 0.0f));
        scalar.push_back(float(q));
        tet.push_back(4 * k + q);
      }
      of.push_back(k / tets_each);
    }
    for (int k = 0; k < n_sub; ++k) subs.push_back(k);
    load();
    tf.n_entries = 2;
    tf.rgba = table.data();
    tf.s_max = 3.0f;
    tf.kappa = 1.0f;
    tf.absorbance_max = 10.0f;
    mb.m = 8;
    mb.renormalize = 1;
    mb.alpha = 5e-5;
    mb.eta = 0.3;
    for (int j = 0; j < 8; ++j) mb.bias[j] = (j & 1) ? 1.0 / (j + 2) : 0.0;
  }
  void load() {
    apc_mesh_desc d = {};
    d.n_vertices = int64_t(scalar.size());
    d.n_tets = int64_t(of.size());
    d.n_subdomains = int(subs.size());
    d.xyz = xyz.data();
    d.scalar = scalar.data();
    d.tet_vertices = tet.data();
    d.tet_subdomain = of.data();
    if (APC(apc_load_mesh)(ctx, &d, &mesh, nullptr) != APC_OK) exit(5);
  }
  apc_view view(int w, int h) const {
    apc_view v = {};
    v.width = w;
    v.height = h;
    v.projection = APC_ORTHOGRAPHIC;
    v.eye[2] = -1.0;
    v.dir[2] = 1.0;
    v.right[0] = 1.0 / w;
    v.down[1] = 1.0 / h;
    v.step = 0.1;
    return v;
  }
  apc_status moments_pass(const apc_view& v, uint32_t flags, int m = 8) {
    return APC(apc_moments_pass)(ctx, mesh, &v, &tf, m, subs.data(), int(subs.size()), moments, flags, nullptr);
  }
  apc_status resolve(const apc_view& v, uint32_t flags) {
    return APC(apc_resolve_pass)(ctx, mesh, &v, &tf, &mb, moments, subs.data(), int(subs.size()), rgba, flags,
                                 nullptr);
  }
  apc_status tiles(const apc_view& v, float* tiles, int32_t* bins, int64_t cap, int64_t* n) {
    return APC(apc_moments_pass_pairs)(ctx, mesh, &v, &tf, 8, subs.data(), int(subs.size()), tiles, bins, cap, n,
                                       nullptr);
  }
};

// A call that returns an error, or only a count, leaves nothing of its own in flight: the fill of the bins (which
// starts before the host knows the totals) has ended, so its buffers -- the static workspace belongs to every
// context and stream of the device -- may serve another frame at once.
int refused_noalloc() {
  Scene s(2);
  g_records = uint64_t(64) << 20;  // more than the 64 MiB hold
  const apc_view v = s.view(64, 64);
  const apc_status st = APC(apc_resolve_pass_noalloc)(s.ctx, s.mesh, &v, &s.tf, &s.mb, s.moments, s.subs.data(), 2,
                                                      s.rgba, 0, nullptr);
  CHECK(st == APC_E_NOMEM);
  CHECK(!in_flight());
  return 0;
}

int refused_overflow() {
  Scene s(2);
  g_records = 10;
  g_pairs = 4;
  CHECK(s.moments_pass(s.view(64, 64), APC_MOMENTS_GLOBAL) == APC_OK);  // (the buffers exist now)
  hipDeviceSynchronize();
  g_records = uint64_t(1) << 31;
  CHECK(s.moments_pass(s.view(64, 56), APC_MOMENTS_GLOBAL) == APC_E_NUMERIC);
  CHECK(!in_flight());
  return 0;
}

int counted_pairs() {
  Scene s(2);
  g_records = 10;
  g_pairs = 4;
  int64_t n = -1;
  const apc_view v = s.view(64, 64);
  CHECK(s.tiles(v, nullptr, nullptr, 0, &n) == APC_OK && n == 4);
  CHECK(!in_flight());
  CHECK(s.tiles(s.view(64, 56), s.moments, reinterpret_cast<int32_t*>(s.rgba), 3, &n) == APC_E_NOMEM && n == 4);
  CHECK(!in_flight());
  return 0;
}

// A frame whose pair numbers cannot be had must not leave an older frame's bins claiming numbers that are gone: the
// older frame, asked for again, is numbered anew into the buffer that its pair list reads.
int lost_numbers() {
  Scene s(2);
  g_records = 10;
  g_pairs = 4;
  const apc_view small = s.view(64, 64);
  CHECK(s.resolve(small, APC_BY_PAIR) == APC_OK);
  g_fail_above = 64 << 10;
  CHECK(s.resolve(s.view(1024, 1024), APC_BY_PAIR) != APC_OK);  // 32768 bins: 128 KiB of numbers
  g_fail_above = SIZE_MAX;
  g_launches.clear();
  CHECK(s.resolve(small, APC_BY_PAIR) == APC_OK);
  uint64_t numbers = 0;
  for (const Launch& l : g_launches) {
    if (l.name.find("k_bin_scan") != std::string::npos) numbers = l.arg[6];
    if (l.name.find("k_pair_list") != std::string::npos) CHECK(numbers && l.arg[2] == numbers);
  }
  return 0;
}

// The buffers that only walking by pairs needs (its numbers, list and moments, in this order) may be refused: the
// frame is then walked per tile, in a launch of a workgroup per tile.
int refused_pair_buffers() {
  const size_t from[3] = {280 << 10, 78 << 10, 40 << 20}, to[3] = {370 << 10, 120 << 10, 100 << 20};
  for (int which = 0; which < 3; ++which) {  // 73728 bins, 20000 pairs: 288 KiB, 80 KiB, 44 MiB and their slack
    Scene s(8);
    g_records = 10;
    g_pairs = 20000;
    g_refuse_from = from[which];
    g_refuse_to = to[which];
    g_refusals = which == 2 ? 2 : 1;  // (the moments are asked for twice: with room and without)
    g_launches.clear();
    CHECK(s.moments_pass(s.view(768, 768), APC_MOMENTS_GLOBAL) == APC_OK);
    CHECK(g_refusals == 0);
    uint64_t walks = 0;
    for (const Launch& l : g_launches)
      if (l.name.find("k_moments") != std::string::npos) walks = l.grid;
    CHECK(walks == 9216);
  }
  return 0;
}

// Launches stay below 2^32 threads in each dimension however large the output: per-subdomain images of 17 GB, more
// pairs than such a launch holds, and sums of an image whose tiles are nearly empty.
int large_images() {
  Scene s(460);
  g_records = 10;
  g_pairs = 460;
  CHECK(s.moments_pass(s.view(1024, 1024), 0) == APC_OK);  // 460 x 9 x 2^20 values
  return 0;
}

int large_pair_lists() {
  Scene s(4200);
  g_records = 10;
  g_pairs = 16384ull * 4200;
  g_launches.clear();
  CHECK(s.moments_pass(s.view(1024, 1024), 0, 4) == APC_OK);
  uint64_t walks = 0;
  for (const Launch& l : g_launches)
    if (l.name.find("k_moments") != std::string::npos) walks = l.grid;
  CHECK(walks == 16384);
  return 0;
}

int thin_images() {
  Scene s(1);
  CHECK(APC(apc_sum_moment_tiles)(s.ctx, s.moments, reinterpret_cast<int32_t*>(s.rgba), 5, 1, 8, 1 << 27, 1, 64,
                                  s.moments, nullptr) == APC_OK);
  uint64_t blocks = 0;
  for (const Launch& l : g_launches)
    if (l.name.find("k_sum_tiles") != std::string::npos) blocks = l.grid * (l.block / 64);
  CHECK(blocks >= 1u << 27);
  return 0;
}

// The buffer of the pairs' moments: at most 256 MiB, twice what the first frame needs, never more than the bins of
// the frame can fill, and in place for a view with more pairs.
int moments_buffer() {
  auto largest = [] {
    size_t n = 0;
    for (auto& m : g_mem) n = m.second > n ? m.second : n;
    return n;
  };
  const size_t tile = 64 * 9 * sizeof(float);
  {
    Scene s(8);
    g_records = 10;
    g_pairs = (size_t(255) << 20) / tile;
    CHECK(s.moments_pass(s.view(1000, 1000), APC_MOMENTS_GLOBAL) == APC_OK);
    CHECK(largest() == size_t(256) << 20);
    APC(apc_destroy)(s.ctx);
  }
  Scene s(8);
  g_pairs = 4000;
  CHECK(s.moments_pass(s.view(512, 512), APC_MOMENTS_GLOBAL) == APC_OK);
  CHECK(largest() == 8000 * tile);
  g_pairs = 7900;
  const size_t held = device_bytes();
  CHECK(s.moments_pass(s.view(512, 504), APC_MOMENTS_GLOBAL) == APC_OK);
  CHECK(largest() == 8000 * tile && device_bytes() - held < (64 << 10));  // (the pairs' list)
  g_pairs = 512 * 504 / 64 * 8;  // every bin
  CHECK(s.moments_pass(s.view(504, 512), APC_MOMENTS_GLOBAL) == APC_OK);
  CHECK(largest() == g_pairs * tile);
  return 0;
}

// Kept pieces belong to the mesh they were made from, not to the next one at its address.
int kept_mesh() {
  Scene s(2);
  g_records = 10;
  g_pairs = 4;
  const apc_view v = s.view(64, 64);
  for (int attempt = 0; attempt < 64; ++attempt) {
    CHECK(s.moments_pass(v, APC_KEEP_PIECES) == APC_OK);
    const apc_mesh old = s.mesh;
    APC(apc_free_mesh)(s.ctx, s.mesh);
    s.load();
    g_launches.clear();
    CHECK(s.resolve(v, 0) == APC_OK);
    for (const Launch& l : g_launches) CHECK(l.name.find("k_eval") == std::string::npos);
    if (s.mesh == old) return 0;
  }
  printf("no address was used again\n");
  return 1;
}

// On a stream that the caller captures: what has to read totals back is refused before anything is launched; bins at
// hand serve stage one (per tile where their pairs have no numbers) and stage two.
int users_capture() {
  Scene s(8);
  g_records = 10;
  g_pairs = 4;
  const apc_view v = s.view(512, 512), w = s.view(512, 504);
  auto walks = [] {
    uint64_t n = 0;
    for (const Launch& l : g_launches)
      if (l.name.find("k_moments") != std::string::npos) n = l.grid;
    return n;
  };
  int64_t n = 0;
  g_captured = true;
  g_launches.clear();
  CHECK(s.moments_pass(v, APC_MOMENTS_GLOBAL) == APC_E_DEVICE);
  CHECK(s.resolve(v, 0) == APC_E_DEVICE);
  CHECK(APC(apc_resolve_pass_noalloc)(s.ctx, s.mesh, &v, &s.tf, &s.mb, s.moments, s.subs.data(), 8, s.rgba, 0,
                                      nullptr) == APC_E_DEVICE);
  CHECK(g_launches.empty());
  g_captured = false;
  CHECK(s.moments_pass(v, APC_MOMENTS_GLOBAL) == APC_OK);
  g_captured = true;
  g_launches.clear();
  CHECK(s.resolve(v, APC_BY_PAIR) == APC_E_ARG);
  CHECK(s.tiles(v, nullptr, nullptr, 0, &n) == APC_E_DEVICE);
  CHECK(g_launches.empty());
  CHECK(s.moments_pass(v, APC_MOMENTS_GLOBAL) == APC_OK && walks() == 4);
  CHECK(s.resolve(v, 0) == APC_OK);
  g_captured = false;
  CHECK(s.resolve(w, 0) == APC_OK);  // binned without numbers
  g_captured = true;
  CHECK(s.moments_pass(w, APC_MOMENTS_GLOBAL) == APC_OK && walks() == 64 * 63);
  CHECK(s.resolve(w, 0) == APC_OK);
  return 0;
}

// The scan of very many bins adds up the sums of its workgroups in two levels, within its scratch memory.
int many_bins() {
  Scene s(72);
  g_records = 10;
  g_pairs = 4;
  CHECK(s.resolve(s.view(8192, 8192), 0) == APC_OK);  // 75.5M bins, 36864 workgroups
  bool two = false;
  for (const Launch& l : g_launches)
    if (l.name.find("k_bin_supers") != std::string::npos) {
      two = true;
      CHECK(l.arg[1] == 36864 && l.grid == 18);
      const auto buf = g_mem.find(reinterpret_cast<void*>(l.arg[0]));
      CHECK(buf != g_mem.end());
      CHECK(l.arg[2] >= l.arg[0] + 8 * 36864 && l.arg[2] + 8 * 18 <= l.arg[0] + buf->second);
    }
  CHECK(two);
  return 0;
}

// Which form stage one takes: <width> <height> <subdomains> <tets of each>.
int route(int w, int h, int n_sub, int tets_each) {
  Scene s(n_sub, tets_each);
  g_records = 100;
  g_pairs = 7;
  for (uint32_t flags : {APC_MOMENTS_GLOBAL, 0u}) {
    g_launches.clear();
    CHECK(s.moments_pass(s.view(w, h), flags) == APC_OK);
    for (const Launch& l : g_launches)
      if (l.name.find("k_moments") != std::string::npos) printf("%s ", l.grid == 7 ? "pairs" : "tiles");
  }
  return 0;
}

}  // namespace

int main(int argc, char** argv) {
  const std::map<std::string, std::function<int()>> cases = {
      {"refused_noalloc", refused_noalloc},
      {"refused_overflow", refused_overflow},
      {"counted_pairs", counted_pairs},
      {"lost_numbers", lost_numbers},
      {"refused_pair_buffers", refused_pair_buffers},
      {"large_images", large_images},
      {"large_pair_lists", large_pair_lists},
      {"thin_images", thin_images},
      {"kept_mesh", kept_mesh},
      {"users_capture", users_capture},
      {"many_bins", many_bins},
      {"moments_buffer", moments_buffer},
  };
  const bool routes = argc == 7 && std::string(argv[2]) == "route";
  if (!routes && (argc != 3 || !cases.count(argv[2]))) return 2;
  g_lib = dlopen(argv[1], RTLD_NOW | RTLD_LOCAL);
  if (!g_lib) {
    printf("%s\n", dlerror());
    return 2;
  }
  return routes ? route(atoi(argv[3]), atoi(argv[4]), atoi(argv[5]), atoi(argv[6])) : cases.at(argv[2])();
}
