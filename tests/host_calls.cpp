// A program that loads libinframind.so on a machine without a GPU and stands in
// for the runtime under it: "device" memory is host memory, kernels are not run,
// and every launch is printed with its kernel, grid and the device current at the
// time. `host_calls LIB SCENARIO` runs one scenario of calls (main below).
#include <dlfcn.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <map>
#include <string>
#include <vector>

#include "../include/inframind.h"

struct Dim3 {
  uint32_t x, y, z;
};
static int g_device = 0, g_cus = 256;   // current device; compute units (< 0: the query fails)
static bool g_log = false;
static std::map<const void*, std::string> g_names;
static Dim3 g_grid, g_block;

// The runtime's functions that the library calls (errors are ints, 0 for success).
extern "C" {
void** __hipRegisterFatBinary(const void*) {
  static void* m = nullptr;
  return &m;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*,
                           int*) {
  g_names[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t, void*) {
  g_grid = grid;
  g_block = block;
  return 0;
}
int __hipPopCallConfiguration(Dim3* grid, Dim3* block, size_t* shared, void** stream) {
  *grid = g_grid;
  *block = g_block;
  *shared = 0;
  *stream = nullptr;
  return 0;
}
int hipLaunchKernel(const void* f, Dim3 grid, Dim3 block, void**, size_t, void*) {
  if (g_log) printf("launch %s grid %u block %u device %d\n", g_names[f].c_str(), grid.x, block.x, g_device);
  return 0;
}
int hipGetDevice(int* d) {
  *d = g_device;
  return 0;
}
int hipSetDevice(int d) {
  g_device = d;
  return 0;
}
int hipDeviceGetAttribute(int* v, int, int) {
  if (g_cus < 0) return 1;
  *v = g_cus;
  return 0;
}
int hipDeviceSynchronize() {
  if (g_log) printf("synchronize device %d\n", g_device);
  return 0;
}
int hipMalloc(void** p, size_t n) {
  *p = calloc(n, 1);
  return *p ? 0 : 2;
}
int hipFree(void* p) {
  free(p);
  return 0;
}
int hipHostMalloc(void** p, size_t n, unsigned) {
  if (g_log) printf("host memory device %d\n", g_device);
  return hipMalloc(p, n);
}
int hipHostFree(void* p) { return hipFree(p); }
int hipMemcpy(void* d, const void* s, size_t n, int) {
  memcpy(d, s, n);
  return 0;
}
int hipMemset(void* d, int v, size_t n) {
  memset(d, v, n);
  return 0;
}
int hipStreamSynchronize(void*) { return 0; }
int hipGetLastError() { return 0; }
const char* hipGetErrorString(int) { return "an error"; }
int hipGetSymbolAddress(void** p, const void*) {
  static char some[64];
  *p = some;
  return 0;
}
}

static void* g_lib;
template <class F>
F* sym(F*, const char* name) {
  return reinterpret_cast<F*>(dlsym(g_lib, name));
}
#define CALL(f) sym(&f, #f)
static int need(im_status s, const char* what) {
  if (s == IM_OK) return 0;
  printf("%s: status %d\n", what, (int)s);
  exit(1);
}

struct Shape {
  int E, M, K, qcap, slots, hidden, layers, dtype, steps;
  int embed = 32;
};
static im_pool* make(const Shape& s) {
  im_pool_desc d{};
  d.n_envs = s.E; d.n_models = s.M; d.n_depths = s.K; d.queue_cap = s.qcap; d.max_slots = s.slots;
  d.embed_dim = s.embed; d.feat_dim = s.embed + 4 * s.M + 1; d.n_layers = s.layers;
  for (int l = 0; l + 1 < s.layers; ++l) d.widths[l] = s.hidden;
  d.widths[s.layers - 1] = s.M * s.K;
  d.dtype = s.dtype; d.max_arrivals_per_env_tick = 1 << 16; d.budget_max = 100; d.max_steps = s.steps;
  static std::vector<float> zeros(1 << 20);
  const float* w[3] = {zeros.data(), zeros.data(), zeros.data()};
  std::vector<int32_t> cap((size_t)s.E * s.M, 1);
  im_pool* p = nullptr;
  need(CALL(im_pool_create)(&d, w, w, zeros.data(), 8, cap.data(), nullptr, nullptr, &p), "im_pool_create");
  return p;
}
static im_arrivals arrivals(int n, int E) {
  static std::vector<int32_t> i32;
  static std::vector<int16_t> i16;
  i32.assign((size_t)n + E + 1, 0);
  i16.assign((size_t)n + 1, 1);
  im_arrivals a{};
  a.offsets = a.q_idx = i32.data();
  a.budget = a.base_svc = a.n_steps = i16.data();
  a.n_total = n;
  return a;
}

// Reads envs [e0, e0 + n) and writes them back.
static void read_and_write(im_pool* p, const Shape& s, int e0, int n, bool write) {
  std::vector<im_env_state> envs(n + 1);
  std::vector<im_model_state> models((size_t)(n + 1) * s.M);
  std::vector<im_slot> slots((size_t)(n + 1) * s.M * s.slots);
  std::vector<im_entry> queues((size_t)(n + 1) * s.M * s.qcap);
  std::vector<int64_t> hist((size_t)(n + 1) * s.M * s.K);
  int32_t t = 0;
  need(CALL(im_read_state)(p, e0, n, &t, envs.data(), models.data(), slots.data(), queues.data(), hist.data()),
       "im_read_state");
  if (!write) return;
  for (im_model_state& m : models) {
    m = im_model_state{};
    m.capacity = m.enabled = 1;
  }
  for (im_slot& x : slots) x = im_slot{-1, 0, 0, 0};
  need(CALL(im_write_state)(p, e0, n, 0, envs.data(), models.data(), slots.data(), queues.data(), hist.data()),
       "im_write_state");
}

int main(int argc, char** argv) {
  if (argc < 3) return 2;
  const std::string what = argv[2];
  g_lib = dlopen(argv[1], RTLD_NOW);
  if (!g_lib) {
    printf("%s\n", dlerror());
    return 2;
  }
  if (what == "other_device") {   // a pool of device 0, used while device 1 is current
    const Shape s{3, 2, 2, 8, 2, 64, 2, IM_F32, 1};
    im_pool* p = make(s);
    g_device = 1;
    g_log = true;
    read_and_write(p, s, 0, 3, true);
    printf("after device %d\n", g_device);
    g_log = false;
    g_device = 0;
    CALL(im_destroy)(p);
    return 0;
  }
  if (what == "no_cu_count") {   // the compute units are not known
    g_cus = -1;
    for (int dtype : {IM_F32, IM_BF16}) {
      for (int hidden : {32, 64, 256}) {
        const Shape s{4, 2, 2, 8, 2, hidden, 3, dtype, 1};
        im_pool* p = make(s);
        for (int n : {1, 100}) {
          std::vector<int32_t> act(n);
          const im_arrivals a = arrivals(n, s.E);
          g_log = true;
          printf("route %d hidden %d rows %d\n", dtype, hidden, n);
          fflush(stdout);
          need(CALL(im_route)(p, &a, act.data(), nullptr, nullptr), "im_route");
          g_log = false;
        }
        CALL(im_destroy)(p);
      }
    }
    return 0;
  }
  if (what == "restore") {   // parts of a pool restored
    const Shape s{3000, 2, 2, 1, 1, 64, 2, IM_F32, 1};
    im_pool* p = make(s);
    for (const int n : {0, 1, 3, 1024, 2000}) {
      printf("envs %d\n", n);
      g_log = true;
      read_and_write(p, s, 1000, n, true);
      g_log = false;
    }
    CALL(im_destroy)(p);
    return 0;
  }
  if (what == "chain_grid") {   // E models slots arrivals hidden cus
    const int E = atoi(argv[3]), n = atoi(argv[6]);
    g_cus = atoi(argv[8]);
    const Shape s{E, atoi(argv[4]), 1, 1, atoi(argv[5]), atoi(argv[7]), 3, IM_F32, 3};
    im_pool* p = make(s);
    std::vector<int32_t> act((size_t)n + E * s.M * s.slots);
    const im_arrivals a = arrivals(n, E);
    g_log = true;
    need(CALL(im_route)(p, &a, act.data(), nullptr, nullptr), "im_route");
    g_log = false;
    CALL(im_destroy)(p);
    return 0;
  }
  if (what == "growing_reads") {   // one env, two, ... of a pool
    const Shape s{200, 4, 2, 64, 2, 64, 2, IM_F32, 1};
    im_pool* p = make(s);
    g_log = true;
    for (int n = 1; n <= s.E; ++n) read_and_write(p, s, 0, n, false);
    g_log = false;
    CALL(im_destroy)(p);
    return 0;
  }
  if (what == "chain_rl") {   // models slots arrivals layers
    const int E = 64, n = atoi(argv[5]);
    g_cus = 8;
    Shape s{E, atoi(argv[3]), 3, 1, atoi(argv[4]), 256, atoi(argv[6]), IM_BF16, 3};
    s.embed = 64;
    im_pool* p = make(s);
    std::vector<int32_t> act((size_t)n + E * s.M * s.slots);
    const im_arrivals a = arrivals(n, E);
    im_policy_out o{};
    o.actions = act.data();
    g_log = true;
    need(CALL(im_route_sample)(p, &a, 1, 0, &o, nullptr), "im_route_sample");
    g_log = false;
    CALL(im_destroy)(p);
    return 0;
  }
  printf("no scenario %s\n", what.c_str());
  return 2;
}
