// Host-side tests of libvgicp.so without a GPU: this program defines the HIP runtime functions that the
// library calls (they take the place of the runtime's, since a program's own symbols come first), with
// device memory in host memory, kernels that do nothing and refusals on demand. What it checks is the
// library's host code: who owns which block of memory, on which device, and what is left after a
// refused allocation. Usage: driver <test>; prints "<test> ok".
#include <algorithm>
#include <atomic>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <thread>
#include <vector>

#include "../../include/vgicp.h"

#define CHECK(c)                                                         \
  do {                                                                   \
    if (!(c)) {                                                          \
      std::printf("%s:%d: %s (%s)\n", __FILE__, __LINE__, #c, vgicp_last_error()); \
      std::exit(1);                                                      \
    }                                                                    \
  } while (0)

// ------------------------------------------------------------------ the runtime

namespace {

struct Alloc {
  size_t bytes;
  int device;
};
struct Launch {  // a launch of batch_kernel
  char *items, *partials;
};
struct Dim3 {
  uint32_t x, y, z;
};
struct Config {
  Dim3 grid, block;
  size_t shared;
  void* stream;
};
struct Graph {
  std::vector<Launch> launches;
};
struct Copy {  // an asynchronous copy that runs at the next wait
  void* to;
  const void* from;
  std::vector<char> then;  // what was there when it was asked for
};

constexpr int kOk = 0, kInvalid = 1, kOutOfMemory = 2;
std::mutex g_mu;
std::map<char*, Alloc> g_live;                 // device memory
std::map<char*, size_t> g_pinned;
std::map<const void*, char*> g_symbols;
size_t g_refuse_above = ~(size_t)0;            // device allocations of more bytes are refused
size_t g_refuse_exactly = 0;                    // and those of this size
size_t g_largest = 0;                          // largest device allocation so far
std::atomic<int> g_launched{0};                // kernels launched
std::atomic<int> g_synchronised{-1};           // device of the last device synchronisation
bool g_refuse_waits = false;                   // synchronisations fail (another thread captures, say)
bool g_defer = false;                          // asynchronous copies run at the next wait
std::vector<Copy> g_copies;
Graph* g_capture = nullptr;
std::vector<Launch> g_ran;                     // executed launches of batch_kernel
thread_local int t_device = 0, t_error = kOk;
thread_local std::vector<Config> t_config;

// Host stub -> device name. The library registers its kernels before this program's globals exist.
std::map<const void*, std::string>& kernels() {
  static auto* m = new std::map<const void*, std::string>;
  return *m;
}

int error(int e) {
  t_error = e;
  return e;
}

// The map build, filter or neighbour search that a thread is in: the block and the pinned report that its
// first kernel set up. Nobody else may be given them before it ends (done).
std::map<const void*, std::thread::id> g_owner;
thread_local const void *t_block = nullptr, *t_report = nullptr;

void own(const void* block, const void* report) {
  std::lock_guard<std::mutex> lk(g_mu);
  t_block = block;
  t_report = report;
  for (const void* p : {block, report}) g_owner[p] = std::this_thread::get_id();
}

void still_owned() {
  std::lock_guard<std::mutex> lk(g_mu);
  for (const void* p : {t_block, t_report})
    if (p && g_owner[p] != std::this_thread::get_id()) {
      std::printf("a block is in two hands\n");
      std::exit(1);
    }
}

void done() { t_block = t_report = nullptr; }

// The allocation that holds p, nullptr when it is not live.
const Alloc* owner(const void* p) {
  std::lock_guard<std::mutex> lk(g_mu);
  auto it = g_live.upper_bound((char*)p);
  if (it == g_live.begin()) return nullptr;
  --it;
  return (char*)p < it->first + it->second.bytes ? &it->second : nullptr;
}

size_t live_count() {
  std::lock_guard<std::mutex> lk(g_mu);
  return g_live.size();
}

}  // namespace

extern "C" {

void** __hipRegisterFatBinary(const void*) {
  static void* binary = nullptr;
  return &binary;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*,
                           void*, void*, int*) {
  kernels()[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim3 g, Dim3 b, size_t shared, void* s) {
  t_config.push_back({g, b, shared, s});
  return kOk;
}
int __hipPopCallConfiguration(Dim3* g, Dim3* b, size_t* shared, void** s) {
  const Config c = t_config.back();
  t_config.pop_back();
  *g = c.grid;
  *b = c.block;
  *shared = c.shared;
  *s = c.stream;
  return kOk;
}
int hipLaunchKernel(const void* f, Dim3, Dim3, void** args, size_t, void*) {
  ++g_launched;
  if (kernels()[f].find("call_init_kernel") != std::string::npos && *(void**)args[2])
    own(*(void**)args[2], *(void**)args[3]);
  still_owned();
  if (kernels()[f].find("12batch_kernel") != std::string::npos) {
    const Launch l = {*(char**)args[2], *(char**)args[6]};
    std::lock_guard<std::mutex> lk(g_mu);
    (g_capture ? g_capture->launches : g_ran).push_back(l);
  }
  return kOk;
}

int hipGetDevice(int* d) {
  *d = t_device;
  return kOk;
}
int hipSetDevice(int d) {
  t_device = d;
  return kOk;
}
int hipDeviceSynchronize() {
  if (g_refuse_waits) return error(kInvalid);
  g_synchronised = t_device;
  return kOk;
}
int hipGetDevicePropertiesR0600(void*, int) { return kInvalid; }  // the library assumes 256 CUs
const char* hipGetErrorString(int) { return "refused"; }
int hipGetLastError() {
  const int e = t_error;
  t_error = kOk;
  return e;
}
int hipGetSymbolAddress(void** p, const void* s) {
  std::lock_guard<std::mutex> lk(g_mu);
  char*& m = g_symbols[s];
  if (!m) m = (char*)std::calloc(1, 1 << 20);
  *p = m;
  return kOk;
}

int hipMalloc(void** p, size_t n) {
  if (n > g_refuse_above || n == g_refuse_exactly) return error(kOutOfMemory);
  char* q = (char*)std::calloc(1, n ? n : 1);
  std::lock_guard<std::mutex> lk(g_mu);
  g_live[q] = {n, t_device};
  if (n > g_largest) g_largest = n;
  *p = q;
  return kOk;
}
int hipFree(void* p) {
  if (!p) return kOk;
  {
    std::lock_guard<std::mutex> lk(g_mu);
    if (g_live.erase((char*)p) == 0) {
      std::printf("hipFree of memory that is not live\n");
      std::exit(1);
    }
  }
  std::free(p);
  return kOk;
}
int hipMallocAsync(void** p, size_t n, void*) { return hipMalloc(p, n); }
int hipFreeAsync(void* p, void*) { return hipFree(p); }
int hipHostMalloc(void** p, size_t n, unsigned) {
  *p = std::calloc(1, n);
  std::lock_guard<std::mutex> lk(g_mu);
  g_pinned[(char*)*p] = n;
  return kOk;
}
int hipHostFree(void* p) {
  std::lock_guard<std::mutex> lk(g_mu);
  g_pinned.erase((char*)p);
  std::free(p);
  return kOk;
}
int hipMemcpy(void* d, const void* s, size_t n, int) {
  std::memcpy(d, s, n);
  return kOk;
}
int hipMemcpyAsync(void* d, const void* s, size_t n, int k, void*) {
  if (!g_defer) return hipMemcpy(d, s, n, k);
  g_copies.push_back({d, s, std::vector<char>((const char*)s, (const char*)s + n)});
  return kOk;
}
int hipMemset(void* d, int v, size_t n) {
  std::memset(d, v, n);
  return kOk;
}
int hipMemsetAsync(void* d, int v, size_t n, void*) { return hipMemset(d, v, n); }

int hipEventCreateWithFlags(void** e, unsigned) {
  *e = std::malloc(1);
  return kOk;
}
int hipEventCreate(void** e) { return hipEventCreateWithFlags(e, 0); }
int hipEventDestroy(void* e) {
  std::free(e);
  return kOk;
}
int hipEventRecord(void*, void*) { return kOk; }
int hipEventSynchronize(void*) { return kOk; }
int hipEventElapsedTime(float* ms, void*, void*) {
  static int n = 0;
  *ms = 1.0f + 0.001f * (float)(n++ % 97);
  return kOk;
}
int hipStreamCreateWithFlags(void** s, unsigned) {
  *s = std::malloc(1);
  return kOk;
}
int hipStreamDestroy(void* s) {
  std::free(s);
  return kOk;
}
int hipStreamSynchronize(void*) {
  if (g_refuse_waits) return error(kInvalid);
  for (const Copy& c : g_copies) {
    if (std::memcmp(c.from, c.then.data(), c.then.size()) != 0) {
      std::printf("the source of a copy changed before it was waited for\n");
      std::exit(1);
    }
    std::memcpy(c.to, c.from, c.then.size());
  }
  g_copies.clear();
  still_owned();
  return kOk;
}
int hipStreamWaitEvent(void*, void*, unsigned) { return kOk; }
int hipStreamBeginCapture(void*, int) {
  g_capture = new Graph;
  return kOk;
}
int hipStreamEndCapture(void*, void** g) {
  *g = g_capture;
  g_capture = nullptr;
  return kOk;
}
int hipGraphInstantiate(void** x, void* g, void*, char*, size_t) {
  *x = new Graph(*(Graph*)g);
  return kOk;
}
int hipGraphDestroy(void* g) {
  delete (Graph*)g;
  return kOk;
}
int hipGraphExecDestroy(void* x) {
  delete (Graph*)x;
  return kOk;
}
int hipGraphLaunch(void* x, void*) {
  std::lock_guard<std::mutex> lk(g_mu);
  for (const Launch& l : ((Graph*)x)->launches) g_ran.push_back(l);
  return kOk;
}

}  // extern "C"

// ------------------------------------------------------------------ the tests

namespace {

// A device pointer of the caller's that nothing on the host reads.
template <typename T>
T* some(size_t i = 1) {
  return reinterpret_cast<T*>(4096 * i);
}

vgicp_voxelmap empty_map() {
  vgicp_voxelmap m = nullptr;
  CHECK(vgicp_build_voxelmap(nullptr, nullptr, 0, 0.5, nullptr, &m) == VGICP_OK);
  return m;
}

vgicp_batch make_batch(vgicp_voxelmap m, const std::vector<int64_t>& sizes) {
  std::vector<vgicp_cloud> clouds;
  std::vector<vgicp_factor> factors;
  for (size_t c = 0; c < sizes.size(); ++c) {
    clouds.push_back({some<float>(), some<float>(), sizes[c]});
    factors.push_back({0, (int32_t)c, 0, 1, 1});
  }
  vgicp_batch b = nullptr;
  CHECK(vgicp_batch_create(&m, 1, clouds.data(), (int32_t)clouds.size(), factors.data(),
                           (int32_t)factors.size(), 2, &b) == VGICP_OK);
  return b;
}

// The memory that a linearization of the batch runs on.
Launch linearize(vgicp_batch b) {
  g_ran.clear();
  CHECK(vgicp_batch_linearize(b, some<double>(), VGICP_ACC_FP64, some<double>(2), some<double>(3),
                              some<double>(4), some<int64_t>(5), nullptr) == VGICP_OK);
  CHECK(g_ran.size() == 1);
  CHECK(owner(g_ran[0].items) && owner(g_ran[0].partials));
  return g_ran[0];
}

bool same(const vgicp_schedule& a, const vgicp_schedule& b) {
  return a.block == b.block && a.tile == b.tile && a.blocks_per_cu == b.blocks_per_cu &&
         a.lookahead == b.lookahead;
}

// A refused allocation fails its own call and nothing after it.
void refusal_is_forgotten() {
  const vgicp_voxelmap m = empty_map();
  const vgicp_batch a = make_batch(m, std::vector<int64_t>(8, 100000));
  const vgicp_schedule small{256, 2048, 4, 4};
  g_refuse_above = 0;
  CHECK(vgicp_batch_set_schedule(a, &small) == VGICP_E_OOM);
  g_refuse_above = ~(size_t)0;
  vgicp_batch_destroy(make_batch(m, {100}));
  // memory that does not come from the kept blocks
  const double* grad = some<double>();
  g_refuse_above = 0;
  CHECK(vgicp_batch_backward(a, grad, VGICP_ACC_FP64, grad, some<double>(2), nullptr, nullptr, nullptr) ==
        VGICP_E_OOM);
  g_refuse_above = ~(size_t)0;
  vgicp_batch_destroy(make_batch(m, {100}));
  vgicp_batch_destroy(a);
  vgicp_destroy_voxelmap(m);
}

// A schedule whose memory is refused leaves the batch as it was: on its old schedule, with memory that
// nobody else is given.
void schedule_refused() {
  const vgicp_voxelmap m = empty_map();
  const std::vector<int64_t> sizes(8, 100000);
  const vgicp_batch a = make_batch(m, sizes);
  const Launch before = linearize(a);
  vgicp_schedule old, now, small{256, 2048, 4, 4};
  CHECK(vgicp_batch_get_schedule(a, &old) == VGICP_OK);
  g_refuse_above = 0;
  CHECK(vgicp_batch_set_schedule(a, &small) == VGICP_E_OOM);
  g_refuse_above = ~(size_t)0;
  CHECK(vgicp_batch_get_schedule(a, &now) == VGICP_OK && same(old, now));
  const vgicp_batch b = make_batch(m, sizes);
  const Launch mine = linearize(a), other = linearize(b);
  CHECK(mine.partials != other.partials && mine.items != other.items);
  CHECK(mine.partials == before.partials && mine.items == before.items);
  // the candidates that fit are timed, the others are skipped, and the batch runs on the choice
  g_refuse_above = 300 << 10;
  vgicp_schedule chosen;
  CHECK(vgicp_batch_autotune(a, some<double>(), VGICP_ACC_FP64, nullptr, &chosen, nullptr) == VGICP_OK);
  CHECK(vgicp_batch_get_schedule(a, &now) == VGICP_OK && same(chosen, now));
  g_refuse_above = ~(size_t)0;
  const Launch tuned = linearize(a);
  CHECK(tuned.partials != other.partials && tuned.items != other.items);
  // and without refusals it changes
  CHECK(vgicp_batch_set_schedule(a, &small) == VGICP_OK);
  CHECK(vgicp_batch_get_schedule(a, &now) == VGICP_OK && same(small, now));
  const Launch changed = linearize(a);
  CHECK(changed.partials != other.partials && changed.items != other.items);
  vgicp_batch_destroy(a);
  vgicp_batch_destroy(b);
  vgicp_destroy_voxelmap(m);
}

// A batch's calls without a device argument of their own work on the batch's device, whichever is
// current, and leave that one current.
void other_device_current() {
  const vgicp_voxelmap m = empty_map();
  const vgicp_batch a = make_batch(m, std::vector<int64_t>(8, 100000));
  const vgicp_schedule small{256, 2048, 4, 4};
  CHECK(hipSetDevice(1) == kOk);
  CHECK(vgicp_batch_set_schedule(a, &small) == VGICP_OK);
  CHECK(t_device == 1 && g_synchronised == 0);
  // what was given back is the other device's memory, and no other's is taken from it
  const vgicp_voxelmap m1 = empty_map();
  const vgicp_batch b = make_batch(m1, std::vector<int64_t>(8, 100000));
  const Launch other = linearize(b);
  CHECK(owner(other.items)->device == 1 && owner(other.partials)->device == 1);
  CHECK(vgicp_batch_refresh(a, nullptr) == VGICP_OK);
  CHECK(t_device == 1);
  CHECK(hipSetDevice(0) == kOk);
  const Launch mine = linearize(a);
  CHECK(owner(mine.items)->device == 0 && owner(mine.partials)->device == 0);
  vgicp_batch_destroy(a);
  vgicp_batch_destroy(b);
  vgicp_destroy_voxelmap(m);
  vgicp_destroy_voxelmap(m1);
}

// The clouds of a batch are put in order together; one large cloud among many small ones does not
// make each of those pay for it. 3.9 M points: 154 MB of copies, at most 160 MB to order them.
void order_memory() {
  const vgicp_voxelmap m = empty_map();
  std::vector<int64_t> sizes(4000, 900);
  sizes[700] = 260000;
  sizes[2900] = 262144;
  g_largest = 0;
  const vgicp_batch b = make_batch(m, sizes);
  CHECK(g_largest <= 200u << 20);
  vgicp_batch_destroy(b);
  vgicp_destroy_voxelmap(m);
}

// The caller's workspace: absent, misaligned and short ones are refused before anything is launched.
void workspace_checks() {
  const vgicp_voxelmap m = empty_map();
  const double T[12] = {1, 0, 0, 0, 0, 1, 0, 0, 0, 0, 1, 0};
  double* out = some<double>(2);
  int64_t need = 0;
  CHECK(vgicp_workspace_size(1000, &need) == VGICP_OK && need > 0);
  auto all = [&](void* ws, int64_t bytes, vgicp_status want) {
    g_launched = 0;
    CHECK(vgicp_linearize_workspace(m, some<float>(), some<float>(), 1000, T, T, 1, VGICP_ACC_FP64, out,
                                    out, out, some<int64_t>(3), nullptr, ws, bytes, nullptr) == want);
    CHECK(vgicp_evaluate_workspace(m, some<float>(), some<float>(), 1000, T, T, VGICP_ACC_FP64, out,
                                   some<int64_t>(3), nullptr, ws, bytes, nullptr) == want);
    CHECK(vgicp_backward_tangent_workspace(m, some<float>(), some<float>(), 1000, T, T, nullptr, nullptr,
                                           1, some<int32_t>(4), out, VGICP_ACC_FP64, out, nullptr, ws,
                                           bytes, nullptr) == want);
    CHECK((g_launched > 0) == (want == VGICP_OK));
  };
  char* ws = some<char>(5);
  all(ws, need, VGICP_OK);
  all(ws + 8, need, VGICP_OK);
  all(nullptr, need, VGICP_E_INVALID_ARG);
  all(ws, -1, VGICP_E_INVALID_ARG);
  for (int off = 1; off < 8; ++off) all(ws + off, need, VGICP_E_INVALID_ARG);
  all(ws, 8, VGICP_E_CAPACITY);
  vgicp_destroy_voxelmap(m);
}

// A call that ends early leaves no copy behind that reads memory of its own.
void copies_of_a_refused_call() {
  const vgicp_voxelmap m = empty_map();
  const vgicp_cloud cloud = {some<float>(), some<float>(), (1 << 18) + 5};
  const vgicp_factor f = {0, 0, 0, 1, 1};
  vgicp_batch b = nullptr;
  g_defer = true;
  g_refuse_exactly = 256 * 129 * sizeof(int);  // the digit counts of the long sort
  CHECK(vgicp_batch_create(&m, 1, &cloud, 1, &f, 1, 2, &b) == VGICP_E_OOM && !b);
  g_refuse_exactly = 0;
  CHECK(hipStreamSynchronize(nullptr) == kOk);
  CHECK(vgicp_batch_create(&m, 1, &cloud, 1, &f, 1, 2, &b) == VGICP_OK);
  CHECK(vgicp_batch_destroy(b) == VGICP_OK && vgicp_destroy_voxelmap(m) == VGICP_OK);
}

// The autotuner times no launch twice in its first stage: with the grid capped at the resident blocks
// (256 CUs here, 4 blocks of 4 waves, 3 for the forms with wide sums) several blocks-per-CU values are one.
void tuned_once() {
  const vgicp_voxelmap m = empty_map();
  const vgicp_batch b = make_batch(m, std::vector<int64_t>(64, 1000000));
  const char* path = std::getenv("VGICP_AUTOTUNE_LOG");
  for (int precision = 0; precision < 4; ++precision) {
    std::remove(path);
    vgicp_schedule chosen;
    CHECK(vgicp_batch_autotune(b, some<double>(), (vgicp_precision)precision, nullptr, &chosen, nullptr) ==
          VGICP_OK);
    const int most = precision == VGICP_ACC_KAHAN_FP32 || precision == VGICP_MATH_FP64 ? 3 : 4;
    std::map<std::vector<int>, int> launches;
    std::FILE* f = std::fopen(path, "r");
    CHECK(f);
    char line[256];
    while (std::fgets(line, sizeof line, f)) {
      int stage, block, tile, per_cu, look;
      if (std::sscanf(line, "%d %d %d %d %d", &stage, &block, &tile, &per_cu, &look) != 5 || stage != 1)
        continue;
      const std::vector<int> launch = {block, tile, look, std::min(per_cu * block / 256, most)};
      CHECK(++launches[launch] == 1);
    }
    std::fclose(f);
    CHECK(launches.size() == (most == 4 ? 54u : 45u));  // 2 x 3 x 3 cuts, 4 + 2 grids (3 + 2)
  }
  vgicp_batch_destroy(b);
  vgicp_destroy_voxelmap(m);
}

// Memory whose users could not be waited for is freed (the runtime's free waits by itself), not kept
// for the next call.
void refused_waits() {
  vgicp_voxelmap m = empty_map();
  vgicp_batch b = make_batch(m, {1000, 2000});
  CHECK(vgicp_release_idle() == VGICP_OK);
  const size_t pinned = g_pinned.size();
  CHECK(pinned == 0);
  g_refuse_waits = true;
  int64_t n = 0;
  CHECK(vgicp_downsample(some<float>(), nullptr, 5000, 0.5, 0.1, some<float>(2), nullptr, 5000, &n,
                         nullptr) == VGICP_E_HIP);
  vgicp_voxelmap other = nullptr;
  CHECK(vgicp_build_voxelmap(nullptr, nullptr, 0, 0.5, nullptr, &other) == VGICP_E_HIP && !other);
  CHECK(vgicp_knn(some<float>(), 5000, 10, 0.0, some<int32_t>(2), nullptr) == VGICP_E_HIP);
  CHECK(vgicp_batch_refresh(b, nullptr) == VGICP_E_HIP);
  CHECK(vgicp_batch_destroy(b) == VGICP_OK);
  CHECK(vgicp_destroy_voxelmap(m) == VGICP_OK);
  g_refuse_waits = false;
  // nothing is left that a next call could be given
  CHECK(live_count() == 0 && g_pinned.empty());
  vgicp_destroy_voxelmap(empty_map());
}

// Maps, filters, neighbour searches and one-shot batches from eight threads: no block is in two hands,
// what is kept is bounded, and the release gives all of it back.
void threads() {
  const double T[24] = {1, 0, 0, 0, 0, 1, 0, 0, 0, 0, 1, 0, 1, 0, 0, 0, 0, 1, 0, 0, 0, 0, 1, 0};
  std::vector<std::thread> all;
  for (int k = 0; k < 8; ++k)
    all.emplace_back([k, &T] {
      vgicp_stream s = some<void>(k + 1);
      for (int i = 0; i < 40; ++i) {
        const int64_t n = 1000 + 7919 * ((k + i) % 5);
        int64_t m = 0;
        CHECK(vgicp_downsample(some<float>(), nullptr, n, 0.5, 0.1, some<float>(2), nullptr, n, &m, s) ==
              VGICP_OK);
        done();
        CHECK(vgicp_knn(some<float>(), n, 10, 0.0, some<int32_t>(2), s) == VGICP_OK);
        done();
        vgicp_voxelmap map = nullptr;
        CHECK(vgicp_build_voxelmap(nullptr, nullptr, 0, 0.5, s, &map) == VGICP_OK);
        done();
        const vgicp_cloud cloud = {some<float>(), some<float>(), n};
        const vgicp_factor f = {0, 0, 0, 1, 1};
        CHECK(vgicp_linearize_batched(&map, 1, &cloud, 1, T, 2, &f, 1, VGICP_ACC_FP64, some<double>(2),
                                      some<double>(3), some<double>(4), some<int64_t>(5), s) == VGICP_OK);
        done();
        CHECK(vgicp_destroy_voxelmap(map) == VGICP_OK);
        done();
      }
    });
  for (auto& t : all) t.join();
  const vgicp_voxelmap m = empty_map();
  vgicp_batch_destroy(make_batch(m, {6000000}));  // 240 MB of copies, among others
  vgicp_batch_destroy(make_batch(m, {4000000}));
  done();
  size_t kept = 0;
  for (const auto& a : g_live) kept += a.second.bytes;
  CHECK(kept > 0 && kept <= (256u << 20) + (1u << 20));  // and the map
  CHECK(vgicp_release_idle() == VGICP_OK);
  CHECK(live_count() == 1 && g_pinned.empty());
  CHECK(vgicp_destroy_voxelmap(m) == VGICP_OK && vgicp_release_idle() == VGICP_OK);
  CHECK(live_count() == 0);
  CHECK(vgicp_release_idle() == VGICP_OK);
  vgicp_destroy_voxelmap(empty_map());  // and the library takes memory again
}

}  // namespace

int main(int argc, char** argv) {
  const std::map<std::string, void (*)()> tests = {
      {"refusal_is_forgotten", refusal_is_forgotten},
      {"schedule_refused", schedule_refused},
      {"other_device_current", other_device_current},
      {"order_memory", order_memory},
      {"workspace_checks", workspace_checks},
      {"copies_of_a_refused_call", copies_of_a_refused_call},
      {"tuned_once", tuned_once},
      {"refused_waits", refused_waits},
      {"threads", threads},
  };
  const auto it = tests.find(argc > 1 ? argv[1] : "");
  if (it == tests.end()) return 2;
  it->second();
  std::printf("%s ok\n", argv[1]);
  return 0;
}
