// Host paths of libmplb on a machine without a GPU.  This program is linked
// with libmplb.so and defines the HIP calls that it makes: device memory is
// host memory, copies happen at once, kernels do nothing.  Failures that a
// real device shows rarely can then be forced, and the calls counted.
//
//   driver CASE     prints "ok" and exits 0 if every expectation holds
#include <hip/hip_runtime_api.h>

#include <atomic>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <future>
#include <new>
#include <vector>

#include "mplb.h"

static int fails = 0;
#define EXPECT(cond)                                             \
  do {                                                           \
    if (!(cond)) {                                               \
      std::printf("FAIL line %d: %s\n", __LINE__, #cond);        \
      std::fflush(stdout);                                       \
      ++fails;                                                   \
    }                                                            \
  } while (0)

// ------------------------------------------------- allocation failures
static thread_local bool no_memory = false;
void* operator new(size_t n) {
  void* p = no_memory ? nullptr : std::malloc(n ? n : 1);
  if (!p) throw std::bad_alloc();
  return p;
}
void* operator new(size_t n, const std::nothrow_t&) noexcept { return no_memory ? nullptr : std::malloc(n ? n : 1); }
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }

// ------------------------------------------------------------ fake HIP
// Two devices; a stream and an event belong to one, and an event is recorded on
// its own device's streams only.
struct FakeStream {
  int device;
};
struct FakeEvent {
  int device;
};
static thread_local int current = 0;
static std::atomic<int> host_allocations{0}, host_live{0}, events_live{0};
static std::atomic<int> copies{0};
static int event_limit = 1 << 20;
struct Launch {
  unsigned blocks, threads;
};
static std::vector<Launch> launches;
static thread_local struct {
  dim3 grid, block;
  size_t shared;
  hipStream_t stream;
} pushed;
static const void *locked_from = nullptr, *locked_to = nullptr;  // page-locked memory of the caller
static std::function<void()> during_host_malloc;
static int device_of(hipStream_t s) { return s ? ((FakeStream*)s)->device : current; }

extern "C" {
hipError_t hipGetDevice(int* d) { *d = current; return hipSuccess; }
hipError_t hipSetDevice(int d) { current = d; return hipSuccess; }
hipError_t hipStreamGetDevice(hipStream_t s, hipDevice_t* d) { *d = device_of(s); return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "fake error"; }
hipError_t hipMalloc(void** p, size_t n) { *p = std::malloc(n); return *p ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  if (during_host_malloc) during_host_malloc();
  ++host_allocations;
  ++host_live;
  *p = std::malloc(n);
  return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipHostFree(void* p) {
  --host_live;
  std::free(p);
  return hipSuccess;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void* p) {
  const bool locked = p >= locked_from && p < locked_to;
  if (!locked) return hipErrorInvalidValue;  // what older runtimes say of pageable memory
  *a = hipPointerAttribute_t{};
  a->type = hipMemoryTypeHost;
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* dst, const void* src, size_t n, hipMemcpyKind, hipStream_t) {
  ++copies;
  std::memcpy(dst, src, n);
  return hipSuccess;
}
hipError_t hipMemsetAsync(void* p, int v, size_t n, hipStream_t) { std::memset(p, v, n); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) {
  if (events_live == event_limit) return hipErrorOutOfMemory;
  ++events_live;
  auto* f = (FakeEvent*)std::malloc(sizeof(FakeEvent));
  f->device = current;
  *e = (hipEvent_t)f;
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { --events_live; std::free((void*)e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  return ((FakeEvent*)e)->device == device_of(s) ? hipSuccess : hipErrorInvalidHandle;
}
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 0; return hipSuccess; }
static char symbol[1 << 20];
hipError_t hipGetSymbolAddress(void** p, const void*) { *p = symbol; return hipSuccess; }
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, hipStream_t s) {
  pushed = {grid, block, shared, s};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shared, hipStream_t* s) {
  *grid = pushed.grid; *block = pushed.block; *shared = pushed.shared; *s = pushed.stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void*, dim3 grid, dim3 block, void**, size_t, hipStream_t) {
  launches.push_back({grid.x, block.x});
  return hipSuccess;
}
hipError_t hipGraphCreate(hipGraph_t*, unsigned) { return hipErrorNotSupported; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
}

// -------------------------------------------------------------- lattices
static mplb_t* make(int nx, int ny, int nz, int precision, int mode, std::vector<char>& arena, bool fill = true) {
  size_t need = 0;
  EXPECT(mplb_required_bytes(nx, ny, nz, precision, mode, &need) == MPLB_OK);
  arena.resize(need + 256);
  char* base = (char*)(((uintptr_t)arena.data() + 255) / 256 * 256);
  const int bc[3] = {0, 0, 0};
  mplb_t* h = nullptr;
  EXPECT(mplb_create(nx, ny, nz, bc, precision, mode, base, need, &h) == MPLB_OK);
  mplb_params p;
  std::memset(&p, 0, sizeof p);
  p.sigma = 1e-3; p.width = 4; p.rho_l = 2; p.rho_g = 1; p.mobility = 0.05; p.A = 0.25; p.nu = 0.1;
  for (double& s : p.s_f) s = 1;
  for (double& l : p.lambda_g) l = 1;
  EXPECT(mplb_set_params(h, &p) == MPLB_OK);
  std::vector<double> phi((size_t)nx * ny * nz, 0.5);
  EXPECT(mplb_init(h, phi.data(), nullptr) == MPLB_OK);
  for (size_t i = 0; i < need && fill; ++i) base[i] = (char)(i * 2654435761u >> 24);  // what a checkpoint has to bring
  return h;
}

// A checkpoint's arrays in the order in which a fresh lattice's arena holds
// them: f of level 0, g of level 0 and the history.
static bool checkpoint_matches(const std::vector<char>& arena, const std::vector<char>& out) {
  uint64_t bytes[3];
  const char* base = (const char*)(((uintptr_t)arena.data() + 255) / 256 * 256);
  const size_t head = 8 + 6 * 4 + 8 + 3 * 8;
  std::memcpy(bytes, out.data() + head - sizeof bytes, sizeof bytes);
  const size_t f = bytes[0], g = bytes[1], hist = bytes[2];
  return head + f + g + hist == out.size() && !std::memcmp(out.data() + head, base, f) &&
         !std::memcmp(out.data() + head + f, base + 2 * f, g) &&
         !std::memcmp(out.data() + head + f + g, base + 2 * f + 2 * g, hist);
}
static size_t checkpoint_bytes(mplb_t* h) {
  size_t n = 0;
  EXPECT(mplb_checkpoint_bytes(h, &n) == MPLB_OK);
  return n;
}

// No memory for the threads that copy a large array out: the calling thread
// copies it alone.
static void copy_without_memory() {
  std::vector<char> arena;
  mplb_t* h = make(64, 64, 100, MPLB_F64, MPLB_CHE_ONLY, arena);
  std::vector<char> out(checkpoint_bytes(h));
  no_memory = true;
  const int rc = mplb_checkpoint(h, out.data(), out.size());
  no_memory = false;
  EXPECT(rc == MPLB_OK && checkpoint_matches(arena, out));
  mplb_destroy(h);
}

// A lattice on a stream of another device than the caller's current one.
static void copy_from_another_device() {
  FakeStream other{1};
  for (int n : {8, 100}) {  // alone, and by several threads
    std::vector<char> arena;
    mplb_t* h = make(64, 64, n, MPLB_F64, MPLB_CHE_ONLY, arena);
    EXPECT(mplb_set_stream(h, &other) == MPLB_OK);
    std::vector<char> out(checkpoint_bytes(h));
    EXPECT(mplb_checkpoint(h, out.data(), out.size()) == MPLB_OK && checkpoint_matches(arena, out));
    EXPECT(current == 0);
    mplb_destroy(h);
  }
}

// No memory for the plan of a batch beyond 512 lattices: refused, and nothing
// has stepped.
static void batch_without_memory() {
  const int count = MPLB_NOALLOC_MAX_LATTICES + 1;
  std::vector<std::vector<char>> arena(count);
  std::vector<mplb_t*> hs;
  for (int i = 0; i < count; ++i) hs.push_back(make(2, 2, 2, MPLB_F32, MPLB_COUPLED, arena[i]));
  no_memory = true;
  int rc = -1;
  try {
    rc = mplb_step_many(hs.data(), count, 3);
  } catch (const std::bad_alloc&) {
  }
  no_memory = false;
  EXPECT(rc == MPLB_E_NOMEM && mplb_step_count(hs[0]) == 0 && mplb_step_count(hs[count - 1]) == 0);
  for (mplb_t* h : hs) mplb_destroy(h);
}

// Pinned staging is allocated for copies that it speeds up, and goes with the
// last lattice.
static void staging_of_short_lives() {
  std::vector<double> out(60 * 60 * 60);
  std::vector<char> arena;
  for (int life = 0; life < 3; ++life) {  // one small lattice at a time, read five times
    mplb_t* h = make(48, 48, 48, MPLB_F32, MPLB_COUPLED, arena);
    for (int f = MPLB_PHI; f <= MPLB_UY; ++f) EXPECT(mplb_read(h, f, out.data()) == MPLB_OK);
    mplb_destroy(h);
  }
  EXPECT(host_allocations == 0 && events_live == 0);
  mplb_t* h = make(60, 60, 60, MPLB_F32, MPLB_COUPLED, arena);
  for (int f = MPLB_PHI; f <= MPLB_UY; ++f) EXPECT(mplb_read(h, f, out.data()) == MPLB_OK);
  EXPECT(host_allocations == 1 && host_live == 1);
  mplb_destroy(h);
  EXPECT(host_live == 0 && events_live == 0);
}

// A read that allocates staging holds up no other.
static void staging_is_allocated_unlocked() {
  std::vector<char> a, b;
  mplb_t* large = make(64, 64, 64, MPLB_F32, MPLB_COUPLED, a);
  mplb_t* small = make(8, 8, 8, MPLB_F32, MPLB_COUPLED, b);
  std::vector<double> out(64 * 64 * 64), other(8 * 8 * 8);
  std::future<int> read;
  bool waited = true;
  during_host_malloc = [&] {
    read = std::async(std::launch::async, [&] { return mplb_read(small, MPLB_PHI, other.data()); });
    waited = read.wait_for(std::chrono::seconds(5)) != std::future_status::ready;
  };
  EXPECT(mplb_read(large, MPLB_PHI, out.data()) == MPLB_OK);
  during_host_malloc = nullptr;
  EXPECT(!waited && read.get() == MPLB_OK);
  mplb_destroy(large);
  mplb_destroy(small);
  EXPECT(host_live == 0 && events_live == 0);
}

// Into the caller's page-locked memory: one copy per array and no staging.
static void copy_to_page_locked() {
  std::vector<char> arena;
  mplb_t* h = make(64, 64, 100, MPLB_F64, MPLB_CHE_ONLY, arena);  // f and the history
  std::vector<char> out(checkpoint_bytes(h));
  locked_from = out.data();
  locked_to = out.data() + out.size();
  copies = 0;
  EXPECT(mplb_checkpoint(h, out.data(), out.size()) == MPLB_OK && checkpoint_matches(arena, out));
  EXPECT(host_allocations == 0 && copies == 2);
  mplb_destroy(h);
}

// Staging that cannot be had whole: the runtime's own copy, and nothing kept.
static void copy_without_events() {
  std::vector<char> arena;
  mplb_t* h = make(64, 64, 100, MPLB_F64, MPLB_CHE_ONLY, arena);
  std::vector<char> out(checkpoint_bytes(h));
  event_limit = 2;
  EXPECT(mplb_checkpoint(h, out.data(), out.size()) == MPLB_OK && checkpoint_matches(arena, out));
  EXPECT(host_allocations > 0 && events_live <= 2);
  mplb_destroy(h);
  EXPECT(host_live == 0 && events_live == 0);
}

// The launches of mplb_step are those that mplb_step_shape names, and the kinds
// that mplb_step_many_kinds names those of a batch's launches.
static const unsigned kThreads[8] = {512, 1024, 512, 512, 256, 512, 512, 1024};  // by kind
static void launches_are_the_shapes() {
  std::vector<char> arena;
  int seen[8] = {};
  const struct {
    int nx, ny, nz;
  } boxes[] = {{9, 8, 7}, {64, 48, 40}, {48, 48, 64}, {96, 33, 34}, {256, 250, 1}, {600, 520, 1}, {64, 64, 280},
               {176, 160, 160}, {64, 272, 260}, {1, 2200, 2100}};
  for (const auto& b : boxes)
    for (int prec = MPLB_F64; prec <= MPLB_F32_BF16; ++prec)
      for (int mode : {MPLB_COUPLED, MPLB_CHE_ONLY, MPLB_COUPLED_Q19}) {
        if (mode != MPLB_CHE_ONLY && (long)b.nx * b.ny * b.nz > 1500000) continue;  // (memory)
        if (mode == MPLB_CHE_ONLY && prec == MPLB_F32_BF16) continue;
        mplb_t* h = make(b.nx, b.ny, b.nz, prec, mode, arena, false);
        EXPECT(mplb_set_check_interval(h, 0) == MPLB_OK);
        for (int rows : {0, 8, 16})
          for (int n : {1, 6}) {
            const int bc[3] = {0, 0, 0};
            int shape[6], one[6];
            const int rc = mplb_step_shape(b.nx, b.ny, b.nz, bc, prec, mode, MPLB_VEL_ZERO, 0, rows, n, shape);
            EXPECT((rc == MPLB_OK) == (mplb_force_tile_rows(h, rows) == MPLB_OK));
            if (rc) continue;
            launches.clear();
            EXPECT(mplb_step(h, n) == MPLB_OK);
            ++seen[shape[0]];
            const bool pair = shape[0] == 7;
            EXPECT((int)launches.size() == (pair ? n - 2 : n));  // six steps: two pairs and two steps
            EXPECT(mplb_step_shape(b.nx, b.ny, b.nz, bc, prec, mode, MPLB_VEL_ZERO, 0, rows, 1, one) == MPLB_OK);
            for (size_t i = 0; i < launches.size(); ++i) {
              const int* s = pair && i >= 2 ? one : shape;
              EXPECT(launches[i].blocks == (unsigned)s[5] && launches[i].threads == kThreads[s[0]]);
            }
          }
        mplb_destroy(h);
      }
  for (int k : seen) EXPECT(k > 0);
}

static void batch_launches_are_the_kinds() {
  const struct {
    int prec, steps, nx, ny, nz, count, kind;
  } batches[] = {{MPLB_F32, 3, 32, 32, 32, 4, 6},        // small as a whole
                 {MPLB_F32, 1, 130, 128, 5, 9, 6},       // flat, but little idle
                 {MPLB_F32, 9, 64, 64, 1, 20, 4},        // idle work of 0.98 M nodes,
                 {MPLB_F32, 9, 64, 64, 1, 21, 0},        // 1.03 M
                 {MPLB_F64, 9, 64, 64, 5, 22, 4},        // in FP64 0.43 M,
                 {MPLB_F64, 9, 64, 64, 5, 23, 0},        // 0.45 M
                 {MPLB_F32, 7, 96, 96, 40, 4, 0},        // 295 MB in few steps,
                 {MPLB_F32, 8, 96, 96, 40, 4, 6},        // in enough for groups
                 {MPLB_F32_F16, 31, 64, 64, 64, 8, 0},   // 243 MB with 16-bit populations
                 {MPLB_F32_F16, 32, 64, 64, 64, 8, 6},
                 {MPLB_F32_BF16, 32, 48, 48, 64, 13, 5}};
  for (const auto& b : batches) {
    std::vector<std::vector<char>> arena(b.count);
    std::vector<mplb_t*> hs;
    for (int i = 0; i < b.count; ++i) hs.push_back(make(b.nx, b.ny, b.nz, b.prec, MPLB_COUPLED, arena[i], false));
    std::vector<int> kinds(b.count, -1);
    EXPECT(mplb_step_many_kinds(hs.data(), b.count, b.steps, kinds.data()) == MPLB_OK);
    for (int k : kinds) EXPECT(k == b.kind);
    launches.clear();
    EXPECT(mplb_step_many_noalloc(hs.data(), b.count, b.steps) == MPLB_OK);
    EXPECT(!launches.empty());
    for (const Launch& l : launches) EXPECT(l.threads == kThreads[b.kind]);
    for (mplb_t* h : hs) mplb_destroy(h);
  }
}

int main(int argc, char** argv) {
  const struct {
    const char* name;
    void (*run)();
  } cases[] = {{"copy_without_memory", copy_without_memory},
               {"batch_without_memory", batch_without_memory},
               {"copy_from_another_device", copy_from_another_device},
               {"copy_without_events", copy_without_events},
               {"copy_to_page_locked", copy_to_page_locked},
               {"launches_are_the_shapes", launches_are_the_shapes},
               {"batch_launches_are_the_kinds", batch_launches_are_the_kinds},
               {"staging_of_short_lives", staging_of_short_lives},
               {"staging_is_allocated_unlocked", staging_is_allocated_unlocked}};
  for (const auto& c : cases)
    if (argc == 2 && !std::strcmp(argv[1], c.name)) {
      c.run();
      std::puts(fails ? "FAILED" : "ok");
      return fails ? 1 : 0;
    }
  std::puts("no such case");
  return 2;
}
