// A stand-in for the HIP runtime, for tests of host logic on machines without a GPU: loaded in front of
// the real runtime, it takes the built library's runtime calls, records its launches and answers as
// the test asks.  No kernel runs; of the store's hash kernel it does what the kernel is specified to
// do (the sums of one launch appear in `partial`), at once or when the stream is next waited for.
// HashRange / HashArgs repeat the layout of paper_2601_11590_amd/csrc/mm_store.hip.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

namespace {
struct Dim3 { uint32_t x, y, z; };
struct HashRange { const uint8_t* data; int64_t bytes; uint64_t salt; uint32_t words, groups, first_block; };
struct HashArgs { int n; uint64_t* partial; uint64_t* result; uint32_t blocks; HashRange r[32]; };

struct Launch { std::string name; Dim3 grid, block; std::string args; };
std::map<const void*, std::string> g_names;
std::vector<Launch> g_launches;
std::vector<std::pair<uint64_t*, uint64_t>> g_late;      // stores of a kernel that still runs
std::map<std::string, long long> g_calls;
long long g_set[8];                                      // see fake_set
enum { kLastError, kCapture, kLate, kLaunchStatus, kSyncStatus, kHostFlags };

std::string g_refuse;                                    // see fake_refuse
int g_refuse_status = 0;
std::string g_keep;                                      // see fake_keep_args
size_t g_keep_bytes = 0;

constexpr uint64_t kP = (1ull << 61) - 1;
uint64_t mul(uint64_t a, uint64_t b) { return (uint64_t)((unsigned __int128)a * b % kP); }

uint64_t hash(const HashRange& r, uint64_t base) {
  uint64_t h = 0;
  auto add = [&](uint64_t w) { h = mul((h + w + 1) % kP, base); };
  add((uint64_t)r.bytes & 0xffffffffu); add((uint64_t)r.bytes >> 32); add(r.salt & 0xffffffffu); add(r.salt >> 32);
  for (int64_t i = 0; i < r.bytes; i += 4) {
    uint32_t w = 0;
    std::memcpy(&w, r.data + i, (size_t)(r.bytes - i < 4 ? r.bytes - i : 4));
    add(w);
  }
  return h;
}

void drain() {
  for (auto& s : g_late) __atomic_store_n(s.first, s.second, __ATOMIC_RELEASE);
  g_late.clear();
}

Dim3 g_grid, g_block;
size_t g_shmem;
void* g_stream;
}  // namespace

extern "C" {

// what: 0 = the thread's uncollected last error, 1 = capture status of every stream, 2 = stores of
// kernels appear late (at the next wait), 3 / 4 = status of launches / of waits for a stream
void fake_set(int what, long long value) { g_set[what] = value; }
// launches of kernels whose name holds `part` fail with `status`
void fake_refuse(const char* part, int status) { g_refuse = part; g_refuse_status = status; }
// launches of kernels whose name holds `part` keep the first `bytes` of their argument for fake_args
void fake_keep_args(const char* part, size_t bytes) { g_keep = part; g_keep_bytes = bytes; }
const void* fake_args(int i) { return g_launches[i].args.data(); }
long long fake_get(int what) { return g_set[what]; }
void fake_drain() { drain(); }
long long fake_calls(const char* name) { return g_calls[name]; }
int fake_all_calls() { int n = 0; for (auto& c : g_calls) n += (int)c.second; return n; }
int fake_launches() { return (int)g_launches.size(); }
void fake_forget() { g_launches.clear(); g_calls.clear(); }
// launch i: name, grid and block sizes
const char* fake_launch(int i, uint32_t* sizes) {
  const Launch& l = g_launches[i];
  const uint32_t v[6] = {l.grid.x, l.grid.y, l.grid.z, l.block.x, l.block.y, l.block.z};
  std::memcpy(sizes, v, sizeof v);
  return l.name.c_str();
}

#define CALL() (++g_calls[__func__])

void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) { g_names[host] = name; }
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim3 g, Dim3 b, size_t s, void* st) { g_grid = g; g_block = b; g_shmem = s; g_stream = st; return 0; }
int __hipPopCallConfiguration(Dim3* g, Dim3* b, size_t* s, void** st) { *g = g_grid; *b = g_block; *s = g_shmem; *st = g_stream; return 0; }

int hipLaunchKernel(const void* f, Dim3 grid, Dim3 block, void** args, size_t, void*) {
  CALL();
  if (g_set[kLaunchStatus]) { g_set[kLastError] = g_set[kLaunchStatus]; return (int)g_set[kLaunchStatus]; }
  if (!g_refuse.empty() && g_names[f].find(g_refuse) != std::string::npos) { g_set[kLastError] = g_refuse_status; return g_refuse_status; }
  g_launches.push_back({g_names[f], grid, block, {}});
  if (g_keep_bytes && g_names[f].find(g_keep) != std::string::npos) g_launches.back().args.assign((const char*)args[0], g_keep_bytes);
  if (g_names[f].find("hash_partial_kernel") != std::string::npos) {
    HashArgs a;
    std::memcpy(&a, args[0], sizeof a);
    const uint64_t base[2] = {0x1D4E2C1B3A596877ull % kP, 0x0F1E2D3C4B5A6978ull % kP};
    std::vector<uint64_t> sums((size_t)a.blocks * 2, 0);
    for (int i = 0; i < a.n; ++i)
      for (int k = 0; k < 2; ++k) sums[(size_t)a.r[i].first_block * 2 + k] = hash(a.r[i], base[k]);
    for (size_t i = 0; i < sums.size(); ++i) g_late.push_back({a.partial + i, sums[i]});
    if (!g_set[kLate]) drain();
  }
  return 0;
}
int hipStreamSynchronize(void*) {
  CALL();
  if (g_set[kSyncStatus]) return (int)g_set[kSyncStatus];
  drain();
  return 0;
}
int hipStreamIsCapturing(void*, int* status) { CALL(); *status = (int)g_set[kCapture]; return 0; }
int hipGetLastError() { CALL(); const int e = (int)g_set[kLastError]; g_set[kLastError] = 0; return e; }
const char* hipGetErrorString(int e) { static char b[32]; std::snprintf(b, sizeof b, "fake error %d", e); return b; }
int hipHostMalloc(void** p, size_t n, unsigned flags) { CALL(); g_set[kHostFlags] = flags; *p = std::calloc(n, 1); return 0; }
int hipHostFree(void* p) { CALL(); std::free(p); return 0; }
int hipGetDevice(int* d) { CALL(); *d = 0; return 0; }
int hipDeviceGetAttribute(int* v, int, int) { CALL(); *v = 256; return 0; }
int hipGetSymbolAddress(void** p, const void*) { static uint64_t area[1 << 17]; CALL(); *p = area; return 0; }
int hipMemcpy(void*, const void*, size_t, int) { CALL(); return 0; }
int hipMemcpyAsync(void*, const void*, size_t, int, void*) { CALL(); return 0; }
int hipMemcpy2DAsync(void*, size_t, const void*, size_t, size_t, size_t, int, void*) { CALL(); return 0; }
int hipMemsetAsync(void*, int, size_t, void*) { CALL(); return 0; }
int hipEventCreate(void** e) { CALL(); *e = (void*)1; return 0; }
int hipEventCreateWithFlags(void** e, unsigned) { CALL(); *e = (void*)1; return 0; }
int hipEventDestroy(void*) { CALL(); return 0; }
int hipEventRecord(void*, void*) { CALL(); return 0; }
int hipEventSynchronize(void*) { CALL(); return 0; }
int hipEventElapsedTime(float* ms, void*, void*) { CALL(); *ms = 0.f; return 0; }

}  // extern "C"
