// Single-node stand-in for the MM Store (paper section 3.2, "Multimodal Cache Pooling" and
// "Fault-Tolerant and Recomputation"): encoded features are kept in a device pool under the
// hash of the multimodal input; a hit returns the stored rows without running the encoder, a
// miss (never stored, or dropped to make room) recomputes them and stores them again.
//
// The paper names neither the hash nor the replacement rule; fixed here:
//   key   two polynomial hashes modulo P = 2^61 - 1 over the input as 32-bit little-endian
//         words (last word zero-padded) behind four header words (byte length low / high, salt
//         low / high):  H_k = sum_j (s_j + 1) R_k^(L - j) mod P.  Every term carries its own
//         power, so the sum can be taken in any order: exact integer arithmetic, bit for bit the
//         value a serial evaluation gives (how the kernel orders it: hash_partial_kernel).
//   pool  a byte arena behind a reserved area of 1 MiB (it held the partial hashes once; entries
//         stay where callers know them to be); entries are contiguous, 256-byte aligned; insert drops least-recently-used entries until a first-fit range
//         (lowest address) is free; a hit makes its entry the most recent.
// The bookkeeping is host code and touches no device memory; only epd_store_hash and
// epd_encode_cached launch work.  Pinned memory is allocated when a store is made, beside its pool, and not
// by its first hash: an allocation there would take 27 us of the call and break a stream capture that
// another thread has under way.
#include "../../include/epd_encode.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdarg>
#include <cstdio>
#include <list>
#include <map>
#include <mutex>
#include <string>
#include <vector>

namespace {

constexpr uint64_t kP = (1ull << 61) - 1;
constexpr uint64_t kBase0 = 0x1D4E2C1B3A596877ull % kP, kBase1 = 0x0F1E2D3C4B5A6978ull % kP;
constexpr uint64_t kAlign = 256;
constexpr uint64_t kScratchBytes = 1ull << 20;
constexpr int kRanges = 32;          // ranges per launch (descriptors travel as kernel arguments)
constexpr int kThreads = 256;
constexpr int kGroup = 4;            // 16-byte loads a thread has in flight = one group of 16 words
constexpr int kSpan = kThreads * 4;            // words a block covers with one load per thread
constexpr int kGroupWords = kSpan * kGroup;    // words a block covers per group (16 KB)
constexpr int kMaxBlocks = 4096;     // blocks per launch, all ranges together
constexpr uint64_t kAbsent = ~0ull;  // no hash: those are below 2^61
constexpr int kAimBlocks = 2048;     // blocks a launch is split into where the input allows

struct Key {
  uint64_t a, b;
  bool operator<(const Key& o) const { return a != o.a ? a < o.a : b < o.b; }
};
struct Entry { uint64_t off, bytes; std::list<Key>::iterator lru; };

std::string fmt(const char* f, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, f);
  vsnprintf(buf, sizeof buf, f, ap);
  va_end(ap);
  return buf;
}

// ---------------------------------------------------------------- arithmetic modulo 2^61 - 1
__host__ __device__ constexpr uint64_t addmod(uint64_t a, uint64_t b) {
  uint64_t r = a + b;                 // < 2^62
  return r >= kP ? r - kP : r;
}
__device__ inline uint64_t mulmod(uint64_t a, uint64_t b) {   // a, b < 2^61
  const uint64_t lo = a * b, hi = __umul64hi(a, b);           // 2^64 = 8 (mod P): a b = 8 hi + lo
  uint64_t r = (lo & kP) + ((lo >> 61) | (hi << 3));          // hi < 2^58
  r = (r & kP) + (r >> 61);
  return r >= kP ? r - kP : r;
}
constexpr uint64_t mulmod_const(uint64_t a, uint64_t b) {     // compile time
  return (uint64_t)((unsigned __int128)a * b % kP);
}
constexpr uint64_t powmod_const(uint64_t r, uint64_t e) {
  uint64_t acc = 1;
  for (; e; e >>= 1, r = mulmod_const(r, r))
    if (e & 1) acc = mulmod_const(acc, r);
  return acc;
}

// Powers the kernel multiplies by.  thread[k][t] moves a thread's sum to the end of its block's
// span, up / down[k][b] = R_k^(+-2^b) move a block's sum to the end of the range.
struct PowerTables {
  uint64_t thread[2][kThreads];
  uint64_t up[2][32], down[2][32];
};
constexpr PowerTables make_tables() {
  PowerTables t{};
  for (int k = 0; k < 2; ++k) {
    const uint64_t r = k ? kBase1 : kBase0, r4 = powmod_const(r, 4);
    uint64_t p = r;
    for (int i = kThreads - 1; i >= 0; --i) { t.thread[k][i] = p; p = mulmod_const(p, r4); }   // R^(4 (255 - t) + 1)
    uint64_t u = r, d = powmod_const(r, kP - 2);              // the inverse
    for (int b = 0; b < 32; ++b) {
      t.up[k][b] = u; t.down[k][b] = d;
      u = mulmod_const(u, u); d = mulmod_const(d, d);
    }
  }
  return t;
}
__constant__ const PowerTables kTables = make_tables();

// Weights of the 16 words of a group, R^(kSpan (3 - i) + 3 - c) for word c of load i, in limbs of
// 21, 20 and 20 bits: a 32-bit word times a limb stays below 2^53, so all products of a group add up
// in 64 bits without any reduction between them -- three multiply-adds per word and hash.
struct GroupWeights {
  uint32_t limb[kGroup * 4][3];
  uint64_t sum;                  // of all weights: the "+ 1" of every word
  uint64_t step;                 // R^kGroupWords
};
constexpr GroupWeights make_weights(uint64_t r) {
  GroupWeights w{};
  for (int i = 0; i < kGroup; ++i)
    for (int c = 0; c < 4; ++c) {
      const uint64_t v = powmod_const(r, (uint64_t)kSpan * (kGroup - 1 - i) + 3 - c);
      w.limb[i * 4 + c][0] = (uint32_t)(v & ((1u << 21) - 1));
      w.limb[i * 4 + c][1] = (uint32_t)((v >> 21) & ((1u << 20) - 1));
      w.limb[i * 4 + c][2] = (uint32_t)(v >> 41);
      w.sum = addmod(w.sum, v);
    }
  w.step = powmod_const(r, kGroupWords);
  return w;
}

struct HashRange {
  const uint8_t* data;
  int64_t bytes;
  uint64_t salt;
  uint32_t words;            // ceil(bytes / 4)
  uint32_t groups;           // groups of kGroupWords words per block
  uint32_t first_block;      // first block of this range in the launch (>= 1 block per range)
};
struct HashArgs {
  int n;
  uint64_t* partial;         // [blocks of the launch][2]
  uint64_t* result;          // [n][2] (hash_final_kernel)
  uint32_t blocks;
  HashRange r[kRanges];
};

__device__ inline uint64_t wave_addmod(uint64_t v, int from) {   // sum over lanes that differ in the bits below `from * 2`
  for (int o = from; o > 0; o >>= 1) v = addmod(v, __shfl_xor((unsigned long long)v, o));
  return v;
}

// R_k^e (e may be negative) by half-wave k = lane / 32, one bit of |e| per lane: five multiplications
// deep, against 62 for square-and-multiply
__device__ inline uint64_t half_wave_power(int64_t e) {
  const int lane = threadIdx.x & 63, b = lane & 31, k = lane >> 5;
  const uint64_t m = (uint64_t)(e < 0 ? -e : e);
  uint64_t v = (m >> b) & 1 ? (e < 0 ? kTables.down[k][b] : kTables.up[k][b]) : 1;
  for (int o = 16; o > 0; o >>= 1) v = mulmod(v, __shfl_xor((unsigned long long)v, o));
  return v;
}

// a += w * weights of group word J, limb by limb
template <int J> __device__ inline void add_word(uint64_t (&a)[2][3], uint32_t w) {
  constexpr GroupWeights g0 = make_weights(kBase0), g1 = make_weights(kBase1);
#pragma unroll
  for (int l = 0; l < 3; ++l) {
    a[0][l] += (uint64_t)w * g0.limb[J][l];
    a[1][l] += (uint64_t)w * g1.limb[J][l];
  }
}
__device__ inline uint64_t fold_limbs(const uint64_t (&a)[3]) {   // a[0] + a[1] 2^21 + a[2] 2^41 mod P, each < 2^57
  uint64_t r = (a[0] & kP) + ((a[1] << 21) & kP) + (a[1] >> 40);
  r = (r & kP) + (r >> 61);
  r += ((a[2] << 41) & kP) + (a[2] >> 20);
  r = (r & kP) + (r >> 61);
  return r >= kP ? r - kP : r;
}

// a += the words of v that exist and their "+ 1"; bit J of `present` = word J lies in the range
template <int J> __device__ inline void add_present(uint64_t (&a)[2][3], const uint32_t (&v)[kGroup * 4], uint32_t present) {
  if constexpr (J < kGroup * 4) {
    const uint32_t one = (present >> J) & 1u;
    add_word<J>(a, one ? v[J] : 0u);
    add_word<J>(a, one);
    add_present<J + 1>(a, v, present);
  }
}

typedef uint32_t u32_any __attribute__((aligned(1)));
typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(1)));

// Bound: integer multiply-adds (v_mad_u64_u32, quarter rate) and HBM about equally.  A block takes
// `groups` groups of 16 KB; a thread has its four 16-byte loads of a group in flight together (any
// byte alignment), folds the 16 words with constant weights (six multiply-adds per word for both
// hashes) and steps its Horner sum by one modular product per group.  The first form -- one thread
// folding 64 consecutive words with a modular product per word, then square-and-multiply for its
// position -- took 61 us for four 9.6 MB clips and 35 us for eight 0.6 MB images (80 blocks); this
// one 13.0 us (3.0 TB/s) and 7.8 us (304 blocks; launch, one round of loads and the block's
// reduction).
__global__ __launch_bounds__(kThreads) void hash_partial_kernel(HashArgs a) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // the range of this block: every lane compares with one range's first block
  const int ri = __popcll(__ballot(lane < a.n && a.r[lane < kRanges ? lane : 0].first_block <= blockIdx.x)) - 1;
  const HashRange g = a.r[__builtin_amdgcn_readfirstlane(ri)];
  const uint32_t blk = blockIdx.x - g.first_block;
  const int64_t wb = (int64_t)blk * g.groups * kGroupWords, we = wb + (int64_t)g.groups * kGroupWords;
  constexpr GroupWeights g0 = make_weights(kBase0), g1 = make_weights(kBase1);
  uint64_t h0 = 0, h1 = 0;
  for (uint32_t q = 0; q < g.groups; ++q) {
    const int64_t w0 = wb + (int64_t)q * kGroupWords;          // first word of the group
    uint64_t acc[2][3] = {};
    uint64_t s0, s1;
    if (w0 + kGroupWords <= (g.bytes >> 2)) {         // whole words only
      const uint8_t* p = g.data + (w0 + tid * 4) * 4;
      u32x4_any v[kGroup];
#pragma unroll
      for (int i = 0; i < kGroup; ++i) v[i] = *(const u32x4_any*)(p + (size_t)i * kSpan * 4);
#define EPD_HASH_LOAD(I) \
      add_word<I * 4>(acc, v[I][0]); add_word<I * 4 + 1>(acc, v[I][1]); add_word<I * 4 + 2>(acc, v[I][2]); add_word<I * 4 + 3>(acc, v[I][3]);
      EPD_HASH_LOAD(0) EPD_HASH_LOAD(1) EPD_HASH_LOAD(2) EPD_HASH_LOAD(3)
#undef EPD_HASH_LOAD
      s0 = addmod(fold_limbs(acc[0]), g0.sum);
      s1 = addmod(fold_limbs(acc[1]), g1.sum);
    } else {                                                   // the range ends inside (or before) this group
      // a word that the range ends in is taken from the range's last four bytes, shifted; all loads
      // are issued before the first is used
      uint32_t v[kGroup * 4] = {}, present = 0;
      if (g.bytes >= 4) {
        const int64_t at0 = min(w0 * 4, g.bytes - 4);          // where the addresses below count from
        const uint32_t ahead = (uint32_t)min(w0 * 4 - at0, (int64_t)4), last = (uint32_t)min(g.bytes - 4 - at0, (int64_t)kGroupWords * 4);
        const uint32_t words = (uint32_t)max((int64_t)0, min((int64_t)g.words - w0, (int64_t)kGroupWords));
#pragma unroll
        for (int j = 0; j < kGroup * 4; ++j) v[j] = *(const u32_any*)(g.data + at0 + min(4u * ((j / 4) * kSpan + tid * 4 + j % 4) + ahead, last));
#pragma unroll
        for (int j = 0; j < kGroup * 4; ++j) {
          const uint32_t w = (j / 4) * kSpan + tid * 4 + j % 4, byte = w * 4 + ahead;
          if (w < words) present |= 1u << j;
          if (byte > last) v[j] >>= 8u * ((byte - last) & 3u);
        }
      } else if (tid == 0 && w0 == 0) {
        for (int i = 0; i < (int)g.bytes; ++i) v[0] |= (uint32_t)g.data[i] << (8 * i);
        present = g.bytes ? 1u : 0u;
      }
      add_present<0>(acc, v, present);
      s0 = fold_limbs(acc[0]);
      s1 = fold_limbs(acc[1]);
    }
    h0 = q ? addmod(mulmod(h0, g0.step), s0) : s0;
    h1 = q ? addmod(mulmod(h1, g1.step), s1) : s1;
  }
  h0 = wave_addmod(mulmod(h0, kTables.thread[0][tid]), 32);
  h1 = wave_addmod(mulmod(h1, kTables.thread[1][tid]), 32);
  __shared__ uint64_t sum[2][kThreads / 64], head[2];
  if (lane == 0) { sum[0][wave] = h0; sum[1][wave] = h1; }
  if (blk == 0 && wave == 1) {
    // header words s_0 .. s_3 stand in front of all data words: powers words + 4 .. words + 1
    const int k = lane >> 5;
    const uint64_t hdr[4] = {(uint64_t)g.bytes & 0xffffffffull, (uint64_t)g.bytes >> 32, g.salt & 0xffffffffull, g.salt >> 32};
    uint64_t t = 0;
    for (int j = 0; j < 4; ++j) t = mulmod(addmod(t, hdr[j] + 1), k ? kBase1 : kBase0);
    t = mulmod(t, half_wave_power((int64_t)g.words));
    if ((lane & 31) == 0) head[k] = t;
  }
  __syncthreads();
  if (wave == 0) {
    const int k = lane >> 5;
    uint64_t v = addmod(addmod(sum[k][0], sum[k][1]), addmod(sum[k][2], sum[k][3]));
    v = mulmod(v, half_wave_power((int64_t)g.words - we));     // negative where the last block runs past the range
    if (blk == 0) v = addmod(v, head[k]);
    // system scope: in host memory the host sees the value as soon as it is there, not at the kernel's end
    if ((lane & 31) == 0) __hip_atomic_store(a.partial + (size_t)blockIdx.x * 2 + k, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}
static_assert(kThreads == 256 && kGroup == 4, "the kernel above is written for four waves and four loads per group");

// one wave per range: modular sum of its blocks' partial hashes
__global__ __launch_bounds__(64) void hash_final_kernel(HashArgs a) {
  const uint32_t b0 = a.r[blockIdx.x].first_block, b1 = (int)blockIdx.x + 1 < a.n ? a.r[blockIdx.x + 1].first_block : a.blocks;
  uint64_t h0 = 0, h1 = 0;
  for (uint32_t b = b0 + threadIdx.x; b < b1; b += 64) {
    h0 = addmod(h0, a.partial[(size_t)b * 2]);
    h1 = addmod(h1, a.partial[(size_t)b * 2 + 1]);
  }
  h0 = wave_addmod(h0, 32);
  h1 = wave_addmod(h1, 32);
  if (threadIdx.x == 0) {
    a.result[blockIdx.x * 2] = h0;
    a.result[blockIdx.x * 2 + 1] = h1;
  }
}

// Partial-hash scratch of epd_store_hash_noalloc: one slot pair per block of one launch.
// Every GPU the library runs on holds its own copy of this array, at its own address, until the
// process ends.  In host code the name is only a handle for hipGetSymbolAddress -- it is not a
// device address and never goes into a kernel argument or a copy.
constexpr size_t kStaticScratchWords = (size_t)kMaxBlocks * 2;
static __device__ __align__(256) uint64_t scratch[kStaticScratchWords];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
uint64_t* g_scratch_ptr[kMaxDevices] = {};     // device address of `scratch` on each device, once known

}  // namespace

struct epd_store {
  char* pool = nullptr;          // device; [0, kScratchBytes) reserved, entries behind it
  uint64_t* partial = nullptr;   // pinned host memory: partial hashes of one launch, written by the kernel
  std::vector<uint64_t*> given_up;         // earlier ones that a kernel may still write, freed at destroy
  uint64_t arena = 0;            // bytes available to entries (multiple of kAlign)
  std::map<Key, Entry> entries;
  std::map<uint64_t, uint64_t> by_off;     // offset -> rounded size
  std::list<Key> lru;                      // front = least recently used
  uint64_t hits = 0, misses = 0, evictions = 0;
  std::string err;
};

namespace {

thread_local std::string g_store_error = "";

uint64_t round_up(uint64_t n) { return (n + kAlign - 1) / kAlign * kAlign; }

// lowest offset of a free range of `need` bytes, or UINT64_MAX
uint64_t first_fit(const epd_store* s, uint64_t need) {
  uint64_t pos = 0;
  for (const auto& kv : s->by_off) {
    if (kv.first - pos >= need) return pos;
    pos = kv.first + kv.second;
  }
  return s->arena - pos >= need ? pos : UINT64_MAX;
}

hipError_t pin_partials(epd_store* s) {
  if (s->partial) return hipSuccess;
  // coherent whatever the environment says: the host reads and resets slots while the kernel runs, and
  // a late write-back over a reset slot would be read as the next launch's sum
  const hipError_t e = hipHostMalloc((void**)&s->partial, (size_t)kMaxBlocks * 16, hipHostMallocPortable | hipHostMallocCoherent);
  if (e != hipSuccess) { s->partial = nullptr; (void)hipGetLastError(); return e; }
  std::fill(s->partial, s->partial + (size_t)kMaxBlocks * 2, kAbsent);
  return e;
}

// A launch whose end could not be waited for may write its slots at any time: they are given up, so
// that no later call takes those sums for its own, and the next call gets others.
void give_up_partials(epd_store* s) {
  s->given_up.push_back(s->partial);
  s->partial = nullptr;
}

// Sum of the `count` pairs at p, each waited for and then marked absent again for the next launch.
// The host looks for the values themselves -- they arrive within microseconds, sooner than the
// runtime reports the stream idle -- and after `patience` looks in vain asks the runtime instead
// (a long queue ahead of the kernel, or a fault, which it reports).
hipError_t take_partials(uint64_t* p, uint32_t count, hipStream_t st, bool& synced, uint64_t key[2]) {
  uint64_t h[2] = {0, 0};
  for (uint32_t i = 0; i < count * 2; ++i) {
    uint64_t v;
    int patience = 100000;
    while ((v = __atomic_load_n(p + i, __ATOMIC_ACQUIRE)) == kAbsent) {
      if (synced) return hipErrorUnknown;              // the kernel has ended without writing it
      if (--patience > 0) continue;
      if (hipError_t e = hipStreamSynchronize(st)) return e;
      synced = true;
    }
    p[i] = kAbsent;
    h[i & 1] = addmod(h[i & 1], v);
  }
  key[0] = h[0];
  key[1] = h[1];
  return hipSuccess;
}

void drop(epd_store* s, std::map<Key, Entry>::iterator it) {
  s->by_off.erase(it->second.off);
  s->lru.erase(it->second.lru);
  s->entries.erase(it);
}

}  // namespace

extern "C" {

epd_status epd_store_create(void* device_pool, uint64_t pool_bytes, epd_store_handle* out) {
  if (!out) { g_store_error = "out is NULL"; return EPD_ERR_INVALID_ARG; }
  if (!device_pool || ((uintptr_t)device_pool % kAlign)) {
    g_store_error = "pool is NULL or not 256-byte aligned"; return EPD_ERR_INVALID_ARG;
  }
  if (pool_bytes < kScratchBytes + kAlign) {
    g_store_error = fmt("pool of %llu bytes is smaller than the %llu-byte scratch area plus one entry",
                        (unsigned long long)pool_bytes, (unsigned long long)kScratchBytes);
    return EPD_ERR_WORKSPACE;
  }
  epd_store* s = new epd_store();
  s->pool = (char*)device_pool;
  s->arena = (pool_bytes - kScratchBytes) / kAlign * kAlign;
  (void)pin_partials(s);         // without a GPU (bookkeeping only) this fails; epd_store_hash asks again
  *out = s;
  return EPD_OK;
}

epd_status epd_store_destroy(epd_store_handle s) {
  if (s && s->partial) (void)hipHostFree(s->partial);
  if (s) for (uint64_t* p : s->given_up) (void)hipHostFree(p);
  delete s;
  return EPD_OK;
}

const char* epd_store_last_error(epd_store_handle s) { return s ? s->err.c_str() : g_store_error.c_str(); }

epd_status epd_store_lookup(epd_store_handle s, const uint64_t key[2], void** device_ptr, uint64_t* bytes) {
  if (!s) { g_store_error = "store is NULL"; return EPD_ERR_INVALID_ARG; }
  if (!key || !device_ptr) { s->err = "a required pointer is NULL"; return EPD_ERR_INVALID_ARG; }
  auto it = s->entries.find(Key{key[0], key[1]});
  if (it == s->entries.end()) { ++s->misses; *device_ptr = nullptr; if (bytes) *bytes = 0; return EPD_MISS; }
  ++s->hits;
  s->lru.splice(s->lru.end(), s->lru, it->second.lru);       // most recent at the back
  *device_ptr = s->pool + kScratchBytes + it->second.off;
  if (bytes) *bytes = it->second.bytes;
  return EPD_OK;
}

epd_status epd_store_insert(epd_store_handle s, const uint64_t key[2], uint64_t bytes, void** device_ptr) {
  if (!s) { g_store_error = "store is NULL"; return EPD_ERR_INVALID_ARG; }
  if (!key || !device_ptr) { s->err = "a required pointer is NULL"; return EPD_ERR_INVALID_ARG; }
  const uint64_t need = round_up(bytes);
  if (bytes == 0 || need > s->arena) {
    s->err = fmt("an entry of %llu bytes can never fit a pool of %llu", (unsigned long long)bytes,
                 (unsigned long long)s->arena);
    *device_ptr = nullptr;
    return EPD_ERR_WORKSPACE;
  }
  const Key k{key[0], key[1]};
  auto old = s->entries.find(k);
  if (old != s->entries.end()) drop(s, old);
  uint64_t off;
  while ((off = first_fit(s, need)) == UINT64_MAX) {
    drop(s, s->entries.find(s->lru.front()));
    ++s->evictions;
  }
  s->lru.push_back(k);
  s->entries[k] = Entry{off, bytes, std::prev(s->lru.end())};
  s->by_off[off] = need;
  *device_ptr = s->pool + kScratchBytes + off;
  return EPD_OK;
}

epd_status epd_store_stats(epd_store_handle s, uint64_t* hits, uint64_t* misses, uint64_t* evictions, uint64_t* entries) {
  if (!s) { g_store_error = "store is NULL"; return EPD_ERR_INVALID_ARG; }
  if (hits) *hits = s->hits;
  if (misses) *misses = s->misses;
  if (evictions) *evictions = s->evictions;
  if (entries) *entries = s->entries.size();
  return EPD_OK;
}

// Describes ranges [i0, i0 + m) in `a` and launches the hash kernel for them; partial hashes go to
// a.partial (set by the caller).  Returns the launch's own status: the runtime's last error may be one
// that the program left behind long before, and the kernel runs all the same.
// Blocks take as many 16 KB groups as keep the launch at about kAimBlocks blocks (two or more waves
// on every SIMD): one group each up to 32 MB, where a block's fixed part -- its reduction and its
// power -- costs about as much as a group.
static hipError_t launch_hash(HashArgs& a, const void* device_data, const uint64_t* offsets, const uint64_t* salts, int i0, int m,
                              hipStream_t st) {
  uint64_t total = 0;
  for (int j = 0; j < m; ++j) total += (offsets[i0 + j + 1] - offsets[i0 + j]) / 4 / kGroupWords + 1;
  const uint32_t groups = (uint32_t)((total + kAimBlocks - 1) / kAimBlocks);
  uint32_t blocks = 0;
  for (int j = 0; j < m; ++j) {
    HashRange& r = a.r[j];
    r.data = (const uint8_t*)device_data + offsets[i0 + j];
    r.bytes = (int64_t)(offsets[i0 + j + 1] - offsets[i0 + j]);
    r.salt = salts[i0 + j];
    r.words = (uint32_t)((r.bytes + 3) / 4);
    r.groups = groups;
    r.first_block = blocks;
    const uint64_t span = (uint64_t)groups * kGroupWords;
    blocks += std::max<uint32_t>(1u, (uint32_t)(((uint64_t)r.words + span - 1) / span));   // <= kAimBlocks + 2 kRanges in all
  }
  a.n = m;
  a.blocks = blocks;
  void* args[] = {&a};
  return hipLaunchKernel((const void*)hash_partial_kernel, dim3(blocks), dim3(kThreads), args, 0, st);
}
static_assert(kAimBlocks + 2 * kRanges <= kMaxBlocks, "partial hashes of one launch");

static bool ranges_ok(const uint64_t* offsets, int n, std::string& err) {
  for (int i = 0; i < n; ++i)
    if (offsets[i + 1] < offsets[i] || offsets[i + 1] - offsets[i] >= (1ull << 33)) {
      err = fmt("range %d: offsets must not decrease and a range holds less than 8 GiB", i);
      return false;
    }
  return true;
}

epd_status epd_store_hash(epd_store_handle s, const void* device_data, const uint64_t* offsets, const uint64_t* salts,
                          int32_t n, uint64_t* keys_out, void* stream) {
  if (!s) { g_store_error = "store is NULL"; return EPD_ERR_INVALID_ARG; }
  if (!device_data || !offsets || !salts || !keys_out || n <= 0) {
    s->err = "a required pointer is NULL or n <= 0"; return EPD_ERR_INVALID_ARG;
  }
  if (!ranges_ok(offsets, n, s->err)) return EPD_ERR_SHAPE;
  hipStream_t st = (hipStream_t)stream;
  // a captured launch would run again with every replay, when nobody takes its sums
  hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
  hipError_t e = hipStreamIsCapturing(st, &capture);
  if (e != hipSuccess || capture != hipStreamCaptureStatusNone) {
    s->err = e != hipSuccess ? fmt("hipStreamIsCapturing: %s", hipGetErrorString(e)) : "the stream is being captured: the call waits for its keys";
    return EPD_ERR_HIP;
  }
  e = pin_partials(s);
  if (e != hipSuccess) { s->err = fmt("pinned memory for the partial hashes: %s", hipGetErrorString(e)); return EPD_ERR_HIP; }
  // The kernel leaves its blocks' partial hashes in host memory and the host adds them up: no second
  // kernel, no copy (the host has to wait for the keys anyway -- they decide what is launched next).
  // A call on four 9.6 MB clips: 92 us with a second kernel, a copy and a wait for the stream (61 us of
  // it in the first form of the kernel), 33 us with the wait only, 28 us taking the values as they come.
  HashArgs a{};
  a.partial = s->partial;
  for (int i0 = 0; i0 < n; i0 += kRanges) {
    const int m = n - i0 < kRanges ? n - i0 : kRanges;
    e = launch_hash(a, device_data, offsets, salts, i0, m, st);
    if (e != hipSuccess) { s->err = fmt("hash launch failed: %s", hipGetErrorString(e)); return EPD_ERR_HIP; }   // nothing was queued
    bool synced = false;
    for (int j = 0; j < m && e == hipSuccess; ++j) {
      const uint32_t b0 = a.r[j].first_block, b1 = j + 1 < m ? a.r[j + 1].first_block : a.blocks;
      e = take_partials(s->partial + (size_t)b0 * 2, b1 - b0, st, synced, keys_out + (size_t)(i0 + j) * 2);
    }
    if (e != hipSuccess) {
      give_up_partials(s);
      s->err = fmt("waiting for the hash kernel failed: %s", hipGetErrorString(e)); return EPD_ERR_HIP;
    }
  }
  return EPD_OK;
}

// The same keys for callers that cannot allocate: the partial hashes go to the library's own
// static device array instead of a pool, the keys to a device buffer of the caller, and the host
// is not waited for.  Nothing here allocates or frees memory (device or pinned), copies, or
// synchronises; the two launches are all the GPU work.
epd_status epd_store_hash_noalloc(const void* device_data, const uint64_t* offsets, const uint64_t* salts, int32_t n,
                                  uint64_t* keys_device_out, void* stream) {
  if (!device_data || !offsets || !salts || !keys_device_out || n <= 0) {
    g_store_error = "a required pointer is NULL or n <= 0"; return EPD_ERR_INVALID_ARG;
  }
  if (n > kRanges) {
    g_store_error = fmt("%d ranges: one call of epd_store_hash_noalloc takes at most %d (its scratch array holds that many)", n, kRanges);
    return EPD_ERR_SHAPE;
  }
  if (!ranges_ok(offsets, n, g_store_error)) return EPD_ERR_SHAPE;
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess || dev < 0 || dev >= kMaxDevices) {
    g_store_error = fmt("no usable current device (%s, device %d)", hipGetErrorString(e), dev); return EPD_ERR_HIP;
  }
  uint64_t* ptr;
  {
    // first call on this device: ask the runtime where this device keeps its copy of the array
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
      void* p = nullptr;
      e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
      if (e != hipSuccess || !p) {
        g_store_error = fmt("hipGetSymbolAddress(scratch) failed on device %d: %s", dev, hipGetErrorString(e)); return EPD_ERR_HIP;
      }
      g_scratch_ptr[dev] = (uint64_t*)p;
    }
    ptr = g_scratch_ptr[dev];
  }
  // Nothing in the array has to start at zero: the first kernel writes the slot of every block the
  // second one reads, so the previous call's contents are simply overwritten.
  HashArgs a{};
  a.partial = ptr;
  a.result = keys_device_out;
  (void)launch_hash(a, device_data, offsets, salts, 0, n, (hipStream_t)stream);   // a failure shows below
  hipLaunchKernelGGL(hash_final_kernel, dim3(n), dim3(64), 0, (hipStream_t)stream, a);
  e = hipGetLastError();
  if (e != hipSuccess) { g_store_error = fmt("hash launch failed: %s", hipGetErrorString(e)); return EPD_ERR_HIP; }
  return EPD_OK;
}

}  // extern "C"
