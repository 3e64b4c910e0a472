// The step in front of the encoder (paper section 3.1: the Encode stage takes the raw
// multimodal input I_m): uint8 pixels -> bilinear resize to the item's patch grid ->
// per-channel normalise -> packed patch rows, the A operand of the patch-embedding GEMM.
//
// The paper does not say how I_m becomes encoder input; this kernel fixes: planar uint8
// frames [C, t*tp, Hs, Ws] per item, bilinear taps at half-pixel centres with the source
// coordinate clamped to the image (no antialiasing, no resampling in time), value
// (v / 255 - mean_c) / std_c, row layout (channel, frame in patch, row in patch, column in
// patch), tokens in raster order over (t, h, w).
//
// Bound: HBM (1 byte in per source pixel, 2 or 4 bytes out per element) once enough loads are in
// flight.  The tap positions are exact integer arithmetic, (2j + 1) * n_in - n_out over 2 * n_out,
// so that equal sizes copy pixels untouched and the weights carry a single rounding.
#include "epd_internal.h"

#include <algorithm>

namespace epd {

struct Tap { int i0; float w1; };

// taps of output sample j along an axis of n_in source and n_out output samples: i0 and i0 + 1
// (clamped by the caller), the second weighted w1.  inv = 1 / (2 n_out): the quotient of the float
// product is off by at most one (it stays below 2^14), which the remainder shows.  The weight is a
// true division (remainder times inv would be rounded twice: mean error 2.2e-8 instead of 0.8e-8).
__device__ __forceinline__ Tap tap(int j, int n_in, int n_out, float inv) {
  const int num = max((2 * j + 1) * n_in - n_out, 0), den = 2 * n_out;
  int q = (int)((float)num * inv), r = num - q * den;
  if (r < 0) { --q; r += den; }
  if (r >= den) { ++q; r -= den; }
  Tap t;
  t.i0 = min(q, n_in - 1);
  t.w1 = (float)r / (float)den;
  return t;
}

// (1 - w) a + w b, the second product rounded first: spelled out, so that the outputs do not follow
// what the compiler makes of the sum
__device__ __forceinline__ float blend(float w, float a, float b) { return fmaf(1.0f - w, a, w * b); }

typedef uint16_t u16_any __attribute__((aligned(1)));

// two neighbouring elements of the output
template <bool BF16> __device__ __forceinline__ void store_pair(char* base, uint32_t off, float v0, float v1) {
  if constexpr (BF16) {
    typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
    bf16x2 w;
    w[0] = (__bf16)v0; w[1] = (__bf16)v1;
    // a stream of output: the clips below 35.1 -> 34.1 us, 32 images 28.3 -> 26.9.  The GEMM that reads the
    // rows next then finds less of them in the caches: 1 us longer behind 10 and 40 MB, 6 us behind 77 MB.
    __builtin_nontemporal_store(w, (bf16x2*)(base + off));
  } else {
    *(float2*)(base + off) = make_float2(v0, v1);
  }
}

// channel and frame of the slab at hand; stays on the last one
struct SlabWalk {
  int c, dt, left;             // left = slabs still ahead of this one
  __device__ __forceinline__ void next(int tp) {
    if (left > 0) { --left; if (++dt == tp) { dt = 0; ++c; } }
  }
};

// base + off with off widened next to the load, so that "scalar base + 32-bit lane offset" stays the
// load's own addressing form
__device__ __forceinline__ uint32_t pixels_at(const uint8_t* base, uint32_t off) {
  asm volatile("" : "+v"(off));
  return *(const u16_any*)(base + (size_t)off);
}

// A thread owns two neighbouring elements at one position of the patch and makes them for every
// channel x frame slab of its token, so that positions and taps are worked out once per token; a
// wave's store is a contiguous run of the output row.  A block takes as many whole tokens of one
// temporal slice as fit 512 threads: frame and output bases are then scalars, and a load is one
// instruction on a 32-bit lane offset.  Two elements per thread and not more, because the lanes of
// one load instruction then cover few source rows: with four or eight per thread a wave touches 16
// or 32 rows per load and the eight images below take 26 us.
// Measured, whole calls on inputs that do not stay in the last-level cache, against one block of
// patch x patch / 8 (or / 2) threads per token with divisions and byte loads per tap: eight images
// of 224 x 224 ... 1080 x 1920 to 448 x 448 48 -> 13 us (the host needs as long to queue one); 2160 x
// 3840 to 1056 x 1888 52 -> 14 us (2.7 TB/s); 64 frames at size, patch 14, 61 -> 38 us (3.1 TB/s; bound
// by HBM and what a wave spends before its first load); the same from 360 x 640 135 -> 70 us (vector
// arithmetic: about 490 instructions per token and position).
template <bool BF16>
__global__ __launch_bounds__(512) void preprocess_kernel(PrepArgs a) {
  // consecutive block ids go to different XCDs (8, each with its own L2): give every XCD a
  // contiguous eighth of the blocks, so that the neighbouring patches that share a 128-byte line
  // of source pixels fetch it through one L2 instead of eight
  const int nb = gridDim.x;
  const int vb = (blockIdx.x & 7) * (nb >> 3) + min((int)(blockIdx.x & 7), nb & 7) + (blockIdx.x >> 3);
  int it = 0;
#pragma unroll
  for (int step = kPrepItems / 2; step > 0; step >>= 1)
    if (it + step < a.n_items && vb >= a.item[it + step].blk_off) it += step;
  const PrepItem& d = a.item[it];
  const int p = a.patch;
  // small quotients in float: (n + 1/2) / k is at least 1 / (2 k) away from any integer
  const int tl = (int)(((float)threadIdx.x + 0.5f) * a.inv_per_token), pos = threadIdx.x - tl * a.per_token;
  const int py = (int)(((float)pos + 0.5f) * a.inv_per_row), px = (pos - py * (p >> 1)) * 2;
  const int blk = vb - d.blk_off, ti = blk / d.slice_blocks, first = (blk - ti * d.slice_blocks) * a.block_tokens;
  const long long plane = (long long)d.hs * d.ws, channel = (long long)(d.t * a.tp) * plane;
  constexpr int ES = BF16 ? 2 : 4;
  char* const out0 = (char*)a.out + ((long long)(d.tok_off + ti * d.h * d.w) * a.pdim) * ES;
  const uint32_t o = (uint32_t)(tl * a.pdim + py * p + px) * ES;
  const uint8_t* const frame0 = a.pixels + d.src_off + (long long)(ti * a.tp) * plane;
  const int slabs = a.channels * a.tp, slab_bytes = p * p * ES;
  const bool same = d.hs == d.h * p && d.ws == d.w * p;   // no resize: the pixels themselves
  const bool narrow = d.ws < 2;                           // rows of one pixel: nothing to load two of
  if (tl >= a.block_tokens || first + tl >= d.h * d.w) return;
  const int row0 = first / d.w, along = first - row0 * d.w + tl;           // along < w + 256
  const int down = (int)(((float)along + 0.5f) * d.inv_cols);
  const int y = (row0 + down) * p + py, x = (along - down * d.w) * p + px;
  char* out = out0 + (long long)first * a.pdim * ES;
  SlabWalk w = {0, 0, slabs - 1};
  if (same) {
    constexpr int kSlabs = 6;      // slabs whose loads a thread has in flight together (of fewer, the last is loaded again)
    const uint32_t f = (uint32_t)(y * d.ws + x);
    for (int s0 = 0; s0 < slabs; s0 += kSlabs) {
      uint32_t q[kSlabs];
      float ac[kSlabs], bc[kSlabs];
#pragma unroll
      for (int k = 0; k < kSlabs; ++k) {
        q[k] = pixels_at(frame0 + w.c * channel + w.dt * plane, f);
        ac[k] = a.a[w.c]; bc[k] = a.b[w.c];
        w.next(a.tp);
      }
#pragma unroll
      for (int k = 0; k < kSlabs; ++k) {
        if (s0 + k >= slabs) break;
        store_pair<BF16>(out, o, fmaf((float)(q[k] & 0xff), ac[k], bc[k]), fmaf((float)(q[k] >> 8), ac[k], bc[k]));
        out += slab_bytes;
      }
    }
    return;
  }
  constexpr int kSlabs = 3;
  const Tap ty = tap(y, d.hs, d.h * p, d.inv_h);
  const uint32_t r0 = (uint32_t)ty.i0 * (uint32_t)d.ws, r1 = (uint32_t)min(ty.i0 + 1, d.hs - 1) * (uint32_t)d.ws;
  float wx[2];
  uint32_t at[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const Tap t = tap(x + i, d.ws, d.w * p, d.inv_w);
    // at or beyond the last pixel centre both taps are the last pixel, the second of the pair loaded
    wx[i] = t.i0 >= d.ws - 1 ? 1.0f : t.w1;
    at[i] = (uint32_t)max(min(t.i0, d.ws - 2), 0);
  }
  for (int s0 = 0; s0 < slabs; s0 += kSlabs) {
    uint32_t q[kSlabs][2][2];                             // two neighbouring pixels of rows r0 and r1 per element
    float ac[kSlabs], bc[kSlabs];
#pragma unroll
    for (int k = 0; k < kSlabs; ++k) {
      const uint8_t* f = frame0 + w.c * channel + w.dt * plane;
      ac[k] = a.a[w.c]; bc[k] = a.b[w.c];
      if (narrow) {
#pragma unroll
        for (int i = 0; i < 2; ++i) { q[k][i][0] = (uint32_t)f[r0] * 0x101u; q[k][i][1] = (uint32_t)f[r1] * 0x101u; }
      } else {
#pragma unroll
        for (int i = 0; i < 2; ++i) { q[k][i][0] = pixels_at(f, r0 + at[i]); q[k][i][1] = pixels_at(f, r1 + at[i]); }
      }
      w.next(a.tp);
    }
#pragma unroll
    for (int k = 0; k < kSlabs; ++k) {
      if (s0 + k >= slabs) break;
      float v[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        float line[2];
#pragma unroll
        for (int r = 0; r < 2; ++r)
          line[r] = blend(wx[i], (float)(q[k][i][r] & 0xff), (float)(q[k][i][r] >> 8));
        v[i] = fmaf(blend(ty.w1, line[0], line[1]), ac[k], bc[k]);
      }
      store_pair<BF16>(out, o, v[0], v[1]);
      out += slab_bytes;
    }
  }
}

void launch_preprocess(PrepArgs& a, hipStream_t s) {
  a.per_token = a.patch * a.patch / 2;          // 2 .. 512 threads
  a.block_tokens = 512 / a.per_token;
  a.inv_per_token = 1.0f / (float)a.per_token;
  a.inv_per_row = 1.0f / (float)(a.patch / 2);
  long long blocks = 0;
  for (int i = 0; i < a.n_items; ++i) {
    PrepItem& d = a.item[i];
    d.blk_off = (int)blocks;
    d.slice_blocks = (d.h * d.w + a.block_tokens - 1) / a.block_tokens;
    d.inv_h = 1.0f / (float)(2 * d.h * a.patch);
    d.inv_w = 1.0f / (float)(2 * d.w * a.patch);
    d.inv_cols = 1.0f / (float)d.w;
    blocks += (long long)d.t * d.slice_blocks;
  }
  const dim3 threads((a.block_tokens * a.per_token + 63) / 64 * 64);
  for (long long b = 0; b < blocks; b += kMaxGrid) {
    // block numbers of an item count from the launch's first block (first_block as an argument took 1 % of
    // the clips' time: 33.45 -> 33.78 us)
    if (b > 0)
      for (int i = 0; i < a.n_items; ++i) a.item[i].blk_off -= kMaxGrid;
    const dim3 grid((unsigned)std::min(blocks - b, (long long)kMaxGrid));
    if (a.out_bf16) hipLaunchKernelGGL(preprocess_kernel<true>, grid, threads, 0, s, a);
    else hipLaunchKernelGGL(preprocess_kernel<false>, grid, threads, 0, s, a);
  }
}

}  // namespace epd
