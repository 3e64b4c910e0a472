// Per-call plan kernels, the fused LayerNorm / RMSNorm kernel and the create-time weight
// reordering of the Encode-stage library (ViT forward, paper section 3.1, Eq. 1).
//
// All of these are bound by memory traffic, not arithmetic: they use wide coalesced
// accesses and wave-level (64 lane) reductions, no matrix cores.
#include "epd_internal.h"

#include <algorithm>

namespace epd {

typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;

// ------------------------------------------------------------------------------ plan
template <typename E> __device__ __forceinline__ int last_not_after(const E* t, int n, int x, int32_t E::*key) {
  // largest i in [0, n) with t[i].*key <= x   (keys increase, t[0].*key = 0)
  int lo = 0, hi = n;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (t[mid].*key <= x) lo = mid; else hi = mid;
  }
  return lo;
}

// Everything a call derives from its metadata, in one launch; a block has one of four roles:
//   rot    (cos, sin) of the (token, pair) entries of 256 / pairs tokens, in double
//   work   bf16: one entry of the attention work list and the vt columns of its tokens; fp32: 256
//          entries (no vt)
//   merge  the source tokens of 256 merged tokens, window rows then columns
//   pad    clears the columns of vt between a segment's end and the next (aligned) start, four
//          channel rows per block: attention multiplies them by exact zeros, so they must be finite
// The rot and pad roles take at most kMaxGrid blocks, which stride over larger tables (STRIDED; a
// kernel of its own, since small calls notice the loops: 0.2 us of 57).
// Up to kPlanInline segments and items the tables are kernel arguments, copied to LDS before they
// are searched.  Bound: latency.  As a copy of the metadata (3 us) plus three kernels, one thread per
// token for all its pairs (15 us), this step cost a call 24 us more: one 256-token image 3.9 us now.
template <bool STRIDED> __global__ __launch_bounds__(256) void plan_kernel(PlanArgs p) {
  __shared__ PlanItem items[kPlanInline];
  __shared__ PlanSeg segs[kPlanInline];
  const int tid = threadIdx.x;
  const PlanItem* item = p.item;
  const PlanSeg* seg = p.seg;
  if (p.inline_tables) {
    if (tid < p.num_items) items[tid] = p.inl_item[tid];
    if (tid < p.num_segments) segs[tid] = p.inl_seg[tid];
    __syncthreads();
    item = items; seg = segs;
  }
  int b = blockIdx.x;
  if (b < p.rot_blocks) {
    RotEntry e;
    do {
      if (!rot_entry(p.T, p.pairs, b, tid, e)) continue;
      const PlanItem& d = item[last_not_after(item, p.num_items, e.tok, &PlanItem::tok)];
      const int local = e.tok - d.tok, t = local / (d.h * d.w), rem = local - t * d.h * d.w, r = rem / d.w;
      const int ax = p.pair_axis[e.pair], coord = ax == 0 ? t : ax == 1 ? r : rem - r * d.w;
      double sn, cs;
      sincos((double)coord * p.pair_freq[e.pair], &sn, &cs);
      p.rot[e.at] = make_float2((float)cs, (float)sn);
    } while (STRIDED && (b += p.rot_blocks) * rot_tokens_per_block(p.pairs) < p.T);
    return;
  }
  b -= p.rot_blocks;
  if (b < p.work_blocks) {
    const int i = p.vcol ? b : b * 256 + tid;
    if (i >= p.num_work) return;
    const PlanSeg& s = seg[last_not_after(seg, p.num_segments, i, &PlanSeg::work0)];
    const int q0 = (i - s.work0) * p.q_tile;
    if (!p.vcol || tid == 0) p.work[i] = AttnWork{s.start + q0, s.start, s.len, s.vcol};
    if (p.vcol)
      for (int t = q0 + tid; t < min(q0 + p.q_tile, s.len); t += 256) p.vcol[s.start + t] = s.vcol + t;
    return;
  }
  b -= p.work_blocks;
  if (b < p.merge_blocks) {
    const int mt = b * 256 + tid;
    if (mt >= p.Tm) return;
    const PlanItem& d = item[last_not_after(item, p.num_items, mt, &PlanItem::mrg)];
    const int m = p.merge, hm = d.h / m, wm = d.w / m, local = mt - d.mrg;
    const int ti = local / (hm * wm), rem = local - ti * hm * wm, i = rem / wm, j = rem - i * wm;
    const int base = d.tok + ti * d.h * d.w;
    for (int di = 0; di < m; ++di)
      for (int dj = 0; dj < m; ++dj)
        p.merge_idx[(size_t)mt * m * m + di * m + dj] = base + (m * i + di) * d.w + m * j + dj;
    return;
  }
  b -= p.merge_blocks;
  const int rows = (p.hidden + 3) / 4;
  do {
    const int sg = b / rows, row = (b - sg * rows) * 4 + (tid >> 6);
    if (row >= p.hidden) continue;
    const PlanSeg& s = seg[sg];
    uint16_t* vt = (uint16_t*)p.vt + (size_t)row * p.vt_stride;
    const int end = s.vcol + (s.len + kVtAlign - 1) / kVtAlign * kVtAlign;
    for (int c = s.vcol + s.len + (tid & 63); c < end; c += 64) vt[c] = 0;
  } while (STRIDED && (b += p.pad_blocks) < p.num_segments * rows);
}

void launch_plan(PlanArgs& p, hipStream_t s) {
  const int rot_tokens = p.pairs > 0 ? rot_tokens_per_block(p.pairs) : 1;
  const int rot = p.pairs > 0 ? (p.T + rot_tokens - 1) / rot_tokens : 0;
  const int pad = p.vt ? p.num_segments * ((p.hidden + 3) / 4) : 0;      // the vt buffer holds 1 KB per unit of it
  p.rot_blocks = std::min(rot, kMaxGrid);
  p.work_blocks = p.vcol ? p.num_work : (p.num_work + 255) / 256;
  p.merge_blocks = p.merge > 1 ? (p.Tm + 255) / 256 : 0;
  p.pad_blocks = std::min(pad, kMaxGrid);
  const dim3 grid(p.rot_blocks + p.work_blocks + p.merge_blocks + p.pad_blocks);
  if (rot > kMaxGrid || pad > kMaxGrid) hipLaunchKernelGGL(plan_kernel<true>, grid, dim3(256), 0, s, p);
  else hipLaunchKernelGGL(plan_kernel<false>, grid, dim3(256), 0, s, p);
}

// ------------------------------------------------------------------------------ norm
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}


template <typename T> __device__ __forceinline__ void ld_param4(const T* p, int i, float* o);
template <> __device__ __forceinline__ void ld_param4<float>(const float* p, int i, float* o) {
  const float4 v = *(const float4*)(p + i);
  o[0] = v.x; o[1] = v.y; o[2] = v.z; o[3] = v.w;
}
template <> __device__ __forceinline__ void ld_param4<__bf16>(const __bf16* p, int i, float* o) {
  const uint2 v = *(const uint2*)(p + i);
  o[0] = __uint_as_float(v.x << 16); o[1] = __uint_as_float(v.x & 0xffff0000u);
  o[2] = __uint_as_float(v.y << 16); o[3] = __uint_as_float(v.y & 0xffff0000u);
}

// One 64-lane wave per token row; the row is held in registers (NV float4 per lane) between
// the statistics pass and the scaling pass, so HBM sees one read and one write per element.
// LayerNorm uses the two-pass mean / centred variance form (biased variance).
template <typename PT, typename OT, int NV>
__global__ __launch_bounds__(256) void norm_kernel(const float* __restrict__ x, const PT* __restrict__ gamma,
                                                   const PT* __restrict__ beta, OT* __restrict__ out,
                                                   int T, int D, float eps, int rms) {
  int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  int lane = threadIdx.x & 63;
  if (row >= T) return;
  const float* xr = x + (size_t)row * D;
  float4 v[NV];
  float sum = 0.f;
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    int c = (i * 64 + lane) * 4;
    v[i] = (c < D) ? *(const float4*)(xr + c) : make_float4(0.f, 0.f, 0.f, 0.f);
    sum += (v[i].x + v[i].y) + (v[i].z + v[i].w);
  }
  float mean = 0.f;
  if (!rms) mean = wave_sum(sum) / (float)D;
  float sq = 0.f;
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    int c = (i * 64 + lane) * 4;
    if (c < D) {
      float a = v[i].x - mean, b = v[i].y - mean, cc = v[i].z - mean, d = v[i].w - mean;
      sq += (a * a + b * b) + (cc * cc + d * d);
    }
  }
  float rstd = 1.0f / sqrtf(wave_sum(sq) / (float)D + eps);   // correctly rounded, once per row
  OT* orow = out + (size_t)row * D;
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    int c = (i * 64 + lane) * 4;
    if (c < D) {
      float y[4] = {v[i].x, v[i].y, v[i].z, v[i].w};
      // the four gains (and shifts) of the chunk come in one load each (c is a multiple of 4)
      float g4[4], b4[4] = {0.f, 0.f, 0.f, 0.f};
      ld_param4(gamma, c, g4);
      if (beta) ld_param4(beta, c, b4);
#pragma unroll
      for (int e = 0; e < 4; ++e) y[e] = (y[e] - mean) * rstd * g4[e] + b4[e];
      if constexpr (sizeof(OT) == 4) {
        *(float4*)((float*)orow + c) = make_float4(y[0], y[1], y[2], y[3]);
      } else {
        bf16x2_t lo, hi;
        lo[0] = (__bf16)y[0]; lo[1] = (__bf16)y[1];
        hi[0] = (__bf16)y[2]; hi[1] = (__bf16)y[3];
        uint2 pk;
        pk.x = *(uint32_t*)&lo; pk.y = *(uint32_t*)&hi;
        *(uint2*)((__bf16*)orow + c) = pk;
      }
    }
  }
}

template <typename PT, typename OT>
static void norm_dispatch(const float* x, const void* g, const void* b, void* out, int T, int D,
                          float eps, bool rms, hipStream_t s) {
  dim3 grid((T + 3) / 4), block(256);
  int nv = (D + 255) / 256;
#define EPD_NORM_CASE(N)                                                                      \
  hipLaunchKernelGGL((norm_kernel<PT, OT, N>), grid, block, 0, s, x, (const PT*)g, (const PT*)b, \
                     (OT*)out, T, D, eps, rms ? 1 : 0)
  if (nv <= 1) EPD_NORM_CASE(1);
  else if (nv <= 2) EPD_NORM_CASE(2);
  else if (nv <= 4) EPD_NORM_CASE(4);
  else if (nv <= 5) EPD_NORM_CASE(5);
  else if (nv <= 8) EPD_NORM_CASE(8);
  else if (nv <= 13) EPD_NORM_CASE(13);
  else if (nv <= 16) EPD_NORM_CASE(16);
  else EPD_NORM_CASE(32);   // D <= 8192 (checked at create)
#undef EPD_NORM_CASE
}

void launch_norm(const float* x, const void* gamma, const void* beta, void* out, int T, int D,
                 float eps, bool rms, bool bf16, hipStream_t s) {
  if (T <= 0) return;
  if (bf16) norm_dispatch<__bf16, __bf16>(x, gamma, beta, out, T, D, eps, rms, s);
  else norm_dispatch<float, float>(x, gamma, beta, out, T, D, eps, rms, s);
}

// ------------------------------------------------------------------------------ create-time reorder
// Rows of the fused QKV weight are reordered inside every Q and K head so that the two
// members (p, p + d/2) of rotary pair p become neighbours (2p, 2p + 1).  Q.K^T is
// unchanged by a permutation applied to both, and the GEMM epilogue can then rotate a pair
// without leaving the lane that owns it.  V rows are copied as they are.
template <typename T>
__global__ __launch_bounds__(256) void permute_qkv_kernel(const T* __restrict__ sw, const T* __restrict__ sb,
                                                          T* __restrict__ dw, T* __restrict__ db,
                                                          int D, int hd) {
  int drow = blockIdx.x;     // destination row in [0, 3D)
  int srow = drow;
  if (drow < 2 * D) {
    int head0 = (drow / hd) * hd;
    int c = drow - head0;
    srow = head0 + (c >> 1) + (c & 1) * (hd >> 1);
  }
  const T* s = sw + (size_t)srow * D;
  T* d = dw + (size_t)drow * D;
  for (int i = threadIdx.x; i < D; i += blockDim.x) d[i] = s[i];
  if (sb && threadIdx.x == 0) db[drow] = sb[srow];
}

void launch_permute_qkv(const void* src_w, const void* src_b, void* dst_w, void* dst_b, int hidden,
                        int num_heads, int head_dim, int elem_bytes, hipStream_t s) {
  (void)num_heads;
  if (elem_bytes == 4)
    hipLaunchKernelGGL(permute_qkv_kernel<float>, dim3(3 * hidden), dim3(256), 0, s, (const float*)src_w,
                       (const float*)src_b, (float*)dst_w, (float*)dst_b, hidden, head_dim);
  else
    hipLaunchKernelGGL(permute_qkv_kernel<uint16_t>, dim3(3 * hidden), dim3(256), 0, s, (const uint16_t*)src_w,
                       (const uint16_t*)src_b, (uint16_t*)dst_w, (uint16_t*)dst_b, hidden, head_dim);
}

// ------------------------------------------------------------------------------ copies
// Several device-to-device copies in one launch (rows of the feature store to and from the
// caller's tensors).  Bound: HBM; one 16 KB piece per block, four 16-byte loads per thread in
// flight, any alignment.  Eight copies of 1.6 MB: 5.5 us (4.7 TB/s read + written) here, eight
// launches of at least as much each as hipMemcpyAsync.
typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(1)));
constexpr int kCopyPiece = 256 * 16 * 4;

__global__ __launch_bounds__(256) void copies_kernel(CopyArgs a) {
  static_assert(kCopyItems == 64, "one lane per item");
  const int lane = threadIdx.x & 63;
  const int i = __builtin_amdgcn_readfirstlane(__popcll(__ballot(lane < a.n && a.first_block[lane] <= (int)blockIdx.x)) - 1);
  const CopyItem c = a.item[i];
  const long long at = (long long)((int)blockIdx.x - a.first_block[i]) * kCopyPiece;
  const char* src = (const char*)c.src + at;
  char *d0 = (char*)c.dst + at, *d1 = c.dst2 ? (char*)c.dst2 + at : nullptr;
  const int left = (int)min((long long)kCopyPiece, c.bytes - at);
  if (left == kCopyPiece) {
    u32x4_any v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = *(const u32x4_any*)(src + (k * 256 + threadIdx.x) * 16);
#pragma unroll
    for (int k = 0; k < 4; ++k) *(u32x4_any*)(d0 + (k * 256 + threadIdx.x) * 16) = v[k];
    if (d1) {
#pragma unroll
      for (int k = 0; k < 4; ++k) *(u32x4_any*)(d1 + (k * 256 + threadIdx.x) * 16) = v[k];
    }
    return;
  }
  for (int o = threadIdx.x * 16; o < left; o += 256 * 16) {
    if (o + 16 <= left) {
      const u32x4_any v = *(const u32x4_any*)(src + o);
      *(u32x4_any*)(d0 + o) = v;
      if (d1) *(u32x4_any*)(d1 + o) = v;
    } else {
      for (int b = o; b < left; ++b) {
        const char v = src[b];
        d0[b] = v;
        if (d1) d1[b] = v;
      }
    }
  }
}

hipError_t launch_copies(CopyArgs& a, hipStream_t s) {
  long long blocks = 0;
  for (int i = 0; i < a.n; ++i) {
    a.first_block[i] = (int)blocks;
    blocks += (a.item[i].bytes + kCopyPiece - 1) / kCopyPiece;
  }
  if (blocks == 0) return hipSuccess;
  void* args[] = {&a};
  return hipLaunchKernel((const void*)copies_kernel, dim3((unsigned)blocks), dim3(256), args, 0, s);
}

// ---------------------------------------------------------------- gamma folding (create time)
__global__ __launch_bounds__(256) void fold_gamma_kernel(uint16_t* __restrict__ w, const uint16_t* __restrict__ gamma,
                                                         long total, int K) {
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  if (i >= total) return;
  const int k = (int)(i % K);
  const float v = __uint_as_float((uint32_t)w[i] << 16) * __uint_as_float((uint32_t)gamma[k] << 16);
  __bf16 r = (__bf16)v;   // round to nearest even
  w[i] = *(uint16_t*)&r;
}

void launch_fold_gamma(void* w, const void* gamma, int N, int K, hipStream_t s) {
  const long total = (long)N * K;
  hipLaunchKernelGGL(fold_gamma_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, (uint16_t*)w,
                     (const uint16_t*)gamma, total, K);
}

}  // namespace epd
