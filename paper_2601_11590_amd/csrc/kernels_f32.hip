// fp32 kernels of the Encode-stage library (ViT forward, paper section 3.1, Eq. 1): the
// configuration whose storage type is fp32 must multiply and accumulate in true fp32.  The
// contractions run on the fp32 matrix instruction, v_mfma_f32_16x16x4_f32 (fused fp32 multiply-adds,
// twice the vector rate); everything else is vector arithmetic.
//
// What bounds the small calls this path serves (one 224 x 224 image: 256 tokens, hidden 256) is
// latency and idle compute units, so work is cut fine: 16 x 16 output tiles whose K is split over the
// waves of a block, 16-query attention tiles whose keys are split over the waves.  Operands go from
// memory straight to registers: the k a lane group supplies to an instruction is arbitrary as long
// as both operands agree, so a lane takes four consecutive k of its row (one 16-byte load) and feeds
// them to four instructions.
#include "epd_internal.h"

#include <algorithm>

namespace epd {

typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));

// ------------------------------------------------------------------------------ GEMM
__device__ __forceinline__ float gelu_f32(float v, int act) {
  if (act == 0) return 0.5f * v * (1.0f + erff(v * 0.70710678118654752440f));
  float u = 0.79788456080286535588f * (v + 0.044715f * v * v * v);
  return 0.5f * v * (1.0f + tanhf(u));
}

// A block of NW waves.  SPLIT: all of them share one 16 T x 16 T tile and take its K in turn, 32 at a
// time, and their sums meet in LDS; otherwise NW = 4 and each has a tile of its own, 2 x 2.
// VEC: rows start 16-byte aligned and K (and a gathered piece) is a multiple of 4; otherwise 16-byte
// loads from any float's address, and the last of a row taken apart.
template <int T, int NW, bool SPLIT, bool VEC>
__global__ __launch_bounds__(64 * NW) void gemm_f32_kernel(GemmArgs g) {
  constexpr int WT = 16 * T, BT = SPLIT ? WT : 2 * WT;       // wave and block tile
  constexpr int LD = BT + 4, COPIES = SPLIT ? NW : 1;
  constexpr int KS = 32;                                     // k per step and wave: two 16-byte loads per row
  __shared__ __attribute__((aligned(16))) float acc_lds[COPIES][BT][LD];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, g4 = lane >> 4;
  const int m0 = blockIdx.y * BT, n0 = blockIdx.x * BT;
  const int wm = SPLIT ? 0 : (wave >> 1) * WT, wn = SPLIT ? 0 : (wave & 1) * WT;
  const float* const A = (const float*)g.A;
  const float* const W = (const float*)g.W;
  const int kc = g.gather ? g.K / g.gather_n : g.K;          // width of one gathered piece

  const float *arow[T], *wrow[T];
  int am[T];
#pragma unroll
  for (int t = 0; t < T; ++t) {                              // rows beyond the matrix repeat the last one: never stored
    am[t] = min(m0 + wm + t * 16 + l16, g.M - 1);
    arow[t] = A + (size_t)am[t] * g.lda;
    wrow[t] = W + (size_t)min(n0 + wn + t * 16 + l16, g.N - 1) * g.K;
  }
  auto load4 = [&](const float* row, int k) {                // row[k .. k + 3], zero from K on
    if constexpr (VEC) {
      const f32x4 v = *(const f32x4*)(row + min(k, g.K - 4));
      return k < g.K ? v : f32x4{0.f, 0.f, 0.f, 0.f};
    } else {
      // 16 bytes at any float's address; four loads of four made K = 1023 slower than 64 x 64 vector tiles were
      // (32 768 x 256: 722 us against 473; 312 this way)
      f32x4 v;
      if (k + 4 <= g.K) {
        v = *(const f32x4_any*)(row + k);
      } else {
#pragma unroll
        for (int c = 0; c < 4; ++c) v[c] = k + c < g.K ? row[k + c] : 0.f;
      }
      return v;
    }
  };
  auto load_a = [&](int t, int k) {
    if (!g.gather) return load4(arow[t], k);
    f32x4 v;
    if constexpr (VEC) {
      const int kk = min(k, g.K - 4), piece = kk / kc;
      v = *(const f32x4*)(A + (size_t)g.gather[(size_t)am[t] * g.gather_n + piece] * g.lda + (kk - piece * kc));
      if (k >= g.K) v = f32x4{0.f, 0.f, 0.f, 0.f};
    } else {
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int kk = min(k + c, g.K - 1), piece = kk / kc;
        v[c] = A[(size_t)g.gather[(size_t)am[t] * g.gather_n + piece] * g.lda + (kk - piece * kc)];
        if (k + c >= g.K) v[c] = 0.f;
      }
    }
    return v;
  };

  f32x4 acc[T][T];                                           // [n][m]: a lane holds 4 consecutive n of one m
#pragma unroll
  for (int i = 0; i < T; ++i)
#pragma unroll
    for (int j = 0; j < T; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  constexpr int KSTEP = SPLIT ? NW * KS : KS;
  f32x4 fa[2][T][2], fw[2][T][2];
  auto fetch = [&](int buf, int k0) {
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        fa[buf][t][h] = load_a(t, k0 + h * 16 + g4 * 4);
        fw[buf][t][h] = load4(wrow[t], k0 + h * 16 + g4 * 4);
      }
  };
  auto multiply = [&](int buf) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int i = 0; i < T; ++i)
#pragma unroll
          for (int j = 0; j < T; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fw[buf][i][h][c], fa[buf][j][h][c], acc[i][j], 0, 0, 0);
  };
  int k0 = SPLIT ? wave * KS : 0;
  if (k0 < g.K) fetch(0, k0);
  for (; k0 < g.K; k0 += 2 * KSTEP) {
    if (k0 + KSTEP < g.K) fetch(1, k0 + KSTEP);
    multiply(0);
    if (k0 + KSTEP >= g.K) break;
    if (k0 + 2 * KSTEP < g.K) fetch(0, k0 + 2 * KSTEP);
    multiply(1);
  }
#pragma unroll
  for (int i = 0; i < T; ++i)
#pragma unroll
    for (int j = 0; j < T; ++j)
      *(f32x4*)&acc_lds[SPLIT ? wave : 0][wm + j * 16 + l16][wn + i * 16 + g4 * 4] = acc[i][j];
  __syncthreads();

  // epilogue: a thread takes 4 consecutive columns (whole rotary pairs) of a row
  const float* bias = (const float*)g.bias;
  float* out = (float*)g.out;
  for (int e = tid; e < BT * BT / 4; e += 64 * NW) {
    const int r = e / (BT / 4), c = (e - r * (BT / 4)) * 4;
    const int m = m0 + r, n = n0 + c;
    if (m >= g.M || n >= g.N) continue;
    f32x4 v = *(const f32x4*)&acc_lds[0][r][c];
#pragma unroll
    for (int w = 1; w < COPIES; ++w) v += *(const f32x4*)&acc_lds[w][r][c];
    const int left = min(4, g.N - n);
    if (bias)
      for (int j = 0; j < left; ++j) v[j] += bias[n + j];
    if (g.epilogue == EPI_QKV && g.rot) {
#pragma unroll
      for (int j = 0; j < 4; j += 2) {
        if (n + j + 1 < g.N && n + j < g.qk_cols) {          // even column; pair = (n + j, n + j + 1)
          const float2 cs = g.rot[(size_t)m * g.rot_pairs + (((n + j) % g.head_dim) >> 1)];
          const float a = v[j], b = v[j + 1];
          v[j] = a * cs.x - b * cs.y;
          v[j + 1] = a * cs.y + b * cs.x;
        }
      }
    }
    if (g.epilogue == EPI_GELU) {
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = gelu_f32(v[j], g.act);
    }
    float* dst = g.epilogue == EPI_RESIDUAL ? g.resid + (size_t)m * g.ldr + n : out + (size_t)m * g.ldo + n;
    if (left == 4 && ((size_t)dst & 15) == 0) {
      if (g.epilogue == EPI_RESIDUAL) v += *(const f32x4*)dst;
      *(f32x4*)dst = v;
    } else {
      for (int j = 0; j < left; ++j) dst[j] = g.epilogue == EPI_RESIDUAL ? dst[j] + v[j] : v[j];
    }
  }
}

template <int T, int NW, bool SPLIT> static void launch_tile_f32(const GemmArgs& g, hipStream_t s) {
  constexpr int BT = SPLIT ? 16 * T : 32 * T;
  const dim3 grid((g.N + BT - 1) / BT, (g.M + BT - 1) / BT);
  const int piece = g.gather ? g.K / g.gather_n : g.K;
  const bool vec = piece % 4 == 0 && g.lda % 4 == 0 && (((size_t)g.A | (size_t)g.W) & 15) == 0;
  if (vec) hipLaunchKernelGGL((gemm_f32_kernel<T, NW, SPLIT, true>), grid, dim3(64 * NW), 0, s, g);
  else hipLaunchKernelGGL((gemm_f32_kernel<T, NW, SPLIT, false>), grid, dim3(64 * NW), 0, s, g);
}

// Tile by how many waves it gives a chip of 1024 SIMDs: 16 x 16 tiles with K split over four waves (or
// eight, where there are few tiles and K is long) up to about four waves per SIMD, then 32 x 32 tiles
// with K split over four, then 64 x 64 blocks of four wave tiles, which read an operand byte least
// often.  One 256-token image (hidden 256, six products of 256 x 256 x 256 ... 1024): 4 - 9 us each, 41
// together, where 64 x 64 tiles of vector arithmetic took 34 - 144 and 428 together.
void launch_gemm_f32(const GemmArgs& g, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0) return;
  const long t16 = (long)((g.M + 15) / 16) * ((g.N + 15) / 16), t32 = (long)((g.M + 31) / 32) * ((g.N + 31) / 32);
  if (t16 <= 256 && g.K >= 512) launch_tile_f32<1, 8, true>(g, s);
  else if (t16 <= 1024) launch_tile_f32<1, 4, true>(g, s);
  else if (t32 <= 2048) launch_tile_f32<2, 4, true>(g, s);
  else launch_tile_f32<2, 4, false>(g, s);
}

// ------------------------------------------------------------------------------ attention
// One block = 16 query rows of one segment and head; its NW waves take the keys in turn, 32 at a
// time, each with its own running maximum and sum (softmax in fp32 with expf), and merge at the end.
// Scores are computed transposed, S^T = K Q^T: a lane then holds the scores of ONE query (lane % 16)
// against keys 4 (lane / 16) .. + 3 of each 16, which is where the second product, O^T = V^T P^T,
// wants its second operand if instruction j takes key 4 (lane / 16) + j from lane group lane / 16.
// 256 tokens, 4 heads of 64: 8.7 us (64 blocks of 8 waves), 232 with one thread per query row.
constexpr int F32_BQ = 16, F32_BKV = 32;

template <int DH, int NW>
__global__ __launch_bounds__(64 * NW) void attn_f32_kernel(AttnArgs a) {
  constexpr int DC = (DH + 15) / 16;       // 16-channel chunks
  constexpr int LDO = DC * 16 + 4;
  __shared__ __attribute__((aligned(16))) float o_lds[NW][F32_BQ][LDO];
  __shared__ float m_lds[NW][F32_BQ], l_lds[NW][F32_BQ];
  const AttnWork w = a.work[blockIdx.x];
  const int head = blockIdx.y, D = a.num_heads * DH;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, g4 = lane >> 4;
  const float* const base = (const float*)a.qkv + head * DH;
  const int seg_end = w.seg_start + w.seg_len;

  // channel 16 i + 4 g4 + c of a row is the k of instruction (i, c) that lane group g4 supplies
  f32x4 q[DC];
  const float* const qrow = base + (size_t)min(w.q0 + l16, seg_end - 1) * a.ld_qkv;
#pragma unroll
  for (int i = 0; i < DC; ++i) {
    const int d = 16 * i + 4 * g4;
    q[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (d < DH) q[i] = *(const f32x4*)(qrow + d) * a.scale;
  }
  f32x4 o[DC];
#pragma unroll
  for (int i = 0; i < DC; ++i) o[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY, l = 0.f;            // of query l16, over the keys this lane group has seen (m: of all groups)

  for (int kv0 = w.seg_start + wave * F32_BKV; kv0 < seg_end; kv0 += NW * F32_BKV) {
    f32x4 kf[2][DC];
    float vf[2][4][DC];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const float* kr = base + D + (size_t)min(kv0 + 16 * b + l16, seg_end - 1) * a.ld_qkv;
#pragma unroll
      for (int i = 0; i < DC; ++i) {
        const int d = 16 * i + 4 * g4;
        kf[b][i] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (d < DH) kf[b][i] = *(const f32x4*)(kr + d);
      }
    }
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float* vr = base + 2 * D + (size_t)min(kv0 + 16 * b + 4 * g4 + j, seg_end - 1) * a.ld_qkv;
#pragma unroll
        for (int i = 0; i < DC; ++i) vf[b][j][i] = vr[min(16 * i + l16, DH - 1)];   // channels beyond DH are never stored
      }
    f32x4 s[2];
    float mt = -INFINITY;
    const float m0 = m;
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      s[b] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int i = 0; i < DC; ++i)
#pragma unroll
        for (int c = 0; c < 4; ++c) s[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[b][i][c], q[i][c], s[b], 0, 0, 0);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        if (kv0 + 16 * b + 4 * g4 + v >= seg_end) s[b][v] = -INFINITY;
        mt = fmaxf(mt, s[b][v]);
      }
    }
    mt = fmaxf(mt, __shfl_xor(mt, 16));
    mt = fmaxf(mt, __shfl_xor(mt, 32));
    m = fmaxf(m, mt);
    // scores may all be -inf (a product beyond the range): those of a wave's share of the keys, of weight
    // zero beside the other waves' -- the maximum subtracted must be finite
    const float mn = m == -INFINITY ? 0.f : m;
    const float alpha = expf(m0 - mn);     // first keys: exp(-inf) = 0
    l *= alpha;
#pragma unroll
    for (int i = 0; i < DC; ++i) o[i] *= alpha;
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        s[b][v] = expf(s[b][v] - mn);      // masked entries: exp(-inf) = 0
        l += s[b][v];
      }
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int i = 0; i < DC; ++i) o[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[b][j][i], s[b][j], o[i], 0, 0, 0);
  }
  l += __shfl_xor(l, 16);
  l += __shfl_xor(l, 32);
#pragma unroll
  for (int i = 0; i < DC; ++i) *(f32x4*)&o_lds[wave][l16][16 * i + 4 * g4] = o[i];
  if (lane < 16) { m_lds[wave][l16] = m; l_lds[wave][l16] = l; }
  __syncthreads();
  for (int e = tid; e < F32_BQ * DH; e += 64 * NW) {
    const int r = e / DH, d = e - r * DH;
    if (w.q0 + r >= seg_end) continue;
    float mx = m_lds[0][r];
#pragma unroll
    for (int x = 1; x < NW; ++x) mx = fmaxf(mx, m_lds[x][r]);
    float num = 0.f, den = 0.f;
#pragma unroll
    for (int x = 0; x < NW; ++x) {
      const float f = expf(m_lds[x][r] - mx);                // a wave without keys: exp(-inf) = 0
      num = fmaf(f, o_lds[x][r][d], num);
      den = fmaf(f, l_lds[x][r], den);
    }
    ((float*)a.out)[(size_t)(w.q0 + r) * a.ld_out + head * DH + d] = num / den;
  }
}

bool launch_attn_f32(const AttnArgs& a, hipStream_t s) {
  if (a.num_work <= 0) return true;
  if (a.q_tile != F32_BQ) return false;
#define EPD_ATTN_F32(DH)                                                                             \
  case DH: {                                                                                         \
    constexpr int NW = DH <= 64 ? 8 : 4;                                                             \
    for (AttnArgs c = a; c.num_work > 0; c.num_work -= kMaxGrid, c.work += kMaxGrid)                 \
      hipLaunchKernelGGL((attn_f32_kernel<DH, NW>), dim3(std::min(c.num_work, kMaxGrid), a.num_heads), \
                         dim3(64 * NW), 0, s, c);                                                    \
    return true;                                                                                     \
  }
  switch (a.head_dim) {
    EPD_ATTN_F32(8);
    EPD_ATTN_F32(16);
    EPD_ATTN_F32(32);
    EPD_ATTN_F32(64);
    EPD_ATTN_F32(72);
    EPD_ATTN_F32(80);
    EPD_ATTN_F32(96);
    EPD_ATTN_F32(128);
    default:
      return false;
  }
#undef EPD_ATTN_F32
}

}  // namespace epd
