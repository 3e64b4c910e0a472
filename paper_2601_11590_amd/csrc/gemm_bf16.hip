// bf16 GEMM family of the Encode-stage library (ViT forward, paper section 3.1, Eq. 1):
// patch embedding, QKV projection with rotary epilogue, attention output projection, the
// two MLP GEMMs and the merger projection all are  C[M,N] = A[M,K] * W[N,K]^T (+bias)  with
// different epilogues.  Written for gfx950: 64-lane waves, v_mfma_f32_16x16x32_bf16 (fp32
// accumulate; at equal flops this shape draws less power than the 32x32x16 one, and under the
// chip's power limit that is clock: +7 % on the large GEMMs with random operands, nothing on
// all-zero ones), operand tiles brought from global memory straight into LDS
// (global_load_lds_dwordx4, no register staging) in a ring of two to four stages.
//
// Tile scheme.  A block of WAVES_M x WAVES_N waves owns a BM x BN output tile; K advances in
// steps of BK.  Both operands are K-contiguous in memory ("NT" form), so one lane's MFMA
// operand (8 consecutive k of one row) is one 16-byte LDS read.  A direct-to-LDS load writes
// the 64 lanes' 16-byte chunks to consecutive LDS addresses, so rows cannot be padded;
// instead the chunk a lane fetches is chosen so that chunk c of row r lands in slot
// c ^ swz(r) of that row, which spreads the 16 rows read by one MFMA operand fetch over all
// bank groups.  The next stages are in flight while stage s is multiplied.  The main loop is the ping-pong loop
// (eight-wave tiles, see PingPong) or a plain ring with one barrier per K step.
//
// Accumulator orientation.  For a 16x16 MFMA result lane l holds column (l % 16) and rows
// 4*(l/16) + v, v = 0..3.  By default the W fragment is fed as the first operand, so "rows"
// are output columns n and the lane's column is a token m: every lane then owns runs of 4
// consecutive n of one token -- 16-byte fp32 / 8-byte bf16 pieces of a row, and the two
// members of a rotary pair (neighbouring n after the create-time reorder) share a lane.  For
// the V third of the QKV projection the operands are swapped, a lane owns 4 consecutive tokens
// of one n, and V is stored transposed ([channel][token]) for the attention kernel's second
// GEMM.
#include "epd_internal.h"

#include <algorithm>
#include <type_traits>

namespace epd {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(4))) float f32x4;

#define EPD_GPTR(p) ((const __attribute__((address_space(1))) void*)(p))
#define EPD_LPTR(p) ((__attribute__((address_space(3))) void*)(p))

__device__ __forceinline__ uint2 pack_bf16x4(float a, float b, float c, float d) {
  bf16x2 lo, hi;
  lo[0] = (__bf16)a; lo[1] = (__bf16)b; hi[0] = (__bf16)c; hi[1] = (__bf16)d;
  uint2 r;
  r.x = *(uint32_t*)&lo; r.y = *(uint32_t*)&hi;
  return r;
}

__device__ __forceinline__ float bf16_bits_to_float(uint32_t b) { return __uint_as_float(b << 16); }

// x * Phi(x) with the Gaussian CDF written through its upper tail,
//   gelu(x) = max(x, 0) - |x| Q(|x|),   Q(a) = erfc(a / sqrt2) / 2 = 2^(a P(a) - 1),
// where P is a degree-5 polynomial fitted (weighted minimax, a in [0, 7.5]) to
// log2(erfc(a / sqrt2)) / a.  The logarithm of the tail is smooth, so one v_exp_f32 and six
// fused multiply-adds reach an absolute error below 2e-6 and a relative error below 1.5e-3 even
// where gelu is of order 1e-12 -- both far below the bf16 rounding of the stored result.
// Beyond a = 7.5 the tail term is below 1e-12 and the exponent is simply held.
__device__ __forceinline__ float gelu_erf_fast(float x) {
  const float a = fminf(fabsf(x), 7.5f);
  float p = fmaf(2.3815253741819458e-05f, a, -0.0006414791230697928f);
  p = fmaf(p, a, 0.007484599623650507f);
  p = fmaf(p, a, -0.05223089570546575f);
  p = fmaf(p, a, -0.459768916243223f);
  p = fmaf(p, a, -1.1509091680606687f);
  const float e = __builtin_amdgcn_exp2f(fmaf(p, a, -1.0f));
  return fmaf(-fabsf(x), e, fmaxf(x, 0.f));
}

__device__ __forceinline__ float gelu_tanh_fast(float x) {
  const float u = 0.79788456080286535588f * fmaf(0.044715f * x * x, x, x);
  const float e = __builtin_amdgcn_exp2f(2.0f * 1.44269504088896340736f * u);
  return x * (1.0f - __builtin_amdgcn_rcpf(1.0f + e));   // x * sigmoid(2u)
}

// (a, b) turned by (cos, sin).  One of the two products of each sum is rounded before it is added;
// which one is spelled out, because the compiler chose differently for different copies of an
// unrolled loop: the last eight rows of a tile (of every 128 rows for the 64-row tiles) had the
// product with the cosine rounded, the others that with the sine.  Kept so, row by row: every tile of
// up to 128 rows then gives a token the same bits, and calls give the bits they gave when 128 x 128
// was the smallest tile.
__device__ __forceinline__ void rotate_pair(float& a, float& b, float cos, float sin, bool sin_last) {
  const float as = a * sin, ac = a * cos, bs = b * sin, bc = b * cos;
  const float ra = sin_last ? fmaf(-b, sin, ac) : fmaf(a, cos, -bs);
  const float rb = sin_last ? fmaf(a, sin, bc) : fmaf(b, cos, as);
  a = ra; b = rb;
}

enum OutKind : int { OUT_BF16 = 0, OUT_F32 = 1 };

// Sum over aligned groups of G = 8 or 16 consecutive lanes; every lane of a group gets the sum.
template <int G> __device__ __forceinline__ float group_sum(float x) {
  static_assert(G == 8 || G == 16, "group size");
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0xB1, 0xF, 0xF, true));   // quad_perm 1,0,3,2
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x4E, 0xF, 0xF, true));   // quad_perm 2,3,0,1
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x141, 0xF, 0xF, true));  // row_half_mirror
  if constexpr (G == 16)
    x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x140, 0xF, 0xF, true));  // row_mirror
  return x;
}

constexpr int ROT_TABLE_ROUNDS = 2;  // rounds of blocks of a QKV launch up to which its rotary table goes through LDS (see the epilogue)
constexpr int MAX_PIECES = 4;       // pieces per gathered row that the ping-pong loop takes

// Rows of a matrix from `base` on, `bytes` of them in all: accesses beyond are dropped (loads give zero), which spares
// the epilogues a branch per access.  A lane that must not take part passes OUTSIDE as its offset.
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
constexpr uint32_t OUTSIDE = 0x80000000u;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_window(const void* base, size_t bytes) {
  // (made of scalars by hand: where the compiler does not see that they are, every access becomes a loop over the lanes)
  const uint64_t p = (uint64_t)base;
  const uint64_t u = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)p) | (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(p >> 32)) << 32;
  return __builtin_amdgcn_make_buffer_rsrc((void*)u, 0, __builtin_amdgcn_readfirstlane((int)bytes), 0x00027000);
}

template <int N> __device__ __forceinline__ void wait_vmcnt() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// Explicit LDS reads and counter waits (see the main loop of gemm_tile for why).
template <int OFF> __device__ __forceinline__ void ds_read_b128(bf16x8& d, uint32_t addr) {
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(d) : "v"(addr), "n"(OFF) : "memory");
}
template <int N, int STRIDE, int BASE, int I = 0> __device__ __forceinline__ void ds_read_rows(bf16x8* d, uint32_t addr) {
  if constexpr (I < N) {
    constexpr int off = BASE + I * STRIDE, hi = off & ~0xffff;   // the offset field holds 16 bits
    ds_read_b128<off - hi>(d[I], addr + (uint32_t)hi);
    ds_read_rows<N, STRIDE, BASE, I + 1>(d, addr);
  }
}
// wait until at most PENDING LDS reads of this wave are outstanding (they return in order),
// then tie the N fragments to the wait so that their consumers cannot be scheduled above it
// The compiler takes the result of an inline ds_read for valid at once: the ties keep the
// consumers behind the wait, and the scheduling barrier keeps any register copy the compiler
// makes for a tie behind it as well -- a copy hoisted above the wait reads a register the LDS
// has not filled yet (seen once, with a variant of the main loop; the generated code of every
// kernel is checked for such copies at build time, check_lds_waits.py).
template <int PENDING, int N, int N2> __device__ __forceinline__ void wait_lds_reads(bf16x8* f, bf16x8* f2) {
  asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(PENDING) : "memory");
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < N; ++i) asm volatile("" : "+v"(f[i]));
#pragma unroll
  for (int i = 0; i < N2; ++i) asm volatile("" : "+v"(f2[i]));
}

// f(integral_constant<int, 0>) ... f(integral_constant<int, N-1>), unrolled at compile time
template <class F, int... I> __device__ __forceinline__ void static_for_seq(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F> __device__ __forceinline__ void static_for(F&& f) {
  static_for_seq(f, std::make_integer_sequence<int, N>{});
}

// Compile-time description of one kernel variant.
template <int BM_, int BN_, int BK_, int WAVES_M_, int WAVES_N_, int MINBLK_, int PARTS_, int STAGES_, bool SPREAD_ = false, int PP_PARTS_ = 0>
struct Tile {
  static constexpr int BM = BM_, BN = BN_, BK = BK_, WAVES_M = WAVES_M_, WAVES_N = WAVES_N_;
  static constexpr int MINBLK = MINBLK_, STAGES = STAGES_;
  static constexpr bool SPREAD = SPREAD_;                // loads of a stage spread over the MFMAs of a step
  static constexpr int PP_PARTS = PP_PARTS_;             // ping-pong main loop: parts of a wave tile's rows, one per phase (0: plain loop)
  static constexpr bool PINGPONG = PP_PARTS > 0;
  static constexpr int NT = 64 * WAVES_M * WAVES_N;
  static constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N, TM = WM / 32, TN = WN / 32;
  static constexpr int TM16 = WM / 16, TN16 = WN / 16;   // 16 x 16 MFMA blocks per wave tile
  static constexpr int PARTS = PARTS_;                   // parts the A blocks of a k step are multiplied in
  static constexpr int STAT_COLS = BN < 128 ? BN : 128;  // columns per sum of squares that the residual epilogue leaves
  static constexpr int CPR = BK / 8;                     // 16-byte chunks per tile row
  static constexpr int LA = BM * CPR / NT, LW = BN * CPR / NT;   // load instructions per thread and stage
  static constexpr int STAGE_BYTES = (BM + BN) * BK * 2;
  static constexpr int LDS_BYTES = STAGES * STAGE_BYTES;
  static_assert(BK == 64, "BK: the main loop is written for two MFMA k steps of 32 per stage");
  static_assert((BM * CPR) % NT == 0 && (BN * CPR) % NT == 0, "tile / thread mismatch");
  static_assert(WM % 32 == 0 && WN % 32 == 0, "wave tile");
  // LDS has 64 banks of 4 bytes: a 16-byte-per-lane read is served 16 lanes (256 bytes) at a
  // time, so 16 consecutive rows must map to 16 different 16-byte columns modulo 256 bytes.
  __device__ static __forceinline__ int swz(int row) { return (row >> 1) & 7; }
};

// Ping-pong main loop (eight waves, WAVES_M = 2, two waves per SIMD).  The two wave rows run half a phase
// apart: while one multiplies, the other fetches its next fragments, so the matrix cores never wait for
// an LDS read, a barrier or the issue of a load.  The rows of a wave tile come in two parts and a K step
// is a phase per part:
//     fragment reads, waited for | barrier | matrix instructions, loads between them | barrier
// and wave row 1 passes one barrier more ahead of the loop (wave row 0 one behind it).  Operands come in
// units: part h of the rows of both wave rows, and all of W.  Unit u of a step is read in phase p(u), and
// its place in the ring is refilled, STAGES steps ahead, with the matrix instructions of phase q(u) > p(u)
// counted from the same step: by then both wave rows have read it, one barrier apart at most.  A wave waits
// for its loads of a unit in the phase before the one that reads it (the barriers between make that hold
// for the loads of all waves) and never for a later one.
//   What it replaced on the large tiles was one barrier per K step, behind which all waves read, waited and
// multiplied together: 256 x 256 x 64 took 3440 clocks of 2048 that the matrix instructions need, now 2390
// (320 x 256: 2930 of 2560).  LDS is not what bounds it (fragment reads run at 256 B per clock and unit, direct-
// to-LDS loads at 64: 768 and 1024 clocks a step).  Four phases a step of a quarter each: 2540; matrix
// instructions at raised priority: no difference.  8192^3, random operands: 1406 -> 1490 TFLOP/s (the chip's
// power limit; all-zero ones 1618 -> 1890), 32768 x 12800 x 3200 with GELU 1244 -> 1316, four clips 450 -> 432 ms.
template <class T> struct PingPong {
  static constexpr int S = T::STAGES, NP = T::PP_PARTS, NU = NP + 1;    // units in the order A0, W [, A1]
  // 16-row fragment blocks per part: ten of rows go as four and six, so that every wave issues as many loads
  static constexpr int NA0 = T::TM16 == 10 ? 4 : T::TM16 / NP, NA1 = T::TM16 - NA0, NW = T::TN16;
  static constexpr int p(int u) { return u / 2; }
  static constexpr int q(int u) { return u / 2 + 1; }
  static constexpr int blocks(int u) { return u == 1 ? NW : u == 2 ? NA1 : NA0; }
  static constexpr int loads(int u) { return (u == 1 ? 4 : 2) * blocks(u) / 4; }   // of 8 rows, 1 KB, per wave and unit
  // With `rem` steps behind the current one: this wave's loads that may be in flight at the wait of phase f
  // (-1: ahead of the loop), or -1 where the next phase reads no unit.  A load of step t (relative to the current
  // one) and unit u is issued in phase (t - S) * NP + q(u); loads are issued in that order.
  static constexpr int in_flight(int rem, int f) {
    int need = -1000000, n = 0;
    for (int t = 0; t <= 1 && t <= rem; ++t)
      for (int u = 0; u < NU; ++u)
        if (t * NP + p(u) == f + 1) { const int r = ((t - S) * NP + q(u)) * NU + u; need = r > need ? r : need; }
    if (need == -1000000) return -1;
    for (int t = 0; t <= rem && t <= 2 * S; ++t)
      for (int u = 0; u < NU; ++u) {
        const int ph = (t - S) * NP + q(u);
        if (ph * NU + u > need && ph < (f < 0 ? 0 : f)) n += loads(u);
      }
    return n;
  }
};

// Fragment reads of the ping-pong loop: blocks of 16 rows of one operand at offset OFF (f[2 * block + k half], k
// halves at a0 and a1), with them two blocks of the other one, and the wait for all of them -- in one
// asm block, so that no result is ever pending outside of it.
#define EPD_DSR(d, a, o) "ds_read_b128 %" #d ", %" #a " offset:%" #o "\n\t"
template <int N, int OFF> __device__ __forceinline__ void read_frags(bf16x8* f, uint32_t a0, uint32_t a1) {
  static_assert(N == 4 || N == 6, "blocks");
  if constexpr (N == 4) {
    asm volatile(EPD_DSR(0, 8, 10) EPD_DSR(2, 8, 11) EPD_DSR(4, 8, 12) EPD_DSR(6, 8, 13)
                 EPD_DSR(1, 9, 10) EPD_DSR(3, 9, 11) EPD_DSR(5, 9, 12) EPD_DSR(7, 9, 13) "s_waitcnt lgkmcnt(0)"
                 : "=&v"(f[0]), "=&v"(f[1]), "=&v"(f[2]), "=&v"(f[3]), "=&v"(f[4]), "=&v"(f[5]), "=&v"(f[6]), "=&v"(f[7])
                 : "v"(a0), "v"(a1), "n"(OFF), "n"(OFF + 2048), "n"(OFF + 4096), "n"(OFF + 6144) : "memory");
  } else {
    asm volatile(EPD_DSR(0, 12, 14) EPD_DSR(2, 12, 15) EPD_DSR(4, 12, 16) EPD_DSR(6, 12, 17)
                 EPD_DSR(8, 12, 18) EPD_DSR(10, 12, 19) EPD_DSR(1, 13, 14) EPD_DSR(3, 13, 15)
                 EPD_DSR(5, 13, 16) EPD_DSR(7, 13, 17) EPD_DSR(9, 13, 18) EPD_DSR(11, 13, 19) "s_waitcnt lgkmcnt(0)"
                 : "=&v"(f[0]), "=&v"(f[1]), "=&v"(f[2]), "=&v"(f[3]), "=&v"(f[4]), "=&v"(f[5]), "=&v"(f[6]), "=&v"(f[7]), "=&v"(f[8]), "=&v"(f[9]), "=&v"(f[10]), "=&v"(f[11])
                 : "v"(a0), "v"(a1), "n"(OFF), "n"(OFF + 2048), "n"(OFF + 4096), "n"(OFF + 6144), "n"(OFF + 8192), "n"(OFF + 10240) : "memory");
  }
}
template <int NA, int NW> __device__ __forceinline__ void read_frags_both(bf16x8* f, uint32_t a0, uint32_t a1, bf16x8* w, uint32_t w0, uint32_t w1) {
  static_assert(NA == 4 && (NW == 2 || NW == 4), "blocks");
  if constexpr (NW == 2) {
    asm volatile(EPD_DSR(8, 14, 16) EPD_DSR(10, 14, 17) EPD_DSR(0, 12, 16) EPD_DSR(2, 12, 17)
                 EPD_DSR(4, 12, 18) EPD_DSR(6, 12, 19) EPD_DSR(9, 15, 16) EPD_DSR(11, 15, 17)
                 EPD_DSR(1, 13, 16) EPD_DSR(3, 13, 17) EPD_DSR(5, 13, 18) EPD_DSR(7, 13, 19) "s_waitcnt lgkmcnt(0)"
                 : "=&v"(f[0]), "=&v"(f[1]), "=&v"(f[2]), "=&v"(f[3]), "=&v"(f[4]), "=&v"(f[5]), "=&v"(f[6]), "=&v"(f[7]), "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2]), "=&v"(w[3])
                 : "v"(a0), "v"(a1), "v"(w0), "v"(w1), "n"(0), "n"(2048), "n"(4096), "n"(6144) : "memory");
  } else {
    asm volatile(EPD_DSR(8, 18, 20) EPD_DSR(10, 18, 21) EPD_DSR(12, 18, 22) EPD_DSR(14, 18, 23)
                 EPD_DSR(0, 16, 20) EPD_DSR(2, 16, 21) EPD_DSR(4, 16, 22) EPD_DSR(6, 16, 23)
                 EPD_DSR(9, 19, 20) EPD_DSR(11, 19, 21) EPD_DSR(13, 19, 22) EPD_DSR(15, 19, 23)
                 EPD_DSR(1, 17, 20) EPD_DSR(3, 17, 21) EPD_DSR(5, 17, 22) EPD_DSR(7, 17, 23) "s_waitcnt lgkmcnt(0)"
                 : "=&v"(f[0]), "=&v"(f[1]), "=&v"(f[2]), "=&v"(f[3]), "=&v"(f[4]), "=&v"(f[5]), "=&v"(f[6]), "=&v"(f[7]), "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2]), "=&v"(w[3]), "=&v"(w[4]), "=&v"(w[5]), "=&v"(w[6]), "=&v"(w[7])
                 : "v"(a0), "v"(a1), "v"(w0), "v"(w1), "n"(0), "n"(2048), "n"(4096), "n"(6144) : "memory");
  }
}
#undef EPD_DSR

template <class T, int EPI, int OUT, bool VMODE, bool GATHER, bool FAST>
__device__ __forceinline__ void gemm_tile(const GemmArgs& g, const int m0, const int n0, char* const lds) {
  constexpr int BM = T::BM, BN = T::BN, BK = T::BK, NT = T::NT, WM = T::WM, WN = T::WN, TM = T::TM, TN = T::TN;
  constexpr int CPR = T::CPR, LA = T::LA, LW = T::LW;
  constexpr int ROWB = BK * 2;               // bytes per tile row
  constexpr int A_BYTES = BM * ROWB, W_BYTES = BN * ROWB;
  constexpr int S = T::STAGES, GL = LA + LW;   // ring stages; loads per thread and stage

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform: keeps LDS bases scalar
  const int wm = wave / T::WAVES_N, wn = wave % T::WAVES_N;
  const int l16 = lane & 15, g4 = lane >> 4;

  const char* zeros = (const char*)g.zeros;
  const int kcw = GATHER ? g.K / g.gather_n : g.K;

  // ---- per-thread load descriptors.  Load instruction `it` of a stage covers LDS chunks
  // it*NT + wave*64 + lane; chunk c is row c / CPR, slot c % CPR, and holds k-chunk
  // slot ^ swz(row) of that row.  One instruction covers RPP = NT / CPR rows (a multiple of
  // 16, so the swizzle of a lane's row is the same for every `it`).
  //   FAST (the caller guarantees that whole tiles of W, and of A unless its rows are gathered, may
  //   be read, also where they run past N or M, and K is a multiple of BK): the address is a wave-
  //   uniform row base, advanced with scalar arithmetic, plus ONE per-lane offset for all loads of an operand.
  //   Otherwise rows beyond M (or N) are clamped to the last valid row -- they only feed
  //   accumulators that are never stored -- and every load keeps its own per-lane offset.
  constexpr int RPP = NT / CPR;
  static_assert(RPP % 16 == 0, "rows per load instruction");
  const char* a_base_ptr = (const char*)g.A + (size_t)m0 * g.lda * 2;
  const int ldw = g.ldw ? g.ldw : g.K;
  const char* w_base_ptr = (const char*)g.W + (size_t)n0 * ldw * 2;
  constexpr int NOFF_A = FAST ? 1 : LA, NOFF_W = FAST ? 1 : LW;
  uint32_t a_off[NOFF_A], w_off[NOFF_W];
#pragma unroll
  for (int it = 0; it < NOFF_A; ++it) {
    const int c = it * NT + tid, row = c / CPR, col = (c % CPR) ^ T::swz(row);
    a_off[it] = (uint32_t)(FAST ? row : min(row, g.M - 1 - m0)) * (uint32_t)g.lda * 2u + col * 16;
  }
#pragma unroll
  for (int it = 0; it < NOFF_W; ++it) {
    const int c = it * NT + tid, row = c / CPR, col = (c % CPR) ^ T::swz(row);
    w_off[it] = (uint32_t)(FAST ? row : min(row, g.N - 1 - n0)) * (uint32_t)ldw * 2u + col * 16;
  }
  // first k of the chunk that load instruction `it` fetches (only the ragged-K and gather paths
  // need it, so it is recomputed there rather than kept in registers)
  auto chunk_k = [&](int it) {
    const int c = it * NT + tid, row = c / CPR;
    return ((c % CPR) ^ T::swz(row)) * 8;
  };

  // GATHER with pieces of whole K steps: a piece is the same for all lanes of a step, and the
  // rows it comes from are fetched when a new piece begins -- per step, the wait for them would
  // empty the ring of loads in flight every time
  // (small tiles: the large ones have no registers to spare for them)
  const bool whole_pieces = GATHER && LA <= 2 && kcw % BK == 0;
  [[maybe_unused]] int cur_piece = -1;
  [[maybe_unused]] int cur_src[LA];

  // TAIL = the K step that may run past K (only the last one, only when K % BK != 0):
  // chunks at k >= K are fetched from a zero buffer instead.
  // LDS: [A stage 0 | A stage 1 | ... | W stage 0 | W stage 1 | ...]
  //   Loads FROM .. TO - 1 of the LA + LW that bring K step k0 / BK into a stage.
  auto issue = [&](auto TAIL, auto FROM, auto TO, int stage, int k0) {
    constexpr bool tail = decltype(TAIL)::value;
    constexpr int from = decltype(FROM)::value, to = decltype(TO)::value;
    char* const sa = lds + stage * A_BYTES;
    char* const sw = lds + S * A_BYTES + stage * W_BYTES;
    const char* ab = a_base_ptr + (size_t)k0 * 2;
    const char* wb = w_base_ptr + (size_t)k0 * 2;
    // gathered operand (a stage's loads are then always issued in one run): the rows of all its
    // loads are fetched ahead of the first one, so that they are waited for once -- a row fetched
    // between two loads is waited for together with every load before it, and the opaque copies
    // below keep the compiler from moving it up (merger of four clips: 2150 us so, 1370 this way)
    static_assert(!GATHER || (from == 0 && to == GL), "a stage's loads in one run");
    [[maybe_unused]] int src[LA], piece[LA];
    if constexpr (GATHER) {
      if (whole_pieces) {
        if (k0 / kcw != cur_piece) {
          cur_piece = k0 / kcw;
#pragma unroll
          for (int it = 0; it < LA; ++it)
            cur_src[it] = g.gather[(size_t)(m0 + min((it * NT + tid) / CPR, g.M - 1 - m0)) * g.gather_n + cur_piece];
        }
#pragma unroll
        for (int it = 0; it < LA; ++it) { piece[it] = cur_piece; src[it] = cur_src[it]; }
      } else {
#pragma unroll
        for (int it = 0; it < LA; ++it) {
          piece[it] = min((k0 + chunk_k(it)) / kcw, g.gather_n - 1);
          src[it] = g.gather[(size_t)(m0 + min((it * NT + tid) / CPR, g.M - 1 - m0)) * g.gather_n + piece[it]];
        }
      }
    }
    // The per-lane offsets pass through an opaque copy here, so that their widening to 64 bits
    // stays next to the load: "scalar base + 32-bit lane offset" is then the load's own
    // addressing form.  Widened once ahead of the loop, every offset would occupy a register
    // pair for the whole loop and every load would need a 64-bit vector add in front of it.
    // (one copy per load: a shared one would let the adds be re-associated into a running
    // 64-bit vector address again)
#pragma unroll
    for (int ld = from; ld < to; ++ld) {
      const bool is_a = ld < LA;
      const int it = is_a ? ld : ld - LA;
      uint32_t off = is_a ? a_off[FAST ? 0 : it] : w_off[FAST ? 0 : it];
      if (!(GATHER && is_a)) asm volatile("" : "+v"(off));
      const char* p;
      if (is_a) {
        if constexpr (GATHER) {
          p = (const char*)g.A + ((size_t)src[it] * g.lda + (k0 + chunk_k(it) - piece[it] * kcw)) * 2;
        } else if constexpr (FAST) {
          p = (ab + (size_t)(it * RPP) * (size_t)g.lda * 2) + (size_t)off;
        } else {
          p = ab + (size_t)off;
        }
      } else {
        if constexpr (FAST) p = (wb + (size_t)(it * RPP) * (size_t)ldw * 2) + (size_t)off;
        else p = wb + (size_t)off;
      }
      if constexpr (tail) { if (k0 + chunk_k(it) >= g.K) p = zeros; }
      __builtin_amdgcn_global_load_lds(EPD_GPTR(p), EPD_LPTR((is_a ? sa : sw) + (it * NT + wave * 64) * 16), 16, 0, 0);
    }
  };
  // Folded RMSNorm (consumer side): scale of row m = rsqrt(mean of squares + eps), from the
  // per-segment sums the producing GEMM left.  Computed first, so that the loads complete in
  // the shadow of the main loop, and kept in LDS behind the stages and the staging area (the
  // barriers of the main loop make it visible to the epilogue).
  float* const row_scale = (float*)(lds + T::LDS_BYTES);
  constexpr bool CONSUMER = EPI == EPI_GELU || EPI == EPI_QKV;
  const bool scaled = CONSUMER && g.stats_in != nullptr;
  // The order of the additions is the same whichever tile left the sums and whichever takes them:
  // sums of 64 columns (stats_n * 64 = K) are added in pairs first, which is how a tile of 128 columns
  // makes one, then 8 segments (hidden 1024) as a tree, any other number one after the other.
  // Hidden 1024: the 8 or (small tiles only) 16 sums of a row are loaded here, ahead of the first
  // operand loads, and only consumed after the first barrier
  static_assert(BM <= NT, "one row scale per thread");
  constexpr int SV = BM * BN <= 128 * 128 ? 4 : 2;       // 16-byte loads held
  const bool halves = g.stats_n * 64 == g.K;             // sums of 64 columns
  const bool scaled_v = scaled && g.K == 1024 && g.stats_n <= 4 * SV;
  float4 st[SV];
  if (scaled_v) {
#pragma unroll
    for (int j = 0; j < SV; ++j) st[j] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (tid < BM) {
      const float4* sp = (const float4*)(g.stats_in + (size_t)min(m0 + tid, g.M - 1) * g.stats_n);
      st[0] = sp[0]; st[1] = sp[1];
      if constexpr (SV == 4) { if (halves) { st[2] = sp[2]; st[3] = sp[3]; } }
    }
  } else if (scaled) {
    for (int r = tid; r < BM; r += NT) {
      const float* sp = g.stats_in + (size_t)min(m0 + r, g.M - 1) * g.stats_n;
      auto segment = [&](int j) { return halves ? sp[2 * j] + sp[2 * j + 1] : sp[j]; };
      float ss = 0.f;
      if (SV == 2 && g.K == 1024) {                      // 16 sums in front of a large tile
        ss = ((segment(0) + segment(1)) + (segment(2) + segment(3))) + ((segment(4) + segment(5)) + (segment(6) + segment(7)));
      } else {
        const int n = halves ? g.stats_n / 2 : g.stats_n;
        for (int j = 0; j < n; ++j) ss += segment(j);
      }
      row_scale[r] = 1.0f / sqrtf(fmaf(ss, g.stats_inv_dim, g.stats_eps));
    }
  } else if (CONSUMER) {
    for (int r = tid; r < BM; r += NT) row_scale[r] = 1.0f;
  }

  // The epilogue's bias values (4 columns per 16-column block of the lane) are fetched here, so that their
  // latency passes in the shadow of the main loop; the largest tile has no registers to spare for them
  // and fetches them in the epilogue
  constexpr int TN16 = T::TN16;
  constexpr bool BIAS_USED = !VMODE && EPI != EPI_RESIDUAL && OUT == OUT_BF16, BIAS_PRE = BIAS_USED && BM * BN <= 256 * 256;
  [[maybe_unused]] uint2 bb[TN16];
  auto load_bias = [&]() {
#pragma unroll
    for (int w = 0; w < TN16; ++w) {
      const int nb = n0 + wn * WN + w * 16 + g4 * 4;
      bb[w] = (g.bias && nb < g.N) ? *(const uint2*)((const uint16_t*)g.bias + nb) : make_uint2(0u, 0u);   // N is a multiple of 4
    }
  };
  if constexpr (BIAS_PRE) load_bias();

  const int nk = (g.K + BK - 1) / BK;
  const bool ragged_k = (g.K % BK) != 0;
  using ALL0 = std::integral_constant<int, 0>;
  using ALLN = std::integral_constant<int, GL>;
  auto issue_step = [&](int stage, int kt) {      // kt < nk
    if constexpr (FAST) {
      issue(std::false_type{}, ALL0{}, ALLN{}, stage, kt * BK);
    } else {
      if (ragged_k && kt == nk - 1) issue(std::true_type{}, ALL0{}, ALLN{}, stage, kt * BK);
      else issue(std::false_type{}, ALL0{}, ALLN{}, stage, kt * BK);
    }
  };

  // acc[i][j][q]: the 32 x 32 block (i, j) of the wave tile as four 16 x 16 MFMA results,
  // q = 2 * (token half) + (column half)
  f32x4 acc[TM][TN][4];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[i][j][q][v] = 0.f;

  // ---- LDS fragment reads.  Issued as explicit ds_read_b128 so that their order against the
  // direct-to-LDS loads and the waits below is exactly the one written here (a compiler-
  // visible LDS read that follows a direct-to-LDS load in program order gets a full wait for
  // that load inserted in front of it, which would serialise the two-stage ring).
  // One fragment = 16 rows x 32 k: lane (l16, g4) reads k chunk 4*ks + g4 of row blk*16 + l16;
  // multiples of 16 keep swz(row) = swz(l16).  A stage is multiplied in 2 * P slices,
  // slice sl = (k step ks = sl / P, part p = sl % P of the A blocks): slice (ks, 0) needs the
  // TN16 W fragments of the k step and the first AP A fragments, the others the next AP A
  // fragments.  W fragments alternate between two buffers by k step, A fragments by slice.
  constexpr int TM16 = T::TM16, P = T::PARTS, AP = TM16 / P, NSL = 2 * P;
  static_assert(TM16 % P == 0 && TN16 + AP <= 15, "slices / LDS counter");
  const uint32_t lds0 = (uint32_t)(size_t)EPD_LPTR(lds);
  // Address of k step 1 = address of k step 0 with bit 6 flipped (chunk slot bit 2; the row
  // base has a zero there); stage and 16-row block go into the instruction's offset field.
  const uint32_t a_rd0 = lds0 + (wm * WM + l16) * ROWB + ((g4 ^ T::swz(l16)) * 16);
  const uint32_t w_rd0 = lds0 + S * A_BYTES + (wn * WN + l16) * ROWB + ((g4 ^ T::swz(l16)) * 16);
  bf16x8 fw[2][TN16], fa[2][AP];
  auto read_slice = [&](auto SL, auto ST) {
    constexpr int sl = decltype(SL)::value, st = decltype(ST)::value, ks = sl / P, p = sl % P;
    if constexpr (p == 0) ds_read_rows<TN16, 16 * ROWB, st * W_BYTES>(&fw[ks][0], w_rd0 ^ (uint32_t)(ks * 64));
    ds_read_rows<AP, 16 * ROWB, st * A_BYTES + p * AP * 16 * ROWB>(&fa[sl & 1][0], a_rd0 ^ (uint32_t)(ks * 64));
  };
  // wait until at most the reads of the next slice are outstanding (none with DRAIN: every
  // read of the wave has returned), then tie the slice's fragments to the wait
  auto wait_slice = [&](auto SL, auto DRAIN) {
    constexpr int sl = decltype(SL)::value, ks = sl / P, p = sl % P;
    constexpr int next_reads = ((sl + 1) % P == 0 ? TN16 : 0) + AP;
    wait_lds_reads<(decltype(DRAIN)::value ? 0 : next_reads), AP, (p == 0 ? TN16 : 0)>(&fa[sl & 1][0], &fw[ks][0]);
  };
  // Multiply slice SL.  Meanwhile (REFILL) its share of the loads that refill the stage before
  // this one is issued, one load after every few matrix instructions: a wave issues in order and
  // the address unit takes a 1 KB load every 18 cycles or so, so a whole stage's loads in one run
  // leave the matrix cores idle for as long as they take.
  constexpr int MPS = AP * TN16;                        // matrix instructions per slice
  constexpr bool LATE_REFILL = TM * TN <= 4;
  constexpr int LSL = S == 2 && NSL > 4 ? NSL / 2 : NSL - 1;    // slices that issue loads (never the last one)
  auto mfmas = [&](auto SL, auto REFILL, int stage, int k0) {
    constexpr int sl = decltype(SL)::value, ks = sl / P, p = sl % P;
    constexpr int l0 = sl < LSL ? GL * sl / LSL : GL, l1 = sl < LSL ? GL * (sl + 1) / LSL : GL, nl = l1 - l0;
    static_for<MPS>([&](auto I) {
      constexpr int i = decltype(I)::value;
      // consecutive MFMAs keep their first operand: measured ~7% faster than alternating it
      constexpr int t = VMODE ? i / TN16 : i % AP, w = VMODE ? i % TN16 : i / AP;
      constexpr int a16 = p * AP + t;
      f32x4& c = acc[a16 >> 1][w >> 1][(a16 & 1) * 2 + (w & 1)];
      if constexpr (VMODE) c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[sl & 1][t], fw[ks][w], c, 0, 0, 0);
      else c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[ks][w], fa[sl & 1][t], c, 0, 0, 0);
      if constexpr (decltype(REFILL)::value && nl > 0) {
        constexpr int b0 = l0 + nl * i / MPS, b1 = l0 + nl * (i + 1) / MPS;
        if constexpr (b1 > b0) {
          __builtin_amdgcn_sched_barrier(0);
          issue(std::false_type{}, std::integral_constant<int, b0>{}, std::integral_constant<int, b1>{}, stage, k0);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    });
  };
  using I0 = std::integral_constant<int, 0>;
  using LAST = std::integral_constant<int, NSL - 1>;

  // What the epilogue adds to or multiplies with the accumulators of a 16-token block: as many fp32 values as it has --
  // of the residual rows (EPI_RESIDUAL, lanes along rows), or cos and sin of the lane's rotary pairs (EPI_QKV).
  // Where all of it is at most 16 loads they are issued behind the last stage hand-over, so that they
  // overlap the last K step; otherwise AUX blocks are kept in flight through the epilogue.
  //   A rotary table that comes through LDS (`table`) needs none of these loads: issued all the same, and waited for
  // ahead of the table, they took the 256 x 128 tile's QKV launch of 12 544 x 960 x 320 from 25.8 to 30.0 us (28.0 without a
  // table).  On its plain loop (K in parts of steps) the entries are not fetched ahead at all: 6272 x 3240 x 1080 80.7 us, 83
  // with the prefetch.
  constexpr int FC = WN / 4, FR = 64 / FC;              // lanes per row of fp32 values, rows per access of a wave
  constexpr bool HAS_AUX = !VMODE && (EPI == EPI_RESIDUAL || EPI == EPI_QKV);
  constexpr bool PREF = HAS_AUX && TM16 * TN16 <= 16 && !(EPI == EPI_QKV && T::PINGPONG && !FAST);
  [[maybe_unused]] constexpr bool ROT_TABLE = HAS_AUX && EPI == EPI_QKV && T::PINGPONG;
  [[maybe_unused]] constexpr int TAB_BYTES = T::LDS_BYTES - T::WAVES_M * T::WAVES_N * 16 * WN * 2;   // what the bf16 staging pieces leave
  const bool table = ROT_TABLE && g.rot && g.rot_lds && BM * g.rot_pairs * 8 <= TAB_BYTES;
  constexpr int AUX = PREF ? TM16 : BM > 256 ? (EPI == EPI_QKV ? 2 : 3) : 4;
  [[maybe_unused]] float4 aux[HAS_AUX ? AUX : 1][TN16];
  const int rows_left = max(0, min(WM, g.M - m0 - wm * WM));       // rows of the wave's tile that exist
  [[maybe_unused]] const uint32_t aux_pitch = EPI == EPI_QKV ? (uint32_t)g.rot_pairs * 8u : (uint32_t)g.ldr * 4u;
  [[maybe_unused]] uint32_t aux_off[EPI == EPI_QKV ? TN16 : 1];
  [[maybe_unused]] __amdgpu_buffer_rsrc_t aux_rows;
  if constexpr (HAS_AUX) {
    aux_rows = row_window((EPI == EPI_QKV ? (const char*)g.rot : (const char*)g.resid) + (size_t)(m0 + wm * WM) * aux_pitch, (size_t)rows_left * aux_pitch);
    if constexpr (EPI == EPI_QKV) {
#pragma unroll
      for (int w = 0; w < TN16; ++w) aux_off[w] = (uint32_t)l16 * aux_pitch + (uint32_t)(((n0 + wn * WN + w * 16 + g4 * 4) % g.head_dim) >> 1) * 8u;
    } else {
      const int n = n0 + wn * WN + (lane % FC) * 4;
      aux_off[0] = n < g.N ? (uint32_t)(lane / FC) * aux_pitch + (uint32_t)n * 4u : OUTSIDE;
    }
  }
  auto load_aux = [&](int b) {
    if constexpr (HAS_AUX) {
#pragma unroll
      for (int w = 0; w < TN16; ++w) {
        const uint32_t off = aux_off[EPI == EPI_QKV ? w : 0] + (uint32_t)(b * 16 + (EPI == EPI_QKV ? 0 : w * FR)) * aux_pitch;
        aux[b % AUX][w] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(aux_rows, off, 0, 0));
      }
    }
  };
  auto prefetch_aux = [&]() {
    if constexpr (PREF) {
      if (EPI == EPI_QKV && (!g.rot || table)) return;
#pragma unroll
      for (int b = 0; b < TM16; ++b) load_aux(b);
    }
  };

  // ---- main loop: a ring of S LDS stages.  The hand-over to the next stage happens before the
  // last slice of the current stage is multiplied: wait for the own loads of the next stage
  // (those of up to S - 2 later ones stay in flight), barrier (everybody's loads landed,
  // everybody finished reading this stage), start reading the next one -- and only then issue the
  // MFMAs of the last slice, which cover the barrier and the LDS latency.  The freed stage is
  // refilled at once, or (SPREAD tiles) between the MFMAs of the next step.
  auto wait_later = [&](int later) {      // loads of at most min(later, S - 2) stages stay in flight
    bool done = false;
    static_for<S - 1>([&](auto I) {
      constexpr int k = S - 2 - decltype(I)::value;
      if (!done && later >= k) { wait_vmcnt<k * GL>(); done = true; }
    });
  };
  static_assert(S >= 2 && (S - 2) * GL < 64, "ring, load counter");
  // the sums of squares held since before the first operand load
  auto store_row_scale = [&]() {
    if (scaled_v && tid < BM) {
      float ss = ((st[0].x + st[0].y) + (st[0].z + st[0].w)) + ((st[1].x + st[1].y) + (st[1].z + st[1].w));
      if constexpr (SV == 4) ss += ((st[2].x + st[2].y) + (st[2].z + st[2].w)) + ((st[3].x + st[3].y) + (st[3].z + st[3].w));
      row_scale[tid] = 1.0f / sqrtf(fmaf(ss, g.stats_inv_dim, g.stats_eps));
    }
  };
  if constexpr (T::PINGPONG && FAST) {
    using PP = PingPong<T>;
    static_assert(T::WAVES_M == 2 && T::WAVES_N == 4 && PP::NP == 2, "ping-pong tile");
    constexpr int NP = PP::NP, NW = PP::NW;
    // a load covers 8 rows that start at a multiple of 8, odd for odd waves: its lanes' offsets are the same for all
    // loads of a wave
    const int lrow = lane >> 3, lcol = ((lane & 7) ^ T::swz((wave & 1) * 8 + lrow)) * 16;
    const uint32_t a_lane = (uint32_t)lrow * (uint32_t)g.lda * 2u + lcol, w_lane = (uint32_t)lrow * (uint32_t)ldw * 2u + lcol;
    // gathered operand: the tile's row numbers lie in LDS, [piece][row]; those of a wave's loads are fetched into
    // registers when a new piece begins (pieces are whole K steps), ahead of the phase that issues the loads
    [[maybe_unused]] const uint32_t idx0 = lds0 + (uint32_t)(T::LDS_BYTES + BM * 4);
    [[maybe_unused]] int src[GATHER ? 2 : 1][GATHER ? 3 : 1], piece[2] = {-1, -1}, kin[2] = {0, 0};
    if constexpr (GATHER) {
      int* const idx = (int*)(lds + T::LDS_BYTES + BM * 4);
      for (int r = tid; r < BM; r += NT)
        for (int c = 0; c < g.gather_n; ++c) idx[c * BM + r] = g.gather[(size_t)min(m0 + r, g.M - 1) * g.gather_n + c];
      __syncthreads();
    }
    auto tile_row = [&](auto U, int j) {     // first row of load j of unit U
      constexpr int u = decltype(U)::value, per = PP::blocks(u) * 2;   // loads per wave row / column
      const int n = j * 8 + wave;
      return (n / per) * (u != 1 ? WM : WN) + (u == 2 ? PP::NA0 * 16 : 0) + (n % per) * 8;
    };
    // called once per step and unit, in order, ahead of the unit's loads
    auto next_rows = [&](auto U) {
      constexpr int u = decltype(U)::value, h = u / 2;
      if constexpr (GATHER && u != 1) {
        kin[h] += BK;
        if (piece[h] < 0 || kin[h] == kcw) {
          kin[h] = 0; ++piece[h];
#pragma unroll
          for (int j = 0; j < PP::loads(u); ++j) {
            const uint32_t at = idx0 + (uint32_t)(piece[h] * BM + tile_row(U, j) + lrow) * 4u;
            int row;
            asm volatile("ds_read_b32 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=v"(row) : "v"(at) : "memory");
            src[h][j] = row;
          }
        }
      }
    };
    auto load = [&](auto U, auto J, int stage, int kt) {
      constexpr int u = decltype(U)::value, j = decltype(J)::value;
      const int row = tile_row(U, j);
      char* const dst = lds + (u != 1 ? stage * A_BYTES : S * A_BYTES + stage * W_BYTES) + row * ROWB;
      if constexpr (GATHER && u != 1) {
        constexpr int h = u / 2;
        const char* from = (const char*)g.A + (size_t)kin[h] * 2 + lcol + (uint64_t)(uint32_t)src[h][j] * ((uint32_t)g.lda * 2u);
        __builtin_amdgcn_global_load_lds(EPD_GPTR(from), EPD_LPTR(dst), 16, 0, 0);
        return;
      }
      uint32_t off = u != 1 ? a_lane : w_lane;
      asm volatile("" : "+v"(off));          // see issue()
      const char* base = u != 1 ? a_base_ptr + ((size_t)row * g.lda + (size_t)kt * BK) * 2 : w_base_ptr + ((size_t)row * ldw + (size_t)kt * BK) * 2;
      __builtin_amdgcn_global_load_lds(EPD_GPTR(base + (size_t)off), EPD_LPTR(dst), 16, 0, 0);
    };
    auto load_unit = [&](auto U, int stage, int kt) {
      next_rows(U);
      static_for<PP::loads(decltype(U)::value)>([&](auto J) { load(U, J, stage, kt); });
    };
    bf16x8 pa[2 * PP::NA1], pw[2 * NW];
    // loads ahead of the loop: everything the loop does not issue
    static_for<S>([&](auto TT) {
      static_for<PP::NU>([&](auto U) {
        constexpr int t = decltype(TT)::value;
        if constexpr ((t - S) * NP + PP::q(decltype(U)::value) < 0) { if (t < nk) load_unit(U, t, t); }
      });
    });
    if (nk >= S) wait_vmcnt<PP::in_flight(2 * S, -1)>();
    else wait_vmcnt<0>();
    __builtin_amdgcn_s_barrier();
    store_row_scale();
    if (wm == 1) __builtin_amdgcn_s_barrier();
    auto phase = [&](auto P, auto REM, int t, int stg) {
      constexpr int p = decltype(P)::value, rem = decltype(REM)::value, NA = p ? PP::NA1 : PP::NA0, NM = NA * NW * 2;
      const uint32_t a0 = a_rd0 + stg * A_BYTES, w0 = w_rd0 + stg * W_BYTES;
      static_for<PP::NU>([&](auto U) {
        constexpr int u = decltype(U)::value, ahead = S + (p - PP::q(u) < 0 ? -1 : 0);
        if constexpr (PP::q(u) % NP == p && ahead <= rem) next_rows(U);
      });
      if constexpr (p == 0) read_frags_both<PP::NA0, NW>(pa, a0, a0 ^ 64u, pw, w0, w0 ^ 64u);
      else read_frags<PP::NA1, PP::NA0 * 2048>(pa, a0, a0 ^ 64u);
      constexpr int keep = PP::in_flight(rem, p);
      if constexpr (keep >= 0) wait_vmcnt<keep>();
      if constexpr (rem == 0 && p == 0) prefetch_aux();
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
      static_for<NM>([&](auto I) {
        constexpr int i = decltype(I)::value, ks = i / (NW * NA), w = i / NA % NW, x = i % NA, a16 = p * PP::NA0 + x;
        f32x4& c = acc[a16 >> 1][w >> 1][(a16 & 1) * 2 + (w & 1)];
        if constexpr (VMODE) c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pa[2 * x + ks], pw[2 * w + ks], c, 0, 0, 0);
        else c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pw[2 * w + ks], pa[2 * x + ks], c, 0, 0, 0);
        // units refilled in this phase, their loads spread over the instructions
        static_for<PP::NU>([&](auto U) {
          constexpr int u = decltype(U)::value, ahead = S + (p - PP::q(u) < 0 ? -1 : 0);
          if constexpr (PP::q(u) % NP == p && ahead <= rem) {
            constexpr int n = PP::loads(u);
            static_for<n>([&](auto J) {
              if constexpr (i == NM * (2 * decltype(J)::value + 1) / (2 * n)) {
                __builtin_amdgcn_sched_barrier(0);
                int ns = stg + ahead; ns = ns >= S ? ns - S : ns;
                load(U, J, ns, t + ahead);
                __builtin_amdgcn_sched_barrier(0);
              }
            });
          }
        });
      });
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
    };
    int t = 0, stg = 0;
    for (; t + S < nk; ++t) {
      static_for<NP>([&](auto P) { phase(P, std::integral_constant<int, 2 * S>{}, t, stg); });
      if (++stg == S) stg = 0;
    }
    static_for<S>([&](auto R) {              // the last S steps: fewer loads, and fewer to wait for
      constexpr int rem = S - 1 - decltype(R)::value;
      if (nk > rem) {
        static_for<NP>([&](auto P) { phase(P, std::integral_constant<int, rem>{}, t, stg); });
        ++t;
        if (++stg == S) stg = 0;
      }
    });
    if (wm == 0) __builtin_amdgcn_s_barrier();
  } else {
  static_for<S - 1>([&](auto ST) { if (nk > decltype(ST)::value) issue_step(decltype(ST)::value, decltype(ST)::value); });
  wait_later(nk - 1);
  __builtin_amdgcn_s_barrier();
  store_row_scale();
  constexpr bool INNER_LOOP = FAST && T::SPREAD;
  if (!INNER_LOOP && nk > S - 1) issue_step(S - 1, S - 1);
  read_slice(I0{}, I0{});

  auto step = [&](auto ST, auto INNER, int kt) {
    constexpr int s = decltype(ST)::value, sp = (s + S - 1) % S;    // sp: the stage to refill, with K step kt + S - 1
    constexpr bool inner = decltype(INNER)::value;                  // a full ring of steps and loads follows
    using SN = std::integral_constant<int, (s + 1) % S>;
    const int k0 = (kt + S - 1) * BK;
    // the fragments of slice sl+1 are requested before slice sl is multiplied
    static_for<NSL - 1>([&](auto SL) {
      read_slice(std::integral_constant<int, decltype(SL)::value + 1>{}, ST);
      wait_slice(SL, std::false_type{});
      mfmas(SL, INNER, sp, k0);
    });
    // last slice: stage hand-over first
    if (inner || kt + 1 < nk) {
      if constexpr (inner) wait_vmcnt<(S - 2) * GL>();
      else wait_later(nk - 2 - kt);
      wait_slice(LAST{}, std::true_type{});
      __builtin_amdgcn_s_barrier();
      if constexpr (!inner && !LATE_REFILL) { if (kt + S < nk) issue_step(s, kt + S); }
      read_slice(I0{}, SN{});
      if constexpr (!inner) { if (kt + 2 >= nk) prefetch_aux(); }          // last hand-over: no operand load follows
    } else {
      wait_slice(LAST{}, std::true_type{});
    }
    mfmas(LAST{}, std::false_type{}, 0, 0);
    if constexpr (!inner && LATE_REFILL) {
      // small wave tiles: the refill of stage s is issued behind the queued MFMAs, so the
      // address arithmetic and load instructions run in their shadow (pinning this order
      // costs registers, which the large wave tiles do not have)
      __builtin_amdgcn_sched_barrier(0);
      if (kt + S < nk) issue_step(s, kt + S);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  int kt = 0;
  if constexpr (INNER_LOOP) {        // no branches while every step refills a stage
    constexpr int AHEAD = S == 2 ? 3 : 2 * S - 2;      // the last hand-over stays with the loop below
    for (; kt + AHEAD < nk; kt += S)
      static_for<S>([&](auto ST) { step(ST, std::true_type{}, kt + decltype(ST)::value); });
  }
  if (INNER_LOOP && kt + S - 1 < nk) issue_step(S - 1, kt + S - 1);
  for (; kt < nk; kt += S)
    static_for<S>([&](auto ST) {
      if (kt + decltype(ST)::value < nk) step(ST, std::false_type{}, kt + decltype(ST)::value);
    });
  if (nk == 1) prefetch_aux();
  }

  // ------------------------------------------------------------------ epilogue
  if constexpr (VMODE) {
    // The MFMA operands are swapped for these tiles, so a lane holds 4 consecutive tokens of
    // one channel: scale and bias are applied there, and 16 channels x up to 128 tokens at a time are staged
    // in a piece of LDS of the wave's own, [channel][token]; a lane then takes 8 consecutive tokens (one 16-byte
    // store) of a channel row.  (Staged by the whole block, channel halves on the 320-row tile: 19.4 k clocks a tile.)
    const uint16_t* bias = (const uint16_t*)g.bias;
    uint16_t* vt = (uint16_t*)g.vt;
    float bv[TN16];
#pragma unroll
    for (int w = 0; w < TN16; ++w) {
      const int n = n0 + wn * WN + w * 16 + l16;
      bv[w] = bias && n < g.N ? bf16_bits_to_float(bias[n]) : 0.f;
    }
    static_assert(T::WAVES_M * T::WAVES_N * 16 * 256 <= T::LDS_BYTES, "transposed staging area");
    char* const stg = lds + wave * 16 * 256;
    __builtin_amdgcn_s_barrier();                        // the operand stages are dead from here on (all reads of them were waited for)
    auto part = [&](auto FIRST, auto COUNT) {            // 16-token blocks FIRST .. FIRST + COUNT - 1 of the wave's rows
      constexpr int b0 = decltype(FIRST)::value, nb = decltype(COUNT)::value;
      constexpr int CHV = 2 * nb, RPV = 64 / CHV;        // 8-token chunks per channel row, rows per read
      auto chunk = [](int row, int c) { return row * (nb * 32) + ((nb == 8 ? c ^ row : nb == 4 ? c ^ T::swz(row) : c ^ ((row >> 2) & 3)) * 16); };
      const int m = m0 + wm * WM + b0 * 16 + (lane % CHV) * 8;
      int4 vc0 = make_int4(0, 0, 0, 0), vc1 = make_int4(0, 0, 0, 0);
      const bool full = m + 7 < g.M;
      if (full) { vc0 = *(const int4*)(g.vcol + m); vc1 = *(const int4*)(g.vcol + m + 4); }
      // eight tokens side by side, or twice four: items whose first token is a multiple of four and not of eight
      const bool eight = full && (vc1.w - vc0.x == 7) && ((vc0.x & 7) == 0);
      const bool fours = full && vc0.w - vc0.x == 3 && vc1.w - vc1.x == 3 && ((vc0.x | vc1.x) & 3) == 0;
#pragma unroll
      for (int w = 0; w < TN16; ++w) {
#pragma unroll
        for (int b = 0; b < nb; ++b) {
          const f32x4 a = acc[(b0 + b) >> 1][w >> 1][((b0 + b) & 1) * 2 + (w & 1)];
          const float4 rs = *(const float4*)(row_scale + wm * WM + (b0 + b) * 16 + g4 * 4);
          *(uint2*)(stg + chunk(l16, b * 2 + (g4 >> 1)) + (g4 & 1) * 8) =
              pack_bf16x4(fmaf(a[0], rs.x, bv[w]), fmaf(a[1], rs.y, bv[w]), fmaf(a[2], rs.z, bv[w]), fmaf(a[3], rs.w, bv[w]));
        }
        asm volatile("" ::: "memory");                   // other lanes' pieces are read below: LDS takes a wave's accesses in order
        uint4 p[16 / RPV];
#pragma unroll
        for (int k = 0; k < 16 / RPV; ++k) p[k] = *(const uint4*)(stg + chunk(k * RPV + lane / CHV, lane % CHV));
        asm volatile("" ::: "memory");
#pragma unroll
        for (int k = 0; k < 16 / RPV; ++k) {
          const int n = n0 + wn * WN + w * 16 + k * RPV + lane / CHV;
          if (n >= g.N || m >= g.M) continue;
          uint16_t* vrow = vt + (size_t)(n - g.qk_cols) * g.vt_stride;
          if (eight) {
            *(uint4*)(vrow + vc0.x) = p[k];
          } else if (fours) {
            *(uint2*)(vrow + vc0.x) = make_uint2(p[k].x, p[k].y);
            *(uint2*)(vrow + vc1.x) = make_uint2(p[k].z, p[k].w);
          } else {
            const uint32_t u[4] = {p[k].x, p[k].y, p[k].z, p[k].w};
            for (int t = 0; t < 8 && m + t < g.M; ++t) vrow[g.vcol[m + t]] = (uint16_t)(u[t >> 1] >> ((t & 1) * 16));
          }
        }
      }
    };
    static_assert(TM16 == 2 || TM16 == 4 || TM16 == 8 || TM16 == 10, "token parts");
    part(I0{}, std::integral_constant<int, TM16 < 8 ? TM16 : 8>{});
    if constexpr (TM16 == 10) part(std::integral_constant<int, 8>{}, std::integral_constant<int, 2>{});
  } else {
    // Everything else goes 16 tokens x WN columns at a time through a piece of LDS of the wave's own, from which it
    // leaves as whole 128- or 256-byte lines: no wave waits for another.  bf16 results are finished where the
    // accumulators stand -- a lane holds four consecutive columns of one token in each 16-column block; fp32 rows
    // (residual stream, fp32 outputs) are turned first, then read and written as rows (from where the
    // accumulators stand an access touches 16 rows of 64 bytes each: residual add of 256 x 256, 35 k clocks).
    //   It replaced passes of the whole block over row or column slices of the tile in fp32, a barrier or two each,
    // with the rotary table copied to LDS or (head_dim 128) read where it was used.  Clocks per 256 x 256 tile:
    // residual add 38.6 k -> 17.8 k (with all units at it, HBM at its limit, 70 k -> 37 k), GELU 19.9 k -> 9.1 k, Q | K with
    // rotary 22 k -> 16 k (its table: 64-byte pieces of rows, half the address unit's rate), plain store 6.0 k -> 3.9 k.
    constexpr bool F32_ROWS = EPI == EPI_RESIDUAL || OUT == OUT_F32;
    constexpr int SROW = WN * (F32_ROWS ? 4 : 2), CH = SROW / 16, RPI = 64 / CH;   // bytes and 16-byte chunks per staged row, rows per read
    constexpr int STG_BYTES = T::WAVES_M * T::WAVES_N * 16 * SROW;
    static_assert(STG_BYTES + T::WAVES_N * BM * 4 <= T::LDS_BYTES, "staging area");
    if constexpr (BIAS_USED && !BIAS_PRE) load_bias();
    __builtin_amdgcn_s_barrier();                        // the operand stages are dead from here on (all reads of them were waited for)
    char* const stg = lds + wave * 16 * SROW;
    // rows of 256 bytes: chunk ^ row; of 128 (64): two (four) rows share the banks' 256 bytes
    auto schunk = [](int row, int c) { return row * SROW + ((SROW == 256 ? c ^ row : SROW == 128 ? c ^ T::swz(row) : c ^ ((row >> 2) & 3)) * 16); };
    if constexpr (F32_ROWS) {
      const int n = n0 + wn * WN + (lane % FC) * 4;      // N is a multiple of 4: all or nothing
      const bool sums = EPI == EPI_RESIDUAL && g.stats_out != nullptr;
      const uint32_t out_pitch = EPI == EPI_RESIDUAL ? (uint32_t)g.ldxb * 2u : (uint32_t)g.ldo * 4u;
      const uint32_t out_off = n < g.N ? (uint32_t)(lane / FC) * out_pitch + (uint32_t)n * (EPI == EPI_RESIDUAL ? 2u : 4u) : OUTSIDE;
      const char* const out0 = EPI == EPI_RESIDUAL ? (const char*)g.xb : (const char*)g.out;      // no bf16 copy wanted: an empty window
      const __amdgpu_buffer_rsrc_t out_rows = row_window(out0 + (size_t)(m0 + wm * WM) * out_pitch, out0 ? (size_t)rows_left * out_pitch : 0);
      float* const part = (float*)(lds + T::WAVES_M * T::WAVES_N * 16 * SROW);   // [WAVES_N][BM] sums of squares per wave
      uint2 br = make_uint2(0u, 0u);
      if (g.bias && n < g.N) br = *(const uint2*)((const uint16_t*)g.bias + n);
      const float b0 = bf16_bits_to_float(br.x & 0xffff), b1 = bf16_bits_to_float(br.x >> 16);
      const float b2 = bf16_bits_to_float(br.y & 0xffff), b3 = bf16_bits_to_float(br.y >> 16);
      [[maybe_unused]] float ss = 0.f;
      if constexpr (HAS_AUX && !PREF) {
#pragma unroll
        for (int b = 0; b < AUX; ++b) load_aux(b);
      }
#pragma unroll
      for (int b = 0; b < TM16; ++b) {
#pragma unroll
        for (int w = 0; w < TN16; ++w) {
          const f32x4 a = acc[b >> 1][w >> 1][(b & 1) * 2 + (w & 1)];
          *(float4*)(stg + schunk(l16, w * 4 + g4)) = make_float4(a[0], a[1], a[2], a[3]);
        }
        asm volatile("" ::: "memory");                 // other lanes' pieces are read below: LDS takes a wave's accesses in order
#pragma unroll
        for (int w = 0; w < TN16; ++w) {
          const int c = b * TN16 + w;                  // rows c * FR + lane / FC of the wave's tile
          const float4 e = *(const float4*)(stg + schunk(w * FR + lane / FC, lane % FC));
          const float v0 = e.x + b0, v1 = e.y + b1, v2 = e.z + b2, v3 = e.w + b3;
          if constexpr (EPI == EPI_RESIDUAL) {
            float4 x = aux[b % AUX][w];
            x.x += v0; x.y += v1; x.z += v2; x.w += v3;
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, x), aux_rows, aux_off[0] + (uint32_t)(c * FR) * aux_pitch, 0, 0);
            // folded RMSNorm (producer side): the raw rows in bf16 for the next GEMM, and their sums of squares per
            // STAT_COLS columns, which are two or four waves' shares; lane c % FC of a row's lanes keeps the sum of its row c
            __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, pack_bf16x4(x.x, x.y, x.z, x.w)), out_rows, out_off + (uint32_t)(c * FR) * out_pitch, 0, 0);
            // (made also where nobody takes them: a branch here would cut the loops into pieces that do not overlap)
            const float r = group_sum<FC>(fmaf(x.x, x.x, fmaf(x.y, x.y, fmaf(x.z, x.z, x.w * x.w))));
            ss = lane % FC == c % FC ? r : ss;
            if (c % FC == FC - 1 || c == TM16 * TN16 - 1) {
              const int row = (c / FC * FC + lane % FC) * FR + lane / FC;
              if (c % FC == FC - 1 || row < WM) part[wn * BM + wm * WM + row] = ss;
            }
          } else {
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, make_float4(v0, v1, v2, v3)), out_rows, out_off + (uint32_t)(c * FR) * out_pitch, 0, 0);
          }
        }
        if constexpr (HAS_AUX && !PREF) { if (b + AUX < TM16) load_aux(b + AUX); }
        asm volatile("" ::: "memory");
      }
      if (sums) {
        __syncthreads();
        constexpr int SEGS = BN / T::STAT_COLS, WPS = T::WAVES_N / SEGS;
        static_assert(WPS == 2 || WPS == 4, "waves per sum");
        for (int r = tid; r < BM * SEGS; r += NT) {
          const int seg = r / BM, ml = r % BM, m = m0 + ml;
          const float* const p = part + seg * WPS * BM + ml;
          float sum = p[0] + p[BM];
          if constexpr (WPS == 4) sum += p[2 * BM] + p[3 * BM];
          if (m < g.M && n0 + seg * T::STAT_COLS < g.N) g.stats_out[(size_t)m * g.stats_n + n0 / T::STAT_COLS + seg] = sum;
        }
      }
    } else {
      uint16_t* const outp = (uint16_t*)g.out;
      const int ns = n0 + wn * WN + (lane % CH) * 8;     // first column of the lane's 16-byte piece of a staged row
      const uint32_t out_pitch = (uint32_t)g.ldo * 2u, out_off = ns < g.N ? (uint32_t)(lane / CH) * out_pitch + (uint32_t)ns * 2u : OUTSIDE;
      const __amdgpu_buffer_rsrc_t out_rows = row_window(outp + (size_t)(m0 + wm * WM) * g.ldo, (size_t)rows_left * out_pitch);
      float bias[TN16][4], qs[TN16];
#pragma unroll
      for (int w = 0; w < TN16; ++w) {
        bias[w][0] = bf16_bits_to_float(bb[w].x & 0xffff); bias[w][1] = bf16_bits_to_float(bb[w].x >> 16);
        bias[w][2] = bf16_bits_to_float(bb[w].y & 0xffff); bias[w][3] = bf16_bits_to_float(bb[w].y >> 16);
        // the softmax scale (in log2 units) rides on Q: one rounding of q * scale instead of
        // a multiply per score in the attention kernel
        qs[w] = n0 + wn * WN + w * 16 + g4 * 4 < g.q_cols ? g.q_scale : 1.0f;
      }
      // Large tiles: the rotary table's rows for the tile's tokens are one slab of memory, which comes to LDS in whole
      // lines behind the staging pieces (its 16-byte chunks swizzled, so that 16 tokens' entries lie in different
      // banks); fetched from memory where they are used, entries are 64-byte pieces of 16 rows per access, at half the
      // address unit's rate and once per wave: 6272 x 3072 x 1024 44.2 -> 40.2 us in 320 x 256 tiles, the call of eight
      // images 5570 -> 5434 us.  Only in launches of up to two rounds of the units the call runs on.  Longer ones in 256 x 128
      // tiles lose alone (12 544 x 3264 x 1088 109.8 -> 113.4 us, 18 816 x 3600 x 1200 230 -> 240).  In 256 x 256 and 320 x 256
      // tiles they gain alone (37 632 x 3072 x 1024 246 -> 232, 25 088 x 3840 x 1280 237 -> 234) and whole calls go
      // either way, the clock of the attention beside them with it: 20 ... 48 images at hidden 1024 0.9 % less, 32 ragged images
      // the same, 10 ... 14 k tokens at hidden 1152 the same, 20 k 0.7 % and five resolutions 1.5 % more.  So the line does not
      // stand where a call of every width would have it; it keeps what was measured to lose out.
      const uint32_t trb = (uint32_t)g.rot_pairs * 8u, cpr = trb / 16;          // bytes and 16-byte chunks per token
      auto swr = [&](int row) { return cpr == 16 || cpr == 32 ? row & 15 : cpr == 8 ? (row >> 1) & 7 : 0; };
      char* const tab = lds + STG_BYTES;
      [[maybe_unused]] uint32_t tab_off[TN16];
      if constexpr (ROT_TABLE) {
        if (table) {
          const float inv = 1.0f / (float)cpr;
          for (int c0 = wave * 64; c0 < BM * (int)cpr; c0 += NT) {
            const int c = c0 + lane, row = (int)(((float)c + 0.5f) * inv), pos = c - row * (int)cpr;
            const char* from = (const char*)g.rot + (size_t)min(m0 + row, g.M - 1) * trb + (pos ^ swr(row)) * 16;
            __builtin_amdgcn_global_load_lds(EPD_GPTR(from), EPD_LPTR(tab + c0 * 16), 16, 0, 0);
          }
#pragma unroll
          for (int w = 0; w < TN16; ++w)
            tab_off[w] = (uint32_t)(wm * WM + l16) * trb + (uint32_t)((((n0 + wn * WN + w * 16 + g4 * 4) % g.head_dim) >> 2) ^ swr(l16)) * 16u;
          wait_vmcnt<0>();
          __builtin_amdgcn_s_barrier();
        }
      }
      // VARIANT 1: tanh instead of erf (GELU), rotary embedding (QKV; 2: from the table in LDS), rows that do not start on
      // 16 bytes (STORE; N and ldo are multiples of 8) -- outside of the loops, so that these are one
      // block of code in which loads, arithmetic and stores of different tokens overlap
      auto rows = [&](auto VARIANT) {
        constexpr int variant = decltype(VARIANT)::value;
        if constexpr (variant == 1 && HAS_AUX && !PREF) {
#pragma unroll
          for (int b = 0; b < AUX; ++b) load_aux(b);
        }
#pragma unroll
        for (int b = 0; b < TM16; ++b) {
          const int ml = wm * WM + b * 16 + l16;
          const float rs = CONSUMER ? row_scale[ml] : 1.0f;
#pragma unroll
          for (int w = 0; w < TN16; ++w) {
            const f32x4 a = acc[b >> 1][w >> 1][(b & 1) * 2 + (w & 1)];
            float v0 = fmaf(a[0], rs, bias[w][0]), v1 = fmaf(a[1], rs, bias[w][1]), v2 = fmaf(a[2], rs, bias[w][2]), v3 = fmaf(a[3], rs, bias[w][3]);
            if constexpr (EPI == EPI_GELU) {
              if constexpr (variant == 0) { v0 = gelu_erf_fast(v0); v1 = gelu_erf_fast(v1); v2 = gelu_erf_fast(v2); v3 = gelu_erf_fast(v3); }
              else { v0 = gelu_tanh_fast(v0); v1 = gelu_tanh_fast(v1); v2 = gelu_tanh_fast(v2); v3 = gelu_tanh_fast(v3); }
            } else if constexpr (EPI == EPI_QKV) {
              if constexpr (variant != 0) {
                const float4 cs = variant == 2 ? *(const float4*)(tab + tab_off[w] + (uint32_t)(b * 16) * trb) : aux[b % AUX][w];
                const bool sin_last = b == TM16 - 1 && (BM >= 128 ? ml >= BM - 8 : (m0 & 64) && ml >= 56);
                rotate_pair(v0, v1, cs.x, cs.y, sin_last);
                rotate_pair(v2, v3, cs.z, cs.w, sin_last);
              }
              v0 *= qs[w]; v1 *= qs[w]; v2 *= qs[w]; v3 *= qs[w];
            }
            *(uint2*)(stg + schunk(l16, w * 2 + (g4 >> 1)) + (g4 & 1) * 8) = pack_bf16x4(v0, v1, v2, v3);
          }
          if constexpr (variant == 1 && HAS_AUX && !PREF) { if (b + AUX < TM16) load_aux(b + AUX); }
          asm volatile("" ::: "memory");                 // other lanes' pieces are read below: LDS takes a wave's accesses in order
#pragma unroll
          for (int k = 0; k < 16 / RPI; ++k) {
            const int r = k * RPI + lane / CH;
            const uint4 v = *(const uint4*)(stg + schunk(r, lane % CH));
            if constexpr (EPI == EPI_STORE && variant == 1) {
              const int m = m0 + wm * WM + b * 16 + r;
              const uint32_t u[4] = {v.x, v.y, v.z, v.w};
              if (m < g.M && ns < g.N)
                for (int t = 0; t < 8; ++t) outp[(size_t)m * g.ldo + ns + t] = (uint16_t)(u[t >> 1] >> ((t & 1) * 16));
            } else {
              __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), out_rows, out_off + (uint32_t)(b * 16 + k * RPI) * out_pitch, 0, 0);
            }
          }
          asm volatile("" ::: "memory");
          if constexpr (BM > 256) __builtin_amdgcn_sched_barrier(0);
        }
      };
      if ((EPI == EPI_GELU && g.act != 0) || (EPI == EPI_QKV && g.rot) || (EPI == EPI_STORE && ((size_t)outp & 15))) {
        if constexpr (ROT_TABLE) { if (table) { rows(std::integral_constant<int, 2>{}); return; } }
        rows(std::integral_constant<int, 1>{});
      } else {
        rows(std::integral_constant<int, 0>{});
      }
    }
  }
}

// Consecutive hardware block ids go to different XCDs (8 per chip, each with its own 4 MB
// L2).  Remap so that every XCD walks a contiguous range of tile numbers, and number the tiles
// in groups of `group_m` row tiles swept column by column: the tiles an XCD runs at the same
// time then form a compact rectangle whose A panels stay in its L2 while W panels stream
// through once, instead of every XCD re-reading all of W for every row of tiles.
__device__ __forceinline__ int xcd_remap(int bid, int nblocks) {
  const int q = nblocks >> 3, r = nblocks & 7;
  const int xcd = bid & 7, idx = bid >> 3;
  return xcd * q + min(xcd, r) + idx;
}

__device__ __forceinline__ void tile_coords(int t, int tiles_m, int tiles_n, int group_m, int& tm, int& tn) {
  const int per_group = group_m * tiles_n;
  const int grp = t / per_group, local = t - grp * per_group;
  const int first = grp * group_m;
  const int rows = min(group_m, tiles_m - first);
  tn = local / rows;
  tm = first + (local - tn * rows);
}

// TAG changes nothing in the code: it gives the two residual GEMMs of a block (attention output
// projection, second MLP GEMM) kernel names of their own, so that a profile lists them apart.
template <class T, int EPI, int OUT, bool GATHER, bool FAST, int TAG>
__global__ __launch_bounds__(T::NT, T::MINBLK) void gemm_bf16_kernel(GemmArgs g) {
  // + per-row scales of the epilogue + the row numbers of a gathered operand (ping-pong loop)
  __shared__ __attribute__((aligned(1024))) char lds[T::LDS_BYTES + T::BM * 4 + (GATHER && FAST ? T::BM * MAX_PIECES * 4 : 0)];
  const int tiles_n = (g.N + T::BN - 1) / T::BN, tiles_m = (g.M + T::BM - 1) / T::BM;
  int tm, tn;
  tile_coords(xcd_remap(blockIdx.x, gridDim.x), tiles_m, tiles_n, g.group_m, tm, tn);
  const int m0 = tm * T::BM, n0 = tn * T::BN;
  if constexpr (EPI == EPI_QKV) {
    if (n0 >= g.qk_cols) {
      gemm_tile<T, EPI, OUT, true, false, FAST>(g, m0, n0, lds);
      return;
    }
  }
  gemm_tile<T, EPI, OUT, false, GATHER, FAST>(g, m0, n0, lds);
}

static int num_cus() {
  static int n = [] {
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v <= 0)
      v = 256;
    return v;
  }();
  return n;
}

template <class T, int EPI, int OUT, bool GATHER>
static void launch_cfg(const GemmArgs& g, hipStream_t s) {
  const int tiles_m = (g.M + T::BM - 1) / T::BM, tiles_n = (g.N + T::BN - 1) / T::BN;
  const long blocks = (long)T::MINBLK * (g.compute_units > 0 ? g.compute_units : num_cus());     // of one round
  GemmArgs a = g;
  a.rot_lds = EPI == EPI_QKV && (long)tiles_m * tiles_n <= ROT_TABLE_ROUNDS * blocks;
  if (a.group_m <= 0) {
    // keep the A panels of one group (group_m x BM rows x K) within about 2 MB of the 4 MB L2
    const long panel = (long)T::BM * g.K * 2;
    a.group_m = (int)std::max(1L, std::min((long)tiles_m, (2L << 20) / std::max(panel, 1L)));
    // Long K (panels beyond the cache) and a wide output: the 32 tiles an XCD runs at a time still
    // advance through K together, so what has to stay cached is their current K window, not whole
    // panels.  Four row tiles per group make that set 4 x 8 tiles (12 operand panels) instead of
    // 1 x 32 (33 panels): +5 % on 32768 x 12800 x 3200 and 32768 x 9600 x 3200; narrow outputs
    // (13 column tiles) measured best with the panel rule alone.
    if (tiles_n >= 24) a.group_m = std::max(a.group_m, 4);
    // Few rows against a large weight matrix (the merger projection): with row groups every
    // XCD streams all of W.  When the whole grid runs in at most two rounds, number the tiles
    // column by column instead, so that an XCD owns a block of columns: W is then fetched
    // once in total and the (smaller) A once per XCD.
    if ((long)g.N > 2L * g.M && (long)tiles_m * tiles_n <= 2 * blocks) a.group_m = tiles_m;
  }
  a.group_m = std::min(a.group_m, tiles_m);
  if constexpr (!GATHER) {
    if (g.overread_a && g.overread_w && g.K % T::BK == 0) {
      if (EPI == EPI_RESIDUAL && g.name_tag == 1)
        hipLaunchKernelGGL((gemm_bf16_kernel<T, EPI, OUT, false, true, (EPI == EPI_RESIDUAL ? 1 : 0)>), dim3(tiles_m * tiles_n), dim3(T::NT), 0, s, a);
      else
        hipLaunchKernelGGL((gemm_bf16_kernel<T, EPI, OUT, false, true, 0>), dim3(tiles_m * tiles_n), dim3(T::NT), 0, s, a);
      return;
    }
  }
  if constexpr (GATHER && T::PINGPONG) {
    if (g.overread_w && g.gather_n <= MAX_PIECES && g.K % (g.gather_n * T::BK) == 0) {
      hipLaunchKernelGGL((gemm_bf16_kernel<T, EPI, OUT, true, true, 0>), dim3(tiles_m * tiles_n), dim3(T::NT), 0, s, a);
      return;
    }
  }
  hipLaunchKernelGGL((gemm_bf16_kernel<T, EPI, OUT, GATHER, false, 0>), dim3(tiles_m * tiles_n), dim3(T::NT), 0, s, a);
}

// 256 x 128 serves QKV where 2 * hidden is not a multiple of 256, and narrow outputs (plan_tiles).  Ping-pong loop: 1385
// clocks a K step of 1024; 25 088 x 3264 x 1088 270 -> 204 us (128 x 128 tiles: 198).
//            BM   BN  BK  WM WN MINBLK PARTS STAGES
using T0 = Tile<256, 256, 64, 2, 4, 1, 4, 2, false, 2>;   // 8 waves, 128x64 wave tiles, 128 KB LDS, one block per CU
using T2 = Tile<256, 128, 64, 2, 4, 1, 4, 3, false, 2>;   // 8 waves, 128x32 wave tiles, 144 KB LDS, one block per CU
using T4 = Tile<128, 128, 64, 2, 2, 2, 4, 2>;   // 4 waves, 64x64 wave tiles, 64 KB LDS, two blocks per CU
using T5 = Tile<320, 256, 64, 2, 4, 1, 5, 2, false, 2>;   // 8 waves, 160x64 wave tiles, 144 KB LDS, one block per CU

using T7 = Tile<64, 64, 64, 2, 2, 2, 1, 4, true>;    // 4 waves, 32x32 wave tiles, 64 KB LDS, two blocks per CU
using T8 = Tile<64, 128, 64, 2, 2, 2, 1, 3, true>;   // 4 waves, 32x64 wave tiles, 72 KB LDS, two blocks per CU

// Tile choice.  Both large tiles run one block per compute unit, so an output whose number of
// tiles is not a multiple of the unit count pays a whole tile time for its last, partial round,
// and nothing hides their epilogues.  The 128 x 128 tile runs two blocks per unit (the epilogue of
// one hides behind the main loop of the other) and quantises four times finer, but its main loop
// is the slowest.  The 320 x 256 tile moves the fewest operand bytes per flop.  A launch is priced
// by a model: the time of one round of blocks is, per 256 x 256 of output area,
// alpha * K / 1024 + eps[epilogue]  microseconds:
//                  alpha   eps: store / GELU   residual add (K >= 2048)   QKV + rotary
//   256 x 256      22.6        13.2               39.4 (25.0)                 21.9
//   320 x 256      21.8        11.7               39.4 (24.5)                 24.8
//   128 x 128      32.8         4.6               23.8                        19.6
// All but the figures in brackets were fitted to launch times inside encoder calls (where the chip sits at its
// power limit; loops of one GEMM alone rank the tiles differently) when the large tiles still had one barrier per K step and
// block-wide epilogues.  Since then launches in them have become 4 to 20 % shorter (73 896 x 3072 x 1024 in 256 x 256 tiles:
// the model says 623 us, measured 469; 32 768 x 9600 x 3200: 1758 and 1617), those in 128 x 128 tiles, which kept their
// loop, 0 to 12 %: the ranking leans towards the small tile.  Every tile forced on residual adds of 3136 ... 31 360 rows,
// hidden 1024, 1152 and 1600 (profiles/residual_tiles.txt): from K = 2048 on what is planned is within 3 % of the best tile in 79 of
// 84 launches (8 % off in the worst); at K = 1280 ... 1792 in 36 of 63, and up to 15 % off where 128 x 128 tiles are taken
// and 256 x 256 would be faster (12 544 x 1024 x 1280: 56.0 and 48.9 us).  Whole batches, all products
// (profiles/gemm_tile_model_fit.txt): 22 of 25 planned launches within 3 % of the best tile; behind it are the output
// projections of 73 896 and 85 500 rows (275 us in 128 x 128 tiles, 241 in 320 x 256; 316 and 289) and the merger of 1568 (84, 63 in 256 x 128).
bool gemm_bf16_tile_known(int t) { return t == 0 || t == 2 || t == 4 || t == 5 || t == 7 || t == 8; }
struct TileShape { int bm, bn, blocks, cfg; double alpha, eps[4]; };   // eps indexed by Epilogue
// Few rows: 64 x 64 and 64 x 128 tiles, whose stages are refilled three and two steps ahead between
// the matrix instructions.  Their main loops are slower still per output (LDS reads), but a call
// with one to four images has too few large tiles to occupy the chip, and each of those takes as
// long as on a full one: 784 x 1024 x 4096 is 56 tiles of 128 x 128 in 61 us, 208 of 64 x 64 in 21
// (784 x 3072 x 1024: 23 us, 64 x 128 tiles 16).  They are offered while they fit two rounds of
// blocks; beyond, the large tiles fill the chip themselves (3136 x 3072 x 1024: 1 round of 256 x 256
// tiles 32 us, 64 x 64 in four rounds 44).  Their constants rank, they do not predict: measured in
// calls with every tile forced, 196 ... 4608 tokens at hidden 1024, 1152 and 3200 (profiles/gemm_tile_few_rows.txt), the tile
// chosen is within 3 % of the fastest in 59 of 70 launches and within 11 % in all but one (merger of 1152 rows: 74 us, 59 in
// 256 x 128), while the model is off by up to a factor of two on single launches.
constexpr TileShape kShape256 = {256, 256, 1, 0, 22.6, {13.2, 13.2, 39.4, 21.9}};
constexpr TileShape kShape320 = {320, 256, 1, 5, 21.8, {11.7, 11.7, 39.4, 24.8}};
constexpr TileShape kShape128 = {128, 128, 2, 4, 32.8, {4.6, 4.6, 23.8, 19.6}};
constexpr TileShape kShape64 = {64, 64, 2, 7, 39.0, {41.0, 41.0, 59.0, 41.0}};
constexpr TileShape kShape64x128 = {64, 128, 2, 8, 33.3, {22.5, 22.5, 36.7, 22.7}};
constexpr double kSecondLaunch = 4.0;      // what a second launch of the same GEMM adds (gap + ramp), same unit

constexpr TileShape kShape256x128 = {256, 128, 1, 2, 19.3, {30.0, 30.0, 30.0, 30.0}};
// Against a long K the large tiles' residual add costs less: the tiles of a launch drift apart, and not all of them
// are at HBM together (73 896 x 1024 x 4096: 558 us in 256 x 256 tiles, 543 in 320 x 256; 20 676 x 1152 x 4352: 218 in 256 x
// 256, 240 in 128 x 128; 28 224 x 1152 x 4352: 277 in 320 x 256, 326 in 128 x 128).  The line at 2048 is on the safe side: no
// launch of 4704 ... 36 064 rows, hidden 768 ... 1600, K = 2048, 2560, 3072 or 4096 takes longer than in the tiles that the constants
// for a short K chose, on the kernels of then; below the line the large tiles gain already (see above).
constexpr int kLongK = 2048;
constexpr double kLongEps256 = 25.0, kLongEps320 = 24.5;

static double tile_cost(int M, int N, int K, int epi, const TileShape& t, long cus) {
  const long tiles = (long)((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn);
  const long slots = cus * t.blocks;
  double eps = t.eps[epi & 3];
  if (epi == EPI_RESIDUAL && K >= kLongK) eps = t.bm == 320 ? kLongEps320 : t.bm == 256 && t.bn == 256 ? kLongEps256 : eps;
  const double per_round = (double)t.blocks * t.bm * t.bn / 65536.0 * (t.alpha * K / 1024.0 + eps);
  return (double)((tiles + slots - 1) / slots) * per_round;
}

// How to cover an M x N output: one launch of `tile`, or (body_rows > 0) the first body_rows rows
// with `tile` and the rest with smaller ones (`tail_tile`).  The second form cuts the output behind the last
// full round of the large tile, so that what would have been a partial round of whole-tile
// times becomes a round of small tiles: 32768 x 3200 in 256 x 256 tiles is 1664 tiles = 6.5
// rounds, priced 7; cut after 30208 rows it is 6 rounds plus 500 small tiles.
struct TilePlan { int tile, body_rows; double cost; int tail_tile; };

static TilePlan plan_tiles(int M, int N, int K, int epi, bool may_split, long cus) {
  TilePlan best = {0, 0, tile_cost(M, N, K, epi, kShape256, cus), 0};
  const double keep = 0.98 * best.cost;          // the plain 256 x 256 launch stays unless clearly beaten
  auto offer = [&](int tile, int body_rows, double cost, int tail_tile = 0) {
    if (cost < keep && cost < best.cost) best = {tile, body_rows, cost, tail_tile};
  };
  offer(kShape128.cfg, 0, tile_cost(M, N, K, epi, kShape128, cus));
  offer(kShape320.cfg, 0, tile_cost(M, N, K, epi, kShape320, cus));
  for (const TileShape* t : {&kShape64, &kShape64x128}) {
    const long tiles = (long)((M + t->bm - 1) / t->bm) * ((N + t->bn - 1) / t->bn);
    if (tiles <= 2 * cus * t->blocks) offer(t->cfg, 0, tile_cost(M, N, K, epi, *t, cus));
  }
  auto one_round_256x128 = [&](int rows) { return epi == EPI_RESIDUAL && K >= kLongK && (long)((rows + 255) / 256) * ((N + 127) / 128) <= cus; };
  // Narrow outputs against a long K in one round of 256 x 128 tiles: 6272 x 1024 x 4096 56 us against 61 in 128 x 128
  // tiles and 78 in 256 x 256; K = 2048 36.7 and 38.4.  (Only this is priced by kShape256x128's constants.  Against a short K
  // 128 x 128 tiles take as long: K = 1024 25.2 and 25.4 us, 1536 32.2 and 32.5.  In several
  // rounds the larger tiles, which move fewer operand bytes, are faster: 20 676 x 1152 x 4352 227 us against
  // 218, 73 896 x 1024 x 4096 668 against 543.)
  if (one_round_256x128(M))
    offer(kShape256x128.cfg, 0, tile_cost(M, N, K, epi, kShape256x128, cus));
  if (may_split) {
    for (const TileShape* t : {&kShape256, &kShape320}) {
      const long tm = (M + t->bm - 1) / t->bm, tn = (N + t->bn - 1) / t->bn;
      const long full = tm * tn / cus;                       // complete rounds of the large tile
      if (full < 1 || (tm * tn) % cus == 0) continue;
      const long body_tm = std::min(full * cus / tn, (long)(M / t->bm));   // whole row tiles within them
      if (body_tm < 1 || body_tm * t->bm >= M) continue;
      const int body_rows = (int)body_tm * t->bm;
      // the tail in 128 x 128 tiles, or in one round of 256 x 128 against a long K (2112 x 3200 x 12800: 202 us in the former)
      const int rest = M - body_rows;
      double tail = tile_cost(rest, N, K, epi, kShape128, cus);
      int tail_tile = kShape128.cfg;
      if (one_round_256x128(rest)) {
        const double c = tile_cost(rest, N, K, epi, kShape256x128, cus);
        if (c < tail) { tail = c; tail_tile = kShape256x128.cfg; }
      }
      offer(t->cfg, body_rows, tile_cost(body_rows, N, K, epi, *t, cus) + tail + kSecondLaunch, tail_tile);
    }
  }
  return best;
}

template <int EPI, int OUT, bool GATHER>
static void launch_epi(const GemmArgs& g, hipStream_t s) {
  int t = g.tile_cfg > 0 ? g.tile_cfg - 1 : -1;   // tile_cfg: set by the tuning hook of the C ABI, or by a split
  if (!gemm_bf16_tile_known(t)) t = plan_tiles(g.M, g.N, g.K, g.epilogue, false, g.compute_units > 0 ? g.compute_units : num_cus()).tile;
  if (EPI == EPI_QKV && (t == 0 || t == 5) && g.qk_cols % 256 != 0) t = 2;
  switch (t) {
    case 0: launch_cfg<T0, EPI, OUT, GATHER>(g, s); break;
    case 2: launch_cfg<T2, EPI, OUT, GATHER>(g, s); break;
    case 5: launch_cfg<T5, EPI, OUT, GATHER>(g, s); break;
    case 7: launch_cfg<T7, EPI, OUT, GATHER>(g, s); break;
    case 8: launch_cfg<T8, EPI, OUT, GATHER>(g, s); break;
    default: launch_cfg<T4, EPI, OUT, GATHER>(g, s); break;
  }
}

constexpr int kQkvBN = 128;

static void launch_gemm_bf16_whole(const GemmArgs& g, hipStream_t s);

// a forced tile, gathered rows, or Q | K columns that do not end on a 256-column boundary (those
// run the 256 x 128 tile): one launch
static bool may_split_rows(const GemmArgs& g) {
  return g.tile_cfg == 0 && !g.gather && !(g.epilogue == EPI_QKV && g.qk_cols % 256 != 0);
}

void plan_gemm_bf16(const GemmArgs& g, int compute_units, int* tile_rows, int* tile_cols, int* body_rows) {
  const long cus = compute_units > 0 ? compute_units : (g.compute_units > 0 ? g.compute_units : num_cus());
  int t = g.tile_cfg > 0 ? g.tile_cfg - 1 : -1, body = 0;
  if (!gemm_bf16_tile_known(t)) {
    const TilePlan p = plan_tiles(g.M, g.N, g.K, g.epilogue, may_split_rows(g), cus);
    t = p.tile; body = p.body_rows;
  }
  if (g.epilogue == EPI_QKV && (t == 0 || t == 5) && g.qk_cols % 256 != 0) t = 2;
  *tile_rows = t == 7 || t == 8 ? 64 : t == 4 ? 128 : t == 5 ? 320 : 256;
  *tile_cols = t == 7 ? 64 : t == 0 || t == 5 ? 256 : 128;
  *body_rows = body;
}

int gemm_bf16_stat_cols(const GemmArgs& g) {
  int rows, cols, body;
  plan_gemm_bf16(g, 0, &rows, &cols, &body);
  return cols < 128 ? cols : 128;
}

void launch_gemm_bf16(const GemmArgs& g, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0) return;
  const TilePlan plan = may_split_rows(g) ? plan_tiles(g.M, g.N, g.K, g.epilogue, true, g.compute_units > 0 ? g.compute_units : num_cus()) : TilePlan{0, 0, 0.0, 0};
  if (plan.body_rows <= 0) { launch_gemm_bf16_whole(g, s); return; }
  const int mb = plan.body_rows;
  GemmArgs body = g, tail = g;
  body.M = mb; body.tile_cfg = plan.tile + 1;
  tail.M = g.M - mb; tail.tile_cfg = plan.tail_tile + 1;
  // everything indexed by the output row moves down by mb rows (vt is indexed through vcol)
  tail.A = (const __bf16*)g.A + (size_t)mb * g.lda;
  if (g.out) tail.out = g.out_f32 ? (void*)((float*)g.out + (size_t)mb * g.ldo) : (void*)((__bf16*)g.out + (size_t)mb * g.ldo);
  if (g.resid) tail.resid = g.resid + (size_t)mb * g.ldr;
  if (g.xb) tail.xb = (__bf16*)g.xb + (size_t)mb * g.ldxb;
  if (g.stats_out) tail.stats_out = g.stats_out + (size_t)mb * g.stats_n;
  if (g.stats_in) tail.stats_in = g.stats_in + (size_t)mb * g.stats_n;
  if (g.rot) tail.rot = g.rot + (size_t)mb * g.rot_pairs;
  if (g.vcol) tail.vcol = g.vcol + mb;
  launch_gemm_bf16_whole(body, s);
  launch_gemm_bf16_whole(tail, s);
}

static void launch_gemm_bf16_whole(const GemmArgs& g, hipStream_t s) {
  switch (g.epilogue) {
    case EPI_STORE:
      if (g.gather) launch_epi<EPI_STORE, OUT_BF16, true>(g, s);
      else if (g.out_f32) launch_epi<EPI_STORE, OUT_F32, false>(g, s);
      else launch_epi<EPI_STORE, OUT_BF16, false>(g, s);
      break;
    case EPI_GELU:
      launch_epi<EPI_GELU, OUT_BF16, false>(g, s);
      break;
    case EPI_RESIDUAL:
      launch_epi<EPI_RESIDUAL, OUT_F32, false>(g, s);
      break;
    case EPI_QKV:
      if (g.qk_cols % kQkvBN == 0) {
        launch_epi<EPI_QKV, OUT_BF16, false>(g, s);
      } else {
        // a column tile would straddle the K | V boundary: run the two parts separately
        GemmArgs qk = g;
        qk.N = g.qk_cols;
        launch_epi<EPI_QKV, OUT_BF16, false>(qk, s);
        GemmArgs v = g;
        v.W = (const __bf16*)g.W + (size_t)g.qk_cols * (g.ldw ? g.ldw : g.K);
        v.bias = g.bias ? (const void*)((const __bf16*)g.bias + g.qk_cols) : nullptr;
        v.N = g.N - g.qk_cols;
        v.qk_cols = 0;
        launch_epi<EPI_QKV, OUT_BF16, false>(v, s);
      }
      break;
  }
}

}  // namespace epd
