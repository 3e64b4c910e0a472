// Calls of the library's internal bf16 GEMM launcher with operands of the test's choice, for the stand-in
// runtime: addresses are made up, nothing is read.
#include "epd_internal.h"

#include <cstring>

extern "C" {

// may_read: 1 = rows past the end of A, 2 = rows past the end of W
void shim_gemm(int M, int N, int K, int epilogue, int gather_n, int may_read, int tile, int compute_units) {
  epd::GemmArgs g;
  std::memset((void*)&g, 0, sizeof g);
  g.A = (const void*)0x10000; g.W = (const void*)0x20000; g.out = (void*)0x30000; g.resid = (float*)0x40000;
  g.M = M; g.N = N; g.K = K; g.lda = gather_n ? K / gather_n : K; g.ldo = N; g.ldr = N; g.epilogue = epilogue;
  if (gather_n) { g.gather = (const int32_t*)0x50000; g.gather_n = gather_n; }
  g.overread_a = may_read & 1; g.overread_w = (may_read >> 1) & 1;
  g.tile_cfg = tile + 1; g.compute_units = compute_units;
  g.qk_cols = N / 3 * 2; g.head_dim = 64; g.rot = (const float2*)0x60000; g.rot_pairs = 32;
  epd::launch_gemm_bf16(g, nullptr);
}

size_t shim_args_size() { return sizeof(epd::GemmArgs); }
int shim_rot_lds(const void* args) { return ((const epd::GemmArgs*)args)->rot_lds; }

}  // extern "C"
