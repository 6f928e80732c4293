// Split-K bf16 GEMM for gfx950, C = A B^T for products with too few 256 x 256 output tiles to
// fill the chip (a decode step's projections: 24 x 4096 outputs are 16 such tiles, for 256
// CUs). A workgroup takes 16 NB rows and 16 NJ columns of C and splits K over its waves, so the
// grid has (M / 16 NB) (N / 16 NJ) workgroups; the waves' fp32 partial sums meet in LDS once
// and are added in wave order.
//
// What bounds it is the rate at which a CU's vector memory path delivers operand lines (about
// 75 B/ns with the loads below): every operand byte of a workgroup's K panels comes once per
// workgroup, (NB + NJ) 32 K bytes. Each wave stages its own K pieces (64 elements, one 128-byte
// line of every row) in a private slice of LDS by direct loads of 8 rows x 128 bytes per
// instruction, kDepth pieces deep, and needs no barrier until the end. Loading the MFMA fragments
// straight into registers instead (16 rows x 64 bytes per instruction, so every line is touched
// by two instructions) took 18.7 us where this takes 11.2 (24 x 4096 x 7168, 5.3 TB/s of weights),
// and 53 us against 23 (256 x 4096 x 7168).
#pragma once
#include "xs_common.hpp"

namespace xs {
namespace skinny {

struct Args {
  const char* a;
  int64_t lda_bytes;
  const char* b;
  int64_t ldb_bytes;
  char* c;
  int64_t ldc_bytes;
  int M, K;
};

// v_mfma_f32_16x16x32_bf16 with the weight fragment first: lane l holds row l % 16 of either
// operand at K elements 8 (l / 16) .. + 7, and accumulates columns 4 (l / 16) .. + 3 of output
// row l % 16. In a staged piece, logical 16-byte part c of row r sits at c ^ ((r >> 1) & 7).
template <int NB, int NJ, int kDepth, int kWaves>
__global__ __launch_bounds__(kWaves * 64) void gemm_kernel(Args p) {
  constexpr int kRows = 16 * NB, kCols = 16 * NJ, kThreads = kWaves * 64;
  constexpr int kPitch = kCols + 4;                  // floats per row of a partial sum
  constexpr int kPiece = (kRows + kCols) * 128;      // bytes of one staged piece, B rows first
  constexpr int kLoads = 2 * (NB + NJ);              // loads of one piece
  constexpr int kStageBytes = kWaves * kDepth * kPiece, kRedBytes = kWaves * kRows * kPitch * 4;
  __shared__ __attribute__((aligned(16))) char smem[kStageBytes > kRedBytes ? kStageBytes : kRedBytes];
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i = lane & 15, g = lane >> 4;
  lds_char* const lds = (lds_char*)smem + w * kDepth * kPiece;
  const int n0 = blockIdx.x * kCols, m0 = blockIdx.y * kRows;
  const int rows = min(kRows, p.M - m0);
  const v4i ra = buffer_rsrc(p.a + m0 * p.lda_bytes, static_cast<uint32_t>((rows - 1) * p.lda_bytes + 2 * p.K));
  const v4i rb = buffer_rsrc(p.b + n0 * p.ldb_bytes, static_cast<uint32_t>((kCols - 1) * p.ldb_bytes + 2 * p.K));
  // load n of an operand fills its rows 8 n .. + 7 of a piece
  uint32_t oa[2 * NB], ob[2 * NJ];
  const int lr = lane >> 3, lp = lane & 7;
#pragma unroll
  for (int n = 0; n < 2 * NB; ++n)
    oa[n] = static_cast<uint32_t>((8 * n + lr) * p.lda_bytes + ((lp ^ ((4 * n + (lr >> 1)) & 7)) << 4));
#pragma unroll
  for (int n = 0; n < 2 * NJ; ++n)
    ob[n] = static_cast<uint32_t>((8 * n + lr) * p.ldb_bytes + ((lp ^ ((4 * n + (lr >> 1)) & 7)) << 4));
  const int pieces = p.K / 64;
  const int p0 = pieces * w / kWaves, p1 = pieces * (w + 1) / kWaves;   // this wave's pieces
  f32x4 acc[NB][NJ];
#pragma unroll
  for (int x = 0; x < NB; ++x)
#pragma unroll
    for (int y = 0; y < NJ; ++y) acc[x][y] = f32x4{0.f, 0.f, 0.f, 0.f};
  // piece pc into slot s; past the wave's range every lane points past the buffers (their ends
  // lie below 2^31), so the number of loads in flight stays the same
  auto load = [&](int s, int pc) {
    const uint32_t k = pc < p1 ? static_cast<uint32_t>(pc) * 128u : 0x80000000u;
#pragma unroll
    for (int n = 0; n < 2 * NJ; ++n) load_lds16(rb, ob[n] + k, lds + s * kPiece + n * 1024);
#pragma unroll
    for (int n = 0; n < 2 * NB; ++n) load_lds16(ra, oa[n] + k, lds + s * kPiece + kCols * 128 + n * 1024);
  };
  const int swz = (i >> 1) & 7;
#pragma unroll
  for (int s = 0; s < kDepth; ++s) load(s, p0 + s);
  for (int pc = p0; pc < p1; pc += kDepth) {
#pragma unroll
    for (int s = 0; s < kDepth; ++s) {
      if (pc + s >= p1) break;
      wait_vm<(kDepth - 1) * kLoads>();              // piece pc + s has landed
      bf16x8 bf[2][NJ], af[2][NB];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int o = ((4 * h + g) ^ swz) << 4;
#pragma unroll
        for (int y = 0; y < NJ; ++y) bf[h][y] = *(const lds_bf16x8*)(lds + s * kPiece + (16 * y + i) * 128 + o);
#pragma unroll
        for (int x = 0; x < NB; ++x)
          af[h][x] = *(const lds_bf16x8*)(lds + s * kPiece + (kCols + 16 * x + i) * 128 + o);
      }
      __builtin_amdgcn_s_waitcnt(0xC07F);            // lgkmcnt(0): the slot has been read
      asm volatile("" ::: "memory");
      load(s, pc + s + kDepth);
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int x = 0; x < NB; ++x)
#pragma unroll
          for (int y = 0; y < NJ; ++y)
            acc[x][y] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bf[h][y], af[h][x], acc[x][y], 0, 0, 0);
    }
  }
  wait_vm<0>();
  __syncthreads();                                   // no load is in flight: the LDS is free
  float* const red = reinterpret_cast<float*>(smem);
#pragma unroll
  for (int x = 0; x < NB; ++x)
#pragma unroll
    for (int y = 0; y < NJ; ++y)
      *reinterpret_cast<f32x4*>(red + (w * kRows + 16 * x + i) * kPitch + 16 * y + 4 * g) = acc[x][y];
  __syncthreads();
  for (int u = tid; u < rows * (kCols / 4); u += kThreads) {
    const int r = u / (kCols / 4), c = 4 * (u % (kCols / 4));
    f32x4 s = *reinterpret_cast<const f32x4*>(red + r * kPitch + c);
#pragma unroll
    for (int x = 1; x < kWaves; ++x) s += *reinterpret_cast<const f32x4*>(red + (x * kRows + r) * kPitch + c);
    uint2 v;
    v.x = pack_bf16x2(s[0], s[1]);
    v.y = pack_bf16x2(s[2], s[3]);
    *reinterpret_cast<uint2*>(p.c + (m0 + r) * p.ldc_bytes + static_cast<int64_t>(n0 + c) * 2) = v;
  }
}

}  // namespace skinny
}  // namespace xs
