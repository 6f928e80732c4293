// MFMA cores for tiles of at most 128 rows: an expert with few tokens, or the last rows of one.
// Such a tile is bound by streaming its 256 weight rows, and the 256-row cores spend half of
// their LDS and of their loads on activation rows that do not exist. Here the activation
// stages hold 64 or 128 rows, the LDS that is saved holds more stages (the loads in flight per
// CU are what the weight stream's rate hangs on), and every wave multiplies all the rows by its
// own share of the columns. One barrier per K step; the loads of stage kt + S - 1 go into the
// slot of stage kt - 1, S stages in all. Loads past K, and of activation rows that do not exist,
// are issued out of the buffers' range: nothing is fetched (every line counts: a CU's load path
// is what bounds the quantized tiles), and the number in flight is the same in every step.
//
// The products are summed by the same MFMAs in the same K order as in the 256-row cores: the
// results' bits do not depend on which core ran.
#pragma once
#include "xs_gemm_mx.hpp"

namespace xs {

constexpr int kSmallRows = 128;
constexpr uint32_t kBufBytes = 0x80000000u;   // descriptors span 2 GiB; offsets from here on fetch nothing
static_assert(kLdsBytes >= 4 * (64 + kBN) * kBK * 2, "four stages of 64 activation rows");

// Per-lane offset o (kBufBytes for a row that does not exist) plus the K offset k, or, past the
// last stage, out of range. (The or keeps a missing row's offset from wrapping.)
__device__ __forceinline__ uint32_t at_stage(uint32_t o, uint32_t k, bool in) {
  return (o + (in ? k : 0u)) | (in ? 0u : kBufBytes);
}

// ------------------------------------------------------------------------------ bf16
// acc[i]: rows 32 i + lane % 32; columns of wave w 32 w + 8 (q / 4) + 4 (lane / 32) + q % 4.
typedef f32x16 AccSmall[4];

// B tile row -> weight row: a wave's 32 rows are 16 gate and the 16 matching up rows.
__device__ __forceinline__ int b_row_small(int r, int n0, int half, bool swiglu) {
  return swiglu ? n0 + ((r >> 4) & 1) * half + (r >> 5) * 16 + (r & 15) : n0 + r;
}

struct SmallTile {
  v4i ra, rb;
  uint32_t oa[2], ob[4];
};

template <int NI>
__device__ __forceinline__ void mainloop_small(const SmallTile& t, int nk, AccSmall& acc, char* lds_raw) {
  constexpr int kAL = (NI + 1) / 2;                       // A loads per wave and stage: 64 rows each
  constexpr int kABytes = kAL * 64 * kBK * 2, kStageBytes = kABytes + kOpBytes;
  constexpr int S = kLdsBytes / kStageBytes;              // 4 (up to 64 rows) or 3 stages
  constexpr int kL = kAL + 4;
  lds_char* const lds = (lds_char*)lds_raw;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int swz = (lane >> 1) & 7, khalf = lane >> 5;
  const int arow = (lane & 31) * kBK * 2, brow = kABytes + (32 * w + (lane & 31)) * kBK * 2;
  auto issue = [&](int kt, int slot) {
    lds_char* st = lds + slot * kStageBytes;
    const uint32_t k = static_cast<uint32_t>(kt) * (kBK * 2);
#pragma unroll
    for (int i = 0; i < 4; ++i) load_lds16(t.rb, at_stage(t.ob[i], k, kt < nk), st + kABytes + (8 * i + w) * 1024);
#pragma unroll
    for (int i = 0; i < kAL; ++i) load_lds16(t.ra, at_stage(t.oa[i], k, kt < nk), st + (8 * i + w) * 1024);
  };
#pragma unroll
  for (int s = 0; s + 1 < S; ++s) issue(s, s);
  int slot = 0, fill = S - 1;
  for (int kt = 0; kt < nk; ++kt) {
    wait_vm<(S - 2) * kL>();
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    const lds_char* st = lds + slot * kStageBytes;
    bf16x8 bf[4], af[4][NI];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      const int piece = ((2 * kk + khalf) ^ swz) << 4;
      bf[kk] = *(const lds_bf16x8*)(st + brow + piece);
#pragma unroll
      for (int i = 0; i < NI; ++i) af[kk][i] = *(const lds_bf16x8*)(st + arow + i * 32 * kBK * 2 + piece);
    }
    asm volatile("" ::: "memory");
    issue(kt + S - 1, fill);
    fill = slot;
    slot = slot + 1 == S ? 0 : slot + 1;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
#pragma unroll
      for (int i = 0; i < NI; ++i) acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bf[kk], af[kk][i], acc[i], 0, 0, 0);
  }
  wait_vm<0>();
}

// As gemm_mainloop, for 1 <= a_rows <= kSmallRows; every operand byte of the tile within 2 GiB of A
// and B. Returns the number of 32-row blocks. Ends with a block barrier.
__device__ __forceinline__ int gemm_mainloop_small(const uint16_t* A, int64_t lda, int a_rows, const uint16_t* B,
                                                   int64_t ldb, int b_n0, int b_half, bool swiglu, int K,
                                                   AccSmall& acc, char* lds) {
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  SmallTile t;
  t.ra = buffer_rsrc(A, kBufBytes);
  t.rb = buffer_rsrc(B, kBufBytes);
  const int lr = lane >> 3, lp = lane & 7;
  const int c16 = (lp ^ ((4 * w + (lr >> 1)) & 7)) * 16;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = 64 * i + 8 * w + lr;
    if (i < 2) t.oa[i] = r < a_rows ? static_cast<uint32_t>(r * lda * 2 + c16) : kBufBytes;
    t.ob[i] = static_cast<uint32_t>(b_row_small(r, b_n0, b_half, swiglu) * ldb * 2 + c16);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int q = 0; q < 16; ++q) acc[i][q] = 0.f;
  const int nk = uniform_here(K / kBK), ni = __builtin_amdgcn_readfirstlane((a_rows + 31) >> 5);
  switch (ni) {
    case 1: mainloop_small<1>(t, nk, acc, lds); break;
    case 2: mainloop_small<2>(t, nk, acc, lds); break;
    case 3: mainloop_small<3>(t, nk, acc, lds); break;
    default: mainloop_small<4>(t, nk, acc, lds); break;
  }
  __syncthreads();
  return ni;
}

// Accumulators -> bf16 rows in LDS, pitch kEpiPitch, and with SwiGLU 128 columns at kEpiPitchH.
__device__ __forceinline__ void stage_tile_small(const AccSmall& acc, int ni, char* lds) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (i >= ni) break;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      uint2 v;
      v.x = pack_bf16x2(acc[i][4 * g], acc[i][4 * g + 1]);
      v.y = pack_bf16x2(acc[i][4 * g + 2], acc[i][4 * g + 3]);
      const int row = 32 * i + (lane & 31), col = 32 * w + 8 * g + 4 * (lane >> 5);
      *reinterpret_cast<uint2*>(lds + (row * kEpiPitch + col) * 2) = v;
    }
  }
}

__device__ __forceinline__ void stage_swiglu_small(const AccSmall& acc, int ni, char* lds) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (i >= ni) break;
#pragma unroll
    for (int g = 0; g < 2; ++g) {   // columns 8 g + .. of the wave's 16 gate columns, and the up ones
      float h[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float gt = acc[i][4 * g + q], up = acc[i][8 + 4 * g + q];
        h[q] = gt * __builtin_amdgcn_rcpf(1.f + __expf(-gt)) * up;
      }
      uint2 v;
      v.x = pack_bf16x2(h[0], h[1]);
      v.y = pack_bf16x2(h[2], h[3]);
      const int row = 32 * i + (lane & 31), col = 16 * w + 8 * g + 4 * (lane >> 5);
      *reinterpret_cast<uint2*>(lds + (row * kEpiPitchH + col) * 2) = v;
    }
  }
}

// ------------------------------------------------------------------------------ MX
// acc[i][j]: rows 32 i + lane % 32; columns of wave w 64 w + 32 j + 8 (q / 4) + 4 (lane / 32) + q % 4.
typedef f32x16 AccMxSmall[4][2];

struct MxSmallTile {
  v4i ra, rb, rsa, rsb;
  uint32_t oa[4], ob[8];
  uint32_t osa, osb;          // this lane's scale row (16 bytes of group 0)
  uint32_t sa_grp, sb_grp;    // bytes from one scale group to the next
};

// Loads of the stages newer than stage kt (position p in its scale group of G stages) that are in
// flight at its boundary: stages kt + 1 .. kt + S - 2, two more in each that opens a scale group.
constexpr int mx_small_newer(int p, int S, int L, int G) {
  int n = 0;
  for (int j = p + 1; j <= p + S - 2; ++j) n += L + (j % G == 0 ? 2 : 0);
  return n;
}

// A stage is one whole 128-byte line of every weight row: 128 K elements of E4M3 codes, 256 of
// E2M1 (with 64-byte stages every E2M1 line was loaded in two halves).
template <int NI, bool BF4>
__device__ __forceinline__ void mainloop_mx_small(const MxSmallTile& t, int nk, AccMxSmall& acc, char* lds_raw) {
  constexpr int kW = BF4 ? 2 : 1;                         // 128-element pieces (scale words) per stage
  constexpr int kG = 4 / kW;                              // stages per scale group
  constexpr int kAPart = NI * 32 * 128;                   // A bytes of one 128-element piece
  constexpr int kABytes = kW * kAPart, kStageBytes = kABytes + kBN * 128;
  constexpr int kFit = kMxScaleOff / kStageBytes;
  // the group of stage kt + S - 1 goes into the buffer of the group two before it, whose last words
  // every wave has read before the barrier of stage kt only if S <= kG + 1
  constexpr int S = kFit < kG + 1 ? kFit : kG + 1;        // stages: E4M3 weights 4 or 3, E2M1 3 or 2
  constexpr int kL = NI * kW + 8;                         // loads per wave: A 32 rows, B 32 rows x 128 bytes each
  constexpr int kFmtB = BF4 ? 4 : 0;
  static_assert(S >= 2, "stages");
  typedef __attribute__((address_space(3))) v4i_t lds_v4i;
  typedef __attribute__((address_space(3))) uint32_t lds_u32;
  lds_char* const lds = (lds_char*)lds_raw;
  const int lane = lane_id_here();   // not held across other tiles (the 256-row core needs every register)
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int swz = (lane >> 1) & 7, h = lane >> 5;
  const uint32_t sel = h ? 0x0C0C0301u : 0x0C0C0200u;     // bytes h and 2 + h of a scale word
  const int arow = (lane & 31) * 128, brow = kABytes + (64 * w + (lane & 31)) * 128;
  const int asc = kMxScaleOff + (lane & 31) * 16, bsc = kMxScaleOff + kBM * 16 + (64 * w + (lane & 31)) * 16;
  // stage kt into `slot`; a stage that opens a scale group also brings the group's 16 bytes per
  // row (A rows 64 (w % 2) + lane: two waves load the same ones; B rows 64 w + lane)
  auto issue = [&](int kt, int slot, auto opens) {
    lds_char* st = lds + slot * kStageBytes;
    const bool in = kt < nk;
    const uint32_t k = static_cast<uint32_t>(kt) * 128u;
#pragma unroll
    for (int i = 0; i < 8; ++i) load_lds16(t.rb, at_stage(t.ob[i], k, in), st + kABytes + (4 * i + w) * 1024);
#pragma unroll
    for (int c = 0; c < kW; ++c)
#pragma unroll
      for (int i = 0; i < NI; ++i)
        load_lds16(t.ra, at_stage(t.oa[i], k * kW + c * 128u, in), st + c * kAPart + (4 * i + w) * 1024);
    if constexpr (decltype(opens)::value) {
      const uint32_t g = static_cast<uint32_t>(kt) / kG;
      lds_char* sc = lds + kMxScaleOff + (g & 1) * kMxScaleBuf;
      load_lds16(t.rsa, at_stage(t.osa, g * t.sa_grp, in), sc + (w & 1) * 1024);
      load_lds16(t.rsb, at_stage(t.osb, g * t.sb_grp, in), sc + kBM * 16 + w * 1024);
    }
  };
  int slot = 0, fill = S - 1;
  auto stage = [&](int kt, auto pos) {
    constexpr int p = decltype(pos)::value;
    wait_vm<mx_small_newer(p, S, kL, kG)>();
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    const lds_char* st = lds + slot * kStageBytes;
    const int sg = ((kt / kG) & 1) * kMxScaleBuf + 4 * kW * p;
    int sa[kW][NI], sb[kW][2];
    v8i_t a[2 * kW][NI], b[2 * kW][2];
#pragma unroll
    for (int c = 0; c < kW; ++c) {
#pragma unroll
      for (int i = 0; i < NI; ++i) sa[c][i] = static_cast<int>(*(const lds_u32*)(lds + sg + 4 * c + asc + i * 512));
#pragma unroll
      for (int j = 0; j < 2; ++j) sb[c][j] = static_cast<int>(*(const lds_u32*)(lds + sg + 4 * c + bsc + j * 512));
    }
    auto frag = [&](int row_off, int kk) {
      const v4i_t lo = *(const lds_v4i*)(st + row_off + (((4 * kk + h) ^ swz) << 4));
      const v4i_t hi = *(const lds_v4i*)(st + row_off + (((4 * kk + 2 + h) ^ swz) << 4));
      return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    };
#pragma unroll
    for (int kk = 0; kk < 2 * kW; ++kk) {
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        if constexpr (BF4) {   // 32 codes per lane: piece 2 kk + h of the line
          const v4i_t v = *(const lds_v4i*)(st + brow + j * 32 * 128 + (((2 * kk + h) ^ swz) << 4));
          b[kk][j] = __builtin_shufflevector(v, v, 0, 1, 2, 3, -1, -1, -1, -1);
        } else {
          b[kk][j] = frag(brow + j * 32 * 128, kk);
        }
      }
#pragma unroll
      for (int i = 0; i < NI; ++i) a[kk][i] = frag((kk >> 1) * kAPart + arow + i * 32 * 128, kk & 1);
    }
    asm volatile("" ::: "memory");
    issue(kt + S - 1, fill, std::integral_constant<bool, (p + S - 1) % kG == 0>{});
    fill = slot;
    slot = slot + 1 == S ? 0 : slot + 1;
#pragma unroll
    for (int c = 0; c < kW; ++c) {
#pragma unroll
      for (int i = 0; i < NI; ++i) sa[c][i] = static_cast<int>(__builtin_amdgcn_perm(sa[c][i], sa[c][i], sel));
#pragma unroll
      for (int j = 0; j < 2; ++j) sb[c][j] = static_cast<int>(__builtin_amdgcn_perm(sb[c][j], sb[c][j], sel));
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(b[2 * c][j], a[2 * c][i], acc[i][j], kFmtB, 0, 0,
                                                                      sb[c][j], 0, sa[c][i]);
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(b[2 * c + 1][j], a[2 * c + 1][i], acc[i][j], kFmtB, 0,
                                                                      1, sb[c][j], 1, sa[c][i]);
    }
  };
  const std::true_type yes;
  const std::false_type no;
#pragma unroll
  for (int s = 0; s + 1 < S; ++s) {
    if (s % kG == 0) issue(s, s, yes);
    else issue(s, s, no);
  }
  for (int kt = 0; kt < nk; kt += kG) {   // K is a multiple of 512: whole scale groups
    stage(kt, std::integral_constant<int, 0>{});
    stage(kt + 1, std::integral_constant<int, 1>{});
    if constexpr (kG == 4) {
      stage(kt + 2, std::integral_constant<int, 2>{});
      stage(kt + 3, std::integral_constant<int, 3>{});
    }
  }
  wait_vm<0>();
}

// As gemm_mainloop_mx, for 1 <= a_rows <= kSmallRows; every operand and scale byte of the tile
// within 2 GiB of its base. Returns the number of 32-row blocks. Ends with a block barrier.
template <bool BF4>
__device__ __forceinline__ int gemm_mainloop_mx_small(const uint8_t* A, int64_t lda, const uint8_t* As, int64_t a_srow,
                                                      int64_t a_sgrp, int a_rows, const uint8_t* B, int64_t ldb,
                                                      const uint8_t* Bs, int64_t b_srow, int64_t b_sgrp, int b_n0,
                                                      int b_half, bool swiglu, int K, AccMxSmall& acc, char* lds) {
  const int lane = lane_id_here();
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  MxSmallTile t;
  t.ra = buffer_rsrc(A, kBufBytes);
  t.rb = buffer_rsrc(B, kBufBytes);
  t.rsa = buffer_rsrc(As, kBufBytes);
  t.rsb = buffer_rsrc(Bs, kBufBytes);
  const int lr = lane >> 3, lp = lane & 7;
  const int c16 = (lp ^ ((4 * w + (lr >> 1)) & 7)) * 16;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int r = 32 * i + 8 * w + lr;
    if (i < 4) t.oa[i] = r < a_rows ? static_cast<uint32_t>(r * lda + c16) : kBufBytes;
    t.ob[i] = static_cast<uint32_t>(b_row_map(r, b_n0, b_half, swiglu) * ldb + c16);
  }
  const int sr = 64 * (w & 1) + lane;
  t.osa = sr < a_rows ? static_cast<uint32_t>(sr * a_srow) : kBufBytes;
  t.osb = static_cast<uint32_t>(b_row_map(64 * w + lane, b_n0, b_half, swiglu) * b_srow);
  t.sa_grp = static_cast<uint32_t>(a_sgrp);
  t.sb_grp = static_cast<uint32_t>(b_sgrp);
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int q = 0; q < 16; ++q) acc[i][j][q] = 0.f;
  const int nk = uniform_here(K / (BF4 ? 256 : 128)), ni = __builtin_amdgcn_readfirstlane((a_rows + 31) >> 5);
  switch (ni) {
    case 1: mainloop_mx_small<1, BF4>(t, nk, acc, lds); break;
    case 2: mainloop_mx_small<2, BF4>(t, nk, acc, lds); break;
    case 3: mainloop_mx_small<3, BF4>(t, nk, acc, lds); break;
    default: mainloop_mx_small<4, BF4>(t, nk, acc, lds); break;
  }
  __syncthreads();
  return ni;
}

// Accumulators -> bf16 rows in LDS, pitch kEpiPitch.
__device__ __forceinline__ void stage_tile_mx_small(const AccMxSmall& acc, int ni, char* lds) {
  const int lane = lane_id_here(), w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (i >= ni) break;
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        uint2 v;
        v.x = pack_bf16x2(acc[i][j][4 * g], acc[i][j][4 * g + 1]);
        v.y = pack_bf16x2(acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]);
        const int row = 32 * i + (lane & 31), col = 64 * w + 32 * j + 8 * g + 4 * (lane >> 5);
        *reinterpret_cast<uint2*>(lds + (row * kEpiPitch + col) * 2) = v;
      }
  }
}

// SwiGLU and quantization of block w of the tile's 128 output columns (stage_swiglu_mxq).
__device__ __forceinline__ void stage_swiglu_mxq_small(const AccMxSmall& acc, int ni, char* lds) {
  const int lane = lane_id_here(), w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (i >= ni) break;
    swiglu_mxq_block(acc[i][0], acc[i][1], 32 * i + (lane & 31), w, lane >> 5, lds);
  }
}

}  // namespace xs
