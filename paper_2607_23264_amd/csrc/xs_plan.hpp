// The expert FFN's scheduler plan, computed from the local experts' row counts: scheduler rows
// of up to 256 (or 128) rows per expert, the Expert-Wave boundaries (App. A.2), the h row offsets, and
// the cleared readiness and claim counters. Shared by the plan kernel and by the layout's
// scan kernel, which plans right after it has the expert totals.
#pragma once
#include "xs_common.hpp"

namespace xs {

struct PlanArgs {
  int e_begin, n_experts, cap, P1, P2, wave_tiles;
  int* meta;           // [0] rows P, [1] waves, [2] wave-list length, [3] computed rows,
                       // [8], [9] claim counters, [10] workgroups done (FFN), [11] blocks done
                       // (dispatch)
  int* row_expert;
  int* exp_m;
  int* exp_rowfirst;
  int* exp_hrow;
  int* exp_block;      // rows of the expert's blocks; not in meta, whose line the claims keep busy
  int* wave_pos;
  int* wave_row;
  int* l1_done;
  // Blocks of 128 rows where those are at most this many Linear-1 tiles (0: never), and the scheduler
  // rows that the tables hold
  int half_tiles, max_rows;
};

// Inclusive prefix sum over the wave's lanes, by DPP (no LDS round trips): shifts within rows of 16,
// then each row's last lane onto the rows after it.
__device__ __forceinline__ int wave_inclusive_scan(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, false);   // row_shr 1, 2, 4, 8
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xF, 0xF, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xA, 0xF, false);   // row_bcast 15 into rows 1 and 3
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xC, 0xF, false);   // row_bcast 31 into rows 2 and 3
  return x;
}

// Exclusive prefix sum of v over the block's threads in order (at most 16 waves, whole ones):
// a scan inside each wave, then of the waves' totals. ws is 16 ints of LDS; `total` receives the
// block's sum. Begins and ends with a block barrier.
__device__ __forceinline__ int block_exclusive_scan(int v, int* ws, int& total) {
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int waves = blockDim.x >> 6;
  const int x = wave_inclusive_scan(v);
  lds_sync();
  if (lane == 63) ws[wv] = x;
  lds_sync();
  const int sums = wave_inclusive_scan(lane < waves ? ws[lane & 15] : 0);   // lanes past the waves add nothing
  total = __builtin_amdgcn_readlane(sums, 63);
  const int before = wv ? __builtin_amdgcn_readlane(sums, wv - 1) : 0;
  lds_sync();
  return before + x - v;
}

// s_m[x] (LDS): local expert x's rows, clipped to its window; s_first (LDS, n_experts) and ws
// (LDS, 16 ints) are this function's scratch. Called by every thread of one block of at least
// n_experts threads, in whole waves; begins with a block barrier. One thread per expert: one
// thread for all of them took most of the scan launch (32 experts: 5 us).
__device__ __forceinline__ void plan_rows(const PlanArgs& pa, const int* s_m, int* s_first, int* ws) {
  const int i = threadIdx.x, n = pa.n_experts;
  lds_sync();
  const int m = i < n ? s_m[i] : 0;
  int bm = 256, mt = (m + 255) / 256, rows, hrows;
  int first = block_exclusive_scan(mt, ws, rows);
  const int hrow = block_exclusive_scan(m, ws, hrows);
  if (rows > 0 && rows * pa.P1 <= pa.half_tiles) {
    int rows_half;
    const int mt_half = (m + 127) / 128, first_half = block_exclusive_scan(mt_half, ws, rows_half);
    if (rows_half * pa.P1 <= pa.half_tiles && rows_half <= pa.max_rows) {
      bm = 128;
      mt = mt_half;
      first = first_half;
      rows = rows_half;
    }
  }
  if (i < n) {
    pa.exp_m[i] = m;
    pa.exp_rowfirst[i] = first;
    pa.exp_hrow[i] = hrow;
    pa.exp_block[i] = bm;
    s_first[i] = first + mt;   // the row after the expert's last
    for (int p = first; p < first + mt; ++p) pa.row_expert[p] = i;
  }
  for (int p = i; p < rows; p += blockDim.x) pa.l1_done[p] = 0;
  lds_sync();
  if (i == 0) {
    // expert waves: whole experts until a wave has wave_tiles Linear-1 tiles
    int nw = 0, last = 0, prev = 0, wl1 = 0;
    pa.wave_row[0] = 0;
    pa.wave_pos[0] = 0;
    for (int x = 0; x < n; ++x) {
      const int end = s_first[x];
      wl1 += (end - prev) * pa.P1;
      prev = end;
      if (wl1 >= pa.wave_tiles && end > last) {
        ++nw;
        pa.wave_row[nw] = end;
        pa.wave_pos[nw] = end * (pa.P1 + pa.P2);
        last = end;
        wl1 = 0;
      }
    }
    if (rows > last) {
      ++nw;
      pa.wave_row[nw] = rows;
      pa.wave_pos[nw] = rows * (pa.P1 + pa.P2);
    }
    pa.meta[0] = rows;
    pa.meta[1] = nw;
    pa.meta[2] = rows * (pa.P1 + pa.P2);
    pa.meta[3] = hrows;
    pa.meta[8] = 0;    // claim counters (dynamic claiming)
    pa.meta[9] = 0;
    pa.meta[10] = 0;   // workgroups done (the FFN's window signal)
    pa.meta[11] = 0;   // blocks done (the dispatch's window signal)
  }
}

// The rest of the layout, done by the dispatch launch of the fused layer (see dispatch_kernel).
struct FinArgs {
  int src, n_src, cap, n_chunks, n_disp_blocks;
  const int* idx_all;          // [n_src][T][k]; null: plain dispatch
  int rows_final;              // slot_row holds final rows; only row_src is left, of every source
  int* slot_row_all;
  const int* chunk_base;
  const int* src_base;
  const int* expert_offsets;
  int* row_src;
  int* done;
};

}  // namespace xs
