// Dispatch through bounded destination rings (Sec. 4.3: an eligible Linear-1 tile needs a free
// destination ring slot; App. A.2: the scheduler checks ring-slot readiness before emission).
//
// Each destination d owns a ring of S slots. An entry is one token row plus a header listing
// the rows of d's dispatch window it goes to: every (token, k) slot of that destination when
// deduplicating, one slot otherwise. Entries of a ring are numbered in token order (then k slot
// order) by a prefix scan before the dispatch; entry n lives in slot n mod S.
//
// Lifetime protocol (per slot two words, counting completed uses):
//   pub[s] = u + 1  entry n = u S + s is written (its producer's stores have completed);
//   rel[s] = u + 1  it has been copied out (by its consumer).
// The producer of entry n waits for rel[n mod S] == n / S (entry n - S released), writes the
// row and header, then publishes. Its consumer sees pub == n / S + 1, copies the row into every
// listed window row, then releases the slot.
//
// Agents are waves, with no workgroup barrier in the protocol: even waves produce their tokens'
// entries in token order, odd waves consume. A consumer owns every Q-th entry of a ring (or, with
// fewer consumers than rings, whole rings), so claiming takes no atomic; it looks at several of
// its entries at once, one per lane, and consumes whichever are published.
//
// Coherence: on this GPU a release that another XCD must observe writes back the L2, and an
// acquire invalidates it (agent and system scope cost the same, measured). With such fences, even
// one per 32 entries, the dispatch of 2048 rows of 14 KiB through 256-slot rings took 857 us,
// without any 150. So no ring byte is left in an L2: rows, headers and flags are stored with the
// system-scope bits (sc0 sc1: written through to memory), a producer publishes once its stores
// have completed (vmcnt 0), and consumers load with the same bits, past the L2. Only the window
// rows, which are read after the kernel, are cached. What bounds wide rings now is memory: every
// row is written and read once more than by the plain dispatch (575 MB in those 150 us).
//
// Progress: every wave is resident. The earliest entry not yet published (in token order) has
// a producer that waits at most for an earlier entry of its ring, which is published, and whose
// consumer waits for no particular entry; a producer publishes what it has written before it
// waits. Every wait is bounded: on time-out an agent reports XS_ETIMEOUT and raises an abort word
// that makes every other wait give up, so the grid always drains.
#include <algorithm>

#include "xs_common.hpp"

namespace xs {
namespace ring {

constexpr int kThreads = 256;         // four waves; every wave is an independent agent
constexpr int kMaxK = 32;
constexpr int kLine = 32;             // ints per 128-byte line: one counter per line
constexpr int kChunk = 64;            // tokens numbered by one wave of the rank kernel
constexpr int kPieces = 8;            // 16-byte pieces of a row per lane in flight (with 16, 4 % faster,
                                      // the kernel needs 174 registers: see the launch bounds)
constexpr int kLook = 8;              // entries a consumer looks at at once
constexpr int kCoherent = 17;         // buffer cache policy: sc0 | sc1, system scope

struct RingArgs {
  const char* x;               // token rows, x_stride bytes apart
  int64_t x_stride;
  int row_bytes;               // payload bytes per entry (a multiple of 16)
  int T, k, E, S, dedup;
  const int* idx;              // [T][k] routed experts
  const int* slot_row;         // [T][k] window row of each (token, k) slot
  WinSet win;                  // dispatch windows
  char* ring[XS_MAX_WINDOWS];  // ring memory per destination: S slots of slot_bytes
  int64_t slot_bytes;          // from one slot to the next (no upper bound)
  uint32_t entry_bytes;        // payload, then 1 + k header ints
  int* entry_no;               // [T][k] entry number of each (token, k) slot in its ring, less its
                               //        chunk's base
  int* chunk_base;             // [T / kChunk][W] entries of the ring from earlier chunks
  int* total;                  // [W] entries per destination, one per line
  int* abort_word;
  int* pub;                    // [W][S]
  int* rel;                    // [W][S]
  int* stats;                  // optional [2W]: entries, producer stalls
  int* status;
  int64_t timeout_ticks;
};

// Entry numbers within each chunk of 64 tokens, the chunks' entries per ring, and a clean control
// block. One wave per chunk, one token per lane: entries of a ring are numbered in token order
// (and k slot order within a token without dedup), a prefix sum over the lanes by ballots of the
// counts' bits.
__global__ __launch_bounds__(kThreads) void ring_rank_kernel(RingArgs a) {
  const int W = a.win.n;
  const int epw = a.E / W;
  const int64_t gid = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x;
  const int64_t words = static_cast<int64_t>(W) * a.S;
  for (int64_t i = gid; i < words; i += static_cast<int64_t>(gridDim.x) * kThreads) {
    a.pub[i] = 0;
    a.rel[i] = 0;
  }
  if (gid == 0) *a.abort_word = 0;
  const int lane = threadIdx.x & 63;
  const int c = blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
  if (c * kChunk >= a.T) return;
  const int t = c * kChunk + lane;
  const int* idx = a.idx + static_cast<int64_t>(t) * a.k;
  int* no = a.entry_no + static_cast<int64_t>(t) * a.k;
  // the token's destinations, held in registers (reading the indices again for every destination
  // took 22 us at 2048 tokens, k = 8, W = 8)
  int dst[kMaxK];
#pragma unroll
  for (int j = 0; j < kMaxK; ++j) dst[j] = j < a.k && t < a.T ? idx[j] : -1;
#pragma unroll
  for (int j = 0; j < kMaxK; ++j)
    if (j < a.k) dst[j] = dst[j] >= 0 && dst[j] < a.E ? dst[j] / epw : -1;
  const uint64_t below = (1ull << lane) - 1;
  const int bits = a.dedup ? 1 : 32 - __builtin_clz(a.k);
  for (int d = 0; d < W; ++d) {
    int n = 0;
#pragma unroll
    for (int j = 0; j < kMaxK; ++j)
      if (j < a.k) n += dst[j] == d;
    if (a.dedup) n = n > 0;
    int before = 0, all = 0;
    for (int b = 0; b < bits; ++b) {
      const uint64_t m = __ballot((n >> b) & 1);
      before += __builtin_popcountll(m & below) << b;
      all += __builtin_popcountll(m) << b;
    }
#pragma unroll
    for (int j = 0; j < kMaxK; ++j)
      if (j < a.k && dst[j] == d) {
        no[j] = before;
        before += !a.dedup;
      }
    if (lane == 0) a.chunk_base[static_cast<int64_t>(c) * W + d] = all;
  }
}

// The chunks' counts -> bases, and the totals: one wave per ring.
__global__ __launch_bounds__(1024) void ring_scan_kernel(RingArgs a) {
  const int W = a.win.n, lane = threadIdx.x & 63;
  const int chunks = (a.T + kChunk - 1) / kChunk;
  for (int d = threadIdx.x >> 6; d < W; d += 16) {
    int base = 0;
    for (int c0 = 0; c0 < chunks; c0 += 64) {
      int* p = a.chunk_base + static_cast<int64_t>(c0 + lane) * W + d;
      const int v = c0 + lane < chunks ? *p : 0;
      int x = v;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(x, o);
        if (lane >= o) x += y;
      }
      if (c0 + lane < chunks) *p = base + x - v;
      base += __shfl(x, 63);
    }
    if (lane == 0) {
      a.total[d * kLine] = base;
      if (a.stats) {
        a.stats[d] = base;
        a.stats[W + d] = 0;
      }
    }
  }
}

__device__ __forceinline__ bool aborted(const RingArgs& a) {
  return __hip_atomic_load(a.abort_word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
}

__device__ __forceinline__ void give_up(const RingArgs& a) {
  set_status(a.status, XS_ETIMEOUT);
  __hip_atomic_store(a.abort_word, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ int bcast(int v) { return __builtin_amdgcn_readfirstlane(v); }

typedef __attribute__((address_space(1))) u32x4 gv4;

// A buffer over the entry in one ring slot (wave-uniform address). Its range is the entry's bytes and not
// the slots' distance, which may not fit a descriptor's 32 bits.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t slot_buffer(const RingArgs& a, int d, int s) {
  const uint64_t p = reinterpret_cast<uint64_t>(a.ring[d] + static_cast<int64_t>(s) * a.slot_bytes);
  const uint64_t u = static_cast<uint64_t>(static_cast<uint32_t>(bcast(static_cast<int>(p)))) |
                     static_cast<uint64_t>(static_cast<uint32_t>(bcast(static_cast<int>(p >> 32)))) << 32;
  return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(u), 0, static_cast<int>(a.entry_bytes), 0x00020000);
}

// Copies published entry m of ring d out and releases its slot (wave-uniform m, d).
__device__ __forceinline__ void consume(const RingArgs& a, int d, int m, int lane) {
  const int s = m % a.S;
  const auto slot = slot_buffer(a, d, s);
  const int pieces = a.row_bytes >> 4;
  const int word = lane <= a.k ? __builtin_amdgcn_raw_buffer_load_b32(slot, a.row_bytes + 4 * lane, 0, kCoherent) : 0;
  int n = 0, my_row = -1;
  for (int p0 = 0; p0 < pieces; p0 += 64 * kPieces) {
    u32x4 v[kPieces];
#pragma unroll
    for (int q = 0; q < kPieces; ++q) {
      const int p = p0 + q * 64 + lane;
      if (p < pieces) v[q] = __builtin_amdgcn_raw_buffer_load_b128(slot, p * 16, 0, kCoherent);
    }
    if (p0 == 0) {
      n = bcast(word);
      if (n < 0 || n > a.k) {               // never written by a producer: report, copy nothing
        if (lane == 0) set_status(a.status, XS_EBADINPUT);
        n = 0;
      }
      my_row = __shfl(word, min(lane + 1, 63));
    }
    for (int i = 0; i < n; ++i) {
      const int r = __shfl(my_row, i);
      if (r < 0 || r >= a.win.cap[d]) {
        if (lane == 0 && p0 == 0) set_status(a.status, XS_ECAPACITY);
        continue;
      }
      char* dst = a.win.base[d] + static_cast<int64_t>(r) * a.win.stride[d];
#pragma unroll
      for (int q = 0; q < kPieces; ++q) {
        const int p = p0 + q * 64 + lane;
        if (p < pieces) *(gv4*)(dst + p * 16) = v[q];
      }
    }
  }
  // the stores above waited for the slot's loads (a load no row needed may be overwritten)
  asm volatile("" ::: "memory");
  if (lane == 0)
    __hip_atomic_store(a.rel + static_cast<int64_t>(d) * a.S + s, m / a.S + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Lane i of a consumer follows the entries m, m + step, ... of ring d; every published one is
// consumed, in any order. Until all are consumed, or the call is aborted.
__device__ __forceinline__ void consume_all(const RingArgs& a, int d, int m, int step, int lane) {
  const int tot = d >= 0 ? a.total[d * kLine] : 0;
  uint64_t t0 = wall_ticks();
  for (int it = 1;; ++it) {
    const bool left = m < tot;
    if (!__ballot(left)) return;
    const bool ready = left && __hip_atomic_load(a.pub + static_cast<int64_t>(d) * a.S + m % a.S, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_SYSTEM) == m / a.S + 1;
    asm volatile("" ::: "memory");
    uint64_t todo = __ballot(ready);
    if (!todo) {
      int stop = 0;
      if (lane == 0) {
        if ((it & 15) == 0 && aborted(a)) stop = 1;
        else if (wall_ticks() - t0 > static_cast<uint64_t>(a.timeout_ticks)) { give_up(a); stop = 1; }
      }
      if (bcast(stop)) return;
      __builtin_amdgcn_s_sleep(2);
      continue;
    }
    for (; todo; todo &= todo - 1) {
      const int i = __builtin_ctzll(todo);
      consume(a, bcast(__shfl(d, i)), bcast(__shfl(m, i)), lane);
    }
    if (ready) m += step;
    t0 = wall_ticks();
  }
}

// Produces token t's entries: lane j holds slot j's destination (d, -1: none), window row and entry
// number. Every entry whose slot is free is written, then all of them are published; until none
// is left. False on abort.
__device__ __forceinline__ bool produce(const RingArgs& a, int t, int d, int en, int row, int lane) {
  // the first lane of each entry stands for it, with the entry's lanes in `mask`
  uint64_t mask = 0, todo = 0;
  for (uint64_t rest = __ballot(d >= 0); rest;) {
    const int lead = __builtin_ctzll(rest);
    const int dd = __shfl(d, lead);
    const uint64_t m = a.dedup ? __ballot(d == dd) : 1ull << lead;
    if ((m >> lane) & 1) mask = m;
    todo |= 1ull << lead;
    rest &= ~m;
  }
  const int s = d >= 0 ? en % a.S : 0, u = d >= 0 ? en / a.S : 0;
  const int64_t word = d >= 0 ? static_cast<int64_t>(d) * a.S + s : 0;
  const char* src = a.x + static_cast<int64_t>(t) * a.x_stride;
  const int pieces = a.row_bytes >> 4;
  uint64_t t0 = wall_ticks();
  for (int it = 0; todo; ++it) {
    const bool wait = (todo >> lane) & 1;
    // a slot's first use needs no look
    const bool ready = wait && (u == 0 || __hip_atomic_load(a.rel + word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM) == u);
    asm volatile("" ::: "memory");
    if (it == 0 && wait && !ready && a.stats) atomicAdd(a.stats + a.win.n + d, 1);
    const uint64_t now = __ballot(ready);
    if (!now) {
      int stop = 0;
      if (lane == 0) {
        if ((it & 15) == 15 && aborted(a)) stop = 1;
        else if (wall_ticks() - t0 > static_cast<uint64_t>(a.timeout_ticks)) { give_up(a); stop = 1; }
      }
      if (bcast(stop)) return false;
      __builtin_amdgcn_s_sleep(4);
      continue;
    }
    for (int p0 = 0; p0 < pieces; p0 += 64 * kPieces) {
      u32x4 v[kPieces];
#pragma unroll
      for (int q = 0; q < kPieces; ++q) {
        const int p = p0 + q * 64 + lane;
        if (p < pieces) v[q] = *(const gv4*)(src + p * 16);
      }
      for (uint64_t w = now; w; w &= w - 1) {
        const int i = __builtin_ctzll(w);
        const auto slot = slot_buffer(a, bcast(__shfl(d, i)), bcast(__shfl(s, i)));
#pragma unroll
        for (int q = 0; q < kPieces; ++q) {
          const int p = p0 + q * 64 + lane;
          if (p < pieces) __builtin_amdgcn_raw_buffer_store_b128(v[q], slot, p * 16, 0, kCoherent);
        }
      }
    }
    // headers: the number of rows, then the rows in ascending k slot order
    for (uint64_t w = now; w; w &= w - 1) {
      const int i = __builtin_ctzll(w);
      const auto slot = slot_buffer(a, bcast(__shfl(d, i)), bcast(__shfl(s, i)));
      const uint64_t m = static_cast<uint64_t>(static_cast<uint32_t>(__shfl(static_cast<int>(mask), i))) |
                         static_cast<uint64_t>(static_cast<uint32_t>(__shfl(static_cast<int>(mask >> 32), i))) << 32;
      if ((m >> lane) & 1)
        __builtin_amdgcn_raw_buffer_store_b32(row, slot, a.row_bytes + 4 * (1 + __builtin_popcountll(m & ((1ull << lane) - 1))),
                                              0, kCoherent);
      if (lane == 0) __builtin_amdgcn_raw_buffer_store_b32(__builtin_popcountll(m), slot, a.row_bytes, 0, kCoherent);
    }
    // published once every store of this wave has reached memory
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (ready) __hip_atomic_store(a.pub + word, u + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    todo &= ~now;
    t0 = wall_ticks();
  }
  return true;
}

// four waves per SIMD, two of them this call's: a second call on another stream is resident too
__global__ __launch_bounds__(kThreads, 4) void ring_dispatch_kernel(RingArgs a) {
  const int lane = threadIdx.x & 63;
  const int agents = gridDim.x * (kThreads / 64);
  const int me = bcast(blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6));
  const int W = a.win.n;
  const int epw = a.E / W;
  const int half = agents / 2, id = me / 2;
  if (me & 1) {
    if (half >= W) {
      // ring id % W; of its consumers as many as it has slots (no more entries are ever ready)
      const int d = id % W, q = id / W;
      const int Q = min((half - d + W - 1) / W, a.S);
      if (q < Q) consume_all(a, lane < kLook ? d : -1, q + lane * Q, kLook * Q, lane);
    } else {
      const int d = id + lane * half;
      consume_all(a, lane < XS_MAX_WINDOWS && d < W ? d : -1, 0, 1, lane);
    }
    return;
  }
  for (int t = id; t < a.T; t += half) {
    // lane j < k holds slot j's destination, window row and entry number
    int d = -1, r = -1, en = 0;
    if (lane < a.k) {
      const int64_t q = static_cast<int64_t>(t) * a.k + lane;
      const int e = a.idx[q];
      if (e < 0 || e >= a.E) {
        set_status(a.status, XS_EBADINPUT);
      } else {
        d = e / epw;
        r = a.slot_row[q];
        en = a.entry_no[q] + a.chunk_base[static_cast<int64_t>(t / kChunk) * W + d];
      }
    }
    if (!produce(a, t, d, en, r, lane)) return;
  }
}

}  // namespace ring
}  // namespace xs

// ------------------------------------------------------------------------------ host side
namespace xs_host {
int signal_windows(const xs::WinSet& ws, hipStream_t st);
int persistent_grid(int max_producers);
}  // namespace xs_host

namespace {

int64_t align16(int64_t v) { return (v + 15) / 16 * 16; }

// Control block in the workspace: total [W], one counter per 128-byte line, the abort word on a
// line of its own, then pub and rel [W][S] each.
constexpr int64_t kCtrlTotal = 0, kCtrlAbort = XS_MAX_WINDOWS * 32, kCtrlPub = kCtrlAbort + 32;
int64_t chunks_of(int32_t T) { return (static_cast<int64_t>(T) + xs::ring::kChunk - 1) / xs::ring::kChunk; }
// control words, then the entry numbers [T][k] and the chunk bases [chunks][W]
int64_t ctrl_ints(int32_t T, int32_t k, int32_t W, int32_t S) {
  return kCtrlPub + 2 * static_cast<int64_t>(W) * S + static_cast<int64_t>(T) * k + chunks_of(T) * W;
}

}  // namespace

extern "C" int xs_ring_slot_bytes(int32_t H, int32_t k, int64_t* bytes) {
  if (!bytes || H < 8 || H % 8 || k < 1 || k > xs::ring::kMaxK) return XS_EINVAL;
  *bytes = align16(static_cast<int64_t>(H) * 2 + 4 * (1 + static_cast<int64_t>(k)));
  return XS_OK;
}

extern "C" int xs_dispatch_ring_workspace_bytes(int32_t T, int32_t k, int32_t W, int32_t slots, int64_t* bytes) {
  if (!bytes || T < 0 || k < 1 || W < 1 || W > XS_MAX_WINDOWS || slots < 1) return XS_EINVAL;
  *bytes = ctrl_ints(T, k, W, slots) * 4;
  return XS_OK;
}

extern "C" int xs_dispatch_ring(const void* x, int32_t T, int32_t H, const int32_t* topk_idx,
                                const int32_t* slot_row, int32_t k, int32_t E, const xs_window* win,
                                int32_t W, const xs_window* rings, int32_t dedup, int32_t max_producers,
                                int64_t spin_timeout_us, void* workspace, int64_t workspace_bytes,
                                int32_t* stats, int32_t* dev_status, void* stream) {
  using namespace xs;
  if (!x || !topk_idx || !slot_row || !win || !rings || !dev_status || T < 0 || k < 1 ||
      k > ring::kMaxK || k > E || E < 1 || W < 1 || W > XS_MAX_WINDOWS || E % W || (dedup != 0 && dedup != 1) ||
      max_producers < 0 || spin_timeout_us < 0)
    return XS_EINVAL;
  if (H < 8 || H % 8 || (reinterpret_cast<uintptr_t>(x) & 15)) return XS_EUNSUPPORTED;
  int64_t slot_bytes = 0;
  xs_ring_slot_bytes(H, k, &slot_bytes);
  const int32_t S = static_cast<int32_t>(rings[0].capacity_rows);
  if (S < 1 || rings[0].capacity_rows > (1 << 20)) return XS_EINVAL;
  ring::RingArgs a{};
  for (int d = 0; d < W; ++d) {
    if (!rings[d].base || rings[d].capacity_rows != S || rings[d].row_stride_bytes < slot_bytes ||
        rings[d].row_stride_bytes % 16 || (reinterpret_cast<uintptr_t>(rings[d].base) & 15))
      return XS_EINVAL;
    a.ring[d] = static_cast<char*>(rings[d].base);
  }
  if (rings[0].row_stride_bytes != rings[W - 1].row_stride_bytes) return XS_EINVAL;
  for (int d = 0; d < W; ++d)
    if (rings[d].row_stride_bytes != rings[0].row_stride_bytes) return XS_EINVAL;
  int64_t need = 0;
  xs_dispatch_ring_workspace_bytes(T, k, W, S, &need);
  if (!workspace || workspace_bytes < need) return XS_EWORKSPACE;
  const int rc = xs_host::make_winset(win, W, static_cast<int64_t>(H) * 2, &a.win);
  if (rc) return rc;
  int* ctrl = static_cast<int*>(workspace);
  a.x = static_cast<const char*>(x);
  a.x_stride = static_cast<int64_t>(H) * 2;
  a.row_bytes = H * 2;
  a.T = T;
  a.k = k;
  a.E = E;
  a.S = S;
  a.dedup = dedup;
  a.idx = topk_idx;
  a.slot_row = slot_row;
  a.slot_bytes = rings[0].row_stride_bytes;
  a.entry_bytes = static_cast<uint32_t>(static_cast<int64_t>(H) * 2 + 4 * (1 + k));
  a.total = ctrl + kCtrlTotal;
  a.abort_word = ctrl + kCtrlAbort;
  a.pub = ctrl + kCtrlPub;
  a.rel = a.pub + static_cast<int64_t>(W) * S;
  a.entry_no = a.rel + static_cast<int64_t>(W) * S;
  a.chunk_base = a.entry_no + static_cast<int64_t>(T) * k;
  a.stats = stats;
  a.status = dev_status;
  a.timeout_ticks = xs_host::ns_to_ticks((spin_timeout_us > 0 ? spin_timeout_us : 2000000) * 1000);
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (T > 0) {
    // a wave per chunk of tokens, and enough threads to clear the slots' words
    const int64_t blocks = std::max((chunks_of(T) + 3) / 4, std::min<int64_t>(1024, static_cast<int64_t>(W) * S / 1024));
    hipLaunchKernelGGL(ring::ring_rank_kernel, dim3(static_cast<unsigned>(blocks)), dim3(ring::kThreads), 0, st, a);
    if (xs_host::launch_status()) return XS_EHIP;
  }
  hipLaunchKernelGGL(ring::ring_scan_kernel, dim3(1), dim3(1024), 0, st, a);
  if (xs_host::launch_status()) return XS_EHIP;
  if (T > 0) {
    // two workgroups (eight agent waves) per CU, all resident; no more than a producer per token
    const int grid = std::min((T + 1) / 2, 2 * xs_host::persistent_grid(max_producers));
    hipLaunchKernelGGL(ring::ring_dispatch_kernel, dim3(grid), dim3(ring::kThreads), 0, st, a);
    if (xs_host::launch_status()) return XS_EHIP;
  }
  return xs_host::signal_windows(a.win, st);
}
