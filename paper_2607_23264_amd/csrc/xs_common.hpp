// Shared device/host helpers of the gfx950 store-path library.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "xstage.h"

namespace xs {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kWave = 64;

// Window set passed by value to kernels (host xs_window array, copied into the kernel
// arguments so that device code never dereferences host memory).
struct WinSet {
  char* base[XS_MAX_WINDOWS];
  int64_t cap[XS_MAX_WINDOWS];
  int64_t stride[XS_MAX_WINDOWS];
  uint32_t* flag[XS_MAX_WINDOWS];
  int n;
};

// First error wins.
__device__ __forceinline__ void set_status(int32_t* st, int32_t code) {
  if (st) atomicCAS(st, 0, code);
}

// fp32 -> bf16 bits, round to nearest even; NaN stays a quiet NaN.
__device__ __forceinline__ uint32_t f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (u >> 16) | 0x40u;
  u += 0x7fffu + ((u >> 16) & 1u);
  return u >> 16;
}

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

// Two fp32 -> packed bf16 (lo in bits 0..15) with gfx950's v_cvt_pk_bf16_f32: round to
// nearest even, as f2bf, in one instruction and without a branch.
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  const bf16x2_t b = __builtin_convertvector(f32x2{lo, hi}, bf16x2_t);
  return __builtin_bit_cast(uint32_t, b);
}

__device__ __forceinline__ float bf_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

__device__ __forceinline__ uint64_t wall_ticks() { return wall_clock64(); }

// ------------------------------------------------------------------- direct loads into LDS
typedef __attribute__((address_space(3))) char lds_char;
typedef __attribute__((address_space(3))) bf16x8 lds_bf16x8;
typedef int v4i __attribute__((ext_vector_type(4)));

// A raw buffer descriptor over [base, base + bytes), wave-uniform: loads past its end fetch nothing.
// A memory instruction may read an SGPR that a vector instruction (readfirstlane) wrote only five
// wait states later, which the compiler does not see to for the assembly below: hence the s_nop.
__device__ __forceinline__ v4i buffer_rsrc(const void* base, uint32_t bytes) {
  const uint64_t b = reinterpret_cast<uint64_t>(base);
  v4i r = {static_cast<int>(__builtin_amdgcn_readfirstlane(static_cast<uint32_t>(b))),
           static_cast<int>(__builtin_amdgcn_readfirstlane(static_cast<uint32_t>(b >> 32)) & 0xFFFF),
           static_cast<int>(bytes), 0x00020000};
  asm("s_nop 4" : "+s"(r));
  return r;
}

// One 16-byte piece per lane from the buffer at voff (+ soff) into LDS at dst + 16 lane. Issued from
// assembly so that the compiler does not count it: it would wait for every load in flight
// before each LDS read (for transposing reads it cannot tell the two apart); the kernel waits itself,
// with vmcnt. A load into LDS may not directly follow the write of M0 that gives its address
// (one wait state), which the compiler does not see to around assembly: hence the s_nop.
__device__ __forceinline__ void load_lds16(v4i rsrc, uint32_t voff, const lds_char* dst) {
  const uint32_t m0v = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(dst));
  asm volatile("s_nop 0\n\tbuffer_load_dwordx4 %0, %1, 0 offen lds" :: "v"(voff), "s"(rsrc), "{m0}"(m0v) : "memory");
}
__device__ __forceinline__ void load_lds16(v4i rsrc, uint32_t voff, int soff, const lds_char* dst) {
  const uint32_t m0v = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(dst));
  asm volatile("s_nop 0\n\tbuffer_load_dwordx4 %0, %1, %2 offen lds"
               :: "v"(voff), "s"(rsrc), "s"(soff), "{m0}"(m0v) : "memory");
}

// A store past the L2 (agent scope, written through to memory): once it has completed (vmcnt), an
// agent-scope acquire on any XCD sees it, without the release that writes back the whole L2. Not
// counted by the compiler: the kernel waits with wait_vm. (The registers of a store of more than 64
// bits may be written again two wait states later; the compiler does not see to that here.)
__device__ __forceinline__ void store_through16(void* p, u32x4 v) {
  asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" :: "v"(p), "v"(v) : "memory");
}
__device__ __forceinline__ void store_through4(void* p, uint32_t v) {
  asm volatile("global_store_dword %0, %1, off sc1" :: "v"(p), "v"(v) : "memory");
}

// A uniform value, taken where it stands: what follows from it is computed there and not hoisted
// out of a persistent kernel's tile loop, where it would hold (and spill) registers across tiles.
__device__ __forceinline__ int uniform_here(int v) {
  asm volatile("" : "+s"(v));
  return v;
}

// Workgroup barrier for data exchanged in LDS only: global stores may still be in flight
// (__syncthreads waits until they have reached memory, a microsecond or two each time).
__device__ __forceinline__ void lds_sync() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

template <int V>
__device__ __forceinline__ void wait_vm() {   // s_waitcnt vmcnt(V) only
  static_assert(V >= 0 && V < 64);
  __builtin_amdgcn_s_waitcnt(0x0F70 | (V & 15) | ((V >> 4) << 14));
  asm volatile("" ::: "memory");
}

// Busy-wait for `ticks` wall-clock ticks without touching memory.
__device__ __forceinline__ void spin_ticks(uint64_t ticks) {
  if (!ticks) return;
  uint64_t t0 = wall_clock64();
  while (wall_clock64() - t0 < ticks) __builtin_amdgcn_s_sleep(1);
}

}  // namespace xs

// ------------------------------------------------------------------------------ host side
namespace xs_host {

// Validates a host window array and copies it into a kernel-argument WinSet.
// row_bytes: bytes each row must hold. Returns XS_OK or XS_EINVAL.
int make_winset(const xs_window* win, int32_t W, int64_t row_bytes, xs::WinSet* out);

int launch_status();                      // XS_OK, or XS_EHIP if the last launch failed
double wall_rate_hz();                    // wall-clock tick rate of the current device
int num_cus();                            // compute units of the current device
int64_t ns_to_ticks(int64_t ns);

}  // namespace xs_host
