// Loads that go from memory straight into LDS.
#pragma once
#include "sea_internal.h"

namespace sea {

#if defined(__HIPCC__)

// raw buffer resource, word 3: 32-bit data format, no swizzle; loads past num_records return zero
constexpr int kBufferFlags = 0x00020000;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// 16 bytes per lane from a buffer straight into LDS: lane l of the wave writes at + 8 l.  `at` and the resource (the
// words of buffer_words) are wave-uniform.  Nothing the compiler does waits for these loads: lds_loads_done() does, and
// the barrier behind it makes the waves' pieces each other's.  (The builtin for this load makes the compiler wait for
// it in front of every transpose read, i.e. in the middle of the step that it is meant to run under.)
__device__ __forceinline__ u32x4 buffer_words(const void* base, uint32_t bytes) {
  const uint64_t p = reinterpret_cast<uint64_t>(base);
  return u32x4{static_cast<uint32_t>(p), static_cast<uint32_t>(p >> 32) & 0xffffu, bytes, static_cast<uint32_t>(kBufferFlags)};
}
// The memory side needs whole 4-byte words.  Tensors of 2-byte elements that start between two of them (their rows are
// whole words apart, so all loads of a tensor go the same way) pass through registers: load16_odd asks for a piece,
// park16 puts it where buffer_load_lds16 would.
// The five wait states in front of a load are for a resource whose words come from vector instructions just before (read
// lanes, a scalar that the compiler spilled among them): the compiler does not see the load and keeps no distance itself.
__device__ __forceinline__ void buffer_load_lds16(u32x4 r, uint16_t* at, uint32_t byte_off) {
  const uint32_t lds = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) void*)at));
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(lds), "v"(byte_off), "s"(r) : "memory", "m0");
}
// two pieces a lane, which share those wait states
__device__ __forceinline__ void buffer_load_lds16(u32x4 r, uint16_t* at0, uint32_t off0, uint16_t* at1, uint32_t off1) {
  const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) void*)at0));
  const uint32_t lds1 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) void*)at1));
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tbuffer_load_dwordx4 %2, %4, 0 offen lds\n\t"
               "s_mov_b32 m0, %1\n\ts_nop 0\n\tbuffer_load_dwordx4 %3, %4, 0 offen lds"
               ::"s"(lds0), "s"(lds1), "v"(off0), "v"(off1), "s"(r) : "memory", "m0");
}
__device__ __forceinline__ u32x4 load16_odd(u32x4 r, uint32_t byte_off) {
  typedef uint32_t anywhere __attribute__((ext_vector_type(4), aligned(2)));
  const auto* base = reinterpret_cast<const __attribute__((address_space(1))) char*>(r[0] | (static_cast<uint64_t>(r[1]) << 32));
  return *reinterpret_cast<const __attribute__((address_space(1))) anywhere*>(base + byte_off);
}
__device__ __forceinline__ void park16(uint16_t* at, u32x4 v) { reinterpret_cast<u32x4*>(at)[threadIdx.x & 63] = v; }
__device__ __forceinline__ void buffer_load_lds16_odd(u32x4 r, uint16_t* at, uint32_t byte_off) { park16(at, load16_odd(r, byte_off)); }
// buffer_load_lds16 with 4 bytes per lane: lane l writes word l
__device__ __forceinline__ void buffer_load_lds4(u32x4 r, uint32_t* at, uint32_t byte_off) {
  const uint32_t lds = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) void*)at));
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tbuffer_load_dword %1, %2, 0 offen lds" ::"s"(lds), "v"(byte_off), "s"(r) : "memory", "m0");
}
__device__ __forceinline__ void lds_loads_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
// waits until at most n (uniform, below eight) of the loads asked for last are on their way
__device__ __forceinline__ void lds_loads_pending(int n) {
  switch (n) {
    case 1: asm volatile("s_waitcnt vmcnt(1)" ::: "memory"); break;
    case 2: asm volatile("s_waitcnt vmcnt(2)" ::: "memory"); break;
    case 3: asm volatile("s_waitcnt vmcnt(3)" ::: "memory"); break;
    case 4: asm volatile("s_waitcnt vmcnt(4)" ::: "memory"); break;
    case 5: asm volatile("s_waitcnt vmcnt(5)" ::: "memory"); break;
    case 6: asm volatile("s_waitcnt vmcnt(6)" ::: "memory"); break;
    case 7: asm volatile("s_waitcnt vmcnt(7)" ::: "memory"); break;
    default: lds_loads_done(); break;
  }
}

#endif  // __HIPCC__

// does a tensor start between two 4-byte words?
inline bool starts_odd(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 3) != 0; }

}  // namespace sea
