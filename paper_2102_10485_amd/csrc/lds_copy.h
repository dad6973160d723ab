// Copies from global memory straight into LDS, bounds-checked buffers, and LDS reads that transpose.
#pragma once

#include <type_traits>

#include "common.h"

namespace gan {

// 16 bytes per lane from a buffer straight into LDS: the wave's 64 lanes fill the 1 KiB starting at lds_base
// (wave-uniform) in lane order; a lane whose byte offset lies outside the buffer (NO_ROW below) delivers zeros,
// which is how padding taps, rows past a model's end and columns past N are filled.  Completion is counted by
// vmcnt like any vector load.
typedef int int4v __attribute__((ext_vector_type(4)));
constexpr unsigned NO_ROW = 0xffffffffu;
__device__ inline int4v make_rsrc(const void* base, unsigned long long bytes) {
  const unsigned long long p = (unsigned long long)base;
  int4v r;
  r.x = __builtin_amdgcn_readfirstlane((int)(unsigned)p);
  r.y = __builtin_amdgcn_readfirstlane((int)((unsigned)(p >> 32) & 0xffffu));                 // stride 0: raw buffer
  r.z = __builtin_amdgcn_readfirstlane((int)(unsigned)(bytes > 0xfffffff0ull ? 0xfffffff0ull : bytes));
  r.w = 0x00020000;
  return r;
}
__device__ inline __amdgpu_buffer_rsrc_t buffer_of(const void* base, unsigned long long bytes) {      // the same for the load builtins
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)(unsigned)(bytes > 0xfffffff0ull ? 0xfffffff0ull : bytes), 0x00020000);
}
// The wave-uniform part of the offset (which tap, which channels) travels in a scalar register.
__device__ inline void load16_to_lds(const int4v& rsrc, unsigned byte_off, unsigned uniform_off, unsigned lds_base) {
  asm volatile("s_mov_b32 m0, %3\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, %2 offen lds"
               : : "v"(byte_off), "s"(rsrc), "s"(__builtin_amdgcn_readfirstlane((int)uniform_off)), "s"(__builtin_amdgcn_readfirstlane((int)lds_base)) : "memory", "m0");
}
// The same with the LDS address as a scalar base and a constant, which then takes no register of its own.
template <int LDS_OFF>
__device__ inline void load16_to_lds_at(const int4v& rsrc, unsigned byte_off, unsigned uniform_off, int lds_base) {
  asm volatile("s_add_u32 m0, %3, %4\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, %2 offen lds"
               : : "v"(byte_off), "s"(rsrc), "s"(__builtin_amdgcn_readfirstlane((int)uniform_off)), "s"(lds_base), "n"(LDS_OFF) : "memory", "m0", "scc");
}
// wait until at most N loads are still in flight
template <int N>
__device__ inline void wait_vm() {
  static_assert(N <= 63, "vmcnt range");
  asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory");
}

// ds_read_b64_tr_b16: within each block of 16 lanes, lane i receives element i % 4 of the 8-byte groups addressed by lanes
// i / 4, 4 + i / 4, 8 + i / 4, 12 + i / 4.
typedef short short4v __attribute__((ext_vector_type(4)));
__device__ inline uint2 lds_read_tr16(const unsigned char* p) {
  const short4v v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) short4v*)(p));
  return __builtin_bit_cast(uint2, v);
}

template <int I, int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<I + 1, N>(f);
  }
}

}  // namespace gan
