// Buffer-load and LDS helpers of the LDS-ring GEMM kernels (gemm.hip): raw
// buffer resources with 31-bit offsets, 16-byte loads
// straight into LDS (buffer_load ... lds), explicit wait counts and 16-byte
// LDS fragment reads.  Device code only; nothing here is part of the ABI.
#pragma once

#include <type_traits>
#include <utility>

#include "cts_internal.h"

namespace cts {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
constexpr uint32_t kOob = 0x80000000u;   // every operand is < 2^31 bytes

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, uint32_t nbytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), static_cast<short>(0),
                                           static_cast<int>(nbytes), 0x00020000);
}

__device__ __forceinline__ u32x4 load16(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  return __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0);
}

template <int BK> __device__ __forceinline__ int swz_key(int row) {
  if (BK == 128) return row & 15;
  return BK == 64 ? ((row >> 1) & 7) : ((row >> 2) & 3);
}

// The inline assembly below exists only in the device compilation pass (the
// host pass of a HIP translation unit never executes kernel bodies).
template <int N> __device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
#endif
}

template <int N> __device__ __forceinline__ void wait_lgkmcnt() {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(N) : "memory");
#endif
}

// Workgroup barrier for ordinary LDS data: waits for this wave's LDS
// operations only, and not, as __syncthreads does, for every load it has in
// flight into LDS.
__device__ __forceinline__ void lds_barrier() {
  wait_lgkmcnt<0>();
  __builtin_amdgcn_s_barrier();
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("" ::: "memory");
#endif
}

// 16-byte LDS read issued as assembly: its completion is waited for with
// wait_lgkmcnt, and pin() ties the fragment to that wait.
__device__ __forceinline__ void lds_read16(bf16x8& dst, uint32_t addr) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("ds_read_b128 %0, %1" : "=v"(dst) : "v"(addr) : "memory");
#endif
}

// The same at addr + OFF (0 <= OFF < 65536): the offset goes into the
// instruction, so reads a constant apart share one address register.
template <int OFF> __device__ __forceinline__ void lds_read16_at(bf16x8& dst, uint32_t addr) {
  static_assert(OFF >= 0 && OFF < 65536, "16-bit offset");
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "n"(OFF) : "memory");
#endif
}

// 8- and 4-byte LDS reads and writes as assembly, waited for with
// wait_lgkmcnt: the compiler would first wait for every load in flight into
// LDS, which it cannot tell apart from them.
__device__ __forceinline__ void lds_read8(uint64_t& dst, uint32_t addr) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("ds_read_b64 %0, %1" : "=v"(dst) : "v"(addr) : "memory");
#endif
}
__device__ __forceinline__ void lds_read4(uint32_t& dst, uint32_t addr) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("ds_read_b32 %0, %1" : "=v"(dst) : "v"(addr) : "memory");
#endif
}
__device__ __forceinline__ void lds_write8(uint32_t addr, uint64_t v) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("ds_write_b64 %0, %1" ::"v"(addr), "v"(v) : "memory");
#endif
}
__device__ __forceinline__ void lds_write4(uint32_t addr, uint32_t v) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("ds_write_b32 %0, %1" ::"v"(addr), "v"(v) : "memory");
#endif
}

// 16-byte buffer load of each lane straight into LDS: lane l's chunk lands at
// lds + 16*l (lds must be the same for the whole wave); out-of-range lanes
// write zeros.
__device__ __forceinline__ void load16_lds(__amdgpu_buffer_rsrc_t r, char* lds, uint32_t voff,
                                           uint32_t soff = 0) {
#if defined(__HIP_DEVICE_COMPILE__)
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)lds, 16, voff,
                                           soff, 0, 0);
#endif
}

__device__ __forceinline__ void pin(bf16x8& v) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("" : "+v"(v));
#endif
}

__device__ __forceinline__ void pin(uint64_t& v) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("" : "+v"(v));
#endif
}

__device__ __forceinline__ void pin(uint32_t& v) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("" : "+v"(v));
#endif
}

// f(0), ..., f(N - 1), the index a compile-time constant
template <typename F, int... I>
__device__ __forceinline__ void unrolled_steps(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F> __device__ __forceinline__ void unrolled(F&& f) {
  unrolled_steps(f, std::make_integer_sequence<int, N>{});
}

}  // namespace cts
