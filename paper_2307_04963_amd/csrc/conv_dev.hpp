// Device helpers shared by the bf16 convolution kernels: vector types, the
// epilogues' arithmetic, loads straight into LDS and barriers.
#pragma once

#include "gelu.hpp"
#include "kernels.hpp"

namespace dycl {
namespace k {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void* lds_void_ptr;

// round to nearest even (v_cvt_pk_bf16_f32; NaN stays NaN), as every
// kernel's epilogue
__device__ __forceinline__ uint16_t f2bf(float f) { return __builtin_bit_cast(uint16_t, static_cast<__bf16>(f)); }

__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  const bf16x2 v = {static_cast<__bf16>(lo), static_cast<__bf16>(hi)};
  return __builtin_bit_cast(uint32_t, v);
}

__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float(static_cast<uint32_t>(h) << 16); }

// the element row (image * HoWo + pixel) that layer row `row` maps to
// through an image list (null: itself)
__device__ __forceinline__ size_t row_at(const int32_t* rows, int row, int HoWo) {
  if (!rows) return static_cast<size_t>(row);
  const int img = row / HoWo;
  return static_cast<size_t>(rows[img]) * HoWo + (row - img * HoWo);
}

template <int ACT>
__device__ __forceinline__ float act_t(float v) {
  if (ACT == ACT_RELU) return v > 0.f ? v : 0.f;
  if (ACT == ACT_GELU) return gelu_f32(v);
  if (ACT == ACT_TANH) return tanhf(v);
  return v;
}

__device__ __forceinline__ float apply_act(float v, int act) {
  if (act == ACT_RELU) return v > 0.f ? v : 0.f;
  if (act == ACT_GELU) return gelu_f32(v);
  if (act == ACT_TANH) return tanhf(v);
  return v;
}

__device__ __forceinline__ float sigmoidf(float v) { return 1.0f / (1.0f + expf(-v)); }

// Wait until at most N vector-memory operations of this thread are still in
// flight (loads complete in order, so every older one - the tile about to be
// read - has landed), then barrier.  Inline asm with a memory clobber keeps
// the compiler from moving LDS reads across it and from widening the wait.
template <int N>
__device__ __forceinline__ void wait_vm_barrier() {
  static_assert(N >= 0 && N < 64, "vmcnt is 6 bits");
  asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(N) : "memory");
}

// 16 bytes per lane from a raw buffer straight into LDS at `lds` + 16 * lane:
// the buffer spans `bytes` from `base`, and a load at or past its end (an
// offset of 2^31 or more included) writes zeros instead of reading memory.
__device__ __forceinline__ void buffer_load_lds16(const void* base, uint32_t bytes, uint32_t offset, lds_void_ptr lds) {
  const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, bytes, 0x00020000);
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, lds, 16, offset, 0, 0, 0);
}

// 16 bytes per lane from a raw buffer of `bytes` from `base`; zeros at or past its end
__device__ __forceinline__ u32x4 buffer_load16(const void* base, uint32_t bytes, uint32_t offset) {
  const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, bytes, 0x00020000);
  return __builtin_amdgcn_raw_buffer_load_b128(r, offset, 0, 0);
}

// 16 bytes per lane to a raw buffer of `bytes` from `base`; a store at or
// past its end is dropped.
__device__ __forceinline__ void buffer_store16(void* base, uint32_t bytes, uint32_t offset, u32x4 v) {
  const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(base, 0, bytes, 0x00020000);
  __builtin_amdgcn_raw_buffer_store_b128(v, r, offset, 0, 0);
}

// (M0, which the loads below set, is a reserved register: the compiler is told
// of the write and keeps nothing there, which is all the warning is about)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"

// 16 bytes per lane from `src` (per lane) straight into LDS at `lds` + 16 *
// lane (the same for all lanes).  Unlike the builtin the compiler does not
// track it: it places no waits before LDS reads on its account (it cannot
// tell the stages of one buffer apart and would wait for every load in
// flight), so whoever issues it waits for it before the barrier that releases
// the data.  No register is written.
__device__ __forceinline__ void load_lds16(const void* src, const void* lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
               :
               : "s"((lds_void_ptr)(lds)), "v"(src)
               : "memory", "m0");
}

// the same from `base` (the same for all lanes) + a byte offset per lane
__device__ __forceinline__ void load_lds16(const void* base, uint32_t offset, const void* lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
               :
               : "s"((lds_void_ptr)(lds)), "v"(offset), "s"(base)
               : "memory", "m0");
}

// the same from a raw buffer: `offset` (per lane) past its end brings zeros;
// `add` (the same for all lanes) moves the address within it
__device__ __forceinline__ void buffer_lds16(u32x4 rsrc, uint32_t offset, uint32_t add, const void* lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
               :
               : "s"((lds_void_ptr)(lds)), "v"(offset), "s"(rsrc), "s"(add)
               : "memory", "m0");
}

#pragma clang diagnostic pop

// a raw buffer's descriptor, in scalar registers
__device__ __forceinline__ u32x4 raw_buffer(const void* base, uint32_t bytes) {
  const uint64_t b = reinterpret_cast<uint64_t>(base);
  return u32x4{static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<uint32_t>(b))),
               static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<uint32_t>(b >> 32) & 0xffffu)),
               static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(bytes)), 0x00020000u};
}

// every load and LDS access of this thread done, then barrier; waits that the
// compiler sees, so it adds none of its own for the loads that they cover
__device__ __forceinline__ void seen_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0);
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }
__device__ __forceinline__ void all_barrier() { asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

}  // namespace k
}  // namespace dycl
