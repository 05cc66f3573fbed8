// Device-side helpers shared by the libtg kernels (gfx950, wave64).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace tg {

constexpr int kWave = 64;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float bf16_to_f32(uint16_t b) {
  return __uint_as_float(static_cast<uint32_t>(b) << 16);
}

// float32 -> bf16, round to nearest even. The conversion compiles to
// v_cvt_pk_bf16_f32 (one instruction for a pair); for every non-NaN input it
// gives the bits of adding 0x7fff plus the lowest kept bit and truncating
// (checked on an MI355X over all 2^32 float32 patterns); NaN stays NaN.
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint16_t f32_to_bf16(float f) {
  return __builtin_bit_cast(uint16_t, (__bf16)f);
}

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  const bf16x2_t v = {(__bf16)lo, (__bf16)hi};
  return __builtin_bit_cast(uint32_t, v);
}

__device__ __forceinline__ int lane_id() { return __lane_id(); }

// Waits until at most n of the wave's vector-memory loads are in flight.
#define TG_WAIT_VM(n) \
  __builtin_amdgcn_s_waitcnt(((n) & 0xF) | (((n) >> 4) << 14) | (0x7 << 4) | (0xF << 8))

__device__ __forceinline__ void block_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

typedef __attribute__((address_space(3))) uint16_t lds_u16;

// One 16-byte global -> LDS transfer per lane; the wave's 64 chunks land at
// consecutive 16-byte positions starting at the (wave-uniform) `lds` row.
__device__ __forceinline__ void load_lds16(__amdgpu_buffer_rsrc_t rsrc, lds_u16* lds, int voffset,
                                           int soffset) {
#if defined(__HIP_DEVICE_COMPILE__)
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (__attribute__((address_space(3))) void*)lds, 16,
                                           voffset, soffset, 0, 0);
#endif
}

// Raw buffer resource over [base, base + bytes); loads beyond it return 0.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)bytes, 0x00020000);
}

}  // namespace tg
