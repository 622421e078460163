// wave_pair.h -- memory access of kernels whose lanes own two x-adjacent points
// (wave_kernels_pair.hip, wave_kernels_block.hip).

#pragma once

#include "wave_point.h"

namespace wave {
namespace {

typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

// pair access per storage type: load two values (byte offset of the first),
// store two values
template <class S> struct PairIO;
template <> struct PairIO<StF32> {
  static __device__ __forceinline__ f32x2 ld(__amdgpu_buffer_rsrc_t r, uint32_t vo, uint32_t so) {
    const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(r, (int)vo, (int)so, 0);
    return f32x2{__uint_as_float(v[0]), __uint_as_float(v[1])};
  }
  static __device__ __forceinline__ f32x2 ld1(__amdgpu_buffer_rsrc_t r, uint32_t vo, uint32_t so) {
    const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(r, (int)vo, (int)so, kLdOnce);
    return f32x2{__uint_as_float(v[0]), __uint_as_float(v[1])};
  }
  static __device__ __forceinline__ void st(__amdgpu_buffer_rsrc_t r, uint32_t vo, uint32_t so,
                                            float a, float b) {
    __builtin_amdgcn_raw_buffer_store_b64(u32x2{__float_as_uint(a), __float_as_uint(b)}, r,
                                          (int)vo, (int)so, kSt);
  }
};
template <> struct PairIO<StBF16> {
  static __device__ __forceinline__ f32x2 unpack(uint32_t v) {
    return f32x2{__uint_as_float(v << 16), __uint_as_float(v & 0xffff0000u)};
  }
  static __device__ __forceinline__ f32x2 ld(__amdgpu_buffer_rsrc_t r, uint32_t vo, uint32_t so) {
    return unpack(__builtin_amdgcn_raw_buffer_load_b32(r, (int)vo, (int)so, 0));
  }
  static __device__ __forceinline__ f32x2 ld1(__amdgpu_buffer_rsrc_t r, uint32_t vo, uint32_t so) {
    return unpack(__builtin_amdgcn_raw_buffer_load_b32(r, (int)vo, (int)so, kLdOnce));
  }
  static __device__ __forceinline__ void st(__amdgpu_buffer_rsrc_t r, uint32_t vo, uint32_t so,
                                            float a, float b) {
    const uint32_t v = (uint32_t)StBF16::enc(a) | ((uint32_t)StBF16::enc(b) << 16);
    __builtin_amdgcn_raw_buffer_store_b32(v, r, (int)vo, (int)so, kSt);
  }
};
template <> struct PairIO<StBF16SR> : PairIO<StBF16> {};
template <> struct PairIO<StF16> {
  static __device__ __forceinline__ f32x2 unpack(uint32_t v) {
    return f32x2{(float)__builtin_bit_cast(_Float16, (uint16_t)(v & 0xffffu)),
                 (float)__builtin_bit_cast(_Float16, (uint16_t)(v >> 16))};
  }
  static __device__ __forceinline__ f32x2 ld(__amdgpu_buffer_rsrc_t r, uint32_t vo, uint32_t so) {
    return unpack(__builtin_amdgcn_raw_buffer_load_b32(r, (int)vo, (int)so, 0));
  }
  static __device__ __forceinline__ f32x2 ld1(__amdgpu_buffer_rsrc_t r, uint32_t vo, uint32_t so) {
    return unpack(__builtin_amdgcn_raw_buffer_load_b32(r, (int)vo, (int)so, kLdOnce));
  }
  static __device__ __forceinline__ void st(__amdgpu_buffer_rsrc_t r, uint32_t vo, uint32_t so,
                                            float a, float b) {
    const uint32_t v = (uint32_t)__builtin_bit_cast(uint16_t, StF16::enc(a)) |
                       ((uint32_t)__builtin_bit_cast(uint16_t, StF16::enc(b)) << 16);
    __builtin_amdgcn_raw_buffer_store_b32(v, r, (int)vo, (int)so, kSt);
  }
};

__device__ __forceinline__ f32x2 ld_f32x2(__amdgpu_buffer_rsrc_t r, uint32_t vo, uint32_t so,
                                          bool once) {
  const u32x2 v = once ? __builtin_amdgcn_raw_buffer_load_b64(r, (int)vo, (int)so, kLdOnce)
                       : __builtin_amdgcn_raw_buffer_load_b64(r, (int)vo, (int)so, 0);
  return f32x2{__uint_as_float(v[0]), __uint_as_float(v[1])};
}

}  // namespace
}  // namespace wave
