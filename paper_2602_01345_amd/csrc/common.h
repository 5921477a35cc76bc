// Device-side helpers shared by the gfx950 kernels of this library.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#define NOVA_WAVE 64

typedef __bf16 bf16_t;
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float bf16_bits_to_f32(uint32_t h) { return __uint_as_float(h << 16); }

// element load/store with widening to fp32 (T = float or bf16_t)
template <typename T> __device__ __forceinline__ float ld_f32(const T* p) { return (float)*p; }
template <typename T> __device__ __forceinline__ void st_f32(T* p, float v) { *p = (T)v; }

// 16-byte vector of T as fp32 lanes
template <typename T> struct Vec16;
template <> struct Vec16<float> {
  static constexpr int N = 4;
  f32x4 v;
  __device__ __forceinline__ void load(const float* p) { v = *reinterpret_cast<const f32x4*>(p); }
  __device__ __forceinline__ void store(float* p) const { *reinterpret_cast<f32x4*>(p) = v; }
  __device__ __forceinline__ float get(int i) const { return v[i]; }
  __device__ __forceinline__ void set(int i, float x) { v[i] = x; }
};
template <> struct Vec16<bf16_t> {
  static constexpr int N = 8;
  bf16x8 v;
  __device__ __forceinline__ void load(const bf16_t* p) { v = *reinterpret_cast<const bf16x8*>(p); }
  __device__ __forceinline__ void store(bf16_t* p) const { *reinterpret_cast<bf16x8*>(p) = v; }
  __device__ __forceinline__ float get(int i) const { return (float)v[i]; }
  __device__ __forceinline__ void set(int i, float x) { v[i] = (bf16_t)x; }
};

// Global -> LDS: 16 bytes per lane from base + lane_off + off (bytes; base and off wave-uniform) into 1 KB of LDS at dst.
// Offsets have 32 bits and are bounded at 2^31 - 1: loads from there on give zeros.
typedef __attribute__((address_space(3))) void* lptr_t;
__device__ __forceinline__ void fill_lds(const bf16_t* base, char* dst, uint32_t lane_off, uint32_t off) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(
      __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(base), 0, 0x7FFFFFFF, 0x00020000), (lptr_t)dst, 16, lane_off, off, 0, 0);
}

constexpr float kNormEps = 1e-6f;          // of the LayerNorms

// Per-image keep counts (the reduction ratios of Sec. 3.3, "Dual-Linkage Acceleration", are per instance): the
// kept rows of image b are slots [0, k_b) of its kpitch-row segment, and it holds its own number of prior K/V rows.
// Null pointers mean "uniform": every image keeps kpitch rows / holds P prior rows.  Values are clamped, so a
// count the host never saw cannot send a kernel out of bounds.
__device__ __forceinline__ int image_count(const int32_t* __restrict__ k_rows, int b, int kpitch) {
  if (!k_rows) return kpitch;
  const int v = k_rows[b];
  return v < 0 ? 0 : (v > kpitch ? kpitch : v);
}
__device__ __forceinline__ int image_prior(const int32_t* __restrict__ kv_rows, int b, int P) {
  if (!kv_rows) return P;
  const int v = kv_rows[b];
  return v < 0 ? 0 : (v > P ? P : v);
}

// Wave-wide sum / maximum on the DPP cross-lane paths of the vector ALU (quads, half rows, rows of 16, then the two
// row broadcasts), read back from lane 63 as a wave-uniform scalar: six dependent vector instructions and no trip
// through the LDS crossbar, which is what a butterfly of lane shuffles costs six times over.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_or(float v, float identity) {
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(identity), __float_as_int(v), CTRL, ROW_MASK, 0xF, false));
}
// (of each sixteen lanes, in all of them)
__device__ __forceinline__ float row16_sum(float v) {
  v += dpp_or<0xB1, 0xF>(v, 0.0f);
  v += dpp_or<0x4E, 0xF>(v, 0.0f);
  v += dpp_or<0x141, 0xF>(v, 0.0f);
  return v + dpp_or<0x140, 0xF>(v, 0.0f);
}
__device__ __forceinline__ float wave_sum(float v) {
  v += dpp_or<0xB1, 0xF>(v, 0.0f);          // quad_perm [1,0,3,2]
  v += dpp_or<0x4E, 0xF>(v, 0.0f);          // quad_perm [2,3,0,1]
  v += dpp_or<0x141, 0xF>(v, 0.0f);         // row_half_mirror
  v += dpp_or<0x140, 0xF>(v, 0.0f);         // row_mirror: every lane holds the sum of its row of 16
  v += dpp_or<0x142, 0xA>(v, 0.0f);         // row_bcast15 into rows 1 and 3
  v += dpp_or<0x143, 0xC>(v, 0.0f);         // row_bcast31 into rows 2 and 3: lane 63 holds the total
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}
__device__ __forceinline__ float wave_max(float v) {
  v = fmaxf(v, dpp_or<0xB1, 0xF>(v, -INFINITY));
  v = fmaxf(v, dpp_or<0x4E, 0xF>(v, -INFINITY));
  v = fmaxf(v, dpp_or<0x141, 0xF>(v, -INFINITY));
  v = fmaxf(v, dpp_or<0x140, 0xF>(v, -INFINITY));
  v = fmaxf(v, dpp_or<0x142, 0xA>(v, -INFINITY));
  v = fmaxf(v, dpp_or<0x143, 0xC>(v, -INFINITY));
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

// Division of 0 <= n < 2^31 by d >= 1 through inv = div_inv(d), made once on the host: the high half of n * inv is the
// quotient or one less.
inline uint32_t div_inv(int d) { return 0xFFFFFFFFu / (uint32_t)(d > 0 ? d : 1); }
__device__ __forceinline__ int div_by(int n, int d, uint32_t inv, int& rem) {
  int q = (int)__umulhi((uint32_t)n, inv);
  rem = n - q * d;
  if (rem >= d) { ++q; rem -= d; }
  return q;
}
