// What the prompt-attention kernels (flash.hip, flash_short.hip) share: lane
// exchanges and the rotary embedding.
#pragma once
#include "common.h"

namespace qsvd {

constexpr int kFaK = 64;        // keys per tile
constexpr float kFaLog2e = 1.4426950408889634f;

// v_permlane32_swap (v_permlane16_swap) with both registers holding a value:
// a and b then hold this lane's and lane l ^ 32's (l ^ 16's), at vector-ALU
// latency (issued as asm with both registers read-write; the s_nop covers the
// hazard of a vector write just before).
__device__ __forceinline__ void fa_swap32(uint32_t& a, uint32_t& b) {
  asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(a), "+v"(b));
}
__device__ __forceinline__ void fa_swap16(uint32_t& a, uint32_t& b) {
  asm volatile("s_nop 1\n\tv_permlane16_swap_b32 %0, %1" : "+v"(a), "+v"(b));
}
// Max and sum over lanes l, l ^ 32, both receiving it.
__device__ __forceinline__ float fa_pair_max(float x) {
  uint32_t a = __builtin_bit_cast(uint32_t, x), b = a;
  fa_swap32(a, b);
  return fmaxf(__builtin_bit_cast(float, a), __builtin_bit_cast(float, b));
}
__device__ __forceinline__ float fa_pair_sum(float x) {
  uint32_t a = __builtin_bit_cast(uint32_t, x), b = a;
  fa_swap32(a, b);
  return __builtin_bit_cast(float, a) + __builtin_bit_cast(float, b);
}
// ... and over lanes l, l ^ 16, l ^ 32, l ^ 48.
__device__ __forceinline__ float fa_rows4_max(float x) {
  uint32_t a = __builtin_bit_cast(uint32_t, fa_pair_max(x)), b = a;
  fa_swap16(a, b);
  return fmaxf(__builtin_bit_cast(float, a), __builtin_bit_cast(float, b));
}
__device__ __forceinline__ float fa_rows4_sum(float x) {
  uint32_t a = __builtin_bit_cast(uint32_t, fa_pair_sum(x)), b = a;
  fa_swap16(a, b);
  return __builtin_bit_cast(float, a) + __builtin_bit_cast(float, b);
}

// Rotary embedding: the rotate-half pairs (a[e], b[e]) of channels j0 + e are
// turned by the angle pos * theta^(-2j/dh).  freq[j] holds
// theta^(-2j/dh) / (2 pi), so the angle in revolutions is formed and reduced
// to [0, 1) in fp64; sine and cosine then come from the hardware's
// revolution-based instructions in fp32, and the turned rows are rounded to
// fp16 for the matrix cores, like the unturned ones.
__device__ __forceinline__ double fa_freq(int j, int dh, double log2_theta) {
  return exp2(-2.0 * j / dh * log2_theta) * 0.15915494309189533576888376337251;
}
__device__ __forceinline__ void fa_angle(int pos, double freq, float* c, float* s) {
  const float x = (float)__builtin_amdgcn_fract((double)pos * freq);
  *c = __builtin_amdgcn_cosf(x);
  *s = __builtin_amdgcn_sinf(x);
}
__device__ __forceinline__ void fa_turn8(f16x8& a, f16x8& b, const float* c, const float* s) {
  f16x8 ra, rb;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const float fa = (float)a[e], fb = (float)b[e];
    ra[e] = (_Float16)(fa * c[e] - fb * s[e]);
    rb[e] = (_Float16)(fb * c[e] + fa * s[e]);
  }
  a = ra;
  b = rb;
}
__device__ __forceinline__ void fa_rope8(f16x8& a, f16x8& b, int pos, const double* freq) {
  float c[8], s[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) fa_angle(pos, freq[e], &c[e], &s[e]);
  fa_turn8(a, b, c, s);
}

}  // namespace qsvd
