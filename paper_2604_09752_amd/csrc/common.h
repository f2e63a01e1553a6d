// Device helpers shared by the decode and verify kernels (gfx950, wave64).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#define AIO_WAVE 64
#define AIO_DEV __device__ __forceinline__

// bf16 -> fp32 is a 16-bit shift; both halves of a packed dword.
AIO_DEV float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
AIO_DEV float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }
AIO_DEV float bf16_to_f32(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

// fp32 -> bf16 bits, round to nearest even (NaN kept quiet).
AIO_DEV uint16_t f32_to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

AIO_DEV float fp16_to_f32(uint16_t h) { return (float)__builtin_bit_cast(_Float16, h); }

// Sum over aligned groups of `width` lanes (a power of two <= 64).
template <int WIDTH>
AIO_DEV float group_sum(float v) {
#pragma unroll
  for (int off = WIDTH / 2; off >= 1; off >>= 1) v += __shfl_xor(v, off, AIO_WAVE);
  return v;
}

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// 16-byte streaming load of weights (read once per token: no reuse to keep).
AIO_DEV uint4 ld_stream(const uint4* p) {
  const u32x4 v = __builtin_nontemporal_load((const u32x4*)p);
  return make_uint4(v.x, v.y, v.z, v.w);
}

// dot of 8 bf16 (one uint4) with 8 fp32 activations.
AIO_DEV float dot8_bf16(uint4 w, const float4 a, const float4 b, float acc) {
  acc = fmaf(bf16_lo(w.x), a.x, acc);
  acc = fmaf(bf16_hi(w.x), a.y, acc);
  acc = fmaf(bf16_lo(w.y), a.z, acc);
  acc = fmaf(bf16_hi(w.y), a.w, acc);
  acc = fmaf(bf16_lo(w.z), b.x, acc);
  acc = fmaf(bf16_hi(w.z), b.y, acc);
  acc = fmaf(bf16_lo(w.w), b.z, acc);
  acc = fmaf(bf16_hi(w.w), b.w, acc);
  return acc;
}

// int8 byte j of a dword, sign-extended, as fp32 (exact).
AIO_DEV float i8_at(uint32_t w, int j) { return (float)(int8_t)(w >> (8 * j)); }

// dot of 4 int8 (one dword) with 4 fp32 activations.
AIO_DEV float dot4_i8(uint32_t w, const float4 a, float acc) {
  acc = fmaf(i8_at(w, 0), a.x, acc);
  acc = fmaf(i8_at(w, 1), a.y, acc);
  acc = fmaf(i8_at(w, 2), a.z, acc);
  acc = fmaf(i8_at(w, 3), a.w, acc);
  return acc;
}

// One DPP lane move of a float (a VALU operation: no LDS round trip).
template <int CTRL>
AIO_DEV float dpp_mov(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}

// Sum over aligned groups of 8 or 16 lanes; every lane of a group receives
// the same total.  Each step adds a lane's value to that of a partner in the
// other half of its current group: lane ^ 1, lane ^ 2 (quad permutations),
// then the mirror lane of the other quad (row_half_mirror) and, for 16, of
// the other half row (row_mirror).
template <int WIDTH>
AIO_DEV float group_sum_dpp(float v) {
  static_assert(WIDTH == 8 || WIDTH == 16, "DPP sums cover 8 or 16 lanes");
  v += dpp_mov<0xB1>(v);   // quad_perm [1, 0, 3, 2]
  v += dpp_mov<0x4E>(v);   // quad_perm [2, 3, 0, 1]
  v += dpp_mov<0x141>(v);  // row_half_mirror
  if (WIDTH == 16) v += dpp_mov<0x140>(v);  // row_mirror
  return v;
}

// Lane exchanges between the halves and between the rows of 16 of a wave, as
// VALU swaps (an LDS exchange takes an LDS round trip and its wait):
//   swap32: a = {a.lo, b.lo}, b = {a.hi, b.hi}   (lanes 0-31, 32-63)
//   swap16: a = {a0, b0, a2, b2}, b = {a1, b1, a3, b3}   (rows of 16 lanes)
AIO_DEV void swap32(float& a, float& b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  a = __uint_as_float(r[0]);
  b = __uint_as_float(r[1]);
}
AIO_DEV void swap16(float& a, float& b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  a = __uint_as_float(r[0]);
  b = __uint_as_float(r[1]);
}

// The value of lane ^ 4: lanes with bit 2 clear read four lanes up (row_shl:4),
// the others four lanes down (row_shr:4).
AIO_DEV float dpp_xor4(float v) {
  const int x = __float_as_int(v);
  const int t = __builtin_amdgcn_update_dpp(0, x, 0x104, 0xF, 0x5, false);
  return __int_as_float(__builtin_amdgcn_update_dpp(t, x, 0x114, 0xF, 0xA, false));
}

// Sum and maximum over the 64 lanes of a wave; every lane receives the same
// total.  VALU steps, where exchanges through LDS take six round trips.  The sum
// exchanges over lane bits 5 to 0 in that order (results behind a short cache
// depend on the order of sums: see the test of their bits).
AIO_DEV float half_wave_sum(float v) {
  float o = v;
  swap16(v, o);
  v += o;
  v += dpp_mov<0x128>(v);  // row_ror:8, lane ^ 8
  v += dpp_xor4(v);
  v += dpp_mov<0x4E>(v);  // lane ^ 2
  return v + dpp_mov<0xB1>(v);  // lane ^ 1
}
AIO_DEV float wave_sum(float v) {
  float o = v;
  swap32(v, o);
  return half_wave_sum(v + o);
}
// The sum of x^2, the lower half's squares fused into the first exchange.
AIO_DEV float wave_sum_sq(float x) {
  float o = x;
  swap32(x, o);
  return half_wave_sum(fmaf(x, x, o * o));
}
AIO_DEV float wave_max(float v) {
  v = fmaxf(v, dpp_mov<0xB1>(v));
  v = fmaxf(v, dpp_mov<0x4E>(v));
  v = fmaxf(v, dpp_mov<0x141>(v));
  v = fmaxf(v, dpp_mov<0x140>(v));
  float o = v;
  swap16(v, o);
  v = fmaxf(v, o);
  o = v;
  swap32(v, o);
  return fmaxf(v, o);
}
