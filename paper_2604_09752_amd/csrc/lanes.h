// Lane exchanges, division and device-coherent access of the verify and prefill
// kernels (the step kernel does not use them).
#pragma once

#include "common.h"

// Division by a number the host knows: n / d as the high half of a product, for
// the n below the limit given to make_udiv (inv 0: divide).  A division by a
// kernel argument is some 30 instructions in a row (64-bit: over 100), on the
// path to a kernel's first loads.  Without them: verify of the 1B, 3 rows at
// 1531, 1142 -> 1127 us (7B, 9 rows at 2048, 3443 -> 3417), prefill of 23 rows of
// the 1B 2011 -> 1988, 2048 rows 14706 -> 14643.
struct UDiv {
  unsigned inv, d;
};
inline UDiv make_udiv(unsigned d, unsigned limit) {
  // 2^32 / d rounded up is exact while n d <= 2^32
  const bool ok = d > 1 && (uint64_t)limit * d <= (1ull << 32);
  return UDiv{ok ? (unsigned)(((1ull << 32) + d - 1) / d) : 0u, d};
}
AIO_DEV int udiv(int n, const UDiv& v) {
  if (v.inv) return (int)__umulhi((unsigned)n, v.inv);
  return v.d == 1 ? n : (int)((unsigned)n / v.d);
}

// log2 of a head dimension (64 or 128).
AIO_DEV int hd_shift(int hd) { return hd == 128 ? 7 : 6; }

// Maximum over aligned groups of 8 lanes, as group_sum_dpp sums them.
AIO_DEV float group_max8_dpp(float v) {
  v = fmaxf(v, dpp_mov<0xB1>(v));
  v = fmaxf(v, dpp_mov<0x4E>(v));
  return fmaxf(v, dpp_mov<0x141>(v));
}

// Transposing LDS read of 16-bit values.  In each group of 16 lanes, lanes 4 e
// .. 4 e + 3 give the addresses of the four quarters (4 values, 8 bytes each)
// of row e, and lane i receives column i of the four rows: {row 0, .., row
// 3}[i].  `p` points into LDS.
typedef short i16x4 __attribute__((ext_vector_type(4)));
AIO_DEV uint2 lds_read_tr16(const void* p) {
  const i16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (__attribute__((address_space(3))) i16x4*)p);
  return __builtin_bit_cast(uint2, v);
}

// Device-coherent access for sums that workgroups hand to one another (K slices,
// attention splits): written through to memory and read past the (per-XCD) L2, so
// the hand-over needs no fence that writes back or drops a whole L2 (with fences, it
// cost about 40 us per product).  The arrival counters are vector atomics at device
// scope.
AIO_DEV void st_agent(float* p, float v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
AIO_DEV float ld_agent(const float* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
AIO_DEV int atomic_add_agent(int* p, int v) {
  return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
AIO_DEV int atomic_load_agent(const int* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
AIO_DEV void atomic_store_agent(int* p, int v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Wait for this wave's LDS operations; also a compiler barrier, so no LDS access
// moves across it.  Lanes of one wave exchange data through LDS without a workgroup
// barrier (the waves of a workgroup run different numbers of iterations).
AIO_DEV void wave_lds_sync() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }
