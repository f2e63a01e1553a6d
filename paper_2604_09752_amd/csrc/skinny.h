// Staging of the skinny products: the verify's (up to 10 rows) and those of
// short prompt chunks (up to 32).  Included by one kernel source each.
#pragma once

#include "aio.h"
#include "common.h"

namespace {

// The skinny GEMM runs 8 waves per workgroup: more weight loads in flight
// per CU, and the K range of a workgroup split eight ways.
constexpr int kGBlock = 512;
constexpr int kGWaves = kGBlock / AIO_WAVE;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(1))) const u32x4 gl_u32x4;

AIO_DEV bf16x8 as_bf16x8(uint4 u) { return __builtin_bit_cast(bf16x8, u); }

// 16-byte loads through a global-address-space pointer.  Selected from a
// table the pointer's address space is unknown, and a flat load also counts
// against the LDS wait counter: every LDS wait would then wait for the
// weights in flight as well.
AIO_DEV uint4 ldg_nt(const void* p) {
  const u32x4 v = __builtin_nontemporal_load((gl_u32x4*)p);
  return make_uint4(v.x, v.y, v.z, v.w);
}
AIO_DEV uint4 ldg(const void* p) {
  const u32x4 v = *(gl_u32x4*)p;
  return make_uint4(v.x, v.y, v.z, v.w);
}

// The k of the two MFMA fragments a lane holds in a block of 32 k (lane
// half kh = l / 32): for bf16, k .. k+7 and k+16 .. k+23 from block + 8 kh;
// for int8, the 16 consecutive k from block + 16 kh.  Weights (frag_lds)
// and activations use the same k, so the permutation cancels.
template <int WFMT>
AIO_DEV int vk_lo(int block, int kh) { return WFMT == AIO_WFMT_BF16 ? block + 8 * kh : block + 16 * kh; }
template <int WFMT>
AIO_DEV int vk_hi(int block, int kh) { return WFMT == AIO_WFMT_BF16 ? block + 16 + 8 * kh : block + 16 * kh + 8; }

// Weights reach the MFMA through LDS in stages of 256 k per row (64 rows:
// 32 KB of bf16, 16 KB of int8), two stages in flight per workgroup.  Read
// straight into the MFMA operand layout, every load instruction would span
// 32 rows at 16-32 bytes each; staged, consecutive lanes read consecutive
// 16-byte chunks of one row, and the 64 rows of a stage go to LDS with a
// 16-byte skew per row, so that the fragment reads (32 rows at one column)
// spread over the banks.  Stages of 1 KB per row (64 KB, one workgroup per
// CU) measured slower: 5.16 against 4.89 ms per 7B bf16 verify.
template <int WFMT>
struct VStage {
  static constexpr int KC = 256;                                     // k per stage
  static constexpr int RB = KC * (WFMT == AIO_WFMT_BF16 ? 2 : 1);    // bytes of a row
  static constexpr int RS = RB + 16;                                 // LDS row stride
  static constexpr int CPR = RB / 16;                                // 16-byte chunks per row
  static constexpr int NLD = 64 * CPR / kGBlock;                     // loads per thread
  static constexpr int BPS = KC / 32;                                // 32-k blocks per stage
  static constexpr int BPW = BPS / kGWaves;                          // blocks per wave
};

// Two bf16x8 MFMA fragments of one staged row for the wave's block of 32 k
// (the same k as vk_lo / vk_hi give for the activations).
template <int WFMT>
AIO_DEV void frag_lds(const char* rowl, int wblock, int kh, bf16x8& lo, bf16x8& hi) {
  if constexpr (WFMT == AIO_WFMT_BF16) {
    const char* p = rowl + (size_t)(wblock * 32 + 8 * kh) * 2;
    lo = __builtin_bit_cast(bf16x8, *(const uint4*)p);
    hi = __builtin_bit_cast(bf16x8, *(const uint4*)(p + 32));
  } else {
    const uint4 u = *(const uint4*)(rowl + wblock * 32 + 16 * kh);
    uint32_t w[4] = {u.x, u.y, u.z, u.w};
    uint32_t o[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      // two int8 -> two bf16 (exact: |q| <= 127 has <= 7 significant bits)
      const uint32_t src = w[i / 2];
      const int sh = (i & 1) * 16;
      const float f0 = (float)(int8_t)(src >> sh);
      const float f1 = (float)(int8_t)(src >> (sh + 8));
      o[i] = (__float_as_uint(f0) >> 16) | (__float_as_uint(f1) & 0xffff0000u);
    }
    lo = __builtin_bit_cast(bf16x8, make_uint4(o[0], o[1], o[2], o[3]));
    hi = __builtin_bit_cast(bf16x8, make_uint4(o[4], o[5], o[6], o[7]));
  }
}

// LDS of a skinny-GEMM workgroup (the eight waves' sums meet in one step there,
// and the epilogue's operands are requested before the loop.  Two steps, half
// of the waves adding to the other half's, and late requests took 0.5 to 1.0
// us more per product, at the verify's rows and positions: O 7B 12.2 -> 11.6,
// int8 11.0 -> 10.0, 1B 7.6 -> 6.9; down 22.0 -> 21.3, 18.3 -> 17.4, 10.6 ->
// 10.1): the weight stage during the product, then the waves' partial tiles [waves][T] of [32][33] (with four tiles each 16
// floats longer, so that the two rows of a pair, two tiles apart, lie in
// different halves of the banks, as they do with two tiles).
template <int T>
constexpr int kVRedTile = 32 * 33 + (T == 4 ? 16 : 0);
template <int WFMT, int T>
constexpr int vgemm_lds(int stage_rows) {
  constexpr int red = (int)sizeof(float) * kGWaves * T * kVRedTile<T>;
  return stage_rows * VStage<WFMT>::RS > red ? stage_rows * VStage<WFMT>::RS : red;
}

}  // namespace
