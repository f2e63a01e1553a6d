// Lane exchanges of the verify and prefill kernels (the step kernel does not
// use them).
#pragma once

#include "common.h"

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
