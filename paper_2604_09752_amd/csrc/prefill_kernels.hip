// Prefill: a prompt of R rows at positions pos0 .. pos0 + R - 1 in one pass
// of prompt-length matrix products (M = R), for gfx950.  This is the probe's
// single forward over its templated request: every row's K and V go to the
// cache, and the last row's logits come out.
//
// Per layer: QKV GEMM (+norm scale, RoPE, K/V append) -> pattn (causal
// flash attention; row r sees positions [0, pos0 + r]) -> O GEMM
// (+residual, x g for the next norm) -> gate/up GEMM (+norm scale, SwiGLU)
// -> down GEMM (+residual, x g).  The RMSNorm is folded into the products:
// its factor 1 / sqrt(mean(x^2) + eps) is one number per row, so a residual
// product writes x g (not yet normalised) and the sums of squares of x over
// 64-column blocks, and the consuming product scales its outputs by the
// row's factor.  Only layer 0's embedding rows go through pnorm.  The last
// row then goes through the final RMSNorm and the LM head of the verify
// path.
//
// Precision.  Activations stay fp32 between kernels.  The GEMMs run on MFMA
// (v_mfma_f32_16x16x32_bf16) with every activation split exactly into three
// bf16 terms as it is staged in LDS (a = t0 + t1 + t2), so the products keep
// fp32 accuracy (two terms leave 2^-18, which measurably loosens the cache
// rows of deeper layers).  Weights are exact in bf16 (int8 weights
// convert exactly; their fp16 per-output-channel scale applies in the
// epilogue).  Attention splits the queries and the softmax weights into
// three terms as well.
#include <math.h>
#include <algorithm>

#include "aio_internal.h"
#include "common.h"
#include "lanes.h"
#include "skinny.h"

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

AIO_DEV f32x16 mfma(const bf16x8& a, const bf16x8& b, const f32x16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// Terms of the activation split.
constexpr int kNT = 3;

// Three-term bf16 split by truncation, for fp32 bits `a`: t0 = the top 16
// bits of a, t1 those of r1 = a - t0, t2 those of r1 - t1.  Both
// subtractions are exact and r1 - t1 has at most 8 significant bits, so a =
// t0 + t1 + t2 exactly (for a normal, as every activation here is).
// Returned as fp32 bit patterns with the low 16 bits clear (the bf16 in the
// high half); branch-free.  (Rounding to nearest instead costs several
// times the operations, and in the stage loader its registers spilled.)
AIO_DEV void split3t(uint32_t a, uint32_t (&t)[kNT]) {
  t[0] = a & 0xffff0000u;
  const float r1 = __uint_as_float(a) - __uint_as_float(t[0]);
  t[1] = __float_as_uint(r1) & 0xffff0000u;
  t[2] = __float_as_uint(r1 - __uint_as_float(t[1])) & 0xffff0000u;
}

// Two floats as bf16 (round to nearest even) in one word, the first low.
AIO_DEV uint32_t pack_bf16x2(float lo, float hi) {
  return (uint32_t)f32_to_bf16(lo) | ((uint32_t)f32_to_bf16(hi) << 16);
}

// ------------------------------------------------------------- RMSNorm rows

struct PNormArgs {
  float* x;                // [R][d] residual rows (layer 0: written from the embedding)
  const uint16_t* embed;   // layer 0: embedding table, else null
  const int32_t* tokens;   // [R] (layer 0)
  const uint16_t* gain;
  float* act;              // [R][lda]: x g
  int lda;
  int d;
  float* ss;               // [R][d / 64] sums of squares of x over 64-column blocks
};

constexpr int kNormThreads = 256;

// One workgroup per row (layer 0): x from the embedding table, x g, and the
// row's sums of squares of x per 64-column block.
__global__ __launch_bounds__(kNormThreads) void k_pnorm(PNormArgs a) {
  const int r = blockIdx.x, tid = threadIdx.x;
  float* xr = a.x + (size_t)r * a.d;
  const uint16_t* emb = a.embed ? a.embed + (size_t)a.tokens[r] * a.d : nullptr;
  float* out = a.act + (size_t)r * a.lda;
  // a wave covers one 64-column block per pass (d is a multiple of 64)
  for (int e0 = 0; e0 < a.d; e0 += kNormThreads) {
    const int e = e0 + tid;
    float v = 0.f;
    if (e < a.d) {
      if (emb) {
        v = bf16_to_f32(emb[e]);
        xr[e] = v;
      } else {
        v = xr[e];
      }
      out[e] = v * bf16_to_f32(a.gain[e]);
    }
    const float sq = wave_sum_sq(v);
    if ((tid & (AIO_WAVE - 1)) == 0 && e < a.d) a.ss[(size_t)r * (a.d / 64) + e / 64] = sq;
  }
}

// --------------------------------------------------------------------- GEMM

// A workgroup of WN x WR waves computes a tile of 64 WN weight rows (2 WN
// blocks of 32, in "units" of 128 rows, the granule of the row mapping
// below) by 16 PB WR prompt rows, every term of each.  Wave (wn, wr) owns
// row blocks 2 wn ("lo") and 2 wn + 1 ("hi") and PB blocks of 16 prompt
// rows, so the two rows an epilogue combines (a RoPE pair, gate and up) sit
// in one lane.
//
// What bounds a long prompt is the card's power: in the products the clock
// falls from 2.4 to about 1.9 GHz (1.56 in a large library matrix product).
// So the products are 16 x 16 x 32 MFMAs, which draw less than 32 x 32 x 16
// ones (register-resident products of such operands: 2050 against 1780
// TFLOP/s; the 1B's 2048-row QKV product 98 -> 88 us, gate/up 248 -> 232),
// consecutive ones share an operand (2110), and the tile is as large as the
// accumulators allow (256 x 128: 27 % less LDS traffic per product than 256 x
// 64).  1B, 2048 rows, per layer: QKV 140 -> 88, O 63 -> 53, gate/up 308 ->
// 230, down 161 -> 126 us, about 1.2 PFLOP/s of MFMA work, where a library
// matrix product reaches 1.3.
//
// Weights and activations pass through LDS in stages of 32 k, double
// buffered: the next stages' global loads are in flight in registers while
// the current one is multiplied.  An LDS row is 64 bytes (32 k); its 16-byte
// chunk c is kept at place c ^ f(row / 4 mod 4), f = 0, 2, 3, 1.  Any such
// permutation spreads 16 consecutive lanes of a fragment read (one chunk of
// 16 rows) over the 64 banks; but the hardware serves a 16-byte read in
// groups that take lanes 0-3, 12-15, 20-23 and 24-27 (then 4-11, 16-19 and
// 28-31) together, and this one also keeps those apart (conflict cycles of
// the 2048-row gate/up product 14 % of its cycles -> 0; 236 -> 232 us).
// (Activations kept as the three terms between the products, split once by
// their producer: no splitting here, but half as many bytes again to stage;
// gate/up 268 -> 279 us.)
constexpr int kPfMaxKs = 8;  // most K slices of a prefill product
constexpr int kUnit = 128;   // weight rows per unit of the row mapping (block_src)
constexpr int kKT = 32;      // k per stage
constexpr int kRowB = kKT * 2;
constexpr int kMB = 4;       // blocks of 16 weight rows per wave

// Byte of chunk c of LDS row `row` (of either operand).
AIO_DEV int lds_chunk(int row, int c) {
  const int q1 = (row >> 3) & 1, q0 = (row >> 2) & 1;
  return row * kRowB + ((c ^ ((q0 ^ q1) << 1 | q1)) << 4);
}

// With KG > 1, KG such groups of waves share the tile, group kg multiplying
// the kg-th 32 k of every stage of 32 KG k; their sums meet in LDS at the
// end.  At a short prompt a workgroup has a CU to itself and a stage's time
// is its chain of waits (barrier, LDS, products), about 0.5 us whatever its
// width, so KG times the k per stage is nearly KG times the rate.
template <int WN, int WR, int PB, int NS, int KG>
struct PTile {
  static constexpr int kWN = WN, kWR = WR, kPB = PB, kKG = KG;
  static constexpr int kNS = NS;                            // stages of loads in flight
  static constexpr int GG = WN * WR * AIO_WAVE;             // threads of a group
  static constexpr int GT = KG * GG;                        // threads
  static constexpr int BM = 16 * kMB * WN;                  // weight rows
  static constexpr int BN = 16 * PB * WR;                   // prompt rows
  static constexpr int SK = KG * kKT;                       // k per stage
  static constexpr int kBand = 512 / BN;                    // rows of tiles in a band (ptile_id)
  static constexpr int UPT = BM / kUnit;                    // units per tile
  static constexpr int BCols = kNT * BN;                    // activation columns
  static constexpr int BLd = BN * (SK / 4) / GT;            // 16-byte activation loads per thread
  static constexpr int SubB = (BM + BCols) * kRowB;         // 32 k: weight rows + activation columns
  static constexpr int StageB = KG * SubB;
  static constexpr int RedB = (KG - 1) * 16 * kMB * PB * GG;  // the groups' sums
  static constexpr int Lds = 2 * StageB;
  static_assert(BN * (SK / 4) % GT == 0, "whole activation loads per thread");
  static_assert(RedB <= Lds, "the groups' sums fit the stage buffers");
};

enum PEpi { PE_QKV = 0, PE_RESID = 1, PE_SWIGLU = 2 };

struct PGemmArgs {
  const float* act;     // [R][lda] activations (split into terms on the way to LDS)
  int lda;
  int R;
  const void* w0;       // QKV: wq | SWIGLU: w_gate | RESID: the matrix
  const void* w1;       // QKV: wk | SWIGLU: w_up
  const void* w2;       // QKV: wv
  const uint16_t* s0;
  const uint16_t* s1;
  const uint16_t* s2;
  int N, K;             // QKV: N = (H + 2 Hkv) hd virtual rows; SWIGLU: F; RESID: rows
  float* out;           // QKV: q [R][H hd] | RESID: x [R][N]
  int ldo;
  float* act_out;       // SWIGLU: [R][lda_out]
  int lda_out;
  uint16_t* kc;         // QKV: cache of the layer, [Hkv][max_ctx][hd]
  uint16_t* vc;
  const float2* rope;   // [max_ctx][hd / 2] (cos, sin)
  int pos0, H, Hkv, hd, max_ctx;
  // K split over workgroups (grid.z) when the tiles alone are too few: all
  // but the last slice of a tile to arrive write their partial tile through
  // to fix; tcnt[tile] counts arrivals (low half) and writes (high half)
  int ks;
  float* fix;           // [tiles][ks, or 1 for ks == 2][values per lane][lanes of a group]
  int* tcnt;            // [tiles], zero between products
  int* err;             // the handle's status word: set if a wait gave up
  // the folded RMSNorm: QKV and SWIGLU scale output row r by 1 / sqrt(sum
  // of ss_in[r][0 .. nss) / K + eps); RESID (with act_next) writes x g_next
  // to act_next and ss_out[r][n / 64] for its columns
  const float* ss_in;
  float* ss_out;
  int nss;
  float eps;
  float* act_next;
  int lda_next;
  const uint16_t* g_next;
  // divisions of ptile_id: by the tiles of a whole band, and by the rows of
  // tiles of the last, shorter one
  UDiv by_band, by_tail;
};

// Where block `blk` (0..3) of unit `bx` reads its 32 rows: matrix index
// (0, 1, 2 = w0, w1, w2), first row in that matrix, and the number of valid
// rows (0 for a block past the end).
struct BlockSrc {
  int mat, row0, valid;
  int vrow0;  // QKV: virtual row of the block's first row
};

template <int EPI>
AIO_DEV BlockSrc block_src(const PGemmArgs& a, int bx, int blk) {
  BlockSrc b{0, 0, 0, 0};
  if constexpr (EPI == PE_QKV) {
    const int nheads = a.H + 2 * a.Hkv;
    int head, off;
    if (a.hd == 128) {
      head = bx;
      off = (blk & 1) * 64 + (blk >> 1) * 32;  // blocks 0..3 -> 0, 64, 32, 96
    } else {
      head = 2 * bx + (blk >> 1);
      off = (blk & 1) * 32;
    }
    if (head >= nheads) return b;
    const int vr = head * a.hd + off;
    const int qrows = a.H * a.hd, krows = a.Hkv * a.hd;
    b.vrow0 = vr;
    b.valid = 32;
    if (vr >= qrows + krows) { b.mat = 2; b.row0 = vr - qrows - krows; }
    else if (vr >= qrows) { b.mat = 1; b.row0 = vr - qrows; }
    else { b.mat = 0; b.row0 = vr; }
  } else if constexpr (EPI == PE_SWIGLU) {
    // blocks: gate f0, up f0, gate f0 + 32, up f0 + 32
    const int f = bx * 64 + (blk >> 1) * 32;
    b.mat = blk & 1;
    b.row0 = f;
    b.valid = f < a.N ? min(32, a.N - f) : 0;
  } else {
    const int n = bx * kUnit + blk * 32;
    b.row0 = n;
    b.valid = n < a.N ? min(32, a.N - n) : 0;
  }
  return b;
}

// One of the three weight matrices, selected arithmetically (an indexed
// local array would live in scratch memory).
AIO_DEV const char* pick_mat(const PGemmArgs& a, int mat) {
  const uint64_t b0 = (uint64_t)a.w0;
  const uint64_t d1 = (uint64_t)a.w1 - b0, d2 = (uint64_t)a.w2 - b0;
  return (const char*)(b0 + (uint64_t)(mat == 1) * d1 + (uint64_t)(mat == 2) * d2);
}

// Global loads of stage st: A_LD 16-byte weight chunks and BLd activation
// chunks per thread.
template <int WFMT, int SK, int A_LD, int BLD>
AIO_DEV void gload_stage(const char* const (&aptr)[A_LD], const float* const (&bptr)[BLD],
                         int st, uint4 (&ra)[A_LD], uint4 (&rb)[BLD]) {
  constexpr int wbytes = WFMT == AIO_WFMT_BF16 ? 2 : 1;
  const size_t ko = (size_t)st * SK;
#pragma unroll
  for (int j = 0; j < A_LD; ++j) ra[j] = *(const uint4*)(aptr[j] + ko * wbytes);
#pragma unroll
  for (int j = 0; j < BLD; ++j) rb[j] = *(const uint4*)(bptr[j] + ko);
}

// The same chunks into an LDS stage buffer: int8 widened to bf16 (exact:
// |q| <= 127); each activation value split into its three bf16 terms, one
// 8-byte store per term column (4 consecutive k).
template <int WFMT, int A_LD, int BLD>
AIO_DEV void lstore_stage(char* buf, const int (&alds)[A_LD], const int (&blds)[BLD],
                          const uint4 (&ra)[A_LD], const uint4 (&rb)[BLD]) {
  // (vector stores: a uint4 struct copy is a memcpy, which keeps the
  // register sets in scratch memory)
#pragma unroll
  for (int j = 0; j < A_LD; ++j) {
    if constexpr (WFMT == AIO_WFMT_BF16) {
      const u32x4 w = {ra[j].x, ra[j].y, ra[j].z, ra[j].w};
      *(u32x4*)(buf + alds[j]) = w;
    } else {
      const uint32_t w[4] = {ra[j].x, ra[j].y, ra[j].z, ra[j].w};
      uint32_t o[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const uint32_t sw = w[i / 2];
        const int sh = (i & 1) * 16;
        const float f0 = (float)(int8_t)(sw >> sh), f1 = (float)(int8_t)(sw >> (sh + 8));
        o[i] = (__float_as_uint(f0) >> 16) | (__float_as_uint(f1) & 0xffff0000u);
      }
      // 16 weights: chunks c and c ^ 1 of the row (c even, so the swizzled
      // places are one 32-byte pair, in one order or the other)
      const u32x4 w0 = {o[0], o[1], o[2], o[3]}, w1 = {o[4], o[5], o[6], o[7]};
      *(u32x4*)(buf + alds[j]) = w0;
      *(u32x4*)(buf + (alds[j] ^ 16)) = w1;
    }
  }
#pragma unroll
  for (int j = 0; j < BLD; ++j) {
    uint32_t t[4][kNT];
    split3t(rb[j].x, t[0]);
    split3t(rb[j].y, t[1]);
    split3t(rb[j].z, t[2]);
    split3t(rb[j].w, t[3]);
#pragma unroll
    for (int k = 0; k < kNT; ++k) {
      const u32x2 w = {(t[0][k] >> 16) | t[1][k], (t[2][k] >> 16) | t[3][k]};
      *(u32x2*)(buf + blds[j] + k * 32 * kRowB) = w;
    }
  }
}

// MFMA fragments of a stage: the wave's weight rows, and the three terms of
// one block of 16 prompt rows (LDS columns are ordered [32 prompt
// rows][term][row]).
struct AFrag {
  bf16x8 v[kMB];
};
struct BFrag {
  bf16x8 v[kNT];
};

AIO_DEV void afrag_load(AFrag& f, const char* p) {
#pragma unroll
  for (int m = 0; m < kMB; ++m) f.v[m] = as_bf16x8(*(const uint4*)(p + m * 16 * kRowB));
}
// Block p of the wave's prompt rows, b0 its first block's address.
AIO_DEV void bfrag_load(BFrag& f, const char* b0, int p) {
  b0 += ((p >> 1) * kNT * 32 + (p & 1) * 16) * kRowB;
#pragma unroll
  for (int t = 0; t < kNT; ++t) f.v[t] = as_bf16x8(*(const uint4*)(b0 + t * 32 * kRowB));
}

// Products of one block of prompt rows.  The first term's go to hi, the
// second's and third's (2^-8 of it and below, so rounding their sum in fp32
// costs nothing next to hi's own rounding) to lo.  Consecutive products
// share an operand (the rows go back and forth), which saves power.
AIO_DEV void frag_mma(const AFrag& a, const BFrag& b, f32x4 (&hi)[kMB], f32x4 (&lo)[kMB]) {
#pragma unroll
  for (int i = 0; i < kNT; ++i) {
    const int t = i == 0 ? 1 : (i == 1 ? 0 : 2);
#pragma unroll
    for (int j = 0; j < kMB; ++j) {
      const int m = i == 1 ? kMB - 1 - j : j;
      f32x4& acc = t == 0 ? hi[m] : lo[m];
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.v[m], b.v[t], acc, 0, 0, 0);
    }
  }
}

// The logical (weight tile, prompt-row tile, K slice) of this workgroup.
// Workgroups go to the 8 XCDs round-robin by linear id, and each XCD has its
// own L2; so the linear ids are renumbered to give every XCD a contiguous
// run of the logical order, in which the tiles go down bands of up to 512
// prompt rows per weight tile.  The workgroups that run at once on one
// XCD then share a few weight tiles and a few activation tiles in its L2,
// instead of each bringing its own from memory (when it was introduced:
// 2048 tokens 20.8 -> 18.9 ms).  A product split over K keeps the hardware
// order: renumbered, the workgroups of one XCD would all read one K slice,
// whose rows' equal k offsets share a few HBM channels (128 tokens 3.31 ->
// 3.49 ms).
struct PTileId {
  int bx, by, kz;
};
template <class Tl>
AIO_DEV PTileId ptile_id(const PGemmArgs& a) {
  PTileId t;
  if (gridDim.z > 1) {
    t.bx = (int)blockIdx.x;
    t.by = (int)blockIdx.y;
    t.kz = (int)blockIdx.z;
    return t;
  }
  const int nx = (int)gridDim.x, ny = (int)gridDim.y, g = nx * ny;
  const int lin = (int)(blockIdx.x + gridDim.x * blockIdx.y);
  // XCD lin % 8 holds g / 8 workgroups, the first g % 8 XCDs one more
  const int xcd = lin & 7, rem = xcd * (g / 8) + min(xcd, g & 7) + (lin >> 3);
  t.kz = 0;
  constexpr int kBand = Tl::kBand;
  const int by0 = udiv(rem, a.by_band) * kBand;
  const int in = rem - by0 * nx;
  if (ny - by0 >= kBand) {
    t.bx = in / kBand;
    t.by = by0 + in % kBand;
  } else {
    t.bx = udiv(in, a.by_tail);
    t.by = by0 + in - t.bx * (ny - by0);
  }
  return t;
}

// The four fp16 scales from s, as floats.
AIO_DEV void scale4(const uint16_t* s, float (&f)[4]) {
  const uint2 u = *(const uint2*)s;
  f[0] = fp16_to_f32((uint16_t)u.x);
  f[1] = fp16_to_f32((uint16_t)(u.x >> 16));
  f[2] = fp16_to_f32((uint16_t)u.y);
  f[3] = fp16_to_f32((uint16_t)(u.y >> 16));
}

// Epilogue of a wave: its 64 weight rows (the 32-row block slo and the one after
// it, both whole or both past the end) by its PB blocks of 16 prompt rows from row
// rw0.  Lane (c16, g) holds, for prompt row rw0 + 16 p + c16, rows 16 m + 4 g
// .. + 3 of the 64 in y[p][m].  inv: the norm factors of the wave's prompt
// rows (QKV and SWIGLU).  Everything it reads is requested before the first
// store (a load after a store that may alias it would wait its own round
// trip: 16 of them in turn in a residual tile).
template <int WFMT, int EPI, int PB>
AIO_DEV void pgemm_epi(const PGemmArgs& a, const BlockSrc& slo, int rw0, int c16, int g,
                       const float* inv, const f32x4 (&y)[PB][kMB]) {
  if (!slo.valid) return;
  if constexpr (EPI == PE_RESID) {
    float4 xv[PB][kMB];
    float gn[kMB][4], sc[kMB][4];
#pragma unroll
    for (int m = 0; m < kMB; ++m) {
      const int n = slo.row0 + 16 * m + 4 * g;  // (adjacent blocks)
      if (a.act_next) {
        const uint2 u = *(const uint2*)(a.g_next + n);
        gn[m][0] = bf16_lo(u.x);
        gn[m][1] = bf16_hi(u.x);
        gn[m][2] = bf16_lo(u.y);
        gn[m][3] = bf16_hi(u.y);
      }
      if constexpr (WFMT == AIO_WFMT_INT8) scale4(a.s0 + n, sc[m]);
    }
#pragma unroll
    for (int p = 0; p < PB; ++p) {
      const float* xrow = a.out + (size_t)min(rw0 + 16 * p + c16, a.R - 1) * a.ldo;
#pragma unroll
      for (int m = 0; m < kMB; ++m)
        xv[p][m] = *(const float4*)(xrow + slo.row0 + 16 * m + 4 * g);
    }
#pragma unroll
    for (int p = 0; p < PB; ++p) {
      const int r = rw0 + 16 * p + c16;
      const bool live = r < a.R;
      float sq = 0.f;  // the lane's sum of squares of the new x
#pragma unroll
      for (int m = 0; m < kMB; ++m) {
        const int n = slo.row0 + 16 * m + 4 * g;
        float x[4] = {xv[p][m].x, xv[p][m].y, xv[p][m].z, xv[p][m].w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float v = y[p][m][e];
          if constexpr (WFMT == AIO_WFMT_INT8) v *= sc[m][e];
          x[e] += v;
          sq = fmaf(x[e], x[e], sq);
        }
        if (live) {
          *(float4*)(a.out + (size_t)r * a.ldo + n) = make_float4(x[0], x[1], x[2], x[3]);
          if (a.act_next)
            *(float4*)(a.act_next + (size_t)r * a.lda_next + n) =
                make_float4(x[0] * gn[m][0], x[1] * gn[m][1], x[2] * gn[m][2], x[3] * gn[m][3]);
        }
      }
      // the wave's 64 columns are one block of the sums for row r, 16 of
      // them in each lane group
      if (a.act_next) {
        sq += __shfl_xor(sq, 16, AIO_WAVE);
        sq += __shfl_xor(sq, 32, AIO_WAVE);
        if (live && g == 0) a.ss_out[(size_t)r * a.nss + slo.row0 / 64] = sq;
      }
    }
  } else if constexpr (EPI == PE_SWIGLU) {
    float sg[2][4], su[2][4];
    if constexpr (WFMT == AIO_WFMT_INT8) {
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        scale4(a.s0 + slo.row0 + 16 * q + 4 * g, sg[q]);
        scale4(a.s1 + slo.row0 + 16 * q + 4 * g, su[q]);
      }
    }
#pragma unroll
    for (int p = 0; p < PB; ++p) {
      const int r = rw0 + 16 * p + c16;
      if (r >= a.R) continue;
      const float rs = inv[16 * p + c16];
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        float h[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float gt = y[p][q][e] * rs, up = y[p][q + 2][e] * rs;
          if constexpr (WFMT == AIO_WFMT_INT8) {
            gt *= sg[q][e];
            up *= su[q][e];
          }
          h[e] = gt / (1.f + expf(-gt)) * up;
        }
        *(float4*)(a.act_out + (size_t)r * a.lda_out + slo.row0 + 16 * q + 4 * g) =
            make_float4(h[0], h[1], h[2], h[3]);
      }
    }
  } else {
    // QKV: the pair (row, row + hd/2) of a head section in blocks lo and hi;
    // the lane's rows come in runs of 4, stored as one vector each (q fp32,
    // the K / V cache bf16)
    const int half = a.hd / 2, mat = slo.mat;
    float sl[2][4], sh[2][4];
    if constexpr (WFMT == AIO_WFMT_INT8) {
      const uint16_t* s = (mat == 0 ? a.s0 : (mat == 1 ? a.s1 : a.s2)) + slo.row0 + 4 * g;
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        scale4(s + 16 * q, sl[q]);
        scale4(s + half + 16 * q, sh[q]);
      }
    }
    // cos, sin of the rows' four consecutive angles (ii is a multiple of 4)
    float4 cs[PB][2][2];
    if (mat < 2) {
#pragma unroll
      for (int p = 0; p < PB; ++p)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const int ii = (slo.vrow0 + 16 * q + 4 * g) & (a.hd - 1);
          const float4* t = (const float4*)(a.rope + (size_t)(a.pos0 + min(rw0 + 16 * p + c16,
                                                                           a.R - 1)) * half + ii);
          cs[p][q][0] = t[0];
          cs[p][q][1] = t[1];
        }
    }
#pragma unroll
    for (int p = 0; p < PB; ++p) {
      const int r = rw0 + 16 * p + c16;
      if (r >= a.R) continue;
      const float rs = inv[16 * p + c16];
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const int row = slo.row0 + 16 * q + 4 * g;            // first of 4 rows in its matrix
        const int ii = (slo.vrow0 + 16 * q + 4 * g) & (a.hd - 1);  // its index in the head (< hd / 2)
        float lo[4], hi[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          lo[e] = y[p][q][e] * rs;
          hi[e] = y[p][q + 2][e] * rs;
          if constexpr (WFMT == AIO_WFMT_INT8) {
            lo[e] *= sl[q][e];
            hi[e] *= sh[q][e];
          }
        }
        if (mat < 2) {
          const float4 c0 = cs[p][q][0], c1 = cs[p][q][1];
          const float co[4] = {c0.x, c0.z, c1.x, c1.z}, si[4] = {c0.y, c0.w, c1.y, c1.w};
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float r0v = lo[e] * co[e] - hi[e] * si[e];
            const float r1v = hi[e] * co[e] + lo[e] * si[e];
            lo[e] = r0v;
            hi[e] = r1v;
          }
        }
        if (mat == 0) {
          float* qp = a.out + (size_t)r * a.ldo + row;
          *(float4*)qp = make_float4(lo[0], lo[1], lo[2], lo[3]);
          *(float4*)(qp + half) = make_float4(hi[0], hi[1], hi[2], hi[3]);
        } else {
          uint16_t* c = (mat == 1 ? a.kc : a.vc) +
                        ((size_t)(row >> hd_shift(a.hd)) * a.max_ctx + a.pos0 + r) * a.hd + ii;
          *(uint2*)c = make_uint2(pack_bf16x2(lo[0], lo[1]), pack_bf16x2(lo[2], lo[3]));
          *(uint2*)(c + half) = make_uint2(pack_bf16x2(hi[0], hi[1]), pack_bf16x2(hi[2], hi[3]));
        }
      }
    }
  }
}

// Scheduling of N MFMAs with a share of a stage's split and stores between
// them.
template <int N>
AIO_DEV void sched_mix() {
#pragma unroll
  for (int i = 0; i < N; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);  // MFMA
    __builtin_amdgcn_sched_group_barrier(0x002, 7, 0);  // VALU
    __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);  // LDS write
  }
}

template <int WFMT, int EPI, class Tl>
__global__ __launch_bounds__(Tl::GT, 2) void k_pgemm(PGemmArgs a) {
  constexpr int kGT = Tl::GT, kBM = Tl::BM, kBLd = Tl::BLd, kStageB = Tl::StageB;
  constexpr int PB = Tl::kPB;
  extern __shared__ __align__(16) char smem[];
  const int tid = threadIdx.x, lane = tid & (AIO_WAVE - 1), wid = tid / AIO_WAVE;
  constexpr int KG = Tl::kKG, kGG = Tl::GG;
  const int kg = wid / (Tl::kWN * Tl::kWR);
  const int wn = wid % Tl::kWN, wr = wid / Tl::kWN % Tl::kWR;
  const int c16 = lane & 15, g = lane >> 4;  // row of a fragment, lane group
  const PTileId tid3 = ptile_id<Tl>(a);
  const int bx = tid3.bx, r0 = tid3.by * Tl::BN;
  constexpr int wbytes = WFMT == AIO_WFMT_BF16 ? 2 : 1;

  // Staging assignments.  A: row ra of the tile (block ra / 32), 16-byte
  // chunk ca of 32 k (bf16: 4 chunks of 8 weights; int8: 2 chunks of 16
  // weights, widened to 32 bytes in LDS) of the stage's KG.  B: prompt row r0
  // + p, 8 chunks of 4 fp32 per 32 k; its terms t go to the LDS activation
  // columns (p / 32 kNT + t) 32 + p % 32.
  constexpr int A_CPR = WFMT == AIO_WFMT_BF16 ? 4 : 2;
  constexpr int A_LD = kBM * A_CPR * KG / kGT;
  const char* aptr[A_LD];
  int alds[A_LD];
#pragma unroll
  for (int j = 0; j < A_LD; ++j) {
    const int f = j * kGT + tid, ra = f / (A_CPR * KG), cs = f % (A_CPR * KG);
    const int sub = cs / A_CPR, ca = cs % A_CPR;
    const int blk = ra >> 5;  // block of the tile: unit UPT bx + blk / 4, block blk % 4 of it
    const BlockSrc s = block_src<EPI>(a, Tl::UPT * bx + (blk >> 2), blk & 3);
    int row = s.row0 + ((ra & 31) < s.valid ? (ra & 31) : 0);
    if (s.valid == 0) row = 0;  // a block past the end reads row 0 of w0 (discarded)
    const char* w = s.valid ? pick_mat(a, s.mat) : (const char*)a.w0;
    aptr[j] = w + ((size_t)row * a.K + (size_t)cs * (16 / wbytes)) * wbytes;
    alds[j] = sub * Tl::SubB + lds_chunk(ra, ca * (2 / wbytes));
  }
  const float* bptr[kBLd];
  int blds[kBLd];
#pragma unroll
  for (int j = 0; j < kBLd; ++j) {
    const int f = j * kGT + tid, p = f / (8 * KG), cs = f % (8 * KG), c = cs % 8;
    const int row = r0 + p;
    bptr[j] = a.act + (size_t)(row < a.R ? row : a.R - 1) * a.lda + cs * 4;
    blds[j] = cs / 8 * Tl::SubB + lds_chunk(kBM + (p / 32) * kNT * 32 + (p % 32), c / 2) + (c & 1) * 8;
  }
  // fragment reads: lane (c16, g) takes chunk g of row c16 of a block
  const int aoff = kg * Tl::SubB + lds_chunk(wn * 16 * kMB + c16, g);
  const int boff = kg * Tl::SubB + lds_chunk(kBM + wr * (PB / 2) * kNT * 32 + c16, g);
  f32x4 hi[PB][kMB], lo[PB][kMB];
#pragma unroll
  for (int p = 0; p < PB; ++p)
#pragma unroll
    for (int m = 0; m < kMB; ++m) hi[p][m] = lo[p][m] = f32x4{0.f, 0.f, 0.f, 0.f};

  // this workgroup's stages [sA, sB) of K (all of them unless K is split).
  // NS register sets keep NS stages' loads in flight (a stage's loads take a
  // memory round trip, its products a fraction of one): stage sA + i goes
  // through set i mod NS; loads past sB re-read the last stage and are not
  // used.
  constexpr int NS = Tl::kNS;
  const int nst = a.K / Tl::SK, kz = tid3.kz;
  const int ksh = __builtin_ctz(a.ks);  // a power of two
  const int sA = (kz * nst) >> ksh, sB = ((kz + 1) * nst) >> ksh, sL = sB - 1;
  uint4 ra[NS][A_LD], rb[NS][kBLd];
#pragma unroll
  for (int i = 0; i < NS; ++i) gload_stage<WFMT, Tl::SK>(aptr, bptr, min(sA + i, sL), ra[i], rb[i]);
  // the folded norm's row factors of the tile's prompt rows, GT / BN threads
  // per row (their loads queue behind the first stages'; the barrier below
  // publishes them)
  __shared__ float inv_rows[Tl::BN];
  if constexpr (EPI != PE_RESID) {
    constexpr int TPR = kGT / Tl::BN;
    const int j = tid / TPR, part = tid % TPR;
    const float* ssr = a.ss_in + (size_t)min(r0 + j, a.R - 1) * a.nss;
    float s0 = 0.f, s1 = 0.f, s2 = 0.f, s3 = 0.f;
    int c = part;
    for (; c + 3 * TPR < a.nss; c += 4 * TPR) {
      s0 += ssr[c];
      s1 += ssr[c + TPR];
      s2 += ssr[c + 2 * TPR];
      s3 += ssr[c + 3 * TPR];
    }
    for (; c < a.nss; c += TPR) s0 += ssr[c];
    float sum = (s0 + s1) + (s2 + s3);
#pragma unroll
    for (int off = TPR / 2; off >= 1; off >>= 1) sum += __shfl_xor(sum, off, AIO_WAVE);
    if (part == 0) inv_rows[j] = rsqrtf(sum / (float)a.K + a.eps);
  }
  lstore_stage<WFMT>(smem, alds, blds, ra[0], rb[0]);
  __syncthreads();
  gload_stage<WFMT, Tl::SK>(aptr, bptr, min(sA + NS, sL), ra[0], rb[0]);
  // Stage i (of sA ..): its weight fragments fa and its first block of
  // prompt rows f0 are in registers.  During the first half of the blocks'
  // products the other blocks are read, and stage i + 1 is split and stored
  // to the other LDS buffer.  Then, after the barrier, its register set is
  // refilled with stage i + 1 + NS and the next stage's first fragments are
  // requested, ahead of the second half's products, which cover their
  // latency.  The scheduling barriers keep these parts in this order:
  // without them the compiler moved a set's loads to just before their use,
  // and nothing was in flight.
  AFrag fa, na;
  BFrag f0, fb[PB];
  afrag_load(fa, smem + aoff);
  bfrag_load(f0, smem + boff, 0);
  auto step = [&](int i, uint4 (&RA)[A_LD], uint4 (&RB)[kBLd]) {
    const char* cur = smem + (i & 1) * kStageB;
    char* nxt = smem + ((i + 1) & 1) * kStageB;
#pragma unroll
    for (int p = 1; p < PB; ++p) bfrag_load(fb[p], cur + boff, p);
    __builtin_amdgcn_sched_barrier(0);
    frag_mma(fa, f0, hi[0], lo[0]);
#pragma unroll
    for (int p = 1; p < PB / 2; ++p) frag_mma(fa, fb[p], hi[p], lo[p]);
    lstore_stage<WFMT>(nxt, alds, blds, RA, RB);
    sched_mix<kMB * kNT * PB / 4>();
    __builtin_amdgcn_sched_barrier(0);
    __syncthreads();
    gload_stage<WFMT, Tl::SK>(aptr, bptr, min(sA + i + 1 + NS, sL), RA, RB);
    afrag_load(na, nxt + aoff);
    bfrag_load(f0, nxt + boff, 0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int p = PB / 2; p < PB; ++p) frag_mma(fa, fb[p], hi[p], lo[p]);
    __builtin_amdgcn_sched_barrier(0);
    fa = na;
  };
  const int ns = sB - sA;
  int i = 0;
  for (; i + NS < ns; i += NS) {
#pragma unroll
    for (int u = 0; u < NS; ++u) step(i + u, ra[(u + 1) % NS], rb[(u + 1) % NS]);
  }
  // the last 1 .. NS stages
#pragma unroll
  for (int u = 0; u < NS - 1; ++u) {
    if (i + 1 >= ns) break;
    step(i, ra[(u + 1) % NS], rb[(u + 1) % NS]);
    ++i;
  }
  {
    const char* cur = smem + (i & 1) * kStageB;
    frag_mma(fa, f0, hi[0], lo[0]);
#pragma unroll
    for (int p = 1; p < PB; ++p) {
      bfrag_load(fb[p], cur + boff, p);
      frag_mma(fa, fb[p], hi[p], lo[p]);
    }
  }

  // the tile's sums over the three terms
#pragma unroll
  for (int p = 0; p < PB; ++p)
#pragma unroll
    for (int m = 0; m < kMB; ++m) hi[p][m] += lo[p][m];
  constexpr int PV = 4 * kMB;  // values of a lane per block of prompt rows
  const int gtid = tid % kGG;  // thread of its group
  if constexpr (KG > 1) {
    // the groups' sums, added in group order by group 0
    __syncthreads();
    float* red = (float*)smem + gtid;
    if (kg > 0) {
#pragma unroll
      for (int p = 0; p < PB; ++p)
#pragma unroll
        for (int v = 0; v < PV; ++v)
          red[((kg - 1) * PB * PV + p * PV + v) * kGG] = hi[p][v / 4][v % 4];
    }
    __syncthreads();
    if (kg == 0) {
#pragma unroll
      for (int k = 1; k < KG; ++k)
#pragma unroll
        for (int p = 0; p < PB; ++p)
#pragma unroll
          for (int v = 0; v < PV; ++v)
            hi[p][v / 4][v % 4] += red[((k - 1) * PB * PV + p * PV + v) * kGG];
    }
  }
  if (a.ks > 1) {
    // K split.  Each slice takes a ticket when its product is done (the low
    // half of the tile's counter).  All but the last to arrive write their
    // partial tile through to memory and count it written (the high half);
    // the last keeps its own in registers, waits for the others' writes, and
    // adds all of them in slice order, so the sum is the same whatever the
    // arrival order.  The others hold their tickets, so they are running, their
    // first waves past their products: the wait is short and never for a
    // workgroup that has not started.  It relies on the counter being zero at
    // entry, and is bounded in case it is not (the step kernel's limit; the
    // status word then says that results are invalid).  Partials are element-major: every store
    // and load instruction of a wave covers 256 contiguous bytes.  Lanes of
    // prompt rows past R move nothing: at a short prompt most of the tile's
    // rows are.  Two slices need one slot per tile, more need one each.
    const int tile = tid3.by * (int)gridDim.x + bx;
    const size_t slot = (size_t)PV * PB * kGG;  // floats of one partial tile
    const int nslot = a.ks == 2 ? 1 : a.ks;
    float* fix = a.fix + (size_t)tile * nslot * slot + gtid;
    __shared__ int ticket_s;
    if (tid == 0) ticket_s = atomic_add_agent(a.tcnt + tile, 1) & 0xffff;
    __syncthreads();
    if (ticket_s < a.ks - 1) {
      float* mine = fix + (a.ks == 2 ? 0 : kz) * slot;
      if (kg == 0) {
#pragma unroll
        for (int p = 0; p < PB; ++p)
          if (r0 + (wr * PB + p) * 16 + c16 < a.R) {
#pragma unroll
            for (int v = 0; v < PV; ++v) st_agent(mine + (p * PV + v) * kGG, hi[p][v / 4][v % 4]);
          }
      }
      __builtin_amdgcn_s_waitcnt(0);
      __syncthreads();
      if (tid == 0) atomic_add_agent(a.tcnt + tile, 0x10000);
      return;
    }
    if (tid == 0) {
      unsigned spins = 0;
      while ((atomic_load_agent(a.tcnt + tile) >> 16) != a.ks - 1) {
        __builtin_amdgcn_s_sleep(1);
        if ((++spins & 63u) == 0 && (spins > kSpinLimit || atomic_load_agent(a.err))) {
          atomic_store_agent(a.err, 1);
          break;
        }
      }
      atomic_store_agent(a.tcnt + tile, 0);  // ready for the next product
    }
    __syncthreads();
    if (kg > 0) return;
#pragma unroll
    for (int p = 0; p < PB; ++p) {
      if (r0 + (wr * PB + p) * 16 + c16 >= a.R) continue;
      float sum[PV];
      if (a.ks == 2) {  // (the two slices' sum does not depend on their order)
#pragma unroll
        for (int v = 0; v < PV; ++v) sum[v] = ld_agent(fix + (p * PV + v) * kGG);
#pragma unroll
        for (int v = 0; v < PV; ++v) sum[v] += hi[p][v / 4][v % 4];
      } else {
        // four slices' values are requested together (a round trip each)
#pragma unroll
        for (int v = 0; v < PV; ++v) sum[v] = 0.f;
        for (int k0 = 0; k0 < a.ks; k0 += 4) {
          float pv[4][PV];
#pragma unroll
          for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int v = 0; v < PV; ++v)
              pv[k][v] = ld_agent(fix + (k0 + k) * slot + (p * PV + v) * kGG);
#pragma unroll
          for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int v = 0; v < PV; ++v) sum[v] += k0 + k == kz ? hi[p][v / 4][v % 4] : pv[k][v];
        }
      }
#pragma unroll
      for (int v = 0; v < PV; ++v) hi[p][v / 4][v % 4] = sum[v];
    }
  }
  if (kg > 0) return;

  const int blk = 2 * wn;  // the wave's first block of 32 weight rows in the tile
  const BlockSrc slo = block_src<EPI>(a, Tl::UPT * bx + (blk >> 2), blk & 3);
  pgemm_epi<WFMT, EPI, PB>(a, slo, r0 + wr * PB * 16, c16, g,
                           EPI == PE_RESID ? nullptr : inv_rows + wr * PB * 16, hi);
}

// ------------------------------------------------------ causal attention

struct PAttnArgs {
  const float* q;       // [R][H hd] rotated queries
  int ldq;
  const uint16_t* kc;   // [Hkv][max_ctx][hd]
  const uint16_t* vc;
  float* act;           // [R][lda]: the output, at columns h hd ..
  int lda;
  int R, pos0, H, Hkv, max_ctx;
  float scale_log2;     // log2(e) / sqrt(hd)
  UDiv by_g, by_hpx;    // divisions by H / Hkv and by H / 8
};

constexpr int kAW = 4;  // waves per workgroup: they split the key blocks

template <int HD>
struct AttnLds {
  static constexpr int QROW = HD * 2 + 16;        // bytes per query row of one term
  static constexpr int QBYTES = 3 * 32 * QROW;     // three terms of 32 queries
  static constexpr int VROW = HD * 2 + 16;         // bytes per key row of a value tile
  static constexpr int VBYTES = 32 * VROW;         // one wave's value tile (32 keys)
  static constexpr int OROW = HD + 1;              // floats per combined output row (padded)
  static constexpr int OBYTES = 2 * 32 * OROW * 4 + 2 * 2 * 32 * 4;  // combine: 2 waves' O, m, l
  static constexpr int TAIL = kAW * VBYTES > OBYTES ? kAW * VBYTES : OBYTES;
  static constexpr int BYTES = QBYTES + TAIL;
};

// One workgroup per (32 query rows, head): wave w takes key blocks w, w + 4,
// ... of 32 keys.  Per block: S^T = K Q^T on MFMA (A = 32 key rows from the
// cache, B = the queries' three bf16 terms from LDS), the online softmax per
// query (one query per lane pair), then O^T += V^T P^T (B = the softmax
// weights' three terms straight from the score tile's registers: register v
// = 8 c2 + e of lane half kh holds key 8 (v / 4) + 4 kh + v % 4; A = the value
// rows of those keys, staged in LDS row by row and read with the transposing
// LDS read).  The waves' (max, sum, output) states are merged through LDS at
// the end.
// Vector instructions bound it (MFMAs do not hide them): the value tile
// gathered by 16-bit reads, 64 and 32 packs per block, the output rescaled
// and the mask applied at every block took 79 us at 2048 rows of the 1B (16
// heads); the transposing reads, and both of the others only where needed,
// 69.5 (7B, 1000 rows: 53 -> 44).  The first block requested ahead of the
// query split, and no merge for a single block: 23 rows 12.3 -> 5.2 us.
template <int HD>
__global__ __launch_bounds__(kAW * AIO_WAVE, 2) void k_pattn(PAttnArgs a) {
  using Lds = AttnLds<HD>;
  extern __shared__ __align__(16) char smem[];
  char* qs = smem;                  // [3][32][QROW]
  char* tail = smem + Lds::QBYTES;  // per wave: value tile; at the end: the merge
  const int tid = threadIdx.x, lane = tid & (AIO_WAVE - 1), wid = tid / AIO_WAVE;
  const int rl = lane & 31, kh = lane >> 5;
  // Query tiles in reverse: a causal tile's work grows with its position,
  // and workgroups start in index order, so the longest start first.  With
  // a multiple of 8 heads, each XCD (workgroups go to the 8 XCDs
  // round-robin by linear id) takes H / 8 consecutive heads, whose keys and
  // values (shared through G) then stay in its own L2 instead of being
  // read by all eight; its heads' tiles interleave, longest first.
  int qt = (int)blockIdx.x, h = (int)blockIdx.y;
  if (gridDim.y % 8 == 0) {
    const int lin = (int)(blockIdx.x + gridDim.x * blockIdx.y);
    const int hpx = (int)gridDim.y / 8, j = lin / 8;
    qt = udiv(j, a.by_hpx);
    h = (lin % 8) * hpx + j - qt * hpx;
  }
  const int q0 = ((int)gridDim.x - 1 - qt) * 32;
  const int kvh = udiv(h, a.by_g);
  const int rows = min(32, a.R - q0);
  const int n_keys = a.pos0 + q0 + rows;  // keys the block's last row sees
  const int nkb = (n_keys + 31) / 32;

  // queries, scaled to log2 units and split into three bf16 terms, four
  // consecutive dims per thread and pass
  float4 qv[32 * HD / 4 / (kAW * AIO_WAVE)];
#pragma unroll
  for (int i = 0; i < 32 * HD / 4 / (kAW * AIO_WAVE); ++i) {
    const int e = i * kAW * AIO_WAVE + tid, qq = e / (HD / 4), dim = e % (HD / 4) * 4;
    qv[i] = *(const float4*)(a.q + (size_t)(q0 + min(qq, rows - 1)) * a.ldq + (size_t)h * HD + dim);
  }
  // (the first block's keys and values follow the queries: loads complete in
  // order, so waiting for the queries leaves them in flight)
  const uint16_t* kbase = a.kc + (size_t)kvh * a.max_ctx * HD;
  const uint16_t* vbase = a.vc + (size_t)kvh * a.max_ctx * HD;
  // Block kb's key fragments (A operand: key row rl, dims 16 c + 8 kh ..) and
  // value chunks (16 bytes of 8 dims, row-major) into registers; keys past
  // n_keys read key 0.  The next block of the wave is requested while the
  // current one is multiplied.
  constexpr int NKC = HD / 16, VCH = 32 * HD / 8, NVL = VCH / AIO_WAVE;
  uint4 kr[NKC], vr[NVL];
  auto load_block = [&](int kb) {
    const int j0 = kb * 32;
    const int key = j0 + rl < n_keys ? j0 + rl : 0;
    const uint16_t* krow = kbase + (size_t)key * HD;
#pragma unroll
    for (int c = 0; c < NKC; ++c) kr[c] = *(const uint4*)(krow + c * 16 + 8 * kh);
#pragma unroll
    for (int it = 0; it < NVL; ++it) {
      const int f = it * AIO_WAVE + lane, kk = f / (HD / 8), d0 = (f % (HD / 8)) * 8;
      const int vkey = j0 + kk < n_keys ? j0 + kk : 0;
      vr[it] = *(const uint4*)(vbase + (size_t)vkey * HD + d0);
    }
  };
  load_block(min(wid, nkb - 1));
#pragma unroll
  for (int i = 0; i < 32 * HD / 4 / (kAW * AIO_WAVE); ++i) {
    const int e = i * kAW * AIO_WAVE + tid, qq = e / (HD / 4), dim = e % (HD / 4) * 4;
    uint32_t t[4][kNT];
    split3t(__float_as_uint(qv[i].x * a.scale_log2), t[0]);
    split3t(__float_as_uint(qv[i].y * a.scale_log2), t[1]);
    split3t(__float_as_uint(qv[i].z * a.scale_log2), t[2]);
    split3t(__float_as_uint(qv[i].w * a.scale_log2), t[3]);
#pragma unroll
    for (int k = 0; k < kNT; ++k) {
      const u32x2 w = {(t[0][k] >> 16) | t[1][k], (t[2][k] >> 16) | t[3][k]};
      *(u32x2*)(qs + (k * 32 + qq) * Lds::QROW + dim * 2) = w;
    }
  }
  __syncthreads();

  // this lane's query: row q0 + rl sees keys [0, lim]
  const int lim = a.pos0 + q0 + (rl < rows ? rl : rows - 1);
  char* vt = tail + wid * Lds::VBYTES;
  constexpr int NHB = HD / 32;
  f32x16 o[NHB];
#pragma unroll
  for (int hb = 0; hb < NHB; ++hb)
#pragma unroll
    for (int i = 0; i < 16; ++i) o[hb][i] = 0.f;
  float m = -INFINITY, lsum = 0.f;

  // transposing reads of the value tile: this lane's address serves key e of
  // four and dims 4 q .. + 3 of its group's 16
  const char* vtr = vt + (4 * kh + (lane & 15) / 4) * Lds::VROW +
                    ((lane >> 4 & 1) * 16 + (lane & 3) * 4) * 2;

  for (int kb = wid; kb < nkb; kb += kAW) {
    const int j0 = kb * 32;
    // value rows -> LDS, row by row (a vector store: a uint4 struct copy
    // would go through scratch memory)
#pragma unroll
    for (int it = 0; it < NVL; ++it) {
      const int f = it * AIO_WAVE + lane, kk = f / (HD / 8), d0 = (f % (HD / 8)) * 8;
      const u32x4 wv = {vr[it].x, vr[it].y, vr[it].z, vr[it].w};
      *(u32x4*)(vt + kk * Lds::VROW + d0 * 2) = wv;
    }
    // scores: S^T[key i][query j] over the HD dims, three query terms
    f32x16 s;
#pragma unroll
    for (int i = 0; i < 16; ++i) s[i] = 0.f;
#pragma unroll
    for (int c = 0; c < NKC; ++c) {
      const bf16x8 ak = as_bf16x8(kr[c]);
#pragma unroll
      for (int t = 0; t < 3; ++t) {
        const bf16x8 bq =
            as_bf16x8(*(const uint4*)(qs + (t * 32 + rl) * Lds::QROW + (c * 16 + 8 * kh) * 2));
        s = mfma(ak, bq, s);
      }
    }
    // the wave's next block (the last one re-reads itself: no branch, so
    // the fragments stay in registers)
    load_block(kb + kAW < nkb ? kb + kAW : kb);
    // causal mask and online softmax for this lane's query (column rl)
    // (only a block with keys past the first row's own needs the mask)
    if (j0 + 31 > a.pos0 + q0) {
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int key = j0 + 8 * (v / 4) + 4 * kh + (v % 4);
        if (key > lim) s[v] = -INFINITY;
      }
    }
    float mx = s[0];
#pragma unroll
    for (int v = 1; v < 16; ++v) mx = fmaxf(mx, s[v]);
    mx = fmaxf(mx, __shfl_xor(mx, 32, AIO_WAVE));
    const float mnew = fmaxf(m, mx);
    // (the hardware exp2: every argument is <= 0, and exp2(-inf) = 0; a block
    // that raises no query's maximum, as most after the first few, leaves the
    // output as it is: c would be 1)
    const bool raised = __any(mnew > m);
    const float c = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m - mnew);
    const float mref = mnew == -INFINITY ? 0.f : mnew;
    float p[16];
    float ps = 0.f;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      p[v] = __builtin_amdgcn_exp2f(s[v] - mref);
      ps += p[v];
    }
    if (raised) {
      lsum *= c;
#pragma unroll
      for (int hb = 0; hb < NHB; ++hb)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[hb][i] *= c;
    }
    lsum += ps;
    m = mnew;
    wave_lds_sync();  // the value tile is in LDS
    // O^T += V^T P^T, two chunks of 16 keys, three terms of the weights
#pragma unroll
    for (int c2 = 0; c2 < 2; ++c2) {
      // the weights split by truncation: t0 = the top 16 bits of p, t1 those
      // of p - t0, t2 = p - t0 - t1 (exact: 8 significant bits each)
      uint32_t tt[3][8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const uint32_t u0 = __float_as_uint(p[8 * c2 + e]) & 0xffff0000u;
        const float r1 = p[8 * c2 + e] - __uint_as_float(u0);
        const uint32_t u1 = __float_as_uint(r1) & 0xffff0000u;
        tt[0][e] = u0;
        tt[1][e] = u1;
        tt[2][e] = __float_as_uint(r1 - __uint_as_float(u1));
      }
      bf16x8 bp[3];
#pragma unroll
      for (int t = 0; t < 3; ++t)
        bp[t] = as_bf16x8(make_uint4((tt[t][0] >> 16) | (tt[t][1] & 0xffff0000u),
                                     (tt[t][2] >> 16) | (tt[t][3] & 0xffff0000u),
                                     (tt[t][4] >> 16) | (tt[t][5] & 0xffff0000u),
                                     (tt[t][6] >> 16) | (tt[t][7] & 0xffff0000u)));
#pragma unroll
      for (int hb = 0; hb < NHB; ++hb) {
        // V^T fragment: dimension hb 32 + rl at this lane's eight keys
        const uint2 v0 = lds_read_tr16(vtr + 16 * c2 * Lds::VROW + hb * 64);
        const uint2 v1 = lds_read_tr16(vtr + (16 * c2 + 8) * Lds::VROW + hb * 64);
        const bf16x8 av = as_bf16x8(make_uint4(v0.x, v0.y, v1.x, v1.y));
#pragma unroll
        for (int t = 0; t < 3; ++t) o[hb] = mfma(av, bp[t], o[hb]);
      }
    }
    wave_lds_sync();  // every read of the value tile is done before the next block's writes
  }
  lsum += __shfl_xor(lsum, 32, AIO_WAVE);

  // merge the waves' states: 2, 3 into 0, 1, then 1 into 0
  __syncthreads();
  float* om = (float*)tail;                 // [2][32][OROW] outputs (rows padded: no bank conflicts)
  float* mm = om + 2 * 32 * Lds::OROW;      // [2][32] max
  float* ll = mm + 2 * 32;                  // [2][32] sum
  auto put = [&](int slot) {
#pragma unroll
    for (int hb = 0; hb < NHB; ++hb)
#pragma unroll
      for (int v = 0; v < 16; ++v)
        om[((size_t)slot * 32 + rl) * Lds::OROW + hb * 32 + 8 * (v / 4) + 4 * kh + (v % 4)] = o[hb][v];
    if (kh == 0) {
      mm[slot * 32 + rl] = m;
      ll[slot * 32 + rl] = lsum;
    }
  };
  auto take = [&](int slot) {
    const float m2 = mm[slot * 32 + rl], l2 = ll[slot * 32 + rl];
    const float M = fmaxf(m, m2);
    const float c1 = m == -INFINITY ? 0.f : exp2f(m - M);
    const float c2 = m2 == -INFINITY ? 0.f : exp2f(m2 - M);
#pragma unroll
    for (int hb = 0; hb < NHB; ++hb)
#pragma unroll
      for (int v = 0; v < 16; ++v)
        o[hb][v] = o[hb][v] * c1 +
                   om[((size_t)slot * 32 + rl) * Lds::OROW + hb * 32 + 8 * (v / 4) + 4 * kh + (v % 4)] * c2;
    lsum = lsum * c1 + l2 * c2;
    m = M;
  };
  if (nkb > 1) {  // (one block: it was wave 0's)
    if (wid >= 2) put(wid - 2);
    __syncthreads();
    if (wid < 2) take(wid);
    __syncthreads();
    if (wid == 1) put(0);
    __syncthreads();
  }
  if (wid != 0) return;
  if (nkb > 1) take(0);
  if (rl >= rows) return;
  const int r = q0 + rl;
  const float inv = 1.f / lsum;
  float* out = a.act + (size_t)r * a.lda + (size_t)h * HD;
  // the lane's dimensions come in runs of 4: one float4 store each
#pragma unroll
  for (int hb = 0; hb < NHB; ++hb)
#pragma unroll
    for (int g = 0; g < 4; ++g)
      *(float4*)(out + hb * 32 + 8 * g + 4 * kh) =
          make_float4(o[hb][4 * g] * inv, o[hb][4 * g + 1] * inv, o[hb][4 * g + 2] * inv,
                      o[hb][4 * g + 3] * inv);
}

// ------------------------------------------- products of a few prompt rows

// Products of at most kSkRows prompt rows.  The tiles of k_pgemm leave such a
// product to few workgroups (the 1B's 128 or 176), and a CU streams no more than
// about 30 bytes per ns of weights from memory, so they should come in equal shares
// through all of them: a workgroup owns np row pairs (k_spair) or 64 rows and a K
// slice (k_sresid) and passes its weights through LDS in stages of 256 k.  Wave w
// multiplies 32-k block w of every stage by all prompt rows: lane rl of a half
// wave reads prompt row rl's 16 activations of the block from memory and splits
// them, and the three terms are three products into 32x32 tiles, hi (first terms)
// and lo.  The waves' tiles meet in LDS.  What bounds it is the bytes through each
// CU, weights and activations together some 45 per ns (every workgroup reads the
// activations of its K slice, which come from a cache).  23 rows of the 1B, in us,
// Short tiles of k_pgemm before and now: QKV 19.5 -> 12.6, O 15.7 -> 10.4, gate/up
// 20.0 -> 18.0, down 21.5 -> 13.7.
constexpr int kSkRows = 32;

struct SkArgs {
  PGemmArgs g;
  int pairs, np;        // k_spair: row pairs of the product and per workgroup
  UDiv by_np, by_nst;   // k_spair: divisions by np and by the K stages of a slice
};
constexpr int kSkPairKs = 4;  // most K slices of a k_spair product

// The three bf16 terms of 8 activations.
AIO_DEV void split_frag(const uint4& a, const uint4& b, bf16x8 (&f)[kNT]) {
  const uint32_t x[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
  uint32_t t[8][kNT];
#pragma unroll
  for (int i = 0; i < 8; ++i) split3t(x[i], t[i]);
#pragma unroll
  for (int k = 0; k < kNT; ++k) {
    uint32_t w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = (t[2 * i][k] >> 16) | t[2 * i + 1][k];
    f[k] = as_bf16x8(make_uint4(w[0], w[1], w[2], w[3]));
  }
}

// The streaming loop of both kernels: rows lrow[] of K weights, k blocks [kbA,
// kbB), stages rotated by rot, NS of them in flight in registers.
template <int WFMT, int NLD, int NS>
struct SkStream {
  using St = VStage<WFMT>;
  static_assert(St::BPW == 1, "one block per wave and stage");
  const char* lrow[NLD];
  int lds_off[NLD];
  int lchunk, wid, rl, kh, kbA, kbB, nst, rot, kend;
  const float* actp;  // prompt row rl (the last one past the rows: not stored)

  AIO_DEV int kb0(int st) const {  // first block of stage st (st < 2 nst)
    const int q = st + rot;
    return kbA + (q >= nst ? q - nst : q) * St::BPS;
  }
  AIO_DEV void load(uint4 (&R)[NLD], uint4 (&A)[4], int st) const {
    constexpr int wbytes = WFMT == AIO_WFMT_BF16 ? 2 : 1;
    const int b0 = kb0(min(st, nst - 1));
    const int off = min(b0 * 32 * wbytes + lchunk * 16, kend);
#pragma unroll
    for (int j = 0; j < NLD; ++j) R[j] = ldg_nt(lrow[j] + off);
    const int block = min(b0 + wid, kbB - 1) * 32;
    const float* lo = actp + vk_lo<WFMT>(block, kh);
    const float* hi = actp + vk_hi<WFMT>(block, kh);
    A[0] = ldg(lo);
    A[1] = ldg(lo + 4);
    A[2] = ldg(hi);
    A[3] = ldg(hi + 4);
  }
  AIO_DEV void stage(char* smem, const uint4 (&R)[NLD]) const {
    __syncthreads();  // every wave is done with the previous stage
#pragma unroll
    for (int j = 0; j < NLD; ++j) {
      const u32x4 w = {R[j].x, R[j].y, R[j].z, R[j].w};
      *(u32x4*)(smem + lds_off[j]) = w;
    }
    __syncthreads();
  }
  // (a block past the end multiplies zeros)
  AIO_DEV void product(const char* smem, const uint4 (&A)[4], int st, f32x16 (&hi)[2],
                       f32x16 (&lo)[2]) const {
    const bool live = kb0(st) + wid < kbB;
    uint4 z[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
      z[i] = make_uint4(live ? A[i].x : 0u, live ? A[i].y : 0u, live ? A[i].z : 0u,
                        live ? A[i].w : 0u);
    bf16x8 wa[2], wb[2], ba[kNT], bb[kNT];
#pragma unroll
    for (int t = 0; t < 2; ++t)
      frag_lds<WFMT>(smem + (t * 32 + rl) * St::RS, wid, kh, wa[t], wb[t]);
    split_frag(z[0], z[1], ba);
    split_frag(z[2], z[3], bb);
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      hi[t] = mfma(wa[t], ba[0], hi[t]);
      lo[t] = mfma(wa[t], ba[1], lo[t]);
      hi[t] = mfma(wb[t], bb[0], hi[t]);
      lo[t] = mfma(wa[t], ba[2], lo[t]);
      lo[t] = mfma(wb[t], bb[1], lo[t]);
      lo[t] = mfma(wb[t], bb[2], lo[t]);
    }
  }
  // All stages; then the wave's tiles to LDS (the caller's barrier follows).
  // `between` runs once the first stages are requested.
  template <class F>
  AIO_DEV void run(char* smem, int rows, F&& between) const {
    f32x16 hi[2], lo[2];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int i = 0; i < 16; ++i) hi[t][i] = lo[t][i] = 0.f;
    uint4 R[NS][NLD], A[NS][4];
#pragma unroll
    for (int i = 0; i < NS; ++i) load(R[i], A[i], i);
    between();
    // a stage's register set is refilled with the stage NS ahead: the weights
    // and activations of NS stages stay in flight through its product
    int st = 0;
    for (; st + NS < nst; st += NS) {
#pragma unroll
      for (int i = 0; i < NS; ++i) {
        stage(smem, R[i]);
        uint4 a[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) a[q] = make_uint4(A[i][q].x, A[i][q].y, A[i][q].z, A[i][q].w);
        __builtin_amdgcn_sched_barrier(0);
        load(R[i], A[i], st + i + NS);
        __builtin_amdgcn_sched_barrier(0);
        product(smem, a, st + i, hi, lo);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
#pragma unroll
    for (int i = 0; i < NS; ++i) {
      if (st + i >= nst) break;
      stage(smem, R[i]);
      product(smem, A[i], st + i, hi, lo);
    }
    __syncthreads();  // the stage buffer becomes the partial-tile buffer
    float* red = (float*)smem;
    if (rl < rows) {
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v)
          red[(wid * 2 + t) * kVRedTile<2> + (8 * (v / 4) + 4 * kh + (v % 4)) * 33 + rl] =
              hi[t][v] + lo[t][v];
    }
  }
};

// Prompt row r of row i of tile t: the waves' sums.
AIO_DEV float sk_sum(const float* red, int t, int i, int r) {
  float s = 0.f;
#pragma unroll
  for (int w = 0; w < kGWaves; ++w) s += red[(w * 2 + t) * kVRedTile<2> + i * 33 + r];
  return s;
}

// QKV and gate/up.  Pairs and their layout as in the tile products' epilogue:
// rows ii and ii + hd / 2 of a head section, or row p of gate and of up.
template <int WFMT, int EPI, int NLD, int NS>
__global__ __launch_bounds__(kGBlock, 1) void k_spair(SkArgs sa) {
  static_assert(EPI == PE_QKV || EPI == PE_SWIGLU, "products of row pairs");
  using St = VStage<WFMT>;
  constexpr int RPL = kGBlock / St::CPR;  // rows a load slot covers
  constexpr int NI = (NLD * RPL * kSkRows + kGBlock - 1) / kGBlock;
  const PGemmArgs& a = sa.g;
  extern __shared__ __align__(16) char smem[];
  __shared__ float inv_s[kSkRows];
  __shared__ int last_s;
  const int tid = threadIdx.x, lane = tid & (AIO_WAVE - 1), wid = tid / AIO_WAVE;
  constexpr int wbytes = WFMT == AIO_WFMT_BF16 ? 2 : 1;
  const int p0 = (int)blockIdx.x * sa.np, np = min(sa.np, sa.pairs - p0);
  const int qrows = a.H * a.hd, krows = a.Hkv * a.hd, half = a.hd / 2;
  SkStream<WFMT, NLD, NS> s;
  s.lchunk = tid % St::CPR;
#pragma unroll
  for (int j = 0; j < NLD; ++j) {
    const int sl = min(j * RPL + tid / St::CPR, 2 * np - 1);
    const bool hi = sl >= np;
    const int p = p0 + (hi ? sl - np : sl);
    int n = p, mat = hi;
    if constexpr (EPI == PE_QKV) {
      const int head = p >> (hd_shift(a.hd) - 1);
      n = head * a.hd + p - head * half + (hi ? half : 0);
      mat = 0;
      if (n >= qrows + krows) { mat = 2; n -= qrows + krows; }
      else if (n >= qrows) { mat = 1; n -= qrows; }
    }
    s.lrow[j] = pick_mat(a, mat) + (size_t)n * a.K * wbytes;
    s.lds_off[j] = ((hi ? 32 : 0) + p - p0) * St::RS + s.lchunk * 16;
  }
  s.wid = wid;
  s.rl = lane & 31;
  s.kh = lane >> 5;
  const int kz = (int)blockIdx.y, ksh = __builtin_ctz(a.ks);
  s.kbA = (kz * (a.K / 32)) >> ksh;
  s.kbB = ((kz + 1) * (a.K / 32)) >> ksh;
  s.nst = (s.kbB - s.kbA + St::BPS - 1) / St::BPS;
  // (by_nst divides by the stages of the longest slice)
  s.rot = min((int)blockIdx.x - udiv(blockIdx.x, sa.by_nst) * (int)sa.by_nst.d, s.nst - 1);
  s.kend = s.kbB * 32 * wbytes - 16;
  s.actp = a.act + (size_t)min(s.rl, a.R - 1) * a.lda;
  // the norm's row factors: wave w sums rows w, w + 8, ...
  float ssp[kSkRows / kGWaves][2];
  s.run(smem, a.R, [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int h = 0; h < kSkRows / kGWaves; ++h) {
      const float* ss = a.ss_in + (size_t)min(wid + kGWaves * h, a.R - 1) * a.nss;
      ssp[h][0] = lane < a.nss ? ss[lane] : 0.f;
      ssp[h][1] = lane + 64 < a.nss ? ss[lane + 64] : 0.f;
    }
  });
#pragma unroll
  for (int h = 0; h < kSkRows / kGWaves; ++h) {
    const int r = wid + kGWaves * h;
    if (r >= a.R) break;
    float p = ssp[h][0] + ssp[h][1];
    for (int c = lane + 128; c < a.nss; c += 64) p += a.ss_in[(size_t)r * a.nss + c];
    const float sum = wave_sum(p);
    if (lane == 0) inv_s[r] = rsqrtf(sum / (float)a.K + a.eps);
  }
  // Two lanes per pair and prompt row, each summing one of the pair's rows;
  // what the epilogue reads besides is requested before the barrier.
  float2 cs[NI];
  float sc[NI];
  const int h = tid & 1;
#pragma unroll
  for (int it = 0; it < NI; ++it) {
    cs[it] = make_float2(1.f, 0.f);
    sc[it] = 1.f;
    if (it * kGBlock >= 2 * np * a.R) break;
    const int e = min((tid + it * kGBlock) >> 1, np * a.R - 1);
    const int r = np == sa.np ? udiv(e, sa.by_np) : e / np, p = p0 + e - r * np;
    if constexpr (EPI == PE_QKV) {
      const int head = p >> (hd_shift(a.hd) - 1), ii = p - head * half, n = head * a.hd + ii;
      if (n < qrows + krows) cs[it] = a.rope[(size_t)(a.pos0 + r) * half + ii];
      if constexpr (WFMT == AIO_WFMT_INT8) {
        const uint16_t* q = n >= qrows + krows ? a.s2 + (n - qrows - krows)
                                               : (n >= qrows ? a.s1 + (n - qrows) : a.s0 + n);
        sc[it] = fp16_to_f32(q[h ? half : 0]);
      }
    } else if constexpr (WFMT == AIO_WFMT_INT8) {
      sc[it] = fp16_to_f32((h ? a.s1 : a.s0)[p]);
    }
  }
  __syncthreads();
  const float* red = (const float*)smem;
  float y[NI];
  float* part = a.fix + ((size_t)blockIdx.x * a.ks * 2 + h) * sa.np * a.R;
  const size_t pstep = (size_t)2 * sa.np * a.R;
#pragma unroll
  for (int it = 0; it < NI; ++it) {
    const int e = (tid + it * kGBlock) >> 1;
    if (e >= np * a.R) break;  // (both lanes of a pair)
    const int r = np == sa.np ? udiv(e, sa.by_np) : e / np, i = e - r * np;
    y[it] = sk_sum(red, h, i, r);
    if (a.ks > 1) st_agent(part + kz * pstep + e, y[it]);
  }
  if (a.ks > 1) {
    // as in k_sresid: the last slice to arrive adds all of them in order
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (tid == 0) last_s = atomic_add_agent(a.tcnt + blockIdx.x, 1) == a.ks - 1;
    __syncthreads();
    if (!last_s) return;
    if (tid == 0) atomic_store_agent(a.tcnt + blockIdx.x, 0);  // ready for the next product
    float pv[NI][kSkPairKs];
#pragma unroll
    for (int it = 0; it < NI; ++it) {
      if (it * kGBlock >= 2 * np * a.R) break;
      const int e = min((tid + it * kGBlock) >> 1, np * a.R - 1);
#pragma unroll
      for (int k = 0; k < kSkPairKs; ++k) pv[it][k] = ld_agent(part + (k < a.ks ? k : 0) * pstep + e);
    }
#pragma unroll
    for (int it = 0; it < NI; ++it) {
      if (it * kGBlock >= 2 * np * a.R) break;
      y[it] = 0.f;
#pragma unroll
      for (int k = 0; k < kSkPairKs; ++k)
        if (k < a.ks) y[it] += pv[it][k];
    }
  }
#pragma unroll
  for (int it = 0; it < NI; ++it) {
    const int e = (tid + it * kGBlock) >> 1;
    if (e >= np * a.R) break;
    const int r = np == sa.np ? udiv(e, sa.by_np) : e / np, i = e - r * np, p = p0 + i;
    const float yv = y[it] * inv_s[r] * sc[it];
    const float o = dpp_mov<0xB1>(yv);  // lane ^ 1
    if constexpr (EPI == PE_QKV) {
      // each lane stores its own row of the rotated pair
      const int head = p >> (hd_shift(a.hd) - 1), ii = p - head * half, n = head * a.hd + ii;
      const float v = n < qrows + krows ? yv * cs[it].x + (h ? o : -o) * cs[it].y : yv;
      const int off = h ? half : 0;
      if (n < qrows) {
        a.out[(size_t)r * a.ldo + n + off] = v;
      } else {
        const bool is_k = n < qrows + krows;
        const int g = (n - (is_k ? qrows : qrows + krows)) >> hd_shift(a.hd);
        ((is_k ? a.kc : a.vc) + ((size_t)g * a.max_ctx + a.pos0 + r) * a.hd)[ii + off] = f32_to_bf16(v);
      }
    } else if (h == 0) {
      a.act_out[(size_t)r * a.lda_out + p] = yv / (1.f + expf(-yv)) * o;
    }
  }
}

// O and down: 64 rows of the matrix and one of a.ks K slices per workgroup.
// With ks > 1 every slice writes its sums through to a.fix[slice][R][N], and
// the last one to arrive (a.tcnt) adds them in slice order, then to x.
template <int WFMT, int NS>
__global__ __launch_bounds__(kGBlock, 1) void k_sresid(PGemmArgs a) {
  using St = VStage<WFMT>;
  constexpr int NLD = St::NLD, NI = 64 * kSkRows / kGBlock;
  extern __shared__ __align__(16) char smem[];
  __shared__ int last_s;
  const int tid = threadIdx.x, lane = tid & (AIO_WAVE - 1), wid = tid / AIO_WAVE;
  constexpr int wbytes = WFMT == AIO_WFMT_BF16 ? 2 : 1;
  const int n0 = (int)blockIdx.x * 64, kz = (int)blockIdx.y, ksh = __builtin_ctz(a.ks);
  SkStream<WFMT, NLD, NS> s;
  s.lchunk = tid % St::CPR;
#pragma unroll
  for (int j = 0; j < NLD; ++j) {
    const int r = (j * kGBlock + tid) / St::CPR;
    s.lrow[j] = (const char*)a.w0 + (size_t)(n0 + r) * a.K * wbytes;
    s.lds_off[j] = r * St::RS + s.lchunk * 16;
  }
  const int nkb = a.K / 32;
  s.wid = wid;
  s.rl = lane & 31;
  s.kh = lane >> 5;
  s.kbA = (kz * nkb) >> ksh;
  s.kbB = ((kz + 1) * nkb) >> ksh;
  s.nst = (s.kbB - s.kbA + St::BPS - 1) / St::BPS;
  s.rot = (int)(blockIdx.x % (unsigned)s.nst);
  s.kend = s.kbB * 32 * wbytes - 16;
  s.actp = a.act + (size_t)min(s.rl, a.R - 1) * a.lda;
  // thread -> prompt rows r and output column n of the epilogue
  const int n = n0 + lane;
  float xv[NI], gn = 1.f, sc = 1.f;
  s.run(smem, a.R, [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int it = 0; it < NI; ++it)
      xv[it] = a.out[(size_t)min(wid + kGWaves * it, a.R - 1) * a.ldo + n];
    if (a.act_next) gn = bf16_to_f32(a.g_next[n]);
    if constexpr (WFMT == AIO_WFMT_INT8) sc = fp16_to_f32(a.s0[n]);
  });
  __syncthreads();
  const float* red = (const float*)smem;
  float v[NI];
#pragma unroll
  for (int it = 0; it < NI; ++it) {
    const int r = wid + kGWaves * it;
    if (r >= a.R) break;
    v[it] = sk_sum(red, lane / 32, lane % 32, r) * sc;
    if (a.ks > 1) st_agent(a.fix + ((size_t)kz * a.R + r) * a.N + n, v[it]);
  }
  float pv[NI][kVerifyMaxKs];
  if (a.ks > 1) {
    // every wave's stores have completed (written through) before the slice
    // is counted
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (tid == 0) last_s = atomic_add_agent(a.tcnt + blockIdx.x, 1) == a.ks - 1;
    __syncthreads();
    if (!last_s) return;
    if (tid == 0) atomic_store_agent(a.tcnt + blockIdx.x, 0);  // ready for the next product
#pragma unroll
    for (int it = 0; it < NI; ++it) {
      if (wid + kGWaves * it >= a.R) break;
#pragma unroll
      for (int k = 0; k < kVerifyMaxKs; ++k)
        pv[it][k] = ld_agent(a.fix + ((size_t)(k < a.ks ? k : 0) * a.R + wid + kGWaves * it) * a.N + n);
    }
  }
#pragma unroll
  for (int it = 0; it < NI; ++it) {
    const int r = wid + kGWaves * it;
    if (r >= a.R) break;  // (whole waves)
    float y = v[it];
    if (a.ks > 1) {
      y = 0.f;
#pragma unroll
      for (int k = 0; k < kVerifyMaxKs; ++k)
        if (k < a.ks) y += pv[it][k];
    }
    const float x = xv[it] + y;  // (rounded once at x's magnitude)
    a.out[(size_t)r * a.ldo + n] = x;
    if (a.act_next) {
      a.act_next[(size_t)r * a.lda_next + n] = x * gn;
      const float sq = wave_sum_sq(x);
      if (lane == 0) a.ss_out[(size_t)r * a.nss + blockIdx.x] = sq;
    }
  }
}

// ----------------------------------------------------------------- launchers

hipError_t launch_pnorm(const aio_model& m, const PfBuffers& b, int R, const uint16_t* embed,
                        const void* gain) {
  PNormArgs n{};
  n.x = b.x;
  n.embed = embed;
  n.tokens = b.tokens;
  n.gain = (const uint16_t*)gain;
  n.act = b.actA;
  n.lda = b.lda_a;
  n.d = m.cfg.d_model;
  n.ss = b.ss;
  hipLaunchKernelGGL(k_pnorm, dim3(R), dim3(kNormThreads), 0, m.stream, n);
  return hipGetLastError();
}

// The tile shapes, and what a product takes in each, in microseconds: every
// round of workgroups `round` plus, per 32 k of its K slice, `few` (at most
// half the CUs busy) or `full`; `base` once; a K split `split` plus
// `slice` per slice (scaled by the live share of the tile's prompt rows).
// Fitted to the 1B's and the 7B's four products (bf16) at 19 prompt lengths from
// 23 to 2048, every shape and split measured by kernel trace (the model is
// within 4 to 10 % of them, and the shape it picks within 1.8 % of the best
// one on average, 13 % at worst); int8 takes the same constants unfitted:
//   Big    one workgroup per CU; the fewest bytes and LDS reads per product
//          (2048 rows, 1B: QKV 86 against Wide's 105 us, gate/up 226 / 264)
//   Wide   half the prompt rows: twice the workgroups where Big leaves CUs
//          idle (2048 rows, 1B: O 53 against Big's 78 us unsplit, down
//          126 / 182; 1000 rows, 7B: O 95 / 140)
//   Short  prompts of a few blocks of 16 rows, split over K to cover the CUs
//          (23 rows, 1B: QKV 20.5 against Wide's 23.8 us, O 15.6 / 21.4,
//          gate/up 19.2 / 24.8, down 21.4 / 31.3)
//          (up to 32 rows most products now go to k_spair and k_sresid)
struct PfShape {
  int bm, bn, sk, per_cu;
  double few, full, round, base, split, slice;
};
using Big = PTile<4, 2, 4, 2, 1>;
using Wide = PTile<4, 2, 2, 2, 1>;
using Short = PTile<2, 1, 2, 2, 2>;
template <class Tl>
constexpr PfShape pf_shape(int per_cu, double few, double full, double round, double base,
                           double split, double slice) {
  return PfShape{Tl::BM, Tl::BN, Tl::SK, per_cu, few, full, round, base, split, slice};
}
constexpr PfShape kPfShapes[3] = {
    pf_shape<Big>(1, 0.96, 1.07, 7.3, 3.5, 0.0, 5.6),
    pf_shape<Wide>(1, 0.60, 0.67, 3.3, 5.1, 2.6, 1.7),
    pf_shape<Short>(2, 0.25, 0.43, 2.4, 7.9, 1.1, 0.9),
};

// A product of a layer as the choice of its kernel sees it, and the choice.
struct PfProduct {
  int epi;           // PEpi
  int N, K, R;       // as in PGemmArgs
  int units;         // units of 128 weight rows
  size_t fix_bytes;  // room for the sums of K slices
};
struct PfPlan {
  int kernel;  // a tile shape of kPfShapes, or kPfFewRows: k_spair, k_sresid
  int ks, np;  // K slices; row pairs per workgroup (k_spair)
};
constexpr int kPfFewRows = 3;

// Bytes of the partial tiles of `tiles` tiles split into ks slices.
size_t pf_fix_bytes(const PfShape& s, size_t tiles, int ks) {
  return ks == 1 ? 0 : tiles * (ks == 2 ? 1 : ks) * s.bm * s.bn * 4;
}

// Shape and K split (up to kPfMaxKs, within the fix-up room) with the least
// predicted time.
void pf_choose(const PfProduct& p, int num_cus, size_t counters, int* shape, int* ks) {
  const int units = p.units, R = p.R, K = p.K;
  double best = 1e30;
  for (int i = 0; i < 3; ++i) {
    const PfShape& s = kPfShapes[i];
    const size_t tiles = (size_t)((units * kUnit + s.bm - 1) / s.bm) * ((R + s.bn - 1) / s.bn);
    const long long slots = (long long)s.per_cu * num_cus;
    for (int k = 1; k <= kPfMaxKs; k *= 2) {
      if (k > 1 && (pf_fix_bytes(s, tiles, k) > p.fix_bytes || tiles > counters || K / s.sk < k))
        break;
      const long long wgs = (long long)tiles * k, rem = wgs % slots;
      const double st = (double)K / kKT / k;
      auto round = [&](long long n) {
        return st * (2 * n <= slots ? s.few : s.full) + s.round;
      };
      const double t = s.base + (double)(wgs / slots) * round(slots) + (rem ? round(rem) : 0.0) +
                       (k > 1 ? s.split + s.slice * k * std::min(R, s.bn) / s.bn : 0.0);
      if (t < best) {
        best = t;
        *shape = i;
        *ks = k;
      }
    }
  }
}

template <int WFMT, int EPI, class Tl>
hipError_t launch_pgemm_t(const aio_model& m, const PGemmArgs& g, int units) {
  const dim3 grid((units + Tl::UPT - 1) / Tl::UPT, (g.R + Tl::BN - 1) / Tl::BN, g.ks);
  const void* fn = (const void*)k_pgemm<WFMT, EPI, Tl>;
  hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, Tl::Lds);
  if (e != hipSuccess) return e;
  PGemmArgs a = g;
  const unsigned tiles = grid.x * grid.y, tail = grid.y % Tl::kBand;
  a.by_band = make_udiv(Tl::kBand * grid.x, tiles);
  a.by_tail = make_udiv(tail ? tail : 1, tiles);
  hipLaunchKernelGGL((k_pgemm<WFMT, EPI, Tl>), grid, dim3(Tl::GT), Tl::Lds, m.stream, a);
  return hipGetLastError();
}

// Products of a few prompt rows (SkArgs).  Pairs: one round of workgroups of at
// most 32 pairs (one 32-row tile of each of their rows).
template <int WFMT, int EPI, int NLD, int NS>
hipError_t launch_spair_t(const aio_model& m, const SkArgs& a) {
  constexpr int lds = vgemm_lds<WFMT, 2>(64);
  const void* fn = (const void*)k_spair<WFMT, EPI, NLD, NS>;
  const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_spair<WFMT, EPI, NLD, NS>), dim3((a.pairs + a.np - 1) / a.np, a.g.ks),
                     dim3(kGBlock), lds, m.stream, a);
  return hipGetLastError();
}
template <int WFMT, int NS>
hipError_t launch_sresid_t(const aio_model& m, const PGemmArgs& g) {
  constexpr int lds = vgemm_lds<WFMT, 2>(64);
  const void* fn = (const void*)k_sresid<WFMT, NS>;
  const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_sresid<WFMT, NS>), dim3(g.N / 64, g.ks), dim3(kGBlock), lds, m.stream, g);
  return hipGetLastError();
}

// Pairs per workgroup and K slices of a product of `pairs` row pairs; false
// where it is left to the tile products.  Every workgroup reads the activations
// of its slice: more than 384 KB of them cost what the even shares gain (7B
// QKV, K 4096: 23 rows, 368 KB, 31.6 us against the tiles' 32.6; 32 rows, 512 KB,
// 34.6 / 32.6, int8 32.7 / 30.9), and pairs for half or a quarter of K are
// preferred where 32 allow it (QKV of the 1B, K 2048, 23 rows: 8 pairs each 14.8
// us, 32 of a quarter 12.6).  More than 32 pairs would need a second pair of
// tiles, whose hi and lo do not fit the registers.
bool sk_pairs(const PfProduct& p, int num_cus, size_t counters, int* np, int* ks) {
  const int pairs = p.epi == PE_QKV ? p.N / 2 : p.N;
  for (*ks = kSkPairKs; *ks >= 1; *ks /= 2) {
    *np = (pairs * *ks + num_cus - 1) / num_cus;
    if (*np > 32) continue;
    const size_t tiles = (size_t)(pairs + *np - 1) / *np;
    if (*ks > 1 && (p.K / 32 / (*ks * kGWaves) < 2 || tiles > counters ||
                    tiles * *ks * 2 * *np * p.R * 4 > p.fix_bytes))
      continue;
    return p.R <= kSkRows && (size_t)4 * p.R * p.K / *ks <= 384 * 1024;
  }
  return false;
}

// K slices of k_sresid: as far as there are CUs and every wave keeps two blocks,
// and the slices' sums fit the fix-up room.
int sk_resid_slices(const PfProduct& p, int num_cus, size_t counters) {
  const int nkb = p.K / 32, tiles = p.N / 64;
  int ks = 1;
  while (tiles * ks < num_cus && 2 * ks <= kVerifyMaxKs && nkb / (2 * ks * kGWaves) >= 2 &&
         (size_t)tiles <= counters && (size_t)2 * ks * p.R * p.N * 4 <= p.fix_bytes)
    ks *= 2;
  return ks;
}

PfPlan pf_plan(const PfProduct& p, int num_cus, size_t counters) {
  PfPlan c{kPfFewRows, 1, 0};
  if (p.epi == PE_RESID && p.R <= kSkRows)
    c.ks = sk_resid_slices(p, num_cus, counters);
  else if (p.epi == PE_RESID || !sk_pairs(p, num_cus, counters, &c.np, &c.ks)) {
    c.np = 0;
    pf_choose(p, num_cus, counters, &c.kernel, &c.ks);
  }
  return c;
}

// Bytes of scratch that are idle during a product of a chunk of R rows and hold the
// partial sums of its K slices (sized by R alone, so that the split, and with it
// the order of the sums, does not depend on how much scratch there is).
enum PfWhich { PF_QKV = 0, PF_O = 1, PF_GU = 2, PF_DOWN = 3 };
size_t pf_idle_bytes(const aio_config& c, int which, int R) {
  const size_t d = (size_t)c.d_model, F = (size_t)c.ffn_dim, Hd = (size_t)c.n_heads * c.head_dim;
  const size_t words[4] = {d + F, F, Hd + std::max(d, Hd), Hd};
  return 4 * (size_t)R * words[which];
}

// The product as pf_plan takes it; the workspace's fix-up region serves where it is
// the larger one.
PfProduct pf_product(const aio_config& c, const WsLayout& lay, int which, int R) {
  PfProduct p{};
  const int Hd = c.n_heads * c.head_dim;
  p.epi = which == PF_QKV ? PE_QKV : (which == PF_GU ? PE_SWIGLU : PE_RESID);
  p.N = which == PF_QKV ? Hd + 2 * c.n_kv_heads * c.head_dim : (which == PF_GU ? c.ffn_dim : c.d_model);
  p.K = which == PF_O ? Hd : (which == PF_DOWN ? c.ffn_dim : c.d_model);
  p.R = R;
  p.units = which == PF_GU ? (p.N + 63) / 64 : (p.N + kUnit - 1) / kUnit;
  p.fix_bytes = std::max(pf_idle_bytes(c, which, R), lay.pfix_bytes);
  return p;
}

template <int WFMT, int EPI>
hipError_t launch_sk(const aio_model& m, const PGemmArgs& g, const PfPlan& plan) {
  if constexpr (EPI == PE_RESID) {
    return launch_sresid_t<WFMT, 2>(m, g);
  } else {
    SkArgs a{};
    a.g = g;
    a.pairs = EPI == PE_QKV ? g.N / 2 : g.N;
    a.np = plan.np;
    a.by_np = make_udiv((unsigned)a.np, (unsigned)(a.np * kSkRows));
    constexpr int bps = VStage<WFMT>::BPS;
    const int slice = (g.K / 32 + g.ks - 1) / g.ks;  // blocks of the longest slice
    a.by_nst = make_udiv((unsigned)((slice + bps - 1) / bps), (unsigned)a.pairs);
    if constexpr (WFMT == AIO_WFMT_BF16) {
      if (a.np <= 8) return launch_spair_t<WFMT, EPI, 1, 3>(m, a);
      if (a.np <= 16) return launch_spair_t<WFMT, EPI, 2, 3>(m, a);
      if (a.np <= 24) return launch_spair_t<WFMT, EPI, 3, 2>(m, a);
      return launch_spair_t<WFMT, EPI, 4, 2>(m, a);
    } else {
      if (a.np <= 16) return launch_spair_t<WFMT, EPI, 1, 3>(m, a);
      return launch_spair_t<WFMT, EPI, 2, 3>(m, a);
    }
  }
}

// Launch of product `which` of a chunk of g.R rows.  The partial sums of a K split
// go to the scratch that is idle during this product (idle), or to the workspace's
// region where that is larger.
template <int WFMT, int EPI>
hipError_t launch_pgemm_w(const aio_model& m, const PGemmArgs& g0, int which, void* idle) {
  const PfProduct p = pf_product(m.cfg, m.lay, which, g0.R);
  const PfPlan plan = pf_plan(p, m.num_cus, m.lay.pcnt_n);
  PGemmArgs g = g0;
  g.N = p.N;
  g.K = p.K;
  g.ks = plan.ks;
  g.fix = pf_idle_bytes(m.cfg, which, g.R) < m.lay.pfix_bytes ? m.at<float>(m.lay.pfix) : (float*)idle;
  g.tcnt = m.at<int>(m.lay.pcnt);
  g.err = m.at<int>(m.lay.sync) + kSyncErr;
  if (plan.kernel == kPfFewRows) return launch_sk<WFMT, EPI>(m, g, plan);
  if (plan.kernel == 0) return launch_pgemm_t<WFMT, EPI, Big>(m, g, p.units);
  if (plan.kernel == 1) return launch_pgemm_t<WFMT, EPI, Wide>(m, g, p.units);
  return launch_pgemm_t<WFMT, EPI, Short>(m, g, p.units);
}

template <int EPI>
hipError_t launch_pgemm(const aio_model& m, const PGemmArgs& g, int which, void* idle) {
  if (m.cfg.wfmt == AIO_WFMT_INT8) return launch_pgemm_w<AIO_WFMT_INT8, EPI>(m, g, which, idle);
  return launch_pgemm_w<AIO_WFMT_BF16, EPI>(m, g, which, idle);
}

template <int HD>
hipError_t launch_pattn_t(const aio_model& m, const PAttnArgs& t) {
  const void* fn = (const void*)k_pattn<HD>;
  hipError_t e =
      hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, AttnLds<HD>::BYTES);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_pattn<HD>, dim3((t.R + 31) / 32, t.H), dim3(kAW * AIO_WAVE),
                     AttnLds<HD>::BYTES, m.stream, t);
  return hipGetLastError();
}

}  // namespace

int aio_prefill_plan(const aio_config* c, int rows, int num_cus, int32_t* out) {
  const int rc = aio_check_config(c);
  if (rc) return rc;
  if (rows < 1 || num_cus < 1 || !out) return AIO_EINVAL;
  const WsLayout lay = aio_ws_layout(*c);
  for (int which = 0; which < 4; ++which) {
    const PfPlan p = pf_plan(pf_product(*c, lay, which, rows), num_cus, lay.pcnt_n);
    out[3 * which] = p.kernel;
    out[3 * which + 1] = p.ks;
    out[3 * which + 2] = p.np;
  }
  return AIO_OK;
}

size_t aio_prefill_row_bytes(const aio_config& c) {
  const size_t d = (size_t)c.d_model, Hd = (size_t)c.n_heads * c.head_dim, F = (size_t)c.ffn_dim;
  const size_t ka = d > Hd ? d : Hd;
  return 4 + 4 * d + 4 * Hd + 4 * ka + 4 * d + 4 * F + 4 * (d / 64);
}

PfBuffers aio_prefill_buffers(const aio_config& c, char* base, int rcap) {
  PfBuffers b{};
  const size_t d = (size_t)c.d_model, Hd = (size_t)c.n_heads * c.head_dim, F = (size_t)c.ffn_dim;
  auto al = [](size_t v) { return (v + 255u) & ~(size_t)255u; };
  size_t off = 0;
  b.rcap = rcap;
  b.lda_a = (int)(d > Hd ? d : Hd);
  b.lda_b = (int)F;
  b.tokens = (int32_t*)(base + off); off = al(off + 4 * (size_t)rcap);
  b.x = (float*)(base + off); off = al(off + 4 * d * rcap);
  b.q = (float*)(base + off); off = al(off + 4 * Hd * rcap);
  b.actA = (float*)(base + off); off = al(off + 4 * (size_t)b.lda_a * rcap);
  b.actN = (float*)(base + off); off = al(off + 4 * d * rcap);
  b.actB = (float*)(base + off); off = al(off + 4 * (size_t)b.lda_b * rcap);
  b.ss = (float*)(base + off); off = al(off + 4 * (d / 64) * rcap);
  b.bytes = off;
  return b;
}

// One chunk of R <= b.rcap prompt rows at positions pos0 .. pos0 + R - 1;
// their tokens are in b.tokens.  On return (enqueued) the cache holds their
// K/V rows in every layer and b.x row R - 1 the last row's final residual.
hipError_t aio_launch_prefill_chunk(const aio_model& m, const PfBuffers& b, int R, int pos0) {
  const aio_config& c = m.cfg;
  const int d = c.d_model, H = c.n_heads, Hkv = c.n_kv_heads, hd = c.head_dim;
  const int nss = d / 64;
  hipError_t e;
  // layer 0's input rows: the embeddings, with x g and the sums of squares
  // for its attention norm; every later norm input comes from the residual
  // product before it
  if ((e = launch_pnorm(m, b, R, (const uint16_t*)m.embed, m.layers[0].attn_norm)) != hipSuccess)
    return e;
  for (int l = 0; l < c.n_layers; ++l) {
    const aio_layer_weights& L = m.layers[(size_t)l];
    const bool last = l + 1 == c.n_layers;

    PGemmArgs g{};
    g.act = b.actA; g.lda = b.lda_a; g.R = R;
    g.ss_in = b.ss; g.nss = nss; g.eps = c.rms_eps;
    g.w0 = L.wq; g.w1 = L.wk; g.w2 = L.wv;
    g.s0 = (const uint16_t*)L.sq; g.s1 = (const uint16_t*)L.sk; g.s2 = (const uint16_t*)L.sv;
    g.out = b.q; g.ldo = H * hd;
    g.kc = m.kv_layer(l, 0); g.vc = m.kv_layer(l, 1);
    g.rope = m.rope; g.pos0 = pos0;
    g.H = H; g.Hkv = Hkv; g.hd = hd; g.max_ctx = c.max_ctx;
    // (the last argument of a product: activations idle meanwhile, for the partial
    // sums of a K split)
    if ((e = launch_pgemm<PE_QKV>(m, g, PF_QKV, b.actN)) != hipSuccess) return e;

    PAttnArgs t{};
    t.q = b.q; t.ldq = H * hd;
    t.kc = g.kc; t.vc = g.vc;
    t.act = b.actA; t.lda = b.lda_a;
    t.R = R; t.pos0 = pos0; t.H = H; t.Hkv = Hkv; t.max_ctx = c.max_ctx;
    t.by_g = make_udiv((unsigned)(H / Hkv), (unsigned)H);
    t.by_hpx = make_udiv((unsigned)std::max(H / 8, 1), (unsigned)H * (unsigned)((R + 31) / 32));
    t.scale_log2 = (float)(1.4426950408889634 / sqrt((double)hd));
    e = hd == 128 ? launch_pattn_t<128>(m, t) : launch_pattn_t<64>(m, t);
    if (e != hipSuccess) return e;

    PGemmArgs o{};
    o.act = b.actA; o.lda = b.lda_a; o.R = R;
    o.w0 = L.wo; o.s0 = (const uint16_t*)L.so;
    o.out = b.x; o.ldo = d;
    o.act_next = b.actN; o.lda_next = d;
    o.g_next = (const uint16_t*)L.ffn_norm; o.ss_out = b.ss; o.nss = nss;
    if ((e = launch_pgemm<PE_RESID>(m, o, PF_O, b.actB)) != hipSuccess) return e;

    PGemmArgs gu{};
    gu.act = b.actN; gu.lda = d; gu.R = R;
    gu.ss_in = b.ss; gu.nss = nss; gu.eps = c.rms_eps;
    gu.w0 = L.w_gate; gu.w1 = L.w_up;
    gu.s0 = (const uint16_t*)L.s_gate; gu.s1 = (const uint16_t*)L.s_up;
    gu.act_out = b.actB; gu.lda_out = b.lda_b;
    if ((e = launch_pgemm<PE_SWIGLU>(m, gu, PF_GU, b.q)) != hipSuccess) return e;

    PGemmArgs dn{};
    dn.act = b.actB; dn.lda = b.lda_b; dn.R = R;
    dn.w0 = L.w_down; dn.s0 = (const uint16_t*)L.s_down;
    dn.out = b.x; dn.ldo = d;
    if (!last) {
      dn.act_next = b.actA; dn.lda_next = b.lda_a;
      dn.g_next = (const uint16_t*)m.layers[(size_t)l + 1].attn_norm;
      dn.ss_out = b.ss; dn.nss = nss;
    }
    if ((e = launch_pgemm<PE_RESID>(m, dn, PF_DOWN, b.q)) != hipSuccess) return e;
  }
  return hipSuccess;
}
