// Verify forward (prompt-lookup verification): M = k + 1 <= 10 rows at
// positions pos .. pos + k in one pass over the weights, for gfx950.
//
// At M rows a projection does ~M flops per weight byte (8-16 flop/B), close
// to the fp32 VALU ridge, so the matrix products run on MFMA
// (v_mfma_f32_32x32x16_bf16).  MFMA inputs are bf16; to keep fp32-level
// accuracy each fp32 activation a is split exactly into three bf16 terms,
// a = t0 + t1 + t2 + O(2^-27 a) (t0 = bf16(a), t1 = bf16(a - t0),
// t2 = bf16(a - t0 - t1); each subtraction is exact in fp32), and the three
// terms of all M rows form the 3M <= 30 columns of one 32-column B operand.
// Weights are the A operand (32 output channels per tile); int8 weights
// convert to bf16 exactly (|q| <= 127) and their fp16 scale is applied in the
// epilogue.
//
// RMSNorm is folded into the products around it.  Its scale
// 1 / sqrt(mean(x_r^2) + eps) is one number per row, so it commutes with the
// product: the GEMM that consumes a normed row multiplies the split of x * g
// and scales its result by the row's factor, which it forms from the row's
// sums of squares over 64-column chunks (written by whoever completed those
// columns of x, summed in chunk order).
//
// Per layer: QKV GEMM (+norm scale, RoPE, K/V append) -> vattn_mma (causal
// split-KV on MFMA, row r sees positions [0, pos + r]; the last split of a
// head merges the head's splits and writes the split output) -> O GEMM
// (+residual, split of x * g_ffn, sums of squares) -> gate/up GEMM (+norm
// scale, SwiGLU, split) -> down GEMM (+residual, split of x * g for the next
// layer or the final norm); then the LM head GEMM (+norm scale) -> logits
// [M][V].  Layer 0's input (the embedding rows) goes through vnorm.
#include <math.h>
#include <algorithm>

#include "aio_internal.h"
#include "common.h"
#include "lanes.h"
#include "skinny.h"

namespace {

constexpr int kMaxRows = AIO_MAX_VERIFY_ROWS;

// Up to this many visible positions a verify's sums keep one order.  There the new
// rows attend mostly to one another, so a K or V element whose fp32 value rounds
// the other way moves everything after it: two orders of the gate/up sums put the
// cache rows of a 7B verify of 4 rows at position 17 up to 1.1e-3 apart (each as
// far from a 64-bit evaluation), 7e-4 at 40, some 2e-4 at 260 and less beyond (at
// the median: over 960 inputs at 260 to 14000 positions 4.5e-4 at most).  So gate/up
// runs in the order of k_vgemm_sk up to here, some 4 us per layer of a 7B slower
// than k_vpair, which takes it beyond; QKV keeps its workgroups inside blocks of 32
// pairs, and a single attention split folds its waves one by one (256: one split, a
// key block per wave).  The other kernels have one order at any length.
constexpr int kOrderKeys = 256;

enum Epi { EPI_QKV = 0, EPI_RESID = 1, EPI_SWIGLU = 2, EPI_STORE = 3 };

// Exact three-term bf16 split of an fp32 value.
AIO_DEV void split3(float a, uint16_t& t0, uint16_t& t1, uint16_t& t2) {
  t0 = f32_to_bf16(a);
  const float r1 = a - bf16_to_f32(t0);
  t1 = f32_to_bf16(r1);
  const float r2 = r1 - bf16_to_f32(t1);
  t2 = f32_to_bf16(r2);
}

AIO_DEV void store_split(uint16_t* act, int lda, int M, int r, int col, float v) {
  uint16_t t0, t1, t2;
  split3(v, t0, t1, t2);
  act[(size_t)r * lda + col] = t0;
  act[(size_t)(M + r) * lda + col] = t1;
  act[(size_t)(2 * M + r) * lda + col] = t2;
}

// ------------------------------------------------------------ RMSNorm rows

struct VNormArgs {
  float* x;                 // [M][d] residual rows
  const uint16_t* embed;    // layer 0: embedding table (tokens from state), else null
  const uint16_t* gain;
  uint16_t* act;            // [32][lda] split of x * g
  int lda, d, M;
  float* ss;                // [M][d / 64] sums of squares of x over 64-column chunks
  const aio_state* st;
};

// One workgroup of 1024 threads per row r (in layer 0 x_r is the embedding
// row of the row's token, written to x): the split of x_r * g and the sums of
// squares of x_r per 64-column chunk.  Wave w holds chunks w, w + 16, ...
constexpr int kNormBlock = 1024;

__global__ __launch_bounds__(kNormBlock) void k_vnorm(VNormArgs a) {
  const int r = blockIdx.x, tid = threadIdx.x;
  const uint16_t* emb = a.embed ? a.embed + (size_t)a.st->token[r] * a.d : nullptr;
  float* xr = a.x + (size_t)r * a.d;
  for (int e = tid; e < a.d; e += kNormBlock) {  // wave-uniform: d % 64 == 0
    float v;
    if (emb) {
      v = bf16_to_f32(emb[e]);
      xr[e] = v;
    } else {
      v = xr[e];
    }
    store_split(a.act, a.lda, a.M, r, e, v * bf16_to_f32(a.gain[e]));
    const float sq = wave_sum_sq(v);
    if ((tid & (AIO_WAVE - 1)) == 0) a.ss[(size_t)r * (a.d / 64) + e / 64] = sq;
  }
}

// ------------------------------------------------------------- skinny GEMM

struct VGemmArgs {
  const uint16_t* act;      // [32][lda] bf16, columns j = term * M + row
  int lda;
  const void* w0;           // QKV: wq | SWIGLU: w_gate | else the matrix
  const void* w1;           // QKV: wk | SWIGLU: w_up
  const void* w2;           // QKV: wv
  const uint16_t* s0;
  const uint16_t* s1;
  const uint16_t* s2;
  int N, K, M;
  float* out;               // QKV: q [M][H*hd] | RESID: x [M][N] | STORE: logits [M][N]
  int ldo;
  uint16_t* act_out;        // SWIGLU: split m [32][lda_out]
  int lda_out;
  uint16_t* kc;
  uint16_t* vc;
  const float2* rope;
  int H, Hkv, hd, max_ctx;
  int ks;                   // K splits across workgroups (grid.y); > 1 only for EPI_RESID
  float* part;              // RESID with ks > 1: [ks][M][ldo], slice y's product
  // QKV, SWIGLU, STORE: the act columns are the split of x * g; each output
  // is scaled by 1 / sqrt(sum(ss_in[r][0 .. nt)) / K + eps)
  const float* ss_in;
  int nt;
  float eps;
  // RESID: completes x (ldo == N == d), then writes act_next = split of
  // x * g_next and ss_out [M][N / 64]; cnt [N / 64] counts arrived slices
  int* cnt;
  const uint16_t* g_next;
  uint16_t* act_next;
  float* ss_out;
  int pairs, np;            // QKV, SWIGLU: row pairs of the product and per workgroup
  int pos;                  // QKV: position of the first row
  UDiv by_np, by_nst;       // divisions by np and by the K stages (QKV, SWIGLU)
  // stream-K SWIGLU: `units` units in ranges of each or each + 1; shared tile
  // pairs' sums in skpart, their arrivals counted in skcnt
  int units, each, rest;
  float* skpart;
  int* skcnt;
};

// Register sets of weight stages in flight per workgroup (three measured
// slower: 4.56 against 4.20 ms per 7B bf16 verify, the extra registers
// leaving one workgroup per CU).
constexpr int kVNB = 2;

// Each workgroup owns T = 2 tiles of 32 output channels and one of a.ks
// slices of K (grid.y).  Its weights pass through LDS in stages (VStage),
// two stages in flight in registers; wave w multiplies block w of every
// stage, and the 8 waves' partial 32x32 tiles are summed in LDS at the end.
// Lane l of a wave covers tile row (l % 32) and 16 of the 32 k of a block
// (vk_lo, vk_hi): MFMA "a" takes 8 of them and MFMA "b" the other 8; the B
// operand (activation column l % 32) is loaded with the same k, so the k
// permutation cancels.
template <int WFMT, int T>
struct VFrag {
  bf16x8 wa[T], wb[T], ba, bb;
};

template <int WFMT, int T>
AIO_DEV void vmma(const VFrag<WFMT, T>& f, bool col_live, f32x16 (&acc)[T]) {
  // dead columns (past the 3M split terms) multiply zeros
  const bf16x8 z = __builtin_bit_cast(bf16x8, make_uint4(0u, 0u, 0u, 0u));
  const bf16x8 ba = col_live ? f.ba : z, bb = col_live ? f.bb : z;
#pragma unroll
  for (int t = 0; t < T; ++t) {
    acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.wa[t], ba, acc[t], 0, 0, 0);
    acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.wb[t], bb, acc[t], 0, 0, 0);
  }
}

// The waves' partial tiles to LDS (D layout: lane l, register v -> column j =
// l % 32, row i = 8 * (v / 4) + 4 * (l / 32) + (v % 4); only columns with a
// term of a row).
template <int T>
AIO_DEV void vred_put(float* red, int wid, int rl, int kh, bool col_live,
                      const f32x16 (&acc)[T]) {
  if (!col_live) return;
#pragma unroll
  for (int t = 0; t < T; ++t)
#pragma unroll
    for (int v = 0; v < 16; ++v)
      red[(wid * T + t) * kVRedTile<T> + (8 * (v / 4) + 4 * kh + (v % 4)) * 33 + rl] = acc[t][v];
}
// Row r of output i of tile t: every wave's sums of the three split terms, waves
// w and w + 4 first (an order that results behind a short cache keep to).
template <int T>
AIO_DEV float vred_sum(const float* red, int t, int i, int r, int M) {
  constexpr int kHalf = kGWaves / 2, kNext = kHalf * T * kVRedTile<T>;
  float s = 0.f;
#pragma unroll
  for (int w = 0; w < kHalf; ++w) {
    const float* p = red + (w * T + t) * kVRedTile<T> + i * 33 + r;
    s += (p[0] + p[kNext]) + (p[M] + p[M + kNext]) + (p[2 * M] + p[2 * M + kNext]);
  }
  return s;
}

// What the epilogue of verify row r of pair p reads besides the sums: cos and
// sin of the pair's angle (QKV: q and k), the int8 scales.
struct PairIn {
  float2 cs;
  float s0, s1;
};
template <int WFMT, int EPI>
AIO_DEV PairIn vpair_in(const VGemmArgs& a, int p, int r) {
  PairIn in{make_float2(1.f, 0.f), 1.f, 1.f};
  if constexpr (EPI == EPI_QKV) {
    const int qrows = a.H * a.hd, krows = a.Hkv * a.hd, half = a.hd / 2;
    const int head = p >> (hd_shift(a.hd) - 1), ii = p - head * half, n = head * a.hd + ii;
    if (n < qrows + krows) in.cs = a.rope[(size_t)(a.pos + r) * half + ii];
    if constexpr (WFMT == AIO_WFMT_INT8) {
      // both rows of the pair lie in the same (q, k or v) section
      const uint16_t* sc = n >= qrows + krows ? a.s2 + (n - qrows - krows)
                                              : (n >= qrows ? a.s1 + (n - qrows) : a.s0 + n);
      in.s0 = fp16_to_f32(sc[0]);
      in.s1 = fp16_to_f32(sc[half]);
    }
  } else if constexpr (WFMT == AIO_WFMT_INT8) {
    in.s0 = fp16_to_f32(a.s0[p]);
    in.s1 = fp16_to_f32(a.s1[p]);
  }
  return in;
}

// Epilogue of verify row r of pair p of a QKV or gate/up product, from the
// pair's two norm-scaled sums y0, y1:
//   QKV: pair p = rows ii and ii + hd / 2 of a head section, rotated at
//     position pos + r, to q or to the K / V cache;
//   SWIGLU: row p of gate and of up, silu(g) u split into act_out.
template <int WFMT, int EPI>
AIO_DEV void vpair_epi(const VGemmArgs& a, const PairIn& in, int p, int r, float y0, float y1) {
  if constexpr (WFMT == AIO_WFMT_INT8) {
    y0 *= in.s0;
    y1 *= in.s1;
  }
  if constexpr (EPI == EPI_QKV) {
    const int qrows = a.H * a.hd, krows = a.Hkv * a.hd, half = a.hd / 2;
    const int head = p >> (hd_shift(a.hd) - 1), ii = p - head * half, n = head * a.hd + ii;
    float lo = y0, hi = y1;
    if (n < qrows + krows) {
      lo = fmaf(y0, in.cs.x, -(y1 * in.cs.y));
      hi = fmaf(y1, in.cs.x, y0 * in.cs.y);
    }
    if (n < qrows) {
      a.out[(size_t)r * a.ldo + n] = lo;
      a.out[(size_t)r * a.ldo + n + half] = hi;
    } else {
      const bool is_k = n < qrows + krows;
      const int g = (n - (is_k ? qrows : qrows + krows)) >> hd_shift(a.hd);
      uint16_t* c = (is_k ? a.kc : a.vc) + ((size_t)g * a.max_ctx + a.pos + r) * a.hd;
      c[ii] = f32_to_bf16(lo);
      c[ii + half] = f32_to_bf16(hi);
    }
  } else {
    store_split(a.act_out, a.lda_out, a.M, r, p, y0 / (1.f + expf(-y0)) * y1);
  }
}

// Norm factors of rows: wave w sums the chunk sums of rows w and w + 8, lane
// l taking chunks l, l + 64, ...; ssp holds the first two of each, requested
// earlier.
AIO_DEV void vnorm_request(const VGemmArgs& a, int wid, int lane, float (&ssp)[2][2]) {
  static_assert(kMaxRows <= 2 * kGWaves, "two rows per wave");
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int r = wid + kGWaves * h;
    ssp[h][0] = ssp[h][1] = 0.f;
    if (r < a.M) {
      const float* ssr = a.ss_in + (size_t)r * a.nt;
      if (lane < a.nt) ssp[h][0] = ssr[lane];
      if (lane + 64 < a.nt) ssp[h][1] = ssr[lane + 64];
    }
  }
}
AIO_DEV void vnorm_finish(const VGemmArgs& a, int wid, int lane, const float (&ssp)[2][2],
                          float* inv_s) {
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int r = wid + kGWaves * h;
    if (r < a.M) {
      float p = ssp[h][0] + ssp[h][1];
      for (int c = lane + 128; c < a.nt; c += 64) p += a.ss_in[(size_t)r * a.nt + c];
      const float sum = wave_sum(p);
      if (lane == 0) inv_s[r] = rsqrtf(sum / (float)a.K + a.eps);
    }
  }
}

template <int WFMT, int EPI>
__global__ __launch_bounds__(kGBlock) void k_vgemm(VGemmArgs a) {
  constexpr int T = 2;
  using St = VStage<WFMT>;
  extern __shared__ __align__(16) char smem[];
  float* red = (float*)smem;
  __shared__ float inv_s[kMaxRows];
  __shared__ int last_s;
  const int tid = threadIdx.x, lane = tid & (AIO_WAVE - 1), wid = tid / AIO_WAVE;
  const int rl = lane & 31, kh = lane >> 5;
  const size_t wbytes = WFMT == AIO_WFMT_BF16 ? 2 : 1;

  const int tile_row[T] = {(int)blockIdx.x * 64, (int)blockIdx.x * 64 + 32};
  const bool col_live = rl < 3 * a.M;
  // (requested here and added only in the epilogue, so no wait in the
  // product is spent on them)
  float ssp[2][2];
  if (EPI != EPI_RESID) vnorm_request(a, wid, lane, ssp);
  // dead columns read row 0 (in bounds) and are zeroed before the product
  const uint16_t* actp = a.act + (size_t)(col_live ? rl : 0) * a.lda;

  // This workgroup's K slice in stages of BPS blocks of 32 k; wave w
  // multiplies blocks w, w + 8, ... of every stage.
  constexpr int BPS = St::BPS, BPW = St::BPW;
  const int nkb = a.K / 32;
  const int ks = (int)blockIdx.y;
  const int kbA = ks * nkb / a.ks, kbB = (ks + 1) * nkb / a.ks;
  const int nst = (kbB - kbA + BPS - 1) / BPS;
  // Workgroup b takes its stages starting at stage b mod nst (and wraps).
  // Every row of W is K * wbytes apart, a multiple of the HBM channel
  // interleave, so the same k offset of all rows lies in the same few
  // channels: in step, every workgroup would read the same channels at
  // once.
  const int rot = nst > 0 ? (int)(blockIdx.x % (unsigned)nst) : 0;
  auto kb0 = [&](int st) {  // first 32-k block of stage st (st < 2 nst)
    const int p = st + rot;
    return kbA + (p >= nst ? p - nst : p) * BPS;
  };
  f32x16 acc[T];
#pragma unroll
  for (int t = 0; t < T; ++t)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[t][i] = 0.f;

  // staging: load j of this thread is chunk c of stage row r (r < 64: tile
  // r / 32, tile row r % 32); chunks past the slice re-read its last chunk
  const char* lrow[St::NLD];
  int lds_off[St::NLD], lchunk[St::NLD];
#pragma unroll
  for (int j = 0; j < St::NLD; ++j) {
    const int f = j * kGBlock + tid, r = f / St::CPR, c = f % St::CPR;
    int n = tile_row[r / 32] + r % 32;
    if (n >= a.N) n = a.N - 1;
    lrow[j] = (const char*)a.w0 + (size_t)n * a.K * wbytes;
    lds_off[j] = r * St::RS + c * 16;
    lchunk[j] = c;
  }
  const int kend = kbB * 32 * (int)wbytes - 16;  // last 16-byte chunk of the slice
  // A stage's weight chunks and this wave's activation fragments of it are
  // requested together, so waiting for one stage never waits for the
  // other stage's loads (vector loads complete in order); a block past the
  // slice re-reads the slice's last block and is not multiplied.
  auto gload_w = [&](uint4 (&R)[St::NLD], int st) {
#pragma unroll
    for (int j = 0; j < St::NLD; ++j) {
      int off = kb0(st) * 32 * (int)wbytes + lchunk[j] * 16;
      off = off < kend ? off : kend;
      R[j] = ldg_nt(lrow[j] + off);
    }
  };
  auto gload_a = [&](uint4 (&A)[BPW][2], int st) {
#pragma unroll
    for (int j = 0; j < BPW; ++j) {
      const int block = min(kb0(st) + wid + kGWaves * j, kbB - 1);
      A[j][0] = ldg(actp + vk_lo<WFMT>(block * 32, kh));
      A[j][1] = ldg(actp + vk_hi<WFMT>(block * 32, kh));
    }
  };
  auto stage = [&](const uint4 (&R)[St::NLD]) {
    __syncthreads();  // every wave is done with the previous stage
#pragma unroll
    for (int j = 0; j < St::NLD; ++j) {
      const u32x4 w = {R[j].x, R[j].y, R[j].z, R[j].w};
      *(u32x4*)(smem + lds_off[j]) = w;
    }
    __syncthreads();
  };
  // Branch-free: a block past the slice multiplies zeros, so every path
  // through the loop has the same loads in flight and each wait names only
  // the stage it needs.
  auto product = [&](int st, const uint4 (&A)[BPW][2]) {
#pragma unroll
    for (int j = 0; j < BPW; ++j) {
      const int wb = wid + kGWaves * j;
      const bool live = col_live && kb0(st) + wb < kbB;
      VFrag<WFMT, T> f;
#pragma unroll
      for (int t = 0; t < T; ++t)
        frag_lds<WFMT>(smem + (t * 32 + rl) * St::RS, wb, kh, f.wa[t], f.wb[t]);
      f.ba = __builtin_bit_cast(bf16x8, A[j][0]);
      f.bb = __builtin_bit_cast(bf16x8, A[j][1]);
      vmma(f, live, acc);
    }
  };
  // One stage: its weights go to LDS, the register set is refilled with the
  // weights kVNB stages ahead before the product (so kVNB stages stay in
  // flight through it), and the activation fragments after it.  Loads past
  // the slice re-read its last chunk.
  auto step = [&](uint4 (&R)[St::NLD], uint4 (&A)[BPW][2], int st) {
    stage(R);
    __builtin_amdgcn_sched_barrier(0);
    gload_w(R, st + kVNB);
    __builtin_amdgcn_sched_barrier(0);
    product(st, A);
    __builtin_amdgcn_sched_barrier(0);
    gload_a(A, st + kVNB);
    __builtin_amdgcn_sched_barrier(0);
  };
  if (nst > 0) {
    static_assert(kVNB == 2, "two register sets");
    uint4 R0[St::NLD], R1[St::NLD];
    uint4 A0[BPW][2], A1[BPW][2];
    gload_w(R0, 0);
    gload_a(A0, 0);
    gload_w(R1, 1);
    gload_a(A1, 1);
    int st = 0;
    for (; st + kVNB < nst; st += kVNB) {
      step(R0, A0, st);
      step(R1, A1, st + 1);
    }
    stage(R0);
    product(st, A0);
    if (st + 1 < nst) {
      stage(R1);
      product(st + 1, A1);
    }
  }
  __syncthreads();  // the stage buffer becomes the partial-tile buffer
  vred_put<T>(red, wid, rl, kh, col_live, acc);
  if (EPI != EPI_RESID) vnorm_finish(a, wid, lane, ssp, inv_s);

  // Thread -> verify row r, output column n (one row per wave and pass).  The
  // inputs of the residual epilogue are requested before the sums.
  const int M = a.M;
  constexpr int NI = (64 * kMaxRows + kGBlock - 1) / kGBlock;
  float v[NI], xn[NI], gn[NI], sc[NI];
#pragma unroll
  for (int it = 0; it < NI; ++it) {
    if (it * kGBlock >= 64 * M) break;
    const int e = min(tid + it * kGBlock, 64 * M - 1), r = e / 64;
    const int n = min((int)blockIdx.x * 64 + e % 64, a.N - 1);
    if constexpr (EPI == EPI_RESID) {
      xn[it] = a.out[(size_t)r * a.ldo + n];
      gn[it] = bf16_to_f32(a.g_next[n]);
    }
    if constexpr (WFMT == AIO_WFMT_INT8) sc[it] = fp16_to_f32(a.s0[n]);
  }
  __syncthreads();
#pragma unroll
  for (int it = 0; it < NI; ++it) {
    const int e = tid + it * kGBlock, r = e / 64, c = e % 64, n = (int)blockIdx.x * 64 + c;
    if (e >= 64 * M || n >= a.N) break;
    v[it] = vred_sum<T>(red, c / 32, c % 32, r, M);
    if constexpr (EPI != EPI_RESID) v[it] *= inv_s[r];
    if constexpr (WFMT == AIO_WFMT_INT8) v[it] *= sc[it];
    if constexpr (EPI == EPI_RESID) {
      // K split over workgroups: each slice stores its part of the product;
      // the slice that arrives last adds them in slice order
      if (a.ks > 1) st_agent(a.part + ((size_t)blockIdx.y * M + r) * a.ldo + n, v[it]);
    } else {
      a.out[(size_t)r * a.ldo + n] = v[it];
    }
  }
  if constexpr (EPI == EPI_RESID) {
    const int nt = a.N / 64;
    float pv[NI][kVerifyMaxKs];
    if (a.ks > 1) {
      // every wave's part stores have completed (written through) before
      // the slice is counted; the last slice to arrive (in whatever order)
      // then reads the others' parts, which the count shows are in memory
      __builtin_amdgcn_s_waitcnt(0);
      __syncthreads();
      if (tid == 0) last_s = atomic_add_agent(a.cnt + blockIdx.x, 1) == a.ks - 1;
      __syncthreads();
      if (!last_s) return;
      if (tid == 0) atomic_store_agent(a.cnt + blockIdx.x, 0);  // ready for the next product
      // every slot is requested before the first is added (slots past ks
      // read slot 0 and add nothing)
#pragma unroll
      for (int it = 0; it < NI; ++it) {
        if (it * kGBlock >= 64 * M) break;
        const int e = min(tid + it * kGBlock, 64 * M - 1), r = e / 64;
        const int n = (int)blockIdx.x * 64 + e % 64;
#pragma unroll
        for (int k = 0; k < kVerifyMaxKs; ++k)
          pv[it][k] = ld_agent(a.part + ((size_t)(k < a.ks ? k : 0) * M + r) * a.ldo + n);
      }
    }
#pragma unroll
    for (int it = 0; it < NI; ++it) {
      const int e = tid + it * kGBlock, r = e / 64, n = (int)blockIdx.x * 64 + e % 64;
      if (e >= 64 * M) break;  // (whole waves)
      float x = xn[it];
      if (a.ks > 1) {
#pragma unroll
        for (int k = 0; k < kVerifyMaxKs; ++k)
          if (k < a.ks) x += pv[it][k];
      } else {
        x += v[it];
      }
      a.out[(size_t)r * a.ldo + n] = x;
      store_split(a.act_next, a.lda, M, r, n, x * gn[it]);
      const float sq = wave_sum_sq(x);
      if (lane == 0) a.ss_out[(size_t)r * nt + blockIdx.x] = sq;
    }
  }
}

// The QKV product and, behind all but a short cache (kOrderKeys), gate/up: outputs
// in pairs of weight rows (QKV: rows ii and ii + hd / 2 of a head section, SWIGLU:
// the same row of gate and up).  Workgroup b owns the np pairs from np b: as many
// as spread the product evenly over the CUs, up to 64, so every CU streams the same
// bytes in one workgroup.  Measured (7B: 9 rows at 2048, 1B: 3 rows at 1531), in us:
// gate/up against k_vgemm_sk 7B bf16 (43 pairs) 38.2 -> 34.0, int8 27.0 -> 23.3, 1B
// (22 pairs) 15.3 -> 11.1; QKV of the 1B (8 pairs; 32 before, on 64 CUs) 10.8 ->
// 7.7.  Other np (22 to 64) were within 3 % or slower.
//   QKV starts its K stages by the block of 32 pairs that a workgroup begins in (7B
// bf16, 24 pairs: 20.1 us; by its own index 22.5).  Behind a short cache it takes a
// power of two of pairs, at most 32, and so lies in one block: the sums are the same
// whatever np (32 pairs in place of 24 on the 7B: bf16 23.0 us, int8 16.4 for 15.6).
//
// As in k_vgemm, the weights pass through LDS in stages of 256 k, with NS
// stages in flight in registers, and wave w multiplies 32-k block w of every
// stage; NB blocks of 32 pairs (rows past np hold whatever the buffer held:
// each row of the result depends on its own weight row only), NLD 16-byte
// loads per thread and stage.
template <int WFMT, int NB, int NLD, int NS>
struct VPair {
  static constexpr int T = 2 * NB;                              // 32-row tiles
  static constexpr int Lds = vgemm_lds<WFMT, T>(32 * T);
  static constexpr int RPL = kGBlock / VStage<WFMT>::CPR;       // rows a load slot covers
  static constexpr int Pairs = NLD * RPL / 2;                   // most pairs
  static constexpr int NI = (2 * Pairs * kMaxRows + kGBlock - 1) / kGBlock;  // sums per thread
};

template <int WFMT, int EPI, int NB, int NLD, int NS>
__global__ __launch_bounds__(kGBlock, 1) void k_vpair(VGemmArgs a) {
  static_assert(EPI == EPI_QKV || EPI == EPI_SWIGLU, "products of row pairs");
  using St = VStage<WFMT>;
  using Vp = VPair<WFMT, NB, NLD, NS>;
  constexpr int T = Vp::T, BPW = St::BPW;
  static_assert(BPW == 1, "one block per wave and stage");
  extern __shared__ __align__(16) char smem[];
  float* red = (float*)smem;
  __shared__ float inv_s[kMaxRows];
  const int tid = threadIdx.x, lane = tid & (AIO_WAVE - 1), wid = tid / AIO_WAVE;
  const int rl = lane & 31, kh = lane >> 5;
  constexpr int wbytes = WFMT == AIO_WFMT_BF16 ? 2 : 1;
  const int M = a.M;
  const bool col_live = rl < 3 * M;
  const int p0 = (int)blockIdx.x * a.np, np = min(a.np, a.pairs - p0);

  // staging: load j of this thread is chunk lchunk of the row in slot j
  // (slot s < np: the lo row of pair p0 + s, then the hi rows; slots past
  // them repeat the last row)
  const char* lrow[NLD];
  int lds_off[NLD];
  const int lchunk = tid % St::CPR;
#pragma unroll
  for (int j = 0; j < NLD; ++j) {
    const int s = min(j * Vp::RPL + tid / St::CPR, 2 * np - 1);
    const bool hi = s >= np;
    const int p = p0 + (hi ? s - np : s);
    const char* w;
    int n;
    if constexpr (EPI == EPI_QKV) {
      const int half = a.hd / 2, head = p >> (hd_shift(a.hd) - 1);
      const int qrows = a.H * a.hd, krows = a.Hkv * a.hd;
      n = head * a.hd + p - head * half + (hi ? half : 0);
      w = (const char*)a.w0;
      if (n >= qrows + krows) { w = (const char*)a.w2; n -= qrows + krows; }
      else if (n >= qrows) { w = (const char*)a.w1; n -= qrows; }
    } else {
      n = p;
      w = (const char*)(hi ? a.w1 : a.w0);
    }
    lrow[j] = w + (size_t)n * a.K * wbytes;
    lds_off[j] = ((hi ? 32 * NB : 0) + p - p0) * St::RS + lchunk * 16;
  }
  const uint16_t* actp = a.act + (size_t)(col_live ? rl : 0) * a.lda;
  const int nkb = a.K / 32, nst = (nkb + St::BPS - 1) / St::BPS;
  // the stages start at stage b mod nst and wrap (see k_vgemm); b counts blocks of
  // 32 pairs in QKV, workgroups in SWIGLU
  const int rb = EPI == EPI_QKV ? p0 / 32 : (int)blockIdx.x;
  const int rot = rb - udiv(rb, a.by_nst) * nst;
  auto kb0 = [&](int st) {  // first 32-k block of stage st (st < 2 nst)
    const int q = st + rot;
    return (q >= nst ? q - nst : q) * St::BPS;
  };
  const int kend = a.K * wbytes - 16;  // last 16-byte chunk of a row
  auto gload_w = [&](uint4 (&R)[NLD], int st) {
    const int off = min(kb0(min(st, nst - 1)) * 32 * wbytes + lchunk * 16, kend);
#pragma unroll
    for (int j = 0; j < NLD; ++j) R[j] = ldg_nt(lrow[j] + off);
  };
  auto gload_a = [&](uint4 (&A)[2], int st) {
    const int block = min(kb0(min(st, nst - 1)) + wid, nkb - 1);
    A[0] = ldg(actp + vk_lo<WFMT>(block * 32, kh));
    A[1] = ldg(actp + vk_hi<WFMT>(block * 32, kh));
  };
  auto stage = [&](const uint4 (&R)[NLD]) {
    __syncthreads();  // every wave is done with the previous stage
#pragma unroll
    for (int j = 0; j < NLD; ++j) {
      const u32x4 w = {R[j].x, R[j].y, R[j].z, R[j].w};
      *(u32x4*)(smem + lds_off[j]) = w;
    }
    __syncthreads();
  };
  f32x16 acc[T];
#pragma unroll
  for (int t = 0; t < T; ++t)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[t][i] = 0.f;
  // branch-free: a block past the end multiplies zeros
  auto product = [&](int st, const uint4 (&A)[2]) {
    const bool live = col_live && kb0(st) + wid < nkb;
    VFrag<WFMT, T> f;
#pragma unroll
    for (int t = 0; t < T; ++t)
      frag_lds<WFMT>(smem + (t * 32 + rl) * St::RS, wid, kh, f.wa[t], f.wb[t]);
    f.ba = __builtin_bit_cast(bf16x8, A[0]);
    f.bb = __builtin_bit_cast(bf16x8, A[1]);
    vmma(f, live, acc);
  };
  uint4 R[NS][NLD], A[NS][2];
#pragma unroll
  for (int i = 0; i < NS; ++i) {
    gload_w(R[i], i);
    gload_a(A[i], i);
  }
  float ssp[2][2];
  vnorm_request(a, wid, lane, ssp);
  // One stage: its weights go to LDS, its register set is refilled with the
  // weights NS stages ahead before the product (so NS stages stay in flight
  // through it), and the activation fragments after it.  Loads past the end
  // re-read the last stage.
  auto step = [&](uint4 (&Rs)[NLD], uint4 (&As)[2], int st) {
    stage(Rs);
    __builtin_amdgcn_sched_barrier(0);
    gload_w(Rs, st + NS);
    __builtin_amdgcn_sched_barrier(0);
    product(st, As);
    __builtin_amdgcn_sched_barrier(0);
    gload_a(As, st + NS);
    __builtin_amdgcn_sched_barrier(0);
  };
  int st = 0;
  for (; st + NS < nst; st += NS) {
#pragma unroll
    for (int i = 0; i < NS; ++i) step(R[i], A[i], st + i);
  }
#pragma unroll
  for (int i = 0; i < NS; ++i) {
    if (st + i >= nst) break;
    stage(R[i]);
    product(st + i, A[i]);
  }
  __syncthreads();  // the stage buffer becomes the partial-tile buffer
  vred_put<T>(red, wid, rl, kh, col_live, acc);
  vnorm_finish(a, wid, lane, ssp, inv_s);
  // Two lanes per pair and verify row, each summing one of the pair's rows.
  PairIn in[Vp::NI];
  const int h = tid & 1;
#pragma unroll
  for (int it = 0; it < Vp::NI; ++it) {
    if (it * kGBlock >= 2 * np * M) break;
    const int e = min((tid + it * kGBlock) >> 1, np * M - 1), r = np == a.np ? udiv(e, a.by_np) : e / np;
    in[it] = vpair_in<WFMT, EPI>(a, p0 + e - r * np, r);
  }
  __syncthreads();
#pragma unroll
  for (int it = 0; it < Vp::NI; ++it) {
    const int e = (tid + it * kGBlock) >> 1;
    if (e >= np * M) break;  // (both lanes of a pair)
    const int r = np == a.np ? udiv(e, a.by_np) : e / np, i = e - r * np;
    const float y = vred_sum<T>(red, h * NB + i / 32, i % 32, r, M) * inv_s[r];
    const float o = __shfl_xor(y, 1, AIO_WAVE);
    if (h == 0) vpair_epi<WFMT, EPI>(a, in[it], p0 + i, r, y, o);
  }
}

// Stream-K form of the gate/up product, behind a short cache (kOrderKeys).  The
// product's units, a tile pair (32 rows of gate and of up) times a stage of 256 k,
// are dealt out in equal contiguous ranges in (tile pair, stage) order, one range
// per workgroup and one workgroup per CU; the register pipeline (two stages in
// flight, as in k_vgemm) runs on across tile pairs.  A tile pair inside the range
// gets its epilogue as soon as its last stage is multiplied; a pair the range
// shares with its neighbours (at most one at each end) keeps its sums in registers
// until the range is done, then writes them through to skpart at its slot (its rank
// among the pair's workgroups) and counts itself in skcnt; the last to arrive adds
// the slots in slot order and runs the epilogue.
constexpr int kSkMaxC = kVerifySkMaxC;  // most workgroups sharing one tile pair

template <int WFMT>
__global__ __launch_bounds__(kGBlock, 1) void k_vgemm_sk(VGemmArgs a) {
  constexpr int T = 2;
  using St = VStage<WFMT>;
  extern __shared__ __align__(16) char smem[];
  float* red = (float*)smem;
  __shared__ float inv_s[kMaxRows];
  __shared__ int last_s[2];
  const int tid = threadIdx.x, lane = tid & (AIO_WAVE - 1), wid = tid / AIO_WAVE;
  const int rl = lane & 31, kh = lane >> 5;
  constexpr int wbytes = WFMT == AIO_WFMT_BF16 ? 2 : 1;
  const int M = a.M;
  const bool col_live = rl < 3 * M;
  static_assert(St::BPW == 1, "one block per wave and stage");
  const int nkb = a.K / 32, nst = (nkb + St::BPS - 1) / St::BPS;
  // range [u0, u1) of workgroup b: b U / G to (b + 1) U / G
  const unsigned G = gridDim.x, gb = blockIdx.x;
  const int u0 = (int)(gb * (unsigned)a.each + gb * (unsigned)a.rest / G);
  const int u1 = (int)((gb + 1) * (unsigned)a.each + (gb + 1) * (unsigned)a.rest / G);
  // workgroup whose range holds unit u
  auto owner = [&](int u) { return (int)(((unsigned)(u + 1) * G - 1) / (unsigned)a.units); };

  const uint16_t* actp = a.act + (size_t)(col_live ? rl : 0) * a.lda;
  // staging: load j of this thread is chunk lchunk of stage row j RPL + tid / CPR
  // (row < 32: tile 0, else tile 1, of whichever pair the unit belongs to)
  constexpr int RPL = kGBlock / St::CPR;
  const int lchunk = tid % St::CPR, lrow = tid / St::CPR;
  const int kend = a.K * wbytes - 16;  // last 16-byte chunk of a row
  // loads past the range re-read its last unit (and are not multiplied)
  auto gload_w = [&](uint4 (&R)[St::NLD], int u) {
    const int uu = min(u, u1 - 1), tp = udiv(uu, a.by_nst), s = uu - tp * nst;
    const int off = min(s * St::KC * wbytes + lchunk * 16, kend);
#pragma unroll
    for (int j = 0; j < St::NLD; ++j) {
      const int rr = j * RPL + lrow;
      const char* w = (const char*)(rr >= 32 ? a.w1 : a.w0);
      R[j] = ldg_nt(w + (size_t)(tp * 32 + (rr & 31)) * a.K * wbytes + off);
    }
  };
  auto gload_a = [&](uint4 (&A)[2], int u) {
    const int uu = min(u, u1 - 1), s = uu - udiv(uu, a.by_nst) * nst;
    const int block = min(s * St::BPS + wid, nkb - 1) * 32;
    A[0] = ldg(actp + vk_lo<WFMT>(block, kh));
    A[1] = ldg(actp + vk_hi<WFMT>(block, kh));
  };
  auto stage = [&](const uint4 (&R)[St::NLD]) {
    __syncthreads();  // every wave is done with the previous stage
#pragma unroll
    for (int j = 0; j < St::NLD; ++j) {
      const u32x4 w = {R[j].x, R[j].y, R[j].z, R[j].w};
      *(u32x4*)(smem + (j * RPL + lrow) * St::RS + lchunk * 16) = w;
    }
    __syncthreads();
  };
  f32x16 acc[T];
  auto zero_acc = [&]() {
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[t][i] = 0.f;
  };
  // branch-free: a block past the end multiplies zeros
  auto product = [&](int u, const uint4 (&A)[2]) {
    const int s = u - udiv(u, a.by_nst) * nst;
    VFrag<WFMT, T> f;
#pragma unroll
    for (int t = 0; t < T; ++t)
      frag_lds<WFMT>(smem + (t * 32 + rl) * St::RS, wid, kh, f.wa[t], f.wb[t]);
    f.ba = __builtin_bit_cast(bf16x8, A[0]);
    f.bb = __builtin_bit_cast(bf16x8, A[1]);
    vmma(f, col_live && s * St::BPS + wid < nkb, acc);
  };

  uint4 R[2][St::NLD], A[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    gload_w(R[i], u0 + i);
    gload_a(A[i], u0 + i);
  }
  float ssp[2][2];
  vnorm_request(a, wid, lane, ssp);
  vnorm_finish(a, wid, lane, ssp, inv_s);  // (published by the first stage's barriers)
  const int er = tid / 32, ei = tid % 32;  // this thread's epilogue element
  // the range's shared tile pairs: [0] the one it starts in, [1] the one it ends in
  // (-1: none), and this thread's sums of them
  int ptp[2] = {-1, -1};
  float py[2][T] = {{0.f, 0.f}, {0.f, 0.f}};
  auto finish = [&](int tp, float y0, float y1) {
    const int p = tp * 32 + ei;
    vpair_epi<WFMT, EPI_SWIGLU>(a, vpair_in<WFMT, EPI_SWIGLU>(a, p, er), p, er, y0 * inv_s[er],
                                y1 * inv_s[er]);
  };
  zero_acc();
  // After the product of unit u: if u ends a segment (the last unit of a tile pair
  // or of the range), sum it over the waves and finish or keep it.
  auto seg_end = [&](int u) {
    const int tp = udiv(u, a.by_nst);
    if (u + 1 != u1 && u + 1 != (tp + 1) * nst) return;
    __syncthreads();  // the stage buffer becomes the partial-tile buffer
    vred_put<T>(red, wid, rl, kh, col_live, acc);
    __syncthreads();
    zero_acc();
    float y[T] = {0.f, 0.f};
    if (tid < 32 * M) {
#pragma unroll
      for (int t = 0; t < T; ++t) y[t] = vred_sum<T>(red, t, ei, er, M);
    }
    // (the next stage() starts with a barrier: every read is done before it writes)
    const bool head = u0 > tp * nst;  // the segment starts inside the pair
    if (!head && u + 1 == (tp + 1) * nst) {
      if (tid < 32 * M) finish(tp, y[0], y[1]);
    } else if (head || tp * nst == u0) {
      ptp[0] = tp;
      py[0][0] = y[0];
      py[0][1] = y[1];
    } else {
      ptp[1] = tp;
      py[1][0] = y[0];
      py[1][1] = y[1];
    }
  };
  auto step = [&](uint4 (&Rs)[St::NLD], uint4 (&As)[2], int u) {
    stage(Rs);
    __builtin_amdgcn_sched_barrier(0);
    gload_w(Rs, u + 2);
    __builtin_amdgcn_sched_barrier(0);
    product(u, As);
    __builtin_amdgcn_sched_barrier(0);
    gload_a(As, u + 2);
    __builtin_amdgcn_sched_barrier(0);
    seg_end(u);
  };
  int u = u0;
  for (; u + 2 <= u1; u += 2) {
    step(R[0], A[0], u);
    step(R[1], A[1], u + 1);
  }
  if (u < u1) {
    stage(R[0]);
    product(u, A[0]);
    seg_end(u);
  }

  // shared tile pairs: write the sums through, count, and the last of the pair's
  // workgroups adds the slots in order and finishes it
  if (ptp[0] < 0 && ptp[1] < 0) return;
  int ncon[2] = {0, 0};
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    if (ptp[p] < 0) continue;
    const int first = ptp[p] * nst, g0 = owner(first);
    ncon[p] = owner(first + nst - 1) - g0 + 1;
    if (tid < 32 * M) {
      float* dst = a.skpart + ((size_t)ptp[p] * kSkMaxC + (gb - g0)) * (kMaxRows * 64) + er * 64 + ei;
      st_agent(dst, py[p][0]);
      st_agent(dst + 32, py[p][1]);
    }
  }
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  if (tid == 0) {
#pragma unroll
    for (int p = 0; p < 2; ++p)
      last_s[p] = ptp[p] >= 0 && atomic_add_agent(a.skcnt + ptp[p], 1) == ncon[p] - 1;
  }
  __syncthreads();
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    if (!last_s[p]) continue;
    if (tid == 0) atomic_store_agent(a.skcnt + ptp[p], 0);  // ready for the next product
    if (tid < 32 * M) {
      const float* src = a.skpart + (size_t)ptp[p] * kSkMaxC * (kMaxRows * 64) + er * 64 + ei;
      float v0[kSkMaxC], v1[kSkMaxC];
#pragma unroll
      for (int k = 0; k < kSkMaxC; ++k) {
        const int kk = k < ncon[p] ? k : 0;
        v0[k] = ld_agent(src + (size_t)kk * (kMaxRows * 64));
        v1[k] = ld_agent(src + (size_t)kk * (kMaxRows * 64) + 32);
      }
      float y0 = 0.f, y1 = 0.f;
#pragma unroll
      for (int k = 0; k < kSkMaxC; ++k)
        if (k < ncon[p]) {
          y0 += v0[k];
          y1 += v1[k];
        }
      finish(ptp[p], y0, y1);
    }
  }
}

// ------------------------------------------------------- causal attention

struct VAttnArgs {
  const float* q;       // [M][H*hd]
  const uint16_t* kc;   // [Hkv][max_ctx][hd]
  const uint16_t* vc;
  float* part_o;        // [M][H][S][hd]
  float* part_ml;       // [M][H][S][2]
  int pos;              // position of the first row
  int H, Hkv, max_ctx, S, M;
  int blocks, more;     // key blocks per split, and how many splits take one more
  UDiv by_g;            // query heads per kv head
  float scale_log2;
  // k_vattn_mma: the last split of head h to finish merges the head's
  // splits into act (split o [32][lda]); cnt [H] counts finished splits
  int* cnt;
  uint16_t* act;
  int lda;
};

// Causal attention of the M verify rows on MFMA.  One workgroup of kVAW
// waves per (split s, query head h); the split takes key blocks [kbA, kbB)
// of 32 keys, and wave w the blocks kbA + w, kbA + w + kVAW, ...  The
// products are 16 x 16 x 32 MFMAs (lane l: row or column l % 16 of a tile,
// k = 8 (l / 16) .. + 7 of the operands, rows 4 (l / 16) .. + 3 of the
// result): 16 query columns cover the M <= 10 rows with half the dead work
// of a 32-column tile.  Per block:
//   S^T = K Q^T, two tiles of 16 keys: A = key rows straight from the cache
//     (exact bf16), B = the M queries' three bf16 terms (log2-scaled) from
//     LDS; columns past M multiply zeros.  The three terms accumulate into
//     one tile, so column r of S^T is row r's scores in fp32-level
//     precision.  Lane l holds keys 4 (l / 16) .. + 3 of both tiles;
//   online softmax per query column (causal mask j <= pos + r), the max
//     over a column's four lane groups by two exchanges;
//   O^T += V^T P^T: B = the softmax weights' three bf16 terms straight from
//     registers (k slots 8 g .. 8 g + 7 of lane group g are its own keys of
//     tile 0 then tile 1), A = the value tile (staged in LDS row by row,
//     read back through transposing LDS reads in that key order).
//     (Transposing on the way in, with one 16-bit store per element, put
//     16 lanes on one bank and tripled the kernel's time.)
// The next block's keys and values are requested before the current one is
// multiplied.  Every wave then leaves its (max, sum, output) state of the
// live rows in LDS, and one pass combines the waves in wave order into the
// split's unnormalized state, written to part_o / part_ml; the head's last
// split to finish merges all of them (vattn_merge).
//
// Eight waves, one block each (more where a context needs more splits than
// the CUs or the merge take): the blocks a wave streams one after the other are
// the kernel's critical path, about 2 us each at 2K context.  With the
// weights of the fold computed per wave and a merge of one round trip: 7B, 9
// rows at 2048, 17.5 -> 15.1 us, 1B, 3 rows at 1531, 13.2 -> 10.7.  Up to 256
// positions there is one split with a block per wave.
constexpr int kVAW = 8;
static_assert(kVattnBlocksPerSplit == kVAW, "a key block per wave");

template <int HD>
struct VAttnLds {
  static constexpr int QROW = HD * 2 + 16;                 // bytes per query row of one term
  static constexpr int QR = kMaxRows + 1;                   // query rows per term (+ a zero row)
  static constexpr int QBYTES = 3 * QR * QROW;              // three terms of the M queries
  static constexpr int VROW = HD * 2 + 16;                  // bytes per key row of a value tile
  static constexpr int VBYTES = 32 * VROW;                  // one wave's value tile
  static constexpr int OROW = HD + 1;                       // floats per wave output row
  static constexpr int OBYTES = kVAW * kMaxRows * OROW * 4 + 2 * kVAW * kMaxRows * 4;
  static constexpr int TAIL = kVAW * VBYTES > OBYTES ? kVAW * VBYTES : OBYTES;
  static constexpr int BYTES = QBYTES + TAIL;
};

// Key (within the block) of k slot 8 g + j of the P V product: the softmax
// weight register j of lane group g, keys 4 g .. + 3 of tile 0, then of tile 1.
AIO_DEV int vattn_key(int g, int j) { return 16 * (j >> 2) + 4 * g + (j & 3); }

typedef float f32x4 __attribute__((ext_vector_type(4)));

// Block kb's key fragments (A operand of tile tt: key row 16 tt + l % 16,
// dims 32 c + 8 (l / 16) ..) and value chunks (16 bytes each, row-major);
// keys past n_keys read key 0.
template <int HD>
AIO_DEV void vattn_load(const uint16_t* kbase, const uint16_t* vbase, int kb, int n_keys,
                        int lane, uint4 (&kr)[HD / 16], uint4 (&vr)[32 * HD / 8 / AIO_WAVE]) {
  const int r16 = lane & 15, g = lane >> 4, j0 = kb * 32;
#pragma unroll
  for (int tt = 0; tt < 2; ++tt) {
    const int key = j0 + 16 * tt + r16 < n_keys ? j0 + 16 * tt + r16 : 0;
    const uint16_t* krow = kbase + (size_t)key * HD;
#pragma unroll
    for (int c = 0; c < HD / 32; ++c) kr[tt * (HD / 32) + c] = *(const uint4*)(krow + c * 32 + 8 * g);
  }
#pragma unroll
  for (int it = 0; it < 32 * HD / 8 / AIO_WAVE; ++it) {
    const int f = it * AIO_WAVE + lane, kk = f / (HD / 8), d0 = (f % (HD / 8)) * 8;
    const int vkey = j0 + kk < n_keys ? j0 + kk : 0;
    vr[it] = *(const uint4*)(vbase + (size_t)vkey * HD + d0);
  }
}

// Merge of head h's S <= 64 splits for the M rows (by the split that finished
// last; the others' states are in memory, read past the caches).  The splits'
// (max, sum) pairs of a row, one per lane (of 8 lanes up to eight splits, else
// of a wave), become their weights 2^(m - max m) / sum; every output element
// adds its splits' outputs with them, in split order (a single split's is divided
// by its sum).  The outputs of the
// first eight splits are requested with the pairs, so up to eight splits take
// one round trip.
template <int HD>
AIO_DEV void vattn_merge(const VAttnArgs& a, int h, float (*wts)[64]) {
  constexpr int NT = kVAW * AIO_WAVE, NI = (kMaxRows * HD + NT - 1) / NT;
  const int M = a.M, S = a.S, tid = threadIdx.x, lane = tid & (AIO_WAVE - 1), wid = tid / AIO_WAVE;
  const bool few = S <= 8;
  float mv[2], lv[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    if (few && q > 0) break;
    const int r = min(few ? tid / 8 : wid + kVAW * q, M - 1), sp = few ? tid & 7 : lane;
    const float* ml = a.part_ml + ((size_t)r * a.H + h) * S * 2;
    mv[q] = ld_agent(ml + 2 * min(sp, S - 1));
    lv[q] = ld_agent(ml + 2 * min(sp, S - 1) + 1);
  }
  const float* po[NI];
  float ov[NI][8];
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    if (i * NT >= M * HD) break;
    const int e = min(tid + i * NT, M * HD - 1), r = e / HD;
    po[i] = a.part_o + ((size_t)r * a.H + h) * S * HD + e % HD;
#pragma unroll
    for (int j = 0; j < 8; ++j) ov[i][j] = ld_agent(po[i] + (size_t)min(j, S - 1) * HD);
  }
  if (few) {
    const float m = (tid & 7) < S ? mv[0] : -INFINITY;
    const float mx = group_max8_dpp(m);
    const float w = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m - mx);
    const float l = group_sum_dpp<8>((tid & 7) < S ? w * lv[0] : 0.f);
    if (tid < 8 * M) wts[tid / 8][tid & 7] = S == 1 ? l : (l > 0.f ? w / l : 0.f);
  } else {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int r = wid + kVAW * q;
      const float m = lane < S ? mv[q] : -INFINITY;
      const float mx = wave_max(m);
      const float w = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m - mx);
      const float l = wave_sum(lane < S ? w * lv[q] : 0.f);
      if (r < M) wts[r][lane] = l > 0.f ? w / l : 0.f;
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int e = tid + i * NT, r = e / HD, dim = e % HD;
    if (e >= M * HD) break;
    float o = 0.f;
    if (S == 1) {
      const float l = wts[r][0];
      o = l > 0.f ? ov[i][0] / l : 0.f;
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (j < S) o += ov[i][j] * wts[r][j];
    }
    for (int s0 = 8; s0 < S; s0 += 8) {
      float x[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) x[j] = ld_agent(po[i] + (size_t)min(s0 + j, S - 1) * HD);
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (s0 + j < S) o += x[j] * wts[r][s0 + j];
    }
    store_split(a.act, a.lda, M, r, h * HD + dim, o);
  }
}

template <int HD>
__global__ __launch_bounds__(kVAW * AIO_WAVE, 1) void k_vattn_mma(VAttnArgs a) {
  using Lds = VAttnLds<HD>;
  extern __shared__ __align__(16) char smem[];
  char* qs = smem;                  // [3][QR][QROW]; row kMaxRows of each term is zero
  char* tail = smem + Lds::QBYTES;  // per wave: value tile; at the end: the waves' states
  const int tid = threadIdx.x, lane = tid & (AIO_WAVE - 1), wid = tid / AIO_WAVE;
  const int col = lane & 15, g = lane >> 4;  // query column, lane group
  const int s = blockIdx.x, h = blockIdx.y, M = a.M;
  const int kvh = udiv(h, a.by_g);
  const int pos = a.pos;
  const int n_keys = pos + M;  // the last row sees keys [0, pos + M - 1]
  const int kbA = s * a.blocks + min(s, a.more), kbB = kbA + a.blocks + (s < a.more);

  const uint16_t* kbase = a.kc + (size_t)kvh * a.max_ctx * HD;
  const uint16_t* vbase = a.vc + (size_t)kvh * a.max_ctx * HD;
  constexpr int NDT = HD / 16;           // 16-dim tiles of the output
  constexpr int NCH = HD / 32;           // 32-dim chunks of a key row
  constexpr int NVL = 32 * HD / 8 / AIO_WAVE;  // 16-byte value chunks per lane
  // The queries are requested first, then the wave's first key block:
  // loads complete in order, so waiting for the queries leaves the block in
  // flight.
  constexpr int NT = kVAW * AIO_WAVE;
  constexpr int NQ = (kMaxRows * HD + NT - 1) / NT;
  float qv[NQ];
#pragma unroll
  for (int i = 0; i < NQ; ++i) {
    const int e = tid + i * NT, qq = e / HD, dim = e % HD;
    qv[i] = e < M * HD ? a.q[(size_t)qq * a.H * HD + (size_t)h * HD + dim] : 0.f;
  }
  uint4 kr[2 * NCH], vr[NVL];
  int kb = kbA + wid;
  vattn_load<HD>(kbase, vbase, max(min(kb, kbB - 1), 0), n_keys, lane, kr, vr);

  // queries, scaled to log2 units and split into three bf16 terms
#pragma unroll
  for (int i = 0; i < NQ; ++i) {
    const int e = tid + i * NT, qq = e / HD, dim = e % HD;
    if (e < M * HD) {
      uint16_t t0, t1, t2;
      split3(qv[i] * a.scale_log2, t0, t1, t2);
      *(uint16_t*)(qs + (0 * Lds::QR + qq) * Lds::QROW + dim * 2) = t0;
      *(uint16_t*)(qs + (1 * Lds::QR + qq) * Lds::QROW + dim * 2) = t1;
      *(uint16_t*)(qs + (2 * Lds::QR + qq) * Lds::QROW + dim * 2) = t2;
    }
  }
  for (int e = tid; e < 3 * HD; e += NT)
    *(uint16_t*)(qs + ((e / HD) * Lds::QR + kMaxRows) * Lds::QROW + (e % HD) * 2) = 0;
  __syncthreads();

  // this lane's query column col: row col sees keys [0, lim]
  const bool live = col < M;
  const int lim = pos + (live ? col : M - 1);
  // columns past the M rows read the zero row: their columns of S^T are zero
  const char* qrow = qs + (live ? col : kMaxRows) * Lds::QROW;
  char* vt = tail + wid * Lds::VBYTES;
  // transposing reads of the value tile: this lane's address serves key 4 g +
  // e (and 16 + ..) and dims 4 q .. + 3 of a 16-dim tile
  const char* vtr = vt + (4 * g + col / 4) * Lds::VROW + (col & 3) * 8;
  f32x4 o[NDT];
#pragma unroll
  for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
    for (int i = 0; i < 4; ++i) o[dt][i] = 0.f;
  float m = -INFINITY, lsum = 0.f;

  for (; kb < kbB; kb += kVAW) {
    const int j0 = kb * 32;
    // value rows -> LDS (a vector store: a uint4 struct copy is a memcpy,
    // which keeps vr in scratch memory)
#pragma unroll
    for (int it = 0; it < NVL; ++it) {
      const int f = it * AIO_WAVE + lane, kk = f / (HD / 8), d0 = (f % (HD / 8)) * 8;
      const u32x4 w = {vr[it].x, vr[it].y, vr[it].z, vr[it].w};
      *(u32x4*)(vt + kk * Lds::VROW + d0 * 2) = w;
    }
    // scores S^T[key][query] over the HD dims, three query terms, two
    // tiles of 16 keys.  The query fragments of chunk c + 1 are requested
    // before the products of chunk c.
    f32x4 sc[2];
#pragma unroll
    for (int tt = 0; tt < 2; ++tt)
#pragma unroll
      for (int i = 0; i < 4; ++i) sc[tt][i] = 0.f;
    bf16x8 qf[2][3];
#pragma unroll
    for (int t = 0; t < 3; ++t)
      qf[0][t] = as_bf16x8(*(const uint4*)(qrow + t * Lds::QR * Lds::QROW + 8 * g * 2));
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      if (c + 1 < NCH) {
#pragma unroll
        for (int t = 0; t < 3; ++t)
          qf[(c + 1) & 1][t] = as_bf16x8(
              *(const uint4*)(qrow + t * Lds::QR * Lds::QROW + ((c + 1) * 32 + 8 * g) * 2));
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int tt = 0; tt < 2; ++tt) {
        const bf16x8 ak = as_bf16x8(kr[tt * NCH + c]);
#pragma unroll
        for (int t = 0; t < 3; ++t)
          sc[tt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ak, qf[c & 1][t], sc[tt], 0, 0, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    // the next block's keys and values are in flight during the softmax and
    // the P V product (the last block re-reads itself: no branch, so the
    // fragments stay in registers)
    vattn_load<HD>(kbase, vbase, kb + kVAW < kbB ? kb + kVAW : kb, n_keys, lane, kr, vr);
    // causal mask (only a block holding keys past pos needs it; the test is
    // the same for the whole wave) and online softmax for this lane's query
    // column; register j = 4 tt + v holds key j0 + vattn_key(g, j)
    float sv[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) sv[j] = sc[j >> 2][j & 3];
    if (j0 + 31 > pos) {
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (j0 + vattn_key(g, j) > lim) sv[j] = -INFINITY;
    }
    float mx = sv[0];
#pragma unroll
    for (int j = 1; j < 8; ++j) mx = fmaxf(mx, sv[j]);
    mx = fmaxf(mx, __shfl_xor(mx, 16, AIO_WAVE));
    mx = fmaxf(mx, __shfl_xor(mx, 32, AIO_WAVE));
    const float mnew = fmaxf(m, mx);
    // while every key so far is masked, mnew is -inf: subtract 0 instead, so
    // exp2(-inf - 0) = 0 gives the zero weights (and o, lsum stay 0)
    const float mref = mnew == -INFINITY ? 0.f : mnew;
    const float cf = __builtin_amdgcn_exp2f(m - mref);
    float p[8];
    float ps = 0.f;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      p[j] = __builtin_amdgcn_exp2f(sv[j] - mref);
      ps += p[j];
    }
    lsum = lsum * cf + ps;
    m = mnew;
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
      for (int i = 0; i < 4; ++i) o[dt][i] *= cf;
    // the weights split by truncation: t0 = the top 16 bits of p, t1 those
    // of p - t0, t2 = p - t0 - t1 (exact: 8 significant bits each, 24 in
    // all), without the rounding's branches
    bf16x8 bp[3];
    {
      uint32_t tt[3][8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const uint32_t u0 = __float_as_uint(p[e]) & 0xffff0000u;
        const float r1 = p[e] - __uint_as_float(u0);
        const uint32_t u1 = __float_as_uint(r1) & 0xffff0000u;
        const float r2 = r1 - __uint_as_float(u1);
        tt[0][e] = u0;
        tt[1][e] = u1;
        tt[2][e] = __float_as_uint(r2);
      }
#pragma unroll
      for (int t = 0; t < 3; ++t)
        bp[t] = as_bf16x8(make_uint4((tt[t][0] >> 16) | (tt[t][1] & 0xffff0000u),
                                     (tt[t][2] >> 16) | (tt[t][3] & 0xffff0000u),
                                     (tt[t][4] >> 16) | (tt[t][5] & 0xffff0000u),
                                     (tt[t][6] >> 16) | (tt[t][7] & 0xffff0000u)));
    }
    wave_lds_sync();  // the value tile is in LDS
    // O^T += V^T P^T per 16-dim tile, three terms of the weights
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt) {
      // V^T fragment: dimension 16 dt + col at this lane group's eight keys
      const uint2 v0 = lds_read_tr16(vtr + dt * 32);
      const uint2 v1 = lds_read_tr16(vtr + 16 * Lds::VROW + dt * 32);
      const bf16x8 av = as_bf16x8(make_uint4(v0.x, v0.y, v1.x, v1.y));
#pragma unroll
      for (int t = 0; t < 3; ++t)
        o[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bp[t], o[dt], 0, 0, 0);
    }
    wave_lds_sync();  // every read of the value tile is done before the next block's writes
  }
  lsum += __shfl_xor(lsum, 16, AIO_WAVE);
  lsum += __shfl_xor(lsum, 32, AIO_WAVE);

  // every wave's state of the live rows -> LDS (over the value tiles)
  __syncthreads();
  float* om = (float*)tail;                    // [kVAW][kMaxRows][OROW] outputs
  float* mm = om + kVAW * kMaxRows * Lds::OROW;  // [kVAW][kMaxRows] max
  float* ll = mm + kVAW * kMaxRows;            // [kVAW][kMaxRows] sum
  if (live) {
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        om[(wid * kMaxRows + col) * Lds::OROW + dt * 16 + 4 * g + v] = o[dt][v];
    if (g == 0) {
      mm[wid * kMaxRows + col] = m;
      ll[wid * kMaxRows + col] = lsum;
    }
  }
  __syncthreads();

  // The split's state of its M rows, written through to memory: (max, sum) in
  // log2 units and the unnormalized output.  Thread 8 r + w gives wave w's weight
  // in row r: 2^(m - max m), with which the waves' outputs are added in wave order;
  // or, for a single split, the two weights of step w of folding them one by one
  // (the state so far by c1, the wave's by c2: 2^ their maxima minus the new
  // maximum), the order that results behind a short cache keep to (for 9 rows of
  // the 7B at 2048 it took 15.7 us, the sum 15.3).
  static_assert(kVAW == 8, "a group of 8 lanes holds a row's waves");
  __shared__ float wts[kMaxRows][64];
  const bool chain = a.S == 1;
  if (tid < 8 * kMaxRows) {
    const int r = tid / 8, w = tid & 7;
    const float mw = r < M ? mm[w * kMaxRows + r] : -INFINITY;
    if (chain) {
      float before = -INFINITY;
#pragma unroll
      for (int j = 0; j < kVAW - 1; ++j)
        if (j < w && r < M) before = fmaxf(before, mm[j * kMaxRows + r]);
      const float after = fmaxf(before, mw);
      wts[r][2 * w] = before == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(before - after);
      wts[r][2 * w + 1] = mw == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mw - after);
      if (w == kVAW - 1 && r < M) st_agent(a.part_ml + ((size_t)r * a.H + h) * 2, after);
    } else {
      const float ms = group_max8_dpp(mw);
      const float wt = mw == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mw - ms);
      const float ls = group_sum_dpp<8>(r < M ? wt * ll[w * kMaxRows + r] : 0.f);
      wts[r][w] = wt;
      if (w == 0 && r < M) {
        float* ml = a.part_ml + (((size_t)r * a.H + h) * a.S + s) * 2;
        st_agent(ml, ms);
        st_agent(ml + 1, ls);
      }
    }
  }
  __syncthreads();
  for (int e = tid; e < M * HD; e += NT) {
    const int r = e / HD, dim = e % HD;
    float os = 0.f;
    if (chain) {
      float ls = 0.f;
#pragma unroll
      for (int w = 0; w < kVAW; ++w) {
        os = fmaf(os, wts[r][2 * w], om[(w * kMaxRows + r) * Lds::OROW + dim] * wts[r][2 * w + 1]);
        ls = fmaf(ls, wts[r][2 * w], ll[w * kMaxRows + r] * wts[r][2 * w + 1]);
      }
      if (dim == 0) st_agent(a.part_ml + ((size_t)r * a.H + h) * 2 + 1, ls);
    } else {
#pragma unroll
      for (int w = 0; w < kVAW; ++w) os += wts[r][w] * om[(w * kMaxRows + r) * Lds::OROW + dim];
    }
    st_agent(a.part_o + (((size_t)r * a.H + h) * a.S + s) * HD + dim, os);
  }
  // count the split; the last of head h's splits to arrive merges them
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  __shared__ int last_s;
  if (tid == 0) last_s = atomic_add_agent(a.cnt + h, 1) == a.S - 1;
  __syncthreads();
  if (!last_s) return;
  if (tid == 0) atomic_store_agent(a.cnt + h, 0);  // ready for the next layer
  vattn_merge<HD>(a, h, wts);
}

// Launch with `blocks` tile pairs.  A residual-add product with fewer tile
// pairs than CUs also splits K over workgroups, as far as every wave keeps
// at least two blocks of 32 k (at most kVerifyMaxKs slices); the others run
// one K slice per workgroup.  Split slices store their products in the vpart
// region and count themselves in vcnt.
template <int EPI>
hipError_t launch_vgemm(const aio_model& m, const VGemmArgs& g, int blocks) {
  VGemmArgs a = g;
  a.ks = 1;
  a.nt = m.cfg.d_model / 64;
  a.eps = m.cfg.rms_eps;
  if (EPI == EPI_RESID) {
    const int nkb = a.K / 32;
    while (blocks * a.ks < m.num_cus && 2 * a.ks <= kVerifyMaxKs &&
           nkb / (2 * a.ks * kGWaves) >= 2)
      a.ks *= 2;
    a.part = m.at<float>(m.lay.vpart);
    a.cnt = m.at<int>(m.lay.vcnt);
    a.ss_out = m.at<float>(m.lay.vss);
  } else {
    a.ss_in = m.at<float>(m.lay.vss);
  }
  const dim3 grid(blocks, a.ks);
  if (m.cfg.wfmt == AIO_WFMT_INT8) {
    constexpr int lds = vgemm_lds<AIO_WFMT_INT8, 2>(64);
    const hipError_t e = hipFuncSetAttribute((const void*)k_vgemm<AIO_WFMT_INT8, EPI>,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_vgemm<AIO_WFMT_INT8, EPI>), grid, dim3(kGBlock), lds, m.stream, a);
  } else {
    constexpr int lds = vgemm_lds<AIO_WFMT_BF16, 2>(64);
    const hipError_t e = hipFuncSetAttribute((const void*)k_vgemm<AIO_WFMT_BF16, EPI>,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_vgemm<AIO_WFMT_BF16, EPI>), grid, dim3(kGBlock), lds, m.stream, a);
  }
  return hipGetLastError();
}

template <int WFMT, int EPI, int NB, int NLD, int NS>
hipError_t launch_vpair_t(const aio_model& m, const VGemmArgs& a) {
  using Vp = VPair<WFMT, NB, NLD, NS>;
  const void* fn = (const void*)k_vpair<WFMT, EPI, NB, NLD, NS>;
  const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, Vp::Lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_vpair<WFMT, EPI, NB, NLD, NS>), dim3((a.pairs + a.np - 1) / a.np),
                     dim3(kGBlock), Vp::Lds, m.stream, a);
  return hipGetLastError();
}

// Launch of a product of `pairs` row pairs (k_vpair), in as few rounds of one
// workgroup per CU as workgroups of at most 64 pairs allow, each round full; QKV
// behind a short cache takes the least power of two of pairs that makes one round,
// at most 32.  The load slots of a workgroup (16 rows of bf16, 32 of int8) round
// its pairs up; few of them leave registers for more stages in flight.
template <int EPI>
hipError_t launch_vpair(const aio_model& m, const VGemmArgs& g, int pairs) {
  VGemmArgs a = g;
  a.ks = 1;
  a.nt = m.cfg.d_model / 64;
  a.eps = m.cfg.rms_eps;
  a.ss_in = m.at<float>(m.lay.vss);
  a.pairs = pairs;
  if (EPI == EPI_QKV && g.pos + g.M <= kOrderKeys) {
    a.np = 1;
    while (a.np < 32 && a.np * m.num_cus < pairs) a.np *= 2;
  } else {
    const int rounds = (pairs + 64 * m.num_cus - 1) / (64 * m.num_cus);
    a.np = (pairs + rounds * m.num_cus - 1) / (rounds * m.num_cus);
  }
  constexpr int kStageBlocks = VStage<AIO_WFMT_BF16>::BPS;
  static_assert(kStageBlocks == VStage<AIO_WFMT_INT8>::BPS, "one stage length");
  a.by_nst = make_udiv((unsigned)((a.K / 32 + kStageBlocks - 1) / kStageBlocks), (unsigned)pairs);
  a.by_np = make_udiv((unsigned)a.np, (unsigned)(a.np * kMaxRows));
  constexpr int I8 = AIO_WFMT_INT8, BF = AIO_WFMT_BF16;
  if (m.cfg.wfmt == AIO_WFMT_INT8) {
    if (a.np <= 16) return launch_vpair_t<I8, EPI, 1, 1, 4>(m, a);
    if (a.np <= 32) return launch_vpair_t<I8, EPI, 1, 2, 2>(m, a);
    if (a.np <= 48) return launch_vpair_t<I8, EPI, 2, 3, 2>(m, a);
    return launch_vpair_t<I8, EPI, 2, 4, 2>(m, a);
  }
  if (a.np <= 8) return launch_vpair_t<BF, EPI, 1, 1, 4>(m, a);
  if (a.np <= 16) return launch_vpair_t<BF, EPI, 1, 2, 4>(m, a);
  if (a.np <= 24) return launch_vpair_t<BF, EPI, 1, 3, 2>(m, a);
  if (a.np <= 32) return launch_vpair_t<BF, EPI, 1, 4, 2>(m, a);
  if (a.np <= 48) return launch_vpair_t<BF, EPI, 2, 6, 2>(m, a);
  return launch_vpair_t<BF, EPI, 2, 8, 2>(m, a);
}

// Stream-K launch of the gate/up product of `tiles` tile pairs: one workgroup per
// CU, but every range at least `per` units long, so that at most kSkMaxC - 1
// ranges meet in one tile pair (a pair of nst units spans at most 1 + ceil((nst -
// 1) / per) ranges).
hipError_t launch_vgemm_sk(const aio_model& m, const VGemmArgs& g, int tiles) {
  VGemmArgs a = g;
  a.ks = 1;
  a.nt = m.cfg.d_model / 64;
  a.eps = m.cfg.rms_eps;
  a.ss_in = m.at<float>(m.lay.vss);
  a.skpart = m.at<float>(m.lay.skpart);
  a.skcnt = m.at<int>(m.lay.skcnt);
  if ((size_t)tiles > m.lay.sk_tiles) return hipErrorInvalidValue;
  constexpr int kStageBlocks = VStage<AIO_WFMT_BF16>::BPS;
  const int nst = (a.K / 32 + kStageBlocks - 1) / kStageBlocks;
  // (at most 2048 pairs of 256 stages and AIO_STEP_MAX_BLOCKS workgroups: the
  // kernel's products of units and workgroups fit 32 bits)
  a.units = tiles * nst;
  const int per = std::max(2, (nst - 1 + kSkMaxC - 3) / (kSkMaxC - 2));
  const int blocks =
      std::max(1, std::min(std::min(m.num_cus, AIO_STEP_MAX_BLOCKS), a.units / per));
  a.each = a.units / blocks;
  a.rest = a.units % blocks;
  a.by_nst = make_udiv((unsigned)nst, (unsigned)a.units);
  const bool i8 = m.cfg.wfmt == AIO_WFMT_INT8;
  const void* fn = i8 ? (const void*)k_vgemm_sk<AIO_WFMT_INT8> : (const void*)k_vgemm_sk<AIO_WFMT_BF16>;
  const int lds = i8 ? vgemm_lds<AIO_WFMT_INT8, 2>(64) : vgemm_lds<AIO_WFMT_BF16, 2>(64);
  const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  if (e != hipSuccess) return e;
  if (i8)
    hipLaunchKernelGGL(k_vgemm_sk<AIO_WFMT_INT8>, dim3(blocks), dim3(kGBlock), lds, m.stream, a);
  else
    hipLaunchKernelGGL(k_vgemm_sk<AIO_WFMT_BF16>, dim3(blocks), dim3(kGBlock), lds, m.stream, a);
  return hipGetLastError();
}

// Split of x * g and chunk sums of squares for the M rows of x (layer 0:
// x is first set to the embedding rows).
hipError_t launch_vnorm(const aio_model& m, float* x, const uint16_t* embed, const void* gain,
                        uint16_t* act, int M) {
  VNormArgs n{};
  n.x = x;
  n.embed = embed;
  n.gain = (const uint16_t*)gain;
  n.act = act;
  n.lda = m.lay.ka;
  n.d = m.cfg.d_model;
  n.M = M;
  n.ss = m.at<float>(m.lay.vss);
  n.st = m.state();
  hipLaunchKernelGGL(k_vnorm, dim3(M), dim3(kNormBlock), 0, m.stream, n);
  return hipGetLastError();
}

template <int HD>
hipError_t launch_vattn_mma(const aio_model& m, const VAttnArgs& t) {
  constexpr int lds = VAttnLds<HD>::BYTES;
  const hipError_t e = hipFuncSetAttribute((const void*)k_vattn_mma<HD>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_vattn_mma<HD>, dim3(t.S, t.H), dim3(kVAW * AIO_WAVE), lds, m.stream, t);
  return hipGetLastError();
}

}  // namespace

hipError_t aio_launch_verify(const aio_model& m, int M, int pos, float* logits,
                             bool last_row_only) {
  const aio_config& c = m.cfg;
  const int d = c.d_model, H = c.n_heads, Hkv = c.n_kv_heads, hd = c.head_dim, F = c.ffn_dim;
  const int ka = m.lay.ka;
  // two split-activation buffers: A feeds the QKV / gate-up / LM-head GEMMs,
  // B feeds the O / down GEMMs.
  uint16_t* actA = m.at<uint16_t>(m.lay.act);
  uint16_t* actB = actA + (size_t)32 * ka;
  float* x = m.at<float>(m.lay.x);
  float* q = m.at<float>(m.lay.q);
  hipError_t e = launch_vnorm(m, x, (const uint16_t*)m.embed, m.layers[0].attn_norm, actA, M);
  if (e != hipSuccess) return e;
  for (int l = 0; l < c.n_layers; ++l) {
    const aio_layer_weights& L = m.layers[(size_t)l];
    const void* g_after = l + 1 < c.n_layers ? m.layers[(size_t)l + 1].attn_norm : m.final_norm;

    VGemmArgs g{};
    g.act = actA; g.lda = ka; g.M = M;
    g.w0 = L.wq; g.w1 = L.wk; g.w2 = L.wv;
    g.s0 = (const uint16_t*)L.sq; g.s1 = (const uint16_t*)L.sk; g.s2 = (const uint16_t*)L.sv;
    g.N = (H + 2 * Hkv) * hd; g.K = d;
    g.out = q; g.ldo = H * hd;
    g.kc = m.kv_layer(l, 0); g.vc = m.kv_layer(l, 1);
    g.rope = m.rope; g.pos = pos;
    g.H = H; g.Hkv = Hkv; g.hd = hd; g.max_ctx = c.max_ctx;
    if ((e = launch_vpair<EPI_QKV>(m, g, (H + 2 * Hkv) * (hd / 2))) != hipSuccess) return e;

    VAttnArgs t{};
    t.q = q; t.kc = g.kc; t.vc = g.vc;
    t.part_o = m.at<float>(m.lay.part_o);
    t.part_ml = m.at<float>(m.lay.part_ml);
    t.pos = pos;
    t.H = H; t.Hkv = Hkv; t.max_ctx = c.max_ctx; t.S = m.lay.splits; t.M = M;
    t.scale_log2 = (float)(1.4426950408889634 / sqrt((double)hd));
    // splits of kVattnBlocksPerSplit key blocks, but no more workgroups than
    // CUs: a workgroup takes a whole CU, and a second round of workgroups
    // pays the queries' prologue and the merges again (at 32K, 64 splits per
    // head cost 9.2 ms per 7B verify).
    const int nkb = (pos + M + 31) / 32;
    const int s_cap = std::max(1, std::min(m.lay.vsplits, m.num_cus / H));
    t.S = std::max(1, std::min(s_cap, (nkb + kVattnBlocksPerSplit - 1) / kVattnBlocksPerSplit));
    t.blocks = nkb / t.S;
    t.more = nkb % t.S;
    t.by_g = make_udiv((unsigned)(H / Hkv), (unsigned)H);
    t.cnt = m.at<int>(m.lay.vacnt);
    t.act = actB;
    t.lda = ka;
    if ((e = hd == 128 ? launch_vattn_mma<128>(m, t) : launch_vattn_mma<64>(m, t)) != hipSuccess)
      return e;

    VGemmArgs o{};
    o.act = actB; o.lda = ka; o.M = M;
    o.w0 = L.wo; o.s0 = (const uint16_t*)L.so;
    o.N = d; o.K = H * hd; o.out = x; o.ldo = d;
    o.g_next = (const uint16_t*)L.ffn_norm; o.act_next = actA;
    if ((e = launch_vgemm<EPI_RESID>(m, o, d / 64)) != hipSuccess) return e;

    VGemmArgs gu{};
    gu.act = actA; gu.lda = ka; gu.M = M;
    gu.w0 = L.w_gate; gu.w1 = L.w_up;
    gu.s0 = (const uint16_t*)L.s_gate; gu.s1 = (const uint16_t*)L.s_up;
    gu.N = F; gu.K = d; gu.act_out = actB; gu.lda_out = ka;
    e = pos + M <= kOrderKeys ? launch_vgemm_sk(m, gu, F / 32) : launch_vpair<EPI_SWIGLU>(m, gu, F);
    if (e != hipSuccess) return e;

    VGemmArgs dn{};
    dn.act = actB; dn.lda = ka; dn.M = M;
    dn.w0 = L.w_down; dn.s0 = (const uint16_t*)L.s_down;
    dn.N = d; dn.K = F; dn.out = x; dn.ldo = d;
    dn.g_next = (const uint16_t*)g_after; dn.act_next = actA;
    if ((e = launch_vgemm<EPI_RESID>(m, dn, d / 64)) != hipSuccess) return e;
  }
  if (last_row_only) {
    // the last row's final RMSNorm and LM head only (a prefill of M tokens)
    if (M > 1 && (e = hipMemcpyAsync(x, x + (size_t)(M - 1) * d, (size_t)d * sizeof(float),
                                     hipMemcpyDeviceToDevice, m.stream)) != hipSuccess)
      return e;
    return aio_launch_lm_rows(m, 1, logits);
  }
  VGemmArgs lm{};
  lm.act = actA; lm.lda = ka; lm.M = M;
  lm.w0 = m.lm_head; lm.s0 = (const uint16_t*)m.s_lm_head;
  lm.N = c.vocab; lm.K = d; lm.out = logits; lm.ldo = c.vocab;
  return launch_vgemm<EPI_STORE>(m, lm, (c.vocab + 63) / 64);
}

hipError_t aio_launch_lm_rows(const aio_model& m, int rows, float* logits) {
  const aio_config& c = m.cfg;
  uint16_t* actA = m.at<uint16_t>(m.lay.act);
  float* x = m.at<float>(m.lay.x);
  hipError_t e = launch_vnorm(m, x, nullptr, m.final_norm, actA, rows);
  if (e != hipSuccess) return e;
  VGemmArgs lm{};
  lm.act = actA; lm.lda = m.lay.ka; lm.M = rows;
  lm.w0 = m.lm_head; lm.s0 = (const uint16_t*)m.s_lm_head;
  lm.N = c.vocab; lm.K = c.d_model; lm.out = logits; lm.ldo = c.vocab;
  return launch_vgemm<EPI_STORE>(m, lm, (c.vocab + 63) / 64);
}
