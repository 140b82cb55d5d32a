// Device building blocks for the message-passing kernels (gfx950, wave64).
//
// Row-block layout.  A wave works on blocks of 16 rows (edges or nodes).
// Lane l handles row j = l % 16 of the block and lane group g = l / 16.  For
// a feature vector of width W (a multiple of 16) the lane holds W/4 values:
//   v[4*b + r]  <->  feature 16*b + 4*g + r      (b < W/16, r < 4)
// so the four lanes of a row together hold the whole row, each lane as W/16
// contiguous float4 chunks.  This is exactly the accumulator layout of the
// 16x16 MFMA instructions when the product is computed transposed
// (output features x rows), which lets the output of one Linear feed the
// next one with no data movement: the K ordering of each product is permuted
// to match, and the weight fragments are packed in that order.
//
// Weight fragments.  A product out[f][row] = sum_k A[f][k] in[k][row] with
// A of shape [M][K] is stored as
//   FP32 (v_mfma_f32_16x16x4f32):  frag[(mb*(K/4) + s)*64 + lane]
//        = A[16*mb + lane%16][16*(s/4) + 4*(lane/16) + s%4]
//   BF16 (v_mfma_f32_16x16x32_bf16): frag16[(mb*(K/32) + t)*64 + lane] =
//        8 values q = 0..7 of A[16*mb + lane%16][32*t + 16*(q/4) + 4*(lane/16) + q%4]
// and the input operand of step s (FP32) is in[s], of step t (BF16) is
// in[8t .. 8t+7], directly in the row-block layout.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mp {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ int lane_id() { return threadIdx.x & 63; }

// ------------------------------------------------------------------ loads

// Load the row-block slice of a W-wide row (ptr = start of the row).
// Lane (j, g) moves features 16b + 4g .. +3, so one instruction covers half
// of each 128-byte line of a row.  All row traffic uses ordinary cached
// loads and stores: L2 then merges the two halves of a line (non-temporal
// stores wrote about 40% more bytes than the arrays hold, and non-temporal
// loads measured slower as well).
template <int W>
__device__ __forceinline__ void load_row(const float* __restrict__ ptr, int g, float (&v)[W / 4]) {
#pragma unroll
  for (int b = 0; b < W / 16; ++b) {
    const float4 t = *reinterpret_cast<const float4*>(ptr + 16 * b + 4 * g);
    v[4 * b + 0] = t.x;
    v[4 * b + 1] = t.y;
    v[4 * b + 2] = t.z;
    v[4 * b + 3] = t.w;
  }
}

template <int W>
__device__ __forceinline__ void store_row(float* __restrict__ ptr, int g, const float (&v)[W / 4]) {
#pragma unroll
  for (int b = 0; b < W / 16; ++b)
    *reinterpret_cast<float4*>(ptr + 16 * b + 4 * g) =
        make_float4(v[4 * b + 0], v[4 * b + 1], v[4 * b + 2], v[4 * b + 3]);
}

// BF16 storage of a row (round to nearest even) and its FP32 read-back.

typedef __bf16 v4bf __attribute__((ext_vector_type(4)));
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
template <int W>
__device__ __forceinline__ void store_row_bf16(__bf16* __restrict__ ptr, int g, const float (&v)[W / 4]) {
#pragma unroll
  for (int b = 0; b < W / 16; ++b) {
    const v4bf t = {(__bf16)v[4 * b], (__bf16)v[4 * b + 1], (__bf16)v[4 * b + 2], (__bf16)v[4 * b + 3]};
    *reinterpret_cast<u32x2*>(ptr + 16 * b + 4 * g) = __builtin_bit_cast(u32x2, t);
  }
}
template <int W>
__device__ __forceinline__ void load_row_bf16(const __bf16* __restrict__ ptr, int g, float (&v)[W / 4]) {
#pragma unroll
  for (int b = 0; b < W / 16; ++b) {
    const v4bf t = __builtin_bit_cast(v4bf, *reinterpret_cast<const u32x2*>(ptr + 16 * b + 4 * g));
    v[4 * b + 0] = (float)t[0];
    v[4 * b + 1] = (float)t[1];
    v[4 * b + 2] = (float)t[2];
    v[4 * b + 3] = (float)t[3];
  }
}

// Row `row` of an [n][W] array stored as FP32 or (BF) BF16.
template <int W, bool BF>
__device__ __forceinline__ void store_row_t(void* __restrict__ base, int64_t row, int g, const float (&v)[W / 4]) {
  if constexpr (BF)
    store_row_bf16<W>(reinterpret_cast<__bf16*>(base) + row * W, g, v);
  else
    store_row<W>(reinterpret_cast<float*>(base) + row * W, g, v);
}
template <int W, bool BF>
__device__ __forceinline__ void load_row_t(const void* __restrict__ base, int64_t row, int g, float (&v)[W / 4]) {
  if constexpr (BF)
    load_row_bf16<W>(reinterpret_cast<const __bf16*>(base) + row * W, g, v);
  else
    load_row<W>(reinterpret_cast<const float*>(base) + row * W, g, v);
}

// Per-feature vector (bias, LayerNorm gain) in row-block layout.
template <int W>
__device__ __forceinline__ void load_vec(const float* __restrict__ p, int g, float (&v)[W / 4]) {
  load_row<W>(p, g, v);
}

// An opaque zero: adding it to an LDS offset inside a loop keeps the
// compiler from hoisting every weight-fragment read out of the loop (which
// would pin the whole matrix in registers and cut occupancy).
__device__ __forceinline__ int opaque_zero() {
  int z = 0;
  asm volatile("" : "+v"(z));
  return z;
}

// ------------------------------------------------------------- GEMMs

// acc[f] += sum_k A[f][k] in[k]  (A packed as FP32 fragments; MB = M/16,
// KB = K/16).  Independent output blocks are interleaved so consecutive
// MFMAs do not depend on each other.
// ROT: the fragments sit in LDS in the rotated layout of stage_frags_rot
// (element o of 64-float chunk c at c*64 + (o + c%4) % 64); chunk
// mb*4KB + s has c%4 = s%4.
template <int MB, int KB, bool ROT = false>
__device__ __forceinline__ void gemm_f32(const float* __restrict__ frag, const float (&in)[4 * KB],
                                         float (&acc)[4 * MB], int lane) {
  v4f c[MB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) c[mb] = v4f{acc[4 * mb], acc[4 * mb + 1], acc[4 * mb + 2], acc[4 * mb + 3]};
#pragma unroll
  for (int s = 0; s < 4 * KB; ++s) {
    const int l = ROT ? ((lane + (s & 3)) & 63) : lane;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
      c[mb] = __builtin_amdgcn_mfma_f32_16x16x4f32(frag[(mb * 4 * KB + s) * 64 + l], in[s], c[mb], 0, 0, 0);
  }
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    acc[4 * mb] = c[mb][0];
    acc[4 * mb + 1] = c[mb][1];
    acc[4 * mb + 2] = c[mb][2];
    acc[4 * mb + 3] = c[mb][3];
  }
}

// acc += W^T in for a square H x H matrix W stored as FP32 fragments (the
// layout gemm_f32 reads for W in).  Fragment element (mb, s, lane i + 16k)
// holds W[16 mb + i][f(s, k)] with f(s, k) = 16 (s/4) + 4k + s%4, the
// feature order of the row-block layout; W^T's element for step s, output
// block mb' and lane (i, k) is W[f(s, k)][16 mb' + i], found at fragment
// (s/4, 4 mb' + i%4, lane 4k + s%4 + 16 (i/4)).  One LDS read per MFMA as
// in gemm_f32, so the transposed matrix need not be stored.  In the packed
// layout the 64 lanes of one read reach only 16 LDS banks (lanes with equal
// i/4 and k but different i%4 read the same bank of four fragments); in the
// rotated layout (ROT) they reach 64 distinct banks.
template <int H, bool ROT = false>
__device__ __forceinline__ void gemm_f32_tr(const float* __restrict__ frag, const float (&in)[H / 4],
                                            float (&acc)[H / 4], int lane) {
  constexpr int MB = H / 16, S = H / 4;
  const int i = lane & 15, k = lane >> 4;
  v4f c[MB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) c[mb] = v4f{acc[4 * mb], acc[4 * mb + 1], acc[4 * mb + 2], acc[4 * mb + 3]};
#pragma unroll
  for (int s = 0; s < S; ++s) {
    // fragment (s/4) S + 4 mb + i%4 (its chunk index is i%4 mod 4), element s%4 + 4k + 16 (i/4)
    const int o = (s & 3) + 4 * k + 16 * (i >> 2);
    const int lane_off = (i & 3) * 64 + (ROT ? ((o + (i & 3)) & 63) : o);
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
      c[mb] = __builtin_amdgcn_mfma_f32_16x16x4f32(frag[((s >> 2) * S + 4 * mb) * 64 + lane_off], in[s], c[mb], 0,
                                                   0, 0);
  }
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    acc[4 * mb] = c[mb][0];
    acc[4 * mb + 1] = c[mb][1];
    acc[4 * mb + 2] = c[mb][2];
    acc[4 * mb + 3] = c[mb][3];
  }
}

// acc += W^T in for an M x K matrix W stored as FP32 fragments (the layout
// gemm_f32 reads for W in): in holds M features, acc K.  The same
// transposed addressing as gemm_f32_tr, with the fragment row-block
// stride of a K-wide matrix (gemm_f32_tr is the case M = K = H).
template <int M, int K, bool ROT = false>
__device__ __forceinline__ void gemm_f32_tr_mk(const float* __restrict__ frag, const float (&in)[M / 4],
                                               float (&acc)[K / 4], int lane) {
  constexpr int MB = K / 16, S = K / 4, STEPS = M / 4;
  const int i = lane & 15, k = lane >> 4;
  v4f c[MB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) c[mb] = v4f{acc[4 * mb], acc[4 * mb + 1], acc[4 * mb + 2], acc[4 * mb + 3]};
#pragma unroll
  for (int s = 0; s < STEPS; ++s) {
    const int o = (s & 3) + 4 * k + 16 * (i >> 2);
    const int lane_off = (i & 3) * 64 + (ROT ? ((o + (i & 3)) & 63) : o);
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
      c[mb] = __builtin_amdgcn_mfma_f32_16x16x4f32(frag[((s >> 2) * S + 4 * mb) * 64 + lane_off], in[s], c[mb], 0,
                                                   0, 0);
  }
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    acc[4 * mb] = c[mb][0];
    acc[4 * mb + 1] = c[mb][1];
    acc[4 * mb + 2] = c[mb][2];
    acc[4 * mb + 3] = c[mb][3];
  }
}

__device__ __forceinline__ v8bf to_bf8(const float* x) {
  v8bf r;
#pragma unroll
  for (int q = 0; q < 8; ++q) r[q] = (__bf16)x[q];  // round to nearest even
  return r;
}

template <int MB, int KB>
__device__ __forceinline__ void gemm_bf16(const uint4* __restrict__ frag, const float (&in)[4 * KB],
                                          float (&acc)[4 * MB], int lane) {
  static_assert(KB % 2 == 0, "BF16 products need K to be a multiple of 32");
  constexpr int T = KB / 2;
  v4f c[MB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) c[mb] = v4f{acc[4 * mb], acc[4 * mb + 1], acc[4 * mb + 2], acc[4 * mb + 3]};
#pragma unroll
  for (int t = 0; t < T; ++t) {
    const v8bf b = to_bf8(&in[8 * t]);
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      const uint4 a = frag[(mb * T + t) * 64 + lane];
      c[mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, a), b, c[mb], 0, 0, 0);
    }
  }
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    acc[4 * mb] = c[mb][0];
    acc[4 * mb + 1] = c[mb][1];
    acc[4 * mb + 2] = c[mb][2];
    acc[4 * mb + 3] = c[mb][3];
  }
}

// ------------------------------- FP32 products on the BF16 matrix unit
//
// An FP32 value is the exact sum of three BF16 parts, x = h + m + l: h its
// upper half, m the rounded remainder, l what then is left (8 + 8 + 8 bits).
// Six of the nine part products give W x: the dropped m*l, l*m and l*l are
// below 2^-23 of |w||x| and symmetric, and the products summed are exact in
// FP32.  The five small ones are summed apart and added once, so the large
// sum takes K/32 roundings instead of the FP32 instruction's K/4: against FP64
// (normal values) the rms error is 5.0e-8 of the result at K = 64 and 3.9e-8 at
// 32, with v_mfma_f32_16x16x4f32 1.44e-7 and 1.03e-7; one product alone is off by
// up to 2.1e-7 (FP32: 6e-8).  With m*l and l*m that would be 6.0e-8, and 4.8e-8 over
// 64 terms: no case measured came nearer to FP64 by them, and the FP32 forward took
// 7%, the width-32 deep layers 13% longer.  The rate: six
// v_mfma_f32_16x16x32_bf16 take 96 cycles for what eight 32-cycle FP32 instructions
// do, and unlike those they issue beside vector instructions.
//
// An infinite operand has no parts: its remainder is inf - inf, so every output
// it reaches is NaN.  The kernels look for one (a NaN among their results, or an
// infinite weight met while staging, stage_wfrag) and then compute those rows
// again with FP32 instructions (mp_exact.hpp), whose infinities are those of FP32
// arithmetic.  Only sums over rows keep the parts' result: a weight gradient with
// an infinite factor is not finite either way.
//
// Op<BF, W>: a W-wide row in the row-block layout as matrix operand; lane
// value q of chunk t is in[8t + q].
template <bool BF, int W>
struct Op;
template <int W>
struct Op<true, W> {
  v8bf h[W / 32];
};
template <int W>
struct Op<false, W> {
  v8bf h[W / 32], m[W / 32], l[W / 32];
};

typedef uint32_t v4u __attribute__((ext_vector_type(4)));

__device__ __forceinline__ void split3_pair(float x0, float x1, uint32_t& h, uint32_t& m, uint32_t& l) {
  const uint32_t b0 = __builtin_bit_cast(uint32_t, x0), b1 = __builtin_bit_cast(uint32_t, x1);
  h = __builtin_amdgcn_perm(b1, b0, 0x07060302);  // upper halves
  float r0 = x0 - __builtin_bit_cast(float, b0 & 0xffff0000u);
  float r1 = x1 - __builtin_bit_cast(float, b1 & 0xffff0000u);
  m = __builtin_bit_cast(uint32_t, v2bf{(__bf16)r0, (__bf16)r1});
  r0 -= __builtin_bit_cast(float, m << 16);
  r1 -= __builtin_bit_cast(float, m & 0xffff0000u);
  l = __builtin_bit_cast(uint32_t, v2bf{(__bf16)r0, (__bf16)r1});
}
__device__ __forceinline__ void split3_8(const float* x, v8bf& h, v8bf& m, v8bf& l) {
  v4u hh, mm, ll;
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    uint32_t a, b, c;
    split3_pair(x[2 * p], x[2 * p + 1], a, b, c);
    hh[p] = a;
    mm[p] = b;
    ll[p] = c;
  }
  h = __builtin_bit_cast(v8bf, hh);
  m = __builtin_bit_cast(v8bf, mm);
  l = __builtin_bit_cast(v8bf, ll);
}

template <int W>
__device__ __forceinline__ void make_op(const float (&x)[W / 4], Op<true, W>& o) {
#pragma unroll
  for (int t = 0; t < W / 32; ++t) o.h[t] = to_bf8(&x[8 * t]);
}
template <int W>
__device__ __forceinline__ void make_op(const float (&x)[W / 4], Op<false, W>& o) {
#pragma unroll
  for (int t = 0; t < W / 32; ++t) split3_8(&x[8 * t], o.h[t], o.m[t], o.l[t]);
}

#define MP_MFMA_BF16(A, B, C) __builtin_amdgcn_mfma_f32_16x16x32_bf16(A, B, C, 0, 0, 0)

// acc += W in over K/32 chunks, W's operand of (chunk t, output block mb) from
// wf(t, mb, part) with part 0, 1, 2 = h, m, l (BF16: part 0 only).
// How a product meets its accumulator: it starts from it (the large part
// products are summed onto it), starts from zero and replaces it, or starts
// from zero and is added at the end times `sc` (one rounding; eight more
// registers).
enum Acc { ACC_START, ACC_SET, ACC_ADD };

template <int MB, int T, Acc MODE, class F>
__device__ __forceinline__ void gemm_op(F&& wf, const Op<true, 32 * T>& in, float (&acc)[4 * MB], float = 1.f) {
  v4f c[MB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
    c[mb] = MODE == ACC_SET ? v4f{0.f, 0.f, 0.f, 0.f}
                            : v4f{acc[4 * mb], acc[4 * mb + 1], acc[4 * mb + 2], acc[4 * mb + 3]};
#pragma unroll
  for (int t = 0; t < T; ++t) {
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) c[mb] = MP_MFMA_BF16(wf(t, mb, 0), in.h[t], c[mb]);
  }
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[4 * mb + r] = c[mb][r];
  }
}
template <int MB, int T, Acc MODE, class F>
__device__ __forceinline__ void gemm_op(F&& wf, const Op<false, 32 * T>& in, float (&acc)[4 * MB], float sc = 1.f) {
  // two output blocks at a time: each weight part is read once, and no two
  // consecutive matrix instructions add to the same registers.  With one chunk
  // the large product comes last on the small ones' sum (one rounding at full
  // size, no second accumulator).  The instruction then cuts the small sum's low
  // bits downwards, a mean error of 2^-27 of a term where two sums leave 2^-33;
  // an adjoint, whose errors add up over millions of rows in the bias gradients,
  // takes its rows by random sign (row_sign), so this one cancels as well (in two
  // sums the width-32 deep layers take 3% longer and are no nearer to FP64).
  constexpr int G = MB % 2 == 0 ? 2 : 1;
  constexpr bool ONE = T == 1;
#pragma unroll
  for (int m0 = 0; m0 < MB; m0 += G) {
    v4f ch[G], cs[G];
#pragma unroll
    for (int i = 0; i < G; ++i) {
      const int mb = m0 + i;
      cs[i] = v4f{0.f, 0.f, 0.f, 0.f};
      ch[i] = MODE == ACC_START ? v4f{acc[4 * mb], acc[4 * mb + 1], acc[4 * mb + 2], acc[4 * mb + 3]} : cs[i];
    }
#pragma unroll
    for (int t = 0; t < T; ++t) {
      v8bf wh[G], wm[G], wl[G];
#pragma unroll
      for (int i = 0; i < G; ++i) {
        wl[i] = wf(t, m0 + i, 2);
        wm[i] = wf(t, m0 + i, 1);
        wh[i] = wf(t, m0 + i, 0);
      }
#pragma unroll
      for (int i = 0; i < G; ++i) cs[i] = MP_MFMA_BF16(wl[i], in.h[t], cs[i]);
#pragma unroll
      for (int i = 0; i < G; ++i) cs[i] = MP_MFMA_BF16(wm[i], in.m[t], cs[i]);
#pragma unroll
      for (int i = 0; i < G; ++i) cs[i] = MP_MFMA_BF16(wh[i], in.l[t], cs[i]);
#pragma unroll
      for (int i = 0; i < G; ++i) cs[i] = MP_MFMA_BF16(wm[i], in.h[t], cs[i]);
      if constexpr (ONE) {
#pragma unroll
        for (int i = 0; i < G; ++i) cs[i] = MP_MFMA_BF16(wh[i], in.m[t], cs[i]);
#pragma unroll
        for (int i = 0; i < G; ++i) cs[i] = MP_MFMA_BF16(wh[i], in.h[t], cs[i]);
      } else {
#pragma unroll
        for (int i = 0; i < G; ++i) ch[i] = MP_MFMA_BF16(wh[i], in.h[t], ch[i]);
#pragma unroll
        for (int i = 0; i < G; ++i) cs[i] = MP_MFMA_BF16(wh[i], in.m[t], cs[i]);
      }
    }
#pragma unroll
    for (int i = 0; i < G; ++i) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float& o = acc[4 * (m0 + i) + r];
        const float v = ONE ? cs[i][r] : ch[i][r] + cs[i][r];
        o = MODE == ACC_ADD ? fmaf(sc, v, o) : ONE && MODE == ACC_START ? o + v : v;
      }
    }
  }
}

// A weight matrix in device memory: element (r, c) at p[r*ld + c], or with
// trans at p[c*ld + r].
struct WView {
  const float* p;
  int ld, trans;
};
// Four consecutive floats, 16-byte aligned (al) or not.
__device__ __forceinline__ float4 load4w(const float* __restrict__ p, bool al) {
  return al ? *reinterpret_cast<const float4*>(p) : make_float4(p[0], p[1], p[2], p[3]);
}
__device__ __forceinline__ bool w_aligned(const WView& w) {
  return (reinterpret_cast<uintptr_t>(w.p) & 15) == 0 && (w.ld & 3) == 0;
}

// Weights in LDS as MFMA fragments: BF16 products one BF16 matrix, FP32
// products its three parts one after the other.  Staged by the kernel itself
// from the FP32 matrix (a few KB per workgroup of a persistent grid, so no
// packing launch is needed before it).  A weight whose upper part would round
// to infinity keeps its upper half instead.
__host__ __device__ constexpr size_t w_bytes(int M, int K, bool bf) { return size_t(M) * K * 2 * (bf ? 1 : 3); }

template <bool BF>
__device__ __forceinline__ void split_w8(const float* x, v8bf& h, v8bf& m, v8bf& l) {
  if constexpr (BF) {
    h = to_bf8(x);
  } else {
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const uint32_t b = __builtin_bit_cast(uint32_t, x[q]);
      __bf16 hq = (__bf16)x[q];
      if ((b & 0x7fffffffu) >= 0x7f7f8000u)
        hq = __builtin_bit_cast(__bf16, (uint16_t)(b >> 16));
      const float r = x[q] - (float)hq;
      const __bf16 mq = (__bf16)r;
      h[q] = hq;
      m[q] = mq;
      l[q] = (__bf16)(r - (float)mq);
    }
  }
}

template <int N>
__device__ __forceinline__ bool any_inf(const float (&x)[N]) {
  bool r = false;
#pragma unroll
  for (int i = 0; i < N; ++i) r |= fabsf(x[i]) == __builtin_inff();
  return r;
}

// Stage the M x K matrix w as fragments: 16-byte piece (mb*(K/32) + t)*64 +
// lane holds A[16 mb + lane%16][32t + 16(q/4) + 4(lane/16) + q%4], q = 0..7;
// the parts M*K*2 bytes apart.  All threads of the workgroup; no barrier.
// Returns whether this thread met an infinite weight (FP32).
template <bool BF, int M, int K>
__device__ __forceinline__ bool stage_wfrag(void* __restrict__ dst, const WView& w) {
  bool odd = false;
  constexpr int T = K / 32;
  uint4* d = reinterpret_cast<uint4*>(dst);
  const bool al = w_aligned(w);
  for (int e = threadIdx.x; e < M * K / 8; e += blockDim.x) {
    const int lane = e % 64, t = (e / 64) % T, mb = e / (64 * T);
    const int row = 16 * mb + lane % 16, col = 32 * t + 4 * (lane / 16);
    float x[8];
    if (!w.trans) {
      const float4 a = load4w(w.p + (int64_t)row * w.ld + col, al);
      const float4 b = load4w(w.p + (int64_t)row * w.ld + col + 16, al);
      x[0] = a.x, x[1] = a.y, x[2] = a.z, x[3] = a.w;
      x[4] = b.x, x[5] = b.y, x[6] = b.z, x[7] = b.w;
    } else {
#pragma unroll
      for (int q = 0; q < 8; ++q) x[q] = w.p[(int64_t)(col + 16 * (q / 4) + q % 4) * w.ld + row];
    }
    v8bf h, m, l;
    split_w8<BF>(x, h, m, l);
    d[e] = __builtin_bit_cast(uint4, h);
    if constexpr (!BF) {
      odd |= any_inf(x);
      d[e + M * K / 8] = __builtin_bit_cast(uint4, m);
      d[e + 2 * (M * K / 8)] = __builtin_bit_cast(uint4, l);
    }
  }
  return odd;
}

// Whether any thread of the workgroup staged an infinite weight: each wave leaves
// its own answer in `slots` (one int per wave), and reads all after the barrier
// that ends the staging.
__device__ __forceinline__ void note_odd(int* __restrict__ slots, bool odd) {
  const uint64_t any = __ballot(odd);
  if ((threadIdx.x & 63) == 0) slots[threadIdx.x / 64] = any != 0;
}
__device__ __forceinline__ bool read_odd(const int* __restrict__ slots) {
  int o = 0;
  for (int w = 0; w < (int)blockDim.x / 64; ++w) o |= slots[w];
  return __builtin_amdgcn_readfirstlane(o) != 0;
}
__device__ __forceinline__ bool any_nan(float x) { return __ballot(x != x) != 0; }

// acc += W in, W staged by stage_wfrag.
template <bool BF, int M, int K>
__device__ __forceinline__ void gemm_wf(const void* __restrict__ w, const Op<BF, K>& in, float (&acc)[M / 4],
                                        int lane) {
  const uint4* f = reinterpret_cast<const uint4*>(w) + lane;
  constexpr int T = K / 32;
  gemm_op<M / 16, T, ACC_START>(
      [&](int t, int mb, int part) {
        return __builtin_bit_cast(v8bf, f[(part * (M / 16) * T + mb * T + t) * 64]);
      },
      in, acc);
}
template <bool BF, int M, int K>
__device__ __forceinline__ void gemm_wf(const void* __restrict__ w, const float (&in)[K / 4], float (&acc)[M / 4],
                                        int lane) {
  Op<BF, K> o;
  make_op(in, o);
  gemm_wf<BF, M, K>(w, o, acc, lane);
}

// Dispatch on the GEMM operand type.  frag points at the fragments of one
// matrix (FP32: M*K floats; BF16: M*K bf16 values).
template <bool BF, int MB, int KB, bool ROT = false>
__device__ __forceinline__ void gemm(const void* frag, const float (&in)[4 * KB], float (&acc)[4 * MB], int lane) {
  static_assert(!(BF && ROT), "the rotated layout is an FP32 fragment layout");
  if constexpr (BF)
    gemm_bf16<MB, KB>(reinterpret_cast<const uint4*>(frag), in, acc, lane);
  else
    gemm_f32<MB, KB, ROT>(reinterpret_cast<const float*>(frag), in, acc, lane);
}

// ---------------------------------------------- row-major BF16 tiles in LDS
//
// [rows][W] BF16 with the 8-byte chunk c of row r at chunk c ^ stg_swz(r):
// with 32 chunks per LDS bank cycle the 32 lanes of a half wave hit all banks
// once, in row accesses (16 rows, two chunks each) and in the transposing
// reads below (8 rows, four chunks each), with no padding.
template <int W>
__device__ __forceinline__ int stg_swz(int row) {
  constexpr int U = W / 4;                 // 8-byte chunks per row
  constexpr int RP = U >= 32 ? 1 : 32 / U;  // rows per 256 bytes of LDS
  constexpr int KR = 8 / RP;               // such groups in 8 rows
  const int k = (row & 15) / RP;
  return ((k & (KR - 1)) << 2) | (((k / KR) & 1) << 1);
}

// MFMA operand of a tile, its rows along K: lane (i, kk) receives feature 16 fb + i
// of rows r0 + 4 kk + 0..3 and r0 + 16 + 4 kk + 0..3 (r0 a multiple of 16; the same
// row order for both operands of a product).
// tr_base: the lane's address for feature block fb.
typedef __attribute__((address_space(3))) v4bf lds_v4bf;
template <int W>
__device__ __forceinline__ const char* tr_base(const void* __restrict__ tile, int fb, int lane) {
  const int row = 4 * (lane >> 4) + ((lane & 15) >> 2);
  return reinterpret_cast<const char*>(tile) + row * (W * 2) + (((4 * fb + (lane & 3)) ^ stg_swz<W>(row)) * 8);
}
__device__ __forceinline__ v4bf tr_read4(const char* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_v4bf*)(p));
}
template <int W>
__device__ __forceinline__ v8bf tr_read8(const char* base, int r0) {
  const v4bf lo = tr_read4(base + r0 * (W * 2)), hi = tr_read4(base + (r0 + 16) * (W * 2));
  return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}

// Row `row` of an operand into a tile (FP32: three tiles, part_bytes apart), its
// sign bits flipped by `flip`.
template <int W>
__device__ __forceinline__ void put_row(char* __restrict__ t, int g, int sz, const v8bf (&v)[W / 32], uint32_t flip) {
#pragma unroll
  for (int b = 0; b < W / 16; ++b) {
    const v4u q = __builtin_bit_cast(v4u, v[b / 2]);
    const u32x2 c = b % 2 ? u32x2{q[2], q[3]} : u32x2{q[0], q[1]};
    *reinterpret_cast<u32x2*>(t + ((4 * b + g) ^ sz) * 8) = u32x2{c[0] ^ flip, c[1] ^ flip};
  }
}
template <int W>
__device__ __forceinline__ void stage_op(void* __restrict__ tile, int part_bytes, int row, int g,
                                         const Op<false, W>& o, uint32_t flip = 0) {
  const int sz = stg_swz<W>(row);
  char* t = reinterpret_cast<char*>(tile) + row * (W * 2);
  put_row<W>(t, g, sz, o.h, flip);
  put_row<W>(t + part_bytes, g, sz, o.m, flip);
  put_row<W>(t + 2 * part_bytes, g, sz, o.l, flip);
}

// Weights row major in LDS for both products: gemm_wn reads W's operand,
// lane (i, g) columns 32 t + 4 g + 0..3 and 32 t + 16 + 4 g + 0..3 of row
// 16 mb + i, gemm_wt (W^T in) reads the same copy through the transposing
// load.  Groups of 16 rows are 16 bytes apart, so that no two 8-byte reads of
// an operand lie a multiple of 512 bytes from another's: the compiler would
// pair those into one read and then move every register into place (147 of
// 1425 vector instructions per block of the FP32 edge adjoint).
__host__ __device__ constexpr int wrow_at(int row, int K) { return row * (K * 2) + (row >> 4) * 16; }
__host__ __device__ constexpr int wrow_part(int M, int K) { return wrow_at(M, K); }
__host__ __device__ constexpr size_t wrow_bytes(int M, int K, bool bf) { return size_t(wrow_part(M, K)) * (bf ? 1 : 3); }

// Stage the M x K matrix w (not transposed).  All threads of the workgroup; no
// barrier.  Returns whether this thread met an infinite weight (FP32).
template <bool BF, int M, int K>
__device__ __forceinline__ bool stage_wrow(void* __restrict__ dst, const WView& w) {
  bool odd = false;
  const bool al = w_aligned(w);
  for (int e = threadIdx.x; e < M * K / 8; e += blockDim.x) {
    const int row = e / (K / 8), c = e % (K / 8) * 2;  // chunks c, c + 1
    const float4 a = load4w(w.p + (int64_t)row * w.ld + 4 * c, al);
    const float4 b = load4w(w.p + (int64_t)row * w.ld + 4 * c + 4, al);
    const float x[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
    v8bf p[3];
    split_w8<BF>(x, p[0], p[1], p[2]);
    const int sz = stg_swz<K>(row);
    char* t = reinterpret_cast<char*>(dst) + wrow_at(row, K);
#pragma unroll
    for (int q = 0; q < (BF ? 1 : 3); ++q) {
      const v4u v = __builtin_bit_cast(v4u, p[q]);
      *reinterpret_cast<u32x2*>(t + q * wrow_part(M, K) + (c ^ sz) * 8) = u32x2{v[0], v[1]};
      *reinterpret_cast<u32x2*>(t + q * wrow_part(M, K) + ((c + 1) ^ sz) * 8) = u32x2{v[2], v[3]};
    }
    if constexpr (!BF) odd |= any_inf(x);
  }
  return odd;
}
// One operand fragment of W (chunk t of K, output block mb of M) and of W^T
// (chunk t of M, output block mb of K).
template <int M, int K>
__device__ __forceinline__ v8bf wn_frag(const char* __restrict__ w, int t, int mb, int part, int lane) {
  const int i = lane & 15, g = lane >> 4, sz = stg_swz<K>(i);
  const char* q = w + i * (K * 2) + part * wrow_part(M, K) + wrow_at(16 * mb, K);
  const v4bf lo = __builtin_bit_cast(v4bf, *reinterpret_cast<const u32x2*>(q + ((8 * t + g) ^ sz) * 8));
  const v4bf hi = __builtin_bit_cast(v4bf, *reinterpret_cast<const u32x2*>(q + ((8 * t + 4 + g) ^ sz) * 8));
  return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}
template <int M, int K>
__device__ __forceinline__ v8bf wt_frag(const char* __restrict__ w, int t, int mb, int part, int lane) {
  const char* q = tr_base<K>(w + part * wrow_part(M, K), mb, lane);
  const v4bf lo = tr_read4(q + wrow_at(32 * t, K)), hi = tr_read4(q + wrow_at(32 * t + 16, K));
  return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}
// acc += W in (ACC_SET: acc = W in)
template <bool BF, int M, int K, Acc MODE = ACC_START>
__device__ __forceinline__ void gemm_wn(const char* __restrict__ w, const Op<BF, K>& in, float (&acc)[M / 4],
                                        int lane) {
  // at K = 32 neighbouring row groups are within a paired read's reach: hide
  // that they share a base
  const char* w1 = w + (K == 32 ? opaque_zero() : 0);
  gemm_op<M / 16, K / 32, MODE>(
      [&](int t, int mb, int part) { return wn_frag<M, K>(mb % 2 ? w1 : w, t, mb, part, lane); }, in, acc);
}
// acc += W^T in (ACC_SET: acc = W^T in)
template <bool BF, int M, int K, Acc MODE = ACC_START>
__device__ __forceinline__ void gemm_wt(const char* __restrict__ w, const Op<BF, M>& in, float (&acc)[K / 4],
                                        int lane, float sc = 1.f) {
  gemm_op<K / 16, M / 32, MODE>([&](int t, int mb, int part) { return wt_frag<M, K>(w, t, mb, part, lane); }, in,
                                acc, sc);
}

// All fragments of a small FP32 matrix, read ahead of the product.
template <int T, int MB>
struct WFrags {
  v8bf f[T][MB][3];
  template <int M, int K>
  __device__ __forceinline__ void load_n(const char* __restrict__ w, int lane) {
    static_assert(T == K / 32 && MB == M / 16, "plain product");
    const char* w1 = w + (K == 32 ? opaque_zero() : 0);
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int p = 0; p < 3; ++p) f[t][mb][p] = wn_frag<M, K>(mb % 2 ? w1 : w, t, mb, p, lane);
  }
  template <int M, int K>
  __device__ __forceinline__ void load_t(const char* __restrict__ w, int lane) {
    static_assert(T == M / 32 && MB == K / 16, "transposed product");
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int p = 0; p < 3; ++p) f[t][mb][p] = wt_frag<M, K>(w, t, mb, p, lane);
  }
  template <Acc MODE>
  __device__ __forceinline__ void gemm(const Op<false, 32 * T>& in, float (&acc)[4 * MB]) const {
    gemm_op<MB, T, MODE>([&](int t, int mb, int part) { return f[t][mb][part]; }, in, acc);
  }
};

// Bytes of the packed fragments of an M x K matrix.
__host__ __device__ constexpr size_t frag_bytes(int M, int K, bool bf) { return size_t(M) * K * (bf ? 2 : 4); }

// --------------------------------------------------- elementwise helpers

// ELU with alpha = 1.  The negative branch uses the hardware exponential
// (v_exp_f32 on a prescaled argument, a few ulp): exp(z) - 1 is then off by
// at most ~1e-7 in absolute terms for z <= 0, far below FP32 tolerances.
__device__ __forceinline__ float elu(float z) { return z > 0.f ? z : __expf(z) - 1.f; }
__device__ __forceinline__ float elu_deriv(float z) { return z > 0.f ? 1.f : __expf(z); }
// ELU'(h) from u = ELU(h): 1 for h > 0, else exp(h) = u + 1.  u > 0 exactly
// when h > 0, and then u + 1 >= 1, so min(u + 1, 1) is the same value in
// two instructions instead of four.
__device__ __forceinline__ float elu_deriv_from_value(float u) { return fminf(u + 1.f, 1.f); }

// Sum over the four lanes that share a row (lane groups g = 0..3), on the
// matrix unit: v_mfma_f32_16x16x4f32 with A = 1 and B[k][j] = the value of
// lane j + 16k gives D[i][j] = sum over k for every i, and lane j + 16g
// receives D[4g..4g+3][j].  One FP32 MFMA instead of two dependent LDS
// permutes; must be called with all lanes active.
__device__ __forceinline__ float row_sum(float s) {
  const v4f d = __builtin_amdgcn_mfma_f32_16x16x4f32(1.f, s, v4f{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
  return d[0];
}

// LayerNorm statistics (biased variance) of a W-wide row in row-block layout.
template <int W>
__device__ __forceinline__ void ln_stats(const float (&v)[W / 4], float eps, float& mean, float& rstd) {
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < W / 4; ++i) s += v[i];
  mean = row_sum(s) * (1.f / W);
  float q = 0.f;
#pragma unroll
  for (int i = 0; i < W / 4; ++i) {
    const float d = v[i] - mean;
    q += d * d;
  }
  const float var = row_sum(q) * (1.f / W);
  rstd = 1.f / sqrtf(var + eps);
}

// --------------------------------------------- small first/last Linears

// Stage W[rows][k] (k <= 4) into LDS as [rows][4], zero padded, with the
// whole block (callers synchronise afterwards).
__device__ __forceinline__ void stage_small(float* __restrict__ dst, const float* __restrict__ W, int rows, int k) {
  for (int t = threadIdx.x; t < rows * 4; t += blockDim.x) {
    const int r = t >> 2, c = t & 3;
    dst[t] = c < k ? W[r * k + c] : 0.f;
  }
}

// z[f] += sum_k W0[f][k] in[k] for the lane's features, W0 staged as [H][4].
template <int H>
__device__ __forceinline__ void small_in_linear(const float* __restrict__ w0s, const float (&in)[4], int g,
                                                float (&z)[H / 4]) {
#pragma unroll
  for (int i = 0; i < H / 4; ++i) {
    const int f = 16 * (i / 4) + 4 * g + (i % 4);
    const float4 w = *reinterpret_cast<const float4*>(w0s + 4 * f);
    z[i] += w.x * in[0] + w.y * in[1] + w.z * in[2] + w.w * in[3];
  }
}

// ------------------------------------------- segmented sums over 16 lanes

// DPP row_shr:n within each 16-lane row; lanes j < n read 0.
template <int CTRL>
__device__ __forceinline__ float dpp_f(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ int dpp_i(int x) {
  return __builtin_amdgcn_update_dpp(0, x, CTRL, 0xf, 0xf, true);
}
constexpr int DPP_ROW_SHR1 = 0x111, DPP_ROW_SHR2 = 0x112, DPP_ROW_SHR4 = 0x114, DPP_ROW_SHR8 = 0x118;
constexpr int DPP_ROW_ROR1 = 0x121;  // lane j reads lane (j-1) mod 16

// Inclusive segmented scan over the 16 lanes j of each lane group.  key
// identifies the segment (equal keys are contiguous in j) and must be
// nonzero, because lanes shifted in from outside the row read key 0.
template <int N>
__device__ __forceinline__ void seg_scan16(float (&v)[N], int key) {
  // Each step adds the value `off` lanes back when that lane is in the same
  // segment, written as v += shifted * (0 or 1) so the shift folds into the
  // multiply-add as a DPP operand.  Steps 4 and 8 are skipped (uniformly for
  // the wave) when no segment in the block is that long.
#define MP_SEG_STEP(CTRL)                                     \
  {                                                           \
    const float same = dpp_i<CTRL>(key) == key ? 1.f : 0.f;   \
    _Pragma("unroll") for (int i = 0; i < N; ++i)             \
      v[i] = fmaf(dpp_f<CTRL>(v[i]), same, v[i]);             \
  }
  MP_SEG_STEP(DPP_ROW_SHR1)
  MP_SEG_STEP(DPP_ROW_SHR2)
  if (__ballot(dpp_i<DPP_ROW_SHR4>(key) == key) != 0) {
    MP_SEG_STEP(DPP_ROW_SHR4)
    if (__ballot(dpp_i<DPP_ROW_SHR8>(key) == key) != 0) MP_SEG_STEP(DPP_ROW_SHR8)
  }
#undef MP_SEG_STEP
}

// Value of the lane whose index j (within its 16-lane group) differs in
// bit M (M = 1, 2, 4, 8): DPP quad permutations for 1 and 2, a 16-lane
// rotation by 8 for 8, and a bitmask swizzle (xor 4) for 4.
template <int M>
__device__ __forceinline__ float lane_xor16(float x) {
  const int v = __builtin_bit_cast(int, x);
  if constexpr (M == 1)
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xf, 0xf, false));  // [1,0,3,2]
  else if constexpr (M == 2)
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xf, 0xf, false));  // [2,3,0,1]
  else if constexpr (M == 4)
    return __builtin_bit_cast(float, __builtin_amdgcn_ds_swizzle(v, 0x101F));  // and 0x1f, xor 4
  else
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, v, 0x128, 0xf, 0xf, false));  // row_ror:8
}

// One halving step of a reduce-scatter over the 16 lanes j of a lane
// group: the lane keeps the half of its N values selected by bit M of j
// and adds the partner's copy of that half (the partner sends the half it
// does not keep).
template <int N, int M>
__device__ __forceinline__ void sum16_half(const float (&in)[N], float (&out)[N / 2], int j) {
  const bool hi = (j & M) != 0;
#pragma unroll
  for (int q = 0; q < N / 2; ++q) {
    const float lo_v = in[q], hi_v = in[q + N / 2];
    out[q] = (hi ? hi_v : lo_v) + lane_xor16<M>(hi ? lo_v : hi_v);
  }
}

// Sum over the 16 lanes of each lane group, scattered: on return lane j
// holds in out[c] the sum over the group's lanes of v[j * (N / 16) + c]
// (N a multiple of 16).  Four halving steps (bits 8, 4, 2, 1 of j), N - N/16
// exchanged values in all; the additions are in a fixed order, so the sums
// are bitwise reproducible.
template <int N>
__device__ __forceinline__ void sum16_scatter(const float (&v)[N], float (&out)[N / 16], int j) {
  static_assert(N % 16 == 0, "sum16_scatter needs a multiple of 16 values");
  float a8[N / 2], a4[N / 4], a2[N / 8];
  sum16_half<N, 8>(v, a8, j);
  sum16_half<N / 2, 4>(a8, a4, j);
  sum16_half<N / 4, 2>(a4, a2, j);
  sum16_half<N / 8, 1>(a2, out, j);
}

// Value of lane 15 of the same lane group, delivered to lane 0 (and lane
// j+1 receives lane j, which callers ignore).
__device__ __forceinline__ float from_prev_lane(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), DPP_ROW_ROR1, 0xf, 0xf, false));
}
__device__ __forceinline__ int from_prev_lane_i(int x) {
  return __builtin_amdgcn_update_dpp(0, x, DPP_ROW_ROR1, 0xf, 0xf, false);
}

// ----------------------------------------- static wave schedules over rows

// Split rows [0, n_rows) into n_parts contiguous ranges with about equal
// edge counts: part p starts at the first row whose first edge index is at
// least floor(p * E / n_parts); the last part ends at n_rows.
__device__ __forceinline__ int64_t lower_bound_i32(const int32_t* __restrict__ a, int64_t n, int64_t key) {
  int64_t lo = 0, hi = n;
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    if ((int64_t)a[mid] < key) lo = mid + 1; else hi = mid;
  }
  return lo;
}
__device__ __forceinline__ void part_rows(const int32_t* __restrict__ rowptr, int64_t n_rows, int64_t n_parts,
                                          int64_t p, int64_t& r0, int64_t& r1) {
  const int64_t E = rowptr[n_rows];
  r0 = (p == 0) ? 0 : lower_bound_i32(rowptr, n_rows + 1, (p * E) / n_parts);
  r1 = (p + 1 >= n_parts) ? n_rows : lower_bound_i32(rowptr, n_rows + 1, ((p + 1) * E) / n_parts);
  if (r0 > n_rows) r0 = n_rows;
  if (r1 > n_rows) r1 = n_rows;
  if (r1 < r0) r1 = r0;
}

// Tiled schedule for the edge kernels.  The rows are cut into n_tiles
// row-aligned tiles of about equal edge count (tile boundaries precomputed by
// k_tiles).  Workgroups are dealt round robin to the 8 XCDs, so workgroup b
// runs on XCD b % 8; each XCD takes one contiguous eighth of the tiles, and
// inside it the XCD's waves take consecutive tiles in turn.  All waves of an
// XCD thus sweep a compact window of rows together, and a node row gathered
// by edges a few planes apart is still in that XCD's L2.
struct TileSched {
  int64_t t0, t1;    // this group's tile range
  int64_t rank, nr;  // block rank inside the group, blocks in the group
};
__device__ __forceinline__ TileSched tile_sched(int64_t n_tiles) {
  const int64_t G = gridDim.x, V = G < 8 ? G : 8;
  const int64_t vx = blockIdx.x % V;
  TileSched s;
  s.rank = blockIdx.x / V;
  s.nr = (G - vx + V - 1) / V;
  s.t0 = vx * n_tiles / V;
  s.t1 = (vx + 1) * n_tiles / V;
  return s;
}

// Dynamic tile order: the tiles are cut into V contiguous ranges (one per
// XCD, V = min(grid, 8), workgroup b on XCD b % V as in tile_sched); a wave
// takes the next tile of its XCD's range from an atomic counter, and once
// that range is empty moves on to the next XCD's range, and so on.
// Returns -1 when every range is exhausted.  Tiles are row aligned, so a
// tile's results do not depend on which wave computes it: the order is
// dynamic but the results stay bitwise reproducible.
__device__ __forceinline__ int64_t queue_next(int32_t* queue, int64_t n_tiles, int64_t V, int x0, int& q) {
  while (q < V) {
    const int x = (int)((x0 + q) % V);
    const int64_t t0 = x * n_tiles / V, t1 = (x + 1) * n_tiles / V;
    int old = 0;
    if ((threadIdx.x & 63) == 0) old = atomicAdd(queue + x, 1);
    old = __builtin_amdgcn_readfirstlane(old);
    const int64_t t = t0 + old;
    if (t < t1) return t;
    ++q;
  }
  return -1;
}

// XCD-aware block numbering: the dispatcher hands consecutive workgroups to
// the 8 XCDs in turn; renumber so that each XCD gets one contiguous eighth
// of the work (its L2 then sees neighbouring rows).
__device__ __forceinline__ int64_t xcd_block(int64_t b, int64_t nb) {
  const int64_t per = (nb + 7) / 8;
  const int64_t x = b % 8, i = b / 8;
  const int64_t full = nb % 8 == 0 ? 8 : nb % 8;  // XCDs that get `per` blocks
  // blocks dealt round robin: XCD x receives per or per-1 blocks
  const int64_t start = x < full ? x * per : full * per + (x - full) * (per - 1);
  return start + i;
}

}  // namespace mp
