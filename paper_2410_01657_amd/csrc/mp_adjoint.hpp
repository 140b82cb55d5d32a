// Pieces shared by the adjoint kernels: weight gradients of FP32 products, sums
// over a workgroup's rows.
#pragma once
#include <algorithm>

#include "mp_device.hpp"
#include "mp_exact.hpp"
#include "mp_kernels.hpp"

namespace mp {

constexpr size_t kLdsLimit = 160 * 1024 - 1024;
constexpr int kWaves = 4;  // waves per workgroup in the row-MLP lock-step kernels

// Sum a per-lane row-block vector over all 16*NW rows of the workgroup of NW waves
// (16 lanes each) in a fixed order and write the W sums to dst, added in FP64 (once
// per kernel; in FP32 these 16*NW roundings were most of the error of a bias
// gradient: 280k edges at H = 64, db1 1.2e-4 against 0.5e-4), each column by as many
// threads as there are.  Uses `scratch` (at least 16*NW*W floats of LDS, aligned to
// 8 bytes); contains barriers.
template <int W, int NW = kWaves>
__device__ __forceinline__ void block_sum_vec(const float (&v)[W / 4], float* __restrict__ scratch,
                                              float* __restrict__ dst, int wave, int lane) {
  const int j = lane & 15, g = lane >> 4;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < W / 4; ++i) scratch[(wave * 16 + j) * W + 16 * (i / 4) + 4 * g + (i % 4)] = v[i];
  __syncthreads();
  constexpr int P = 64 * NW / W > 0 ? 64 * NW / W : 1, R = 16 * NW / P;  // threads per column, rows each
  static_assert(64 * NW >= W && R * P == 16 * NW, "a thread per column and more");
  const int c = threadIdx.x % W, q = threadIdx.x / W;
  double s = 0.;
#pragma unroll 8
  for (int r = q * R; r < (q + 1) * R; ++r) s += scratch[r * W + c];
  if constexpr (P > 1) {
    double* part = reinterpret_cast<double*>(scratch);
    __syncthreads();
    part[q * W + c] = s;
    __syncthreads();
    if (q == 0) {
#pragma unroll
      for (int k = 1; k < P; ++k) s += part[k * W + c];
    }
  }
  if (q == 0) dst[c] = (float)s;
  __syncthreads();
}

// The BF16 matrix instruction loses low bits of its partial sums downwards: a
// bias of some 2^-27 of a term, nothing in one product, but a weight gradient
// adds millions of terms of either sign and the bias then outgrows their sum
// (3.5M edges: 4.5e-6 of a weight gradient, 1.5e-6 with FP32 instructions).
// Every other wave therefore sums the gradients of its rows negated, so the bias
// cancels within a workgroup, whatever the grid: 0.9e-6.  Only the staged factor
// is negated (dw_flip: the sign bits of a packed pair, with the row's own sign);
// what a kernel writes per edge or node does not depend on the wave that computes
// it.
//
// The products of an adjoint have such a bias themselves (2^-27 of a term at
// K = 32, 2^-33 above), which adds up in the bias gradients (0.67M edges at
// H = 32: 3.6e-6 of db1, 0.7e-6 without).  So a row goes through them times a sign
// that its own gradient decides, +1 or -1 about as often: by the number of bits of
// the sign and the mantissa, so that equal rows take the same, opposite rows the
// opposite one and powers of two change nothing.  v: one value of the row per lane
// group.
__device__ __forceinline__ float row_sign(float v) {
  const uint32_t b = __builtin_bit_cast(uint32_t, row_sum(v)) & 0x807fffffu;
  return __builtin_bit_cast(float, 0x3f800000u | ((uint32_t)__popc(b) << 31));
}
__device__ __forceinline__ uint32_t dw_flip(int wave, float row) {
  const uint32_t b = __builtin_bit_cast(uint32_t, row) & 0x80000000u;
  return (wave & 1 ? 0x80008000u : 0u) ^ (b | b >> 16);
}
__device__ __forceinline__ float dw_sign(int wave) { return wave & 1 ? -1.f : 1.f; }

// FP32 weight gradients dW += G^T A (and, with SUM, the column sums of G) over
// the 16 rows one wave holds, from the three BF16 parts of both factors staged
// in that wave's own LDS tiles (stage_op, 16 rows): no other wave takes part,
// so nothing waits.  Sixteen rows fill half of the matrix instruction's 32-long
// reduction; the other half takes the same rows of another part: [Gh|Gm]
// [Ah|Am] = hh + mm, [Gh|Gm] [Am|Ah] = hm + mh, [Gh|Gl] [Al|Ah] = hl + lh, so
// three instructions do the six products, added straight onto the running sum
// (fewer roundings than the FP32 instruction's four).  The column sums are
// products with ones, [Gh|Gm] [1|1] and [Gh|Gl] [0|1]: on the vector unit they
// would move through the accumulation registers every block.
template <int GW, int AW, bool SUM>
struct DwWave {
  static constexpr int FB = GW / 16, KB = AW / 16;
  static constexpr int GP = 16 * GW * 2, AP = 16 * AW * 2;  // bytes of one part
  static constexpr int TILE_G = 3 * GP, TILE_A = 3 * AP;
  v4f acc[FB * KB], cs[SUM ? FB : 1];
  __device__ __forceinline__ void zero() {
#pragma unroll
    for (int n = 0; n < FB * KB; ++n) acc[n] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int n = 0; n < (SUM ? FB : 1); ++n) cs[n] = v4f{0.f, 0.f, 0.f, 0.f};
  }
  static __device__ __forceinline__ v8bf two(const char* p0, const char* p1) {
    return __builtin_shufflevector(tr_read4(p0), tr_read4(p1), 0, 1, 2, 3, 4, 5, 6, 7);
  }
  // The operands of one block, so that a caller can read them early and put
  // the products where they overlap vector work.
  struct Frags {
    v8bf hm[KB], mh[KB], lh[KB], ghm[FB], ghl[FB];
  };
  static __device__ __forceinline__ void load(Frags& f, const char* __restrict__ tG, const char* __restrict__ tA,
                                              int lane) {
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
      const char* p = tr_base<AW>(tA, kb, lane);
      f.hm[kb] = two(p, p + AP);
      f.mh[kb] = two(p + AP, p);
      f.lh[kb] = two(p + 2 * AP, p);
    }
#pragma unroll
    for (int fb = 0; fb < FB; ++fb) {
      const char* p = tr_base<GW>(tG, fb, lane);
      f.ghm[fb] = two(p, p + GP);
      f.ghl[fb] = two(p, p + 2 * GP);
    }
  }
  __device__ __forceinline__ void mma(const Frags& f) {
    const uint32_t one2 = 0x3F803F80u;
#pragma unroll
    for (int fb = 0; fb < FB; ++fb) {
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) acc[fb * KB + kb] = MP_MFMA_BF16(f.ghl[fb], f.lh[kb], acc[fb * KB + kb]);
      if constexpr (SUM) cs[fb] = MP_MFMA_BF16(f.ghl[fb], __builtin_bit_cast(v8bf, (v4u{0, 0, one2, one2})), cs[fb]);
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) acc[fb * KB + kb] = MP_MFMA_BF16(f.ghm[fb], f.mh[kb], acc[fb * KB + kb]);
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) acc[fb * KB + kb] = MP_MFMA_BF16(f.ghm[fb], f.hm[kb], acc[fb * KB + kb]);
      if constexpr (SUM)
        cs[fb] = MP_MFMA_BF16(f.ghm[fb], __builtin_bit_cast(v8bf, (v4u{one2, one2, one2, one2})), cs[fb]);
    }
  }
  __device__ __forceinline__ void add(const char* __restrict__ tG, const char* __restrict__ tA, int lane) {
    Frags f;
    load(f, tG, tA, lane);
    mma(f);
  }
  // Add the NW waves' sums, G staged with dw_flip, in wave order and write them:
  // dst [GW][AW], with SUM dst_cs [GW].  Uses NW * GW * AW floats of `scratch`;
  // contains barriers.
  template <int NW>
  __device__ __forceinline__ void store(float* __restrict__ scratch, float* __restrict__ dst,
                                        float* __restrict__ dst_cs, int wave, int lane) {
    const float sgn = dw_sign(wave);
    __syncthreads();
#pragma unroll
    for (int n = 0; n < FB * KB; ++n) {
#pragma unroll
      for (int v = 0; v < 4; ++v)
        scratch[(wave * GW + 16 * (n / KB) + 4 * (lane >> 4) + v) * AW + 16 * (n % KB) + (lane & 15)] = sgn * acc[n][v];
    }
    __syncthreads();
    for (int t = threadIdx.x; t < GW * AW; t += blockDim.x) {
      float sum = 0.f;
#pragma unroll
      for (int w = 0; w < NW; ++w) sum += scratch[w * GW * AW + t];
      dst[t] = sum;
    }
    __syncthreads();
    if constexpr (SUM) {
      if ((lane & 15) == 0) {
#pragma unroll
        for (int fb = 0; fb < FB; ++fb) {
#pragma unroll
          for (int v = 0; v < 4; ++v) scratch[wave * GW + 16 * fb + 4 * (lane >> 4) + v] = sgn * cs[fb][v];
        }
      }
      __syncthreads();
      for (int t = threadIdx.x; t < GW; t += blockDim.x) {
        float sum = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) sum += scratch[w * GW + t];
        dst_cs[t] = sum;
      }
      __syncthreads();
    }
  }
};

// Keep a wave's LDS stores ahead of its own reads of other lanes' data (LDS
// operations of one wave complete in order).
__device__ __forceinline__ void wave_lds_fence() {
  asm volatile("" ::: "memory");
}

}  // namespace mp
