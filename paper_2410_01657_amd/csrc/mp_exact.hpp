// FP32 products with FP32 matrix instructions, for rows with an infinite operand on
// the paths that otherwise form them from BF16 parts.
//
// None of this runs for finite values.  The row kernels test each block of 16 rows
// and compute it again at once (their output may take an input's place).  The edge
// kernels only note a NaN per block and run the wave's tiles again at their end, once
// its last sum is stored (in the dynamic tile order: a tile after its last block):
// their loops then hold no branch, and its registers stand beside no weight
// gradients.
#pragma once
#include "mp_device.hpp"
#include "mp_edge.hpp"

namespace mp {

// acc += A in with FP32 instructions, A(m, k) read from device memory, of any
// alignment.  For the rare block with an infinite operand.
template <int M, int K, class F>
__device__ __forceinline__ void gemm_exact_of(F&& el, const float (&in)[K / 4], float (&acc)[M / 4], int lane) {
  const int l = lane + opaque_zero(), i = l & 15, k = l >> 4;  // no address held outside the branch
  v4f c[M / 16];
#pragma unroll
  for (int mb = 0; mb < M / 16; ++mb) c[mb] = v4f{acc[4 * mb], acc[4 * mb + 1], acc[4 * mb + 2], acc[4 * mb + 3]};
#pragma unroll
  for (int s = 0; s < K / 4; ++s) {
    if (s % 4 == 0) __builtin_amdgcn_sched_barrier(0);  // few weights in flight
#pragma unroll
    for (int mb = 0; mb < M / 16; ++mb)
      c[mb] = __builtin_amdgcn_mfma_f32_16x16x4f32(el(16 * mb + i, 16 * (s / 4) + 4 * k + s % 4), in[s], c[mb], 0, 0, 0);
  }
#pragma unroll
  for (int mb = 0; mb < M / 16; ++mb) {
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[4 * mb + r] = c[mb][r];
  }
}
template <int M, int K>  // W M x K
__device__ __forceinline__ void gemm_exact(const WView& w, const float (&in)[K / 4], float (&acc)[M / 4], int lane) {
  gemm_exact_of<M, K>([&](int m, int k) { return w.p[(int64_t)m * w.ld + k]; }, in, acc, lane);
}
template <int M, int K>  // W^T in
__device__ __forceinline__ void gemm_exact_t(const WView& w, const float (&in)[M / 4], float (&acc)[K / 4], int lane) {
  gemm_exact_of<K, M>([&](int m, int k) { return w.p[(int64_t)k * w.ld + m]; }, in, acc, lane);
}

// The Linears after an MLP's first, with gemm_exact: u[l] = ELU(z), z = bias(l) +
// W(l) u[l] for l = 0 .. NL - 1, and back: g = (W(l)^T g) ELU'(u[l]).
template <int H, int NL, class FW, class FB>
__device__ __forceinline__ void exact_forward(FW&& W, FB&& bias, float (&z)[H / 4], float (&u)[NL][H / 4], int lane) {
#pragma unroll
  for (int l = 0; l < NL; ++l) {
#pragma unroll
    for (int i = 0; i < H / 4; ++i) u[l][i] = elu(z[i]);
    load_vec<H>(bias(l), lane >> 4, z);
    gemm_exact<H, H>(W(l), u[l], z, lane);
  }
}
template <int H, int NL, class FW>
__device__ __forceinline__ void exact_adjoint(FW&& W, const float (&u)[NL][H / 4], float (&g)[H / 4], int lane) {
#pragma unroll
  for (int l = NL - 1; l >= 0; --l) {
    float t[H / 4];
#pragma unroll
    for (int i = 0; i < H / 4; ++i) t[i] = 0.f;
    gemm_exact_t<H, H>(W(l), g, t, lane);
#pragma unroll
    for (int i = 0; i < H / 4; ++i) g[i] = t[i] * elu_deriv_from_value(u[l][i]);
  }
}
// Adjoint of y = LN(z) for the gradient g at y, in place.
template <int W>
__device__ __forceinline__ void ln_adjoint(float (&z)[W / 4], float (&g)[W / 4], const float* __restrict__ gain,
                                           float eps, int lane) {
  float mean, rstd, gam[W / 4], s1 = 0.f, s2 = 0.f;
  ln_stats<W>(z, eps, mean, rstd);
  load_vec<W>(gain, lane >> 4, gam);
#pragma unroll
  for (int i = 0; i < W / 4; ++i) {
    z[i] = (z[i] - mean) * rstd;
    g[i] *= gam[i];
    s1 += g[i];
    s2 += g[i] * z[i];
  }
  s1 = row_sum(s1) * (1.f / W);
  s2 = row_sum(s2) * (1.f / W);
#pragma unroll
  for (int i = 0; i < W / 4; ++i) g[i] = rstd * (g[i] - s1 - z[i] * s2);
}

// One tile of the edge update (k_edge_fwd) again.  pre(ri, sj, e, z): the first
// pre-activation z; W, bias: the Linears after the first; gain: LayerNorm gain and
// shift, H floats each, or null.
template <int H, int NL, class PRE, class FW, class FB>
__device__ __forceinline__ void exact_edge_tile(const DevGraph& gr, int64_t tile, const float* __restrict__ e_in,
                                                float* __restrict__ e_out, float* __restrict__ a_out, bool am,
                                                float* __restrict__ carry, PRE&& pre, FW&& W, FB&& bias,
                                                const float* __restrict__ gain, float eps, int lane) {
  const int j = lane & 15, g = lane >> 4;
  const int64_t e0 = gr.tile_e[tile], e1 = gr.tile_e[tile + 1];
  int carry_key = 0;
#pragma unroll 1
  for (int64_t base = e0; base < e1; base += 16) {
    EdgeIdx ix;
    ix.fetch(gr, base + j, e1, e1 - 1);
    const int64_t k = base + j;
    const bool valid = k < e1;
    float ev[H / 4], z[H / 4], u[NL][H / 4];
    load_row<H>(e_in + (valid ? k : e1 - 1) * H, g, ev);
    pre(ix.ri, ix.sj, ev, z);
    exact_forward<H, NL>(W, bias, z, u, lane);
    if (gain) {
      float mean, rstd, ga[H / 4], be[H / 4];
      ln_stats<H>(z, eps, mean, rstd);
      load_vec<H>(gain, g, ga);
      load_vec<H>(gain + H, g, be);
#pragma unroll
      for (int i = 0; i < H / 4; ++i) z[i] = (z[i] - mean) * rstd * ga[i] + be[i];
    }
    const float inv_d = 1.f / (float)ix.md;
#pragma unroll
    for (int i = 0; i < H / 4; ++i) ev[i] += z[i];
    if (valid && e_out) store_row<H>(e_out + k * H, g, ev);
#pragma unroll
    for (int i = 0; i < H / 4; ++i) z[i] = (am ? z[i] : ev[i]) * inv_d;
    edge_gp<H>(z, carry, carry_key, valid ? ix.ri + 1 : -1, valid && ix.nx != ix.ri, a_out + (int64_t)ix.ri * H, j, g);
  }
}

// One tile of the edge adjoint again, but for its weight gradients: g_e_in, g_h and
// g_P.  w0: the edge part of the first Linear; gain: null without LayerNorm.
template <int H, int NL, class PRE, class FW, class FB>
__device__ __forceinline__ void exact_edge_adjoint_tile(const DevGraph& gr, int64_t tile,
                                                        const float* __restrict__ e_in,
                                                        const float* __restrict__ g_e_out,
                                                        const float* __restrict__ g_a, float* __restrict__ g_e_in,
                                                        float* __restrict__ g_h, float* __restrict__ g_P, bool am,
                                                        float* __restrict__ carry, PRE&& pre, const WView& w0, FW&& W,
                                                        FB&& bias, const float* __restrict__ gain, float eps, int lane) {
  const int j = lane & 15, g = lane >> 4;
  const int64_t e0 = gr.tile_e[tile], e1 = gr.tile_e[tile + 1];
  int carry_key = 0;
#pragma unroll 1
  for (int64_t base = e0; base < e1; base += 16) {
    EdgeIdx ix;
    ix.fetch(gr, base + j, e1, e1 - 1);
    const int64_t k = base + j;
    const bool valid = k < e1;
    const int64_t kk = valid ? k : e1 - 1;
    const float inv_d = 1.f / (float)ix.md;
    float z[H / 4], t[H / 4], ge[H / 4], u[NL][H / 4];
    load_row<H>(e_in + kk * H, g, t);
    pre(ix.ri, ix.sj, t, z);
    exact_forward<H, NL>(W, bias, z, u, lane);
    load_row<H>(g_a + (int64_t)ix.ri * H, g, t);
    if (g_e_out) {
      load_row<H>(g_e_out + kk * H, g, ge);
    } else {
#pragma unroll
      for (int i = 0; i < H / 4; ++i) ge[i] = 0.f;
    }
#pragma unroll
    for (int i = 0; i < H / 4; ++i) {
      const float v = t[i] * inv_d + ge[i];
      t[i] = valid ? v : 0.f;
      if (!am) ge[i] = t[i];
    }
    if (gain) ln_adjoint<H>(z, t, gain, eps, lane);
    exact_adjoint<H, NL>(W, u, t, lane);
    gemm_exact_t<H, H>(w0, t, ge, lane);
    if (valid) {
      store_row<H>(g_e_in + k * H, g, ge);
      store_row<H>(g_h + k * H, g, t);
    }
    // lanes past the tile's last edge hold t = 0 and a key of their own
    edge_gp<H>(t, carry, carry_key, valid ? ix.ri + 1 : -1, valid && ix.nx != ix.ri, g_P + (int64_t)ix.ri * H, j, g);
  }
}

}  // namespace mp
