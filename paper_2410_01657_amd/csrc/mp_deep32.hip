// Deep MLPs of hidden width 32 on the matrix unit (Table I's large model:
// five extra H -> H layers in every MLP), for the consistent layer (Eq. 4a-e,
// Eq. 3).  Up to kDeep32MaxHidden extra layers; deeper ones, and widths 8 and
// 16, run on the row-per-thread kernels.
//
// A wave holds 16 rows (edges or nodes) in the row-block layout, eight values
// per lane, and takes them through the whole MLP: at this width a Linear is
// two output blocks of one 32-long product each, in FP32 from three BF16 parts
// (Op<false, 32>), so a layer's output operand is the next one's input with no
// data movement.  One row per thread spent 1024 FMA issue cycles per layer and
// 16 rows at half rate (each weight a broadcast LDS read); here it is 192.
//
// Adjoint: the activations of a block stay on chip (FP32 values in registers,
// their parts in LDS as the factors of the weight gradients), and each wave
// sums the gradients of all its matrices itself (DwWave, 16 registers each).
// The row-per-thread form writes a record of 576 floats per edge and reads it
// back for the weight gradients: 2.3 KB each way beside 0.5 KB of inputs and
// outputs.  The first edge Linear is split over its input as in the wide
// layers: P = W0a x + b0 and Q = W0b x once per node (k_proj), and their
// adjoint, the sums over receivers and senders, in k_gq.
//
// Five extra layers, 3.5M edges, 0.63M nodes, one layer forward and adjoint:
// 9.41 -> 2.95 ms (edge adjoint with its weight gradients 5.2 -> 1.73 ms, edge
// forward 1.63 -> 0.61, node adjoint 0.66 and its weight gradients -> 0.31, sender
// sums 0.26 -> 0.18).  With its one wave per SIMD the edge adjoint has the matrix
// unit busy in 27% of the cycles and issues vector instructions in 50%, a quarter of
// the matrix cycles beside them: what does not overlap adds up.
#include "mp_adjoint.hpp"

namespace mp {

namespace {

constexpr int kH = 32, kNF = kH / 4;
constexpr int64_t kHid = kH * kH + kH;  // parameters of one hidden Linear

// Offsets in the flat parameter array of an MLP with K inputs.
constexpr int64_t off_b0(int K) { return (int64_t)kH * K; }
constexpr int64_t off_hid(int K, int l) { return off_b0(K) + kH + l * kHid; }  // l = NH: the last Linear

// Per-feature vectors in LDS: b0, hidden biases, last bias, gain, shift.
template <int NH>
constexpr int n_vecs() { return NH + 4; }
template <int NH>
__device__ __forceinline__ void stage_vecs(float* __restrict__ v, const float* __restrict__ theta, int K, int ln) {
  for (int t = threadIdx.x; t < n_vecs<NH>() * kH; t += blockDim.x) {
    const int q = t / kH, f = t % kH;
    v[t] = q == 0 ? theta[off_b0(K) + f]
           : q <= NH + 1 ? theta[off_hid(K, q - 1) + kH * kH + f]
           : ln ? theta[off_hid(K, NH + 1) + (q - NH - 2) * kH + f]
                : 0.f;
  }
}

// The Linears after the first of an MLP with K inputs: matrices in device memory,
// biases in LDS (stage_vecs).
struct Rest {
  const float* theta;
  int K;
  __device__ __forceinline__ WView operator()(int l) const { return WView{theta + off_hid(K, l), kH, 0}; }
  struct Bias {
    const float* v;
    __device__ __forceinline__ const float* operator()(int l) const { return v + (l + 1) * kH; }
  };
};

// ------------------------------------------------------------------ forward

template <int NH, int K>
struct Fwd32 {
  static constexpr size_t W0 = w_bytes(kH, K, false), W1 = w_bytes(kH, kH, false);
  static constexpr size_t WB = W0 + (NH + 1) * W1;
  static constexpr size_t VECS = n_vecs<NH>() * kH * sizeof(float);
  static constexpr int NW = WB > 50 * 1024 ? 8 : 4;  // two workgroups per CU, or four and more

  // odd: see note_odd
  static __device__ __forceinline__ void stage(char* __restrict__ w, float* __restrict__ v, int* __restrict__ odd,
                                               const float* __restrict__ theta, int ln) {
    bool o = stage_wfrag<false, kH, K>(w, WView{theta, K, 0});
#pragma unroll
    for (int l = 0; l <= NH; ++l)
      o |= stage_wfrag<false, kH, kH>(w + W0 + l * W1, WView{theta + off_hid(K, l), kH, 0});
    stage_vecs<NH>(v, theta, K, ln);
    note_odd(odd, o);
  }
  // y = [LN] MLP(in); odd(y): called with the last Linear's output
  template <class F>
  static __device__ __forceinline__ void run(const char* __restrict__ w, const float* __restrict__ v,
                                             const Op<false, K>& in, int ln, float eps, int lane, float (&y)[kNF],
                                             F&& odd) {
    const int g = lane >> 4;
    float u[kNF];
    load_vec<kH>(v, g, u);
    gemm_wf<false, kH, K>(w, in, u, lane);
#pragma unroll
    for (int l = 0; l <= NH; ++l) {
#pragma unroll
      for (int i = 0; i < kNF; ++i) u[i] = elu(u[i]);
      load_vec<kH>(v + (l + 1) * kH, g, y);
      gemm_wf<false, kH, kH>(w + W0 + l * W1, u, y, lane);
#pragma unroll
      for (int i = 0; i < kNF; ++i) u[i] = y[i];
    }
    odd(y);
    if (ln) {
      float mean, rstd, gam[kNF], bet[kNF];
      ln_stats<kH>(y, eps, mean, rstd);
      load_vec<kH>(v + (NH + 2) * kH, g, gam);
      load_vec<kH>(v + (NH + 3) * kH, g, bet);
#pragma unroll
      for (int i = 0; i < kNF; ++i) y[i] = (y[i] - mean) * rstd * gam[i] + bet[i];
    }
  }
};

// Operand of a row [a, b, ...] of 32-wide pieces: piece p.
template <int K>
__device__ __forceinline__ void put_piece(Op<false, K>& o, int p, const float (&x)[kNF]) {
  split3_8(x, o.h[p], o.m[p], o.l[p]);
}
// Eq. 4a-b, as k_edge_fwd: one row-aligned tile at a time per wave, the
// aggregate by a segmented scan over the 16 edges of a block.
template <int NH>
__global__ __launch_bounds__((64 * Fwd32<NH, 96>::NW), 4) void k_deep32_edge_fwd(DeepEdgeArgs a) {
  using F = Fwd32<NH, 96>;
  extern __shared__ uint4 smem[];
  char* wl = reinterpret_cast<char*>(smem);
  float* vecs = reinterpret_cast<float*>(wl + F::WB);
  float* carry = vecs + n_vecs<NH>() * kH + (threadIdx.x / 64) * kH + (threadIdx.x / 16 % 4) * kNF;
  int* odd = reinterpret_cast<int*>(vecs + (n_vecs<NH>() + F::NW) * kH);
  F::stage(wl, vecs, odd, a.theta, a.ln);
  __syncthreads();
  const bool wodd = read_odd(odd);
  const DevGraph& gr = a.g;
  const int lane = lane_id(), j = lane & 15, g = lane >> 4;
  const TileSched ts = tile_sched(gr.n_tiles);
  bool nan = false;  // an infinite operand met (or a NaN)
  for (int64_t tile = ts.t0 + ts.rank * F::NW + threadIdx.x / 64; tile < ts.t1; tile += ts.nr * F::NW) {
    const int64_t r0 = gr.tile_r[tile], r1 = gr.tile_r[tile + 1];
    const int64_t e0 = gr.tile_e[tile], e1 = gr.tile_e[tile + 1];
    const int64_t e_last = e1 > e0 ? e1 - 1 : 0;
    int carry_key = 0;
    EdgeIdx ix;
    ix.fetch(gr, e0 + j, e1, e_last);
    ix.settle();
    for (int64_t base = e0; base < e1; base += 16) {
      const int oz = opaque_zero();
      const int64_t k = base + j;
      const bool valid = k < e1;
      const int ri = ix.ri, sj = ix.sj;
      const float inv_d = 1.f / (float)ix.md;
      const bool last = valid && ix.nx != ri;
      const int key = valid ? ri + 1 : -1;
      ix.fetch(gr, k + 16, e1, e_last);
      float xi[kNF], xj[kNF], ev[kNF], m[kNF];
      load_row<kH>(a.e_in + (valid ? k : e_last) * kH, g, ev);
      load_row<kH>(a.x + (int64_t)ri * kH, g, xi);
      load_row<kH>(a.x + (int64_t)sj * kH, g, xj);
      __builtin_amdgcn_sched_barrier(0);
      Op<false, 96> in;
      put_piece(in, 0, xi);
      put_piece(in, 1, xj);
      put_piece(in, 2, ev);
      F::run(wl + oz, vecs + oz, in, a.ln, a.eps, lane, m, [&](float (&y)[kNF]) { nan |= y[0] != y[0]; });
#pragma unroll
      for (int i = 0; i < kNF; ++i) ev[i] += m[i];
      if (valid) store_row<kH>(a.e_out + k * kH, g, ev);
#pragma unroll
      for (int i = 0; i < kNF; ++i) ev[i] = (a.am ? m[i] : ev[i]) * inv_d;
      edge_gp<kH>(ev, carry, carry_key, key, last, a.a_out + (int64_t)ri * kH, j, g);
    }
    zero_empty_rows<kH>(gr, r0, r1, a.a_out, lane);
  }
  if (!wodd && !__ballot(nan)) return;
  auto pre = [&](int ri, int sj, const float (&e)[kNF], float (&z)[kNF]) {
    float x[kNF];
    load_vec<kH>(vecs, g, z);
    load_row<kH>(a.x + (int64_t)ri * kH, g, x);
    gemm_exact<kH, kH>(WView{a.theta, 96, 0}, x, z, lane);
    load_row<kH>(a.x + (int64_t)sj * kH, g, x);
    gemm_exact<kH, kH>(WView{a.theta + kH, 96, 0}, x, z, lane);
    gemm_exact<kH, kH>(WView{a.theta + 2 * kH, 96, 0}, e, z, lane);
  };
  for (int64_t tile = ts.t0 + ts.rank * F::NW + threadIdx.x / 64; tile < ts.t1; tile += ts.nr * F::NW)
    exact_edge_tile<kH, NH + 1>(gr, tile, a.e_in, a.e_out, a.a_out, a.am, carry, pre, Rest{a.theta, 96},
                                Rest::Bias{vecs}, a.ln ? vecs + (NH + 2) * kH : nullptr, a.eps, lane);
}

// Eq. 4e: x' = x + MLP([a*, x]).
template <int NH>
__global__ __launch_bounds__((64 * Fwd32<NH, 64>::NW), 4) void k_deep32_node_fwd(DeepRowArgs a) {
  using F = Fwd32<NH, 64>;
  extern __shared__ uint4 smem[];
  char* wl = reinterpret_cast<char*>(smem);
  float* vecs = reinterpret_cast<float*>(wl + F::WB);
  int* odd = reinterpret_cast<int*>(vecs + n_vecs<NH>() * kH);
  F::stage(wl, vecs, odd, a.theta, a.ln);
  __syncthreads();
  const bool wodd = read_odd(odd);
  const int lane = lane_id(), j = lane & 15, g = lane >> 4;
  const int64_t n = a.n_rows, nblk = (n + 15) / 16;
  for (int64_t blk = (int64_t)blockIdx.x * F::NW + threadIdx.x / 64; blk < nblk; blk += (int64_t)gridDim.x * F::NW) {
    const int oz = opaque_zero();
    const int64_t row = blk * 16 + j, rr = std::min<int64_t>(row, n - 1);
    float s[kNF], x[kNF], y[kNF];
    load_row<kH>(a.src_a + rr * kH, g, s);
    load_row<kH>(a.src_b + rr * kH, g, x);
    __builtin_amdgcn_sched_barrier(0);
    Op<false, 64> in;
    put_piece(in, 0, s);
    put_piece(in, 1, x);
    F::run(wl + oz, vecs + oz, in, a.ln, a.eps, lane, y, [&](float (&z)[kNF]) {
      if (!wodd && !any_nan(z[0])) return;
      float again[kNF], u[NH + 1][kNF];
      const int l = lane + oz;
      const float* v = vecs + oz;
      load_vec<kH>(v, g, z);
      load_row<kH>(a.src_a + rr * kH, g, again);
      gemm_exact<kH, kH>(WView{a.theta, 64, 0}, again, z, l);
      load_row<kH>(a.src_b + rr * kH, g, again);
      gemm_exact<kH, kH>(WView{a.theta + kH, 64, 0}, again, z, l);
      exact_forward<kH, NH + 1>(Rest{a.theta, 64}, Rest::Bias{v}, z, u, l);
    });
#pragma unroll
    for (int i = 0; i < kNF; ++i) y[i] += x[i];
    if (row < n) store_row<kH>(a.out + row * kH, g, y);
  }
}

// ------------------------------------------------------------------ adjoint

// K inputs of the first matrix (32: an edge's e, the node parts of the
// pre-activation given; 64: a node's [a*, x]).
template <int NH, int K>
struct Bwd32 {
  static constexpr size_t W0 = wrow_bytes(kH, K, false), W1 = wrow_bytes(kH, kH, false);
  static constexpr size_t WB = W0 + (NH + 1) * W1;
  static constexpr size_t VECS = n_vecs<NH>() * kH * sizeof(float);
  static constexpr bool NODE = K != kH;  // the edge form's b0 is k_gq's
  using Dw0 = DwWave<kH, K, NODE>;
  using Dw1 = DwWave<kH, kH, true>;
  // one wave's tiles: the input, u_0 .. u_NH, and one gradient
  static constexpr size_t T0 = Dw0::TILE_A, T1 = Dw1::TILE_A;
  static constexpr size_t WTILE = T0 + (NH + 1) * T1 + Dw1::TILE_G;
  static constexpr size_t CARRY = kH * sizeof(float);  // per wave
  // the shallowest eight waves, two per SIMD; the others take the registers
  // (and more layers the LDS) of one: at two per SIMD they spill
  static constexpr int OCC = NH <= (K == kH ? 0 : 1) ? 2 : 1, NW = 4 * OCC;
  static constexpr size_t LDS = NW * (WTILE + CARRY) + WB + VECS + NW * sizeof(int);
  static_assert(LDS <= kLdsLimit && NW * WTILE >= NW * kH * K * sizeof(float), "weights, tiles, final sums in LDS");
  static_assert(NW * WTILE >= 16 * NW * kH * sizeof(float), "row sums in LDS");

  Dw0 d0;
  Dw1 d1[NH + 1];  // hidden Linears, then the last
  float dga[kNF], dbe[kNF];

  __device__ __forceinline__ void zero() {
    d0.zero();
#pragma unroll
    for (int l = 0; l <= NH; ++l) d1[l].zero();
#pragma unroll
    for (int i = 0; i < kNF; ++i) dga[i] = dbe[i] = 0.f;
  }
  // w0: the first matrix's columns used here (K of them, leading dimension ld)
  static __device__ __forceinline__ void stage(char* __restrict__ w, float* __restrict__ v, int* __restrict__ odd,
                                               const float* __restrict__ theta, const float* __restrict__ w0, int ld,
                                               int ln) {
    bool o = stage_wrow<false, kH, K>(w, WView{w0, ld, 0});
#pragma unroll
    for (int l = 0; l <= NH; ++l)
      o |= stage_wrow<false, kH, kH>(w + W0 + l * W1, WView{theta + off_hid(ld, l), kH, 0});
    stage_vecs<NH>(v, theta, ld, ln);
    note_odd(odd, o);
  }
  // Forward and adjoint of one block.  z: what the first matrix's product is
  // added to (bias, or P + Q); gE(y): the gradient arriving at the output, zero
  // on absent rows, asked for once the forward is done; done(d, o, sg, nan): called
  // with the first pre-activation's gradient d and its operand, both times the
  // row's sign sg; nan: the forward met an infinite operand (or a NaN).
  template <class GE, class DONE>
  __device__ __forceinline__ void run(const char* __restrict__ w, const float* __restrict__ v, char* __restrict__ tile,
                                      const Op<false, K>& in, float (&z)[kNF], int ln, float eps, int lane,
                                      int wave, GE&& gE, DONE&& done) {
    const int j = lane & 15, g = lane >> 4;
    float u[NH + 1][kNF], y[kNF];
    char* tG = tile + T0 + (NH + 1) * T1;
    // Each matrix's fragments are read one product ahead, and a layer's
    // weight-gradient products are issued beside the next layer's split: a
    // wave alone on its SIMD would wait for every LDS read otherwise.
    WFrags<1, 2> wf;
    wave_lds_fence();
    stage_op<K>(tile, Dw0::AP, j, g, in);
    gemm_wn<false, kH, K>(w, in, z, lane);
#pragma unroll
    for (int l = 0; l <= NH; ++l) {
      wf.template load_n<kH, kH>(w + W0 + l * W1, lane);
      float bias[kNF];
      load_vec<kH>(v + (l + 1) * kH, g, bias);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < kNF; ++i) u[l][i] = elu(z[i]);
      Op<false, kH> o;
      make_op(u[l], o);
      stage_op<kH>(tile + T0 + l * T1, Dw1::AP, j, g, o);
      wf.template gemm<ACC_SET>(o, z);
#pragma unroll
      for (int i = 0; i < kNF; ++i) z[i] += bias[i];
    }
    wf.template load_t<kH, kH>(w + W0 + NH * W1, lane);
    __builtin_amdgcn_sched_barrier(0);
    const bool nan = z[0] != z[0];
    gE(y);
    const float sg = row_sign(y[0]);  // gm carries it from here on
    const uint32_t flip = dw_flip(wave, sg);
    float gm[kNF];
    if (ln) {
      float mean, rstd, gam[kNF];
      load_vec<kH>(v + (NH + 2) * kH, g, gam);
      ln_stats<kH>(z, eps, mean, rstd);
      float s1 = 0.f, s2 = 0.f;
#pragma unroll
      for (int i = 0; i < kNF; ++i) {
        const float xh = (z[i] - mean) * rstd;
        dga[i] += y[i] * xh;
        dbe[i] += y[i];
        const float gx = y[i] * gam[i];
        s1 += gx;
        s2 += gx * xh;
        z[i] = xh;
      }
      s1 = row_sum(s1) * (1.f / kH);
      s2 = row_sum(s2) * (1.f / kH);
      const float rs = rstd * sg, c1 = -rs * s1, c2 = -rs * s2;
#pragma unroll
      for (int i = 0; i < kNF; ++i) gm[i] = fmaf(z[i], c2, fmaf(y[i] * gam[i], rs, c1));
    } else {
#pragma unroll
      for (int i = 0; i < kNF; ++i) gm[i] = y[i] * sg;
    }
    // back through the Linears: gm becomes the gradient at pre-activation l
    typename Dw1::Frags df;
#pragma unroll
    for (int l = NH; l >= 0; --l) {
      Op<false, kH> o;
      make_op(gm, o);
      if (l < NH) {
        d1[l + 1 <= NH ? l + 1 : NH].mma(df);
        // one matrix instruction (16 cycles) per four vector ones
#pragma unroll
        for (int q = 0; q < 14; ++q) {
          __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x2, 4, 0);
        }
      }
      wf.template gemm<ACC_SET>(o, gm);
      wave_lds_fence();
      stage_op<kH>(tG, Dw1::GP, j, g, o, flip);
      wave_lds_fence();
      Dw1::load(df, tG, tile + T0 + l * T1, lane);
      if (l > 0) wf.template load_t<kH, kH>(w + W0 + (l > 0 ? l - 1 : 0) * W1, lane);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < kNF; ++i) gm[i] *= elu_deriv_from_value(u[l][i]);
    }
    Op<false, kH> o;
    make_op(gm, o);
    d1[0].mma(df);
    wave_lds_fence();
    stage_op<kH>(tG, Dw1::GP, j, g, o, flip);
    wave_lds_fence();
    typename Dw0::Frags d0f;
    Dw0::load(d0f, tG, tile, lane);
    done(gm, o, sg, nan);
    d0.mma(d0f);
  }

  // Slab: [dW0 kH * K][db0 (node form only)][hidden W, b pairs][last W, b][dgain, dshift]
  __device__ __forceinline__ void store(float* __restrict__ scratch, float* __restrict__ slab, int ln, int wave,
                                        int lane) {
    float* p = slab + kH * K;
    d0.template store<NW>(scratch, slab, p, wave, lane);
    if constexpr (NODE) p += kH;
#pragma unroll
    for (int l = 0; l <= NH; ++l) {
      d1[l].template store<NW>(scratch, p, p + kH * kH, wave, lane);
      p += kHid;
    }
    if (ln) {
      block_sum_vec<kH, NW>(dga, scratch, p, wave, lane);
      block_sum_vec<kH, NW>(dbe, scratch, p + kH, wave, lane);
    }
  }
};

// Per edge, with the forward recomputed (P_i + Q_j given): g_e, the gradient
// g_h at the first pre-activation (summed per sender by k_gq), its sum g_P over
// the receiver's edges, and every weight gradient except those of W0's node
// parts and b0, which k_gq forms from g_P and the senders' sums.  The
// next block's first rows load while this one is computed.  A wave's weight
// sums round in proportion to their own growing size, so a long run is summed
// in a.passes parts, each its own slab (3.5M edges, NH = 5, gradient error
// against FP64: 9.0e-7 in one part, 7.0e-7 in two; FP32 instructions 8.9e-7).
template <int NH>
__global__ __launch_bounds__((64 * Bwd32<NH, 32>::NW), (Bwd32<NH, 32>::OCC)) void k_deep32_edge_bwd(DeepSplitEdgeArgs a) {
  using B = Bwd32<NH, 32>;
  extern __shared__ uint4 smem[];
  const int lane = lane_id(), j = lane & 15, g = lane >> 4, wave = threadIdx.x / 64;
  char* tile = reinterpret_cast<char*>(smem) + wave * B::WTILE;
  char* wl = reinterpret_cast<char*>(smem) + B::NW * B::WTILE;
  float* vecs = reinterpret_cast<float*>(wl + B::WB);
  float* carry = reinterpret_cast<float*>(wl + B::WB + B::VECS) + wave * kH + g * kNF;
  int* slots = reinterpret_cast<int*>(wl + B::WB + B::VECS + B::NW * B::CARRY);
  B::stage(wl, vecs, slots, a.theta, a.theta + 64, 96, a.ln);
  __syncthreads();
  const bool wodd = read_odd(slots);
  const DevGraph& gr = a.g;
  const TileSched ts = tile_sched(gr.n_tiles);
  B acc;
  const int passes = NH ? a.passes : 1;
  bool odd = false;  // an infinite operand met (or a NaN)
  for (int p = 0; p < passes; ++p) {
    acc.zero();
    const int64_t p0 = ts.t0 + (ts.t1 - ts.t0) * p / passes, p1 = ts.t0 + (ts.t1 - ts.t0) * (p + 1) / passes;
    for (int64_t tl = p0 + ts.rank * B::NW + wave; tl < p1; tl += ts.nr * B::NW) {
      const int64_t r0 = gr.tile_r[tl], r1 = gr.tile_r[tl + 1];
      const int64_t e0 = gr.tile_e[tl], e1 = gr.tile_e[tl + 1];
      const int64_t e_last = e1 > e0 ? e1 - 1 : 0;
      int carry_key = 0;
      EdgeIdx ic, in;
      float ne[kNF], np[kNF], nq[kNF];
      auto load = [&](int64_t k, const EdgeIdx& x) {
        load_row<kH>(a.e_in + (k < e1 ? k : e_last) * kH, g, ne);
        load_row<kH>(a.P + (int64_t)x.ri * kH, g, np);
        load_row<kH>(a.Q + (int64_t)x.sj * kH, g, nq);
      };
      auto settle = [&]() {
#pragma unroll
        for (int i = 0; i < kNF; ++i) asm volatile("" : "+v"(ne[i]), "+v"(np[i]), "+v"(nq[i]));
      };
      ic.fetch(gr, e0 + j, e1, e_last);
      in.fetch(gr, e0 + 16 + j, e1, e_last);
      ic.settle();
      load(e0 + j, ic);
      in.settle();
      settle();
      for (int64_t base = e0; base < e1; base += 16) {
        const int ln = lane + opaque_zero(), oz = opaque_zero();
        const int64_t k = base + j;
        const bool valid = k < e1;
        const int64_t kk = valid ? k : e_last;
        const int ri = ic.ri;
        const float inv_d = 1.f / (float)ic.md;
        const bool last = valid && ic.nx != ri;
        const int key = valid ? ri + 1 : -1;
        float z[kNF], ga[kNF], go[kNF], ge[kNF];
        Op<false, kH> oe;
        make_op(ne, oe);
#pragma unroll
        for (int i = 0; i < kNF; ++i) z[i] = np[i] + nq[i];
        load_row<kH>(a.g_a + (int64_t)ri * kH, g, ga);
        if (a.g_e_out) {
          load_row<kH>(a.g_e_out + kk * kH, g, go);
        } else {
#pragma unroll
          for (int i = 0; i < kNF; ++i) go[i] = 0.f;
        }
        load(k + 16, in);
        ic = in;
        in.fetch(gr, k + 32, e1, e_last);
        __builtin_amdgcn_sched_barrier(0);
        acc.run(
            wl + oz, vecs + oz, tile, oe, z, a.ln, a.eps, ln, wave,
            [&](float (&y)[kNF]) {
#pragma unroll
              for (int i = 0; i < kNF; ++i) {
                const float s = ga[i] * inv_d + go[i];
                y[i] = valid ? s : 0.f;
                // the residual path; message aggregation leaves Eq. 4b's part out
                ge[i] = a.am ? go[i] : y[i];
              }
            },
            [&](float (&d)[kNF], const Op<false, kH>& o, float sg, bool nan) {
              gemm_wt<false, kH, kH, ACC_ADD>(wl + oz, o, ge, ln, sg);
              settle();
              in.settle();
#pragma unroll
              for (int i = 0; i < kNF; ++i) d[i] *= sg;
              odd |= nan || ge[0] != ge[0];
              if (valid) {
                store_row<kH>(a.g_e_in + k * kH, g, ge);
                store_row<kH>(a.g_h + k * kH, g, d);
              }
              edge_gp<kH>(d, carry, carry_key, key, last, a.g_P + (int64_t)ri * kH, j, g);
            });
      }
      zero_empty_rows<kH>(gr, r0, r1, a.g_P, lane);
    }
    acc.store(reinterpret_cast<float*>(smem), a.part + ((int64_t)p * gridDim.x + blockIdx.x) * a.slab, a.ln, wave, lane);
  }
  if (!wodd && !__ballot(odd)) return;
  auto pre = [&](int ri, int sj, const float (&e)[kNF], float (&z)[kNF]) {
    float q[kNF];
    load_row<kH>(a.P + (int64_t)ri * kH, g, z);
    load_row<kH>(a.Q + (int64_t)sj * kH, g, q);
#pragma unroll
    for (int i = 0; i < kNF; ++i) z[i] += q[i];
    gemm_exact<kH, kH>(WView{a.theta + 64, 96, 0}, e, z, lane);
  };
  for (int p = 0; p < passes; ++p) {  // the tiles this wave ran, in its passes
    const int64_t p0 = ts.t0 + (ts.t1 - ts.t0) * p / passes, p1 = ts.t0 + (ts.t1 - ts.t0) * (p + 1) / passes;
    for (int64_t tl = p0 + ts.rank * B::NW + wave; tl < p1; tl += ts.nr * B::NW)
      exact_edge_adjoint_tile<kH, NH + 1>(gr, tl, a.e_in, a.g_e_out, a.g_a, a.g_e_in, a.g_h, a.g_P, a.am, carry, pre,
                                          WView{a.theta + 64, 96, 0}, Rest{a.theta, 96}, Rest::Bias{vecs},
                                          a.ln ? vecs + (NH + 2) * kH : nullptr, a.eps, lane);
  }
}

// Adjoint of the node update: g_a (gradient at a*) and g_x = g_out + the MLP's
// part, and all its weight gradients.
template <int NH>
__global__ __launch_bounds__((64 * Bwd32<NH, 64>::NW), (Bwd32<NH, 64>::OCC)) void k_deep32_node_bwd(DeepSplitNodeArgs a) {
  using B = Bwd32<NH, 64>;
  extern __shared__ uint4 smem[];
  const int lane = lane_id(), j = lane & 15, g = lane >> 4, wave = threadIdx.x / 64;
  char* tile = reinterpret_cast<char*>(smem) + wave * B::WTILE;
  char* wl = reinterpret_cast<char*>(smem) + B::NW * B::WTILE;
  float* vecs = reinterpret_cast<float*>(wl + B::WB);
  int* odd = reinterpret_cast<int*>(wl + B::WB + B::VECS + B::NW * B::CARRY);
  B::stage(wl, vecs, odd, a.theta, a.theta, 64, a.ln);
  __syncthreads();
  const bool wodd = read_odd(odd);
  B acc;
  acc.zero();
  const int64_t n = a.n_rows, nblk = (n + 15) / 16;
  for (int64_t blk = (int64_t)blockIdx.x * B::NW + wave; blk < nblk; blk += (int64_t)gridDim.x * B::NW) {
    const int ln = lane + opaque_zero(), oz = opaque_zero();
    const int64_t row = blk * 16 + j, rr = std::min<int64_t>(row, n - 1);
    const bool valid = row < n;
    float s[kNF], x[kNF], go[kNF], z[kNF], gi[2 * kNF];
    load_row<kH>(a.a_star + rr * kH, g, s);
    load_row<kH>(a.x + rr * kH, g, x);
    load_row<kH>(a.g_out + rr * kH, g, go);
    __builtin_amdgcn_sched_barrier(0);
    Op<false, 64> o;
    put_piece(o, 0, s);
    put_piece(o, 1, x);
    load_vec<kH>(vecs + oz, g, z);
    acc.run(
        wl + oz, vecs + oz, tile, o, z, a.ln, a.eps, ln, wave,
        [&](float (&y)[kNF]) {
#pragma unroll
          for (int i = 0; i < kNF; ++i) y[i] = valid ? go[i] : 0.f;
        },
        [&](float (&d)[kNF], const Op<false, kH>& od, float sg, bool nan) {
#pragma unroll
          for (int i = 0; i < kNF; ++i) {
            gi[i] = 0.f;
            gi[kNF + i] = go[i];
          }
          gemm_wt<false, kH, 64, ACC_ADD>(wl + oz, od, gi, ln, sg);
          if (wodd || __ballot(nan || gi[0] != gi[0])) {
            float again[kNF], zz[kNF], u[NH + 1][kNF];
            const float* v = vecs + oz;
            load_vec<kH>(v, g, zz);
            load_row<kH>(a.a_star + rr * kH, g, again);
            gemm_exact<kH, kH>(WView{a.theta, 64, 0}, again, zz, ln);
            load_row<kH>(a.x + rr * kH, g, again);
            gemm_exact<kH, kH>(WView{a.theta + kH, 64, 0}, again, zz, ln);
            exact_forward<kH, NH + 1>(Rest{a.theta, 64}, Rest::Bias{v}, zz, u, ln);
            load_row<kH>(a.g_out + rr * kH, g, d);
#pragma unroll
            for (int i = 0; i < kNF; ++i) {
              gi[i] = 0.f;
              gi[kNF + i] = d[i];
              d[i] = valid ? d[i] : 0.f;
            }
            if (a.ln) ln_adjoint<kH>(zz, d, v + (NH + 2) * kH, a.eps, ln);
            exact_adjoint<kH, NH + 1>(Rest{a.theta, 64}, u, d, ln);
            gemm_exact_t<kH, 64>(WView{a.theta, 64, 0}, d, gi, ln);
          }
          if (valid) {
            store_row<kH>(a.g_a + row * kH, g, *reinterpret_cast<float(*)[kNF]>(gi));
            store_row<kH>(a.g_x + row * kH, g, *reinterpret_cast<float(*)[kNF]>(gi + kNF));
          }
        });
  }
  acc.store(reinterpret_cast<float*>(smem), a.part + blockIdx.x * a.slab, a.ln, wave, lane);
}

// ---------------------------------------------------------------- launchers

template <int NH>
hipError_t edge_fwd(const DeepEdgeArgs& a, int64_t waves, hipStream_t s) {
  using F = Fwd32<NH, 96>;
  constexpr size_t lds = F::WB + F::VECS + F::NW * (kH * sizeof(float) + sizeof(int));
  auto kern = k_deep32_edge_fwd<NH>;
  (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  hipLaunchKernelGGL(kern, dim3((unsigned)((waves + F::NW - 1) / F::NW)), dim3(64 * F::NW), lds, s, a);
  return hipGetLastError();
}
template <int NH>
hipError_t node_fwd(const DeepRowArgs& a, int64_t waves, hipStream_t s) {
  using F = Fwd32<NH, 64>;
  constexpr size_t lds = F::WB + F::VECS + F::NW * sizeof(int);
  auto kern = k_deep32_node_fwd<NH>;
  (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  hipLaunchKernelGGL(kern, dim3((unsigned)((waves + F::NW - 1) / F::NW)), dim3(64 * F::NW), lds, s, a);
  return hipGetLastError();
}
template <int NH>
hipError_t edge_bwd(const DeepSplitEdgeArgs& a, int grid, hipStream_t s) {
  using B = Bwd32<NH, 32>;
  auto kern = k_deep32_edge_bwd<NH>;
  (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)B::LDS);
  hipLaunchKernelGGL(kern, dim3(grid), dim3(64 * B::NW), B::LDS, s, a);
  return hipGetLastError();
}
template <int NH>
hipError_t node_bwd(const DeepSplitNodeArgs& a, int grid, hipStream_t s) {
  using B = Bwd32<NH, 64>;
  auto kern = k_deep32_node_bwd<NH>;
  (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)B::LDS);
  hipLaunchKernelGGL(kern, dim3(grid), dim3(64 * B::NW), B::LDS, s, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_deep32_edge_fwd(const DeepEdgeArgs& a, hipStream_t s) {
  // two waves per tile until the 4096 the chip holds are in flight
  const int64_t waves = std::max<int64_t>(1, std::min<int64_t>(4096, 2 * a.g.n_tiles));
  switch (a.NH) {
    case 0: return edge_fwd<0>(a, waves, s);
    case 1: return edge_fwd<1>(a, waves, s);
    case 2: return edge_fwd<2>(a, waves, s);
    case 3: return edge_fwd<3>(a, waves, s);
    case 4: return edge_fwd<4>(a, waves, s);
    case 5: return edge_fwd<5>(a, waves, s);
  }
  return hipErrorInvalidValue;
}
hipError_t launch_deep32_node_fwd(const DeepRowArgs& a, hipStream_t s) {
  const int64_t waves = std::max<int64_t>(1, std::min<int64_t>(4096, (a.n_rows + 15) / 16));
  switch (a.NH) {
    case 0: return node_fwd<0>(a, waves, s);
    case 1: return node_fwd<1>(a, waves, s);
    case 2: return node_fwd<2>(a, waves, s);
    case 3: return node_fwd<3>(a, waves, s);
    case 4: return node_fwd<4>(a, waves, s);
    case 5: return node_fwd<5>(a, waves, s);
  }
  return hipErrorInvalidValue;
}
hipError_t launch_deep32_edge_bwd(const DeepSplitEdgeArgs& a, int grid, hipStream_t s) {
  switch (a.NH) {
    case 0: return edge_bwd<0>(a, grid, s);
    case 1: return edge_bwd<1>(a, grid, s);
    case 2: return edge_bwd<2>(a, grid, s);
    case 3: return edge_bwd<3>(a, grid, s);
    case 4: return edge_bwd<4>(a, grid, s);
    case 5: return edge_bwd<5>(a, grid, s);
  }
  return hipErrorInvalidValue;
}
hipError_t launch_deep32_node_bwd(const DeepSplitNodeArgs& a, int grid, hipStream_t s) {
  switch (a.NH) {
    case 0: return node_bwd<0>(a, grid, s);
    case 1: return node_bwd<1>(a, grid, s);
    case 2: return node_bwd<2>(a, grid, s);
    case 3: return node_bwd<3>(a, grid, s);
    case 4: return node_bwd<4>(a, grid, s);
    case 5: return node_bwd<5>(a, grid, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace mp
