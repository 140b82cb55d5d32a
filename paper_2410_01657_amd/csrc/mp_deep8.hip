// Deep layers of hidden width 8 (Table I's small model: two extra H -> H layers
// in every MLP): the edge update and the adjoint, for up to kDeep8MaxHidden extra
// layers.
//
// At this width a matrix-unit tile is mostly padding for the MLP itself, so a
// thread runs whole rows with FP32 FMAs on weights broadcast from LDS, two rows
// per thread: a broadcast read feeds four FMAs per row, and with one row the
// LDS reads take longer than the FMAs.  The activations stay in registers, and
// the weight gradients, sums over rows of 8 x 8 outer products, are formed at
// once: a wave lays its 64 rows' factors out column by column in LDS and two
// products fill one 16 x 16 FP32 matrix-unit tile (gradient blocks l, l + 1
// against their inputs).  The record-writing form that serves the other widths
// and depths writes 96 floats per edge for a later pass to read.  As in the
// wide layers, the first edge Linear's node parts are split off: P = W0a x + b0,
// Q = W0b x per node, their adjoint from the sums of g_h over each node's edges.
// 6.3M edges, two extra layers: edge adjoint with its weight gradients 1.31 ms
// in that form, 0.29 ms here (137 bytes per edge: 0.18 ms at the copy rate).
#include "mp_adjoint.hpp"

namespace mp {

namespace {

constexpr int kH = 8;
constexpr int64_t kHid = kH * kH + kH;
constexpr int kWav = 4;              // waves per workgroup
constexpr int kCS = 68;              // column stride of the staged factors (64 rows, padded)
constexpr int kStage = 32 * kCS;     // floats per wave: 16 gradient and 16 input columns

constexpr int64_t off_b0(int K) { return (int64_t)kH * K; }
constexpr int64_t off_hid(int K, int l) { return off_b0(K) + kH + l * kHid; }  // l = NH: the last Linear

__device__ __forceinline__ int zero_after(float a, float b) {
  int z = 0;
  asm volatile("" : "+v"(z) : "v"(a), "v"(b));
  return z;
}

// z[q] += W x[q] for the NQ rows q; W [8][LD] in LDS, M columns.  Four rows of
// weights in flight at a time (each read waits for the previous four sums).
template <int M, int LD, int NQ>
__device__ __forceinline__ void lin2(const float* __restrict__ W, const float (&x)[NQ][M], float (&z)[NQ][kH]) {
#pragma unroll
  for (int o = 0; o < kH; ++o) {
    if (o % 4 == 0) W += o ? zero_after(z[0][o - 1], z[NQ - 1][o - 1]) : opaque_zero();
#pragma unroll
    for (int c = 0; c < M; c += 4) {
      const float4 w = *reinterpret_cast<const float4*>(W + o * LD + c);
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        z[q][o] = fmaf(w.x, x[q][c], z[q][o]);
        z[q][o] = fmaf(w.y, x[q][c + 1], z[q][o]);
        z[q][o] = fmaf(w.z, x[q][c + 2], z[q][o]);
        z[q][o] = fmaf(w.w, x[q][c + 3], z[q][o]);
      }
    }
  }
}
// y[q] = W^T g[q], M columns of W.
template <int M, int LD, int NQ>
__device__ __forceinline__ void lin2_t(const float* __restrict__ W, const float (&g)[NQ][kH], float (&y)[NQ][M]) {
#pragma unroll
  for (int c = 0; c < M; c += 4) {
    W += c ? zero_after(y[0][c - 1], y[NQ - 1][c - 1]) : opaque_zero();
#pragma unroll
    for (int q = 0; q < NQ; ++q) y[q][c] = y[q][c + 1] = y[q][c + 2] = y[q][c + 3] = 0.f;
#pragma unroll
    for (int o = 0; o < kH; ++o) {
      const float4 w = *reinterpret_cast<const float4*>(W + o * LD + c);
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        y[q][c] = fmaf(w.x, g[q][o], y[q][c]);
        y[q][c + 1] = fmaf(w.y, g[q][o], y[q][c + 1]);
        y[q][c + 2] = fmaf(w.z, g[q][o], y[q][c + 2]);
        y[q][c + 3] = fmaf(w.w, g[q][o], y[q][c + 3]);
      }
    }
  }
}

template <int M>
__device__ __forceinline__ void load_vec8(const float* __restrict__ p, float (&v)[M]) {
#pragma unroll
  for (int c = 0; c < M; c += 4) {
    const float4 t = *reinterpret_cast<const float4*>(p + c);
    v[c] = t.x, v[c + 1] = t.y, v[c + 2] = t.z, v[c + 3] = t.w;
  }
}
template <int M>
__device__ __forceinline__ void store_vec8(float* __restrict__ p, const float* v) {
#pragma unroll
  for (int c = 0; c < M; c += 4) *reinterpret_cast<float4*>(p + c) = make_float4(v[c], v[c + 1], v[c + 2], v[c + 3]);
}

// Column block b (of four) of a wave's staged factors.
__device__ __forceinline__ void put_cols(float* __restrict__ st, int b, const float (&v)[kH], int lane) {
#pragma unroll
  for (int c = 0; c < kH; ++c) st[(8 * b + c) * kCS + lane] = v[c];
}
// acc += (blocks 0, 1)^T (blocks 2, 3) over the ROWS staged rows: rows 0..7 x
// columns 0..7 hold block 0 against block 2, rows 8..15 x columns 8..15 block 1
// against block 3 (the rest is not used).  bs, if given, gains the sums of
// column lane % 16 of blocks 0, 1 over this lane's rows.
template <int ROWS = 64>
__device__ __forceinline__ void outer_tile(const float* __restrict__ st, v4f& acc, float* bs, int lane) {
  const float* g = st + (lane & 15) * kCS + 4 * (lane >> 4);
  const float* a = g + 16 * kCS;
#pragma unroll
  for (int r = 0; r < ROWS; r += 16) {
    const float4 gv = *reinterpret_cast<const float4*>(g + r), av = *reinterpret_cast<const float4*>(a + r);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(gv.x, av.x, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(gv.y, av.y, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(gv.z, av.z, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(gv.w, av.w, acc, 0, 0, 0);
    if (bs) *bs += (gv.x + gv.y) + (gv.z + gv.w);
  }
}
// Block `hi` (0: rows and columns 0..7, 1: 8..15) of a tile summed over the
// workgroup's waves (scratch: [wave][256]) and written to dst[8 x ld].
__device__ __forceinline__ void store_block(const v4f& acc, int hi, float* __restrict__ scratch,
                                            float* __restrict__ dst, int ld, int wave, int lane) {
  __syncthreads();
#pragma unroll
  for (int v = 0; v < 4; ++v) scratch[wave * 256 + (4 * (lane >> 4) + v) * 16 + (lane & 15)] = acc[v];
  __syncthreads();
  if (threadIdx.x < 64) {
    const int o = threadIdx.x / 8, c = threadIdx.x % 8;
    float s = 0.f;
    for (int w = 0; w < kWav; ++w) s += scratch[w * 256 + (o + 8 * hi) * 16 + c + 8 * hi];
    dst[o * ld + c] = s;
  }
}
// Columns 8 hi .. of the sums kept by outer_tile, over the lanes and the waves.
__device__ __forceinline__ void store_cols(float v, int hi, float* __restrict__ scratch, float* __restrict__ dst,
                                           int wave, int lane) {
  v += __shfl_xor(v, 16);
  v += __shfl_xor(v, 32);
  __syncthreads();
  if (lane < 16) scratch[wave * 16 + lane] = v;
  __syncthreads();
  if (threadIdx.x < kH) {
    float s = 0.f;
    for (int w = 0; w < kWav; ++w) s += scratch[w * 16 + 8 * hi + threadIdx.x];
    dst[threadIdx.x] = s;
  }
}
// Eight per-lane sums added over the lanes (butterfly) and the waves (in order).
__device__ __forceinline__ void store_sums(float (&v)[kH], float* __restrict__ scratch, float* __restrict__ dst,
                                           int wave, int lane) {
#pragma unroll
  for (int c = 0; c < kH; ++c) {
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) v[c] += __shfl_xor(v[c], o);
  }
  __syncthreads();
  if (lane == 0) {
#pragma unroll
    for (int c = 0; c < kH; ++c) scratch[wave * kH + c] = v[c];
  }
  __syncthreads();
  if (threadIdx.x < kH) {
    float s = 0.f;
    for (int w = 0; w < kWav; ++w) s += scratch[w * kH + threadIdx.x];
    dst[threadIdx.x] = s;
  }
}

// Rows in chunks of `per`: each XCD takes a contiguous eighth of the chunks and
// its waves take them in turn.
struct Chunks {
  int64_t c0, c1, step;
  __device__ __forceinline__ Chunks(int64_t n, int per, int wave) {
    const int64_t nc = (n + per - 1) / per;
    const TileSched ts = tile_sched(nc);
    c0 = ts.t0 + ts.rank * kWav + wave;
    c1 = ts.t1;
    step = ts.nr * kWav;
  }
};

// One MLP's adjoint for NQ rows per thread.  KA 8-wide input blocks take part
// here (edge: e alone, the node parts given in z; node: [a*, x]).
template <int NH, int KA, int NQ>
struct Bwd8 {
  static constexpr int K = 8 * KA;
  // LDS weights: W0 [8][K], hidden W, b pairs, last W, b, gain
  static constexpr int W0 = 0, W1 = kH * K, GAIN = W1 + (NH + 1) * (int)kHid, PAR = GAIN + kH;
  static constexpr int NT = (NH + 1) / 2 + 1 + (KA - 1);  // matrix-unit tiles
  v4f acc[NT];
  float bs[(NH + 1) / 2 + 1];  // column sums of the gradients, as outer_tile forms them
  float dga[kH], dbe[kH];

  __device__ __forceinline__ void zero() {
#pragma unroll
    for (int n = 0; n < NT; ++n) acc[n] = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int n = 0; n < (NH + 1) / 2 + 1; ++n) bs[n] = 0.f;
#pragma unroll
    for (int c = 0; c < kH; ++c) dga[c] = dbe[c] = 0.f;
  }
  // theta: flat parameters of an MLP with KT inputs, of which columns c0.. are used
  static __device__ __forceinline__ void stage(float* __restrict__ L, const float* __restrict__ theta, int KT, int c0,
                                               int ln) {
    for (int t = threadIdx.x; t < kH * K; t += blockDim.x) L[t] = theta[(int64_t)(t / K) * KT + c0 + t % K];
    for (int t = threadIdx.x; t < (NH + 1) * kHid; t += blockDim.x) L[W1 + t] = theta[off_hid(KT, 0) + t];
    for (int t = threadIdx.x; t < kH; t += blockDim.x) L[GAIN + t] = ln ? theta[off_hid(KT, NH + 1) + t] : 0.f;
  }

  // z: the first pre-activation less W0 in; gE(y): the gradients at the output
  // (zero on absent rows); returns the first pre-activation's gradients in z.
  template <class GE>
  __device__ __forceinline__ void run(const float* __restrict__ L, float* __restrict__ st, const float (&in)[NQ][K],
                                      float (&z)[NQ][kH], int ln, float eps, int lane, GE&& gE) {
    float h[NH + 1][NQ][kH], y[NQ][kH], g[NQ][kH];
    lin2<K, K, NQ>(L + W0, in, z);
#pragma unroll
    for (int l = 0; l <= NH; ++l) {
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
#pragma unroll
        for (int c = 0; c < kH; ++c) {
          h[l][q][c] = elu(z[q][c]);
          z[q][c] = 0.f;
        }
      }
      const float* Wl = L + W1 + l * (int)kHid;
#pragma unroll
      for (int q = 0; q < NQ; ++q) load_vec8<kH>(Wl + kH * kH, z[q]);
      lin2<kH, kH, NQ>(Wl, h[l], z);
    }
    gE(y);
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      if (ln) {
        float gain[kH], s = 0.f, v = 0.f, m1 = 0.f, m2 = 0.f;
        load_vec8<kH>(L + GAIN, gain);
#pragma unroll
        for (int c = 0; c < kH; ++c) s += z[q][c];
        const float mean = s * (1.f / kH);
#pragma unroll
        for (int c = 0; c < kH; ++c) v += (z[q][c] - mean) * (z[q][c] - mean);
        const float rstd = 1.f / sqrtf(v * (1.f / kH) + eps);
#pragma unroll
        for (int c = 0; c < kH; ++c) {
          const float xh = (z[q][c] - mean) * rstd;
          dga[c] += y[q][c] * xh;
          dbe[c] += y[q][c];
          g[q][c] = y[q][c] * gain[c];
          m1 += g[q][c];
          m2 += g[q][c] * xh;
          z[q][c] = xh;
        }
        m1 *= 1.f / kH;
        m2 *= 1.f / kH;
#pragma unroll
        for (int c = 0; c < kH; ++c) g[q][c] = rstd * (g[q][c] - m1 - z[q][c] * m2);
      } else {
#pragma unroll
        for (int c = 0; c < kH; ++c) g[q][c] = y[q][c];
      }
    }
    // g = gradient l's pre-activation: l = NH + 1 the output, 0 the first.
    // Gradients 2k and 2k + 1 go through one tile.
    float gp[NQ][kH];  // gradient l + 1
#pragma unroll
    for (int l = NH + 1; l >= 0; --l) {
      if (l % 2 == 0) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
          wave_lds_fence();
          put_cols(st, 0, g[q], lane);
          if (l <= NH) put_cols(st, 1, gp[q], lane);
          if (l > 0)
            put_cols(st, 2, h[l > 0 ? l - 1 : 0][q], lane);
          else
            put_cols(st, 2, *reinterpret_cast<const float(*)[kH]>(&in[q][K - kH]), lane);
          if (l <= NH) put_cols(st, 3, h[l <= NH ? l : NH][q], lane);
          wave_lds_fence();
          outer_tile(st, acc[l / 2], &bs[l / 2], lane);
          if (KA > 1 && l == 0) {
            wave_lds_fence();
            put_cols(st, 2, *reinterpret_cast<const float(*)[kH]>(&in[q][0]), lane);
            wave_lds_fence();
            outer_tile(st, acc[NT - 1], nullptr, lane);
          }
        }
      }
      if (l > 0) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
#pragma unroll
          for (int c = 0; c < kH; ++c) gp[q][c] = g[q][c];
        }
        lin2_t<kH, kH, NQ>(L + W1 + (l > 0 ? l - 1 : 0) * (int)kHid, gp, g);
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
#pragma unroll
          for (int c = 0; c < kH; ++c) g[q][c] *= elu_deriv_from_value(h[l > 0 ? l - 1 : 0][q][c]);
        }
      }
    }
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
#pragma unroll
      for (int c = 0; c < kH; ++c) z[q][c] = g[q][c];
    }
  }

  // Slab: [dW0 8 x K][db0 (node form)][hidden W, b pairs][last W, b][gain, shift]
  __device__ __forceinline__ void store(float* __restrict__ scratch, float* __restrict__ slab, int ln, int wave,
                                        int lane) {
    float* p = slab + kH * K;
    store_block(acc[0], 0, scratch, slab + K - kH, K, wave, lane);
    if constexpr (KA > 1) {
      store_block(acc[NT - 1], 0, scratch, slab, K, wave, lane);
      store_cols(bs[0], 0, scratch, p, wave, lane);
      p += kH;
    }
#pragma unroll
    for (int l = 1; l <= NH + 1; ++l) {
      store_block(acc[l / 2], l % 2, scratch, p, kH, wave, lane);
      store_cols(bs[l / 2], l % 2, scratch, p + kH * kH, wave, lane);
      p += kHid;
    }
    if (ln) {
      store_sums(dga, scratch, p, wave, lane);
      store_sums(dbe, scratch, p + kH, wave, lane);
    }
  }
};

// Two MLP forwards at once, up to the last Linear's output, in z.
template <int NH>
__device__ __forceinline__ void fwd8_tail(const float* __restrict__ L, float (&z)[2][kH]) {
#pragma unroll
  for (int l = 0; l <= NH; ++l) {
    const float* Wl = L + l * (int)kHid;
    float h[2][kH];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
#pragma unroll
      for (int c = 0; c < kH; ++c) h[q][c] = elu(z[q][c]);
      load_vec8<kH>(Wl + kH * kH, z[q]);
    }
    lin2<kH, kH, 2>(Wl, h, z);
  }
}
// LayerNorm of one row, in place.
__device__ __forceinline__ void ln8(const float* __restrict__ gain, float eps, float (&z)[kH]) {
  float s = 0.f, v = 0.f, ga[kH], be[kH];
  load_vec8<kH>(gain, ga);
  load_vec8<kH>(gain + kH, be);
#pragma unroll
  for (int c = 0; c < kH; ++c) s += z[c];
  const float mean = s * (1.f / kH);
#pragma unroll
  for (int c = 0; c < kH; ++c) v += (z[c] - mean) * (z[c] - mean);
  const float rstd = 1.f / sqrtf(v * (1.f / kH) + eps);
#pragma unroll
  for (int c = 0; c < kH; ++c) z[c] = (z[c] - mean) * rstd * ga[c] + be[c];
}

// Edge update and aggregation: a thread walks one receiver's incoming edges
// two at a time, so that a broadcast weight feeds both.  W0 is split as in the
// adjoint: W0a x_i + b0 once per receiver, [W0b | W0c] [x_j, e] per edge.  The
// next pair's rows load while this one is computed.  6.3M edges: 0.26 ms with one
// edge per thread, 0.20 ms here; three waves per SIMD spill and take 0.28.
template <int NH>
__global__ __launch_bounds__(256, 2) void k_deep8_edge_fwd(DeepEdgeArgs a) {
  constexpr int W1 = kH * 16, GAIN = W1 + (NH + 1) * (int)kHid, W0A = GAIN + 2 * kH, B0 = W0A + kH * kH;
  __shared__ float4 par[(B0 + kH) / 4];
  float* L = reinterpret_cast<float*>(par);
  for (int t = threadIdx.x; t < kH * 16; t += blockDim.x) L[t] = a.theta[t / 16 * 24 + kH + t % 16];
  for (int t = threadIdx.x; t < kH * kH; t += blockDim.x) L[W0A + t] = a.theta[t / kH * 24 + t % kH];
  for (int t = threadIdx.x; t < kH; t += blockDim.x) L[B0 + t] = a.theta[off_b0(24) + t];
  for (int t = threadIdx.x; t < (NH + 1) * kHid; t += blockDim.x) L[W1 + t] = a.theta[off_hid(24, 0) + t];
  if (a.ln)
    for (int t = threadIdx.x; t < 2 * kH; t += blockDim.x) L[GAIN + t] = a.theta[off_hid(24, NH + 1) + t];
  __syncthreads();
  // XCD-aware numbering: each XCD's L2 sees a compact window of receivers
  const int64_t i = xcd_block(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x;
  if (i >= a.g.n_rows) return;
  const int k0 = a.g.rowptr[i], k1 = a.g.rowptr[i + 1];
  float p[1][kH], acc[kH], nx[2][kH], ne[2][kH];
  int nd[2];
  auto load = [&](int k) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int kk = std::min(k + q, k1 - 1);
      const int j = a.g.col[kk];
      nd[q] = a.g.mult[kk];
      load_vec8<kH>(a.e_in + (int64_t)kk * kH, ne[q]);
      load_vec8<kH>(a.x + (int64_t)j * kH, nx[q]);
    }
  };
  if (k0 < k1) load(k0);
  {
    float x[1][kH];
    load_vec8<kH>(a.x + i * kH, x[0]);
    load_vec8<kH>(L + B0, p[0]);
    lin2<kH, kH, 1>(L + W0A, x, p);
#pragma unroll
    for (int c = 0; c < kH; ++c) acc[c] = 0.f;
  }
  for (int k = k0; k < k1; k += 2) {
    float in[2][16], z[2][kH];
    int d[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      d[q] = nd[q];
#pragma unroll
      for (int c = 0; c < kH; ++c) {
        in[q][c] = nx[q][c];
        in[q][kH + c] = ne[q][c];
        z[q][c] = p[0][c];
      }
    }
    if (k + 2 < k1) load(k + 2);
    __builtin_amdgcn_sched_barrier(0);
    lin2<16, 16, 2>(L, in, z);
    fwd8_tail<NH>(L + W1, z);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      if (k + q >= k1) continue;
      if (a.ln) ln8(L + GAIN, a.eps, z[q]);
      const float inv_d = 1.f / (float)d[q];
#pragma unroll
      for (int c = 0; c < kH; ++c) {
        const float msg = z[q][c];
        z[q][c] += in[q][kH + c];                     // residual edge update (Eq. 4a)
        acc[c] += (a.am ? msg : z[q][c]) * inv_d;     // Eq. 4b (or the message variant)
      }
      store_vec8<kH>(a.e_out + (int64_t)(k + q) * kH, z[q]);
    }
  }
  store_vec8<kH>(a.a_out + i * kH, acc);
}

// P = W0a x + b0, Q = W0b x: one node per thread.
__global__ __launch_bounds__(256) void k_deep8_proj(int64_t n, const float* __restrict__ x,
                                                    const float* __restrict__ theta, float* __restrict__ P,
                                                    float* __restrict__ Q) {
  __shared__ float4 Ls[34];
  float* L = reinterpret_cast<float*>(Ls);
  for (int t = threadIdx.x; t < 136; t += blockDim.x)
    L[t] = t < 128 ? theta[(t % 64 / 8) * 24 + (t / 64) * 8 + t % 8] : theta[off_b0(24) + t - 128];
  __syncthreads();
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= n) return;
  float xv[kH], p[kH], q[kH];
  load_vec8<kH>(x + r * kH, xv);
  load_vec8<kH>(L + 128, p);
#pragma unroll
  for (int o = 0; o < kH; ++o) {
    q[o] = 0.f;
#pragma unroll
    for (int c = 0; c < kH; ++c) {
      p[o] = fmaf(L[o * 8 + c], xv[c], p[o]);
      q[o] = fmaf(L[64 + o * 8 + c], xv[c], q[o]);
    }
  }
  store_vec8<kH>(P + r * kH, p);
  store_vec8<kH>(Q + r * kH, q);
}

template <int NH>
__global__ __launch_bounds__(64 * kWav, 2) void k_deep8_edge_bwd(DeepSplitEdgeArgs a) {
  using B = Bwd8<NH, 1, 2>;
  __shared__ float4 par[(B::PAR + 3) / 4];
  __shared__ float4 stage[kWav * kStage / 4];
  float* L = reinterpret_cast<float*>(par);
  const int lane = lane_id(), wave = threadIdx.x / 64;
  float* st = reinterpret_cast<float*>(stage) + wave * kStage;
  B::stage(L, a.theta, 24, 16, a.ln);
  __syncthreads();
  B acc;
  acc.zero();
  const int64_t E = a.g.n_edges;
  const Chunks ch(E, 128, wave);
  for (int64_t c = ch.c0; c < ch.c1; c += ch.step) {
    int64_t k[2], kk[2];
    int ri[2], sj[2], md[2];
    float e[2][kH], z[2][kH], qv[2][kH], ge[2][kH], go[2][kH];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      k[q] = c * 128 + 64 * q + lane;
      kk[q] = std::min(k[q], E - 1);
      ri[q] = a.g.recv[kk[q]];
      sj[q] = a.g.col[kk[q]];
      md[q] = a.g.mult[kk[q]];
      load_vec8<kH>(a.e_in + kk[q] * kH, e[q]);
      if (a.g_e_out) {
        load_vec8<kH>(a.g_e_out + kk[q] * kH, go[q]);
      } else {
#pragma unroll
        for (int i = 0; i < kH; ++i) go[q][i] = 0.f;
      }
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      load_vec8<kH>(a.P + (int64_t)ri[q] * kH, z[q]);
      load_vec8<kH>(a.Q + (int64_t)sj[q] * kH, qv[q]);
      load_vec8<kH>(a.g_a + (int64_t)ri[q] * kH, ge[q]);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
#pragma unroll
      for (int i = 0; i < kH; ++i) z[q][i] += qv[q][i];
    }
    acc.run(L, st, e, z, a.ln, a.eps, lane, [&](float (&y)[2][kH]) {
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const float inv_d = 1.f / (float)md[q];
#pragma unroll
        for (int i = 0; i < kH; ++i) {
          const float s = fmaf(ge[q][i], inv_d, go[q][i]);
          y[q][i] = k[q] < E ? s : 0.f;
          // the residual path; message aggregation leaves Eq. 4b's part out
          ge[q][i] = a.am ? go[q][i] : y[q][i];
        }
      }
    });
    float t[2][kH];
    lin2_t<kH, kH, 2>(L + B::W0, z, t);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
#pragma unroll
      for (int i = 0; i < kH; ++i) t[q][i] += ge[q][i];
      if (k[q] < E) {
        store_vec8<kH>(a.g_e_in + k[q] * kH, t[q]);
        store_vec8<kH>(a.g_h + k[q] * kH, z[q]);
      }
    }
  }
  acc.store(reinterpret_cast<float*>(stage), a.part + blockIdx.x * a.slab, a.ln, wave, lane);
}

template <int NH>
__global__ __launch_bounds__(64 * kWav, 2) void k_deep8_node_bwd(DeepSplitNodeArgs a) {
  constexpr int NQ = 1;  // two rows do not fit in the registers
  using B = Bwd8<NH, 2, NQ>;
  __shared__ float4 par[(B::PAR + kH + 3) / 4];
  __shared__ float4 stage[kWav * kStage / 4];
  float* L = reinterpret_cast<float*>(par);
  const int lane = lane_id(), wave = threadIdx.x / 64;
  float* st = reinterpret_cast<float*>(stage) + wave * kStage;
  B::stage(L, a.theta, 16, 0, a.ln);
  for (int t = threadIdx.x; t < kH; t += blockDim.x) L[B::PAR + t] = a.theta[off_b0(16) + t];
  __syncthreads();
  B acc;
  acc.zero();
  const int64_t n = a.n_rows;
  const Chunks ch(n, 64 * NQ, wave);
  for (int64_t c = ch.c0; c < ch.c1; c += ch.step) {
    float in[NQ][2 * kH], z[NQ][kH], go[NQ][kH];
    int64_t r[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      r[q] = (c * NQ + q) * 64 + lane;
      const int64_t rr = std::min(r[q], n - 1);
      load_vec8<kH>(a.a_star + rr * kH, *reinterpret_cast<float(*)[kH]>(&in[q][0]));
      load_vec8<kH>(a.x + rr * kH, *reinterpret_cast<float(*)[kH]>(&in[q][kH]));
      load_vec8<kH>(a.g_out + rr * kH, go[q]);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < NQ; ++q) load_vec8<kH>(L + B::PAR, z[q]);
    acc.run(L, st, in, z, a.ln, a.eps, lane, [&](float (&y)[NQ][kH]) {
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
#pragma unroll
        for (int i = 0; i < kH; ++i) y[q][i] = r[q] < n ? go[q][i] : 0.f;
      }
    });
    float t[NQ][2 * kH];
    lin2_t<2 * kH, 2 * kH, NQ>(L + B::W0, z, t);
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
#pragma unroll
      for (int i = 0; i < kH; ++i) t[q][kH + i] += go[q][i];
      if (r[q] < n) {
        store_vec8<kH>(a.g_a + r[q] * kH, &t[q][0]);
        store_vec8<kH>(a.g_x + r[q] * kH, &t[q][kH]);
      }
    }
  }
  acc.store(reinterpret_cast<float*>(stage), a.part + blockIdx.x * a.slab, a.ln, wave, lane);
}

// Per node: g_P = sum of g_h over its incoming edges, g_Q over the reverses of
// them (its outgoing edges), in CSR order; g_x = g_add + W0a^T g_P + W0b^T g_Q;
// dW0a = sum g_P x^T, dW0b = sum g_Q x^T, db0 = sum g_P.  Bound by the two
// passes over g_h; two lanes share a node, half a row each, so that neighbouring
// lanes read one 32-byte row and six edges' rows fit in flight (6.3M edges: 163 us
// with one lane per node, 114 so).  Slab: [dW0a][dW0b][db0].
__global__ __launch_bounds__(64 * kWav, 4) void k_deep8_gq(Deep8GqArgs a) {
  __shared__ float4 par[32];
  __shared__ float4 stage[kWav * kStage / 4];
  float* L = reinterpret_cast<float*>(par);
  for (int t = threadIdx.x; t < 128; t += blockDim.x) L[t] = a.theta[(t % 64 / 8) * 24 + (t / 64) * 8 + t % 8];
  __syncthreads();
  const int lane = lane_id(), wave = threadIdx.x / 64, hf = lane & 1;
  float* st = reinterpret_cast<float*>(stage) + wave * kStage;
  float* mine = st + 4 * hf * kCS + lane / 2;
  const DevGraph& gr = a.g;
  const int64_t n = gr.n_rows;
  constexpr int CH = 6;
  v4f acc = v4f{0.f, 0.f, 0.f, 0.f};
  float b0 = 0.f;
  const Chunks ch(n, 32, wave);
  for (int64_t c = ch.c0; c < ch.c1; c += ch.step) {
    const int64_t r = c * 32 + lane / 2, rr = std::min(r, n - 1);
    const bool valid = r < n;
    const int k0 = gr.rowptr[rr], k1 = valid ? gr.rowptr[rr + 1] : k0;
    const float* gh = a.g_h + 4 * hf;
    float v[3][4], gx[4];  // g_P, g_Q, x
    load_vec8<4>(a.x + rr * kH + 4 * hf, v[2]);
    load_vec8<4>(a.g_add + rr * kH + 4 * hf, gx);
#pragma unroll
    for (int i = 0; i < 4; ++i) v[0][i] = v[1][i] = 0.f;
    // six edges at a time: their reverse indices first, then all their rows
    for (int kb = k0; kb < k1; kb += CH) {
      int rv[CH];
#pragma unroll
      for (int q = 0; q < CH; ++q) rv[q] = gr.rev[std::min(kb + q, k1 - 1)];
      float ti[CH][4], tj[CH][4];
#pragma unroll
      for (int q = 0; q < CH; ++q) {
        load_vec8<4>(gh + (int64_t)std::min(kb + q, k1 - 1) * kH, ti[q]);
        load_vec8<4>(gh + (int64_t)rv[q] * kH, tj[q]);
      }
#pragma unroll
      for (int q = 0; q < CH; ++q) {
        if (kb + q < k1) {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            v[0][i] += ti[q][i];
            v[1][i] += tj[q][i];
          }
        }
      }
    }
    wave_lds_fence();
#pragma unroll
    for (int b = 0; b < 4; ++b) {
#pragma unroll
      for (int i = 0; i < 4; ++i) mine[(8 * b + i) * kCS] = v[b < 2 ? b : 2][i];
    }
    wave_lds_fence();
    outer_tile<32>(st, acc, &b0, lane);
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      // the whole row: lane l and its neighbour's half (quad_perm 1, 0, 3, 2)
      float g[kH];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float o = __builtin_bit_cast(
            float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v[b][i]), 0xB1, 0xF, 0xF, true));
        g[i] = hf ? o : v[b][i];
        g[4 + i] = hf ? v[b][i] : o;
      }
      const float* W = L + 64 * b + 4 * hf;
#pragma unroll
      for (int o = 0; o < kH; ++o) {
        float w[4];
        load_vec8<4>(W + o * kH, w);
#pragma unroll
        for (int i = 0; i < 4; ++i) gx[i] = fmaf(w[i], g[o], gx[i]);
      }
    }
    if (valid) store_vec8<4>(a.g_x + r * kH + 4 * hf, gx);
  }
  float* slab = a.part + blockIdx.x * a.slab;
  float* scratch = reinterpret_cast<float*>(stage);
  store_block(acc, 0, scratch, slab, kH, wave, lane);
  store_block(acc, 1, scratch, slab + 64, kH, wave, lane);
  store_cols(b0, 0, scratch, slab + 128, wave, lane);
}

}  // namespace

hipError_t launch_deep8_proj(int64_t n, const float* x, const float* theta, float* P, float* Q, hipStream_t s) {
  hipLaunchKernelGGL(k_deep8_proj, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, n, x, theta, P, Q);
  return hipGetLastError();
}
hipError_t launch_deep8_edge_fwd(const DeepEdgeArgs& a, hipStream_t s) {
  const dim3 grid((unsigned)((a.g.n_rows + 255) / 256));
#define MP_CASE(NN)                                                          \
  if (a.NH == NN) {                                                          \
    hipLaunchKernelGGL(k_deep8_edge_fwd<NN>, grid, dim3(256), 0, s, a);      \
    return hipGetLastError();                                                \
  }
  MP_CASE(0) MP_CASE(1) MP_CASE(2) MP_CASE(3) MP_CASE(4) MP_CASE(5)
#undef MP_CASE
  return hipErrorInvalidValue;
}
hipError_t launch_deep8_edge_bwd(const DeepSplitEdgeArgs& a, int grid, hipStream_t s) {
#define MP_CASE(NN)                                                                       \
  if (a.NH == NN) {                                                                       \
    hipLaunchKernelGGL(k_deep8_edge_bwd<NN>, dim3(grid), dim3(64 * kWav), 0, s, a);       \
    return hipGetLastError();                                                             \
  }
  MP_CASE(0) MP_CASE(1) MP_CASE(2) MP_CASE(3) MP_CASE(4) MP_CASE(5)
#undef MP_CASE
  return hipErrorInvalidValue;
}
hipError_t launch_deep8_node_bwd(const DeepSplitNodeArgs& a, int grid, hipStream_t s) {
#define MP_CASE(NN)                                                                       \
  if (a.NH == NN) {                                                                       \
    hipLaunchKernelGGL(k_deep8_node_bwd<NN>, dim3(grid), dim3(64 * kWav), 0, s, a);       \
    return hipGetLastError();                                                             \
  }
  MP_CASE(0) MP_CASE(1) MP_CASE(2) MP_CASE(3) MP_CASE(4) MP_CASE(5)
#undef MP_CASE
  return hipErrorInvalidValue;
}
hipError_t launch_deep8_gq(const Deep8GqArgs& a, int grid, hipStream_t s) {
  hipLaunchKernelGGL(k_deep8_gq, dim3(grid), dim3(64 * kWav), 0, s, a);
  return hipGetLastError();
}

}  // namespace mp
