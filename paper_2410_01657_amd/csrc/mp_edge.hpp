// A 16-edge block's indices and its segmented sum per receiver.
#pragma once
#include "mp_device.hpp"
#include "mp_kernels.hpp"

namespace mp {

// Indices of one edge per lane: receiver, sender, multiplicity, and the next
// edge's receiver (-1 past the tile); past the tile's end those of e_last.
struct EdgeIdx {
  int ri, sj, md, nx;
  __device__ __forceinline__ void fetch(const DevGraph& gr, int64_t k, int64_t e1, int64_t e_last) {
    const int64_t kk = k < e1 ? k : e_last;
    ri = gr.recv[kk];
    sj = gr.col[kk];
    md = gr.mult[kk];
    nx = (k + 1 < e1) ? gr.recv[k + 1] : -1;
  }
  // Complete the loads here: the loop's entry state (or the stores that
  // follow) then has no pending loads, else the compiler's wait for them
  // also drains the stores.
  __device__ __forceinline__ void settle() { asm volatile("" : "+v"(ri), "+v"(sj), "+v"(md), "+v"(nx)); }
};

// rows without incoming edges have g_P = 0
template <int H>
__device__ __forceinline__ void zero_empty_rows(const DevGraph& gr, int64_t r0, int64_t r1, float* __restrict__ g_P,
                                                int lane) {
  for (int64_t r = r0 + (lane >> 2); r < r1; r += 16) {
    if (gr.rowptr[r] == gr.rowptr[r + 1]) {
      float* dst = g_P + r * H;
      for (int c = (lane & 3) * 4; c < H; c += 16) *reinterpret_cast<float4*>(dst + c) = make_float4(0.f, 0.f, 0.f, 0.f);
    }
  }
}

// g_P of one block: segmented sum of gh per receiver, the open row's partial
// sum handed from lane 15 of one block to lane 0 of the next through LDS
// (same wave, so no barrier is needed).  Lanes past the tile's last edge hold
// gh = 0 and a key of their own, so they add nothing to any row's sum.
template <int H>
__device__ __forceinline__ void edge_gp(float (&t)[H / 4], float* __restrict__ carry, int& carry_key, int key,
                                        bool last, float* __restrict__ dst, int j, int g) {
  constexpr int NF = H / 4;
  if (j == 0 && key == carry_key) {
#pragma unroll
    for (int i = 0; i < NF; i += 4) {
      const float4 c = *reinterpret_cast<const float4*>(carry + i);
      t[i] += c.x;
      t[i + 1] += c.y;
      t[i + 2] += c.z;
      t[i + 3] += c.w;
    }
  }
  seg_scan16<NF>(t, key);
  if (last) store_row<H>(dst, g, t);
  if (j == 15) {
#pragma unroll
    for (int i = 0; i < NF; i += 4) *reinterpret_cast<float4*>(carry + i) = make_float4(t[i], t[i + 1], t[i + 2], t[i + 3]);
  }
  carry_key = from_prev_lane_i(key);
}

}  // namespace mp
