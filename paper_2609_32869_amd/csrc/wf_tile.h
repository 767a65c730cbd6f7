// One block's tile of a product whose four waves split k (internal): used by the prompt
// pass (k_pre.hip) and by the several-slot step (k_gemv.hip).
#pragma once
#include "wf_kernels.h"
#include "wf_operand.h"
#include "wf_split.h"

namespace wf {

// The tile of this block (xcd_blocks, wf_split.h: XCD x = block % 8); false for a block past
// the grid of tiles.
__device__ __forceinline__ bool xcd_tile(int nmb, int nnb, int rs, int& mbk, int& nbk) {
  const int x = blockIdx.x & 7, bi = blockIdx.x >> 3;
  const int nrh = (nmb + rs - 1) / rs, ncq = (nnb * rs + 7) / 8;
  mbk = (x % rs) * nrh + bi % nrh;
  nbk = (x / rs) * ncq + bi / nrh;
  return mbk < nmb && bi / nrh < ncq && nbk < nnb;
}

// Rows 8 (lane / 32) .. + 7 of half `half` (16 rows) of a 32 x 32 accumulator, this lane's
// column, + bias, as eight bf16: the two row groups change places between half-waves.
__device__ __forceinline__ uint4 rows8_bf16(const floatx16& c, int half, float bias) {
  uint32_t p[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) p[e] = pack2_bf16(c[8 * half + 2 * e] + bias, c[8 * half + 2 * e + 1] + bias);
  const auto x = __builtin_amdgcn_permlane32_swap(p[0], p[2], false, false);
  const auto y = __builtin_amdgcn_permlane32_swap(p[1], p[3], false, false);
  return make_uint4(x[0], y[0], x[1], y[1]);
}

// The sum over the P planes of A[m, k] W[n, k] for a tile of 32 TI rows from m0 and 32 TJ
// columns from n0: on return wave w holds tiles w Q .. w Q + Q - 1 (tile i TJ + j), Q =
// TI TJ / 4, in `sum`, each as the 32 x 32 x 16 instruction's accumulator (element v: row
// 8 (v / 4) + 4 (lane / 32) + v % 4, column lane % 32).  Wave w takes the 16-wide k units
// w, w + 4, ... of split y of `ny` for the whole tile, so every operand byte is loaded
// by one wave only, straight into registers and D units ahead: no LDS and no barrier
// in the loop.  With the tile split over the waves instead and the fragments staged in
// LDS, each fragment is read by two waves, and that traffic (48 KB per k-step of a 64 x
// 64 three-plane tile) took longer than the matrix work it feeds.
// A: 16-row fragment order, mt row tiles.  W: 16-column (W_F16) or 32-column (W_F32)
// fragment order; either is read by picking each lane's 16 bytes.  Tiles past the
// data re-read the last one; their results are not to be written.
// `red`: float4 [3][R][4][4][64], R = min(Q, 2), free again after the caller's barrier.
template <int P, int WK, int TI, int TJ, int D>
__device__ __forceinline__ void split_tile(const void* a_, int mt, const void* w_, int K, int N, int m0, int n0, int y, int ny,
                                           floatx16* sum, float4 (*red)[TI * TJ / 4 < 2 ? 1 : 2][4][4][64]) {
  constexpr int NW = 4, Q = TI * TJ / NW;
  static_assert(TI * TJ % NW == 0, "the waves finish equal shares");
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lr = lane & 31, lk = lane >> 5;
  const int KS = K / 32, ku = 2 * (KS / ny), u0 = min(y * ku + wv, 2 * KS - 1), n = (ku - wv + NW - 1) / NW;
  // this lane's 16 bytes of each row / column tile (tiles past the data re-read the
  // last one; their results are not written); unit u0 + 4 t lies t strides on
  const uint4* A0 = reinterpret_cast<const uint4*>(a_) + (size_t)(u0 >> 1) * mt * 64 + 32 * (u0 & 1);
  const uint4* W0 = reinterpret_cast<const uint4*>(w_) + (size_t)u0 * (WK == W_F16 ? 32 : 64);
  const size_t plane = (size_t)mt * KS * 64, sa = (size_t)2 * mt * 64;
  constexpr int sw = NW * (WK == W_F16 ? 32 : 64);
  int oa[TI], ow[TJ];
#pragma unroll
  for (int i = 0; i < TI; ++i) oa[i] = min(m0 / 16 + 2 * i + (lr >> 4), mt - 1) * 64 + (lr & 15) + 16 * lk;
#pragma unroll
  for (int j = 0; j < TJ; ++j)
    ow[j] = WK == W_F16 ? min(n0 / 16 + 2 * j + (lr >> 4), (N + 15) / 16 - 1) * KS * 64 + (lr & 15) + 16 * lk
                        : min(n0 / 32 + j, (N + 31) / 32 - 1) * 2 * KS * 64 + lane;
  struct Frag {
    bf16x8 a[P][TI], w[TJ];
  };
  auto load = [&](int t, Frag& f) {  // the wave's unit t (past the end: the last one; with none, some unit of K)
    const int tt = max(min(t, n - 1), 0);
    const uint4 *At = A0 + tt * sa, *Wt = W0 + (size_t)tt * sw;
#pragma unroll
    for (int j = 0; j < TJ; ++j) f.w[j] = __builtin_bit_cast(bf16x8, Wt[ow[j]]);
#pragma unroll
    for (int h = 0; h < P; ++h)
#pragma unroll
      for (int i = 0; i < TI; ++i) f.a[h][i] = __builtin_bit_cast(bf16x8, (At + h * plane)[oa[i]]);
  };
  floatx16 acc[TI][TJ];
#pragma unroll
  for (int i = 0; i < TI; ++i)
#pragma unroll
    for (int j = 0; j < TJ; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
  auto mul = [&](const Frag& f) {
#pragma unroll
    for (int h = 0; h < P; ++h)
#pragma unroll
      for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TJ; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.a[h][i], f.w[j], acc[i][j], 0, 0, 0);
  };
  // D units in flight; the scheduling barriers keep every load where it is issued
  Frag fr[D];
#pragma unroll
  for (int d = 0; d < D; ++d) load(d, fr[d]);
  __builtin_amdgcn_sched_barrier(0);
  int t = 0;
  for (; t + 2 * D <= n; t += D) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      mul(fr[d]);
      __builtin_amdgcn_sched_barrier(0);
      load(t + d + D, fr[d]);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  // units t .. n - 1 are left, the first D of them in flight
  const int rest = n - t - D;
  if (rest > 0) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      mul(fr[d]);
      __builtin_amdgcn_sched_barrier(0);
      load(t + d + D, fr[d]);
      __builtin_amdgcn_sched_barrier(0);
    }
    t += D;
  }
#pragma unroll
  for (int d = 0; d < D; ++d)
    if (t + d < n) mul(fr[d]);

  // the other waves' parts through LDS in the instruction's own order, 16 bytes per lane,
  // R tiles a round
  constexpr int R = Q < 2 ? Q : 2;
#pragma unroll
  for (int q = 0; q < NW * Q; ++q)
    if (q / Q == wv) sum[q % Q] = acc[q / TJ][q % TJ];
#pragma unroll
  for (int r0 = 0; r0 < Q; r0 += R) {
    if (r0 > 0) __syncthreads();
#pragma unroll
    for (int q = 0; q < NW * Q; ++q) {
      const int own = q / Q, r = q % Q - r0;
      if (r < 0 || r >= R || own == wv) continue;
#pragma unroll
      for (int v = 0; v < 4; ++v)
        red[wv < own ? wv : wv - 1][r][v][own][lane] =
            make_float4(acc[q / TJ][q % TJ][4 * v], acc[q / TJ][q % TJ][4 * v + 1], acc[q / TJ][q % TJ][4 * v + 2],
                        acc[q / TJ][q % TJ][4 * v + 3]);
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int s = 0; s < NW - 1; ++s)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const float4 o = red[s][r][v][wv][lane];
          sum[r0 + r][4 * v] += o.x;
          sum[r0 + r][4 * v + 1] += o.y;
          sum[r0 + r][4 * v + 2] += o.z;
          sum[r0 + r][4 * v + 3] += o.w;
        }
  }
}

}  // namespace wf
