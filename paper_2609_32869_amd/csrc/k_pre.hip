// Prompt pass (prefill) over many rows at once, bf16 storage (gfx950, wave64).
//
// The step's kernels take nine rows per slot; a prompt run through them reads
// every weight once per nine positions (large-v3, 227 tokens: 26 passes of 1.4 ms).
// Here the prompts of all slots are cut into parts of 16 consecutive positions (one
// cache page, and the 16 rows of a matrix tile), and one pass runs all parts of
// the call: row part * 16 + i is position pos0 + i of the part's slot.  A block's
// keys and values are appended by its q|k|v product before its attention reads
// the cache, so the parts of one prompt can share the pass.
//
// Operands are P bf16 planes in 16-row fragment order (wf_common.h): P = 3 (hi, mid,
// lo: the exact fp32 value) for handles of one slot and P = 2 (hi, lo: 2^-17) for
// several, as in the step.
#include <algorithm>

#include "wf_common.h"
#include "wf_kernels.h"
#include "wf_operand.h"
#include "wf_tile.h"

namespace wf {

namespace {
// The 8 values of a row's columns k .. k + 7 into the P planes of an operand whose
// 16-byte chunk index is i (planes `plane` chunks apart).
template <int P>
__device__ __forceinline__ void put_planes8(uint4* A, size_t i, size_t plane, const float* v) {
  if constexpr (P == 3) split3x8(v, A[i], A[i + plane], A[i + 2 * plane]);
  else split2x8(v, A[i], A[i + plane]);
}
}  // namespace

// ---------------------------------------------------------------- set-up
// h[row] = E[token] + P[position] of every part's 16 rows (rows past the prompt take
// its last position's; their results are never read).
__global__ void __launch_bounds__(256) k_pre_begin(PreArgs a) {
  const PrePart p = a.parts[blockIdx.x];
  const int nch = a.d >> 3;
  const bf16* E = reinterpret_cast<const bf16*>(a.emb);
  const bf16* Pt = reinterpret_cast<const bf16*>(a.pos);
  for (int t = blockIdx.y * 256 + threadIdx.x; t < kPrePart * nch; t += gridDim.y * 256) {
    const int i = t / nch, c = 8 * (t - i * nch), pos = p.pos0 + min(i, p.nv - 1);
    const int tok = min(max(a.tokens[(size_t)(p.slot - a.slot0) * a.pmax + pos], 0), a.n_vocab - 1);
    const size_t ei = a.emb_kind == W_F32 ? wfrag32_index(tok, c, a.d / 16) : wfrag16_index(tok, c, a.d / 32);
    float e8[8], p8[8];
    ld8(E + ei, e8);
    ld8(Pt + (size_t)pos * a.d + c, p8);
    float4* hr = reinterpret_cast<float4*>(a.h + (size_t)(blockIdx.x * kPrePart + i) * a.d + c);
    hr[0] = make_float4(e8[0] + p8[0], e8[1] + p8[1], e8[2] + p8[2], e8[3] + p8[3]);
    hr[1] = make_float4(e8[4] + p8[4], e8[5] + p8[5], e8[6] + p8[6], e8[7] + p8[7]);
  }
}

// The hidden row of each prompt's last position, for the vocabulary head (row 0 of
// the slot's nine).
__global__ void __launch_bounds__(256) k_pre_last(PreArgs a, float* __restrict__ lasth) {
  const PrePart p = a.parts[blockIdx.x];
  if (!p.last) return;
  const float* src = a.h + (size_t)(blockIdx.x * kPrePart + p.nv - 1) * a.d;
  for (int c = threadIdx.x; c < a.d; c += 256) lasth[(size_t)p.slot * kRows * a.d + c] = src[c];
}

// ---------------------------------------------------------------- residual + LayerNorm
// One block per row, a thread per 8 consecutive columns (d <= 2048): the row takes
// the product's partial sums and bias (nparts > 0; fresh: the row starts at zero),
// goes out as the drafter tap when tapcol >= 0, and its LayerNorm (g non-null)
// becomes the next product's operand.  Memory-bound: every load is issued first
// and 16 bytes wide.
template <int P>
__global__ void __launch_bounds__(256) k_pre_rln(PreLnArgs a) {
  StampScope stamp_scope(a.stamp, blockDim.x);
  __shared__ float red[2][4];
  const int row = blockIdx.x, d = a.d, nch = d >> 3, c = threadIdx.x, cc = min(c, nch - 1);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  const bool act = c < nch, sums = a.nparts > 0, has_ln = a.g != nullptr;
  float* hr = a.h + (size_t)row * d;
  float v[8], pv[kPreMaxSplit][8], bv[8], gv[8], lv[8];
  ld8(hr + 8 * cc, v);
  if (sums) {
#pragma unroll
    for (int p = 0; p < kPreMaxSplit; ++p) ld8(a.part + min(p, a.nparts - 1) * a.pstride + (size_t)row * d + 8 * cc, pv[p]);
    ld8(a.bias + 8 * cc, bv);
  }
  if (has_ln) {
    ld8(a.g + 8 * cc, gv);
    ld8(a.b + 8 * cc, lv);
  }
  float s = 0.f;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    if (sums) {
      float t = 0.f;
#pragma unroll
      for (int p = 0; p < kPreMaxSplit; ++p) t += p < a.nparts ? pv[p][e] : 0.f;
      v[e] = (a.fresh ? 0.f : v[e]) + (t + bv[e]);
    }
    if (!act) v[e] = 0.f;
    s += v[e];
  }
  const size_t ti = afrag16_index(row, a.tapcol >= 0 ? a.tapcol + 8 * cc : 0, a.mt) / 8;
  if (act) {
    if (sums) {
      float4* y = reinterpret_cast<float4*>(hr + 8 * c);
      y[0] = make_float4(v[0], v[1], v[2], v[3]);
      y[1] = make_float4(v[4], v[5], v[6], v[7]);
    }
    if (a.tapcol >= 0) put_planes8<P>(reinterpret_cast<uint4*>(a.tap), ti, (size_t)a.mt * 2 * a.tapld, v);
  }
  if (!has_ln) return;
  s = wave_sum(s);
  if (lane == 0) red[0][w] = s;
  __syncthreads();
  float tot = 0.f;
  for (int i = 0; i < nw; ++i) tot += red[0][i];
  const float mean = tot / (float)d;
  float q = 0.f;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const float cd = v[e] - mean;
    q += act ? cd * cd : 0.f;
  }
  q = wave_sum(q);
  if (lane == 0) red[1][w] = q;
  __syncthreads();
  float qt = 0.f;
  for (int i = 0; i < nw; ++i) qt += red[1][i];
  const float inv = 1.0f / sqrtf(qt / (float)d + 1e-5f);
  if (act) {
    float y[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) y[e] = (v[e] - mean) * inv * gv[e] + lv[e];
    put_planes8<P>(reinterpret_cast<uint4*>(a.out), afrag16_index(row, 8 * c, a.mt) / 8, (size_t)a.mt * 2 * d, y);
  }
}

// ---------------------------------------------------------------- products
// A block per 32 TI x 32 TJ tile (split_tile, wf_tile.h); grid y splits the k units
// (PRE_PART: one buffer of partial sums per split).
template <int EPI, int P, int WK, int TI, int TJ, int D>
__global__ void __launch_bounds__(256, 1) k_pre_gemm(PreGemmArgs a, int nmb, int nnb, int rs) {
  StampScope stamp_scope(a.stamp, 256);
  constexpr int NW = 4, Q = TI * TJ / NW;
  __shared__ float4 red[NW - 1][Q < 2 ? 1 : 2][4][NW][64];
  int mbk, nbk;
  if (!xcd_tile(nmb, nnb, rs, mbk, nbk)) return;
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lr = lane & 31, lk = lane >> 5, m0 = mbk * 32 * TI, n0 = nbk * 32 * TJ;
  floatx16 sum[Q];
  split_tile<P, WK, TI, TJ, D>(a.a, a.mt, a.w, a.K, a.N, m0, n0, blockIdx.y, gridDim.y, sum, red);
  if constexpr (EPI == PRE_GELU) __syncthreads();

  // accumulator v of a 32 x 32 tile: row 8 (v / 4) + 4 (lane / 32) + v % 4, column lane % 32
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int tile = wv * Q + q, nt = n0 + 32 * (tile % TJ), mt0 = m0 + 32 * (tile / TJ), nc = nt + lr;
    if (nt >= a.N || mt0 >= a.M) continue;  // uniform; M and N are multiples of 16 and 32
    const floatx16& c = sum[q];
    const float bias = EPI != PRE_PART ? to_f(a.bias[nc]) : 0.f;
    if constexpr (EPI == PRE_STORE || EPI == PRE_PART) {
      float* y = a.y + (EPI == PRE_PART ? blockIdx.y * a.pstride : 0) + nc;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int row = mt0 + 8 * (v >> 2) + 4 * lk + (v & 3);
        if (row < a.M) y[(size_t)row * a.ldy] = c[v] + bias;
      }
    } else if constexpr (EPI == PRE_QKV) {
      // queries as fp32 rows; keys and values into the page of each 16-row part
      // (keys [page][head][16][64], values [page][head][64][16])
      const int d = a.d, kind = nt < d ? 0 : nt < 2 * d ? 1 : 2, cc = nc - kind * d, head = cc >> 6, dim = cc & 63;
#pragma unroll
      for (int half = 0; half < 2; ++half) {
        const int r0 = mt0 + 16 * half;
        if (r0 >= a.M) continue;
        if (kind == 0) {
#pragma unroll
          for (int v = 0; v < 8; ++v)
            a.y[(size_t)(r0 + 8 * (v >> 2) + 4 * lk + (v & 3)) * a.ldy + nc] = c[8 * half + v] + bias;
        } else {
          const PrePart p = a.parts[r0 / kPrePart];
          const size_t ph = (size_t)a.page_table[p.slot * a.pages_per_slot + p.pos0 / kPage] * a.n_head + head;
          bf16* cache = reinterpret_cast<bf16*>(a.cache) + (kind == 2 ? a.kv_stride : 0) + ph * kPage * kHeadDim;
          if (kind == 1) {
#pragma unroll
            for (int v = 0; v < 8; ++v)
              cache[(8 * (v >> 2) + 4 * lk + (v & 3)) * kHeadDim + dim] = from_f<bf16>(c[8 * half + v] + bias);
          } else {
            *reinterpret_cast<uint4*>(cache + dim * kPage + 8 * lk) = rows8_bf16(c, half, bias);
          }
        }
      }
    } else {
      // GELU into the next product's planes: 16 x 32 half tiles turned around in
      // the wave's own LDS, then 8 consecutive columns of a row per lane
      float* tr = reinterpret_cast<float*>(red) + wv * 16 * 33;
#pragma unroll
      for (int half = 0; half < 2; ++half) {
#pragma unroll
        for (int v = 0; v < 8; ++v) tr[(8 * (v >> 2) + 4 * lk + (v & 3)) * 33 + lr] = gelu_erf(c[8 * half + v] + bias);
        __builtin_amdgcn_wave_barrier();
        const int r = lane >> 2, c8 = 8 * (lane & 3), row = mt0 + 16 * half + r;
        float o[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = tr[r * 33 + c8 + e];
        __builtin_amdgcn_wave_barrier();
        if (row < a.M)
          put_planes8<P>(reinterpret_cast<uint4*>(a.aout), afrag16_index(row, nt + c8, a.mt) / 8, (size_t)a.mt * 2 * a.N, o);
      }
    }
  }
}

// ---------------------------------------------------------------- attention
// One block per (head, group of up to NQ consecutive parts of one slot), four waves;
// wave w takes the 32-key steps w, w + 4, ...: the keys of the slot's pages up to
// the group's last position (self-attention, causal per row), or the acoustic
// frames (cross-attention).  Per step and part the scores S^T = K q^T and O^T = V^T
// P^T run on the matrix cores as in the step's attention kernels (q and p as hi +
// lo planes); each wave keeps running maxima, sums and outputs of its rows (a row
// is one lane's column, so rescaling is a per-lane factor), and the waves meet once
// in LDS.  The blocks of a head walk the same keys side by side, so every step waits
// for a first touch of its lines: ND steps are kept in flight (240 rows, 1500
// frames, one step ahead: 30 us for 6 us of instructions).
namespace {
struct PreKv {
  bf16x8 kt[2][2], vt[4];
};
__device__ __forceinline__ void split_planes(const float* v, bf16x8& hi, bf16x8& lo) {
  uint4 h, l;
  split2x8(v, h, l);
  hi = __builtin_bit_cast(bf16x8, h);
  lo = __builtin_bit_cast(bf16x8, l);
}
__device__ __forceinline__ float quad_rows(float v, bool max) {  // over the four lanes of a row (lane, +16, +32, +48)
  const auto x = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  const float a = __uint_as_float(x[0]), b = __uint_as_float(x[1]);
  v = max ? fmaxf(a, b) : a + b;
  const auto y = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  const float c = __uint_as_float(y[0]), d = __uint_as_float(y[1]);
  return max ? fmaxf(c, d) : c + d;
}
}  // namespace

template <bool CROSS, int P, int NQ, int NW, int ND>
__global__ void __launch_bounds__(NW * 64, NW / 4) k_pre_attn(PreAttnArgs a) {
  StampScope stamp_scope(a.stamp, NW * 64);
  constexpr int kOld = 68;  // padded row of the wave outputs
  __shared__ float wmax[NQ][NW][16], wsum[NQ][NW][16];
  __shared__ float wo[NQ][NW][16][kOld];
  const int head = blockIdx.x;
  const int2 grp = a.groups[blockIdx.y];  // first part, parts
  const PrePart p0 = a.parts[grp.x], pl = a.parts[grp.x + grp.y - 1];
  const int lane = threadIdx.x & 63, n = lane & 15, kg = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // uniform, so the page of a step is a lane read
  const int slot = p0.slot, H = a.n_head;
  const int nkeys = CROSS ? a.n_frames : pl.pos0 + pl.nv, ns = (nkeys + 31) / 32;
  // lane l holds the page of positions 16 l .. (self)
  const int pages = CROSS ? 0 : a.page_table[slot * a.pages_per_slot + min(lane, a.pages_per_slot - 1)];
  const bf16 *Kb, *Vb;
  if constexpr (CROSS) {
    Kb = reinterpret_cast<const bf16*>(a.k) + (size_t)slot * a.d * (a.n_frames + a.vt_frames);
    Vb = Kb + (size_t)H * a.n_frames * kHeadDim + (size_t)head * kHeadDim * a.vt_frames;
    Kb += (size_t)head * a.n_frames * kHeadDim;
  } else {
    Kb = reinterpret_cast<const bf16*>(a.k);
    Vb = reinterpret_cast<const bf16*>(a.v);
  }
  auto load = [&](int s, PreKv& it) {  // step s (past the end: the last one)
    s = min(s, ns - 1);
    if constexpr (CROSS) {
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const bf16x8* kp = reinterpret_cast<const bf16x8*>(Kb + (size_t)min(32 * s + 16 * t + n, a.n_frames - 1) * kHeadDim) + kg;
        it.kt[t][0] = kp[0];
        it.kt[t][1] = kp[4];
      }
#pragma unroll
      for (int dt = 0; dt < 4; ++dt)
        it.vt[dt] = *reinterpret_cast<const bf16x8*>(Vb + vt_index(16 * dt + n, 32 * s + 8 * kg));
    } else {
      const int g0 = __builtin_amdgcn_readlane(pages, 2 * s);
      const int g1 = __builtin_amdgcn_readlane(pages, min(2 * s + 1, a.pages_per_slot - 1));
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const bf16x8* kp = reinterpret_cast<const bf16x8*>(Kb + (((size_t)(t ? g1 : g0) * H + head) * kPage + n) * kHeadDim) + kg;
        it.kt[t][0] = kp[0];
        it.kt[t][1] = kp[4];
      }
      const size_t vpage = (size_t)(kg < 2 ? g0 : g1) * H + head;
#pragma unroll
      for (int dt = 0; dt < 4; ++dt)
        it.vt[dt] = *reinterpret_cast<const bf16x8*>(Vb + (vpage * kHeadDim + 16 * dt + n) * kPage + 8 * (kg & 1));
    }
  };
  PreKv kv[ND];
  float4 qx[NQ][2][2];
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const float* qr = a.q + (size_t)((grp.x + min(q, grp.y - 1)) * kPrePart + n) * a.ldq + head * kHeadDim + 8 * kg;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      qx[q][h][0] = *reinterpret_cast<const float4*>(qr + 32 * h);
      qx[q][h][1] = *reinterpret_cast<const float4*>(qr + 32 * h + 4);
    }
  }
#pragma unroll
  for (int d = 0; d < ND; ++d) load(w + d * NW, kv[d]);
  __builtin_amdgcn_sched_barrier(0);
  bf16x8 qh[NQ][2], ql[NQ][2];
#pragma unroll
  for (int q = 0; q < NQ; ++q)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const float v[8] = {qx[q][h][0].x * 0.125f, qx[q][h][0].y * 0.125f, qx[q][h][0].z * 0.125f, qx[q][h][0].w * 0.125f,
                          qx[q][h][1].x * 0.125f, qx[q][h][1].y * 0.125f, qx[q][h][1].z * 0.125f, qx[q][h][1].w * 0.125f};
      split_planes(v, qh[q][h], ql[q][h]);
    }
  float m[NQ], l[NQ];
  floatx4 o[NQ][4];
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    m[q] = -INFINITY;
    l[q] = 0.f;
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) o[q][dt] = floatx4{0.f, 0.f, 0.f, 0.f};
  }
  // keys up to `full` are seen by every row of the group
  const int full = CROSS ? a.n_frames : p0.pos0 + 1;
  auto step = [&](int s, const PreKv& it) {
    const bool masked = 32 * s + 32 > full;  // uniform
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      // last key that this lane's row sees (rows past the prompt: the prompt's last)
      const int last = CROSS ? a.n_frames - 1 : min(p0.pos0 + 16 * q + n, nkeys - 1);
      floatx4 sc[2];
      float mx = -INFINITY;
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        floatx4 c = {0.f, 0.f, 0.f, 0.f};
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(it.kt[t][0], qh[q][0], c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(it.kt[t][0], ql[q][0], c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(it.kt[t][1], qh[q][1], c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(it.kt[t][1], ql[q][1], c, 0, 0, 0);
        sc[t] = c;
      }
      if (masked) {
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int i = 0; i < 4; ++i) sc[t][i] = 32 * s + 16 * t + 4 * kg + i <= last ? sc[t][i] : -INFINITY;
      }
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) mx = fmaxf(mx, sc[t][i]);
      const float mn = fmaxf(m[q], quad_rows(mx, true));
      const float ms = mn == -INFINITY ? 0.f : mn;  // no key of this row yet
      if (__builtin_amdgcn_ballot_w64(mn != m[q])) {
        const float f = __expf(m[q] - ms);          // 0 before the first key
        l[q] *= f;
#pragma unroll
        for (int dt = 0; dt < 4; ++dt)
#pragma unroll
          for (int i = 0; i < 4; ++i) o[q][dt][i] *= f;
        m[q] = mn;
      }
      float ls = 0.f, pb[8];
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          sc[t][i] = __expf(sc[t][i] - ms);  // 0 where masked
          ls += sc[t][i];
        }
      l[q] += ls;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const auto x = __builtin_amdgcn_permlane32_swap(__float_as_uint(sc[0][i]), __float_as_uint(sc[1][i]), false, false);
        const auto y = __builtin_amdgcn_permlane16_swap(x[0], x[1], false, false);
        pb[i] = __uint_as_float(y[0]);
        pb[4 + i] = __uint_as_float(y[1]);
      }
      bf16x8 ph, plo;
      split_planes(pb, ph, plo);
#pragma unroll
      for (int dt = 0; dt < 4; ++dt) {
        o[q][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(it.vt[dt], ph, o[q][dt], 0, 0, 0);
        o[q][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(it.vt[dt], plo, o[q][dt], 0, 0, 0);
      }
    }
  };
  const int n_steps = (ns - w + NW - 1) / NW;  // none for a wave past the keys
  int t = 0;
  for (; t + ND < n_steps; t += ND) {
#pragma unroll
    for (int d = 0; d < ND; ++d) {
      step(w + (t + d) * NW, kv[d]);
      __builtin_amdgcn_sched_barrier(0);
      load(w + (t + d + ND) * NW, kv[d]);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int d = 0; d < ND; ++d)
    if (t + d < n_steps) step(w + (t + d) * NW, kv[d]);
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const float ls = quad_rows(l[q], false);
    if (lane < 16) {
      wmax[q][w][lane] = m[q];
      wsum[q][w][lane] = ls;
    }
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
      *reinterpret_cast<float4*>(&wo[q][w][n][16 * dt + 4 * kg]) = make_float4(o[q][dt][0], o[q][dt][1], o[q][dt][2], o[q][dt][3]);
  }
  __syncthreads();
  for (int t = threadIdx.x; t < grp.y * 128; t += NW * 64) {
    const int q = t >> 7, r = (t & 127) >> 3, c8 = 8 * (t & 7);
    float M = wmax[q][0][r];
#pragma unroll
    for (int i = 1; i < NW; ++i) M = fmaxf(M, wmax[q][i][r]);  // finite: every row sees position 0
    float L = 0.f, ov[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < NW; ++i) {
      const float f = __expf(wmax[q][i][r] - M);
      L = fmaf(f, wsum[q][i][r], L);
#pragma unroll
      for (int e = 0; e < 8; ++e) ov[e] = fmaf(f, wo[q][i][r][c8 + e], ov[e]);
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) ov[e] /= L;
    put_planes8<P>(reinterpret_cast<uint4*>(a.out), afrag16_index((grp.x + q) * kPrePart + r, head * kHeadDim + c8, a.mt) / 8,
                   (size_t)a.mt * 2 * a.d, ov);
  }
}

// ---------------------------------------------------------------- drafter history
// Keys (RoPE at their positions) and values of the prompt's positions into one
// drafter block's history cache (Appendix A.2), from its k | v rows.
__global__ void __launch_bounds__(256) k_pre_hist(PreHistArgs a) {
  const PrePart p = a.parts[blockIdx.x];
  bf16* Kh = reinterpret_cast<bf16*>(a.kcache);
  bf16* Vh = reinterpret_cast<bf16*>(a.vcache);
  const int nj = a.n_head * 32;
  for (int t = blockIdx.y * 256 + threadIdx.x; t < p.nv * nj; t += gridDim.y * 256) {
    const int i = t / nj, e = t - i * nj, head = e >> 5, j = e & 31, pos = p.pos0 + i;
    const float* kr = a.kv + (size_t)(blockIdx.x * kPrePart + i) * 2 * a.d + head * kHeadDim;
    const float* vr = kr + a.d;
    const float c = a.use_rope ? a.rope[(pos * 32 + j) * 2] : 1.f, sn = a.use_rope ? a.rope[(pos * 32 + j) * 2 + 1] : 0.f;
    const float k1 = kr[j], k2 = kr[j + 32];
    const size_t base = (((size_t)p.slot * a.n_head + head) * a.n_ctx + pos) * kHeadDim;
    Kh[base + j] = from_f<bf16>(k1 * c - k2 * sn);
    Kh[base + j + 32] = from_f<bf16>(k1 * sn + k2 * c);
    Vh[base + j] = from_f<bf16>(vr[j]);
    Vh[base + j + 32] = from_f<bf16>(vr[j + 32]);
  }
}

// ---------------------------------------------------------------- launchers
void pre_begin(const PreArgs& a, int nparts, hipStream_t st) { k_pre_begin<<<dim3(nparts, 4), 256, 0, st>>>(a); }
void pre_last(const PreArgs& a, int nparts, float* lasth, hipStream_t st) { k_pre_last<<<nparts, 256, 0, st>>>(a, lasth); }
void pre_rln(const PreLnArgs& a, int planes, int rows, hipStream_t st) {
  const unsigned nt = (unsigned)((a.d / 8 + 63) / 64 * 64);
  if (planes == 3) k_pre_rln<3><<<rows, nt, 0, st>>>(a);
  else k_pre_rln<2><<<rows, nt, 0, st>>>(a);
}

namespace {
template <int EPI, int P, int WK, int TI, int TJ, int D>
void gemm_launch(const PreGemmArgs& a, int ks, hipStream_t st) {
  const int nmb = (a.M + 32 * TI - 1) / (32 * TI), nnb = (a.N + 32 * TJ - 1) / (32 * TJ);
  const int rs = xcd_row_parts(nmb, nnb, (size_t)32 * TI * (a.K / ks) * 2 * P);
  k_pre_gemm<EPI, P, WK, TI, TJ, D><<<dim3(xcd_blocks(nmb, nnb, rs), ks), 256, 0, st>>>(a, nmb, nnb, rs);
}
int blocks_of(const PreGemmArgs& a, int ti, int tj) {
  return ((a.M + 32 * ti - 1) / (32 * ti)) * ((a.N + 32 * tj - 1) / (32 * tj));
}
// 64 x 64 tiles; with three planes (one block per CU) 64 x 128 where the smaller
// tiles need a second round of blocks and the larger do not (240 rows: 5120 columns
// 24 against 17.5 us, 3840 columns 10 against 15)
template <int EPI, int P, int WK>
void gemm_tile(const PreGemmArgs& a, int ks, hipStream_t st) {
  if (P == 3 && blocks_of(a, 2, 2) * ks > kPreCus && blocks_of(a, 2, 4) * ks <= kPreCus)
    gemm_launch<EPI, P, WK, 2, 4, 4>(a, ks, st);
  else gemm_launch<EPI, P, WK, 2, 2, 5>(a, ks, st);
}
template <int EPI>
void gemm_planes(const PreGemmArgs& a, int planes, int ks, hipStream_t st) {
  if (planes == 3) {
    if constexpr (EPI == PRE_GELU) {  // one-slot handles keep W_1 in 32-column tiles
      if (a.wkind == W_F32) return gemm_tile<EPI, 3, W_F32>(a, ks, st);
    }
    return gemm_tile<EPI, 3, W_F16>(a, ks, st);
  }
  gemm_tile<EPI, 2, W_F16>(a, ks, st);
}
}  // namespace

int pre_gemm(int epi, const PreGemmArgs& a, int planes, hipStream_t st) {
  switch (epi) {
    case PRE_STORE: gemm_planes<PRE_STORE>(a, planes, 1, st); return 1;
    case PRE_GELU: gemm_planes<PRE_GELU>(a, planes, 1, st); return 1;
    case PRE_QKV: gemm_planes<PRE_QKV>(a, planes, 1, st); return 1;
    default: break;
  }
  // partial sums: split k (640 columns or more per split) while the blocks fit one
  // round, long rows twice in any case (864 rows, K = 5120: 39 us unsplit, 34 split)
  const int blocks = planes == 3 && a.K >= 2560 ? blocks_of(a, 2, 4) : blocks_of(a, 2, 2);
  auto can = [&](int ks) { return ks <= kPreMaxSplit && (a.K / 32) % ks == 0 && a.K / ks >= 640; };
  int ks = 1;
  while (can(2 * ks) && blocks * 2 * ks <= kPreCus) ks *= 2;
  if (ks == 1 && a.K >= 2560 && can(2)) ks = 2;
  gemm_planes<PRE_PART>(a, planes, ks, st);
  return ks;
}

template <bool CROSS, int P>
static void attn_launch(const PreAttnArgs& a, int nq, int ngroups, hipStream_t st) {
  const dim3 grid(a.n_head, ngroups);
  if (nq == 1) k_pre_attn<CROSS, P, 1, 8, 4><<<grid, 512, 0, st>>>(a);
  else if (a.n_head * ngroups <= kPreCus) k_pre_attn<CROSS, P, 2, 8, 3><<<grid, 512, 0, st>>>(a);
  else k_pre_attn<CROSS, P, 2, 4, 2><<<grid, 256, 0, st>>>(a);
}
void pre_attn(const PreAttnArgs& a, bool cross, int planes, int nq, int ngroups, hipStream_t st) {
  if (planes == 3) cross ? attn_launch<true, 3>(a, nq, ngroups, st) : attn_launch<false, 3>(a, nq, ngroups, st);
  else cross ? attn_launch<true, 2>(a, nq, ngroups, st) : attn_launch<false, 2>(a, nq, ngroups, st);
}

void pre_hist(const PreHistArgs& a, int nparts, hipStream_t st) { k_pre_hist<<<dim3(nparts, 4), 256, 0, st>>>(a); }

}  // namespace wf
