// Matrix-core GEMM for the request-time products (bf16 operands, fp32
// accumulation): C[m, n] = sum_k A[m, k] B[n, k] (+ bias[n]), A [M, K] and
// B [N, K] row-major bf16 (a weight matrix [out, in] is B as stored), with one
// of several epilogues.  It computes the acoustic keys and values of every
// decoder block for a new request (Appendix A.5) and the products of the
// audio encoder.
//
// Tiling: BMT x 128 output tiles (BMT = 128 or 64; 256 in k_mmw below), k in steps
// of 64, 256 threads = 2 x 2 waves of BMT/2 x 64
// (BMT/64 x 2 tiles of v_mfma_f32_32x32x16_bf16).  A and B tiles are copied
// straight from memory into LDS stages (global_load_lds_dwordx4): two stages one
// k-step ahead for 128-row tiles (two blocks share a CU), four stages three
// k-steps ahead for 64-row tiles (16-byte chunks, chunk q of row r stored at
// q ^ (r & 7) so that the eight rows a wave's lane group reads fall in different
// banks).
// The finished tile goes through LDS again so that every epilogue writes 16-byte
// runs of consecutive elements.
#include <algorithm>

#include "wf_common.h"
#include "wf_kernels.h"
#include "wf_operand.h"
#include "wf_split.h"

namespace wf {

namespace {

typedef __attribute__((address_space(3))) void lds_void;
constexpr int BN = kMmTile, BK = kMmK, NT = 256;
constexpr int kChunksB = BN * BK / 8;  // 16-byte chunks of a B tile (1024)
constexpr int kCt = BN + 1;            // row stride of the staged output tile (floats)


__device__ __forceinline__ uint4 pack8(const float* v) {
  uint4 r;
  r.x = bf16_bits_rne(v[0]) | (bf16_bits_rne(v[1]) << 16);
  r.y = bf16_bits_rne(v[2]) | (bf16_bits_rne(v[3]) << 16);
  r.z = bf16_bits_rne(v[4]) | (bf16_bits_rne(v[5]) << 16);
  r.w = bf16_bits_rne(v[6]) | (bf16_bits_rne(v[7]) << 16);
  return r;
}

}  // namespace

// Four LDS stages, separate objects so that the compiler sees a copy into one
// stage cannot alias reads of another; each holds one k-step's A and B tiles
// (16-byte chunks, chunk c of row r at r * 8 + (c ^ (r & 7))), and after the loop
// two of them hold the output tile's two 64-row halves ([64][kCt] fp32).
constexpr int kStageU4 = (64 * kCt * 4 + 15) / 16;  // >= 2048 chunks of a 128-row A + B stage
static_assert(kStageU4 >= 2 * kChunksB, "stage holds a 128-row k-step");
__shared__ uint4 g_mm0[kStageU4], g_mm1[kStageU4], g_mm2[kStageU4], g_mm3[kStageU4];

template <int EP, int BM, int NS>
__global__ void __launch_bounds__(NT) k_mm(MmArgs a, int nmb, int nnb, int rs) {
  static_assert(NS == 2 || NS == 4, "two or four stages");
  constexpr int kChunksA = BM * BK / 8, JA = kChunksA / NT, MI = BM / 64;
  // copies per wave and k-step: JA of A, 4 of B; a step waits until at most the
  // NS - 2 later k-steps' copies are outstanding (and its earlier LDS reads are done)
  constexpr int kCopies = JA + 4, kVm = (NS - 2) * kCopies;
  constexpr int kWait = (kVm & 15) | ((kVm >> 4) << 14) | (7 << 4) | (0 << 8);
  // XCD x (block % 8) takes row part x % rs of rs and column part x / rs of 8 / rs, row
  // blocks fastest, so the blocks that share an L2 share their rows and columns
  const int x8 = blockIdx.x & 7, bi = blockIdx.x >> 3;
  const int nrh = (nmb + rs - 1) / rs, ncq = (nnb * rs + 7) / 8;
  const int mbk = (x8 % rs) * nrh + bi % nrh, nbk = (x8 / rs) * ncq + bi / nrh;
  if (mbk >= nmb || bi / nrh >= ncq || nbk >= nnb) return;
  const int z = blockIdx.z;
  const bf16* A = a.A + (size_t)z * a.sA;
  const bf16* B = a.B + (size_t)z * a.sB;
  const int m0 = mbk * BM, n0 = nbk * BN;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int wm = w >> 1, wn = w & 1;
  const int nk = a.K / BK;

  // this lane's copy sources: LDS chunk slot s = (w * J + j) * 64 + lane holds row
  // s / 8, chunk (s % 8) ^ (row & 7) of the tile (rows past the matrix re-read its
  // last row; their results are not written)
  const bf16* srcA[JA];
  const bf16* srcB[4];
#pragma unroll
  for (int j = 0; j < JA; ++j) {
    const int slot = (w * JA + j) * 64 + lane, row = slot >> 3, ch = (slot & 7) ^ (row & 7);
    srcA[j] = A + (size_t)min(m0 + row, a.M - 1) * a.lda + 8 * ch;
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int slot = (w * 4 + j) * 64 + lane, row = slot >> 3, ch = (slot & 7) ^ (row & 7);
    srcB[j] = B + (size_t)min(n0 + row, a.N - 1) * a.ldb + 8 * ch;
  }
  auto copy = [&](int kt, uint4* stage) {  // k-step kt (past the last: the last one)
    const int k0 = min(kt, nk - 1) * BK;
#pragma unroll
    for (int j = 0; j < JA; ++j)
      __builtin_amdgcn_global_load_lds((const void*)(srcA[j] + k0), (lds_void*)&stage[(w * JA + j) * 64], 16, 0, 0);
#pragma unroll
    for (int j = 0; j < 4; ++j)
      __builtin_amdgcn_global_load_lds((const void*)(srcB[j] + k0), (lds_void*)&stage[kChunksA + (w * 4 + j) * 64],
                                       16, 0, 0);
  };

  floatx16 acc[MI][2];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int jj = 0; jj < 2; ++jj)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][jj][v] = 0.f;

  // fragment rows of this lane: row (lane % 32) of each 32-row tile, k chunk
  // 2 s + lane / 32 of k-substep s
  const int lr = lane & 31, lk = lane >> 5;
  auto step = [&](int kt, const uint4* la, uint4* nxt) {
    __builtin_amdgcn_s_waitcnt(kWait);
    __builtin_amdgcn_s_barrier();
    copy(kt + NS - 1, nxt);  // every step issues its copies, so the wait count stays exact
    if (kt < nk) {
      const uint4* lb = la + kChunksA;
#pragma unroll
      for (int s = 0; s < BK / 16; ++s) {
        const int q = 2 * s + lk;
        bf16x8 af[MI], bf[2];
#pragma unroll
        for (int i = 0; i < MI; ++i) {
          const int row = wm * (BM / 2) + i * 32 + lr;
          af[i] = __builtin_bit_cast(bf16x8, la[row * 8 + (q ^ (row & 7))]);
        }
#pragma unroll
        for (int jj = 0; jj < 2; ++jj) {
          const int row = wn * 64 + jj * 32 + lr;
          bf[jj] = __builtin_bit_cast(bf16x8, lb[row * 8 + (q ^ (row & 7))]);
        }
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int jj = 0; jj < 2; ++jj)
            acc[i][jj] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[i], bf[jj], acc[i][jj], 0, 0, 0);
      }
    }
  };
  if constexpr (NS == 4) {
    copy(0, g_mm0);
    copy(1, g_mm1);
    copy(2, g_mm2);
    for (int kt = 0; kt < nk; kt += 4) {
      step(kt, g_mm0, g_mm3);
      step(kt + 1, g_mm1, g_mm0);
      step(kt + 2, g_mm2, g_mm1);
      step(kt + 3, g_mm3, g_mm2);
    }
  } else {  // two stages (66 KB of LDS: two blocks per CU), one k-step ahead
    copy(0, g_mm0);
    for (int kt = 0; kt < nk; kt += 2) {
      step(kt, g_mm0, g_mm1);
      step(kt + 1, g_mm1, g_mm0);
    }
  }
  __builtin_amdgcn_s_waitcnt((0 & 15) | (7 << 4) | (15 << 8));  // every copy has landed
  __syncthreads();

  // stage the tile (+ bias, activation) in LDS: acc element v of a 32 x 32 tile is
  // row 8 (v / 4) + 4 (lane / 32) + v % 4, column lane % 32; rows 0..63 in one
  // stage object, 64..127 in another
  float* ct0 = reinterpret_cast<float*>(g_mm0);
  float* ct1 = reinterpret_cast<float*>(g_mm1);
  auto ct = [&](int r) -> float* { return (r < 64 ? ct0 : ct1) + (r & 63) * kCt; };
  const bf16* bias = a.bias ? a.bias + (size_t)z * a.sBias : nullptr;
#pragma unroll
  for (int jj = 0; jj < 2; ++jj) {
    const int cl = wn * 64 + jj * 32 + lr;
    const float bv = bias ? to_f(bias[min(n0 + cl, a.N - 1)]) : 0.f;
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int rl = wm * (BM / 2) + i * 32 + 8 * (v >> 2) + 4 * lk + (v & 3);
        float x = acc[i][jj][v] * a.scale + bv;
        if (EP == MM_BF16_GELU) x = gelu_erf(x);
        ct(rl)[cl] = x;
      }
  }
  __syncthreads();

  if (EP == MM_XKV || EP == MM_QKV_ENC) {
    // columns [0, nrow) row-major bf16 (keys, or queries | keys), columns
    // [nrow, N) values transposed per head: MM_XKV in 256-frame pieces
    // [head][frame / 256][dim][256] after the keys [head][frame][64]; MM_QKV_ENC as
    // [head][dim][ldv] in out2.  Frames from M to the padded count are zeros (between
    // requests, period > 0: what the rows there give).
    const int nrow = EP == MM_XKV ? a.d : 2 * a.d;
    bf16* out = reinterpret_cast<bf16*>(a.out) + (size_t)z * a.sO;
    // row-major part: items (row, 8 columns)
    for (int it = t; it < BM * (BN / 8); it += NT) {
      const int rl = it / (BN / 8), c8 = (it % (BN / 8)) * 8, f = m0 + rl, n = n0 + c8;
      if (f >= a.M || n >= nrow) continue;
      const uint4 pk = pack8(ct(rl) + c8);
      if (EP == MM_XKV) {
        const int head = n >> 6, dim = n & 63;
        *reinterpret_cast<uint4*>(out + ((size_t)head * a.M + f) * kHeadDim + dim) = pk;
      } else {
        *reinterpret_cast<uint4*>(out + (size_t)f * a.ldo + n) = pk;
      }
    }
    // transposed part: items (column, 8 frames)
    for (int it = t; it < BN * (BM / 8); it += NT) {
      const int cl = it / (BM / 8), r8 = (it % (BM / 8)) * 8, n = n0 + cl, f = m0 + r8;
      if (n < nrow || n >= a.N || f >= (a.period > 0 ? a.M : a.vt_frames)) continue;
      const int col = n - nrow, head = col >> 6, dim = col & 63;
      float v[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = f + e < a.M ? ct(r8 + e)[cl] : 0.f;
      const uint4 pk = pack8(v);
      if (EP == MM_XKV) {
        bf16* vt = out + (size_t)a.n_head * a.M * kHeadDim + (size_t)head * kHeadDim * a.vt_frames;
        *reinterpret_cast<uint4*>(vt + vt_index(dim, f)) = pk;
      } else {  // a tile may hold rows of two requests, eight frames from a multiple of 8 are one's
        const int req = a.period > 0 ? f / a.period : 0;
        bf16* vt = reinterpret_cast<bf16*>(a.out2) + (size_t)(z + req) * a.sO2;
        *reinterpret_cast<uint4*>(vt + ((size_t)head * kHeadDim + dim) * a.vt_frames + f - req * a.period) = pk;
      }
    }
    return;
  }
  // row-major outputs: items (row, 8 columns)
  for (int it = t; it < BM * (BN / 8); it += NT) {
    const int rl = it / (BN / 8), c8 = (it % (BN / 8)) * 8, f = m0 + rl, n = n0 + c8;
    if (f >= a.M || n >= a.N) continue;
    const float* src = ct(rl) + c8;
    if (EP == MM_BF16_GELU) {
      bf16* out = reinterpret_cast<bf16*>(a.out) + (size_t)z * a.sO;
      *reinterpret_cast<uint4*>(out + (size_t)f * a.ldo + n) = pack8(src);
    } else {
      float* out = reinterpret_cast<float*>(a.out) + (size_t)z * a.sO + (size_t)f * a.ldo + n;
      float4 lo = make_float4(src[0], src[1], src[2], src[3]), hi = make_float4(src[4], src[5], src[6], src[7]);
      if (EP == MM_GELU_ADD_F32) {
        const float* ad = a.add + (size_t)f * a.ldadd + n;
        lo.x = gelu_erf(lo.x) + ad[0]; lo.y = gelu_erf(lo.y) + ad[1];
        lo.z = gelu_erf(lo.z) + ad[2]; lo.w = gelu_erf(lo.w) + ad[3];
        hi.x = gelu_erf(hi.x) + ad[4]; hi.y = gelu_erf(hi.y) + ad[5];
        hi.z = gelu_erf(hi.z) + ad[6]; hi.w = gelu_erf(hi.w) + ad[7];
      }
      if (EP == MM_RESID) {  // residual rows: each element has exactly one writer
        const float4 o0 = *reinterpret_cast<const float4*>(out), o1 = *reinterpret_cast<const float4*>(out + 4);
        lo.x += o0.x; lo.y += o0.y; lo.z += o0.z; lo.w += o0.w;
        hi.x += o1.x; hi.y += o1.y; hi.z += o1.z; hi.w += o1.w;
      }
      *reinterpret_cast<float4*>(out) = lo;
      *reinterpret_cast<float4*>(out + 4) = hi;
    }
  }
}

// The same products on 256 x 128 tiles, eight waves of 64 x 64 (two per SIMD), for
// launches whose larger tiles still cover the chip: three LDS stages, two k-steps
// ahead.  Within a k-step the fragment reads of the next 16-wide substep and the
// copies of a later k-step are issued between the multiplications, since a wave
// stalls while its copies are taken up.  The finished 32 x 32 tiles are turned
// around in each wave's own LDS.  6144 rows, K = 5120, N = 1280: 1060 TFLOP/s (a large
// library product reaches 1190 on this card); 1500 rows, N = 2560, 34 matrices 0.40 ms
// against 0.47 on the 128-row tiles and 0.53 before those had their XCD order.  256 x
// 256 tiles in two stages: 0.47 ms.
template <int EP>
__global__ void __launch_bounds__(512, 2) k_mmw(MmArgs a, int nmb, int nnb, int rs) {
  constexpr int BM = 256, WC = 2, WR = 4, MI = 2, NJ = 2, NS = 3;
  constexpr int kA = BM * BK / 8, JA = kA / 512, JB = kChunksB / 512, CPW = JA + JB;
  constexpr int kVm = (NS - 2) * CPW;
  constexpr int kWait = (kVm & 15) | ((kVm >> 4) << 14) | (7 << 4) | (0 << 8);
  constexpr int kStage = kA + kChunksB;
  __shared__ uint4 g_mw0[kStage], g_mw1[kStage], g_mw2[kStage];
  const int x8 = blockIdx.x & 7, bi = blockIdx.x >> 3;
  const int nrh = (nmb + rs - 1) / rs, ncq = (nnb * rs + 7) / 8;
  const int mbk = (x8 % rs) * nrh + bi % nrh, nbk = (x8 / rs) * ncq + bi / nrh;
  if (mbk >= nmb || bi / nrh >= ncq || nbk >= nnb) return;
  const int z = blockIdx.z;
  const bf16* A = a.A + (size_t)z * a.sA;
  const bf16* B = a.B + (size_t)z * a.sB;
  const int m0 = mbk * BM, n0 = nbk * BN;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int wm = w / WC, wn = w % WC, lr = lane & 31, lk = lane >> 5;
  const int nk = a.K / BK;
  // copy sources as in k_mm: slot s holds row s / 8, chunk (s % 8) ^ (row & 7)
  const bf16* src[CPW];
#pragma unroll
  for (int j = 0; j < CPW; ++j) {
    const bool isA = j < JA;
    const int slot = (w * (isA ? JA : JB) + (isA ? j : j - JA)) * 64 + lane, row = slot >> 3, ch = (slot & 7) ^ (row & 7);
    src[j] = isA ? A + (size_t)min(m0 + row, a.M - 1) * a.lda + 8 * ch : B + (size_t)min(n0 + row, a.N - 1) * a.ldb + 8 * ch;
  }
  auto copy1 = [&](int j, int k0, uint4* stage) {
    __builtin_amdgcn_global_load_lds((const void*)(src[j] + k0),
                                     (lds_void*)&stage[j < JA ? (w * JA + j) * 64 : kA + (w * JB + j - JA) * 64], 16, 0, 0);
  };
  floatx16 acc[MI][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
  bf16x8 fr[2][MI + NJ];
  auto read1 = [&](const uint4* st, int s, int r, bf16x8* f) {  // fragment r of substep s: rows, then columns
    const int q = 2 * s + lk;
    if (r < MI) {
      const int row = (wm * MI + r) * 32 + lr;
      f[r] = __builtin_bit_cast(bf16x8, st[row * 8 + (q ^ (row & 7))]);
    } else {
      const int row = (wn * NJ + r - MI) * 32 + lr;
      f[r] = __builtin_bit_cast(bf16x8, st[kA + row * 8 + (q ^ (row & 7))]);
    }
  };
  constexpr int NM = MI * NJ, NR = MI + NJ;
  auto kstep = [&](int kt, const uint4* cur, uint4* nxt) {
    __builtin_amdgcn_s_waitcnt(kWait);
    __builtin_amdgcn_s_barrier();
    const int k0 = min(kt + NS - 1, nk - 1) * BK;  // every step issues its copies, so the wait count stays exact
#pragma unroll
    for (int r = 0; r < NR; ++r) read1(cur, 0, r, fr[0]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int m = 0; m < NM; ++m) {
        acc[m / NJ][m % NJ] =
            __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[s & 1][m / NJ], fr[s & 1][MI + m % NJ], acc[m / NJ][m % NJ], 0, 0, 0);
        if (s < 3) {
#pragma unroll
          for (int r = m * NR / NM; r < (m + 1) * NR / NM; ++r) read1(cur, s + 1, r, fr[(s + 1) & 1]);
        }
#pragma unroll
        for (int j = (s * NM + m) * CPW / (4 * NM); j < (s * NM + m + 1) * CPW / (4 * NM); ++j) copy1(j, k0, nxt);
        __builtin_amdgcn_sched_barrier(0);
      }
  };
  auto stage = [&](int i) -> uint4* { return i == 0 ? g_mw0 : i == 1 ? g_mw1 : g_mw2; };
#pragma unroll
  for (int i = 0; i < NS - 1; ++i)
#pragma unroll
    for (int j = 0; j < CPW; ++j) copy1(j, min(i, nk - 1) * BK, stage(i));
  int kt = 0;
  for (; kt + NS <= nk; kt += NS) {
#pragma unroll
    for (int i = 0; i < NS; ++i) kstep(kt + i, stage(i), stage((i + NS - 1) % NS));
  }
#pragma unroll
  for (int i = 0; i < NS - 1; ++i)
    if (kt + i < nk) kstep(kt + i, stage(i), stage((i + NS - 1) % NS));
  __builtin_amdgcn_s_waitcnt((0 & 15) | (7 << 4) | (15 << 8));  // every copy has landed
  __syncthreads();

  // accumulator v of a 32 x 32 tile: row 8 (v / 4) + 4 (lane / 32) + v % 4, column lane % 32
  float* tr = reinterpret_cast<float*>(g_mw0) + w * 16 * 33;
  const bf16* bias = a.bias ? a.bias + (size_t)z * a.sBias : nullptr;
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int nt = n0 + (wn * NJ + j) * 32, nc = nt + lr;
    if (nt >= a.N) continue;  // uniform
    const float bv = bias ? to_f(bias[min(nc, a.N - 1)]) : 0.f;
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      const int mt = m0 + (wm * MI + i) * 32;
      const int nrow = EP == MM_XKV ? a.d : EP == MM_QKV_ENC ? 2 * a.d : 1 << 30;
      floatx16 c = acc[i][j];
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        c[v] = c[v] * a.scale + bv;
        if (EP == MM_BF16_GELU || EP == MM_GELU_ADD_F32) c[v] = gelu_erf(c[v]);
      }
      if (EP == MM_RESID || EP == MM_GELU_ADD_F32) {
        float* out = reinterpret_cast<float*>(a.out) + (size_t)z * a.sO + nc;
        if (nc < a.N) {
          float o[16];
#pragma unroll
          for (int v = 0; v < 16; ++v) {  // every load first (rows past the matrix re-read its last one)
            const int f = min(mt + 8 * (v >> 2) + 4 * lk + (v & 3), a.M - 1);
            o[v] = EP == MM_RESID ? out[(size_t)f * a.ldo] : a.add[(size_t)f * a.ldadd + nc];
          }
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            const int f = mt + 8 * (v >> 2) + 4 * lk + (v & 3);
            if (f < a.M) out[(size_t)f * a.ldo] = c[v] + o[v];
          }
        }
      } else if (nt < nrow) {
        // bf16 rows: half tiles turned around in the wave's LDS, 8 columns per lane
        bf16* out = reinterpret_cast<bf16*>(a.out) + (size_t)z * a.sO;
#pragma unroll
        for (int half = 0; half < 2; ++half) {
#pragma unroll
          for (int v = 0; v < 8; ++v) tr[(8 * (v >> 2) + 4 * lk + (v & 3)) * 33 + lr] = c[8 * half + v];
          __builtin_amdgcn_wave_barrier();
          float o[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) o[e] = tr[(lane >> 2) * 33 + 8 * (lane & 3) + e];
          __builtin_amdgcn_wave_barrier();
          const int f = mt + 16 * half + (lane >> 2), n = nt + 8 * (lane & 3);
          if (f < a.M && n < a.N) {
            if (EP == MM_XKV)
              *reinterpret_cast<uint4*>(out + ((size_t)(n >> 6) * a.M + f) * kHeadDim + (n & 63)) = pack8(o);
            else
              *reinterpret_cast<uint4*>(out + (size_t)f * a.ldo + n) = pack8(o);
          }
        }
      } else {
        // transposed values, zero past the last frame: eight consecutive frames per lane
        const int col = nc - nrow, head = col >> 6, dim = col & 63;
#pragma unroll
        for (int half = 0; half < 2; ++half) {
          const int f = mt + 16 * half + 8 * lk;
          uint32_t p[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int f0 = mt + 16 * half + 8 * (e >> 1) + 4 * lk + 2 * (e & 1);
            p[e] = pack2_bf16(f0 < a.M ? c[8 * half + 2 * e] : 0.f, f0 + 1 < a.M ? c[8 * half + 2 * e + 1] : 0.f);
          }
          const auto x = __builtin_amdgcn_permlane32_swap(p[0], p[2], false, false);
          const auto y = __builtin_amdgcn_permlane32_swap(p[1], p[3], false, false);
          if (f >= (a.period > 0 ? a.M : a.vt_frames)) continue;
          const uint4 pk = make_uint4(x[0], y[0], x[1], y[1]);
          if (EP == MM_XKV) {
            bf16* vt = reinterpret_cast<bf16*>(a.out) + (size_t)z * a.sO + (size_t)a.n_head * a.M * kHeadDim +
                       (size_t)head * kHeadDim * a.vt_frames;
            *reinterpret_cast<uint4*>(vt + vt_index(dim, f)) = pk;
          } else {  // as in k_mm
            const int req = a.period > 0 ? f / a.period : 0;
            bf16* vt = reinterpret_cast<bf16*>(a.out2) + (size_t)(z + req) * a.sO2;
            *reinterpret_cast<uint4*>(vt + ((size_t)head * kHeadDim + dim) * a.vt_frames + f - req * a.period) = pk;
          }
        }
      }
    }
  }
}

// Shapes the kernel assumes: K a multiple of 64, N a multiple of 8, 16-byte
// aligned rows (lda, ldb, ldo multiples of 8), and for the transposed epilogues
// head width 64 with the value columns after the row-major ones.
int mm_check(const MmArgs& a, int ep) {
  if (a.M < 1 || a.N < 1 || a.K < kMmK || a.K % kMmK) return -1;
  if (a.N % 8 || a.lda % 8 || a.ldb % 8 || a.lda < a.K || a.ldb < a.K) return -1;
  if ((ep == MM_BF16_GELU || ep == MM_RESID || ep == MM_GELU_ADD_F32) &&
      (a.ldo % 8 || a.ldo < a.N))
    return -1;
  if (ep == MM_GELU_ADD_F32 && (!a.add || a.ldadd < a.N)) return -1;
  if (ep == MM_XKV && (a.N != 2 * a.d || a.d % kHeadDim || a.vt_frames < a.M || a.vt_frames % kVtPiece)) return -1;
  if (ep == MM_QKV_ENC && (a.N != 3 * a.d || a.d % kHeadDim || (a.period > 0 ? a.period != a.vt_frames || a.M % a.period : a.vt_frames < a.M) || a.vt_frames % 8 || a.ldo % 8 ||
                           a.ldo < 2 * a.d))
    return -1;
  return 0;
}

namespace {
dim3 xcd_grid(const XcdSplit& x, int batch) { return dim3(xcd_blocks(x.nmb, x.nnb, x.rs), 1, batch); }
}  // namespace

template <int BM, int NS>
static void mm_launch(const MmArgs& a, int ep, const XcdSplit& x, int batch, hipStream_t st) {
  const dim3 grid = xcd_grid(x, batch);
  switch (ep) {
    case MM_BF16_GELU: k_mm<MM_BF16_GELU, BM, NS><<<grid, NT, 0, st>>>(a, x.nmb, x.nnb, x.rs); break;
    case MM_RESID: k_mm<MM_RESID, BM, NS><<<grid, NT, 0, st>>>(a, x.nmb, x.nnb, x.rs); break;
    case MM_XKV: k_mm<MM_XKV, BM, NS><<<grid, NT, 0, st>>>(a, x.nmb, x.nnb, x.rs); break;
    case MM_QKV_ENC: k_mm<MM_QKV_ENC, BM, NS><<<grid, NT, 0, st>>>(a, x.nmb, x.nnb, x.rs); break;
    case MM_GELU_ADD_F32: k_mm<MM_GELU_ADD_F32, BM, NS><<<grid, NT, 0, st>>>(a, x.nmb, x.nnb, x.rs); break;
  }
}
static void mmw_launch(const MmArgs& a, int ep, const XcdSplit& x, int batch, hipStream_t st) {
  const dim3 grid = xcd_grid(x, batch);
  switch (ep) {
    case MM_BF16_GELU: k_mmw<MM_BF16_GELU><<<grid, 512, 0, st>>>(a, x.nmb, x.nnb, x.rs); break;
    case MM_RESID: k_mmw<MM_RESID><<<grid, 512, 0, st>>>(a, x.nmb, x.nnb, x.rs); break;
    case MM_XKV: k_mmw<MM_XKV><<<grid, 512, 0, st>>>(a, x.nmb, x.nnb, x.rs); break;
    case MM_QKV_ENC: k_mmw<MM_QKV_ENC><<<grid, 512, 0, st>>>(a, x.nmb, x.nnb, x.rs); break;
    case MM_GELU_ADD_F32: k_mmw<MM_GELU_ADD_F32><<<grid, 512, 0, st>>>(a, x.nmb, x.nnb, x.rs); break;
  }
}

void mm(const MmArgs& a, int ep, int batch, hipStream_t st) {
  const int rows = std::max(a.M, (ep == MM_XKV || ep == MM_QKV_ENC) ? a.vt_frames : a.M);
  const MmTile t = mm_tile(rows, a.N, BN, batch);
  if (t.rows == 256) mmw_launch(a, ep, t.split, batch, st);
  else if (t.rows == 128) mm_launch<128, 2>(a, ep, t.split, batch, st);
  else mm_launch<64, 4>(a, ep, t.split, batch, st);
}

}  // namespace wf
