// Kernels of the Whisper audio encoder (the acoustic memory the drafter and the
// target cross-attend to, Section 3.2) besides its matrix products, which run on
// k_mm: the log-mel frontend, the convolution stem's row gathering, row-wise
// LayerNorm and the fused self-attention.
#include <float.h>

#include "wf_common.h"
#include "wf_kernels.h"
#include "wf_operand.h"

namespace wf {

namespace {

// order-preserving map of fp32 values to signed ints (max over floats = max over keys)
__device__ __forceinline__ int f2key(float f) {
  const int b = __float_as_int(f);
  return b >= 0 ? b : b ^ 0x7fffffff;
}
__device__ __forceinline__ float key2f(int k) { return __int_as_float(k >= 0 ? k : k ^ 0x7fffffff); }

__device__ __forceinline__ float block_max(float v, float* red) {
  for (int o = 32; o; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  const int w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[w] = v;
  __syncthreads();
  float r = red[0];
  for (int i = 1; i < nw; ++i) r = fmaxf(r, red[i]);
  return r;
}

}  // namespace

// One block per frame f of one request: the frame's n_fft samples (reflect-padded
// signal, periodic Hann window), their power spectrum in fp64, the mel filterbank (each
// filter summed over its nonzero bins) and log10 of max(mel, 1e-10), written to
// logmel[f][m]; the request's maximum goes to *gmax as an order-preserving int.
// The transform in two stages (Cooley and Tukey): N = A B, sample B n1 + n2, bin k:
//   S[k mod A][n2] = sum over n1 of x[B n1 + n2] exp(-2 pi i B n1 k / N)
//   X[k] = sum over n2 of S[k mod A][n2] exp(-2 pi i n2 k / N),
// A the divisor of N next below sqrt(N).  The samples are real, so the rows S[A - j] are
// the conjugates of S[j].  Bound by LDS latency along the sums: A + B terms in a row
// instead of N (20 + 20 against 400; four requests of 3000 frames, 128 filters 399 -> 148 us).
__global__ void __launch_bounds__(256) k_logmel(LogmelArgs a, int A) {
  __shared__ double xw[kMaxFft];
  __shared__ __align__(16) double tw[2 * kMaxFft];
  __shared__ double pw[kMaxFft / 2 + 1];
  __shared__ double2 S[kMaxFft + 2];  // A / 2 + 1 rows of B + 1 values: the most for A = 2 (N is even)
  __shared__ float red[4];
  const int f = blockIdx.x, N = a.n_fft, nb = N / 2 + 1, B = N / A;
  a.audio += (size_t)blockIdx.y * a.n_samples;
  a.logmel += (size_t)blockIdx.y * a.n_frames * a.n_mels;
  a.gmax += blockIdx.y;
  for (int i = threadIdx.x; i < N; i += blockDim.x) {
    int s = f * a.hop - N / 2 + i;
    s = s < 0 ? -s : s;
    s = s >= a.n_samples ? 2 * (a.n_samples - 1) - s : s;
    xw[i] = (double)a.audio[s] * a.window[i];
    tw[2 * i] = a.twiddle[2 * i];
    tw[2 * i + 1] = a.twiddle[2 * i + 1];
  }
  __syncthreads();
  const double2* tw2 = reinterpret_cast<const double2*>(tw);
  for (int j = threadIdx.x; j < (A / 2 + 1) * B; j += blockDim.x) {
    const int k1 = j / B, n2 = j - k1 * B, step = B * k1;
    double re = 0.0, im = 0.0;
    int idx = 0;
#pragma unroll 4
    for (int n1 = 0; n1 < A; ++n1) {
      const double x = xw[B * n1 + n2];
      const double2 w = tw2[idx];
      re = fma(x, w.x, re);
      im = fma(x, w.y, im);
      idx += step;
      if (idx >= N) idx -= N;
    }
    S[k1 * (B + 1) + n2] = make_double2(re, im);
  }
  __syncthreads();
  for (int k = threadIdx.x; k < nb; k += blockDim.x) {
    const int k1 = k % A;
    const bool conj = k1 > A / 2;
    const double2* Sr = S + (conj ? A - k1 : k1) * (B + 1);
    double re = 0.0, im = 0.0;
    int idx = 0;
#pragma unroll 4
    for (int n2 = 0; n2 < B; ++n2) {
      const double2 v = Sr[n2], w = tw2[idx];
      const double y = conj ? -v.y : v.y;
      re = fma(v.x, w.x, fma(-y, w.y, re));
      im = fma(v.x, w.y, fma(y, w.x, im));
      idx += k;
      if (idx >= N) idx -= N;
    }
    pw[k] = re * re + im * im;
  }
  __syncthreads();
  float mx = -FLT_MAX;
  for (int m = threadIdx.x; m < a.n_mels; m += blockDim.x) {
    const int lo = a.fband[2 * m], hi = a.fband[2 * m + 1];
    double s = 0.0;
#pragma unroll 8
    for (int k = lo; k < hi; ++k) s = fma(a.filters[(size_t)m * nb + k], pw[k], s);
    const float lg = (float)log10(fmax(s, 1e-10));
    a.logmel[(size_t)f * a.n_mels + m] = lg;
    mx = fmaxf(mx, lg);
  }
  mx = block_max(mx, red);
  if (threadIdx.x == 0) atomicMax(a.gmax, f2key(mx));
}

// every request's maximum starts below every value
__global__ void k_logmel_init(int* gmax, int nreq) {
  if ((int)threadIdx.x < nreq) gmax[threadIdx.x] = f2key(-FLT_MAX);
}

// Clamp and scale the log-mel values ((max(x, max - 8) + 4) / 4) and gather the
// first convolution's rows: A[t][c * 3 + j] = x[t + j - 1][c] (zero outside the
// frames and in the padding columns up to ld), bf16.  Optionally the scaled
// features [n_mels][frames] fp32 for inspection.
__global__ void __launch_bounds__(256) k_logmel_rows(LogmelArgs a) {
  a.logmel += (size_t)blockIdx.y * a.n_frames * a.n_mels;
  a.rows += (size_t)blockIdx.y * a.n_frames * a.ld1;
  const float top = key2f(a.gmax[blockIdx.y]) - 8.f;
  const size_t total = (size_t)a.n_frames * a.ld1;
  for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (size_t)gridDim.x * blockDim.x) {
    const int t = (int)(e / a.ld1), k = (int)(e % a.ld1);
    float v = 0.f;
    if (k < 3 * a.n_mels) {
      const int c = k / 3, j = k - 3 * c, src = t + j - 1;
      if (src >= 0 && src < a.n_frames) v = (fmaxf(a.logmel[(size_t)src * a.n_mels + c], top) + 4.f) * 0.25f;
    }
    a.rows[e] = from_f<bf16>(v);
    if (a.mel_out && k < a.n_mels)
      a.mel_out[(size_t)k * a.n_frames + t] = (fmaxf(a.logmel[(size_t)t * a.n_mels + k], top) + 4.f) * 0.25f;
  }
}

// Rows of the strided second convolution: A[t][c * 3 + j] = z[2 t + j - 1][c]
// (zero outside), t < n_out, from z [n_in][d] bf16.
__global__ void __launch_bounds__(256) k_conv_rows_s2(const bf16* __restrict__ z, bf16* __restrict__ out, int n_in,
                                                      int n_out, int d) {
  const size_t total = (size_t)n_out * d;
  z += (size_t)blockIdx.y * n_in * d;
  out += (size_t)blockIdx.y * 3 * total;
  for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (size_t)gridDim.x * blockDim.x) {
    const int t = (int)(e / d), c = (int)(e % d);
    bf16* o = out + (size_t)t * 3 * d + 3 * c;
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      const int src = 2 * t + j - 1;
      bf16 v;
      v.u = 0;
      if (src >= 0 && src < n_in) v = z[(size_t)src * d + c];
      o[j] = v;
    }
  }
}

// LayerNorm of fp32 rows [rows][d] of each request into bf16 rows (one wave per row,
// biased variance, eps 1e-5, two passes over the row held in registers; d a
// multiple of 4, each lane loading 16-byte runs of four columns).
__global__ void __launch_bounds__(256) k_ln_rows(const float* __restrict__ x, const bf16* __restrict__ g,
                                                 const bf16* __restrict__ b, bf16* __restrict__ out, int rows, int d,
                                                 int in_period, int out_period) {
  constexpr int kMax = kMaxEncD / 256;  // float4 runs per lane
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (row >= rows) return;
  x += (size_t)blockIdx.y * in_period * d;
  out += (size_t)blockIdx.y * out_period * d;
  const float4* xr = reinterpret_cast<const float4*>(x + (size_t)row * d);
  const int n4 = d >> 2;
  float4 v[kMax];
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < kMax; ++i) {
    const int c = lane + 64 * i;
    v[i] = c < n4 ? xr[c] : make_float4(0.f, 0.f, 0.f, 0.f);
    s += (v[i].x + v[i].y) + (v[i].z + v[i].w);
  }
  for (int o = 32; o; o >>= 1) s += __shfl_xor(s, o, 64);
  const float mean = s / d;
  float q = 0.f;
#pragma unroll
  for (int i = 0; i < kMax; ++i) {
    if (lane + 64 * i < n4) {
      const float a0 = v[i].x - mean, a1 = v[i].y - mean, a2 = v[i].z - mean, a3 = v[i].w - mean;
      q += (a0 * a0 + a1 * a1) + (a2 * a2 + a3 * a3);
    }
  }
  for (int o = 32; o; o >>= 1) q += __shfl_xor(q, o, 64);
  const float r = 1.f / sqrtf(q / d + 1e-5f);
#pragma unroll
  for (int i = 0; i < kMax; ++i) {
    const int c = lane + 64 * i;
    if (c < n4) {
      const int col = 4 * c;
      const float o0 = (v[i].x - mean) * r * to_f(g[col]) + to_f(b[col]);
      const float o1 = (v[i].y - mean) * r * to_f(g[col + 1]) + to_f(b[col + 1]);
      const float o2 = (v[i].z - mean) * r * to_f(g[col + 2]) + to_f(b[col + 2]);
      const float o3 = (v[i].w - mean) * r * to_f(g[col + 3]) + to_f(b[col + 3]);
      *reinterpret_cast<uint2*>(out + (size_t)row * d + col) = make_uint2(pack2_bf16(o0, o1), pack2_bf16(o2, o3));
    }
  }
}

// Bidirectional self-attention of one head over all positions, fused, one pass over
// the keys: one block per (128 queries, head), four waves of 32 queries.  Keys and
// transposed values stream through four LDS stages in tiles of 64 keys, copied
// straight from memory (global_load_lds_dwordx4) three tiles ahead of their use.
// Per 32 keys a wave forms S^T = K q^T on v_mfma_f32_32x32x16_bf16, so a lane holds 16
// keys of one query: the reference of its scores (near their maximum) and the sum are per
// lane (one swap of half-waves joins a query's two lanes), p is rounded to bf16 in place
// and two half-wave swaps of the packed pairs make it the B operand of O^T += V^T P^T.
// O and the sum are rescaled only where a reference moved.  Bound by the vector units
// (32 exponentials per lane and tile against 16 matrix instructions).  1500 positions, 20
// heads: 31.9 us; 70 with two passes over the keys and the probabilities through LDS.
namespace {
typedef __attribute__((address_space(3))) void lds_void;
constexpr int kAq = 128, kAk = 64, kAThreads = 256;
// stage layout (16-byte chunks): keys [key * 8 + chunk ^ (key & 7)] then
// transposed values [512 + dim * 8 + chunk ^ (dim & 7)]
constexpr int kStageChunks = 1024;
constexpr int kWaitKV = (8 & 15) | (7 << 4) | (0 << 8); // vmcnt <= 8: two later tiles' key + value copies
constexpr int kWaitAll = (0 & 15) | (7 << 4) | (15 << 8);
}  // namespace

// copies of key tile kt (its index clamped to the last tile) into a stage: wave w
// fills chunks (w * 2 + j) * 64 + lane of the keys and 512 + ... of the values
__device__ __forceinline__ void attn_copy(const EncAttnArgs& a, int head, int kt, int ntile, uint4* stage) {
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, k0 = min(kt, ntile - 1) * kAk;
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int slot = (w * 2 + j) * 64 + lane, r = slot >> 3, ch = (slot & 7) ^ (r & 7);
    const bf16* src = a.qk + (size_t)min(k0 + r, a.n - 1) * a.ldqk + a.d + head * kHeadDim + 8 * ch;
    __builtin_amdgcn_global_load_lds((const void*)src, (lds_void*)&stage[(w * 2 + j) * 64], 16, 0, 0);
  }
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int slot = (w * 2 + j) * 64 + lane, r = slot >> 3, ch = (slot & 7) ^ (r & 7);
    const bf16* src = a.vt + ((size_t)head * kHeadDim + r) * a.Tp + k0 + 8 * ch;
    __builtin_amdgcn_global_load_lds((const void*)src, (lds_void*)&stage[512 + (w * 2 + j) * 64], 16, 0, 0);
  }
}

__global__ void __launch_bounds__(kAThreads) k_enc_attn(EncAttnArgs a) {
  __shared__ uint4 g_att0[kStageChunks], g_att1[kStageChunks], g_att2[kStageChunks], g_att3[kStageChunks];
  const int head = blockIdx.y, q0 = blockIdx.x * kAq;
  a.qk += (size_t)blockIdx.z * a.sqk;
  a.vt += (size_t)blockIdx.z * a.svt;
  a.o += (size_t)blockIdx.z * a.so;
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, lr = lane & 31, lk = lane >> 5;
  const int ntile = (a.n + kAk - 1) / kAk;
  bf16x8 qf[4];
  {
    const int qrow = min(q0 + w * 32 + lr, a.n - 1);
    const bf16* qp = a.qk + (size_t)qrow * a.ldqk + head * kHeadDim + 8 * lk;
#pragma unroll
    for (int s = 0; s < 4; ++s) qf[s] = *reinterpret_cast<const bf16x8*>(qp + 16 * s);
  }
  // scores in units of log2(e) / 8, so the exponential is one instruction
  constexpr float kScale = 0.125f * 1.44269504088896340736f;
  // Scores are formed less a reference of their query (the products' accumulators start at its
  // negative, `nref`), so p = 2^(kScale s) with no rounding of the reference in it.  It becomes
  // the maximum of the first tile with a score above -inf, then moves only when a score
  // passes it by kRaise: p stays below 2^8
  constexpr float kRaise = 8.f / kScale;
  float raise = -INFINITY, l = 0.f;  // l: this lane's share of the sum
  floatx16 nref;
#pragma unroll
  for (int v = 0; v < 16; ++v) nref[v] = 0.f;
  floatx16 o[2];
#pragma unroll
  for (int nt = 0; nt < 2; ++nt)
#pragma unroll
    for (int v = 0; v < 16; ++v) o[nt][v] = 0.f;
  auto step = [&](int kt, const uint4* cur, uint4* nxt) {
    __builtin_amdgcn_s_waitcnt(kWaitKV);
    __builtin_amdgcn_s_barrier();
    attn_copy(a, head, kt + 3, ntile, nxt);  // every step issues its copies: exact wait counts
    if (kt >= ntile) return;
    floatx16 sc[2];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
      sc[kb] = nref;
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int row = kb * 32 + lr;
        const bf16x8 kf = __builtin_bit_cast(bf16x8, cur[row * 8 + ((2 * s + lk) ^ (row & 7))]);
        sc[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[s], sc[kb], 0, 0, 0);
      }
    }
    // lane: query lr, keys kt * 64 + kb * 32 + 8 (v / 4) + 4 lk + v % 4
    if (kt * kAk + kAk > a.n) {
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int v = 0; v < 16; ++v)
          if (kt * kAk + kb * 32 + 8 * (v >> 2) + 4 * lk + (v & 3) >= a.n) sc[kb][v] = -INFINITY;
    }
    float mx = sc[0][0];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int v = 0; v < 16; ++v) mx = fmaxf(mx, sc[kb][v]);
    const auto x = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
    mx = fmaxf(__uint_as_float(x[0]), __uint_as_float(x[1]));
    if (__builtin_amdgcn_ballot_w64(mx > raise)) {
      const float d = mx > raise ? mx : 0.f;
      const float f = raise > 0.f ? __builtin_amdgcn_exp2f(-d * kScale) : 0.f;  // no score yet: l and o are 0
      if (mx > raise) raise = kRaise;
      l *= f;
#pragma unroll
      for (int nt = 0; nt < 2; ++nt)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[nt][v] *= f;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        sc[0][v] -= d;
        sc[1][v] -= d;
        nref[v] -= d;
      }
    }
    float ls = 0.f;
    uint32_t pk[2][8];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int v = 0; v < 16; v += 2) {
        const float p0 = __builtin_amdgcn_exp2f(sc[kb][v] * kScale), p1 = __builtin_amdgcn_exp2f(sc[kb][v + 1] * kScale);
        ls += p0 + p1;
        pk[kb][v >> 1] = pack2_bf16(p0, p1);
      }
    l += ls;
    // values: 16 keys (substep s of key half kb) per instruction; lanes 0..31 need the
    // keys 16 s .. + 7 of their query, lanes 32..63 the keys 16 s + 8 .. + 15
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const auto y0 = __builtin_amdgcn_permlane32_swap(pk[kb][4 * s], pk[kb][4 * s + 2], false, false);
        const auto y1 = __builtin_amdgcn_permlane32_swap(pk[kb][4 * s + 1], pk[kb][4 * s + 3], false, false);
        const bf16x8 pf = __builtin_bit_cast(bf16x8, make_uint4(y0[0], y1[0], y0[1], y1[1]));
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
          const int row = nt * 32 + lr;
          const bf16x8 vf = __builtin_bit_cast(bf16x8, cur[512 + row * 8 + ((4 * kb + 2 * s + lk) ^ (row & 7))]);
          o[nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pf, o[nt], 0, 0, 0);
        }
      }
  };
  attn_copy(a, head, 0, ntile, g_att0);
  attn_copy(a, head, 1, ntile, g_att1);
  attn_copy(a, head, 2, ntile, g_att2);
  for (int kt = 0; kt < ntile; kt += 4) {
    step(kt, g_att0, g_att3);
    step(kt + 1, g_att1, g_att0);
    step(kt + 2, g_att2, g_att1);
    step(kt + 3, g_att3, g_att2);
  }
  __builtin_amdgcn_s_waitcnt(kWaitAll);  // no copy may land in LDS after the block has left
  const auto x = __builtin_amdgcn_permlane32_swap(__float_as_uint(l), __float_as_uint(l), false, false);
  const float inv = 1.f / (__uint_as_float(x[0]) + __uint_as_float(x[1]));
  // O^T: lane holds query lr, dims nt * 32 + 8 (v / 4) + 4 lk + v % 4
  const int q = q0 + w * 32 + lr;
  if (q < a.n) {
    bf16* op = a.o + (size_t)q * a.ldo + head * kHeadDim;
#pragma unroll
    for (int nt = 0; nt < 2; ++nt)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        *reinterpret_cast<uint2*>(op + nt * 32 + 8 * g + 4 * lk) =
            make_uint2(pack2_bf16(o[nt][4 * g] * inv, o[nt][4 * g + 1] * inv), pack2_bf16(o[nt][4 * g + 2] * inv, o[nt][4 * g + 3] * inv));
  }
}

void enc_attention(const EncAttnArgs& a, int n_head, hipStream_t st) {
  k_enc_attn<<<dim3((a.n + kAq - 1) / kAq, n_head, a.nreq), kAThreads, 0, st>>>(a);
}

void logmel(const LogmelArgs& a, hipStream_t st) {
  k_logmel_init<<<1, 64, 0, st>>>(a.gmax, a.nreq);
  int fft_a = 1;
  for (int i = 2; i * i <= a.n_fft; ++i)
    if (a.n_fft % i == 0) fft_a = i;
  k_logmel<<<dim3(a.n_frames, a.nreq), 256, 0, st>>>(a, fft_a);
  const size_t total = (size_t)a.n_frames * a.ld1;
  k_logmel_rows<<<dim3((unsigned)std::min<size_t>((total + 255) / 256, 4096), a.nreq), 256, 0, st>>>(a);
}
void conv_rows_s2(const bf16* z, bf16* out, int n_in, int n_out, int d, int nreq, hipStream_t st) {
  const size_t total = (size_t)n_out * d;
  k_conv_rows_s2<<<dim3((unsigned)std::min<size_t>((total + 255) / 256, 4096), nreq), 256, 0, st>>>(z, out, n_in, n_out, d);
}
void ln_rows(const float* x, const bf16* g, const bf16* b, bf16* out, int rows, int d, int nreq, int in_period,
             int out_period, hipStream_t st) {
  k_ln_rows<<<dim3((rows + 3) / 4, nreq), 256, 0, st>>>(x, g, b, out, rows, d, in_period, out_period);
}

}  // namespace wf
