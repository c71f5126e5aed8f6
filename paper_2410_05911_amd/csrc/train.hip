// Quantisation-aware training step of AECCT on the GPU: the second training phase of Section 6,
// in which the encoder's in-block linear maps are AAP linear layers (Section 4.1) over latent
// fp32 weights.  Forward with Eq. 1 ternarisation of the current weights and Eq. 2 absmax int8
// activations (both passing gradients straight through their rounding), the cross entropy of the
// multiplicative noise, and the backward pass to every parameter.  fp32 throughout, except that a map's
// input is held as what Eq. 2 makes of it, int8 codes and a row scale; every reduction runs in a fixed
// order (split partial sums reduced in index order), so a step is deterministic.
//
// Layouts: activations row-major [rows][features] with row b * L + r for token r of word b;
// weights [in][out] as in the inference ABI.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cfloat>
#include <cmath>

#include "aecct_internal.h"
#include "device_common.h"

namespace aecct {
namespace train {

constexpr int kThreads = 256;

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}

// ------------------------------------------------------------------------------------------
// Eq. 1 on the current latent weights, one block per matrix: gamma = Percentile(|W|, 0.5) (the
// order statistics at floor(pos) and floor(pos) + 1 for pos = (count - 1) / 2, interpolated in
// double and rounded once to fp32), s = fp32(gamma * delta), T = RoundClip(W / fp32(s + eps),
// -1, 1) with rounding half to even (a zero denominator maps a weight to its sign).  The order
// statistics come from a radix selection over the bit patterns of |W| (non-negative floats order
// like their bits) in digits of 12, 10 and 9 bits: the first takes the exponent and four mantissa bits, as
// the exponent alone leaves a wavefront's 64 keys in a few counters whose atomics then run one after the
// other.  A thread holds its keys (up to 64 Ki per matrix, 64 a thread) between the passes, in registers but for
// 31 of those 64, which do not fit beside the work of 1024 threads and go to scratch.  Eight-bit digits read from
// memory per pass took 95 us on 128 x 512 matrices.
// ------------------------------------------------------------------------------------------
using AapJob = TrainAapJob;
constexpr int kAapThreads = 1024, kAapWaves = kAapThreads / 64, kAapBins = 4096;

// The bucket of hist[0 .. bins) (bins a multiple of 512, at most 4096) holding the k-th counted key, and the
// key's rank inside it, to pick.  Every thread sums bins / 1024 or fewer buckets; wavefront totals through ws.
__device__ void select_bucket(const uint32_t *hist, int bins, uint32_t k, uint32_t *ws, uint32_t *pick) {
  const int per = bins > kAapThreads ? bins / kAapThreads : 1, first = threadIdx.x * per;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t t = 0;
  for (int b = 0; b < per; ++b) t += first + b < bins ? hist[first + b] : 0u;
  uint32_t incl = t;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t up = __shfl_up(incl, o, 64);
    if (lane >= o) incl += up;
  }
  if (lane == 63) ws[wave] = incl;
  __syncthreads();
  uint32_t before = 0;
  for (int w = 0; w < wave; ++w) before += ws[w];
  const uint32_t excl = before + incl - t;
  if (excl <= k && k < excl + t) {   // one thread
    uint32_t kk = k - excl;
    int b = first;
    while (kk >= hist[b]) kk -= hist[b++];
    pick[0] = b;
    pick[1] = kk;
  }
  __syncthreads();
}

// HELD: the launch's largest matrix in multiples of 1024 entries, rounded up to 4, 16 or 64
template <int HELD>
__global__ __launch_bounds__(kAapThreads) void k_aap(TrainAapJobs jobs, float eps) {
  __shared__ uint32_t hist[kAapBins];
  __shared__ uint32_t pick[2], ws[kAapWaves], wgt[kAapWaves];
  __shared__ float sden;
  const AapJob J = jobs.j[blockIdx.x];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, count = (int)J.count;
  const uint32_t lo = (uint32_t)((count - 1) / 2);
  const int held = count / kAapThreads;   // whole: d x d and d x 4 d entries of d = 32, 64, 128
  float w[HELD];
#pragma unroll
  for (int e = 0; e < HELD; ++e) {
    w[e] = 0.0f;
    if (e < held) w[e] = J.w[tid + e * kAapThreads];
  }
  uint32_t prefix = 0, mask = 0, k = lo;
#pragma unroll
  for (int pass = 0; pass < 3; ++pass) {
    const int shift = pass == 0 ? 19 : (pass == 1 ? 9 : 0), bins = pass == 0 ? 4096 : (pass == 1 ? 1024 : 512);
    for (int b = tid; b < bins; b += kAapThreads) hist[b] = 0;
    __syncthreads();
#pragma unroll
    for (int e = 0; e < HELD; ++e) {
      const uint32_t key = __float_as_uint(fabsf(w[e]));
      if (e < held && (key & mask) == prefix) atomicAdd(&hist[(key >> shift) & (bins - 1)], 1u);
      if ((e & 3) == 3) __builtin_amdgcn_sched_barrier(0);   // few keys in the making: the held ones fill the registers
    }
    __syncthreads();
    select_bucket(hist, bins, k, ws, pick);
    prefix |= pick[0] << shift;
    mask |= (uint32_t)(bins - 1) << shift;
    k = pick[1];
    __syncthreads();
  }
  const uint32_t a_lo = prefix;
  // the next order statistic: a_lo again if more than lo + 1 keys are <= a_lo, else the least
  // key above it
  uint32_t le = 0, gt = 0xffffffffu;
#pragma unroll
  for (int e = 0; e < HELD; ++e) {
    const uint32_t key = __float_as_uint(fabsf(w[e]));
    if (e < held) {
      if (key <= a_lo) ++le;
      else gt = min(gt, key);
    }
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    le += __shfl_xor(le, o, 64);
    gt = min(gt, (uint32_t)__shfl_xor(gt, o, 64));
  }
  if (lane == 0) {
    ws[wave] = le;
    wgt[wave] = gt;
  }
  __syncthreads();
  if (tid == 0) {
    uint32_t n_le = 0, g = 0xffffffffu;
    for (int u = 0; u < kAapWaves; ++u) {
      n_le += ws[u];
      g = min(g, wgt[u]);
    }
    const uint32_t a_hi = (lo + 1 >= (uint32_t)count || n_le > lo + 1) ? a_lo : g;
    const double pos = 0.5 * (double)(count - 1);
    const double frac = pos - (double)lo;
    const double flo = (double)__uint_as_float(a_lo), fhi = (double)__uint_as_float(a_hi);
    const float gamma = (float)(flo + frac * (fhi - flo));
    const float s = gamma * J.delta[0];
    *J.gamma = gamma;
    *J.scale = s;
    sden = s + eps;
  }
  __syncthreads();
  const float den = sden;
#pragma unroll
  for (int e = 0; e < HELD; ++e) {
    if (e < held) {
      const float x = w[e];
      float r = den == 0.0f ? (x > 0.0f ? 1.0f : (x < 0.0f ? -1.0f : 0.0f)) : rintf(x / den);
      J.t[tid + e * kAapThreads] = fminf(1.0f, fmaxf(-1.0f, r));
    }
    if ((e & 3) == 3) __builtin_amdgcn_sched_barrier(0);
  }
}

// ------------------------------------------------------------------------------------------
// Pre-processing and embedding (Section 3): t = [|y|, 1 - 2 s(y)], X = t E (+ P), and the Eq. 2 codes
// of X with their scale alpha / 127; one wavefront per token row.
//
// Every map's input is kept as Eq. 2 codes (int8, natural layout) and t = alpha / 127 per row; the value
// they stand for is code x t.  The forward maps then are exact integer products scaled once in the
// epilogue, fma(acc, t s, bias), and the weight gradients take the codes as exact bf16 operands.
// ------------------------------------------------------------------------------------------
__global__ __launch_bounds__(kThreads) void k_embed(const float *y, int64_t rows, int n, int L, int d,
                                                    const int32_t *chk_ptr, const int32_t *chk_idx, const float *E,
                                                    const float *P, float *x, float *tv, int8_t *xq, float *tx) {
  const int64_t r = (int64_t)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (r >= rows) return;
  const int64_t w = r / L;
  const int i = (int)(r - w * L);
  const float *yw = y + w * n;
  float t;
  if (i < n) {
    t = fabsf(yw[i]);
  } else {
    int s = 0;
    for (int e = chk_ptr[i - n]; e < chk_ptr[i - n + 1]; ++e) s ^= yw[chk_idx[e]] < 0.0f ? 1 : 0;
    t = s ? -1.0f : 1.0f;
  }
  float v[2], a = 0.0f;   // d <= 128
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int c = lane + 64 * u;
    v[u] = c < d ? fmaf(t, E[(int64_t)i * d + c], P ? P[(int64_t)i * d + c] : 0.0f) : 0.0f;
    if (c < d) x[r * d + c] = v[u];
    a = fmaxf(a, fabsf(v[u]));
  }
  a = wave_max(a);
  const float inv = inv127(a);
#pragma unroll
  for (int u = 0; u < 2; ++u)
    if (lane + 64 * u < d) xq[r * d + lane + 64 * u] = quant_code(v[u], inv);
  if (lane == 0) {
    tv[r] = t;
    tx[r] = a / 127.0f;
  }
}

// ------------------------------------------------------------------------------------------
// fp32 GEMM of the head: C[M][N] = op(A) op(B) + bias[N], op(A) = A [M][K] (lda) or, with TA,
// the transpose of A stored [K][M]; op(B) = B [K][N] (ldb) or, with TB, the transpose of B stored
// [N][K].  64 x 64 output tiles, 64-deep K steps through LDS (the head's short products take one or two:
// 16-deep steps, each with a memory latency of its own, took 39 us in all on BCH(31,16), 128 words),
// 4 x 4 outputs per thread, FMAs in ascending k.  With gridDim.z > 1 each z takes one contiguous k range and writes its raw sum to
// part[z][M][N]; k_gemm_reduce then adds the ranges in index order and applies the epilogue.
// ------------------------------------------------------------------------------------------
constexpr int kVgK = 64;

struct GemmF32 {
  const float *A, *B;
  float *C;
  int64_t M, N, K;
  int64_t lda, ldb, ldc;
  int64_t kchunk;
  const float *bias;    // [N] or null
  float *part;          // [splits][M][N] when split
};

template <bool TA, bool TB>
__global__ __launch_bounds__(kThreads) void k_gemm(GemmF32 g) {
  __shared__ float As[kVgK][64 + 4];
  __shared__ float Bs[kVgK][64 + 4];
  const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
  const int64_t m0 = (int64_t)blockIdx.y * 64, n0 = (int64_t)blockIdx.x * 64;
  const int64_t kb = (int64_t)blockIdx.z * g.kchunk, ke = std::min<int64_t>(g.K, kb + g.kchunk);
  float acc[4][4] = {};
  for (int64_t k0 = kb; k0 < ke; k0 += kVgK) {
    float va[kVgK / 4], vb[kVgK / 4];   // every load of the step before its first LDS store
#pragma unroll
    for (int u = 0; u < kVgK / 4; ++u) {
      const int idx = tid + kThreads * u;
      const int ma = TA ? idx & 63 : idx / kVgK, ka = TA ? idx >> 6 : idx % kVgK;
      const int64_t gm = m0 + ma, gk = k0 + ka;
      va[u] = gm < g.M && gk < ke ? (TA ? g.A[gk * g.lda + gm] : g.A[gm * g.lda + gk]) : 0.0f;
      const int nb = TB ? idx / kVgK : idx & 63, kb2 = TB ? idx % kVgK : idx >> 6;
      const int64_t gn = n0 + nb, gk2 = k0 + kb2;
      vb[u] = gn < g.N && gk2 < ke ? (TB ? g.B[gn * g.ldb + gk2] : g.B[gk2 * g.ldb + gn]) : 0.0f;
    }
#pragma unroll
    for (int u = 0; u < kVgK / 4; ++u) {
      const int idx = tid + kThreads * u;
      As[TA ? idx >> 6 : idx % kVgK][TA ? idx & 63 : idx / kVgK] = va[u];
      Bs[TB ? idx % kVgK : idx >> 6][TB ? idx / kVgK : idx & 63] = vb[u];
    }
    __syncthreads();
    const int kn = (int)std::min<int64_t>(kVgK, ke - k0);
#pragma unroll 8
    for (int kk = 0; kk < kn; ++kk) {
      float a[4], b[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = As[kk][4 * ty + i];
#pragma unroll
      for (int j = 0; j < 4; ++j) b[j] = Bs[kk][4 * tx + j];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(a[i], b[j], acc[i][j]);
    }
    __syncthreads();
  }
  const bool split = gridDim.z > 1;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int64_t r = m0 + 4 * ty + i;
    if (r >= g.M) continue;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int64_t c = n0 + 4 * tx + j;
      if (c >= g.N) continue;
      if (split) {
        g.part[((int64_t)blockIdx.z * g.M + r) * g.N + c] = acc[i][j];
      } else {
        g.C[r * g.ldc + c] = acc[i][j] + (g.bias ? g.bias[c] : 0.0f);
      }
    }
  }
}

// The same product on v_mfma_f32_16x16x4_f32 for operands whose contiguous dimension and leading
// dimensions are multiples of 4 floats (16-byte loads): blocks of 64 x 128 outputs, four wavefronts of
// 32 x 64 (2 x 4 MFMA tiles), k-steps of 32 staged through LDS, the next step's operands loaded into
// registers while the current one is multiplied.  What binds is the number of blocks: tiles of 128 x 128 were
// slower on all three products from LDPC(64,32) to LDPC(1024,512) and 64 to 16384 words (logits of LDPC(256,128), 512
// words 27.3 us, these 18.0; LDPC(1024,512), 2048 words 108.2, these 88.5).  LDS rows of 80 and 144 floats put the
// four k rows an MFMA fragment reads 16 banks apart.  MFMA layout (lane l): A row l & 15 at k = l >> 4,
// B column l & 15 at k = l >> 4, D rows 4 (l >> 4) + i, column l & 15.
typedef float v4f __attribute__((ext_vector_type(4)));
constexpr int kMfRows = 64, kMfTile = 128, kMfK = 32;

__device__ __forceinline__ float4 load4_if(const float *p, bool ok) {
  float4 v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  if (ok) v = *(const float4 *)p;
  return v;
}

template <bool TA, bool TB>
__global__ __launch_bounds__(kThreads) void k_gemm_mfma(GemmF32 g) {
  constexpr int BM = kMfRows, BN = kMfTile, AP = BM / 32, BP = BN / 32, TM = BM / 32;
  __shared__ __attribute__((aligned(16))) float As[kMfK][BM + 16];
  __shared__ __attribute__((aligned(16))) float Bs[kMfK][BN + 16];
  const float *__restrict__ A = g.A;
  const float *__restrict__ B = g.B;
  const int64_t M = g.M, N = g.N, lda = g.lda, ldb = g.ldb;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int wm = (wave >> 1) * (BM / 2), wn = (wave & 1) * 64;
  const int64_t m0 = (int64_t)blockIdx.y * BM, n0 = (int64_t)blockIdx.x * BN;
  const int64_t kb = (int64_t)blockIdx.z * g.kchunk, ke = std::min<int64_t>(g.K, kb + g.kchunk);
  // Thread t stages float4 number t + 256 u of each 32 x W operand tile (W = 64 or 128).  Stored
  // k-major ([k][m] or [k][n]): k row t / (W / 4) + u 1024 / W, columns 4 (t mod W / 4) .. +3.
  // Stored with k contiguous: tile row (t >> 3) + 32 u, k offsets 4 (t & 7) .. +3.
  const int kmA_r = tid / (BM / 4), kmA_c = (tid % (BM / 4)) * 4, kmB_r = tid >> 5, kmB_c = (tid & 31) * 4;
  const int kc_r = tid >> 3, kc_k = (tid & 7) * 4;
  float4 ra[AP], rb[BP];
  v4f acc[TM][4];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
  const int fr = lane >> 4, fc = lane & 15;
  for (int64_t k0 = kb, first = 1; k0 < ke; k0 += kMfK, first = 0) {
    if (first) {
      // the first step's operands (later steps' were read during the previous step)
#pragma unroll
      for (int u = 0; u < AP; ++u) {
        if (TA) {
          const int64_t gk = k0 + kmA_r + u * (1024 / BM);
          ra[u] = load4_if(A + gk * lda + m0 + kmA_c, gk < ke && m0 + kmA_c < M);
        } else {
          const int64_t gm = m0 + kc_r + 32 * u;
          ra[u] = load4_if(A + gm * lda + k0 + kc_k, gm < M && k0 + kc_k < ke);
        }
      }
#pragma unroll
      for (int u = 0; u < BP; ++u) {
        if (TB) {
          const int64_t gn = n0 + kc_r + 32 * u;
          rb[u] = load4_if(B + gn * ldb + k0 + kc_k, gn < N && k0 + kc_k < ke);
        } else {
          const int64_t gk = k0 + kmB_r + 8 * u;
          rb[u] = load4_if(B + gk * ldb + n0 + kmB_c, gk < ke && n0 + kmB_c < N);
        }
      }
    }
#pragma unroll
    for (int u = 0; u < AP; ++u) {
      if (TA) {
        *(float4 *)&As[kmA_r + u * (1024 / BM)][kmA_c] = ra[u];
      } else {
        const int mm = kc_r + 32 * u;
        As[kc_k][mm] = ra[u].x; As[kc_k + 1][mm] = ra[u].y; As[kc_k + 2][mm] = ra[u].z; As[kc_k + 3][mm] = ra[u].w;
      }
    }
#pragma unroll
    for (int u = 0; u < BP; ++u) {
      if (TB) {
        const int nn = kc_r + 32 * u;
        Bs[kc_k][nn] = rb[u].x; Bs[kc_k + 1][nn] = rb[u].y; Bs[kc_k + 2][nn] = rb[u].z; Bs[kc_k + 3][nn] = rb[u].w;
      } else {
        *(float4 *)&Bs[kmB_r + 8 * u][kmB_c] = rb[u];
      }
    }
    __syncthreads();
    const int64_t k1 = k0 + kMfK;
    if (k1 < ke) {
#pragma unroll
      for (int u = 0; u < AP; ++u) {
        if (TA) {
          const int64_t gk = k1 + kmA_r + u * (1024 / BM);
          ra[u] = load4_if(A + gk * lda + m0 + kmA_c, gk < ke && m0 + kmA_c < M);
        } else {
          const int64_t gm = m0 + kc_r + 32 * u;
          ra[u] = load4_if(A + gm * lda + k1 + kc_k, gm < M && k1 + kc_k < ke);
        }
      }
#pragma unroll
      for (int u = 0; u < BP; ++u) {
        if (TB) {
          const int64_t gn = n0 + kc_r + 32 * u;
          rb[u] = load4_if(B + gn * ldb + k1 + kc_k, gn < N && k1 + kc_k < ke);
        } else {
          const int64_t gk = k1 + kmB_r + 8 * u;
          rb[u] = load4_if(B + gk * ldb + n0 + kmB_c, gk < ke && n0 + kmB_c < N);
        }
      }
    }
#pragma unroll
    for (int ks = 0; ks < kMfK / 4; ++ks) {
      float av[TM], bv[4];
#pragma unroll
      for (int t = 0; t < TM; ++t) av[t] = As[4 * ks + fr][wm + 16 * t + fc];
#pragma unroll
      for (int t = 0; t < 4; ++t) bv[t] = Bs[4 * ks + fr][wn + 16 * t + fc];
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[i], bv[j], acc[i][j], 0, 0, 0);
    }
    __syncthreads();
  }
  // split partial sums raw into their slice of part, else with the bias
  const bool split = gridDim.z > 1;
  float *const P = split ? g.part + (int64_t)blockIdx.z * M * N : g.C;
  const int64_t ld = split ? N : g.ldc;
  const float *bias = split ? nullptr : g.bias;
  const bool full = m0 + BM <= M && n0 + BN <= N;
  float bj[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int64_t c = n0 + wn + 16 * j + fc;
    bj[j] = (bias && c < N) ? bias[c] : 0.0f;
  }
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int64_t r = m0 + wm + 16 * i + 4 * fr + v;
      if (!full && r >= M) continue;
      float *prow = P + r * ld + n0 + wn + fc;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (!full && n0 + wn + 16 * j + fc >= N) continue;
        prow[16 * j] = acc[i][j][v] + bj[j];
      }
    }
}

// ------------------------------------------------------------------------------------------
// Input gradients, products with a ternary operand: C[M][N] = D + sum_s scale_s (A_s T_s^T) where T holds
// only -1, 0, +1 (Eq. 1) and A is fp32.  Each fp32 a splits exactly into three bf16 parts, a = hi + mid +
// lo (hi the leading 8 significant bits by truncation, mid the next 8, lo the remaining at most 8), each
// part times a ternary entry is exact, and the three v_mfma_f32_16x16x32_bf16 products accumulate in
// fp32: the result is an fp32-accumulated sum of exact products, as in the fp32 kernels, at the bf16
// matrix rate.  (The MFMA reads a subnormal part as 0, so the split is whole for |a| above about 1e-33; with the
// step's gradients scaled down to 1e-28 the results are the same to 1e-7, at 1e-30 to 1e-4.)  T^T comes pre-packed as bf16 MFMA B fragments (k_pack_tern).  A wave computes 16 rows x
// 16 NJ columns, a block four waves.
// ------------------------------------------------------------------------------------------
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// Up to three ternary matrices in one product, one after another along k (segments of kseg k-steps of
// A's row: the input gradient summed over the query, key and value maps from the packed [rows][3 d]
// gradient).  Segment s has its own fragments and scale; D is an optional addend laid out like C.
struct GemmTern {
  const float *A;
  const uint4 *B[3];       // fragment (nt, kt) at (nt * kt_s + kt) * 64, kt_s the segment's k-steps:
                           // lane l holds column 16 nt + (l & 15), k = 32 kt + 8 (l >> 4) + e, bf16 e = 0..7
  float *C;
  const float *D;
  int64_t M, N, K, lda, ldc;
  const float *scale[3];   // device scalar or null (1)
  int kseg;                // k-steps per k segment (K / 32 when there is one)
};

template <typename T>
__device__ __forceinline__ T pick3(const T (&v)[3], int i) {   // a selected kernel argument, no indexing
  return i == 0 ? v[0] : (i == 1 ? v[1] : v[2]);
}

// Ternary matrix T [R][C] (fp32 -1 / 0 / +1, row-major), one job per blockIdx.y, as
//   kTernBf16T: bf16 B fragments of T^T (k = column, n = row) for the input gradient of Q | K | V;
//   kTernSelT: selector-byte A fragments of T^T (output rows = rows of T, k = columns of T in the order
//   of Hidden below) for k_train_bwd;
//   kTernI8, kTernI8Hidden: int8 A fragments of the transposed forward products (output rows = columns
//   of T, k = rows of T): fragment (t, s), lane l: output 16 t + (l & 15), k-slots 8 (l >> 4) + e in
//   byte e.  Slot k of step s reads input 32 s + k, or (Hidden) input 32 s + 16 (e >> 2) + 4 (l >> 4) +
//   (e & 3): the eight codes that the product before leaves in a lane group.
__global__ __launch_bounds__(kThreads) void k_pack_tern(TernPackJobs jobs) {
  const TernPackJob &J = jobs.j[blockIdx.y];
  const float *T = J.T;
  const int R = J.R, Cc = J.C;
  const int64_t u = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (u >= (int64_t)R * Cc / 8) return;
  const int l = (int)(u & 63), f = (int)(u >> 6), g = l >> 4;
  if (J.mode == kTernBf16T) {
    const int KT = Cc / 32, nt = f / KT, kt = f - nt * KT;
    const int n = 16 * nt + (l & 15), k0 = 32 * kt + 8 * g;
    uint32_t h[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float t = T[(int64_t)n * Cc + k0 + e];
      h[e] = t > 0.0f ? 0x3F80u : (t < 0.0f ? 0xBF80u : 0u);   // bf16 of +1, -1, 0
    }
    ((uint4 *)J.out)[u] = make_uint4(h[0] | h[1] << 16, h[2] | h[3] << 16, h[4] | h[5] << 16, h[6] | h[7] << 16);
    return;
  }
  uint64_t w = 0;
  if (J.mode == kTernSelT) {
    const int S = Cc / 32, t = f / S, s = f - t * S, r = 16 * t + (l & 15);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float v = T[(int64_t)r * Cc + 32 * s + 16 * (e >> 2) + 4 * g + (e & 3)];
      w |= (uint64_t)(v > 0.0f ? 1u : (v < 0.0f ? 2u : 0u)) << (8 * e);
    }
    ((uint64_t *)J.out)[u] = w;
    return;
  }
  const int S = R / 32, t = f / S, s = f - t * S, c = 16 * t + (l & 15);
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int k = 32 * s + (J.mode == kTernI8Hidden ? 16 * (e >> 2) + 4 * g + (e & 3) : 8 * g + e);
    w |= (uint64_t)(uint8_t)(int8_t)T[(int64_t)k * Cc + c] << (8 * e);
  }
  ((uint64_t *)J.out)[u] = w;
}

// the bf16 bit patterns of eight fp32 values that are exact in bf16 (low 16 bits zero)
__device__ __forceinline__ bf16x8 bf16_hi8(const float (&v)[8]) {
  uint4 w;
  w.x = __builtin_amdgcn_perm(__builtin_bit_cast(uint32_t, v[1]), __builtin_bit_cast(uint32_t, v[0]), 0x07060302u);
  w.y = __builtin_amdgcn_perm(__builtin_bit_cast(uint32_t, v[3]), __builtin_bit_cast(uint32_t, v[2]), 0x07060302u);
  w.z = __builtin_amdgcn_perm(__builtin_bit_cast(uint32_t, v[5]), __builtin_bit_cast(uint32_t, v[4]), 0x07060302u);
  w.w = __builtin_amdgcn_perm(__builtin_bit_cast(uint32_t, v[7]), __builtin_bit_cast(uint32_t, v[6]), 0x07060302u);
  return __builtin_bit_cast(bf16x8, w);
}

// the three bf16 parts of eight fp32 values as MFMA operands.  INF: an infinity is its leading part alone, so that
// its products are what the fp32 product gives (infinite, or NaN with a zero); otherwise Inf - Inf makes its
// other parts, and every sum it enters, NaN.  The weight gradients take it, and the input gradients at d = 32:
// 0.2 % of a step at d = 128, 0.5 % at 32 and 64.
template <bool INF>
__device__ __forceinline__ void split_bf16x3(const float4 &x0, const float4 &x1, bf16x8 &ph, bf16x8 &pm, bf16x8 &pl) {
  const float a[8] = {x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w};
  float hi[8], mid[8], lo[8];
  const auto rest = [&](int e, float rm) {
    mid[e] = __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, rm) & 0xFFFF0000u);
    lo[e] = rm - mid[e];
  };
  if constexpr (INF) {
    float rm[8], top = 0.0f;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      hi[e] = __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, a[e]) & 0xFFFF0000u);
      rm[e] = a[e] - hi[e];
      top = fmaxf(top, fabsf(a[e]));
    }
    if (__builtin_expect(__any(top == INFINITY), 0)) {
#pragma unroll
      for (int e = 0; e < 8; ++e) rm[e] = a[e] == hi[e] ? 0.0f : rm[e];
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) rest(e, rm[e]);
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      hi[e] = __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, a[e]) & 0xFFFF0000u);
      rest(e, a[e] - hi[e]);
    }
  }
  ph = bf16_hi8(hi);
  pm = bf16_hi8(mid);
  pl = bf16_hi8(lo);
}

// The MFMA takes the ternary fragment as its first operand and A's as its second, so it forms the
// transposed tile: lane (col, grp) ends with row 16 t + col, columns 16 j + 4 grp .. + 3 of C, one
// 16-byte store (and, with beta, one 16-byte load) per tile.  Both operands of k-step kt + S - 1 are
// loaded before step kt is computed, from a ring of S register slots: the vector-memory counter
// retires loads in issue order, so a B fragment loaded just before its use would also wait for
// every A prefetch issued ahead of it.  C goes out with ordinary stores: the next kernel reads it,
// partly from the caches (nontemporal stores measured slower over a training step).
template <int NJ, int S>
__global__ __launch_bounds__(kThreads) void k_gemm_tern(GemmTern g) {
  const int wave = threadIdx.x >> 6, l = threadIdx.x & 63, col = l & 15, grp = l >> 4;
  const int64_t m0 = (int64_t)blockIdx.y * 64 + 16 * wave, n0 = (int64_t)blockIdx.x * (16 * NJ);
  const int KT = (int)(g.K / 32), ks = g.kseg;
  const int64_t r = m0 + col;
  const float *arow = g.A + (r < g.M ? r : g.M - 1) * g.lda + 8 * grp;   // rows past M: a copy, never stored
  f32x4 acc[NJ];
  float4 o[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    acc[j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    o[j] = float4{0.0f, 0.0f, 0.0f, 0.0f};
  }
  float4 a[S][2];
  uint4 b[S][NJ];
  auto issue = [&](int kt, float4 (&as)[2], uint4 (&bs)[NJ]) {
    const int s = kt / ks;   // the k segment (0 with one)
    const uint4 *bcol = pick3(g.B, s) + (n0 / 16) * ks * 64 + l;
#pragma unroll
    for (int j = 0; j < NJ; ++j) bs[j] = bcol[(j * ks + kt - s * ks) * 64];
    as[0] = *(const float4 *)(arow + 32 * kt);
    as[1] = *(const float4 *)(arow + 32 * kt + 4);
  };
  int kend = ks;   // the current k segment ends before step kend
#pragma unroll
  for (int s = 0; s < S - 1; ++s)
    if (s < KT) issue(s, a[s], b[s]);
  for (int k0 = 0; k0 < KT; k0 += S) {
#pragma unroll
    for (int s = 0; s < S; ++s) {   // step k0 + s sits in slot s
      const int kt = k0 + s;
      if (kt >= KT) break;
      if (kt + S - 1 < KT) issue(kt + S - 1, a[(s + S - 1) % S], b[(s + S - 1) % S]);
      bf16x8 ph, pm, pl;
      split_bf16x3<NJ == 2>(a[s][0], a[s][1], ph, pm, pl);
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const bf16x8 bb = __builtin_bit_cast(bf16x8, b[s][j]);
        acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bb, pl, acc[j], 0, 0, 0);
        acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bb, pm, acc[j], 0, 0, 0);
        acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bb, ph, acc[j], 0, 0, 0);
      }
      if (kt + 1 == kend) {   // a k segment's products, scaled, into o
        const float *sp = pick3(g.scale, kt / ks);
        const float sc = sp ? *sp : 1.0f;
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          o[j].x += sc * acc[j][0];
          o[j].y += sc * acc[j][1];
          o[j].z += sc * acc[j][2];
          o[j].w += sc * acc[j][3];
          acc[j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        }
        kend += ks;
      }
    }
  }
  if (r >= g.M) return;
  float *crow = g.C + r * g.ldc + n0 + 4 * grp;
  const float *drow = g.D ? g.D + r * g.ldc + n0 + 4 * grp : nullptr;
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    float4 u = o[j];
    if (drow) {
      const float4 dv = *(const float4 *)(drow + 16 * j);
      u.x += dv.x;
      u.y += dv.y;
      u.z += dv.z;
      u.w += dv.w;
    }
    *(float4 *)(crow + 16 * j) = u;
  }
}

// Split-k partial products summed in a fixed order: a block covers 64 outputs, its four lanes per
// output sum the splits z = lane, lane + 4, ... and are added in lane order.
__global__ __launch_bounds__(kThreads) void k_gemm_reduce(GemmF32 g, int splits) {
  __shared__ float red[4][64];
  const int cl = threadIdx.x & 63, rl = threadIdx.x >> 6;
  const int64_t e = (int64_t)blockIdx.x * 64 + cl, MN = g.M * g.N;
  float s0 = 0.0f, s1 = 0.0f;
  if (e < MN) {
    int z = rl;
    for (; z + 4 < splits; z += 8) {
      s0 += g.part[(int64_t)z * MN + e];
      s1 += g.part[(int64_t)(z + 4) * MN + e];
    }
    if (z < splits) s0 += g.part[(int64_t)z * MN + e];
  }
  red[rl][cl] = s0 + s1;
  __syncthreads();
  if (rl != 0 || e >= MN) return;
  const float s = ((red[0][cl] + red[1][cl]) + red[2][cl]) + red[3][cl];
  const int64_t r = e / g.N, c = e - r * g.N;
  g.C[r * g.ldc + c] = s + (g.bias ? g.bias[c] : 0.0f);
}

// ------------------------------------------------------------------------------------------
// Forward maps on Eq. 2 codes.  One wavefront per 16-token strip, products transposed on int8 MFMA
// (weights the A operand, from LDS; the strip's tokens the columns), so lane (c, g) = (lane & 15,
// lane >> 4) ends with outputs 16 t + 4 g .. + 3 of token c for every output tile t: one 16-byte
// access per tile in the natural row layout.  int32 sums are exact; the only rounding of a map is
// fma(acc, t s, bias).
//
// k_train_block is the inference path's token block with the backward's inputs written on the way.  The
// separate kernels it stands for (quantise O, output map, LayerNorm, first map, ReLU and quantise,
// second map, LayerNorm) passed every activation through memory in fp32 and wrote the dequantised
// codes as fp32: LDPC(256,128), 256 words, 440 us a layer; this one moves 3 KB a token and takes 93 us (57 at
// the copy's rate).  Strips go out wavefront-major, so that a batch of fewer strips than the card has
// wavefronts spreads over every compute unit (BCH(31,16), 128 words: step 0.42 -> 0.40 ms).
// ------------------------------------------------------------------------------------------
constexpr int kTbWaves = 8;

template <int D>
constexpr size_t qkv_lds() { return (size_t)3 * D * D + (size_t)3 * D * 4; }
template <int D>
constexpr size_t block_lds() { return (size_t)9 * D * D + (size_t)12 * D * 4; }

// `words` 16-byte words to LDS, four loads of a thread in flight at a time (as v4i: a HIP uint4 stored under a
// condition goes through scratch memory with this compiler)
__device__ __forceinline__ void stage16(const void *src, void *dst, int words, int tid) {
  constexpr int NT = kTbWaves * 64;
  for (int u = tid; u < words; u += 4 * NT) {
    v4i r[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) r[k] = ((const v4i *)src)[std::min(u + k * NT, words - 1)];
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (u + k * NT < words) ((v4i *)dst)[u + k * NT] = r[k];
  }
}
__device__ __forceinline__ void stage_vec(const float *src, float *dst, int n, int tid) {
  for (int u = tid; u < n; u += kTbWaves * 64) dst[u] = src[u];
}

template <int D>
__global__ __launch_bounds__(kTbWaves * 64) void k_train_qkv(TrainQkv p) {
  constexpr int S = D / 32, TO = D / 16;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, c = lane & 15, g = lane >> 4;
  uint64_t *fr = (uint64_t *)smem;               // [3][TO][S][64]
  float *bl = (float *)(smem + (size_t)3 * D * D);
#pragma unroll
  for (int m = 0; m < 3; ++m) {
    stage16(p.f[m], fr + (size_t)m * TO * S * 64, D * D / 16, tid);
    stage_vec(p.b[m], bl + m * D, D, tid);
  }
  __syncthreads();
  const float sq[3] = {*p.s[0], *p.s[1], *p.s[2]};
  const int64_t nstrips = (p.rows + 15) / 16, stride = (int64_t)gridDim.x * kTbWaves;
  for (int64_t strip = (int64_t)wave * gridDim.x + blockIdx.x; strip < nstrips; strip += stride) {
    const int64_t tok = strip * 16 + c, tl = tok < p.rows ? tok : p.rows - 1;
    long x[S];
#pragma unroll
    for (int s = 0; s < S; ++s) x[s] = *(const long *)(p.xq + tl * D + 32 * s + 8 * g);
    const float t = p.tx[tl];
    float *out = p.qkv + tok * 3 * D + 4 * g;
#pragma unroll
    for (int m = 0; m < 3; ++m) {
      const float sc = t * sq[m];
#pragma unroll
      for (int o = 0; o < TO; ++o) {
        const v4i acc = mfma_i8_steps<S>([&](int s) { return (long)fr[((m * TO + o) * S + s) * 64 + lane]; },
                                         [&](int s) { return x[s]; }, v4i{0, 0, 0, 0});
        const float4 b = *(const float4 *)(bl + m * D + 16 * o + 4 * g);
        if (tok < p.rows)
          *(float4 *)(out + m * D + 16 * o) =
              make_float4(fmaf((float)acc[0], sc, b.x), fmaf((float)acc[1], sc, b.y), fmaf((float)acc[2], sc, b.z),
                          fmaf((float)acc[3], sc, b.w));
      }
    }
  }
}

// Eq. 2 codes of a token's row held as x[v] = feature 16 (v >> 2) + 4 g + (v & 3): step s's eight codes
// of this lane (the next product's B operand) to xb, and to the natural row q of int8 codes.
template <int S>
__device__ __forceinline__ void store_codes(const float (&x)[8 * S], float inv, int g, bool ok, int8_t *q, long (&xb)[S]) {
#pragma unroll
  for (int s = 0; s < S; ++s) {
    uint32_t b[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) b[k] = quant_bits(x[8 * s + k], inv);
    xb[s] = tb_pack8(b);
    if (ok) {
      *(uint32_t *)(q + 32 * s + 4 * g) = (uint32_t)xb[s];
      *(uint32_t *)(q + 32 * s + 16 + 4 * g) = (uint32_t)((uint64_t)xb[s] >> 32);
    }
  }
}

template <int D>
__global__ __launch_bounds__(kTbWaves * 64) void k_train_block(TrainBlock p) {
  constexpr int V = D / 4, S = D / 32, TO = D / 16, TH = D / 4, SH = D / 8, MW = D / 32;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, c = lane & 15, g = lane >> 4;
  uint64_t *f1 = (uint64_t *)smem, *f2 = f1 + (size_t)TH * S * 64, *fo = f2 + (size_t)TO * SH * 64;
  float *lv = (float *)(smem + (size_t)9 * D * D);   // bo, g1, be1, b2, g2, be2, res_g, res_b, b1 [4 D]
  stage16(p.f1, f1, D * D / 4, tid);
  stage16(p.f2, f2, D * D / 4, tid);
  stage16(p.fo, fo, D * D / 16, tid);
  {
    const float *src[8] = {p.bo, p.g1, p.be1, p.b2, p.g2, p.be2, p.res_g, p.res_b};
#pragma unroll
    for (int k = 0; k < 8; ++k)
      if (src[k]) stage_vec(src[k], lv + k * D, D, tid);
    stage_vec(p.b1, lv + 8 * D, 4 * D, tid);
  }
  __syncthreads();
  const float so = *p.so, s1 = *p.s1, s2 = *p.s2;
  // the lane's fragments and vectors from opaque byte offsets, so that the unrolled reads share one
  // running address each
  uint32_t of1 = (uint32_t)lane * 8u, of2 = (uint32_t)(TH * S * 64 + lane) * 8u, ov = (uint32_t)(9 * D * D) + 16u * (uint32_t)g;
  asm volatile("" : "+v"(of1), "+v"(of2), "+v"(ov));
  const uint64_t *f1l = (const uint64_t *)(smem + of1), *f2l = (const uint64_t *)(smem + of2);
  const float *vl = (const float *)(smem + ov);       // vl[k D + 16 t + i]: vector k, feature 16 t + 4 g + i
  const int64_t nstrips = (p.rows + 15) / 16, stride = (int64_t)gridDim.x * kTbWaves;
  for (int64_t strip = (int64_t)wave * gridDim.x + blockIdx.x; strip < nstrips; strip += stride) {
    const int64_t tok = strip * 16 + c;
    const bool ok = tok < p.rows;
    const int64_t tl = ok ? tok : p.rows - 1;          // padding columns: a copy, never stored
    float x[V];                                        // the residual, then each LayerNorm's output
    long bq[S];
    float sc;
    {
      float ov8[8 * S], om = 0.0f;                     // the output map reads O's features 32 s + 8 g + e
#pragma unroll
      for (int s = 0; s < S; ++s)
#pragma unroll
        for (int k = 0; k < 8; k += 4) {
          const float4 f = *(const float4 *)(p.o + tl * D + 32 * s + 8 * g + k);
          ov8[8 * s + k] = f.x; ov8[8 * s + k + 1] = f.y; ov8[8 * s + k + 2] = f.z; ov8[8 * s + k + 3] = f.w;
        }
#pragma unroll
      for (int t = 0; t < TO; ++t) {
        const float4 f = *(const float4 *)(p.res + tl * D + 16 * t + 4 * g);
        x[4 * t] = f.x; x[4 * t + 1] = f.y; x[4 * t + 2] = f.z; x[4 * t + 3] = f.w;
      }
#pragma unroll
      for (int k = 0; k < 8 * S; ++k) om = fmaxf(om, fabsf(ov8[k]));
      om = tb_token_max(om);
      const float inv = inv127(om);
#pragma unroll
      for (int s = 0; s < S; ++s) {
        uint32_t b[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) b[k] = quant_bits(ov8[8 * s + k], inv);
        bq[s] = tb_pack8(b);
        if (ok) *(long *)(p.oq + tok * D + 32 * s + 8 * g) = bq[s];
      }
      const float t = om / 127.0f;
      if (ok && g == 0) p.to[tok] = t;
      sc = t * so;
    }
    if (p.res_g) {
#pragma unroll
      for (int v = 0; v < V; ++v) x[v] = fmaf(x[v], vl[6 * D + 16 * (v >> 2) + (v & 3)], vl[7 * D + 16 * (v >> 2) + (v & 3)]);
    }
    // x := LN(x), its normalised row and 1 / sigma to xn, rho; returns max |x| over the token
    auto norm = [&](int kg, int kb, float *xn, float *rho) {
      const float mean = tb_token_sum<V>(x) / (float)D;
      float q[V];
#pragma unroll
      for (int v = 0; v < V; ++v) {
        x[v] = x[v] - mean;
        q[v] = x[v] * x[v];
      }
      const float rh = 1.0f / sqrtf(tb_token_sum<V>(q) / (float)D + p.eps);
      float am = 0.0f;
#pragma unroll
      for (int t = 0; t < TO; ++t) {
#pragma unroll
        for (int i = 0; i < 4; ++i) x[4 * t + i] *= rh;
        if (ok) *(float4 *)(xn + tok * D + 16 * t + 4 * g) = make_float4(x[4 * t], x[4 * t + 1], x[4 * t + 2], x[4 * t + 3]);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          x[4 * t + i] = fmaf(x[4 * t + i], vl[kg * D + 16 * t + i], vl[kb * D + 16 * t + i]);
          am = fmaxf(am, fabsf(x[4 * t + i]));
        }
      }
      if (ok && g == 0) rho[tok] = rh;
      return tb_token_max(am);
    };
    // ---- output map, residual, LN1, Eq. 2 ----
#pragma unroll
    for (int o = 0; o < TO; ++o) {
      const v4i acc = mfma_i8_steps<S>([&](int s) { return (long)fo[(o * S + s) * 64 + lane]; }, [&](int s) { return bq[s]; },
                                       v4i{0, 0, 0, 0});
#pragma unroll
      for (int i = 0; i < 4; ++i) x[4 * o + i] += fmaf((float)acc[i], sc, vl[16 * o + i]);
    }
    const float a1 = norm(1, 2, p.xn1, p.rho1);
    long xb[S];
    store_codes<S>(x, inv127(a1), g, ok, p.x1q + tok * D, xb);
    const float t1 = a1 / 127.0f, sc1 = t1 * s1;
    if (ok && g == 0) p.t1[tok] = t1;
    // ---- first feed-forward map: the hidden row in registers, its ReLU mask and maximum ----
    float hid[TH][4], am = 0.0f;
#pragma unroll
    for (int w = 0; w < MW; ++w) {
      uint32_t keep = 0;
#pragma unroll
      for (int o8 = 0; o8 < 8; ++o8) {
        const int o = 8 * w + o8;
        const v4i acc = mfma_i8_steps<S>([&](int s) { return (long)f1l[(o * S + s) * 64]; }, [&](int s) { return xb[s]; },
                                         v4i{0, 0, 0, 0});
        const float4 b = *(const float4 *)(vl + 8 * D + 16 * o);
        const float bb[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          hid[o][i] = fmaf((float)acc[i], sc1, bb[i]);
          keep |= hid[o][i] > 0.0f ? 1u << (4 * o8 + i) : 0u;
          am = fmaxf(am, hid[o][i]);
        }
      }
      if (ok) p.mask[(tok * 4 + g) * MW + w] = keep;
    }
    am = tb_token_max(am + 0.0f);   // +0: a -0 maximum would not order like its bits
    const float invh = inv127(am), tg = am / 127.0f;
    if (ok && g == 0) p.tg[tok] = tg;
    // ---- ReLU and Eq. 2 on the codes, second map ----
    v4i acc2[TO];
#pragma unroll
    for (int o = 0; o < TO; ++o) acc2[o] = v4i{0, 0, 0, 0};
    static_assert(SH % 2 == 0, "k-steps taken in pairs");
#pragma unroll
    for (int st = 0; st < SH; st += 2) {
      long gb[2];
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        uint32_t w[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int o = 2 * (st + j) + h;
          w[h] = relu_codes4(hid[o][0], hid[o][1], hid[o][2], hid[o][3], invh);
          if (ok) *(uint32_t *)(p.gq + tok * 4 * D + 16 * o + 4 * g) = w[h];
        }
        gb[j] = (long)(((uint64_t)w[1] << 32) | w[0]);
      }
#pragma unroll
      for (int o = 0; o < TO; ++o)
        acc2[o] = mfma_i8_16x16x64((long)f2l[(o * SH + st) * 64], (long)f2l[(o * SH + st + 1) * 64], gb[0], gb[1], acc2[o]);
    }
    // ---- residual, LN2, Eq. 2 of the next layer's input ----
    const float sc2 = tg * s2;
#pragma unroll
    for (int o = 0; o < TO; ++o)
#pragma unroll
      for (int i = 0; i < 4; ++i) x[4 * o + i] += fmaf((float)acc2[o][i], sc2, vl[3 * D + 16 * o + i]);
    const float ax = norm(4, 5, p.xn2, p.rho2);
    if (p.x) {
      if (ok)
#pragma unroll
        for (int t = 0; t < TO; ++t)
          *(float4 *)(p.x + tok * D + 16 * t + 4 * g) = make_float4(x[4 * t], x[4 * t + 1], x[4 * t + 2], x[4 * t + 3]);
    } else {
      long nb[S];
      store_codes<S>(x, inv127(ax), g, ok, p.xq + tok * D, nb);
      if (ok && g == 0) p.tx[tok] = ax / 127.0f;
    }
    __builtin_amdgcn_sched_barrier(0);   // strips do not overlap (their registers would not fit)
  }
}

// ------------------------------------------------------------------------------------------
// The token-local half of a layer's backward: LN2, second feed-forward map, ReLU mask, first map, residual,
// LN1, output map, from dX to the gradients of the maps' outputs (dR2, dG, dR1, which the weight
// gradients read) and of O, with both LayerNorms' gain and shift gradients summed on the way.  One
// wavefront per strip, lanes as in k_train_block.  A gradient times a ternary matrix: fp32 splits exactly
// into three bf16 parts whose products are exact (as k_gemm_tern).  The 9 d^2 ternary entries sit in LDS as
// one selector byte each and become bf16 by byte permutes, eight per eight entries, behind the three
// MFMAs they feed; as bf16 they would not fit, and from the L2 their 18 d^2 bytes a strip were what
// k_gemm_tern spent most of its time on.  Separate kernels passed dX1, dR and dG through memory twice
// more and read X-hat twice (LDPC(256,128), 256 words: 385 us a layer; this one 134, its 512 MB of inputs and
// outputs 98 at the copy's rate).
// ------------------------------------------------------------------------------------------
template <int D>
constexpr size_t bwd_lds() { return (size_t)9 * D * D + (size_t)2 * D * 4; }

// selector bytes (0, 1, 2) of ternary entries 0, +1, -1 to bf16: byte k of w selects the high byte 00, 3F,
// BF and the low byte 00, 80, 80
__device__ __forceinline__ bf16x8 sel_bf16(uint64_t w) {
  const uint32_t a = (uint32_t)w, b = (uint32_t)(w >> 32);
  const uint32_t ha = __builtin_amdgcn_perm(0u, 0x00BF3F00u, a), la = __builtin_amdgcn_perm(0u, 0x00808000u, a);
  const uint32_t hb = __builtin_amdgcn_perm(0u, 0x00BF3F00u, b), lb = __builtin_amdgcn_perm(0u, 0x00808000u, b);
  uint4 r;
  r.x = __builtin_amdgcn_perm(ha, la, 0x05010400u);
  r.y = __builtin_amdgcn_perm(ha, la, 0x07030602u);
  r.z = __builtin_amdgcn_perm(hb, lb, 0x05010400u);
  r.w = __builtin_amdgcn_perm(hb, lb, 0x07030602u);
  return __builtin_bit_cast(bf16x8, r);
}

template <int D>
__global__ __launch_bounds__(kTbWaves * 64) void k_train_bwd(TrainBwd p) {
  constexpr int V = D / 4, S = D / 32, TO = D / 16, TH = D / 4, SH = D / 8, MW = D / 32, NC = (V + 15) / 16;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, c = lane & 15, g = lane >> 4;
  uint64_t *f2 = (uint64_t *)smem, *f1 = f2 + (size_t)TH * S * 64, *fo = f1 + (size_t)TO * SH * 64;
  float *lv = (float *)(smem + (size_t)9 * D * D);   // gains of LN2, LN1
  stage16(p.f2, f2, D * D / 4, tid);
  stage16(p.f1, f1, D * D / 4, tid);
  stage16(p.fo, fo, D * D / 16, tid);
  stage_vec(p.g2, lv, D, tid);
  stage_vec(p.g1, lv + D, D, tid);
  __syncthreads();
  const float s2 = *p.s2, s1 = *p.s1, so = *p.so;
  // the lane's fragments from opaque byte offsets: one running address per array, the rest of a read's
  // address in its immediate offset
  uint32_t o2 = (uint32_t)lane * 8u, o1 = (uint32_t)(4 * D * D) + o2, oo = (uint32_t)(8 * D * D) + o2;
  asm volatile("" : "+v"(o2), "+v"(o1), "+v"(oo));
  const uint64_t *f2l = (const uint64_t *)(smem + o2), *f1l = (const uint64_t *)(smem + o1), *fol = (const uint64_t *)(smem + oo);
  // column sums over this wavefront's tokens: lane c of a row of 16 keeps the features v with v mod 16 = c
  float cs[4][NC] = {};
  const int64_t nstrips = (p.rows + 15) / 16, stride = (int64_t)gridDim.x * kTbWaves;
  for (int64_t strip = (int64_t)wave * gridDim.x + blockIdx.x; strip < nstrips; strip += stride) {
    const int64_t tok = strip * 16 + c;
    const bool ok = tok < p.rows;
    const int64_t tl = ok ? tok : p.rows - 1;   // padding columns: a copy, never stored or summed
    // x := the LayerNorm's input gradient from its output gradient x: rho (x g - mean(x g) - xn mean(x g xn));
    // the sums of x xn and x over the strip's tokens to cs[q], cs[q + 1]
    auto norm_bwd = [&](float (&x)[V], const float *xnp, const float *rhop, uint32_t og, int q) {
      asm volatile("" : "+v"(og));   // the gains are read here, not kept from the kernel's start
      const float *gain = (const float *)(smem + og);
      float xn[V], a[V];
#pragma unroll
      for (int t = 0; t < TO; ++t) {
        const float4 f = *(const float4 *)(xnp + tl * D + 16 * t + 4 * g);
        xn[4 * t] = f.x; xn[4 * t + 1] = f.y; xn[4 * t + 2] = f.z; xn[4 * t + 3] = f.w;
      }
      const float rho = rhop[tl];
#pragma unroll
      for (int v = 0; v < V; ++v) {
        const float sa = row16_sum(ok ? x[v] * xn[v] : 0.0f), sb = row16_sum(ok ? x[v] : 0.0f);
        const bool mine = (v & 15) == c;
        cs[q][v >> 4] += mine ? sa : 0.0f;
        cs[q + 1][v >> 4] += mine ? sb : 0.0f;
        asm volatile("" : "+v"(cs[q][v >> 4]), "+v"(cs[q + 1][v >> 4]));   // added now, not kept for later
        x[v] *= gain[16 * (v >> 2) + (v & 3)];
        a[v] = x[v] * xn[v];
        if ((v & 3) == 3) __builtin_amdgcn_sched_barrier(0);
      }
      const float m1 = tb_token_sum<V>(x) / (float)D, m2 = tb_token_sum<V>(a) / (float)D;
#pragma unroll
      for (int v = 0; v < V; ++v) x[v] = rho * (x[v] - m1 - xn[v] * m2);
    };
    auto put = [&](float *dst, const float (&x)[V]) {
      if (ok)
#pragma unroll
        for (int t = 0; t < TO; ++t)
          *(float4 *)(dst + tok * D + 16 * t + 4 * g) = make_float4(x[4 * t], x[4 * t + 1], x[4 * t + 2], x[4 * t + 3]);
    };
    // the three bf16 parts of a row's values as B operands, smallest part last
    auto parts = [&](const float (&x)[V], bf16x8 (&b)[S][3]) {
#pragma unroll
      for (int s = 0; s < S; ++s)
        split_bf16x3<D == 32>(make_float4(x[8 * s], x[8 * s + 1], x[8 * s + 2], x[8 * s + 3]),
                              make_float4(x[8 * s + 4], x[8 * s + 5], x[8 * s + 6], x[8 * s + 7]), b[s][0], b[s][1], b[s][2]);
    };
    auto mac = [&](uint64_t w, const bf16x8 (&b)[3], f32x4 acc) {
      const bf16x8 a = sel_bf16(w);
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b[2], acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b[1], acc, 0, 0, 0);
      return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b[0], acc, 0, 0, 0);
    };
    float x[V];
#pragma unroll
    for (int t = 0; t < TO; ++t) {
      const float4 f = *(const float4 *)(p.dx + tl * D + 16 * t + 4 * g);
      x[4 * t] = f.x; x[4 * t + 1] = f.y; x[4 * t + 2] = f.z; x[4 * t + 3] = f.w;
    }
    norm_bwd(x, p.xn2, p.rho2, (uint32_t)(9 * D * D) + 16u * (uint32_t)g, 0);
    put(p.dr2, x);
    bf16x8 b[S][3];
    parts(x, b);
    f32x4 acc2[TO];
#pragma unroll
    for (int o = 0; o < TO; ++o) acc2[o] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 1
    for (int st = 0; st < SH; ++st) {   // hidden tiles 2 st, 2 st + 1: the hidden gradient, then its share of dX1
      const uint32_t keep = p.mask[(tl * 4 + g) * MW + (st >> 2)] >> (8 * (st & 3));
      float4 h[2];
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        f32x4 acc = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int s = 0; s < S; ++s) acc = mac(f2l[((2 * st + k) * S + s) * 64], b[s], acc);
        __builtin_amdgcn_sched_barrier(0);   // fragments read and expanded further ahead would spill
        h[k] = make_float4((keep >> (4 * k)) & 1u ? s2 * acc[0] : 0.0f, (keep >> (4 * k + 1)) & 1u ? s2 * acc[1] : 0.0f,
                           (keep >> (4 * k + 2)) & 1u ? s2 * acc[2] : 0.0f, (keep >> (4 * k + 3)) & 1u ? s2 * acc[3] : 0.0f);
        if (ok) *(float4 *)(p.dg + tok * 4 * D + 16 * (2 * st + k) + 4 * g) = h[k];
      }
      bf16x8 hb[3];
      split_bf16x3<D == 32>(h[0], h[1], hb[0], hb[1], hb[2]);
#pragma unroll
      for (int o = 0; o < TO; ++o) {
        acc2[o] = mac(f1l[(o * SH + st) * 64], hb, acc2[o]);
        if (o & 1) __builtin_amdgcn_sched_barrier(0);
      }
    }
#pragma unroll
    for (int o = 0; o < TO; ++o)
#pragma unroll
      for (int i = 0; i < 4; ++i) x[4 * o + i] += s1 * acc2[o][i];
    norm_bwd(x, p.xn1, p.rho1, (uint32_t)(9 * D * D + 4 * D) + 16u * (uint32_t)g, 2);
    put(p.dr1, x);
    parts(x, b);
#pragma unroll
    for (int o = 0; o < TO; ++o) {
      f32x4 acc = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int s = 0; s < S; ++s) acc = mac(fol[(o * S + s) * 64], b[s], acc);
      __builtin_amdgcn_sched_barrier(0);
      if (ok) *(float4 *)(p.dO + tok * D + 16 * o + 4 * g) = make_float4(so * acc[0], so * acc[1], so * acc[2], so * acc[3]);
    }
    __builtin_amdgcn_sched_barrier(0);   // strips do not overlap (their registers would not fit)
  }
  // the block's column sums: LN2's gain and shift, LN1's gain and shift
  __syncthreads();
  float (*red)[4 * D] = (float (*)[4 * D])smem;
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int k = 0; k < NC; ++k) {
      const int v = 16 * k + c;
      if (v < V) red[wave][q * D + 16 * (v >> 2) + 4 * g + (v & 3)] = cs[q][k];
    }
  __syncthreads();
  for (int u = tid; u < 4 * D; u += kTbWaves * 64) {
    float s = 0.0f;
#pragma unroll
    for (int w = 0; w < kTbWaves; ++w) s += red[w][u];
    p.lnpart[(int64_t)blockIdx.x * 4 * D + u] = s;
  }
}

// ------------------------------------------------------------------------------------------
// Weight gradients G = Xh^T dY of every map of a layer, Xh = q t per row (codes and scales): the codes
// are exact in bf16 and fp32(t dY) splits exactly into three bf16 parts, so three bf16 MFMAs form fp32
// sums of exact products (as k_gemm_tern), at 16 times the fp32 matrix rate each.  A block takes a
// D x D tile of one map's gradient over a range of rows: per step of 4096 / D rows a thread reads two
// columns of eight rows of either operand and writes them to LDS as MFMA fragments (the contraction
// runs over rows, so a lane needs eight rows of one column), the next step's reads in flight while the
// current one is multiplied.  The bias gradients are the column sums of the dY that pass by.  All four
// products of a layer go out as one launch, their partial sums reduced by one more in a fixed order
// (fp32 MFMAs on fp32 Xh, with a launch, a reduction and a column-sum pass per map: LDPC(256,128),
// 256 words, 480 us a layer; BCH(31,16), 128 words, 160 us).
// ------------------------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(kThreads, 2) void k_train_dw(TrainDwJobs J) {
  constexpr int CP = D / 2, RG = kThreads / CP, RS = 8 * RG, TM = D / 32;
  __shared__ uint4 As[RG][D], Bs[3][RG][D];   // eight rows of a column as bf16
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, fr = lane >> 4, fc = lane & 15;
  const int cp = tid % CP, rg = CP == 64 ? __builtin_amdgcn_readfirstlane(wave) : tid / CP;   // (scalar loads of t)
  // Block to (row range, tile): blocks go to the eight XCDs in turn, and the tiles of a row range read the
  // same rows (dR2 and x1's codes four times each), so they take blocks b, b + 8, ... of one XCD where the
  // ranges are a multiple of eight.
  const int tiles = J.tile0[J.n], b = (int)blockIdx.x, k8 = b >> 3;
  const int split = J.splits % 8 ? b / tiles : k8 / tiles * 8 + (b & 7), bt = J.splits % 8 ? b % tiles : k8 % tiles;
  int ji = 0;
  while (ji + 1 < J.n && bt >= J.tile0[ji + 1]) ++ji;
  const TrainDwJob &j = J.j[ji];
  const int tile = bt - J.tile0[ji], kts = j.K / D, nt = tile / kts, kt = tile - nt * kts;
  const int64_t r0 = (int64_t)split * J.chunk, r1 = std::min<int64_t>(J.rows, r0 + J.chunk);
  const int8_t *qp = j.q + kt * D + 2 * cp;
  const float *yp = j.dy + nt * D + 2 * cp;
  const float *tp = j.t;
  const int64_t K = j.K, ldy = j.ldy;
  uint32_t q[8];
  float2 y[8];
  float t[8];
  auto load = [&](int64_t r) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int64_t row = r + 8 * rg + e;
      const bool ok = row < r1;
      q[e] = ok ? *(const uint16_t *)(qp + row * K) : 0u;
      y[e] = ok ? *(const float2 *)(yp + row * ldy) : make_float2(0.0f, 0.0f);
      t[e] = ok ? tp[row] : 0.0f;
    }
  };
  f32x4 acc[TM][TM];
#pragma unroll
  for (int a = 0; a < TM; ++a)
#pragma unroll
    for (int b = 0; b < TM; ++b) acc[a][b] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  const int wm = (wave >> 1) * (D / 2), wn = (wave & 1) * (D / 2);
  float cs[2] = {0.0f, 0.0f};
  load(r0);
  for (int64_t r = r0; r < r1; r += RS) {
#pragma unroll
    for (int f = 0; f < 2; ++f) {
      float a[8], v[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        a[e] = (float)(int8_t)(q[e] >> (8 * f));
        const float yv = f ? y[e].y : y[e].x;
        cs[f] += yv;
        v[e] = yv * t[e];
      }
      As[rg][2 * cp + f] = __builtin_bit_cast(uint4, bf16_hi8(a));
      bf16x8 ph, pm, pl;
      split_bf16x3<true>(make_float4(v[0], v[1], v[2], v[3]), make_float4(v[4], v[5], v[6], v[7]), ph, pm, pl);
      Bs[0][rg][2 * cp + f] = __builtin_bit_cast(uint4, ph);
      Bs[1][rg][2 * cp + f] = __builtin_bit_cast(uint4, pm);
      Bs[2][rg][2 * cp + f] = __builtin_bit_cast(uint4, pl);
    }
    __syncthreads();
    if (r + RS < r1) load(r + RS);
#pragma unroll
    for (int ks = 0; ks < RS / 32; ++ks) {
      bf16x8 af[TM];
#pragma unroll
      for (int a = 0; a < TM; ++a) af[a] = __builtin_bit_cast(bf16x8, As[4 * ks + fr][wm + 16 * a + fc]);
#pragma unroll
      for (int b = 0; b < TM; ++b) {
#pragma unroll
        for (int pt = 2; pt >= 0; --pt) {   // smallest part first
          const bf16x8 bf = __builtin_bit_cast(bf16x8, Bs[pt][4 * ks + fr][wn + 16 * b + fc]);
#pragma unroll
          for (int a = 0; a < TM; ++a) acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[a], bf, acc[a][b], 0, 0, 0);
        }
      }
    }
    __syncthreads();
  }
  const int64_t slot = (int64_t)split * tiles + bt;
  float *out = J.part + slot * D * D;
#pragma unroll
  for (int a = 0; a < TM; ++a)
#pragma unroll
    for (int b = 0; b < TM; ++b)
#pragma unroll
      for (int v = 0; v < 4; ++v) out[(wm + 16 * a + 4 * fr + v) * D + wn + 16 * b + fc] = acc[a][b][v];
  if (kt == 0) {
    float (*red)[D] = (float (*)[D])As;
    red[rg][2 * cp] = cs[0];
    red[rg][2 * cp + 1] = cs[1];
    __syncthreads();
    if (tid < D) {
      float s = 0.0f;
#pragma unroll
      for (int k = 0; k < RG; ++k) s += red[k][tid];
      J.cpart[slot * D + tid] = s;
    }
  }
}

// The partial sums of k_train_dw added over the row ranges in order: per tile D D / 256 blocks of its
// elements, then one of its column sums; then the LayerNorm sums of k_train_bwd's blocks.
template <int D>
__global__ __launch_bounds__(kThreads) void k_train_dw_reduce(TrainDwJobs J) {
  constexpr int EB = D * D / kThreads;
  const int tile = (int)blockIdx.x / (EB + 1), eb = (int)blockIdx.x - tile * (EB + 1), tid = threadIdx.x;
  if (tile >= J.tile0[J.n]) {   // the LayerNorms' column sums: 16 columns a block, 16 lanes each
    __shared__ float red[16][17];
    const int u = 16 * ((int)blockIdx.x - J.tile0[J.n] * (EB + 1)) + (tid & 15), rl = tid >> 4;
    float s = 0.0f;
    for (int b = rl; b < J.ln_blocks; b += 16) s += J.lnpart[(int64_t)b * 4 * D + u];
    red[rl][tid & 15] = s;
    __syncthreads();
    if (rl == 0) {
#pragma unroll
      for (int k = 1; k < 16; ++k) s += red[k][tid & 15];
      const int q = u / D;
      float *const o = q == 0 ? J.ln[0] : (q == 1 ? J.ln[1] : (q == 2 ? J.ln[2] : J.ln[3]));
      o[u - q * D] = s;
    }
    return;
  }
  int ji = 0;
  while (ji + 1 < J.n && tile >= J.tile0[ji + 1]) ++ji;
  const TrainDwJob &j = J.j[ji];
  const int ti = tile - J.tile0[ji], kts = j.K / D, nt = ti / kts, kt = ti - nt * kts, tiles = J.tile0[J.n];
  const bool col = eb == EB;
  if (col && (kt != 0 || tid >= D)) return;
  const int e = col ? tid : eb * kThreads + tid;
  const float *src = col ? J.cpart + (int64_t)tile * D + e : J.part + (int64_t)tile * D * D + e;
  const int64_t step = (int64_t)tiles * D * (col ? 1 : D);
  float s[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  int z = 0;
  for (; z + 3 < J.splits; z += 4)
#pragma unroll
    for (int u = 0; u < 4; ++u) s[u] += src[(z + u) * step];
  for (; z < J.splits; ++z) s[0] += src[z * step];
  const float v = (s[0] + s[1]) + (s[2] + s[3]);
  const int n = nt * D + (col ? e : e % D), sg = n / j.seg, nc = n - sg * j.seg;
  float *const gw = sg == 0 ? j.gw[0] : (sg == 1 ? j.gw[1] : j.gw[2]);
  float *const gb = sg == 0 ? j.gb[0] : (sg == 1 ? j.gb[1] : j.gb[2]);
  if (col) gb[nc] = v;
  else gw[(int64_t)(kt * D + e / D) * j.seg + nc] = v;
}

// ------------------------------------------------------------------------------------------
// Head-partitioned attention (Section 4.2) of the training step: one thread per (row, head) over
// the row's neighbour list (first ring for heads below h_f, else the second-ring list, which
// holds the union of both rings under CASA); natural-base softmax of q.k / sqrt(d_h) with the
// maximum subtracted.  Forward stores O and the row's log-sum-exp; the backward recomputes
// p_ij = exp(s_ij - lse_i).  The running maximum starts at the lowest finite value: started at -Inf, a first
// key (of a row, or of one of the lanes that share it) whose score is -Inf would give exp(-Inf + Inf) = NaN where its
// weight is 0.  The masks are symmetric, so the key and value gradients are gathered per key row over its
// own list, without atomics.
// ------------------------------------------------------------------------------------------
using AttnT = TrainAttn;

// Thread gid to (row, head): the first-ring heads of every row first (row-major, a row's h_f heads
// on adjacent lanes), then the second-ring heads, so that a wavefront walks one kind of list and
// its lanes run loops of similar length (with both kinds in one wavefront the first-ring lanes idled
// through the longer second-ring lists), while a row's heads of one kind still read adjacent
// stretches of each neighbour's row.
__device__ __forceinline__ void attn_row_head(const AttnT &p, int64_t gid, int64_t &row, int &h) {
  const int64_t n1 = p.rows * p.hf;
  if (gid < n1) {
    row = gid / p.hf;
    h = (int)(gid - row * p.hf);
  } else {
    const int hs = p.heads - p.hf;
    const int64_t g2 = gid - n1;
    row = g2 / hs;
    h = p.hf + (int)(g2 - row * hs);
  }
}

template <int DH>
__device__ __forceinline__ float dot_dh(const float *a, const float *b) {
  float s = a[0] * b[0];
#pragma unroll
  for (int t = 1; t < DH; ++t) s = fmaf(a[t], b[t], s);
  return s;
}

template <int DH>
__global__ __launch_bounds__(kThreads) void k_attn_fwd(AttnT p) {
  const int64_t gid = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (gid >= p.rows * p.heads) return;
  int64_t row;
  int h;
  attn_row_head(p, gid, row, h);
  const int64_t base = (row / p.L) * p.L;
  const int i = (int)(row - base);
  const int32_t *ptr = h < p.hf ? p.m1_ptr : p.m2_ptr, *idx = h < p.hf ? p.m1_idx : p.m2_idx;
  const int d = p.d, ld = 3 * d;
  const float kappa = 1.0f / sqrtf((float)DH);
  float q[DH];
#pragma unroll
  for (int t = 0; t < DH; ++t) q[t] = p.qkv[row * ld + h * DH + t];
  // one pass with a running maximum: when a score raises it, the sum and the accumulated values so
  // far are rescaled by exp(old - new) (each key read once instead of once for the maximum and once
  // for the weights)
  float mu = -FLT_MAX, S = 0.0f, acc[DH] = {};
  for (int e = ptr[i]; e < ptr[i + 1]; ++e) {
    const int64_t j = base + idx[e];
    const float s = dot_dh<DH>(q, p.qkv + j * ld + d + h * DH) * kappa;
    if (s > mu) {
      const float c = expf(mu - s);   // 0 at the first key
      S *= c;
#pragma unroll
      for (int t = 0; t < DH; ++t) acc[t] *= c;
      mu = s;
    }
    const float pe = expf(s - mu);
    S += pe;
#pragma unroll
    for (int t = 0; t < DH; ++t) acc[t] = fmaf(pe, p.qkv[j * ld + 2 * d + h * DH + t], acc[t]);
  }
#pragma unroll
  for (int t = 0; t < DH; ++t) p.o[row * d + h * DH + t] = acc[t] / S;
  p.lse[row * p.heads + h] = mu + logf(S);
}

template <int DH>
__global__ __launch_bounds__(kThreads) void k_attn_bwd_q(AttnT p) {
  const int64_t gid = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (gid >= p.rows * p.heads) return;
  int64_t row;
  int h;
  attn_row_head(p, gid, row, h);
  const int64_t base = (row / p.L) * p.L;
  const int i = (int)(row - base);
  const int32_t *ptr = h < p.hf ? p.m1_ptr : p.m2_ptr, *idx = h < p.hf ? p.m1_idx : p.m2_idx;
  const int d = p.d, ld = 3 * d;
  const float kappa = 1.0f / sqrtf((float)DH);
  float q[DH], go[DH], dq[DH] = {};
#pragma unroll
  for (int t = 0; t < DH; ++t) {
    q[t] = p.qkv[row * ld + h * DH + t];
    go[t] = p.dout[row * d + h * DH + t];
  }
  const float D = dot_dh<DH>(go, p.o + row * d + h * DH);
  const float lse = p.lse[row * p.heads + h];
  for (int e = ptr[i]; e < ptr[i + 1]; ++e) {
    const int64_t j = base + idx[e];
    const float *kj = p.qkv + j * ld + d + h * DH;
    const float pij = expf(dot_dh<DH>(q, kj) * kappa - lse);
    const float ds = pij * (dot_dh<DH>(go, p.qkv + j * ld + 2 * d + h * DH) - D) * kappa;
#pragma unroll
    for (int t = 0; t < DH; ++t) dq[t] = fmaf(ds, kj[t], dq[t]);
  }
#pragma unroll
  for (int t = 0; t < DH; ++t) p.dqkv[row * ld + h * DH + t] = dq[t];
  p.Dv[row * p.heads + h] = D;
}

template <int DH>
__global__ __launch_bounds__(kThreads) void k_attn_bwd_kv(AttnT p) {
  const int64_t gid = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (gid >= p.rows * p.heads) return;
  int64_t row;   // the key / value row j
  int h;
  attn_row_head(p, gid, row, h);
  const int64_t base = (row / p.L) * p.L;
  const int j = (int)(row - base);
  const int32_t *ptr = h < p.hf ? p.m1_ptr : p.m2_ptr, *idx = h < p.hf ? p.m1_idx : p.m2_idx;
  const int d = p.d, ld = 3 * d;
  const float kappa = 1.0f / sqrtf((float)DH);
  float k[DH], v[DH], dk[DH] = {}, dv[DH] = {};
#pragma unroll
  for (int t = 0; t < DH; ++t) {
    k[t] = p.qkv[row * ld + d + h * DH + t];
    v[t] = p.qkv[row * ld + 2 * d + h * DH + t];
  }
  for (int e = ptr[j]; e < ptr[j + 1]; ++e) {    // rows i whose list holds j (symmetric masks)
    const int64_t i = base + idx[e];
    const float *qi = p.qkv + i * ld + h * DH;
    const float *gi = p.dout + i * d + h * DH;
    const float pij = expf(dot_dh<DH>(qi, k) * kappa - p.lse[i * p.heads + h]);
    const float ds = pij * (dot_dh<DH>(gi, v) - p.Dv[i * p.heads + h]) * kappa;
#pragma unroll
    for (int t = 0; t < DH; ++t) {
      dv[t] = fmaf(pij, gi[t], dv[t]);
      dk[t] = fmaf(ds, qi[t], dk[t]);
    }
  }
#pragma unroll
  for (int t = 0; t < DH; ++t) {
    p.dqkv[row * ld + d + h * DH + t] = dk[t];
    p.dqkv[row * ld + 2 * d + h * DH + t] = dv[t];
  }
}

// ------------------------------------------------------------------------------------------
// The same attention with what a row gathers in LDS: one block per word and 16-dimension head group
// (16 / d_h heads), a lane or several per (row, head) of it.  The keys and values of the group (for the key and value
// gradients: the queries and output gradients) sit in 144-byte rows, 16 different 16-byte bank groups
// apart.  A pair costs its 128 bytes of LDS reads and about 50 multiply-adds instead of two gathers from
// the L2 in a chain (training steps: LDPC(256,128), 256 words 12.20 -> 11.26 ms, with the blocks of a word
// on one XCD 10.55 ms; BCH(31,16), 128 words 0.81 -> 0.66 ms); what binds is the one read of Q | K | V, O
// and dO and the one write of the results, in 64-byte pieces.
// ------------------------------------------------------------------------------------------
constexpr int kAlRow = 36;   // floats per LDS row: two 16-float halves and padding

template <int DH>
constexpr size_t attn_lds_bytes(int L) { return (size_t)L * (kAlRow * 4 + 8 * (16 / DH)); }

// rows 0 .. L - 1 of two 16-float column slices (rows la and lb floats apart) side by side into LDS
__device__ __forceinline__ void attn_stage(const float *a, int64_t la, const float *b, int64_t lb, int L, float *dst) {
  for (int u = threadIdx.x; u < L * 8; u += blockDim.x) {
    const int r = u >> 3, c = (u & 3) * 4;
    *(float4 *)(dst + r * kAlRow + ((u & 4) ? 16 : 0) + c) = *(const float4 *)(((u & 4) ? b + r * lb : a + r * la) + c);
  }
}
template <int DH>
__device__ __forceinline__ void attn_vec(float (&x)[DH], const float *p) {
#pragma unroll
  for (int t = 0; t < DH; t += 4) {
    const float4 f = *(const float4 *)(p + t);
    x[t] = f.x; x[t + 1] = f.y; x[t + 2] = f.z; x[t + 3] = f.w;
  }
}
template <int DH>
__device__ __forceinline__ void attn_put(float *p, const float (&x)[DH]) {
#pragma unroll
  for (int t = 0; t < DH; t += 4) *(float4 *)(p + t) = make_float4(x[t], x[t + 1], x[t + 2], x[t + 3]);
}

// Block b's word and head group: blocks go to the eight XCDs in turn, each with an L2 of its own, so the
// groups of a word (64-byte pieces of the same rows) take blocks b, b + 8, b + 16, ... of one XCD.
__device__ __forceinline__ void attn_word_group(const AttnT &p, int G, int64_t &w, int &hg) {
  const int64_t b = blockIdx.x, words = p.rows / p.L, full = words / 8 * 8;
  if (b < full * G) {
    const int64_t k = b >> 3;
    w = k / G * 8 + (b & 7);
    hg = (int)(k % G);
  } else {
    w = b / G;
    hg = (int)(b % G);
  }
}

// Lanes per row: a row of a short code is a chain of up to 28 dependent steps on a block of three
// wavefronts, so its list goes round robin over four adjacent lanes at d_h = 4 and two at d_h = 8 (the
// pieces' sums combined at the end); with 16-dimension heads the rows alone fill the block.  Steps:
// BCH(31,16), 128 words 0.49 -> 0.42 ms, LDPC(128,64), 125 words 0.91 -> 0.88.
template <int DH>
constexpr int attn_split() { return 16 / DH; }
// v of the row's next lane (o = 1) or of its other pair (o = 2)
template <int O>
__device__ __forceinline__ float quad_other(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), O == 1 ? 0xB1 : 0x4E, 0xf, 0xf, true));
}
template <int SP>
__device__ __forceinline__ float row_lanes_sum(float v) {
  if constexpr (SP >= 2) v += quad_other<1>(v);
  if constexpr (SP >= 4) v += quad_other<2>(v);
  return v;
}
template <int SP>
__device__ __forceinline__ float row_lanes_max(float v) {
  if constexpr (SP >= 2) v = fmaxf(v, quad_other<1>(v));
  if constexpr (SP >= 4) v = fmaxf(v, quad_other<2>(v));
  return v;
}

template <int DH>
__global__ __launch_bounds__(1024) void k_attn_fwd_lds(AttnT p) {
  constexpr int HPG = 16 / DH, SP = attn_split<DH>();
  extern __shared__ __attribute__((aligned(16))) float sm_[];
  const int d = p.d, G = d / 16, ld = 3 * d, L = p.L;
  int64_t w;
  int hg;
  attn_word_group(p, G, w, hg);
  const float *base = p.qkv + w * L * ld + 16 * hg;
  attn_stage(base + d, ld, base + 2 * d, ld, L, sm_);
  __syncthreads();
  const float kappa = 1.0f / sqrtf((float)DH);
  const int part = threadIdx.x % SP;
  for (int r = threadIdx.x / SP; r < L * HPG; r += blockDim.x / SP) {
    const int hh = r / L, i = r - hh * L, h = hg * HPG + hh;
    const int32_t *ptr = h < p.hf ? p.m1_ptr : p.m2_ptr, *idx = h < p.hf ? p.m1_idx : p.m2_idx;
    const float *kb = sm_ + hh * DH;
    float q[DH], k[DH], v[DH];
    attn_vec<DH>(q, base + (int64_t)i * ld + hh * DH);
    const int beg = ptr[i] + part, end = ptr[i + 1];
    float mu = -FLT_MAX, S = 0.0f, acc[DH] = {};
    int j = beg < end ? idx[beg] : 0;
    for (int e = beg; e < end; e += SP) {
      const int jn = e + SP < end ? idx[e + SP] : 0;
      attn_vec<DH>(k, kb + j * kAlRow);
      attn_vec<DH>(v, kb + j * kAlRow + 16);
      const float s = dot_dh<DH>(q, k) * kappa;
      if (s > mu) {
        const float c = expf(mu - s);   // 0 at the first key
        S *= c;
#pragma unroll
        for (int t = 0; t < DH; ++t) acc[t] *= c;
        mu = s;
      }
      const float pe = expf(s - mu);
      S += pe;
#pragma unroll
      for (int t = 0; t < DH; ++t) acc[t] = fmaf(pe, v[t], acc[t]);
      j = jn;
    }
    if constexpr (SP > 1) {   // the row's pieces on its largest score (a list is never empty)
      const float top = row_lanes_max<SP>(mu), c = expf(mu - top);   // 0 in a lane without an entry
      mu = top;
      S = row_lanes_sum<SP>(S * c);
#pragma unroll
      for (int t = 0; t < DH; ++t) acc[t] = row_lanes_sum<SP>(acc[t] * c);
    }
    if (part == 0) {
#pragma unroll
      for (int t = 0; t < DH; ++t) acc[t] /= S;
      attn_put<DH>(p.o + (w * L + i) * d + h * DH, acc);
      p.lse[(w * L + i) * p.heads + h] = mu + logf(S);
    }
  }
}

template <int DH>
__global__ __launch_bounds__(1024) void k_attn_bwd_lds(AttnT p) {
  constexpr int HPG = 16 / DH, SP = attn_split<DH>();
  extern __shared__ __attribute__((aligned(16))) float sm_[];
  const int d = p.d, G = d / 16, ld = 3 * d, L = p.L;
  float *ls = sm_ + (size_t)L * kAlRow, *Ds = ls + L * HPG;   // [HPG][L] log-sum-exp, dO . O
  int64_t w;
  int hg;
  attn_word_group(p, G, w, hg);
  const float *base = p.qkv + w * L * ld + 16 * hg, *dob = p.dout + w * L * d + 16 * hg, *ob = p.o + w * L * d + 16 * hg;
  float *gb = p.dqkv + w * L * ld + 16 * hg;
  const float kappa = 1.0f / sqrtf((float)DH);
  const int part = threadIdx.x % SP;
  // query gradients: each row over its keys and values
  attn_stage(base + d, ld, base + 2 * d, ld, L, sm_);
  __syncthreads();
  for (int r = threadIdx.x / SP; r < L * HPG; r += blockDim.x / SP) {
    const int hh = r / L, i = r - hh * L, h = hg * HPG + hh;
    const int32_t *ptr = h < p.hf ? p.m1_ptr : p.m2_ptr, *idx = h < p.hf ? p.m1_idx : p.m2_idx;
    const float *kb = sm_ + hh * DH;
    float q[DH], go[DH], k[DH], v[DH], dq[DH] = {};
    attn_vec<DH>(q, base + (int64_t)i * ld + hh * DH);
    attn_vec<DH>(go, dob + (int64_t)i * d + hh * DH);
    attn_vec<DH>(v, ob + (int64_t)i * d + hh * DH);
    const float D = dot_dh<DH>(go, v), lse = p.lse[(w * L + i) * p.heads + h];
    if (part == 0) {
      ls[hh * L + i] = lse;
      Ds[hh * L + i] = D;
    }
    const int beg = ptr[i] + part, end = ptr[i + 1];
    int j = beg < end ? idx[beg] : 0;
    for (int e = beg; e < end; e += SP) {
      const int jn = e + SP < end ? idx[e + SP] : 0;
      attn_vec<DH>(k, kb + j * kAlRow);
      attn_vec<DH>(v, kb + j * kAlRow + 16);
      const float pij = expf(dot_dh<DH>(q, k) * kappa - lse);
      const float ds = pij * (dot_dh<DH>(go, v) - D) * kappa;
#pragma unroll
      for (int t = 0; t < DH; ++t) dq[t] = fmaf(ds, k[t], dq[t]);
      j = jn;
    }
#pragma unroll
    for (int t = 0; t < DH; ++t) dq[t] = row_lanes_sum<SP>(dq[t]);
    if (part == 0) attn_put<DH>(gb + (int64_t)i * ld + hh * DH, dq);
  }
  __syncthreads();
  // key and value gradients: each key row over the rows whose list holds it (symmetric masks)
  attn_stage(base, ld, dob, d, L, sm_);
  __syncthreads();
  for (int r = threadIdx.x / SP; r < L * HPG; r += blockDim.x / SP) {
    const int hh = r / L, j = r - hh * L, h = hg * HPG + hh;
    const int32_t *ptr = h < p.hf ? p.m1_ptr : p.m2_ptr, *idx = h < p.hf ? p.m1_idx : p.m2_idx;
    const float *qb = sm_ + hh * DH;
    float k[DH], v[DH], q[DH], go[DH], dk[DH] = {}, dv[DH] = {};
    attn_vec<DH>(k, base + (int64_t)j * ld + d + hh * DH);
    attn_vec<DH>(v, base + (int64_t)j * ld + 2 * d + hh * DH);
    const int beg = ptr[j] + part, end = ptr[j + 1];
    int i = beg < end ? idx[beg] : 0;
    for (int e = beg; e < end; e += SP) {
      const int in = e + SP < end ? idx[e + SP] : 0;
      attn_vec<DH>(q, qb + i * kAlRow);
      attn_vec<DH>(go, qb + i * kAlRow + 16);
      const float pij = expf(dot_dh<DH>(q, k) * kappa - ls[hh * L + i]);
      const float ds = pij * (dot_dh<DH>(go, v) - Ds[hh * L + i]) * kappa;
#pragma unroll
      for (int t = 0; t < DH; ++t) {
        dv[t] = fmaf(pij, go[t], dv[t]);
        dk[t] = fmaf(ds, q[t], dk[t]);
      }
      i = in;
    }
#pragma unroll
    for (int t = 0; t < DH; ++t) {
      dk[t] = row_lanes_sum<SP>(dk[t]);
      dv[t] = row_lanes_sum<SP>(dv[t]);
    }
    if (part == 0) {
      attn_put<DH>(gb + (int64_t)j * ld + d + hh * DH, dk);
      attn_put<DH>(gb + (int64_t)j * ld + 2 * d + hh * DH, dv);
    }
  }
}

// ------------------------------------------------------------------------------------------
// Column sums over rows (the head's), deterministic in two passes: A[r][c] (x w[r]) summed over r for each
// of A's C columns.  A block covers cw columns (a power of two up to 64) with 256 / cw row lanes; lane l
// of a block sums the rows l, l + lanes, ... of its chunk (four interleaved partial sums), the lanes are
// combined by a fixed tree in LDS.  Pass one writes a partial row per chunk, pass two sums the partial
// rows with the same kernel.
// ------------------------------------------------------------------------------------------
template <bool HW>
__global__ __launch_bounds__(kThreads) void k_colsum(const float *A, int64_t lda, const float *w, int64_t rows, int C,
                                                     int cw_log2, int64_t chunk, float *out, int64_t ldo) {
  __shared__ float red[kThreads];
  const int cw = 1 << cw_log2, lanes = kThreads >> cw_log2;
  const int cl = threadIdx.x & (cw - 1), rl = threadIdx.x >> cw_log2;
  const int c = blockIdx.x * cw + cl;
  const int64_t r0 = (int64_t)blockIdx.y * chunk, r1 = std::min<int64_t>(rows, r0 + chunk);
  float s[4] = {};
  auto add = [&](int k, int64_t r) { s[k] += HW ? A[r * lda + c] * w[r] : A[r * lda + c]; };
  if (c < C) {
    int64_t r = r0 + rl;
    for (; r + 3 * lanes < r1; r += 4 * lanes) {
      add(0, r);
      add(1, r + lanes);
      add(2, r + 2 * lanes);
      add(3, r + 3 * lanes);
    }
    for (; r < r1; r += lanes) add(0, r);
  }
  red[threadIdx.x] = (s[0] + s[1]) + (s[2] + s[3]);
  __syncthreads();
  for (int st = lanes >> 1; st > 0; st >>= 1) {
    if (rl < st) red[threadIdx.x] += red[threadIdx.x + (st << cw_log2)];
    __syncthreads();
  }
  if (rl == 0 && c < C) out[(int64_t)blockIdx.y * ldo + c] = red[threadIdx.x];
}

// ------------------------------------------------------------------------------------------
// Small elementwise steps.
// ------------------------------------------------------------------------------------------
// z = X w1 + b1 per row (Section 3 head, W_{d->1}); one wavefront per row
__global__ __launch_bounds__(kThreads) void k_rowdot(const float *x, int64_t rows, int d, const float *w1,
                                                     const float *b1, float *z) {
  const int64_t r = (int64_t)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (r >= rows) return;
  float s = 0.0f;
  for (int c = lane; c < d; c += 64) s = fmaf(x[r * d + c], w1[c], s);
  s = wave_sum(s);
  if (lane == 0) z[r] = s + b1[0];
}

// dX = dz w1^T (the head's W_{d->1} backward)
__global__ __launch_bounds__(kThreads) void k_outer(const float *dz, int64_t rows, const float *w1, int d, float *dx) {
  const int64_t e = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (e >= rows * d) return;
  dx[e] = dz[e / d] * w1[e % d];
}

// Loss of the multiplicative noise (Section 6): target z = [y x_s < 0] (x_s = +1 if xs is null),
// l = softplus(-f) + z f = BCE-with-logits(-f, z); df = (z - sigmoid(-f)) / count.  Per-block
// sums of l in part[blockIdx].
__global__ __launch_bounds__(kThreads) void k_loss(const float *f, const float *y, const float *xs, int64_t count,
                                                   float inv_count, float *df, float *part) {
  __shared__ float red[kThreads / 64];
  const int64_t e = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  float l = 0.0f;
  if (e < count) {
    const float fv = f[e];
    const float sg = xs ? xs[e] : 1.0f;
    const float z = y[e] * sg < 0.0f ? 1.0f : 0.0f;
    const float nf = -fv;
    l = fmaxf(nf, 0.0f) + log1pf(expf(-fabsf(nf))) + z * fv;
    const float sig = 1.0f / (1.0f + expf(fv));          // sigmoid(-f)
    df[e] = (z - sig) * inv_count;
  }
  l = wave_sum(l);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = l;
  __syncthreads();
  if (threadIdx.x == 0) {
    float s = 0.0f;
    for (int k = 0; k < kThreads / 64; ++k) s += red[k];
    part[blockIdx.x] = s;
  }
}

__global__ __launch_bounds__(64) void k_loss_final(const float *part, int n, float inv_count, float *loss) {
  if (threadIdx.x != 0) return;
  float s = 0.0f;
  for (int k = 0; k < n; ++k) s += part[k];
  *loss = s * inv_count;
}

// dE[i][c] = sum_b t[b L + i] dX[b L + i][c] (the embedding is t_i E_i): a block takes 32 columns of a token,
// eight lanes over the words per column, added in lane order (one lane per element walked the words
// alone: 104 us at 256 words of LDPC(256,128), 35 us at 128 of BCH(31,16)).
__global__ __launch_bounds__(kThreads) void k_embed_grad(const float *t, const float *dx, int64_t words, int L, int d,
                                                         float *de) {
  __shared__ float red[kThreads / 32][32];
  const int cl = threadIdx.x & 31, bl = threadIdx.x >> 5, c = blockIdx.y * 32 + cl;   // d a multiple of 32
  const int64_t i = blockIdx.x;
  constexpr int kLanes = kThreads / 32;
  float s[4] = {};
  int64_t b = bl;
  for (; b + 3 * kLanes < words; b += 4 * kLanes)
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t r = (b + u * kLanes) * L + i;
      s[u] = fmaf(t[r], dx[r * d + c], s[u]);
    }
  for (; b < words; b += kLanes) s[0] = fmaf(t[b * L + i], dx[(b * L + i) * d + c], s[0]);
  red[bl][cl] = (s[0] + s[1]) + (s[2] + s[3]);
  __syncthreads();
  if (bl == 0) {
    float v = red[0][cl];
#pragma unroll
    for (int k = 1; k < kLanes; ++k) v += red[k][cl];
    de[i * d + c] = v;
  }
}

// The straight-through Eq. 1 gradients of one matrix, one block per matrix: G = Xh^T dY arrives in
// dW; dW = G s / (s + eps) and d delta = gamma sum(G T) - s gamma / (s + eps)^2 sum(G W).
using DeltaJob = TrainDeltaJob;

__global__ __launch_bounds__(kAapThreads) void k_delta_grad(TrainDeltaJobs jobs, float eps) {
  __shared__ float r1[kAapWaves], r2[kAapWaves];
  const DeltaJob J = jobs.j[blockIdx.x];
  const float s = *J.scale, gamma = *J.gamma;
  const float fac = s / (s + eps);
  float a[2] = {0.0f, 0.0f}, b[2] = {0.0f, 0.0f};
  int64_t e = threadIdx.x;
  for (; e + kAapThreads < J.count; e += 2 * kAapThreads) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int64_t x = e + u * kAapThreads;
      const float gv = J.dw[x];
      a[u] = fmaf(gv, J.t[x], a[u]);
      b[u] = fmaf(gv, J.w[x], b[u]);
      J.dw[x] = gv * fac;
    }
  }
  if (e < J.count) {
    const float gv = J.dw[e];
    a[0] = fmaf(gv, J.t[e], a[0]);
    b[0] = fmaf(gv, J.w[e], b[0]);
    J.dw[e] = gv * fac;
  }
  const float sa_ = wave_sum(a[0] + a[1]), sb_ = wave_sum(b[0] + b[1]);
  if ((threadIdx.x & 63) == 0) {
    r1[threadIdx.x >> 6] = sa_;
    r2[threadIdx.x >> 6] = sb_;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    float sa = 0.0f, sb = 0.0f;
    for (int k = 0; k < kAapWaves; ++k) {
      sa += r1[k];
      sb += r2[k];
    }
    const float den = s + eps;
    *J.ddelta = gamma * sa - s * gamma / (den * den) * sb;
  }
}

}  // namespace train

// ------------------------------------------------------------------------------------------
// launch helpers (declared in aecct_internal.h)
// ------------------------------------------------------------------------------------------
namespace {
inline unsigned blocks_for(int64_t n, int per) { return (unsigned)((n + per - 1) / per); }
}

hipError_t train_aap(const TrainAapJobs &jobs, float eps, hipStream_t s) {
  if (jobs.n <= 0) return hipSuccess;
  int64_t most = 0;
  for (int k = 0; k < jobs.n; ++k) {
    if (jobs.j[k].count <= 0 || jobs.j[k].count % train::kAapThreads) return hipErrorInvalidValue;
    most = std::max(most, jobs.j[k].count / train::kAapThreads);
  }
  const dim3 grid((unsigned)jobs.n), block(train::kAapThreads);
  if (most <= 4) hipLaunchKernelGGL(train::k_aap<4>, grid, block, 0, s, jobs, eps);
  else if (most <= 16) hipLaunchKernelGGL(train::k_aap<16>, grid, block, 0, s, jobs, eps);
  else if (most <= 64) hipLaunchKernelGGL(train::k_aap<64>, grid, block, 0, s, jobs, eps);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t train_delta_grad(const TrainDeltaJobs &jobs, float eps, hipStream_t s) {
  if (jobs.n <= 0) return hipSuccess;
  hipLaunchKernelGGL(train::k_delta_grad, dim3((unsigned)jobs.n), dim3(train::kAapThreads), 0, s, jobs, eps);
  return hipGetLastError();
}

hipError_t train_embed(const float *y, int64_t rows, int n, int L, int d, const int32_t *chk_ptr,
                       const int32_t *chk_idx, const float *E, const float *P, float *x, float *t, int8_t *xq, float *tx,
                       hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  if (d > 128) return hipErrorInvalidValue;
  hipLaunchKernelGGL(train::k_embed, dim3(blocks_for(rows, 4)), dim3(train::kThreads), 0, s, y, rows, n, L, d, chk_ptr,
                     chk_idx, E, P, x, t, xq, tx);
  return hipGetLastError();
}

hipError_t train_gemm(bool ta, bool tb, const float *A, int64_t lda, const float *B, int64_t ldb, float *C, int64_t ldc,
                      int64_t M, int64_t N, int64_t K, const float *bias, float *part, int64_t part_floats, int cu_count,
                      hipStream_t s) {
  if (M <= 0 || N <= 0) return hipSuccess;
  if (ta && tb) return hipErrorInvalidValue;
  train::GemmF32 g{A, B, C, M, N, K, lda, ldb, ldc, K, bias, part};
  // the MFMA kernel reads 16-byte vectors along each operand's contiguous dimension
  auto al16 = [](const float *p) { return ((uintptr_t)p & 15u) == 0; };
  const bool mfma = al16(A) && al16(B) && lda % 4 == 0 && ldb % 4 == 0 && (ta ? M : K) % 4 == 0 &&
                    (tb ? K : N) % 4 == 0;
  const int64_t tm = 64, tn = mfma ? train::kMfTile : 64;
  static_assert(train::kMfRows == 64, "rows of a block of either kernel");
  const int64_t tiles = ((M + tm - 1) / tm) * ((N + tn - 1) / tn);
  // split long reductions over k so that about two blocks per compute unit are busy (k chunks of at
  // least 128)
  int64_t splits = std::max<int64_t>(1, std::min<int64_t>((2 * (int64_t)cu_count + tiles - 1) / tiles, (K + 127) / 128));
  splits = std::min<int64_t>(splits, part_floats / (M * N));
  if (splits < 1) splits = 1;
  const int64_t kq = mfma ? train::kMfK : train::kVgK;
  g.kchunk = (((K + splits - 1) / splits) + kq - 1) / kq * kq;
  if (g.kchunk < kq) g.kchunk = kq;
  splits = (K + g.kchunk - 1) / g.kchunk;
  if (splits < 1) splits = 1;
  const dim3 grid((unsigned)((N + tn - 1) / tn), (unsigned)((M + tm - 1) / tm), (unsigned)splits);
  if (mfma) {
    if (ta) hipLaunchKernelGGL((train::k_gemm_mfma<true, false>), grid, dim3(train::kThreads), 0, s, g);
    else if (tb) hipLaunchKernelGGL((train::k_gemm_mfma<false, true>), grid, dim3(train::kThreads), 0, s, g);
    else hipLaunchKernelGGL((train::k_gemm_mfma<false, false>), grid, dim3(train::kThreads), 0, s, g);
  } else if (ta) {
    hipLaunchKernelGGL((train::k_gemm<true, false>), grid, dim3(train::kThreads), 0, s, g);
  } else if (tb) {
    hipLaunchKernelGGL((train::k_gemm<false, true>), grid, dim3(train::kThreads), 0, s, g);
  } else {
    hipLaunchKernelGGL((train::k_gemm<false, false>), grid, dim3(train::kThreads), 0, s, g);
  }
  if (splits > 1)
    hipLaunchKernelGGL(train::k_gemm_reduce, dim3(blocks_for(M * N, 64)), dim3(train::kThreads), 0, s, g,
                       (int)splits);
  return hipGetLastError();
}

hipError_t train_pack_tern(const TernPackJobs &jobs, hipStream_t s) {
  if (jobs.n <= 0) return hipSuccess;
  int64_t lanes = 0;
  for (int i = 0; i < jobs.n; ++i) {
    if (jobs.j[i].R % 32 || jobs.j[i].C % 32) return hipErrorInvalidValue;
    lanes = std::max<int64_t>(lanes, (int64_t)jobs.j[i].R * jobs.j[i].C / 8);   // one lane per 8 entries
  }
  hipLaunchKernelGGL(train::k_pack_tern, dim3(blocks_for(lanes, train::kThreads), (unsigned)jobs.n), dim3(train::kThreads), 0,
                     s, jobs);
  return hipGetLastError();
}

hipError_t train_gemm_tern(const float *A, int64_t lda, const void *const *frag, int nseg, int64_t kseg,
                           const float *const *scale, const float *D, float *C, int64_t ldc, int64_t M, int64_t N,
                           hipStream_t s) {
  if (M <= 0 || N <= 0) return hipSuccess;
  const auto al16 = [](const void *q) { return ((uintptr_t)q & 15u) == 0; };   // 16-byte rows of A, C, D
  if (nseg < 1 || nseg > 3 || kseg <= 0 || kseg % 32 || N % 32 || lda % 4 || ldc % 4 || !al16(A) || !al16(C) || !al16(D))
    return hipErrorInvalidValue;
  train::GemmTern g{A, {}, C, D, M, N, kseg * nseg, lda, ldc, {}, (int)(kseg / 32)};
  for (int k = 0; k < nseg; ++k) {
    g.B[k] = (const uint4 *)frag[k];
    g.scale[k] = scale[k];
  }
  constexpr int S = 3;   // operands two k-steps ahead
  const unsigned gy = (unsigned)((g.M + 63) / 64);
  if (N % 128 == 0)
    hipLaunchKernelGGL((train::k_gemm_tern<8, S>), dim3((unsigned)(N / 128), gy), dim3(train::kThreads), 0, s, g);
  else if (N % 64 == 0)
    hipLaunchKernelGGL((train::k_gemm_tern<4, S>), dim3((unsigned)(N / 64), gy), dim3(train::kThreads), 0, s, g);
  else
    hipLaunchKernelGGL((train::k_gemm_tern<2, S>), dim3((unsigned)(N / 32), gy), dim3(train::kThreads), 0, s, g);
  return hipGetLastError();
}

namespace {
template <int D>
hipError_t qkv_go(const TrainQkv &a, int cu_count, size_t lds_max, hipStream_t s) {
  constexpr size_t lds = train::qkv_lds<D>();
  const int64_t strips = (a.rows + 15) / 16, groups = std::max<int64_t>((strips + train::kTbWaves - 1) / train::kTbWaves, std::min<int64_t>(strips, cu_count));
  const int64_t per_cu = std::max<int64_t>(1, std::min<int64_t>(2, (int64_t)(lds_max / lds)));
  hipLaunchKernelGGL(train::k_train_qkv<D>, dim3((unsigned)std::min<int64_t>(groups, cu_count * per_cu)),
                     dim3(train::kTbWaves * 64), lds, s, a);
  return hipGetLastError();
}
template <int D>
hipError_t block_go(const TrainBlock &a, int cu_count, size_t lds_max, hipStream_t s) {
  constexpr size_t lds = train::block_lds<D>();
  const int64_t strips = (a.rows + 15) / 16, groups = std::max<int64_t>((strips + train::kTbWaves - 1) / train::kTbWaves, std::min<int64_t>(strips, cu_count));
  const int64_t per_cu = std::max<int64_t>(1, std::min<int64_t>(2, (int64_t)(lds_max / lds)));
  hipLaunchKernelGGL(train::k_train_block<D>, dim3((unsigned)std::min<int64_t>(groups, cu_count * per_cu)),
                     dim3(train::kTbWaves * 64), lds, s, a);
  return hipGetLastError();
}
}  // namespace

hipError_t train_set_attributes(size_t lds_max) {
  const void *fns[] = {(const void *)train::k_train_qkv<32>,   (const void *)train::k_train_qkv<64>,
                       (const void *)train::k_train_qkv<128>,  (const void *)train::k_train_block<32>,
                       (const void *)train::k_train_block<64>, (const void *)train::k_train_block<128>,
                       (const void *)train::k_train_bwd<32>,   (const void *)train::k_train_bwd<64>,
                       (const void *)train::k_train_bwd<128>,  (const void *)train::k_attn_fwd_lds<4>, (const void *)train::k_attn_fwd_lds<8>,
                       (const void *)train::k_attn_fwd_lds<16>, (const void *)train::k_attn_bwd_lds<4>,
                       (const void *)train::k_attn_bwd_lds<8>, (const void *)train::k_attn_bwd_lds<16>};
  if (lds_max < train::block_lds<128>()) return hipErrorInvalidValue;
  for (const void *f : fns) {
    const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_max);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

namespace {
template <int D>
hipError_t bwd_go(const TrainBwd &a, int blocks, hipStream_t s) {
  hipLaunchKernelGGL(train::k_train_bwd<D>, dim3((unsigned)blocks), dim3(train::kTbWaves * 64), train::bwd_lds<D>(), s, a);
  return hipGetLastError();
}
}  // namespace

int train_bwd_blocks(int64_t rows, int cu_count) {
  return (int)std::max<int64_t>(1, std::min<int64_t>((rows + 15) / 16, cu_count));
}

hipError_t train_bwd(int d, const TrainBwd &a, int cu_count, hipStream_t s) {
  if (a.rows <= 0) return hipSuccess;
  const int blocks = train_bwd_blocks(a.rows, cu_count);
  switch (d) {
    case 32: return bwd_go<32>(a, blocks, s);
    case 64: return bwd_go<64>(a, blocks, s);
    case 128: return bwd_go<128>(a, blocks, s);
  }
  return hipErrorInvalidValue;
}

hipError_t train_qkv(int d, const TrainQkv &a, int cu_count, size_t lds_max, hipStream_t s) {
  if (a.rows <= 0) return hipSuccess;
  switch (d) {
    case 32: return qkv_go<32>(a, cu_count, lds_max, s);
    case 64: return qkv_go<64>(a, cu_count, lds_max, s);
    case 128: return qkv_go<128>(a, cu_count, lds_max, s);
  }
  return hipErrorInvalidValue;
}

hipError_t train_block(int d, const TrainBlock &a, int cu_count, size_t lds_max, hipStream_t s) {
  if (a.rows <= 0) return hipSuccess;
  switch (d) {
    case 32: return block_go<32>(a, cu_count, lds_max, s);
    case 64: return block_go<64>(a, cu_count, lds_max, s);
    case 128: return block_go<128>(a, cu_count, lds_max, s);
  }
  return hipErrorInvalidValue;
}

int train_dw_splits(int d, int64_t rows, int tiles, int cu_count) {
  // Three blocks per compute unit, as many as the register file holds at d = 128, where a block's range is then at
  // least eight of the kernel's steps (4096 / d rows), else two (a short range is mostly its first loads and its partial
  // sums); at least 128 rows each.  Steps of four layers with two and three blocks, us: BCH(31,16), d = 32, 1000 words
  // 663 / 672, LDPC(128,64), d = 32, 160 words 512 / 524, 512 words 1078 / 1043; d = 64, 200 words 927 / 919, 1024 words
  // 3223 / 3150; BCH(31,16), d = 128, 300 words 923 / 940; LDPC(256,128), d = 128, 256 words 3394 / 3292 (four 3443).
  const auto ranges = [&](int64_t per_cu) { return (per_cu * cu_count + tiles - 1) / tiles; };
  const int64_t want = rows >= ranges(3) * 8 * (4096 / d) ? ranges(3) : ranges(2);
  return (int)std::max<int64_t>(1, std::min<int64_t>(want, (rows + 127) / 128));
}

hipError_t train_weight_grads(int d, TrainDwJobs &J, int cu_count, float *part, int64_t part_floats, hipStream_t s) {
  if (J.rows <= 0 || J.n < 1 || J.n > kTrainDwJobs) return hipErrorInvalidValue;
  J.tile0[0] = 0;
  for (int k = 0; k < J.n; ++k) {
    const TrainDwJob &j = J.j[k];
    if (j.K % d || j.N % d || j.seg % d || j.ldy % 2 || ((uintptr_t)j.dy & 7u) || ((uintptr_t)j.q & 1u)) return hipErrorInvalidValue;
    J.tile0[k + 1] = J.tile0[k] + (j.K / d) * (j.N / d);
  }
  const int tiles = J.tile0[J.n];
  const int rs = 4096 / d;   // rows of one step of the kernel
  int64_t splits = train_dw_splits(d, J.rows, tiles, cu_count);
  if (splits > 8) splits = splits / 8 * 8;
  J.chunk = ((J.rows + splits - 1) / splits + rs - 1) / rs * rs;
  splits = (J.rows + J.chunk - 1) / J.chunk;
  J.splits = (int)splits;
  J.part = part;
  J.cpart = part + splits * tiles * d * d;
  if (splits * tiles * (int64_t)d * (d + 1) > part_floats) return hipErrorInvalidValue;
  const dim3 grid((unsigned)(tiles * splits)), rgrid((unsigned)(tiles * (d * d / train::kThreads + 1) + 4 * d / 16));
  switch (d) {
    case 32:
      hipLaunchKernelGGL(train::k_train_dw<32>, grid, dim3(train::kThreads), 0, s, J);
      hipLaunchKernelGGL(train::k_train_dw_reduce<32>, rgrid, dim3(train::kThreads), 0, s, J);
      break;
    case 64:
      hipLaunchKernelGGL(train::k_train_dw<64>, grid, dim3(train::kThreads), 0, s, J);
      hipLaunchKernelGGL(train::k_train_dw_reduce<64>, rgrid, dim3(train::kThreads), 0, s, J);
      break;
    case 128:
      hipLaunchKernelGGL(train::k_train_dw<128>, grid, dim3(train::kThreads), 0, s, J);
      hipLaunchKernelGGL(train::k_train_dw_reduce<128>, rgrid, dim3(train::kThreads), 0, s, J);
      break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// The LDS form where a word fits (930, 1024 and 1077 tokens at d_h = 4, 8 and 16 with 160 KB) and one block per
// word and head group is no longer than the whole card's gathers.  A block's time goes with the tokens it stages and
// the 16 / d_h rows of each, so short words always take it; longer ones once there is a block for every second
// compute unit, but not at d_h = 4 and d > 32, where the gathers of a row's many heads share cache lines.  Steps of
// two layers, gathers / LDS, us: 384 tokens, d = 64, d_h = 4, 1 word 249 / 265, 32 words 342 / 333; 900 tokens,
// d = 32, d_h = 4, 1 word 222 / 337, 64 words 528 / 528, 160 words 1188 / 1091; d = 64, d_h = 4, 160 words 1584 / 1778;
// d = 64, d_h = 8, 4 words 306 / 350, 64 words 739 / 677; d = 128, d_h = 16, 1074 tokens, 4 words 476 / 501, 64
// words 1728 / 1396.
template <int DH>
static bool attention_in_lds(const TrainAttn &p, int64_t blocks, int cu_count, size_t lds_max) {
  if (train::attn_lds_bytes<DH>(p.L) > lds_max || p.d % 16 || blocks > INT32_MAX) return false;
  return p.L * (1 + 16 / DH) <= 1920 || (2 * blocks >= cu_count && (DH > 4 || p.d == 32));
}

template <int DH>
static hipError_t attention_go(bool backward, const TrainAttn &p, int cu_count, size_t lds_max, hipStream_t s) {
  const size_t lds = train::attn_lds_bytes<DH>(p.L);
  const int64_t blocks = p.rows / p.L * (p.d / 16);
  if (attention_in_lds<DH>(p, blocks, cu_count, lds_max)) {
    const unsigned threads = (unsigned)std::min(1024, (p.L * (16 / DH) * train::attn_split<DH>() + 63) / 64 * 64);
    if (!backward) hipLaunchKernelGGL(train::k_attn_fwd_lds<DH>, dim3((unsigned)blocks), dim3(threads), lds, s, p);
    else hipLaunchKernelGGL(train::k_attn_bwd_lds<DH>, dim3((unsigned)blocks), dim3(threads), lds, s, p);
    return hipGetLastError();
  }
  const dim3 grid(blocks_for(p.rows * p.heads, train::kThreads));
  if (!backward) {
    hipLaunchKernelGGL(train::k_attn_fwd<DH>, grid, dim3(train::kThreads), 0, s, p);
  } else {
    hipLaunchKernelGGL(train::k_attn_bwd_q<DH>, grid, dim3(train::kThreads), 0, s, p);
    hipLaunchKernelGGL(train::k_attn_bwd_kv<DH>, grid, dim3(train::kThreads), 0, s, p);
  }
  return hipGetLastError();
}

hipError_t train_attention(bool backward, int dh, const TrainAttn &p, int cu_count, size_t lds_max, hipStream_t s) {
  if (p.rows <= 0) return hipSuccess;
  switch (dh) {
    case 4: return attention_go<4>(backward, p, cu_count, lds_max, s);
    case 8: return attention_go<8>(backward, p, cu_count, lds_max, s);
    case 16: return attention_go<16>(backward, p, cu_count, lds_max, s);
  }
  return hipErrorInvalidValue;
}

hipError_t train_colsum(const float *A, int64_t lda, const float *w, int64_t rows, int C, float *out, float *part,
                        int64_t part_floats, hipStream_t s) {
  if (C <= 0) return hipSuccess;
  int cwl = 0;
  while ((1 << cwl) < C && cwl < 6) ++cwl;
  const int lanes = train::kThreads >> cwl;
  const unsigned cblocks = blocks_for(C, 1 << cwl);
  // about 1024 blocks in all, each lane summing at least 8 rows
  int64_t chunks = std::min<int64_t>((rows + 8 * lanes - 1) / (8 * lanes), std::max<int64_t>(1, 1024 / cblocks));
  chunks = std::max<int64_t>(1, std::min<int64_t>(chunks, part_floats / C));
  const int64_t chunk = std::max<int64_t>(1, (rows + chunks - 1) / chunks);
  chunks = std::max<int64_t>(1, (rows + chunk - 1) / chunk);
  const auto pass1 = w ? train::k_colsum<true> : train::k_colsum<false>;
  float *o = chunks == 1 ? out : part;
  hipLaunchKernelGGL(pass1, dim3(cblocks, (unsigned)chunks), dim3(train::kThreads), 0, s, A, lda, w, rows, C, cwl, chunk, o,
                     (int64_t)C);
  // pass two over the partial rows: a block per column, its 256 lanes over the partial rows (a few
  // loads a lane, then the LDS tree), which takes a fraction of the 16-lanes-a-column form's time
  if (chunks > 1)
    hipLaunchKernelGGL(train::k_colsum<false>, dim3((unsigned)C, 1), dim3(train::kThreads), 0, s, (const float *)part, (int64_t)C,
                       (const float *)nullptr, chunks, C, 0, chunks, out, (int64_t)C);
  return hipGetLastError();
}

hipError_t train_rowdot(const float *x, int64_t rows, int d, const float *w1, const float *b1, float *z, hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  hipLaunchKernelGGL(train::k_rowdot, dim3(blocks_for(rows, 4)), dim3(train::kThreads), 0, s, x, rows, d, w1, b1, z);
  return hipGetLastError();
}

hipError_t train_outer(const float *dz, int64_t rows, const float *w1, int d, float *dx, hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  hipLaunchKernelGGL(train::k_outer, dim3(blocks_for(rows * d, train::kThreads)), dim3(train::kThreads), 0, s, dz, rows,
                     w1, d, dx);
  return hipGetLastError();
}

hipError_t train_loss(const float *f, const float *y, const float *xs, int64_t count, float *df, float *part,
                      float *loss, hipStream_t s) {
  if (count <= 0) return hipSuccess;
  const unsigned nb = blocks_for(count, train::kThreads);
  const float inv = 1.0f / (float)count;
  hipLaunchKernelGGL(train::k_loss, dim3(nb), dim3(train::kThreads), 0, s, f, y, xs, count, inv, df, part);
  hipLaunchKernelGGL(train::k_loss_final, dim3(1), dim3(64), 0, s, part, (int)nb, inv, loss);
  return hipGetLastError();
}

hipError_t train_embed_grad(const float *t, const float *dx, int64_t words, int L, int d, float *de, hipStream_t s) {
  hipLaunchKernelGGL(train::k_embed_grad, dim3((unsigned)L, (unsigned)(d / 32)), dim3(train::kThreads), 0, s, t, dx, words, L, d,
                     de);
  return hipGetLastError();
}

}  // namespace aecct
