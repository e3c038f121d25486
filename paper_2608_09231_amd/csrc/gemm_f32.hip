// f32 GEMM for the f32 (small) workloads: C = epi(A . W^T + bias) on
// v_mfma_f32_16x16x4_f32 (f32 products and sums).
//
// These layers are short (64 to about a thousand rows, K from 16 to a few
// hundred): latency bounds them, so a tile is small, its operands go straight
// from global memory (L2) into registers as 16-byte runs of K, and one
// work-group's eight waves share K where the tiles alone would leave most CUs
// idle.  Measured on the 80 x 896 x 128 (with the RMS norm) and 80 x 128 x 640
// layers of the 64 + 16 token workload against 64 x 64 tiles with 16-deep LDS
// slices: 25.9 + 4.1 (the norm's own launch) -> 5.8 us and 54.9 -> 7.5 us.
#include <algorithm>

#include "common.h"
#include "kernels.h"

namespace dit {
namespace {

struct ProbF {
  const float* A; int64_t lda;
  const float* W; int64_t ldw;
  const float* bias;
  float* C; int64_t ldc;
  const float* gate;
  float* x; float alpha;  // Euler update (see GemmArgs)
  int M, N, K, flags, gelu_from, gap_at, gap, rms_cols, tiles_n;
};

struct BatchF {
  ProbF p0, p1;
  int tiles0;
};

// Four consecutive values of K, zeros past its end (VEC: K % 4 == 0 and
// 16-byte aligned rows).  Loaded from inside the row in any case: a tested
// load would become a branch, and the next one wait behind it.
template <bool VEC>
__device__ __forceinline__ f32x4_t load4(const float* p, int k, int K) {
  f32x4_t v;
  if constexpr (VEC) {
    v = *(const f32x4_t*)(p + min(k, K - 4));
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = p[min(k + e, K - 1)];
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = k + e < K ? v[e] : 0.f;
  return v;
}

// TS x TS outputs per work-group.  TS = 16 or 32: each of eight waves takes an
// eighth of K for the whole tile; TS = 64: each of four takes a 32 x 32 quarter
// of the tile.  HD: head width of the RMS norm, a divisor of TS (0: none here).
constexpr int waves_of(int ts) { return ts == 64 ? 4 : 8; }

template <int TS, int HD, bool VEC>
__global__ __launch_bounds__(64 * waves_of(TS)) void gemm_f32_kernel(BatchF b) {
  constexpr int KS = TS == 64 ? 1 : 8;  // waves that share K
  constexpr int NB = TS == 16 ? 1 : 2;  // 16 x 16 blocks each way of a wave's part
  __shared__ float part[waves_of(TS)][16 * NB][16 * NB + 1];
  int tile = blockIdx.x;
  const bool second = tile >= b.tiles0;
  const ProbF& p = second ? b.p1 : b.p0;
  if (second) tile -= b.tiles0;
  const int m0 = tile / p.tiles_n * TS, n0 = tile % p.tiles_n * TS;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, lq = lane >> 4;
  const int mw = TS == 64 ? 32 * (wave >> 1) : 0, nw = TS == 64 ? 32 * (wave & 1) : 0;

  // MFMA j of a 16-deep step takes k = 16 s + 4 lq + j from each lane: the
  // order of K inside a step is the same for both operands
  const int steps = (p.K + 15) / 16, per = (steps + KS - 1) / KS;
  const int s0 = KS == 1 ? 0 : wave * per, s1 = min(steps, s0 + per);
  const float *ar[NB], *wr[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    ar[i] = p.A + (int64_t)min(m0 + mw + 16 * i + lr, p.M - 1) * p.lda;
    wr[i] = p.W + (int64_t)min(n0 + nw + 16 * i + lr, p.N - 1) * p.ldw;
  }
  f32x4_t acc[NB][NB] = {};
  // steps whose loads are in flight together: 3 against 5 the same below a few
  // hundred 32 x 32 tiles, 1152 x 1536 x 256 21.3 / 24.3 us, 1152 x 3072 x 1280 156 / 178
  constexpr int U = 3;
  for (int s = s0; s < s1; s += U) {
    f32x4_t a[U][NB], w[U][NB];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (s + u >= s1) break;
      const int k = 16 * (s + u) + 4 * lq;
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        a[u][i] = load4<VEC>(ar[i], k, p.K);
        w[u][i] = load4<VEC>(wr[i], k, p.K);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (s + u >= s1) break;
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
          for (int n = 0; n < NB; ++n)
            acc[i][n] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u][i][j], w[u][n][j], acc[i][n], 0, 0, 0);
    }
  }
  // acc[i][n][r] = C[16 i + 4 lq + r][16 n + lr] of the wave's part
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int n = 0; n < NB; ++n)
#pragma unroll
      for (int r = 0; r < 4; ++r) part[wave][16 * i + 4 * lq + r][16 * n + lr] = acc[i][n][r];
  __syncthreads();

  // thread: four columns of a row; a head is HD / 4 neighbouring threads
  const bool gated = p.flags & DIT_EPI_GATED_RES, silu = p.flags & DIT_EPI_SILU;
  constexpr int TPR = TS / 4, RPP = TS < 256 / TPR ? TS : 256 / TPR;
  if (tid >= TPR * RPP) return;
#pragma unroll
  for (int pass = 0; pass < TS / RPP; ++pass) {
    const int r = pass * RPP + tid / TPR, c = 4 * (tid % TPR);
    const int m = m0 + r;
    float v[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if constexpr (TS == 64) {
        v[e] = part[2 * (r >> 5) + (c >> 5)][r & 31][(c & 31) + e];
      } else {
        v[e] = 0.f;
#pragma unroll
        for (int w = 0; w < KS; w += 2) v[e] += part[w][r][c + e] + part[w + 1][r][c + e];
      }
      const int n = n0 + c + e;
      v[e] += p.bias && n < p.N ? p.bias[n] : 0.f;
    }
    if constexpr (HD > 0) {
      if (n0 + c < p.rms_cols) {  // whole heads: the same for a head's threads
        float ss = v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3];
#pragma unroll
        for (int o = 1; o < HD / 4; o <<= 1) ss += __shfl_xor(ss, o, 64);
        const float sc = rsqrtf(ss / (float)HD + DIT_RMS_EPS);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] *= sc;
      }
    }
    if (m >= p.M) continue;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int n = n0 + c + e;
      if (n >= p.N) continue;
      float y = v[e];
      if (n >= p.gelu_from) y = gelu_tanh_f(y);
      if (silu) y = silu_f(y);
      if (p.x) {
        float* x = p.x + (int64_t)m * p.ldc + n;
        *x = fmaf(p.alpha, y, *x);
        continue;
      }
      float* o = p.C + (int64_t)m * p.ldc + n + (n >= p.gap_at ? p.gap : 0);
      *o = gated ? *o + p.gate[n] * y : y;
    }
  }
}

}  // namespace

hipError_t launch_gemm_f32(const GemmArgs* g, int n, int head_dim, int n_cu, hipStream_t s) {
  if (n < 1 || n > 2) return hipErrorInvalidValue;
  BatchF b;
  int64_t tiles64 = 0, tiles32 = 0;
  int K = g[0].K;
  bool vec = true, rms = false;
  for (int i = 0; i < n; ++i) {
    const GemmArgs& a = g[i];
    tiles64 += (int64_t)((a.M + 63) / 64) * ((a.N + 63) / 64);
    tiles32 += (int64_t)((a.M + 31) / 32) * ((a.N + 31) / 32);
    vec &= a.K % 4 == 0 && a.lda % 4 == 0 && a.ldw % 4 == 0 && !(((uintptr_t)a.A | (uintptr_t)a.W) & 15);
    rms |= a.rms_cols > 0;
    K = std::min(K, a.K);
  }
  // Per launch, us (M x N x K without the norm):
  // - 16 x 16 tiles while they make about one round of the chip (a 32 x 32 tile is
  //   bound by what one CU can load): against 32 x 32, 12 tiles of 32 x 32 (80 x 128 x
  //   640) 6.1 / 9.7, 76 (600 x 128 x 640) 8.7 / 9.8, 72 (80 x 768 x 1280) 8.8 / 15.7;
  //   144 (1152 x 128 x 640) 11.5 / 9.8, 152 (600 x 256 x 640) 11.6 / 10.0.  With the norm
  //   of 32-wide heads they need its launch (1.9 us) beside: from K = 640 on.
  // - 64 x 64 (half the operand reads, K not shared) where they make one round and
  //   32 x 32 four: against 32 x 32, 216 tiles (1152 x 768) K = 256 18.1 / 13.9, 640
  //   29.0 / 30.5, 1280 47 / 56, 3072 95 / 121; 192 (240 x 3072 x 1280) 46 / 41, 480 (600 x
  //   3072 x 1280) 113 / 101, 864 (1152 x 3072) K = 256 55 / 45, 1280 223 / 178 (five
  //   steps' loads in flight).
  const bool few = 10 * tiles32 <= 3 * n_cu && !(rms && head_dim == 32 && K < 640);
  const int ts = few ? 16 : tiles64 <= n_cu && tiles32 > 3 * n_cu && K >= 640 ? 64 : 32;
  const int hd = rms && ts % head_dim == 0 ? head_dim : 0;
  int total = 0;
  for (int i = 0; i < n; ++i) {
    ProbF& p = i ? b.p1 : b.p0;
    p.A = (const float*)g[i].A; p.lda = g[i].lda;
    p.W = (const float*)g[i].W; p.ldw = g[i].ldw;
    p.bias = (const float*)g[i].bias;
    p.C = (float*)g[i].C; p.ldc = g[i].ldc;
    p.gate = g[i].gate;
    p.x = g[i].euler_x; p.alpha = g[i].euler_alpha;
    p.M = g[i].M; p.N = g[i].N; p.K = g[i].K;
    p.flags = g[i].flags; p.gelu_from = g[i].gelu_from; p.gap_at = g[i].gap_at; p.gap = g[i].gap;
    p.rms_cols = g[i].rms_cols;
    p.tiles_n = (p.N + ts - 1) / ts;
    total += (p.M + ts - 1) / ts * p.tiles_n;
    if (i == 0) b.tiles0 = total;
  }
  if (n == 1) b.p1 = b.p0;
  if (total == 0) return hipSuccess;
#define DIT_GEMM_F32(TS_, HD_)                                                                        \
  hipLaunchKernelGGL((vec ? gemm_f32_kernel<TS_, HD_, true> : gemm_f32_kernel<TS_, HD_, false>), dim3(total), \
                     dim3(64 * waves_of(TS_)), 0, s, b)
  if (ts == 64) {
    if (hd == 16) DIT_GEMM_F32(64, 16);
    else if (hd == 32) DIT_GEMM_F32(64, 32);
    else if (hd == 64) DIT_GEMM_F32(64, 64);
    else DIT_GEMM_F32(64, 0);
  } else if (ts == 16) {
    if (hd == 16) DIT_GEMM_F32(16, 16);
    else DIT_GEMM_F32(16, 0);
  } else {
    if (hd == 16) DIT_GEMM_F32(32, 16);
    else if (hd == 32) DIT_GEMM_F32(32, 32);
    else DIT_GEMM_F32(32, 0);
  }
#undef DIT_GEMM_F32
  hipError_t e = hipGetLastError();
  for (int i = 0; i < n && e == hipSuccess && !hd; ++i)  // heads wider than a tile
    if (g[i].rms_cols > 0) e = launch_rms_heads_f32((float*)g[i].C, g[i].ldc, g[i].M, g[i].rms_cols, head_dim, s);
  return e;
}

}  // namespace dit
