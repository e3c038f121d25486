// bf16 GEMM on gfx950 MFMA with the fused epilogues of the DiT blocks:
// C = epi(A . W^T + bias).
//
// A [M,K] and W [N,K] are both K-contiguous (W in nn.Linear [out,in]
// layout), so every MFMA operand is a 16-byte run of K.  Tiles are staged
// through LDS in BK = 64 slices (128-byte rows) by buffer loads with an LDS
// destination, the 16-byte chunks of each row XOR-swizzled by
// ((row >> 1) & 7): two consecutive 128-byte rows fill one 256-byte bank
// cycle, so the fragment reads of 16 consecutive rows hit 16 distinct 16-byte
// bank groups.  The main kernel (256 x 256 tiles, 8 waves of 64 x 128,
// 16x16x32 MFMAs) keeps a ring of five operand slices in LDS: W slices (cold,
// from HBM) arrive two slices ahead of use, A slices one; smaller tiles use a
// two-stage pipeline on 32x32x16 MFMAs.
// Workgroups are remapped so that each of the 8 XCDs walks a contiguous,
// M-grouped range of tiles (its own L2 sees the shared A rows / W columns).
#include <algorithm>
#include <type_traits>
#include <utility>

#include "common.h"
#include "kernels.h"

namespace dit {

namespace {

constexpr int BK = 64;

struct Prob {
  const bf16_t* A; int64_t lda;
  const bf16_t* W; int64_t ldw;
  const bf16_t* bias;
  void* C; int64_t ldc;
  const float* gate;
  int64_t gstride;  // gate vector of row m: gate + (m / gseg) * gstride (gseg > 0)
  int M, N, K;
  int flags, rms_cols, gelu_from, gap_at, gap, gseg;
  int tiles_m, tiles_n;
  bf16_t* vt;  // transposed values (see GemmArgs)
  int vt_col0, vt_heads, vt_ld, vt_split, vt_rows0, vt_key0, vt_rows1, vt_key1;
};

struct Batch {
  Prob p0, p1;
  int tiles0, total;
  // Ring kernel: tiles past `whole` are computed in `parts` shares of K each,
  // as f32 pieces in ws for gemm_finish_kernel; total counts the pieces.
  int whole, parts;
  float* ws;
};

__device__ __forceinline__ int xcd_remap(int bid, int n) {
  const int x = bid & 7, idx = bid >> 3;
  const int q = n >> 3, r = n & 7;
  return x * q + (x < r ? x : r) + idx;
}

// Epilogue over groups of G = min(TN, 4) adjacent 32x32 tiles (one 128-wide
// head when G = 4): bias, optional per-head RMS norm, GELU / SiLU, then
// store (bf16 round, f32, or gated residual).  acc[i][j][r] holds C[m][n]
// with m = m0 + wm*WM + i*32 + 8*(r/4) + 4*lhalf + (r%4) and
// n = n0 + wn*WN + j*32 + lrow.
template <int TM, int TN, int WM, int WN>
__device__ __forceinline__ void epilogue(const Prob& P, f32x16_t (&acc)[TM][TN], int m0, int n0, int wm,
                                         int wn, int lrow, int lhalf) {
  constexpr int G = TN < 4 ? TN : 4;
  const int ncol0 = n0 + wn * WN;
  const bool f32out = P.flags & DIT_EPI_F32;
  const bool gated = P.flags & DIT_EPI_GATED_RES;
  const bool silu = P.flags & DIT_EPI_SILU;
#pragma unroll
  for (int hb = 0; hb < TN / G; ++hb) {
    const int nh = ncol0 + hb * G * 32;   // first column of this group
    const bool rms = G == 4 && nh < P.rms_cols;
    float bv[G], gv[G];
    int col[G];
    bool gl[G], ok[G];
#pragma unroll
    for (int jj = 0; jj < G; ++jj) {
      const int n = nh + jj * 32 + lrow;
      ok[jj] = n < P.N;
      bv[jj] = (P.bias && ok[jj]) ? bf16_to_f32(P.bias[n]) : 0.f;
      gv[jj] = (gated && ok[jj]) ? P.gate[n] : 0.f;
      gl[jj] = n >= P.gelu_from;
      col[jj] = n + (n >= P.gap_at ? P.gap : 0);
    }
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        float v[G];
#pragma unroll
        for (int jj = 0; jj < G; ++jj) v[jj] = acc[i][hb * G + jj][r] + bv[jj];
        if (rms) {
          float ss = 0.f;
#pragma unroll
          for (int jj = 0; jj < G; ++jj) ss += v[jj] * v[jj];
#pragma unroll
          for (int o = 1; o < 32; o <<= 1) ss += __shfl_xor(ss, o, 64);
          const float sc = rsqrtf(ss * (1.f / 128.f) + DIT_RMS_EPS);
#pragma unroll
          for (int jj = 0; jj < G; ++jj) v[jj] *= sc;
        }
        const int m = m0 + wm * WM + i * 32 + 8 * (r >> 2) + 4 * lhalf + (r & 3);
        if (m >= P.M) continue;
#pragma unroll
        for (int jj = 0; jj < G; ++jj) {
          if (!ok[jj]) continue;
          float y = v[jj];
          if (gl[jj]) y = gelu_tanh_f(y);
          if (silu) y = silu_f(y);
          if (f32out) {
            ((float*)P.C)[(int64_t)m * P.ldc + col[jj]] = y;
          } else {
            bf16_t* c = (bf16_t*)P.C + (int64_t)m * P.ldc + col[jj];
            if (gated) y = bf16_to_f32(*c) + gv[jj] * y;
            *c = f32_to_bf16(y);
          }
        }
      }
    }
  }
}

template <int BM, int BN, int WGM, int WGN>
__global__ __launch_bounds__(256) void gemm_bf16_kernel(Batch b) {
  constexpr int WM = BM / WGM, WN = BN / WGN;
  constexpr int TM = WM / 32, TN = WN / 32;
  constexpr int A_LD = BM * BK / (8 * 256);  // 16-byte chunks per thread
  constexpr int B_LD = BN * BK / (8 * 256);
  static_assert(WGM * WGN == 4, "4 waves");
  static_assert(A_LD >= 1 && B_LD >= 1, "tile too small");

  __shared__ __attribute__((aligned(16))) bf16_t smem[2 * (BM + BN) * BK];

  if ((int)blockIdx.x >= b.total) return;
  int lt = xcd_remap(blockIdx.x, b.total);
  const bool second = lt >= b.tiles0;
  Prob P = second ? b.p1 : b.p0;
  if (second) lt -= b.tiles0;

  // M-grouped tile order (8 tile-rows per group).
  constexpr int GROUP = 8;
  const int in_group = GROUP * P.tiles_n;
  const int gid = lt / in_group;
  const int first_m = gid * GROUP;
  const int gsz = min(P.tiles_m - first_m, GROUP);
  const int tm = first_m + (lt % in_group) % gsz;
  const int tn = (lt % in_group) / gsz;
  const int m0 = tm * BM, n0 = tn * BN;
  // per-segment gate vectors: the host admits only BM | gseg, so a tile's
  // rows share one vector
  if (P.gseg > 0) P.gate += (int64_t)(m0 / P.gseg) * P.gstride;

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WGN, wn = wave % WGN;

  // global -> register staging of one BK slice
  uint4 ra[A_LD], rb[B_LD];
  auto gload = [&](int k0) {
#pragma unroll
    for (int i = 0; i < A_LD; ++i) {
      const int q = tid + 256 * i, row = q >> 3, kc = q & 7;
      const int gm = min(m0 + row, P.M - 1);
      const int gk = k0 + kc * 8;
      ra[i] = (gk < P.K) ? *(const uint4*)(P.A + (int64_t)gm * P.lda + gk) : make_uint4(0, 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < B_LD; ++i) {
      const int q = tid + 256 * i, row = q >> 3, kc = q & 7;
      const int gn = min(n0 + row, P.N - 1);
      const int gk = k0 + kc * 8;
      rb[i] = (gk < P.K) ? *(const uint4*)(P.W + (int64_t)gn * P.ldw + gk) : make_uint4(0, 0, 0, 0);
    }
  };
  auto sstore = [&](int stage) {
    bf16_t* sA = smem + stage * (BM + BN) * BK;
    bf16_t* sB = sA + BM * BK;
#pragma unroll
    for (int i = 0; i < A_LD; ++i) {
      const int q = tid + 256 * i, row = q >> 3, kc = q & 7;
      *(uint4*)(sA + row * BK + ((kc ^ ((row >> 1) & 7)) << 3)) = ra[i];
    }
#pragma unroll
    for (int i = 0; i < B_LD; ++i) {
      const int q = tid + 256 * i, row = q >> 3, kc = q & 7;
      *(uint4*)(sB + row * BK + ((kc ^ ((row >> 1) & 7)) << 3)) = rb[i];
    }
  };

  f32x16_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  const int nk = (P.K + BK - 1) / BK;
  gload(0);
  sstore(0);
  __syncthreads();

  const int lrow = lane & 31, lhalf = lane >> 5;
  for (int kt = 0; kt < nk; ++kt) {
    if (kt + 1 < nk) gload((kt + 1) * BK);
    const bf16_t* sA = smem + (kt & 1) * (BM + BN) * BK;
    const bf16_t* sB = sA + BM * BK;
#pragma unroll
    for (int s = 0; s < BK / 16; ++s) {
      const int kc = 2 * s + lhalf;
      bf16x8_t af[TM], bfr[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const int row = wm * WM + i * 32 + lrow;
        uint4 v = *(const uint4*)(sA + row * BK + ((kc ^ ((row >> 1) & 7)) << 3));
        af[i] = __builtin_bit_cast(bf16x8_t, v);
      }
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int row = wn * WN + j * 32 + lrow;
        uint4 v = *(const uint4*)(sB + row * BK + ((kc ^ ((row >> 1) & 7)) << 3));
        bfr[j] = __builtin_bit_cast(bf16x8_t, v);
      }
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[i], bfr[j], acc[i][j], 0, 0, 0);
    }
    if (kt + 1 < nk) sstore((kt + 1) & 1);
    __syncthreads();
  }

  epilogue<TM, TN, WM, WN>(P, acc, m0, n0, wm, wn, lrow, lhalf);
}

// LDS-staged epilogue for waves that own 128 output columns (WN == 128).
// Per 32-row slab: the raw f32 accumulators go to this wave's 16 KB of LDS
// (columns XOR 32 on rows with bit 2 set, so the two lane halves of a write
// hit different banks); then lane l handles rows l/16 + 4p (p = 0..7) and
// columns 4(l%16) + [0,4) and 64 + 4(l%16) + [0,4): bias, per-head RMS (a
// head is the 16 lanes of one row: 4 shuffles), GELU / SiLU, gated
// residual, and 8-byte stores that coalesce to 128 bytes per row.
// Requires N % 8 == 0, gelu_from and gap_at multiples of 4.
// KIND selects a specialised body: EPI_K_STORE (bf16 store; the per-head RMS
// norm, GELU and column gap each apply to whole 128-column groups, so they
// are wave-uniform), EPI_K_GATED (gated residual only), EPI_K_ANY (every
// flag, per column).
enum { EPI_K_STORE = 0, EPI_K_GATED = 1, EPI_K_ANY = 2 };
template <int KIND = EPI_K_ANY>
struct EpiLds {
  const Prob& P;
  int m_base, ncol0, cq, rq, lrow, lhalf;
  bool f32out, gated, silu, rms, gelu_u;
  float bv[2][4], gv[2][4];
  int col[2];
  bool ok[2], gl[2];
  float* slab;

  __device__ __forceinline__ EpiLds(const Prob& P_, int m_base_, int ncol0_, int lrow_, int lhalf_, float* slab_)
      : P(P_), m_base(m_base_), ncol0(ncol0_), lrow(lrow_), lhalf(lhalf_), slab(slab_) {}

  // Flags, column map, bias and gate values of this lane's 8 columns.
  __device__ __forceinline__ void prep() {
    const int lane = lhalf * 32 + lrow;
    cq = lane & 15;
    rq = lane >> 4;
    f32out = KIND == EPI_K_ANY && (P.flags & DIT_EPI_F32);
    gated = KIND == EPI_K_GATED || (KIND == EPI_K_ANY && (P.flags & DIT_EPI_GATED_RES));
    silu = KIND == EPI_K_ANY && (P.flags & DIT_EPI_SILU);
    rms = KIND != EPI_K_GATED && ncol0 < P.rms_cols;
    gelu_u = KIND == EPI_K_STORE && ncol0 >= P.gelu_from;
#pragma unroll
    for (int hh = 0; hh < 2; ++hh) {
      const int n = ncol0 + 64 * hh + 4 * cq;
      ok[hh] = n < P.N;
      gl[hh] = n >= P.gelu_from;
      col[hh] = n + (n >= P.gap_at ? P.gap : 0);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        bv[hh][e] = (P.bias && ok[hh]) ? bf16_to_f32(P.bias[n + e]) : 0.f;
        gv[hh][e] = (gated && ok[hh]) ? P.gate[n + e] : 0.f;
      }
    }
  }

  // Residual values C[m][col .. col+3] of slab i (gated epilogue), loaded
  // before any slab is staged so their latency overlaps the staging.
  __device__ __forceinline__ void load_old(int i, uint2 (&old)[8][2]) const {
#pragma unroll
    for (int p = 0; p < 8; ++p) {
      const int m = min(m_base + i * 32 + rq + 4 * p, P.M - 1);
#pragma unroll
      for (int hh = 0; hh < 2; ++hh)
        old[p][hh] = ok[hh] ? *(const uint2*)((const bf16_t*)P.C + (int64_t)m * P.ldc + col[hh]) : make_uint2(0, 0);
    }
  }

  // One 32-row slab: accumulators -> LDS -> 8-column row segments -> global.
  // Nothing waits on global memory here: a wave's LDS operations complete in
  // order, so neither the read-back nor the next slab's writes need more
  // than the wait for this wave's own slab writes.
  __device__ __forceinline__ void slab_pass(const f32x16_t (&a)[4], int i, const uint2 (&old)[8][2]) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = 8 * (r >> 2) + 4 * lhalf + (r & 3);
        const int c = (j * 32 + lrow) ^ (((row >> 2) & 1) << 5);
        slab[row * 128 + c] = a[j][r];
      }
    slab_rows<1, 5>(i, old);
  }

  // The same for 16 x 16 blocks (a: rows 0..15, b: rows 16..31): lane (lr, lq)
  // holds column lr and rows 4 lq .. 4 lq + 3 of each; columns XOR 16 ((row >> 2) & 3)
  // send the four lane quarters of a write to different banks.
  __device__ __forceinline__ void slab_pass16(const f32x4_t (&a)[8], const f32x4_t (&b)[8], int i,
                                              const uint2 (&old)[8][2], int lr, int lq) {
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int c = (16 * j + lr) ^ (lq << 4);
        slab[(4 * lq + r) * 128 + c] = a[j][r];
        slab[(16 + 4 * lq + r) * 128 + c] = b[j][r];
      }
    slab_rows<3, 4>(i, old);
  }

  // Reads the staged slab back as 8-column row segments (columns XOR
  // ((row >> 2) & MASK) << SH), applies the epilogue and stores.
  template <int MASK, int SH>
  __device__ __forceinline__ void slab_rows(int i, const uint2 (&old)[8][2]) {
    __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0) only
#pragma unroll
    for (int p = 0; p < 8; ++p) {
      const int row = rq + 4 * p;
      const int sw = ((row >> 2) & MASK) << SH;
      float v[2][4];
#pragma unroll
      for (int hh = 0; hh < 2; ++hh) {
        const float4 t = *(const float4*)(slab + row * 128 + ((64 * hh + 4 * cq) ^ sw));
        v[hh][0] = t.x + bv[hh][0]; v[hh][1] = t.y + bv[hh][1];
        v[hh][2] = t.z + bv[hh][2]; v[hh][3] = t.w + bv[hh][3];
      }
      if (KIND != EPI_K_GATED && rms) {
        float ss = 0.f;
#pragma unroll
        for (int hh = 0; hh < 2; ++hh)
#pragma unroll
          for (int e = 0; e < 4; ++e) ss += v[hh][e] * v[hh][e];
#pragma unroll
        for (int o = 1; o < 16; o <<= 1) ss += __shfl_xor(ss, o, 64);
        const float sc = rsqrtf(ss * (1.f / 128.f) + DIT_RMS_EPS);
#pragma unroll
        for (int hh = 0; hh < 2; ++hh)
#pragma unroll
          for (int e = 0; e < 4; ++e) v[hh][e] *= sc;
      }
      const int m = m_base + i * 32 + row;
      if constexpr (KIND == EPI_K_STORE) {
        if (gelu_u)
#pragma unroll
          for (int hh = 0; hh < 2; ++hh)
#pragma unroll
            for (int e = 0; e < 4; ++e) v[hh][e] = gelu_tanh_f(v[hh][e]);
        if (m < P.M)
#pragma unroll
          for (int hh = 0; hh < 2; ++hh)
            if (ok[hh])
              *(uint2*)((bf16_t*)P.C + (int64_t)m * P.ldc + col[hh]) =
                  make_uint2(pack_bf16x2(v[hh][0], v[hh][1]), pack_bf16x2(v[hh][2], v[hh][3]));
        continue;
      } else if constexpr (KIND == EPI_K_GATED) {
        if (m < P.M)
#pragma unroll
          for (int hh = 0; hh < 2; ++hh)
            if (ok[hh]) {
              const uint2 o = old[p][hh];
              const float y0 = __uint_as_float(o.x << 16) + gv[hh][0] * v[hh][0];
              const float y1 = __uint_as_float(o.x & 0xffff0000u) + gv[hh][1] * v[hh][1];
              const float y2 = __uint_as_float(o.y << 16) + gv[hh][2] * v[hh][2];
              const float y3 = __uint_as_float(o.y & 0xffff0000u) + gv[hh][3] * v[hh][3];
              *(uint2*)((bf16_t*)P.C + (int64_t)m * P.ldc + col[hh]) =
                  make_uint2(pack_bf16x2(y0, y1), pack_bf16x2(y2, y3));
            }
        continue;
      }
      if (m < P.M) {
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) {
          if (!ok[hh]) continue;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            if (gl[hh]) v[hh][e] = gelu_tanh_f(v[hh][e]);
            if (silu) v[hh][e] = silu_f(v[hh][e]);
          }
          if (f32out) {
            *(float4*)((float*)P.C + (int64_t)m * P.ldc + col[hh]) =
                make_float4(v[hh][0], v[hh][1], v[hh][2], v[hh][3]);
          } else {
            bf16_t* c = (bf16_t*)P.C + (int64_t)m * P.ldc + col[hh];
            if (gated) {
              const uint2 o = old[p][hh];
              v[hh][0] = __uint_as_float(o.x << 16) + gv[hh][0] * v[hh][0];
              v[hh][1] = __uint_as_float(o.x & 0xffff0000u) + gv[hh][1] * v[hh][1];
              v[hh][2] = __uint_as_float(o.y << 16) + gv[hh][2] * v[hh][2];
              v[hh][3] = __uint_as_float(o.y & 0xffff0000u) + gv[hh][3] * v[hh][3];
            }
            *(uint2*)c = make_uint2(pack_bf16x2(v[hh][0], v[hh][1]), pack_bf16x2(v[hh][2], v[hh][3]));
          }
        }
      }
    }
  }
};

// Runs the slab passes of a wave that owns TM x 32 rows and 128 columns;
// with the gated residual, the old values of every slab (of one slab at a
// time when TM > 2) are requested first.
// Each slab index is a compile-time constant so the accumulators stay in
// registers.
template <int TM, int KIND, size_t... Is>
__device__ __forceinline__ void epilogue_lds_impl(EpiLds<KIND>& e, f32x16_t (&acc)[TM][4], std::index_sequence<Is...>) {
  if constexpr (TM <= 2) {
    uint2 old[TM][8][2];
    if (e.gated) (e.load_old((int)Is, old[Is]), ...);
    (e.slab_pass(acc[Is], (int)Is, old[Is]), ...);
  } else {  // bounded registers: one slab's old values at a time
    auto one = [&](auto i) {
      constexpr int I = decltype(i)::value;
      uint2 old[8][2];
      if (e.gated) e.load_old(I, old);
      e.slab_pass(acc[I], I, old);
    };
    (one(std::integral_constant<int, (int)Is>{}), ...);
  }
}

typedef __attribute__((address_space(3))) void lds_void_t;
typedef __attribute__((address_space(1))) void glb_void_t;

// A DMA config uses the LDS-staged epilogue when its waves own 128 columns
// and its LDS holds one 32 x 128 f32 slab per wave; the host only picks such
// a config for problems that meet the epilogue's alignment conditions.
template <int WN, int NW, int LDS_BYTES>
constexpr bool kLdsEpilogue = WN == 128 && LDS_BYTES >= NW * 32 * 128 * 4;

// s_waitcnt with only the vector-memory counter constrained (gfx9 encoding:
// vmcnt[3:0] | expcnt[6:4] = 7 | lgkmcnt[11:8] = 15 | vmcnt[5:4] at [15:14]).
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt");
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}

// vmcnt(N) and lgkmcnt(0) in one wait (same encoding as wait_vmcnt).
template <int N>
__device__ __forceinline__ void wait_vmcnt_lgkm0() {
  static_assert(N >= 0 && N < 64, "vmcnt");
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | ((N >> 4) << 14));
}

// Workgroup barrier without the workgroup-scope fence of __syncthreads: that
// fence waits for every outstanding global load of the wave, copies to LDS
// included, which would drain the copies a deeper pipeline keeps in flight.
// The memory clobber keeps the compiler from moving memory operations across
// it; callers wait for their own LDS reads and copies first.
__device__ __forceinline__ void barrier_no_fence() { asm volatile("s_barrier" ::: "memory"); }

// 16 bytes per lane from base + voff + soff (bytes, 32-bit offsets) into LDS
// at dst + 16 lane: a raw buffer load with an LDS destination.  Offsets past
// 4 GiB - 1 read zeros; the host admits this path only when every row of
// the operand lies below that bound.
__device__ __forceinline__ void buf_lds16(const void* base, lds_void_t* dst, uint32_t voff, uint32_t soff) {
#if defined(__HIP_DEVICE_COMPILE__)
  const __amdgpu_buffer_rsrc_t r =
      __builtin_amdgcn_make_buffer_rsrc((void*)base, (short)0, (int)0xffffffffu, 0x00020000);
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, dst, 16, voff, soff, 0, 0);
#endif
}

// Direct-to-LDS pipeline (K % BK == 0): BK-deep slices of A and W are copied
// by global_load_lds_dwordx4 (64 lanes x 16 bytes into a contiguous 1 KB per
// instruction: no staging registers), STAGES slices in flight.  A slice row
// has CPR = BK/8 chunks of 16 bytes; RPB = 256/(2 BK) rows share one 256-byte
// bank cycle, and chunk c of row r is stored at c ^ ((r / RPB) % CPR), so the
// fragment reads of 16 consecutive rows hit 16 distinct bank groups.  The
// per-lane source chunk of each copy realises the same swizzle.
template <int BM, int BN, int WGM, int WGN, int BK_, int STAGES>
__global__ __launch_bounds__(64 * WGM * WGN) void gemm_bf16_dma_kernel(Batch b) {
  constexpr int WM = BM / WGM, WN = BN / WGN;
  constexpr int TM = WM / 32, TN = WN / 32;
  constexpr int NW = WGM * WGN;
  constexpr int CPR = BK_ / 8, RPB = 256 / (2 * BK_);
  constexpr int ROWS_PER_INS = 64 / CPR;
  constexpr int A_INS = BM / (ROWS_PER_INS * NW), B_INS = BN / (ROWS_PER_INS * NW);
  constexpr int INS = A_INS + B_INS;                 // copies per wave per slice
  constexpr int STAGE = (BM + BN) * BK_ * 2;         // bytes
  static_assert(A_INS >= 1 && B_INS >= 1 && A_INS * ROWS_PER_INS * NW == BM &&
                    B_INS * ROWS_PER_INS * NW == BN, "tile");
  static_assert(STAGES >= 2 && (STAGES - 2) * INS < 64, "stages");

  __shared__ __attribute__((aligned(1024))) char smem[STAGES * STAGE];

  if ((int)blockIdx.x >= b.total) return;
  int lt = xcd_remap(blockIdx.x, b.total);
  const bool second = lt >= b.tiles0;
  Prob P = second ? b.p1 : b.p0;
  if (second) lt -= b.tiles0;
  constexpr int GROUP = 8;
  const int in_group = GROUP * P.tiles_n;
  const int gid = lt / in_group;
  const int first_m = gid * GROUP;
  const int gsz = min(P.tiles_m - first_m, GROUP);
  const int tm = first_m + (lt % in_group) % gsz;
  const int tn = (lt % in_group) / gsz;
  const int m0 = tm * BM, n0 = tn * BN;
  // per-segment gate vectors: the host admits only BM | gseg, so a tile's
  // rows share one vector
  if (P.gseg > 0) P.gate += (int64_t)(m0 / P.gseg) * P.gstride;

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WGN, wn = wave % WGN;
  const int lrow = lane & 31, lhalf = lane >> 5;

  // per-lane source offsets in bytes (fixed for the whole K loop; the host
  // admits this kernel only when they fit in 32 bits); the slice offset
  // kt * BK * 2 travels in the scalar offset of the buffer load
  uint32_t aoff[A_INS], boff[B_INS];
#pragma unroll
  for (int j = 0; j < A_INS; ++j) {
    const int row = ROWS_PER_INS * (wave * A_INS + j) + lane / CPR;
    const int c = (lane % CPR) ^ ((row / RPB) % CPR);
    aoff[j] = ((uint32_t)min(m0 + row, P.M - 1) * (uint32_t)P.lda + c * 8) * 2u;
  }
#pragma unroll
  for (int j = 0; j < B_INS; ++j) {
    const int row = ROWS_PER_INS * (wave * B_INS + j) + lane / CPR;
    const int c = (lane % CPR) ^ ((row / RPB) % CPR);
    boff[j] = ((uint32_t)min(n0 + row, P.N - 1) * (uint32_t)P.ldw + c * 8) * 2u;
  }
  auto issue = [&](int kt) {
    char* sA = smem + (kt % STAGES) * STAGE;
    char* sB = sA + BM * BK_ * 2;
    const uint32_t so = (uint32_t)kt * BK_ * 2;
#pragma unroll
    for (int j = 0; j < A_INS; ++j) buf_lds16(P.A, (lds_void_t*)(sA + (wave * A_INS + j) * 1024), aoff[j], so);
#pragma unroll
    for (int j = 0; j < B_INS; ++j) buf_lds16(P.W, (lds_void_t*)(sB + (wave * B_INS + j) * 1024), boff[j], so);
  };

  f32x16_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  // The epilogue state (bias, gate, column map) is loaded before the K loop
  // when registers allow (TM <= 2), so those loads are done when the tile is.
  [[maybe_unused]] EpiLds<> epi(P, m0 + wm * TM * 32, n0 + wn * 128, lrow, lhalf, (float*)smem + wave * (32 * 128));
  if constexpr (kLdsEpilogue<WN, NW, STAGES * STAGE> && TM <= 2) epi.prep();

  const int nk = P.K / BK_;
  if constexpr (STAGES == 2 && BK_ == 64) {
    // Two 64-deep slices in LDS, fragments double-buffered in registers: the
    // LDS reads of substep s+1 (and, in substep 0, the copies of the next
    // slice) are interleaved with the 8 MFMAs of substep s; one barrier per
    // slice, the last iteration peeled so the loop body has no branch.
    auto rd = [&](int kt, int s, bf16x8_t(&af)[TM], bf16x8_t(&bfr)[TN]) {
      const char* sA = smem + (kt & 1) * STAGE;
      const char* sB = sA + BM * BK_ * 2;
      const int kc = 2 * s + lhalf;
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const int row = wm * WM + i * 32 + lrow;
        af[i] = __builtin_bit_cast(bf16x8_t, *(const uint4*)(sA + row * (2 * BK_) + ((kc ^ ((row / RPB) % CPR)) << 4)));
      }
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int row = wn * WN + j * 32 + lrow;
        bfr[j] = __builtin_bit_cast(bf16x8_t, *(const uint4*)(sB + row * (2 * BK_) + ((kc ^ ((row / RPB) % CPR)) << 4)));
      }
    };
    auto mm = [&](const bf16x8_t(&af)[TM], const bf16x8_t(&bfr)[TN]) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[i], bfr[j], acc[i][j], 0, 0, 0);
    };
    // Instruction order of one substep, fixed by scheduling groups: one MFMA,
    // then two LDS reads of the next substep (and, with WithCopy, two buffer
    // copies of the next slice), repeated; then the remaining MFMAs.  A
    // scheduling fence closes every substep, so the reads stay one substep
    // ahead of the MFMAs that consume them (two fragment sets live).
    auto sched = [&](auto with_copy) {
      constexpr bool WithCopy = decltype(with_copy)::value;
      constexpr int NM = TM * TN, ND = TM + TN, NG = (ND + 1) / 2;
      static_assert(NM >= NG, "substep shape");
#pragma unroll
      for (int q = 0; q < NG; ++q) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
        if constexpr (WithCopy) __builtin_amdgcn_sched_group_barrier(0x020, 2, 0);  // VMEM read
        __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);  // DS read
      }
      if constexpr (NM > NG) __builtin_amdgcn_sched_group_barrier(0x008, NM - NG, 0);
      __builtin_amdgcn_sched_barrier(0);
    };
    using copy_t = std::integral_constant<bool, true>;
    using nocopy_t = std::integral_constant<bool, false>;
    bf16x8_t a0[TM], b0[TN], a1[TM], b1[TN];
    issue(0);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    rd(0, 0, a0, b0);
    for (int kt = 0; kt < nk - 1; ++kt) {
      issue(kt + 1);  // into the buffer of slice kt-1, which every wave has finished
      rd(kt, 1, a1, b1); mm(a0, b0); sched(copy_t{});
      rd(kt, 2, a0, b0); mm(a1, b1); sched(nocopy_t{});
      rd(kt, 3, a1, b1); mm(a0, b0); sched(nocopy_t{});
      mm(a1, b1);
      wait_vmcnt<0>();  // this wave's copies of slice kt+1 have landed
      __syncthreads();  // everyone's have, and every read of slice kt is done
      rd(kt + 1, 0, a0, b0);
    }
    rd(nk - 1, 1, a1, b1); mm(a0, b0); sched(nocopy_t{});
    rd(nk - 1, 2, a0, b0); mm(a1, b1); sched(nocopy_t{});
    rd(nk - 1, 3, a1, b1); mm(a0, b0); sched(nocopy_t{});
    mm(a1, b1);
  } else {
#pragma unroll
  for (int s = 0; s < STAGES - 1; ++s)
    if (s < nk) issue(s);

  for (int kt = 0; kt < nk; ++kt) {
    // slice kt must have landed (later slices may stay in flight) and this
    // wave's reads of slice kt-1 have returned
    if (nk - 1 - kt >= STAGES - 2) wait_vmcnt_lgkm0<(STAGES - 2) * INS>();
    else __builtin_amdgcn_s_waitcnt(0);
    // then every wave's copies of slice kt are in and slice kt-1 is no longer
    // read.  (__syncthreads would drain the copies in flight: through the entry
    // point 28 x 18432 x 3072 59.4 us, so 43.7; 512 x 3072 x 4096 50.9, 45.5; 64 x
    // 16384 x 1024 32.1, 26.5; at 28 x 52224 x 3072 both are at 81, 4 TB/s.)
    barrier_no_fence();
    if (kt + STAGES - 1 < nk) issue(kt + STAGES - 1);
    const char* sA = smem + (kt % STAGES) * STAGE;
    const char* sB = sA + BM * BK_ * 2;
#pragma unroll
    for (int s = 0; s < BK_ / 16; ++s) {
      const int kc = 2 * s + lhalf;
      bf16x8_t af[TM], bfr[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const int row = wm * WM + i * 32 + lrow;
        af[i] = __builtin_bit_cast(bf16x8_t, *(const uint4*)(sA + row * (2 * BK_) + ((kc ^ ((row / RPB) % CPR)) << 4)));
      }
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int row = wn * WN + j * 32 + lrow;
        bfr[j] = __builtin_bit_cast(bf16x8_t, *(const uint4*)(sB + row * (2 * BK_) + ((kc ^ ((row / RPB) % CPR)) << 4)));
      }
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[i], bfr[j], acc[i][j], 0, 0, 0);
    }
  }
  }
  __syncthreads();  // all waves are done with the slices before the epilogue reuses LDS
  if constexpr (kLdsEpilogue<WN, NW, STAGES * STAGE>) {
    if constexpr (TM > 2) epi.prep();
    epilogue_lds_impl<TM>(epi, acc, std::make_index_sequence<TM>{});
  } else {
    epilogue<TM, TN, WM, WN>(P, acc, m0, n0, wm, wn, lrow, lhalf);
  }
}

// Transposed values straight from the accumulators of a wave that owns 64
// rows x one 128-column head group (4 x 8 blocks of 16 x 16).  In a block,
// lane (lr, lq) holds column lr and rows 4 lq .. 4 lq + 3; with the key order
// of the transposed layout (slot 8 ((k >> 2) & 3) + 4 (k >> 4) + (k & 3)
// inside each 32-key group) those of a pair of blocks are the eight
// consecutive slots from 8 lq, one 16-byte store.  The host admits this only
// for 32-row aligned segments (a pair of blocks is one sequence's keys kb ..
// kb + 31, kb a multiple of 32), or for one sequence in one piece, whose last
// pair may end past its last key inside the padded key range.
__device__ __forceinline__ void store_vt(const Prob& P, const f32x4_t (&acc)[4][8], int m_base, int ncol0,
                                           int lr, int lq) {
  const int h = (ncol0 - P.vt_col0) >> 7;
  float bias[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) bias[j] = P.bias ? bf16_to_f32(P.bias[ncol0 + 16 * j + lr]) : 0.f;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int m = m_base + 32 * i;
    if (m >= P.M) continue;
    int z, key;
    if (m < P.vt_split) {
      z = m / P.vt_rows0;
      key = P.vt_key0 + m % P.vt_rows0;
    } else {
      const int mm = m - P.vt_split;
      z = mm / P.vt_rows1;
      key = P.vt_key1 + mm % P.vt_rows1;
    }
    bf16_t* base = P.vt + ((int64_t)(z * P.vt_heads + h) * 128 + lr) * P.vt_ld + key + 8 * lq;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const f32x4_t &a = acc[2 * i][j], &c = acc[2 * i + 1][j];
      const float b = bias[j];
      *(uint4*)(base + (int64_t)(16 * j) * P.vt_ld) =
          make_uint4(pack_bf16x2(a[0] + b, a[1] + b), pack_bf16x2(a[2] + b, a[3] + b),
                     pack_bf16x2(c[0] + b, c[1] + b), pack_bf16x2(c[2] + b, c[3] + b));
    }
  }
}
// Problem and origin of 256 x 256 tile lt of a launch: M-grouped order, eight
// tile rows per group.
__device__ __forceinline__ void ring_tile(const Batch& b, int lt, Prob& P, int& m0, int& n0) {
  const bool second = lt >= b.tiles0;
  P = second ? b.p1 : b.p0;
  if (second) lt -= b.tiles0;
  constexpr int GROUP = 8;
  const int in_group = GROUP * P.tiles_n;
  const int gid = lt / in_group;
  const int first_m = gid * GROUP;
  const int gsz = min(P.tiles_m - first_m, GROUP);
  m0 = (first_m + (lt % in_group) % gsz) * 256;
  n0 = (lt % in_group) / gsz * 256;
}

constexpr int PIECE_WAVE = 64 * 128;  // floats of a wave's part of a piece, in register order

// 256 x 256 tiles, 8 waves of 64 x 128, BK = 64, with the whole 160 KB of
// LDS as a ring of five 32 KB operand slices: operand i (W slice s = 2s,
// A slice s = 2s + 1) lives in unit i % 5.  W slices are copied two slices
// ahead of use and A slices one ahead: the weights come cold from HBM, while
// A was mostly written just before.
//
// What bounds it is the board's power: under these launches the clock sits at
// 1.9-2.1 GHz (of 2.4) and falls as the MFMAs get busier, so energy per product counts,
// not issue slots.  16x16x32 MFMAs read and write each accumulator once per
// 32 of K (32x32x16: once per 16) for the same fragment reads from LDS, and
// give the same bits.  Measured against 32x32x16 in turn on one card, through
// the entry point: 4608 x 9216 x 3072 with the RMS norm 235.0 -> 223.2 us, 4608 x
// 12288 x 3072 GELU 327 -> 307, 4608 x 3072 x 12288 gated 295 -> 272, 8192^3 plain
// 1356 -> 1413 TFLOP/s, 32760 x 13824 x 5120 GELU 3505 -> 3280 us.  With 32x32x16, four waves of 128 x 128 (two thirds of the LDS
// reads) ran at 0.99 of the eight waves' rate in the main loop and at 0.92-0.96
// over the K = 3072 layers, whose epilogue then has one wave per SIMD.
//
// A 32-deep substep reads its 12 fragments under the first 24 of the previous
// substep's 32 MFMAs (W fragment j is dead after its four MFMAs, so about 16
// fragments are live); a scheduling fence closes each substep.
// Requires K % 64 == 0, K >= 128 and the LDS-staged epilogue's conditions.
template <int KIND>
__global__ __launch_bounds__(512) void gemm_bf16_ring_kernel(Batch b) {
  constexpr int BK_ = 64, WGN = 2;
  constexpr int WM = 64, WN = 128, TM = 4, TN = 8;
  constexpr int UNIT = 256 * BK_ * 2;  // one operand slice
  constexpr int INS = 4;                // 1 KB copies per wave per operand slice
  __shared__ __attribute__((aligned(1024))) char smem[5 * UNIT];

  if ((int)blockIdx.x >= b.total) return;
  const int piece = (int)blockIdx.x - b.whole;  // < 0: a whole tile
  Prob P;
  int m0, n0;
  ring_tile(b, piece < 0 ? xcd_remap(blockIdx.x, b.whole) : b.whole + piece / b.parts, P, m0, n0);
  int nk = P.K / BK_;  // >= 2
  if (piece >= 0) {
    const int part = piece % b.parts, k0 = nk * part / b.parts, k1 = nk * (part + 1) / b.parts;
    P.A += (int64_t)k0 * BK_;
    P.W += (int64_t)k0 * BK_;
    nk = k1 - k0;
  }
  // per-segment gate vectors: the host admits only BM | gseg
  if (P.gseg > 0) P.gate += (int64_t)(m0 / P.gseg) * P.gstride;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WGN, wn = wave % WGN;
  const int lr = lane & 15, lq = lane >> 4;

  // per-lane source byte offsets: copy j of this wave moves rows
  // 8 (4 wave + j) .. + 7 of the slice, 16-byte chunks XOR-swizzled by
  // ((row >> 1) & 7) as in the two-stage kernel
  uint32_t aoff[INS], boff[INS];
#pragma unroll
  for (int j = 0; j < INS; ++j) {
    const int row = 8 * (wave * INS + j) + (lane >> 3);
    const int c = (lane & 7) ^ ((row >> 1) & 7);
    aoff[j] = ((uint32_t)min(m0 + row, P.M - 1) * (uint32_t)P.lda + c * 8) * 2u;
    boff[j] = ((uint32_t)min(n0 + row, P.N - 1) * (uint32_t)P.ldw + c * 8) * 2u;
  }
  auto issue = [&](const bf16_t* base, const uint32_t (&off)[INS], int u, int s) {
    char* d = smem + u;
    const uint32_t so = (uint32_t)s * BK_ * 2;
#pragma unroll
    for (int j = 0; j < INS; ++j) buf_lds16(base, (lds_void_t*)(d + (wave * INS + j) * 1024), off[j], so);
  };
  // this lane's fragment offset inside 16 rows of a unit: row lr, k = 32 s + 8 lq .. + 7
  int loff[2];
#pragma unroll
  for (int s = 0; s < 2; ++s) loff[s] = lr * 128 + (((4 * s + lq) ^ ((lr >> 1) & 7)) << 4);
  auto rd = [&](int uw, int ua, int s, bf16x8_t(&af)[TM], bf16x8_t(&bfr)[TN]) {
    const char* sA = smem + ua + wm * WM * 128 + loff[s];
    const char* sB = smem + uw + wn * WN * 128 + loff[s];
#pragma unroll
    for (int i = 0; i < TM; ++i) af[i] = __builtin_bit_cast(bf16x8_t, *(const uint4*)(sA + i * 16 * 128));
#pragma unroll
    for (int j = 0; j < TN; ++j) bfr[j] = __builtin_bit_cast(bf16x8_t, *(const uint4*)(sB + j * 16 * 128));
  };
  f32x4_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  // bias and column map are loaded before the K loop; the gated epilogue's
  // gate values beside them would spill, and its own loads of the old rows
  // wait after the loop in any case
  EpiLds<KIND> epi(P, m0 + wm * WM, n0 + wn * WN, lane & 31, lane >> 5, (float*)smem + wave * (32 * 128));
  if constexpr (KIND == EPI_K_STORE) epi.prep();
  auto mm = [&](const bf16x8_t(&af)[TM], const bf16x8_t(&bfr)[TN]) {
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int i = 0; i < TM; ++i)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[i], bfr[j], acc[i][j], 0, 0, 0);
  };
  // per MFMA: a fragment read of the next substep after every second one, and
  // the four copies of this substep (if any) spread between them
  auto sched = [&](auto with_copy) {
    constexpr bool WithCopy = decltype(with_copy)::value;
#pragma unroll
    for (int q = 0; q < 32; ++q) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
      if (q % 2 == 1 && q < 24) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);  // DS read
      if (WithCopy && q % 6 == 2 && q < 24) __builtin_amdgcn_sched_group_barrier(0x010, 1, 0);  // VMEM
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  using yes = std::integral_constant<bool, true>;
  using no = std::integral_constant<bool, false>;

  bf16x8_t a0[TM], b0[TN], a1[TM], b1[TN];
  // unit offsets of W kt, A kt, W kt+1, A kt+1, W kt+2
  int u0 = 0, u1 = UNIT, u2 = 2 * UNIT, u3 = 3 * UNIT, u4 = 4 * UNIT;
  issue(P.W, boff, u0, 0);
  issue(P.A, aoff, u1, 0);
  issue(P.W, boff, u2, 1);
  issue(P.A, aoff, u3, 1);
  wait_vmcnt_lgkm0<2 * INS>();  // slice 0 has landed; slice 1 may be in flight
  barrier_no_fence();
  rd(u0, u1, 0, a0, b0);
  // Slice kt.  Its last fragments are in registers after the first substep:
  // there the wave waits for its own copies of slice kt+1 (W slice kt+2 may
  // stay in flight) and meets the others, so that the units of slice kt are
  // free for A slice kt+2 and (a substep later) W slice kt+3, and the first
  // fragments of slice kt+1 are read under the MFMAs of the second substep.
  // MORE: slice kt+2 exists.
  auto slice = [&](int kt, auto more) {
    constexpr bool MORE = decltype(more)::value;
    if constexpr (MORE) issue(P.W, boff, u4, kt + 2);
    rd(u0, u1, 1, a1, b1); mm(a0, b0);
    if constexpr (MORE) sched(yes{}); else sched(no{});
    if constexpr (MORE) wait_vmcnt_lgkm0<INS>();
    else __builtin_amdgcn_s_waitcnt(0);
    barrier_no_fence();
    if constexpr (MORE) issue(P.A, aoff, u0, kt + 2);
    rd(u2, u3, 0, a0, b0); mm(a1, b1);
    if constexpr (MORE) sched(yes{}); else sched(no{});
    const int t0 = u0, t1 = u1;
    u0 = u2; u1 = u3; u2 = u4; u3 = t0; u4 = t1;
  };
  for (int kt = 0; kt < nk - 2; ++kt) slice(kt, yes{});
  slice(nk - 2, no{});
  rd(u0, u1, 1, a1, b1); mm(a0, b0); sched(no{});
  mm(a1, b1);
  if (piece >= 0) {
    float* w = b.ws + ((int64_t)piece * 8 + wave) * PIECE_WAVE + 4 * lane;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) *(f32x4_t*)(w + (i * TN + j) * 256) = acc[i][j];
    return;
  }
  __syncthreads();  // every wave is done with the ring before the epilogue reuses LDS
  if constexpr (KIND == EPI_K_STORE) {
    const int ncol0 = n0 + wn * WN;  // wave-uniform: whole head groups are values or not
    if (P.vt && ncol0 >= P.vt_col0 && ncol0 < P.vt_col0 + 128 * P.vt_heads) {
      store_vt(P, acc, m0 + wm * WM, ncol0, lr, lq);
      return;
    }
  }
  if constexpr (KIND != EPI_K_STORE) epi.prep();
  uint2 old[2][8][2];
  if (epi.gated) { epi.load_old(0, old[0]); epi.load_old(1, old[1]); }
  epi.slab_pass16(acc[0], acc[1], 0, old[0], lr, lq);
  epi.slab_pass16(acc[2], acc[3], 1, old[1], lr, lq);
}

// Adds the pieces of one wave's part (64 x 128) of a tile in the order of K and
// runs the ring kernel's epilogue on the sum.  One wave per work-group: 64
// rows x one head group need nothing from the tile's other parts.
template <int KIND>
__global__ __launch_bounds__(64) void gemm_finish_kernel(Batch b) {
  __shared__ float slab[32 * 128];
  const int t = blockIdx.x >> 3, wave = blockIdx.x & 7;
  Prob P;
  int m0, n0;
  ring_tile(b, b.whole + t, P, m0, n0);
  if (P.gseg > 0) P.gate += (int64_t)(m0 / P.gseg) * P.gstride;
  const int lane = threadIdx.x, wm = wave >> 1, wn = wave & 1, lr = lane & 15, lq = lane >> 4;
  f32x4_t acc[4][8];
  for (int p = 0; p < b.parts; ++p) {
    const float* w = b.ws + (((int64_t)t * b.parts + p) * 8 + wave) * PIECE_WAVE + 4 * lane;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const f32x4_t v = *(const f32x4_t*)(w + (i * 8 + j) * 256);
        acc[i][j] = p ? acc[i][j] + v : v;
      }
  }
  const int ncol0 = n0 + 128 * wn;
  if constexpr (KIND == EPI_K_STORE) {
    if (P.vt && ncol0 >= P.vt_col0 && ncol0 < P.vt_col0 + 128 * P.vt_heads) {
      store_vt(P, acc, m0 + 64 * wm, ncol0, lr, lq);
      return;
    }
  }
  EpiLds<KIND> epi(P, m0 + 64 * wm, ncol0, lane & 31, lane >> 5, slab);
  epi.prep();
  uint2 old[2][8][2];
  if (epi.gated) { epi.load_old(0, old[0]); epi.load_old(1, old[1]); }
  epi.slab_pass16(acc[0], acc[1], 0, old[0], lr, lq);
  epi.slab_pass16(acc[2], acc[3], 1, old[1], lr, lq);
}

// Few rows or few tiles: 32 x NT outputs per work-group, operands straight
// from global memory into the fragments of 16x16x32 MFMAs, K shared by the
// eight waves (NT = 128: by four, the other four take the second 64 columns).
// What bounds it is latency (small models) or the weights' bytes (a few rows
// against a large table), not the matrix cores: many loads in flight from many
// work-groups count, and an LDS pipeline with one slice in flight per
// work-group has neither.  Through the entry point (11 us of it launch and
// wait), against 32 x 256 tiles: 28 x 3072 x 3072 51.6 -> 30.4 us, 240 x 256 x 1280
// 32.7 -> 21.6 us, 240 x 768 x 256 with the norm 23.7 -> 17.9 us.  Three steps'
// loads in flight at 122 registers (two work-groups per CU) beat four at 146.
// Requires K % 8 == 0 and the LDS-staged epilogue's conditions.
template <int NT>
__global__ __launch_bounds__(512, 4) void gemm_bf16_small_kernel(Batch b) {
  constexpr int NH = NT / 64, KS = 8 / NH;  // column halves, waves that share K
  constexpr int LD = 68;                    // floats per staged row of 64
  __shared__ __attribute__((aligned(16))) float part[8][32][LD];

  if ((int)blockIdx.x >= b.total) return;
  int lt = xcd_remap(blockIdx.x, b.total);
  const bool second = lt >= b.tiles0;
  Prob P = second ? b.p1 : b.p0;
  if (second) lt -= b.tiles0;
  const int m0 = lt % P.tiles_m * 32, n0 = lt / P.tiles_m * NT;  // neighbours share the weights
  if (P.gseg > 0) P.gate += (int64_t)(m0 / P.gseg) * P.gstride;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 15, lq = lane >> 4;
  const int ks = wave % KS, nh = wave / KS;
  const bf16_t *ap[2], *wp[4];
#pragma unroll
  for (int i = 0; i < 2; ++i) ap[i] = P.A + (int64_t)min(m0 + 16 * i + lr, P.M - 1) * P.lda;
#pragma unroll
  for (int j = 0; j < 4; ++j) wp[j] = P.W + (int64_t)min(n0 + 64 * nh + 16 * j + lr, P.N - 1) * P.ldw;
  const int steps = (P.K + 31) / 32, per = (steps + KS - 1) / KS;
  const int s0 = ks * per, s1 = min(steps, s0 + per);
  f32x4_t acc[2][4] = {};
  auto load8 = [&](const bf16_t* p, int k) {
    const uint4 v = *(const uint4*)(p + min(k, P.K - 8));
    return __builtin_bit_cast(bf16x8_t, k < P.K ? v : make_uint4(0, 0, 0, 0));
  };
  constexpr int U = 3;  // steps whose loads are in flight together
  for (int s = s0; s < s1; s += U) {
    bf16x8_t a[U][2], w[U][4];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (s + u >= s1) break;
      const int k = 32 * (s + u) + 8 * lq;
#pragma unroll
      for (int j = 0; j < 4; ++j) w[u][j] = load8(wp[j], k);
#pragma unroll
      for (int i = 0; i < 2; ++i) a[u][i] = load8(ap[i], k);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (s + u >= s1) break;
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[u][i], w[u][j], acc[i][j], 0, 0, 0);
    }
  }
  // acc[i][j][r] = C[16 i + 4 lq + r][16 j + lr] of the wave's 32 x 64
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) part[wave][16 * i + 4 * lq + r][16 * j + lr] = acc[i][j][r];
  __syncthreads();

  // 16 threads per row: columns 4 c .. + 3 of each half, added in wave order
  const int row = tid >> 4, c = tid & 15, m = m0 + row;
  float v[NH][4];
#pragma unroll
  for (int h = 0; h < NH; ++h) {
    const int n = n0 + 64 * h + 4 * c;
    f32x4_t t = {};
#pragma unroll
    for (int w = 0; w < KS; ++w) t += *(const f32x4_t*)&part[KS * h + w][row][4 * c];
    uint2 bb = make_uint2(0, 0);
    if (P.bias && n < P.N) {
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const uint32_t x = P.bias[n + 2 * e] | ((uint32_t)P.bias[n + 2 * e + 1] << 16);
        if (e) bb.y = x; else bb.x = x;
      }
    }
    v[h][0] = t[0] + __uint_as_float(bb.x << 16); v[h][1] = t[1] + __uint_as_float(bb.x & 0xffff0000u);
    v[h][2] = t[2] + __uint_as_float(bb.y << 16); v[h][3] = t[3] + __uint_as_float(bb.y & 0xffff0000u);
  }
  if constexpr (NT == 128) {
    if (n0 < P.rms_cols) {  // one 128-wide head per tile
      float ss = 0.f;
#pragma unroll
      for (int h = 0; h < NH; ++h)
#pragma unroll
        for (int e = 0; e < 4; ++e) ss += v[h][e] * v[h][e];
#pragma unroll
      for (int o = 1; o < 16; o <<= 1) ss += __shfl_xor(ss, o, 64);
      const float sc = rsqrtf(ss * (1.f / 128.f) + DIT_RMS_EPS);
#pragma unroll
      for (int h = 0; h < NH; ++h)
#pragma unroll
        for (int e = 0; e < 4; ++e) v[h][e] *= sc;
    }
  }
  if (m >= P.M) return;
#pragma unroll
  for (int h = 0; h < NH; ++h) {
    const int n = n0 + 64 * h + 4 * c;
    if (n >= P.N) continue;
    if (n >= P.gelu_from)
#pragma unroll
      for (int e = 0; e < 4; ++e) v[h][e] = gelu_tanh_f(v[h][e]);
    if (P.flags & DIT_EPI_SILU)
#pragma unroll
      for (int e = 0; e < 4; ++e) v[h][e] = silu_f(v[h][e]);
    const int64_t at = (int64_t)m * P.ldc + n + (n >= P.gap_at ? P.gap : 0);
    if (P.flags & DIT_EPI_F32) {
      *(float4*)((float*)P.C + at) = make_float4(v[h][0], v[h][1], v[h][2], v[h][3]);
      continue;
    }
    uint2* o = (uint2*)((bf16_t*)P.C + at);
    if (P.flags & DIT_EPI_GATED_RES) {
      const uint2 x = *o;
      const float4 g = *(const float4*)(P.gate + n);
      v[h][0] = __uint_as_float(x.x << 16) + g.x * v[h][0];
      v[h][1] = __uint_as_float(x.x & 0xffff0000u) + g.y * v[h][1];
      v[h][2] = __uint_as_float(x.y << 16) + g.z * v[h][2];
      v[h][3] = __uint_as_float(x.y & 0xffff0000u) + g.w * v[h][3];
    }
    *o = make_uint2(pack_bf16x2(v[h][0], v[h][1]), pack_bf16x2(v[h][2], v[h][3]));
  }
}


// Small-N projection (the final layer, N = C <= 128): v[m][c] = sum_k A[m][k] W[c][k]
// + bias[c], or with x != nullptr the Euler update x[m][c] += alpha * v[m][c]
// fused in.  16 RB rows per workgroup, the K range split over 8 waves, MFMA
// 16x16x32 bf16; A rows stream from HBM once, W (N x K, a few hundred KB)
// stays in L2.  The 8 partial tiles are summed through LDS in wave order.
// What bounds it is loads in flight and, at many rows, the L2 reads of W, so
// three steps' loads are issued together and RB = 2 halves those reads.
// Kernel time with four waves, one step in flight and 16 rows -> now: 4096 x 64 x
// 3072 41 -> 21, 1024 x 64 x 3072 28 -> 20, 32760 x 64 x 5120 290 -> 170 us.
template <int NT, int RB>  // N / 16 output tiles, 16-row blocks
__global__ __launch_bounds__(512) void proj_small_n_kernel(const bf16_t* __restrict__ A, int64_t lda,
                                                           const bf16_t* __restrict__ W, int64_t ldw,
                                                           const bf16_t* __restrict__ bias, float* out,
                                                           int64_t ldo, float* x, int64_t ldx, float alpha,
                                                           int M, int K) {
  constexpr int KS = 8, U = 3;
  __shared__ float part[KS][16 * RB][NT * 16 + 1];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int m0 = blockIdx.x * 16 * RB;
  const int lr = lane & 15, lq = lane >> 4;  // row / column within 16, k-quarter of the 32-deep step
  const int ksteps = K / 32, per = (ksteps + KS - 1) / KS;
  const int s0 = wave * per, s1 = min(ksteps, s0 + per);
  f32x4_t acc[RB][NT] = {};
  const bf16_t* ap[RB];
#pragma unroll
  for (int i = 0; i < RB; ++i) ap[i] = A + (int64_t)min(m0 + 16 * i + lr, M - 1) * lda + 8 * lq;
  const bf16_t* wp = W + (int64_t)lr * ldw + 8 * lq;
  for (int st = s0; st < s1; st += U) {
    bf16x8_t a[U][RB], w[U][NT];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (st + u >= s1) break;
#pragma unroll
      for (int i = 0; i < RB; ++i) a[u][i] = __builtin_bit_cast(bf16x8_t, *(const uint4*)(ap[i] + 32 * (st + u)));
#pragma unroll
      for (int j = 0; j < NT; ++j)
        w[u][j] = __builtin_bit_cast(bf16x8_t, *(const uint4*)(wp + (int64_t)16 * j * ldw + 32 * (st + u)));
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (st + u >= s1) break;
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int i = 0; i < RB; ++i)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[u][i], w[u][j], acc[i][j], 0, 0, 0);
    }
  }
  // acc[i][j][r] = C[row 16 i + 4 lq + r][col 16 j + lr]
#pragma unroll
  for (int i = 0; i < RB; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) part[wave][16 * i + 4 * lq + r][16 * j + lr] = acc[i][j][r];
  __syncthreads();
  for (int e = threadIdx.x; e < 16 * RB * NT * 16; e += 512) {
    const int r = e / (NT * 16), c = e % (NT * 16);
    const int m = m0 + r;
    if (m >= M) continue;
    float v = 0.f;
#pragma unroll
    for (int w = 0; w < KS; ++w) v += part[w][r][c];
    if (bias) v += bf16_to_f32(bias[c]);
    if (x) x[(int64_t)m * ldx + c] += alpha * v;
    else out[(int64_t)m * ldo + c] = v;
  }
}

constexpr int SPLIT_MIN_SLICES = 24;

struct Cfg {
  int bm, bn, wn, wg_per_cu, threads, bk;
  bool lds_epi;
  float eff;
  bool dma;
  void (*fn)(Batch);
  int min_k;  // smallest K the kernel's pipeline admits
};

// eff: relative MFMA efficiency of a full tile (measured ordering); the
// chooser minimises rounds x per-round work / eff over the configs a
// problem admits.  The 32 x 128 tiles keep three slices in flight and two
// work-groups per CU, for few rows against many weights: 28 x 52224 x 3072
// 93 -> 80 us (32 x 256 tiles, one slice in flight), 512 x 3072 x 4096 60.7 -> 45.5
// us; past 512 of them 512 x 9216 x 3072 76 against 56 us, 256 x 18432 x 3072 94
// against 79 (but 128 x 18432 x 3072 68 against 84).
#define DIT_DMA_CFG(BM, BN, WGM, WGN, BK_, ST, WPC, EFF)                                      \
  {BM, BN, BN / WGN, WPC, 64 * WGM * WGN, BK_,                                                 \
   kLdsEpilogue<BN / WGN, WGM * WGN, ST * (BM + BN) * BK_ * 2>, EFF, true,                     \
   gemm_bf16_dma_kernel<BM, BN, WGM, WGN, BK_, ST>, 0}
const Cfg kCfgs[] = {
    {256, 256, 128, 1, 512, 64, true, 1.08f, true, gemm_bf16_ring_kernel<EPI_K_ANY>, 128},
    DIT_DMA_CFG(256, 256, 4, 2, 64, 2, 1, 1.00f),
    DIT_DMA_CFG(256, 128, 4, 1, 64, 2, 1, 0.72f),
    DIT_DMA_CFG(128, 128, 4, 1, 64, 2, 2, 0.85f),
    DIT_DMA_CFG(32, 256, 1, 4, 64, 2, 2, 0.45f),
    DIT_DMA_CFG(32, 128, 1, 4, 64, 4, 2, 0.44f),
    {256, 128, 128, 1, 256, 64, false, 0.60f, false, gemm_bf16_kernel<256, 128, 4, 1>, 0},
    {128, 128, 128, 2, 256, 64, false, 0.55f, false, gemm_bf16_kernel<128, 128, 4, 1>, 0},
    {32, 256, 64, 2, 256, 64, false, 0.30f, false, gemm_bf16_kernel<32, 256, 1, 4>, 0},
    // picked by their own rule: plain layers, and those with the per-head norm
    {32, 64, 64, 1, 512, 8, true, 0.f, false, gemm_bf16_small_kernel<64>, 0},
    {32, 128, 128, 1, 512, 8, true, 0.f, false, gemm_bf16_small_kernel<128>, 0},
};
#undef DIT_DMA_CFG
constexpr int kNumCfgs = sizeof(kCfgs) / sizeof(kCfgs[0]), kSmallCfg = kNumCfgs - 2;

Prob make_prob(const GemmArgs& g, int bm, int bn) {
  Prob p;
  p.A = (const bf16_t*)g.A; p.lda = g.lda;
  p.W = (const bf16_t*)g.W; p.ldw = g.ldw;
  p.bias = (const bf16_t*)g.bias;
  p.C = g.C; p.ldc = g.ldc;
  p.gate = g.gate;
  p.gseg = g.gseg; p.gstride = g.gstride;
  p.M = g.M; p.N = g.N; p.K = g.K;
  p.flags = g.flags; p.rms_cols = g.rms_cols;
  p.gelu_from = g.gelu_from; p.gap_at = g.gap_at; p.gap = g.gap;
  p.tiles_m = (g.M + bm - 1) / bm;
  p.tiles_n = (g.N + bn - 1) / bn;
  p.vt = (bf16_t*)g.vt;
  p.vt_col0 = g.vt_col0; p.vt_heads = g.vt_heads; p.vt_ld = g.vt_ld; p.vt_split = g.vt_split;
  p.vt_rows0 = g.vt_rows0; p.vt_key0 = g.vt_key0; p.vt_rows1 = g.vt_rows1; p.vt_key1 = g.vt_key1;
  return p;
}

// Shares of K for the tiles of a ring launch past the last whole round (0:
// they stay whole).  Where they fill at most half the chip, floor(n_cu / rest)
// shares take nk / parts slices (1.2 us each with every CU busy) instead of nk;
// writing, adding and the second launch cost about 20 us.  (Past half the chip
// that is one share: nothing to share.)  Through the entry point, whole tiles
// (or the 128 x 128 ones chosen instead) against shares, us:
//   one whole round: 6144 x 3072 x 15360 (288 tiles) 724 / 429, 6144 x 3072 x 3072
//     161 / 130, 6144 x 4096 x 3072 (384, two shares, 24 slices saved) 174 / 151,
//     4352 x 4096 x 1792 (272, 24 saved) 105 / 89; below 24: 6144 x 4096 x 2560 (20)
//     151 / 151 and 4352 x 4096 x 1280 (16) 86 / 86, but 4352 x 4096 x 1600 (21) 97 / 83
//   two or three, many shares: 16640 x 2048 x 2048 (520, 28 saved) 159 / 147, 16896 x
//     3072 x 2048 (792, 28) 222 / 208
//   three or more, two or three shares: the idle CUs' power goes to the others,
//     so a slice saved is worth less: K = 3072 at 864 tiles 310 / 308, 1152 388 / 396,
//     2376 756 / 762; K = 4096 395 / 390, 497 / 494, 965 / 957; K = 5120 481 / 468, 613 /
//     604, 1193 / 1179
int ring_parts(long tiles, const GemmArgs* g, int n, int n_cu) {
  const long rem = tiles % n_cu;
  if (tiles < n_cu || rem == 0) return 0;
  for (int i = 0; i < n; ++i)
    if (g[i].one_chain) return 0;
  int nk = g[0].K / 64;
  for (int i = 1; i < n; ++i) nk = std::min(nk, g[i].K / 64);
  const int parts = (int)std::min<long>(n_cu / rem, nk / 4);
  if (parts < 2 || nk - nk / parts < SPLIT_MIN_SLICES) return 0;
  return tiles / n_cu >= 3 && parts <= 3 && nk < 64 ? 0 : parts;
}

int pick_cfg(const GemmArgs* g, int n, int n_cu, bool ws) {
  bool rms = false, aligned = true;
  for (int i = 0; i < n; ++i) {
    rms |= g[i].rms_cols > 0;
    aligned &= (g[i].lda % 8) == 0 && (g[i].ldw % 8) == 0;
  }
  bool epi_ok = true;  // conditions of the LDS-staged epilogue
  for (int i = 0; i < n; ++i) {
    epi_ok &= (g[i].N % 8) == 0 && (g[i].ldc % 4) == 0;
    epi_ok &= g[i].gelu_from >= g[i].N || (g[i].gelu_from % 4) == 0;
    epi_ok &= g[i].gap == 0 || ((g[i].gap_at | g[i].gap) % 4) == 0;
  }
  bool off32 = true;  // byte offsets of every A / W row fit the buffer loads' 32 bits
  for (int i = 0; i < n; ++i) {
    off32 &= ((uint64_t)(g[i].M - 1) * g[i].lda + g[i].K) * 2 <= 0xffffffffull;
    off32 &= ((uint64_t)(g[i].N - 1) * g[i].ldw + g[i].K) * 2 <= 0xffffffffull;
  }
  auto admits = [&](const Cfg& k) {
    if (rms && k.wn % 128) return false;
    for (int i = 0; i < n; ++i)
      if (g[i].gseg > 0 && g[i].gseg % k.bm) return false;
    if (!k.dma) return true;
    if (!aligned || !off32 || (k.lds_epi && !epi_ok)) return false;
    for (int i = 0; i < n; ++i)
      if (g[i].K % k.bk || g[i].K < k.min_k) return false;
    return true;
  };
  auto tiles_of = [&](int bm, int bn) {
    long t = 0;
    for (int i = 0; i < n; ++i) t += (long)((g[i].M + bm - 1) / bm) * ((g[i].N + bn - 1) / bn);
    return t;
  };
  // Few tiles: at most one 32 x 64 (with the norm 32 x 128) tile per CU.  Through
  // the entry point, small kernel against 32 x 128 tiles with four slices in
  // LDS: 48 tiles, K = 3072 30.3 / 30.7 us; 80, K = 1920 24.8 / 25.6; 96, K = 256 16.0 /
  // 17.9; 256, K = 1024 22.1 / 21.9; past one per CU 288, K = 3072 46 / 31, 384, K = 1024
  // 25.7 / 21.8.  (K that is no multiple of 64 leaves the register-staged kernel.)
  {
    const int c = kSmallCfg + (rms ? 1 : 0);
    bool one_chain = false;
    for (int i = 0; i < n; ++i) one_chain |= g[i].one_chain;
    if (epi_ok && !one_chain && tiles_of(kCfgs[c].bm, kCfgs[c].bn) <= n_cu) return c;
  }
  // K <= 256: the tile writes dominate, more workgroups stream better
  bool shallow = tiles_of(128, 128) >= n_cu;
  for (int i = 0; i < n; ++i) shallow &= g[i].K <= 256 && g[i].M >= 512;
  if (shallow)
    for (int c = 0; c < kSmallCfg; ++c)
      if (kCfgs[c].bm == 128 && kCfgs[c].bn == 128 && admits(kCfgs[c])) return c;
  int best = -1;
  double best_t = 1e300;
  for (int c = 0; c < kSmallCfg; ++c) {
    const Cfg& k = kCfgs[c];
    if (!admits(k)) continue;
    const long tiles = tiles_of(k.bm, k.bn);
    const long slots = (long)n_cu * k.wg_per_cu;
    double rounds = (double)((tiles + slots - 1) / slots);
    if (c == 0 && ws)
      if (const int parts = ring_parts(tiles, g, n, n_cu))
        rounds = tiles / n_cu + 1.0 / parts + 17.0 * 64 / g[0].K;  // 20 us in slices
    const double t = rounds * k.bm * k.bn * k.wg_per_cu / k.eff;
    if (t < best_t) { best_t = t; best = c; }
  }
  return best;
}

}  // namespace

hipError_t launch_proj_small_n(const void* A, int64_t lda, const void* W, int64_t ldw, const void* bias,
                               float* out, int64_t ldo, float* x, int64_t ldx, float alpha, int M, int N,
                               int K, int n_cu, hipStream_t s) {
  if (K % 32 || N % 16 || N > 128 || M < 1) return hipErrorInvalidValue;
  // 32 rows a work-group where those still give every CU two of them
  const bool two = M >= 32 * 2 * n_cu;
  const dim3 grid((M + (two ? 31 : 15)) / (two ? 32 : 16));
#define DIT_PROJ(NT_)                                                                                  \
  case NT_:                                                                                            \
    hipLaunchKernelGGL((two ? proj_small_n_kernel<NT_, 2> : proj_small_n_kernel<NT_, 1>), grid,        \
                       dim3(512), 0, s, (const bf16_t*)A, lda, (const bf16_t*)W, ldw,                  \
                       (const bf16_t*)bias, out, ldo, x, ldx, alpha, M, K);                            \
    break;
  switch (N / 16) {
    DIT_PROJ(1) DIT_PROJ(2) DIT_PROJ(3) DIT_PROJ(4) DIT_PROJ(5) DIT_PROJ(6) DIT_PROJ(7) DIT_PROJ(8)
    default:
      return hipErrorInvalidValue;
  }
#undef DIT_PROJ
  return hipGetLastError();
}

// The kernel for these problems (config c): the 256 x 256 ring kernel takes
// a specialised epilogue when every problem admits it.
static void (*kernel_for(const GemmArgs* g, int n, int c))(Batch) {
  void (*fn)(Batch) = kCfgs[c].fn;
  if (fn == gemm_bf16_ring_kernel<EPI_K_ANY>) {
    bool store = true, gated = true;
    for (int i = 0; i < n; ++i) {
      const GemmArgs& a = g[i];
      const bool plain = !(a.flags & (DIT_EPI_F32 | DIT_EPI_SILU));
      store &= plain && !(a.flags & DIT_EPI_GATED_RES) && (a.gelu_from >= a.N || a.gelu_from % 128 == 0) &&
               (a.gap == 0 || a.gap_at % 128 == 0);
      gated &= plain && (a.flags & DIT_EPI_GATED_RES) && a.rms_cols == 0 && a.gelu_from >= a.N && a.gap == 0;
    }
    if (store) fn = gemm_bf16_ring_kernel<EPI_K_STORE>;
    else if (gated) fn = gemm_bf16_ring_kernel<EPI_K_GATED>;
  }
  return fn;
}

// The transposed-value output: the store kernel, head groups inside the
// output, no column gap or GELU or RMS over them, 32-row aligned segments
// and key offsets, and 16-byte aligned rows of vt.
static bool vt_ok(const GemmArgs* g, int n, int c) {
  if (c < 0 || kernel_for(g, n, c) != gemm_bf16_ring_kernel<EPI_K_STORE>) return false;
  for (int i = 0; i < n; ++i) {
    const GemmArgs& a = g[i];
    if (!a.vt) continue;
    const int end = a.vt_col0 + 128 * a.vt_heads;
    if (a.vt_heads < 1 || a.vt_col0 % 128 || end > a.N || a.vt_ld % 8 || ((uintptr_t)a.vt & 15)) return false;
    if (a.vt_col0 < a.rms_cols || end > a.gelu_from || (a.gap && end > a.gap_at)) return false;
    // one sequence in one piece may end inside a 32-row block: that block's
    // rows past M repeat row M - 1 (clamped loads), so the keys it writes past
    // the sequence hold finite values that attention masks out
    const bool single = a.vt_split >= a.M && a.vt_rows0 >= a.M;
    if (single) {
      if (a.vt_key0 % 32 || a.vt_key0 + (a.M + 31) / 32 * 32 > a.vt_ld) return false;
    } else if (a.M % 32 || a.vt_rows0 % 32 || a.vt_key0 % 32 || a.vt_rows0 < 1) {
      return false;
    }
    if (a.vt_split < a.M && (a.vt_split % 32 || a.vt_rows1 % 32 || a.vt_key1 % 32 || a.vt_rows1 < 1)) return false;
  }
  return true;
}

bool gemm_bf16_fuses_vt(const GemmArgs* g, int n, int n_cu) {
  if (n < 1 || n > 2) return false;
  return vt_ok(g, n, pick_cfg(g, n, n_cu, true));
}

bool gemm_bf16_uses_ws(const GemmArgs* g, int n, int n_cu) {
  if (pick_cfg(g, n, n_cu, true) != 0) return false;
  long tiles = 0;
  for (int i = 0; i < n; ++i) tiles += (long)((g[i].M + 255) / 256) * ((g[i].N + 255) / 256);
  return ring_parts(tiles, g, n, n_cu) > 0;
}

size_t gemm_bf16_ws_bytes(int n_cu) { return (size_t)n_cu * 8 * PIECE_WAVE * sizeof(float); }

hipError_t launch_gemm_bf16(const GemmArgs* g, int n, hipStream_t stream, int n_cu, float* ws) {
  if (n < 1 || n > 2) return hipErrorInvalidValue;
  for (int i = 0; i < n; ++i)
    if (g[i].gseg < 0 || (g[i].gseg > 0 && (g[i].gseg % 32 || !(g[i].flags & DIT_EPI_GATED_RES))))
      return hipErrorInvalidValue;
  const int c = pick_cfg(g, n, n_cu, ws != nullptr);
  if (c < 0) return hipErrorInvalidValue;
  bool want_vt = false;
  for (int i = 0; i < n; ++i) want_vt |= g[i].vt != nullptr;
  if (want_vt && !vt_ok(g, n, c)) return hipErrorInvalidValue;
  const Cfg& k = kCfgs[c];
  void (*fn)(Batch) = kernel_for(g, n, c);
  Batch b;
  b.p0 = make_prob(g[0], k.bm, k.bn);
  b.p1 = n > 1 ? make_prob(g[1], k.bm, k.bn) : b.p0;
  b.tiles0 = b.p0.tiles_m * b.p0.tiles_n;
  b.total = b.tiles0 + (n > 1 ? b.p1.tiles_m * b.p1.tiles_n : 0);
  if (b.total == 0) return hipSuccess;
  b.whole = b.total;
  b.parts = 1;
  b.ws = ws;
  int rem = 0;
  if (c == 0 && ws)
    if (const int parts = ring_parts(b.total, g, n, n_cu)) {
      rem = b.total % n_cu;
      b.parts = parts;
      b.whole = b.total - rem;
      b.total = b.whole + rem * parts;
    }
  hipLaunchKernelGGL(fn, dim3(b.total), dim3(k.threads), 0, stream, b);
  if (rem) {
    void (*fin)(Batch) = fn == gemm_bf16_ring_kernel<EPI_K_STORE>   ? gemm_finish_kernel<EPI_K_STORE>
                         : fn == gemm_bf16_ring_kernel<EPI_K_GATED> ? gemm_finish_kernel<EPI_K_GATED>
                                                                    : gemm_finish_kernel<EPI_K_ANY>;
    hipLaunchKernelGGL(fin, dim3(8 * rem), dim3(64), 0, stream, b);
  }
  return hipGetLastError();
}

}  // namespace dit
