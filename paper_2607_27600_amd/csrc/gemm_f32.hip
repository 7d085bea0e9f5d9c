// fp32 contractions of the scoring pass (CC_F32 problems): y = x W^T and the LM head with
// its log-sum-exp reduced on the fly, as in lmhead.hip, on the 16x16x4 fp32 MFMA (plain fp32
// multiply-adds, twice the rate of the vector ALUs).
//
// C[m][n] = sum_k A[m][k] B[n][k], both operands K-contiguous.  A workgroup of four waves
// (2 x 2) owns a T x T tile; 32 columns of K at a time go through registers into LDS (rows
// of 36 floats: the 16-byte fragment reads of 16 rows hit every bank once), the next 32
// loaded while the current ones are multiplied.  A lane's 16-byte fragment is four
// consecutive k, one for each of four MFMA steps (both operands agree on which).
// Bound: launch and load latency for small problems, where 64 x 64 tiles leave most of the
// chip idle and 32 x 32 or (LM head) 64 x 32 ones are used instead; the fp32 MFMA rate beyond.
// Against 64 x 64 tiles on the vector ALUs with element-wise loads, a 256 x 128 x 128 product
// went from 19 to 4 us, a 1024 x 256 x 128 LM head from 25 to 6.4 us (9.7 in 64 x 64 tiles);
// scoring 2048 entries of 16 heads of 128 on a 32000 x 1024 head from 11.4 to 1.67 ms.
#include "cc_internal.h"

namespace cc {
namespace {

constexpr int FK = 32, FLD = FK + 4;
constexpr int LMT = 64;   // vocabulary rows per LM-head tile

struct GemmArgsF {
  const float* A;
  const float* B;
  int M, N, K;
  int tiles_n;
  int vec;   // rows of A and B start on 16-byte boundaries and K is a multiple of 4
};

__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// y[m][n], M = entries, N = output features.
struct EpiStoreF {
  float* out;
  template <int MB, int NB>
  __device__ void operator()(const f32x4 (&acc)[MB][NB], const GemmArgsF& g, int tm, int m0w,
                             int n0w, int lane, float* lds) const {
    (void)tm;
    (void)lds;
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        const int n = n0w + j * 16 + (lane & 15);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int m = m0w + i * 16 + 4 * (lane >> 4) + e;
          if (m < g.M && n < g.N) out[int64_t(m) * g.N + n] = acc[i][j][e];
        }
      }
  }
};

__device__ __forceinline__ void lse_merge(float& M, float& S, float m, float s) {
  const float t = fmaxf(M, m);
  if (t == -INFINITY) return;
  S = S * expf(M - t) + s * expf(m - t);
  M = t;
}

// M = vocabulary, N = entries: partial[tm * N + n] = (max, sum exp) over the tile's 64
// vocabulary rows; the lane that holds z[x_n] writes the target logit.
struct EpiLseF {
  float2* partial;
  float* target;
  const int32_t* ids;
  template <int MB, int NB>
  __device__ void operator()(const f32x4 (&acc)[MB][NB], const GemmArgsF& g, int tm, int m0w,
                             int n0w, int lane, float* lds) const {
    static_assert(32 * MB == LMT, "one tile, one partial");
    constexpr int T = 32 * NB;
    const int grp = lane >> 4, c16 = lane & 15, wave = threadIdx.x >> 6;
    float2* red = reinterpret_cast<float2*>(lds);   // [2][T]
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const int n = n0w + j * 16 + c16;
      const int id = n < g.N ? ids[n] : -1;
      float mx = -INFINITY, sm = 0.f;
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (m0w + i * 16 + 4 * grp + e < g.M) mx = fmaxf(mx, acc[i][j][e]);
      const float ref = mx == -INFINITY ? 0.f : mx;   // a lane without rows, or of -inf logits, adds 0
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int m = m0w + i * 16 + 4 * grp + e;
          if (m < g.M) {
            sm += expf(acc[i][j][e] - ref);
            if (m == id) target[n] = acc[i][j][e];
          }
        }
#pragma unroll
      for (int off = 16; off < 64; off <<= 1) {
        const float m2 = __shfl_xor(mx, off), s2 = __shfl_xor(sm, off);
        lse_merge(mx, sm, m2, s2);
      }
      if (grp == 0) red[(wave >> 1) * T + (wave & 1) * 16 * NB + j * 16 + c16] = make_float2(mx, sm);
    }
    __syncthreads();
    const int n = n0w - (wave & 1) * 16 * NB + threadIdx.x;   // tile column threadIdx.x
    if (threadIdx.x < T && n < g.N) {
      float2 a = red[threadIdx.x];
      const float2 b = red[T + threadIdx.x];
      lse_merge(a.x, a.y, b.x, b.y);
      partial[int64_t(tm) * g.N + n] = a;
    }
  }
};

// Tiles of 32 MB x 32 NB.
template <int MB, int NB, class Epi>
__global__ __launch_bounds__(256) void gemm_tn_f32(GemmArgsF g, Epi epi) {
  constexpr int TM = 32 * MB, TN = 32 * NB;   // MB, NB: also the float4 a thread loads of each operand
  __shared__ __attribute__((aligned(16))) float lds[(TM + TN) * FLD];
  float* As = lds;
  float* Bs = lds + TM * FLD;
  const int tm = blockIdx.x / g.tiles_n, tn = blockIdx.x % g.tiles_n;
  const int m0 = tm * TM, n0 = tn * TN;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int grp = lane >> 4, r16 = lane & 15;
  const int wm = wave >> 1, wn = wave & 1;
  float4 ra[MB], rb[NB];
  auto load1 = [&](const float* X, int row, int rows, int k) {
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    if (row >= rows) return v;
    const float* p = X + int64_t(row) * g.K + k;
    if (g.vec) {
      if (k < g.K) v = *reinterpret_cast<const float4*>(p);
    } else {
      if (k < g.K) v.x = p[0];
      if (k + 1 < g.K) v.y = p[1];
      if (k + 2 < g.K) v.z = p[2];
      if (k + 3 < g.K) v.w = p[3];
    }
    return v;
  };
  auto load = [&](int k0) {
#pragma unroll
    for (int i = 0; i < MB; ++i) ra[i] = load1(g.A, m0 + ((i * 256 + tid) >> 3), g.M, k0 + (tid & 7) * 4);
#pragma unroll
    for (int i = 0; i < NB; ++i) rb[i] = load1(g.B, n0 + ((i * 256 + tid) >> 3), g.N, k0 + (tid & 7) * 4);
  };
  f32x4 acc[MB][NB];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[i][j] = f32x4{};
  load(0);
  for (int k0 = 0; k0 < g.K; k0 += FK) {
    __syncthreads();
#pragma unroll
    for (int i = 0; i < MB; ++i)
      *reinterpret_cast<float4*>(As + ((i * 256 + tid) >> 3) * FLD + (tid & 7) * 4) = ra[i];
#pragma unroll
    for (int i = 0; i < NB; ++i)
      *reinterpret_cast<float4*>(Bs + ((i * 256 + tid) >> 3) * FLD + (tid & 7) * 4) = rb[i];
    __syncthreads();
    if (k0 + FK < g.K) load(k0 + FK);
#pragma unroll
    for (int ks = 0; ks < FK / 16; ++ks) {
      float4 fa[MB], fb[NB];
#pragma unroll
      for (int i = 0; i < MB; ++i)
        fa[i] = *reinterpret_cast<const float4*>(As + (wm * 16 * MB + i * 16 + r16) * FLD + ks * 16 + grp * 4);
#pragma unroll
      for (int i = 0; i < NB; ++i)
        fb[i] = *reinterpret_cast<const float4*>(Bs + (wn * 16 * NB + i * 16 + r16) * FLD + ks * 16 + grp * 4);
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) {
          acc[i][j] = mfma4(fa[i].x, fb[j].x, acc[i][j]);
          acc[i][j] = mfma4(fa[i].y, fb[j].y, acc[i][j]);
          acc[i][j] = mfma4(fa[i].z, fb[j].z, acc[i][j]);
          acc[i][j] = mfma4(fa[i].w, fb[j].w, acc[i][j]);
        }
    }
  }
  __syncthreads();
  epi(acc, g, tm, m0 + wm * 16 * MB, n0 + wn * 16 * NB, lane, lds);
}

GemmArgsF make_args(const float* a, const float* b, int M, int N, int K) {
  GemmArgsF g;
  g.A = a;
  g.B = b;
  g.M = M;
  g.N = N;
  g.K = K;
  g.vec = K % 4 == 0 && ((reinterpret_cast<uintptr_t>(a) | reinterpret_cast<uintptr_t>(b)) & 15u) == 0;
  return g;
}

int64_t tiles(int rows, int t) { return (int64_t(rows) + t - 1) / t; }

}  // namespace

int lmhead_f32_vocab_tile() { return LMT; }

hipError_t launch_linear_f32(const float* x, const float* w, float* y, int M, int N, int K,
                             hipStream_t s) {
  GemmArgsF g = make_args(x, w, M, N, K);
  EpiStoreF e{y};
  // below one 64 x 64 tile per CU the quarter tiles keep four times as many CUs busy
  if (tiles(M, 64) * tiles(N, 64) >= 256) {
    g.tiles_n = int(tiles(N, 64));
    hipLaunchKernelGGL((gemm_tn_f32<2, 2, EpiStoreF>), dim3(unsigned(tiles(M, 64) * g.tiles_n)),
                       dim3(256), 0, s, g, e);
  } else {
    g.tiles_n = int(tiles(N, 32));
    hipLaunchKernelGGL((gemm_tn_f32<1, 1, EpiStoreF>), dim3(unsigned(tiles(M, 32) * g.tiles_n)),
                       dim3(256), 0, s, g, e);
  }
  return hipGetLastError();
}

hipError_t launch_lmhead_f32(const LmHeadLaunch& a, hipStream_t s) {
  GemmArgsF g = make_args(static_cast<const float*>(a.w_lm), static_cast<const float*>(a.u), a.V,
                          a.N, a.D);
  EpiLseF e{a.partial, a.target, a.ids};
  // below one 64 x 64 tile per CU 32 entries a tile keep twice as many CUs busy, each with half
  // the chain of MFMAs (the partials stay those of 64 vocabulary rows)
  if (tiles(a.V, LMT) * tiles(a.N, 64) >= 256) {
    g.tiles_n = int(tiles(a.N, 64));
    hipLaunchKernelGGL((gemm_tn_f32<2, 2, EpiLseF>), dim3(unsigned(tiles(a.V, LMT) * g.tiles_n)),
                       dim3(256), 0, s, g, e);
  } else {
    g.tiles_n = int(tiles(a.N, 32));
    hipLaunchKernelGGL((gemm_tn_f32<2, 1, EpiLseF>), dim3(unsigned(tiles(a.V, LMT) * g.tiles_n)),
                       dim3(256), 0, s, g, e);
  }
  return hipGetLastError();
}

}  // namespace cc
