// Elementwise steps of the full counter-causal pass (Sec. 3.1: every layer runs with fresh
// queries at the original position ids against the stored keys/values): the embedding
// gather into the fp32 residual stream, RMSNorm to the bf16 GEMM input, and the rotary
// angle table.  The GEMMs (with RoPE / residual / SwiGLU epilogues) live in projections.hip.
#include <type_traits>

#include "cc_internal.h"

namespace cc {
namespace {

// One entry's row: h = x (+ part[0] + ... + part[S - 1], in slice order: the row is read once for
// the sum of a split projection and the norm), y = bf16(RMSNorm(h) gamma).  EMBED: x is row ids[n]
// (n without ids) of a bf16 matrix, else h itself.  A few KB a workgroup: its length is its round
// trips to memory, so a thread's U pieces of 4, with all their slices, are loaded at once and stay
// in registers between the two halves.  (From a loop over the pieces, with the row read again for
// the second half: 512 rows of 3584 with 8 slices 16.6 -> 13.2 us, without slices 5.3 -> 5.1.)
template <int NT, int U, bool EMBED>
__device__ __forceinline__ void norm_row(int n, const u16* __restrict__ embed, const int32_t* __restrict__ ids,
                                         const float* __restrict__ part, int S, int64_t count,
                                         float* __restrict__ h, const u16* __restrict__ gamma,
                                         u16* __restrict__ y, int D, float eps) {
  __shared__ float wsum[NT / 64];
  float* x = h + int64_t(n) * D;
  const u16* row = EMBED ? embed + int64_t(ids ? ids[n] : n) * D : nullptr;
  float4 v[U];
  uint2 gm[U];
  int at[U];   // clamped: loads need no branch, and what lies past the row is not used
#pragma unroll
  for (int u = 0; u < U; ++u) {
    at[u] = min((u * NT + int(threadIdx.x)) * 4, D - 4);
    gm[u] = *reinterpret_cast<const uint2*>(gamma + at[u]);
    if constexpr (EMBED) {
      const uint2 w = *reinterpret_cast<const uint2*>(row + at[u]);
      v[u].x = __uint_as_float(w.x << 16);
      v[u].y = __uint_as_float(w.x & 0xffff0000u);
      v[u].z = __uint_as_float(w.y << 16);
      v[u].w = __uint_as_float(w.y & 0xffff0000u);
    } else {
      v[u] = *reinterpret_cast<const float4*>(x + at[u]);
    }
  }
  if (!EMBED && part) {
    const float* p = part + int64_t(n) * D;
    float4 t[U];
#pragma unroll
    for (int u = 0; u < U; ++u) t[u] = *reinterpret_cast<const float4*>(p + at[u]);
#pragma unroll 4
    for (int sl = 1; sl < S; ++sl) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const float4 w = *reinterpret_cast<const float4*>(p + sl * count + at[u]);
        t[u].x += w.x;
        t[u].y += w.y;
        t[u].z += w.z;
        t[u].w += w.w;
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      v[u].x += t[u].x;
      v[u].y += t[u].y;
      v[u].z += t[u].z;
      v[u].w += t[u].w;
    }
  }
  float ss = 0.f;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    if ((u * NT + int(threadIdx.x)) * 4 < D) {
      if (EMBED || part) *reinterpret_cast<float4*>(x + at[u]) = v[u];
      ss += v[u].x * v[u].x + v[u].y * v[u].y + v[u].z * v[u].z + v[u].w * v[u].w;
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) ss += __shfl_xor(ss, off);
  if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = ss;
  __syncthreads();
  float tot = 0.f;
#pragma unroll
  for (int w = 0; w < NT / 64; ++w) tot += wsum[w];
  const float r = rsqrtf(tot / float(D) + eps);
  u16* out = y + int64_t(n) * D;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int i = (u * NT + int(threadIdx.x)) * 4;
    if (i < D) {
      const float g0 = __uint_as_float(gm[u].x << 16), g1 = __uint_as_float(gm[u].x & 0xffff0000u);
      const float g2 = __uint_as_float(gm[u].y << 16), g3 = __uint_as_float(gm[u].y & 0xffff0000u);
      uint2 o;
      o.x = pack_bf2(v[u].x * r * g0, v[u].y * r * g1);
      o.y = pack_bf2(v[u].z * r * g2, v[u].w * r * g3);
      *reinterpret_cast<uint2*>(out + i) = o;
    }
  }
}

// Rows beyond the registers of a workgroup: the pieces in a loop, read again for the second half
// (each thread reads only what it wrote).
constexpr int WNT = 1024;
template <bool EMBED>
__device__ __forceinline__ void norm_wide_row(int n, const u16* __restrict__ embed,
                                              const int32_t* __restrict__ ids, const float* __restrict__ part,
                                              int S, int64_t count, float* __restrict__ h,
                                              const u16* __restrict__ gamma, u16* __restrict__ y, int D,
                                              float eps) {
  __shared__ float wsum[WNT / 64];
  float* x = h + int64_t(n) * D;
  const u16* row = EMBED ? embed + int64_t(ids ? ids[n] : n) * D : nullptr;
  float ss = 0.f;
  for (int i = threadIdx.x; i < D; i += WNT) {
    float v = EMBED ? bf2f(row[i]) : x[i];
    if (!EMBED && part) {
      const float* p = part + int64_t(n) * D + i;
      float t = p[0];
      for (int sl = 1; sl < S; ++sl) t += p[sl * count];
      v += t;
    }
    if (EMBED || part) x[i] = v;
    ss += v * v;
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) ss += __shfl_xor(ss, off);
  if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = ss;
  __syncthreads();
  float tot = 0.f;
#pragma unroll
  for (int w = 0; w < WNT / 64; ++w) tot += wsum[w];
  const float r = rsqrtf(tot / float(D) + eps);
  for (int i = threadIdx.x; i < D; i += WNT) y[int64_t(n) * D + i] = f2bf(x[i] * r * bf2f(gamma[i]));
}

template <int NT, int U>
__global__ __launch_bounds__(NT) void rmsnorm_kernel(const float* __restrict__ part, int S,
                                                     float* __restrict__ h, const u16* __restrict__ gamma,
                                                     u16* __restrict__ y, int D, float eps) {
  const int64_t count = int64_t(gridDim.x) * D;
  if constexpr (U > 0)
    norm_row<NT, U, false>(int(blockIdx.x), nullptr, nullptr, part, S, count, h, gamma, y, D, eps);
  else
    norm_wide_row<false>(int(blockIdx.x), nullptr, nullptr, part, S, count, h, gamma, y, D, eps);
}

// One thread per (entry, frequency).  The angle is formed and reduced in fp64 so large
// positions keep full fp32 accuracy in cos/sin.
struct RopeArgs {
  const int32_t* pos;
  const int32_t* cu;
  int n_seqs, N, half, head_dim;
  double theta;
  float2* rot;
};
__device__ __forceinline__ void rope_angle(const RopeArgs& a, int64_t idx) {
  if (idx >= int64_t(a.N) * a.half) return;
  const int n = int(idx / a.half), e = int(idx % a.half);
  int p;
  if (a.pos) {
    p = a.pos[n];
  } else {
    int lo = 0, hi = a.n_seqs - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (a.cu[mid] <= n) lo = mid; else hi = mid - 1;
    }
    p = n - a.cu[lo];
  }
  const double inv = pow(a.theta, -2.0 * double(e) / double(a.head_dim));
  double sn, cs;
  sincos(double(p) * inv, &sn, &cs);
  a.rot[idx] = make_float2(float(cs), float(sn));
}

// What a pass does before its first projection, in one launch: the rotary table (the first
// rope_blocks workgroups) and, for every entry, the row's gather into the residual stream and its
// first norm.  512 entries of 3584: 6.9 us, 15.4 in three launches; 768: 8.2 and 18.
template <int NT, int U>
__global__ __launch_bounds__(NT) void enter_kernel(RopeArgs rope, int rope_blocks,
                                                   const u16* __restrict__ embed,
                                                   const int32_t* __restrict__ ids, float* __restrict__ h,
                                                   const u16* __restrict__ gamma, u16* __restrict__ y, int D,
                                                   float eps) {
  if (int(blockIdx.x) < rope_blocks)
    rope_angle(rope, int64_t(blockIdx.x) * NT + threadIdx.x);
  else if constexpr (U > 0)
    norm_row<NT, U, true>(int(blockIdx.x) - rope_blocks, embed, ids, nullptr, 0, 0, h, gamma, y, D, eps);
  else
    norm_wide_row<true>(int(blockIdx.x) - rope_blocks, embed, ids, nullptr, 0, 0, h, gamma, y, D, eps);
}

// Threads and pieces a thread (0: the loops) by the width of a row, so that no thread is without work.
template <class F>
hipError_t by_width(int D, F f) {
  using std::integral_constant;
  if (D <= 1024) return f(integral_constant<int, 256>{}, integral_constant<int, 1>{});
  if (D <= 4096) return f(integral_constant<int, 512>{}, integral_constant<int, 2>{});
  if (D <= 16384) return f(integral_constant<int, 1024>{}, integral_constant<int, 4>{});
  return f(integral_constant<int, WNT>{}, integral_constant<int, 0>{});
}

}  // namespace

hipError_t launch_enter(const void* embed, const int32_t* ids, const int32_t* pos, const int32_t* cu,
                        int n_seqs, float2* rot, float* h, const void* gamma, void* y, int N, int D,
                        int head_dim, double theta, float eps, hipStream_t s) {
  if (N == 0) return hipSuccess;
  const RopeArgs rope{pos, cu, n_seqs, N, head_dim / 2, head_dim, theta, rot};
  return by_width(D, [&](auto nt, auto u) {
    constexpr int NT = decltype(nt)::value, U = decltype(u)::value;
    const int rb = int((int64_t(N) * rope.half + NT - 1) / NT);
    hipLaunchKernelGGL((enter_kernel<NT, U>), dim3(unsigned(rb + N)), dim3(NT), 0, s, rope, rb,
                       static_cast<const u16*>(embed), ids, h, static_cast<const u16*>(gamma),
                       static_cast<u16*>(y), D, eps);
    return hipGetLastError();
  });
}

hipError_t launch_residual_rmsnorm(const float* part, int S, float* h, const void* gamma, void* y,
                                   int N, int D, float eps, hipStream_t s) {
  if (N == 0) return hipSuccess;
  return by_width(D, [&](auto nt, auto u) {
    constexpr int NT = decltype(nt)::value, U = decltype(u)::value;
    hipLaunchKernelGGL((rmsnorm_kernel<NT, U>), dim3(N), dim3(NT), 0, s, part, S, h,
                       static_cast<const u16*>(gamma), static_cast<u16*>(y), D, eps);
    return hipGetLastError();
  });
}

}  // namespace cc
