// Dense projections of the scoring pass on the bf16 contraction of gemm_tile.h: the output
// projection of the fast variant (y = x W^T), and those of a full layer with their epilogues:
// W_q with the rotary embedding, gate/up with SwiGLU, and W_o and W_down into the fp32
// residual stream.
#include <algorithm>

#include "gemm_tile.h"

namespace cc {
namespace {

// y[n][m] in bf16, n an entry, m a feature.
template <int MB, int NB>
struct EpiStore {
  u16* out;
  int vec;   // 8-byte stores: rows start on 8-byte boundaries
  __device__ void operator()(const f32x4 (&acc)[MB][NB], const TileArgs& g, int, int, int m0w,
                             int n0w, int lane, char*) const {
    const int grp = lane >> 4, c = lane & 15;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const int n = n0w + b * 16 + c;
      if (n >= g.N) continue;
      u16* row = out + int64_t(n) * g.M;
#pragma unroll
      for (int a = 0; a < MB; ++a) {
        const int m = m0w + a * 16 + grp * 4;
        if (vec) {
          if (m < g.M)
            *reinterpret_cast<uint2*>(row + m) = make_uint2(pack_bf2(acc[a][b][0], acc[a][b][1]),
                                                            pack_bf2(acc[a][b][2], acc[a][b][3]));
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (m + e < g.M) row[m + e] = f2bf(acc[a][b][e]);
        }
      }
    }
  }
};

// The bf16 results of a wave's pairs.  w[a] holds this lane's two results of block a (pairs
// 8 a + 2 grp, + 1): two blocks exchange lane groups so that a lane stores four consecutive
// results, 8 bytes (block a + (grp & 1), results 4 (grp >> 1) ..); a last odd block goes out
// 4 bytes a lane.  at(i): where the 8 results of block i go.
template <int MB, class At>
__device__ __forceinline__ void store_pairs(const uint32_t (&w)[MB], int grp, At at) {
#pragma unroll
  for (int a = 0; a + 1 < MB; a += 2) {
    const auto x = __builtin_amdgcn_permlane16_swap(w[a], w[a + 1], false, false);
    u16* p = at(a + (grp & 1));
    if (p) *reinterpret_cast<uint2*>(p + 4 * (grp >> 1)) = make_uint2(x[0], x[1]);
  }
  if constexpr (MB % 2 != 0) {
    u16* p = at(MB - 1);
    if (p) *reinterpret_cast<uint32_t*>(p + 2 * grp) = w[MB - 1];
  }
}

// Query projection: pairs (e, e + 64) of a head rotated to the entry's position, q[n][M] bf16.
template <int MB, int NB>
struct EpiRope {
  u16* out;
  const float2* rot;   // [N][64] (cos, sin) of position * theta^(-2e/128)
  __device__ void operator()(const f32x4 (&acc)[MB][NB], const TileArgs& g, int, int, int m0w,
                             int n0w, int lane, char*) const {
    const int grp = lane >> 4, c = lane & 15;
    const int p0 = m0w / 2, np = g.M / 2;   // pair of block 0, pairs in all
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const int n = n0w + b * 16 + c, nr = min(n, g.N - 1);
      uint32_t lo[MB], up[MB];
#pragma unroll
      for (int a = 0; a < MB; ++a) {
        const float4 cs = *reinterpret_cast<const float4*>(rot + int64_t(nr) * 64 + ((p0 + a * 8) & 63) + 2 * grp);
        const f32x4 v = acc[a][b];
        lo[a] = pack_bf2(v[0] * cs.x - v[2] * cs.y, v[1] * cs.z - v[3] * cs.w);
        up[a] = pack_bf2(v[2] * cs.x + v[0] * cs.y, v[3] * cs.z + v[1] * cs.w);
      }
      u16* row = out + int64_t(n) * g.M;
      auto at = [&](int a) -> u16* {
        const int p = p0 + a * 8;
        return n < g.N && p < np ? row + (p >> 6) * 128 + (p & 63) : nullptr;
      };
      store_pairs<MB>(lo, grp, at);
      store_pairs<MB>(up, grp, [&](int a) -> u16* { u16* p = at(a); return p ? p + 64 : nullptr; });
    }
  }
};

// act[n][f] = silu(gate) * up, bf16.
template <int MB, int NB>
struct EpiSwiglu {
  u16* act;
  __device__ void operator()(const f32x4 (&acc)[MB][NB], const TileArgs& g, int, int, int m0w,
                             int n0w, int lane, char*) const {
    const int grp = lane >> 4, c = lane & 15;
    const int f0 = m0w / 2, F = g.M / 2;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const int n = n0w + b * 16 + c;
      uint32_t w[MB];
#pragma unroll
      for (int a = 0; a < MB; ++a) {
        const f32x4 v = acc[a][b];
        w[a] = pack_bf2(v[0] / (1.f + expf(-v[0])) * v[2], v[1] / (1.f + expf(-v[1])) * v[3]);
      }
      u16* row = act + int64_t(n) * F;
      store_pairs<MB>(w, grp, [&](int a) -> u16* {
        const int f = f0 + a * 8;
        return n < g.N && f < F ? row + f : nullptr;
      });
    }
  }
};

// h[n][m] += acc, the fp32 residual stream (M a multiple of 4).
template <int MB, int NB>
struct EpiResidual {
  float* h;
  __device__ void operator()(const f32x4 (&acc)[MB][NB], const TileArgs& g, int, int, int m0w,
                             int n0w, int lane, char*) const {
    const int grp = lane >> 4, c = lane & 15;
    // two blocks of residual values are loaded together (rows and columns clamped, so no load
    // is conditional): one memory round trip for 2 NB 16-byte values instead of one each
#pragma unroll
    for (int a0 = 0; a0 < MB; a0 += 2) {
      float4 r[2][NB];
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int b = 0; b < NB; ++b) {
          const int n = min(n0w + b * 16 + c, g.N - 1), m = min(m0w + (a0 + i) * 16 + grp * 4, g.M - 4);
          if (a0 + i < MB) r[i][b] = *reinterpret_cast<const float4*>(h + int64_t(n) * g.M + m);
        }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int b = 0; b < NB; ++b) {
          const int a = a0 + i;
          if (a >= MB) continue;
          const int n = n0w + b * 16 + c, m = m0w + a * 16 + grp * 4;
          if (n < g.N && m < g.M)
            *reinterpret_cast<float4*>(h + int64_t(n) * g.M + m) =
                make_float4(r[i][b].x + acc[a][b][0], r[i][b].y + acc[a][b][1],
                            r[i][b].z + acc[a][b][2], r[i][b].w + acc[a][b][3]);
        }
    }
  }
};

// Split-K: the fp32 sums of one slice of K, part[slice][n][m] (M a multiple of 4).
template <int MB, int NB>
struct EpiPartial {
  float* part;
  __device__ void operator()(const f32x4 (&acc)[MB][NB], const TileArgs& g, int, int sl, int m0w,
                             int n0w, int lane, char*) const {
    const int grp = lane >> 4, c = lane & 15;
    float* p = part + int64_t(sl) * g.M * g.N;
#pragma unroll
    for (int a = 0; a < MB; ++a)
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        const int n = n0w + b * 16 + c, m = m0w + a * 16 + grp * 4;
        if (n < g.N && m < g.M)
          *reinterpret_cast<float4*>(p + int64_t(n) * g.M + m) =
              make_float4(acc[a][b][0], acc[a][b][1], acc[a][b][2], acc[a][b][3]);
      }
  }
};

// Tile shapes (MB, NB, SA, SB): the rings as deep as 160 KB allow.
struct Shape {
  int mb, nb;
};
constexpr Shape kShapes[] = {{8, 4}, {7, 4}, {5, 4}, {4, 4}, {8, 3}, {6, 2}, {4, 2}, {2, 2}, {4, 1}, {2, 1}};
constexpr int kNShapes = int(sizeof(kShapes) / sizeof(kShapes[0]));

// The tile shape and the number of K slices of an M x N x K product, by estimated time.  A
// workgroup's k-tile takes the longer of its matrix work (7 TFLOP/s a CU) and its loads
// (80 GB/s a CU out of the caches), a workgroup 4 us more for its first loads and its
// epilogue, and the CU that has the most workgroups decides; slices add their fp32 partial
// sums, written and read again at 5 TB/s, and a reduce kernel.  Fitted to 1805 timings of
// M 3584 .. 37888, N 256 .. 4096, K 3584 .. 18944 with 12 shapes and 1 .. 12 slices, cold
// weights: the shape it picks is on average 0.5% and at most 7% slower than the best one.
// Examples, 256 x 256 tiles (5 slices at most) against the picked shape: 3584 x 512 x 3584,
// 40 us (32 and its reduce) against 26; 37888 x 512 x 3584 (296 tiles: a second wave of 40)
// 192 against 128; 3584 x 512 x 18944 109 against 82.
struct TilePlan {
  int shape, slices;
};
TilePlan plan_tiles(int M, int N, int K, bool may_split) {
  const int64_t nk = K / 64;
  TilePlan best{0, 1};
  if (M == 0 || N == 0) return best;   // an empty cache: no tiles
  double best_us = 1e300;
  for (int i = 0; i < kNShapes; ++i) {
    const int tm = 32 * kShapes[i].mb, tn = 64 * kShapes[i].nb;
    const int64_t tiles = ((int64_t(M) + tm - 1) / tm) * ((int64_t(N) + tn - 1) / tn);
    const double ktile = std::max(tm * tn * 128e-6 / 7.0, (tm + tn) * 0.128 / 80.0);
    const int most = may_split ? int(std::min<int64_t>({12, nk / 4, 1024 / tiles})) : 1;
    for (int s = 1; s <= std::max(1, most); ++s) {
      const int64_t kt = (nk + s - 1) / s;
      if (s > 1 && (nk + kt - 1) / kt != s) continue;   // the same as fewer slices
      const int64_t rounds = ((tiles * s + 7) / 8 + 31) / 32;
      const double mb = double(M) * N * 4e-6;
      const double us = double(rounds) * (double(kt) * ktile + 4.0) + (s > 1 ? 5.0 + (s + 2) * mb / 5.0 : 0.0);
      if (us < best_us) {
        best_us = us;
        best = {i, s};
      }
    }
  }
  return best;
}

template <int AM, template <int, int> class Epi, class... E>
hipError_t launch_shape(const TilePlan& p, const TileArgs& g, hipStream_t s, E... e) {
  if (g.K >= kWideRow) return launch_tile<4, 4, 4, 3, AM, true>(g, Epi<4, 4>{e...}, p.slices, s);
  switch (p.shape) {
    case 0: return launch_tile<8, 4, 3, 2, AM>(g, Epi<8, 4>{e...}, p.slices, s);
    case 1: return launch_tile<7, 4, 3, 2, AM>(g, Epi<7, 4>{e...}, p.slices, s);
    case 2: return launch_tile<5, 4, 3, 3, AM>(g, Epi<5, 4>{e...}, p.slices, s);
    case 3: return launch_tile<4, 4, 4, 3, AM>(g, Epi<4, 4>{e...}, p.slices, s);
    case 4: return launch_tile<8, 3, 3, 2, AM>(g, Epi<8, 3>{e...}, p.slices, s);
    case 5: return launch_tile<6, 2, 4, 4, AM>(g, Epi<6, 2>{e...}, p.slices, s);
    case 6: return launch_tile<4, 2, 5, 5, AM>(g, Epi<4, 2>{e...}, p.slices, s);
    case 7: return launch_tile<2, 2, 6, 6, AM>(g, Epi<2, 2>{e...}, p.slices, s);
    case 8: return launch_tile<4, 1, 6, 6, AM>(g, Epi<4, 1>{e...}, p.slices, s);
    default: return launch_tile<2, 1, 8, 8, AM>(g, Epi<2, 1>{e...}, p.slices, s);
  }
}

TileArgs make_args(const void* w, const void* x, int M, int N, int K) {
  TileArgs g{};
  g.A = static_cast<const u16*>(w);
  g.B = static_cast<const u16*>(x);
  g.M = M;
  g.N = N;
  g.K = K;
  return g;
}

}  // namespace

hipError_t launch_linear(int dtype, const void* x, const void* w, void* y, int M, int N, int K,
                         hipStream_t s) {
  if (M == 0 || N == 0) return hipSuccess;
  if (dtype != CC_BF16)
    return launch_linear_f32(static_cast<const float*>(x), static_cast<const float*>(w),
                             static_cast<float*>(y), M, N, K, s);
  const int vec = N % 4 == 0 && (reinterpret_cast<uintptr_t>(y) & 7u) == 0;
  return launch_shape<A_ROWS, EpiStore>(plan_tiles(N, M, K, false), make_args(w, x, N, M, K), s,
                                        static_cast<u16*>(y), vec);
}

int gemm_split_slices(int M, int N, int K) { return plan_tiles(N, M, K, true).slices; }

hipError_t launch_qproj_rope(const void* wq, const void* a, void* q, const float2* rot, int N,
                             int D, int HD, hipStream_t s) {
  if (N == 0) return hipSuccess;
  return launch_shape<A_ROPE, EpiRope>(plan_tiles(HD, N, D, false), make_args(wq, a, HD, N, D), s,
                                       static_cast<u16*>(q), rot);
}

hipError_t launch_linear_residual_norm(const void* x, const void* w, float* h, const void* gamma,
                                       void* y, int M, int N, int K, float eps, float* part,
                                       hipStream_t s) {
  if (M == 0) return hipSuccess;
  const TilePlan p = plan_tiles(N, M, K, true);
  const TileArgs g = make_args(w, x, N, M, K);
  hipError_t err = p.slices > 1 ? launch_shape<A_ROWS, EpiPartial>(p, g, s, part)
                                : launch_shape<A_ROWS, EpiResidual>(p, g, s, h);
  if (err != hipSuccess) return err;
  return launch_residual_rmsnorm(p.slices > 1 ? part : nullptr, p.slices, h, gamma, y, M, N, eps, s);
}

hipError_t launch_gate_up_swiglu(const void* w_gate, const void* w_up, const void* b, void* act,
                                 int N, int D, int F, hipStream_t s) {
  if (N == 0) return hipSuccess;
  TileArgs g = make_args(w_gate, b, 2 * F, N, D);
  g.A2 = static_cast<const u16*>(w_up);
  return launch_shape<A_GATED, EpiSwiglu>(plan_tiles(2 * F, N, D, false), g, s, static_cast<u16*>(act));
}

}  // namespace cc
