// The LM head of the scoring pass (Eq. (5) read as -log P): z = W_lm u for every cached entry,
// reduced on the fly to a per-(entry, 256-word vocabulary tile) pair (max z, sum exp(z - max));
// the lane that holds z[x_i] in its accumulators writes the target logit from them; a combine
// kernel turns these into logsumexp(z) - z[x_i].  The [N][V] logits never leave registers.
// The contraction is that of gemm_tile.h on bf16 rows, packed bf16 rows or E4M3 codes: the
// vocabulary is the MFMA row dimension, so a lane holds 4 MB logits of each of its entries
// and the reduction over the vocabulary is mostly in-lane.
// Also here: the packing of the weight, the E4M3 quantization and the transpose behind the
// W_o-folded weight.  The fp32 LM head is in gemm_f32.hip.
#include "gemm_tile.h"

namespace cc {
namespace {

constexpr int VT = 256;   // vocabulary rows per tile (MB = 8)

__device__ __forceinline__ uint4 ld16(const u16* p) { return *reinterpret_cast<const uint4*>(p); }

// Writes partial[tm * N + n] = (max, sumexp) over the workgroup's 256 vocabulary rows.  The
// epilogue runs while the matrix cores idle, so it is kept to one max and one exp-accumulate
// per logit; only workgroups on the vocabulary edge take the masked variant.  The four lane
// groups of an entry combine by shuffles, the two wave rows through LDS.
// Target gather: the cached token x_n of entry n lies in exactly one vocabulary tile, one
// wave row of it and one lane group; that lane writes target[n] = its accumulator for row
// x_n (times the scales below), so the target logit and the log-sum-exp come from the
// same accumulators.  The ids are loaded first and the selection runs only in waves where
// some lane owns a target (about 3% of them at a vocabulary of 128k).
// An FP8 LM head passes the dequantization scales: the logit is acc * sw * su[n]
// (su per entry, sw for the whole matrix); without them the factor is 1 and the
// arithmetic is unchanged.
template <int NB>
struct EpiLse {
  static constexpr int MB = VT / 32;
  float2* partial;
  float* target;               // [N] target logits z[x_n]
  const int32_t* ids;          // [N] cached token ids
  const float* su = nullptr;   // [N] per-entry scale, or null
  const float* sw = nullptr;   // [1] matrix scale (device), with su
  template <bool EDGE>
  __device__ __forceinline__ void reduce(const f32x4 (&acc)[MB][NB], int rows, int grp,
                                         const float (&f)[NB], float (&mx)[NB], float (&sm)[NB]) const {
#pragma unroll
    for (int b = 0; b < NB; ++b) mx[b] = -INFINITY;
#pragma unroll
    for (int a = 0; a < MB; ++a)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const bool ok = !EDGE || a * 16 + 4 * grp + e < rows;
#pragma unroll
        for (int b = 0; b < NB; ++b)
          if (ok) mx[b] = fmaxf(mx[b], acc[a][b][e]);
      }
    float mc[NB], c[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      // logits are acc * f (f >= 0), so their max is mx * f; a lane whose rows are all
      // past the edge keeps max = -inf and sum = 0
      if (mx[b] != -INFINITY) mx[b] *= f[b];
      mc[b] = mx[b] == -INFINITY ? 0.f : mx[b] * kLog2e;
      c[b] = kLog2e * f[b];
      sm[b] = 0.f;
    }
#pragma unroll
    for (int a = 0; a < MB; ++a)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const bool ok = !EDGE || a * 16 + 4 * grp + e < rows;
#pragma unroll
        for (int b = 0; b < NB; ++b)
          if (ok) sm[b] += fast_exp2(fmaf(acc[a][b][e], c[b], -mc[b]));
      }
  }
  __device__ void operator()(const f32x4 (&acc)[MB][NB], const TileArgs& g, int tm, int, int m0w,
                             int n0w, int lane, char* lds) const {
    const int grp = lane >> 4, c16 = lane & 15;
    const int wave = threadIdx.x >> 6, wm = wave >> 2, wn = wave & 3;
    float2* red = reinterpret_cast<float2*>(lds);   // [2][64 NB] pairs
    // target rows relative to this wave's first vocabulary row (loaded before the
    // reduction so their latency hides behind it)
    int rt[NB];
    float f[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const int n = min(n0w + b * 16 + c16, g.N - 1);
      rt[b] = ids[n] - m0w;
      f[b] = su ? sw[0] * su[n] : 1.f;
    }
    float mx[NB], sm[NB];
    if (tm * VT + VT <= g.M)
      reduce<false>(acc, 0, grp, f, mx, sm);
    else
      reduce<true>(acc, g.M - m0w, grp, f, mx, sm);
    // row r of the wave's 128 sits in block r / 16, element r % 4 of lane group (r / 4) % 4
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const int r = rt[b];
      const bool own = n0w + b * 16 + c16 < g.N && uint32_t(r) < uint32_t(16 * MB) && ((r >> 2) & 3) == grp;
      if (__any(own)) {
        const int idx = (r >> 4) * 4 + (r & 3);
        float z = 0.f;
#pragma unroll
        for (int a = 0; a < MB; ++a)
#pragma unroll
          for (int e = 0; e < 4; ++e) z = idx == a * 4 + e ? acc[a][b][e] : z;
        if (own) target[n0w + b * 16 + c16] = z * f[b];
      }
    }
    auto fold = [](float& M, float& S, float m2, float s2) {
      const float t = fmaxf(M, m2);
      S = t == -INFINITY ? 0.f : S * exp2f((M - t) * kLog2e) + s2 * exp2f((m2 - t) * kLog2e);
      M = t;
    };
#pragma unroll
    for (int b = 0; b < NB; ++b) {
#pragma unroll
      for (int off = 16; off < 64; off <<= 1) {
        const float m2 = __shfl_xor(mx[b], off), s2 = __shfl_xor(sm[b], off);
        fold(mx[b], sm[b], m2, s2);
      }
      if (grp == 0) red[(wm * 4 + wn) * 16 * NB + b * 16 + c16] = make_float2(mx[b], sm[b]);
    }
    __syncthreads();
    const int t = threadIdx.x, n = n0w - wn * 16 * NB + t;   // tile column t
    if (t < 64 * NB && n < g.N) {
      float2 p = red[t];
      const float2 q = red[64 * NB + t];
      fold(p.x, p.y, q.x, q.y);
      partial[int64_t(tm) * g.N + n] = p;
    }
  }
};

// Packed operand layout (cc_pack_lmhead): per 256-row tile and 32-column step one 16 KB block,
// row r of the tile at bytes 64 r .. 64 r + 63, its 16-byte chunk c (columns 8 c .. 8 c + 7 of
// the step) at chunk position c ^ ((r >> 1) & 3); rows past the last are zero.  The weight is
// then read in contiguous 1 KB runs instead of 128-byte row pieces, which matters where the
// weight's bytes bound the product (128256 x 4096 at 200 entries: 232 against 272 us; at 4096
// entries both take 2.99 ms).  The XOR keeps the 16-byte fragment reads free of bank conflicts.
constexpr int PK_ROWS = 256, PK_K = 32;
constexpr int PK_BLOCK = PK_ROWS * PK_K;          // elements per packed block (16 KB)

// One thread per 16-byte chunk; consecutive threads walk a row (reads of whole rows),
// each group of four writes the 64 bytes of one packed row.
__global__ __launch_bounds__(256) void pack_rows_kernel(const u16* __restrict__ x, int R,
                                                        int K, int64_t ldx, int64_t n_chunks,
                                                        u16* __restrict__ out) {
  const int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x;
  if (i >= n_chunks) return;
  const int nsteps = K / PK_K;
  const int c = int(i & 3);
  const int64_t rs = i >> 2;
  const int s = int(rs % nsteps);
  const int64_t row = rs / nsteps;
  const int r = int(row % PK_ROWS);
  const int64_t t = row / PK_ROWS;
  const uint4 v = row < R ? ld16(x + row * ldx + s * PK_K + c * 8) : make_uint4(0, 0, 0, 0);
  u16* dst = out + (t * nsteps + s) * PK_BLOCK + r * PK_K + ((c ^ ((r >> 1) & 3)) * 8);
  *reinterpret_cast<uint4*>(dst) = v;
}

// E4M3 quantization: amax = max |x| over a row (or the matrix), codes = E4M3(x * (448 /
// amax)) rounded to nearest even by the conversion instruction, scale = amax / 448 (fp32
// throughout; an all-zero row gives codes 0 and scale 0).  Rows are read four elements
// per load (8 bytes of bf16 or 16 bytes of fp32; cols is a multiple of 4).
struct Quad {
  float v[4];
};
template <class T>
__device__ __forceinline__ Quad ld4(const T* p);
template <>
__device__ __forceinline__ Quad ld4<u16>(const u16* p) {
  const uint2 u = *reinterpret_cast<const uint2*>(p);
  return Quad{{__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xffff0000u),
               __uint_as_float(u.y << 16), __uint_as_float(u.y & 0xffff0000u)}};
}
template <>
__device__ __forceinline__ Quad ld4<float>(const float* p) {
  const float4 f = *reinterpret_cast<const float4*>(p);
  return Quad{{f.x, f.y, f.z, f.w}};
}

__device__ __forceinline__ float block_max_256(float v, float* red) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = fmaxf(v, __shfl_xor(v, off));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  v = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
  __syncthreads();
  return v;
}

template <class T>
__device__ __forceinline__ float row_amax(const T* row, int cols, float* red) {
  float m = 0.f;
  for (int c = threadIdx.x * 4; c < cols; c += 1024) {
    const Quad q = ld4<T>(row + c);
    m = fmaxf(m, fmaxf(fmaxf(fabsf(q.v[0]), fabsf(q.v[1])), fmaxf(fabsf(q.v[2]), fabsf(q.v[3]))));
  }
  return block_max_256(m, red);
}

template <class T>
__device__ __forceinline__ void quantize_row(const T* row, int cols, float amax, uint8_t* q) {
  const float inv = amax > 0.f ? 448.f / amax : 0.f;
  uint32_t* out = reinterpret_cast<uint32_t*>(q);
  for (int c = threadIdx.x * 4; c < cols; c += 1024) {
    const Quad x = ld4<T>(row + c);
    int v = __builtin_amdgcn_cvt_pk_fp8_f32(x.v[0] * inv, x.v[1] * inv, 0, false);
    v = __builtin_amdgcn_cvt_pk_fp8_f32(x.v[2] * inv, x.v[3] * inv, v, true);
    out[c >> 2] = uint32_t(v);
  }
}

// one scale per row: a workgroup per row reads it twice (the second pass hits the cache)
template <class T>
__global__ __launch_bounds__(256) void quantize_rows_kernel(const T* __restrict__ x, int cols,
                                                            uint8_t* __restrict__ q,
                                                            float* __restrict__ scale) {
  __shared__ float red[4];
  const int64_t r = blockIdx.x;
  const float amax = row_amax<T>(x + r * cols, cols, red);
  if (threadIdx.x == 0) scale[r] = amax / 448.f;
  quantize_row<T>(x + r * cols, cols, amax, q + r * cols);
}

// one scale for the matrix: row maxima, their maximum, then the codes
template <class T>
__global__ __launch_bounds__(256) void row_amax_kernel(const T* __restrict__ x, int cols,
                                                       float* __restrict__ amax) {
  __shared__ float red[4];
  const float m = row_amax<T>(x + int64_t(blockIdx.x) * cols, cols, red);
  if (threadIdx.x == 0) amax[blockIdx.x] = m;
}

__global__ __launch_bounds__(1024) void max_reduce_kernel(const float* __restrict__ v, int64_t n,
                                                          float* __restrict__ out) {
  __shared__ float red[16];
  float m = 0.f;
  for (int64_t i = threadIdx.x; i < n; i += 1024) m = fmaxf(m, v[i]);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    float t = red[0];
    for (int w = 1; w < 16; ++w) t = fmaxf(t, red[w]);
    out[0] = t;
  }
}

template <class T>
__global__ __launch_bounds__(256) void quantize_matrix_kernel(const T* __restrict__ x, int cols,
                                                              const float* __restrict__ amax,
                                                              uint8_t* __restrict__ q,
                                                              float* __restrict__ scale) {
  const int64_t r = blockIdx.x;
  if (r == 0 && threadIdx.x == 0) scale[0] = amax[0] / 448.f;
  quantize_row<T>(x + r * cols, cols, amax[0], q + r * cols);
}

// ------------------------------------------------------------------ LSE combine

// One workgroup per E entries: thread (group gi, entry e) folds the vocabulary tiles gi, gi + 64,
// ... of entry e (E consecutive entries read 8 E contiguous bytes of a tile's row of partials; up
// to 512 tiles are eight loads per thread, all in flight at once), then the 64 groups are folded by
// shuffles within each wave and across the waves in LDS.  Bound by latency below some thousands of
// entries: a batch of eight is summed against one maximum (a fold tile by tile is a chain of as many
// exponentials), and few entries take E = 4, for four times the workgroups; beyond, E = 16 reads
// whole cache lines.  Fold tile by tile in E = 16 -> now: 512 entries of 594 tiles 9.4 -> 6.2 us,
// 200 entries of 501 tiles 8.6 -> 4.6, 4096 entries (E = 16) 10.0 -> 7.4.
// The groups fold in one order for either E (pairs, pairs of pairs, up to 16 groups, then the four
// sums), so that the scores of an entry are the same bits whatever the number of entries beside it.
constexpr int CMB_G = 64;

// (M, S) += (m, s): S is the sum of exponentials against the maximum M.
__device__ __forceinline__ void lse_fold(float& M, float& S, float m, float s) {
  const float t = fmaxf(M, m), ref = t == -INFINITY ? 0.f : t;
  S = fmaf(S, expf(M - ref), s * expf(m - ref));   // (written out: the contraction is part of the order)
  M = t;
}

// The same for Q pairs at once.
template <int Q>
__device__ __forceinline__ void lse_fold(float& M, float& S, const float2 (&p)[Q]) {
  float t = M;
#pragma unroll
  for (int q = 0; q < Q; ++q) t = fmaxf(t, p[q].x);
  const float ref = t == -INFINITY ? 0.f : t;
  float sum = S * expf(M - ref);
#pragma unroll
  for (int q = 0; q < Q; ++q) sum = fmaf(p[q].y, expf(p[q].x - ref), sum);
  S = sum;
  M = t;
}

template <int E>
__global__ __launch_bounds__(E * CMB_G) void lse_combine(const float2* partial, int n_tiles,
                                                         const float* target, const int32_t* cu,
                                                         int n_seqs, int n_frozen, int N,
                                                         float* scores, float* lse_out) {
  constexpr int NWV = E * CMB_G / 64;
  __shared__ float2 red[NWV][E];
  const int e = threadIdx.x % E, gi = threadIdx.x / E;
  const int n = blockIdx.x * E + e;
  const bool writer = gi == 0 && n < N;
  float z = 0.f;
  bool none = false;   // the sequence's last entry, or a frozen one: no score
  if (writer) {
    z = target[n];
    // sequence of entry n: the last b with cu[b] <= n
    int lo = 0, hi = n_seqs - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (cu[mid] <= n) lo = mid; else hi = mid - 1;
    }
    none = n == cu[lo + 1] - 1 || n - cu[lo] < n_frozen;
  }
  float M = -INFINITY, S = 0.f;
  if (n < N) {
    // eight independent loads in flight per thread (tiles past the end fold as empty)
    for (int t0 = gi; t0 < n_tiles; t0 += 8 * CMB_G) {
      float2 p[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const int t = t0 + q * CMB_G;
        p[q] = t < n_tiles ? partial[int64_t(t) * N + n] : make_float2(-INFINITY, 0.f);
      }
      lse_fold(M, S, p);
    }
  }
  // the groups of an entry within a wave fold by shuffles, then the waves' results through LDS
#pragma unroll
  for (int off = E; off < 64; off <<= 1) {
    const float m2 = __shfl_xor(M, off), s2 = __shfl_xor(S, off);
    lse_fold(M, S, m2, s2);
  }
  if ((threadIdx.x & 63) < E) red[threadIdx.x >> 6][e] = make_float2(M, S);
  __syncthreads();
  if (writer) {
    constexpr int W = NWV / 4;   // waves that share 16 groups
    float2 p[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float2 w[W];
#pragma unroll
      for (int i = 0; i < W; ++i) w[i] = red[r * W + i][e];
#pragma unroll
      for (int off = 1; off < W; off <<= 1)
#pragma unroll
        for (int i = 0; i < W; i += 2 * off) lse_fold(w[i].x, w[i].y, w[i + off].x, w[i + off].y);
      p[r] = w[0];
    }
    M = -INFINITY;
    S = 0.f;
    lse_fold(M, S, p);
    const float lse = M + logf(S);
    // -log P >= 0: for a near-certain token (z[x_n] the row maximum, every other term
    // tiny) rounding in the exponentials and the logarithm can take the difference a few
    // ulps below zero; it is clamped there (a NaN stays NaN)
    const float d = lse - z;
    scores[n] = none ? INFINITY : (d < 0.f ? 0.f : d);
    if (lse_out) lse_out[n] = lse;
  }
}

// out[c][r] = in[r][c] for an in [rows][cols] matrix: 64x64 tiles through LDS (one
// padding column, so the column reads hit distinct banks).  Used once per model to lay
// W_o out K-contiguous for the fused LM-head weight.
template <class T>
__global__ __launch_bounds__(256) void transpose_kernel(const T* __restrict__ in, T* __restrict__ out,
                                                        int rows, int cols) {
  __shared__ T tile[64][65];
  const int r0 = blockIdx.y * 64, c0 = blockIdx.x * 64;
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  for (int i = ty; i < 64; i += 4) {
    const int r = r0 + i, c = c0 + tx;
    if (r < rows && c < cols) tile[i][tx] = in[int64_t(r) * cols + c];
  }
  __syncthreads();
  for (int i = ty; i < 64; i += 4) {
    const int c = c0 + i, r = r0 + tx;
    if (c < cols && r < rows) out[int64_t(c) * rows + r] = tile[tx][i];
  }
}

}  // namespace

hipError_t launch_transpose(int dtype, const void* in, void* out, int rows, int cols,
                            hipStream_t s) {
  if (rows == 0 || cols == 0) return hipSuccess;
  const dim3 grid((cols + 63) / 64, (rows + 63) / 64);
  if (dtype == CC_BF16)
    hipLaunchKernelGGL(transpose_kernel<u16>, grid, dim3(256), 0, s, static_cast<const u16*>(in),
                       static_cast<u16*>(out), rows, cols);
  else
    hipLaunchKernelGGL(transpose_kernel<float>, grid, dim3(256), 0, s,
                       static_cast<const float*>(in), static_cast<float*>(out), rows, cols);
  return hipGetLastError();
}

int lmhead_vocab_tile(int dtype) { return dtype == CC_BF16 ? VT : lmhead_f32_vocab_tile(); }

size_t packed_rows_bytes(int64_t rows, int cols) {
  return size_t((rows + PK_ROWS - 1) / PK_ROWS) * PK_ROWS * size_t(cols) * 2;
}

hipError_t launch_pack_rows(const void* x, int64_t rows, int cols, int64_t ldx, void* out,
                            hipStream_t s) {
  const int64_t tiles = (rows + PK_ROWS - 1) / PK_ROWS;
  const int64_t n_chunks = tiles * PK_ROWS * (cols / PK_K) * 4;
  if (n_chunks == 0) return hipSuccess;
  hipLaunchKernelGGL(pack_rows_kernel, dim3(unsigned((n_chunks + 255) / 256)), dim3(256), 0, s,
                     static_cast<const u16*>(x), int(rows), cols, ldx, n_chunks,
                     static_cast<u16*>(out));
  return hipGetLastError();
}

namespace {
// Tile width by estimated time: rounds of 256 workgroups, each its k-tiles (us below, bound by loads
// at 64 entries and by matrix work at 256; the same for bf16 and E4M3), the first loads and the
// epilogue; a last round that leaves CUs idle runs up to 30% quicker.  Over 1026 timings of
// vocabularies 4000 .. 152064, K 1024 .. 4096, 16 .. 4096 entries and the three weight forms the
// width it picks is on average 0.1% and at most 7% slower than the best one; the cheapest cover of the
// entries, without regard to rounds, is 8% and up to 80% (4000 x 1024 at 256 entries: 26 us in
// one column of 16 tiles, 15 in four; 16000 x 2048 at 770: 71 us in five columns of 315 tiles, 59 in
// four of 252).
int lmhead_nb(int V, int N, int K) {
  const double us[4] = {0.66, 0.88, 1.15, 1.47};
  const int64_t tiles_m = (int64_t(V) + VT - 1) / VT;
  int best = 4;
  double least = 1e300;
  for (int nb = 4; nb >= 1; --nb) {
    const int64_t tiles = tiles_m * ((int64_t(N) + 64 * nb - 1) / (64 * nb));
    const int64_t full = tiles / 256, left = tiles % 256;
    const double rounds = full == 0 ? 1.0 : double(full) + (left ? 0.7 + 0.3 * double(left) / 256.0 : 0.0);
    const double c = rounds * (double(K / 64) * us[nb - 1] + 2.0 + nb);
    if (c < least) {
      least = c;
      best = nb;
    }
  }
  return best;
}

template <int AM>
hipError_t launch_lmhead_gemm(const void* w, const void* u, int V, int N, int K, float2* partial,
                              float* target, const int32_t* ids, const float* su, const float* sw,
                              hipStream_t s) {
  TileArgs g{};
  g.A = static_cast<const u16*>(w);
  g.B = static_cast<const u16*>(u);
  g.M = V;
  g.N = N;
  g.K = K;
  if (K >= kWideRow)
    return launch_tile<8, 3, 3, 2, AM, true>(g, EpiLse<3>{partial, target, ids, su, sw}, 1, s);
  switch (lmhead_nb(V, N, K)) {
    case 1: return launch_tile<8, 1, 4, 4, AM>(g, EpiLse<1>{partial, target, ids, su, sw}, 1, s);
    case 2: return launch_tile<8, 2, 3, 3, AM>(g, EpiLse<2>{partial, target, ids, su, sw}, 1, s);
    case 3: return launch_tile<8, 3, 3, 2, AM>(g, EpiLse<3>{partial, target, ids, su, sw}, 1, s);
    default: return launch_tile<8, 4, 3, 2, AM>(g, EpiLse<4>{partial, target, ids, su, sw}, 1, s);
  }
}

hipError_t launch_combine(const float2* partial, int n_vt, const float* target, const int32_t* cu,
                          int n_seqs, int n_frozen, int N, float* scores, float* lse, hipStream_t s) {
  // Four entries a workgroup until these are two workgroups a CU (figures at the kernel).
  if (N <= 2048)
    hipLaunchKernelGGL(lse_combine<4>, dim3((N + 3) / 4), dim3(4 * CMB_G), 0, s, partial, n_vt, target, cu,
                       n_seqs, n_frozen, N, scores, lse);
  else
    hipLaunchKernelGGL(lse_combine<16>, dim3((N + 15) / 16), dim3(16 * CMB_G), 0, s, partial, n_vt, target, cu,
                       n_seqs, n_frozen, N, scores, lse);
  return hipGetLastError();
}
}  // namespace

hipError_t launch_lmhead(const LmHeadLaunch& a, hipStream_t s) {
  if (a.N == 0) return hipSuccess;
  hipError_t err;
  if (a.dtype != CC_BF16)
    err = launch_lmhead_f32(a, s);
  else if (a.w_packed)
    err = launch_lmhead_gemm<A_PACKED>(a.w_packed, a.u, a.V, a.N, a.D, a.partial, a.target, a.ids, nullptr,
                                       nullptr, s);
  else
    err = launch_lmhead_gemm<A_ROWS>(a.w_lm, a.u, a.V, a.N, a.D, a.partial, a.target, a.ids, nullptr,
                                     nullptr, s);
  if (err != hipSuccess) return err;
  const int vt = lmhead_vocab_tile(a.dtype);
  return launch_combine(a.partial, (a.V + vt - 1) / vt, a.target, a.cu_d, a.n_seqs, a.n_frozen, a.N,
                        a.scores, a.lse, s);
}

hipError_t launch_quantize_e4m3(int dtype, const void* x, int64_t rows, int cols, int per_row,
                                uint8_t* q, float* scale, float* amax_ws, hipStream_t s) {
  if (rows == 0 || cols == 0) return hipSuccess;
  const bool bf = dtype == CC_BF16;
  if (per_row) {
    if (bf)
      hipLaunchKernelGGL(quantize_rows_kernel<u16>, dim3(rows), dim3(256), 0, s,
                         static_cast<const u16*>(x), cols, q, scale);
    else
      hipLaunchKernelGGL(quantize_rows_kernel<float>, dim3(rows), dim3(256), 0, s,
                         static_cast<const float*>(x), cols, q, scale);
    return hipGetLastError();
  }
  if (bf)
    hipLaunchKernelGGL(row_amax_kernel<u16>, dim3(rows), dim3(256), 0, s,
                       static_cast<const u16*>(x), cols, amax_ws);
  else
    hipLaunchKernelGGL(row_amax_kernel<float>, dim3(rows), dim3(256), 0, s,
                       static_cast<const float*>(x), cols, amax_ws);
  hipLaunchKernelGGL(max_reduce_kernel, dim3(1), dim3(1024), 0, s, amax_ws, rows, amax_ws + rows);
  if (bf)
    hipLaunchKernelGGL(quantize_matrix_kernel<u16>, dim3(rows), dim3(256), 0, s,
                       static_cast<const u16*>(x), cols, amax_ws + rows, q, scale);
  else
    hipLaunchKernelGGL(quantize_matrix_kernel<float>, dim3(rows), dim3(256), 0, s,
                       static_cast<const float*>(x), cols, amax_ws + rows, q, scale);
  return hipGetLastError();
}

hipError_t launch_lmhead_fp8(const LmHeadFp8Launch& a, hipStream_t s) {
  if (a.N == 0) return hipSuccess;
  hipError_t err = launch_quantize_e4m3(a.dtype, a.u, a.N, a.D, 1, a.uq, a.su, a.amax_ws, s);
  if (err != hipSuccess) return err;
  // rows of D codes are D/2 16-bit units
  err = launch_lmhead_gemm<A_FP8>(a.wq, a.uq, a.V, a.N, a.D / 2, a.partial, a.target, a.ids, a.su, a.sw, s);
  if (err != hipSuccess) return err;
  return launch_combine(a.partial, (a.V + VT - 1) / VT, a.target, a.cu_d, a.n_seqs, a.n_frozen, a.N,
                        a.scores, a.lse, s);
}

}  // namespace cc
