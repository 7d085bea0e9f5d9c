// Counter-causal attention in fp32 (the kernel family of attention.hip for CC_F32 problems):
// every cached entry i attends only to later entries j > i of its own sequence.
//
// S^T = K Q^T and O^T = V^T P^T on the 16x16x4 fp32 MFMA (plain fp32 multiply-adds).  One
// workgroup owns 32 rows, a row being one (position, query head of the GQA group) pair; its W
// waves share those rows and take every W-th 16-key tile each, so a row's serial chain is that
// part of its keys, and their (max, sum, output) triples are merged through LDS.  W is 4, or 8 for
// launches that leave CUs idle (launch_f32 has the rule).  A lane's column of the MFMA output is
// one row, so the online softmax needs two shuffles per tile.  The k index of an MFMA is free to choose as long as both operands
// agree, and is chosen so that every operand arrives by 16-byte loads straight from the
// cache and P needs no data movement at all:
//   S^T: lane group grp of four holds dims grp*d/4 .. +d/4-1 of its key row (step s takes
//        dim grp*d/4 + s from every group);
//   O^T: step e takes key 4 grp + e, which is where S^T left P's element e; row r of output
//        block db is dim r*d/16 + db, so a lane's V values for all blocks are contiguous.
// Bound: latency for the small problems fp32 is used for (one thread per row and 128 rows
// per workgroup left 4 workgroups at 256 entries of 2 heads, each a serial chain of 256
// keys: 281 us; now 13 us), fp32 MFMA rate beyond (one query row costs 4 d operations a key).
#include "cc_internal.h"

namespace cc {
namespace {

constexpr int F_ROWS = 32;   // rows per workgroup
constexpr int F_BN = 16;     // keys per tile

template <class Items>
struct AttnArgsF {
  const float* q;
  float* o;
  Items items;
  KvView k, v;
  int layer;
  int hq, g;
  float scale;
  int inclusive;
};

typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));   // q: only 4-byte aligned

__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ bool non_finite(float x) {
  return (__float_as_uint(x) & 0x7f800000u) == 0x7f800000u;
}

template <int D, bool PAGED, int W, class Items>
__global__ __launch_bounds__(64 * W) void attn_cc_f32(AttnArgsF<Items> a) {
  constexpr int DL = D / 4;     // dims a lane holds of a key (or query) row
  constexpr int DB = D / 16;    // output blocks; dims a lane holds of a value row
  constexpr int OLD = D + 4;    // padded row of the merge buffer
  __shared__ __attribute__((aligned(16))) float os[W][F_ROWS][OLD];
  __shared__ float ms[W][F_ROWS], ls[W][F_ROWS];
  const AttnItem it = a.items.item(blockIdx.x);
  const int b = it.seq, kvh = it.kvh, row0 = it.rb * F_ROWS;
  const int seq0 = it.seq0, n = it.n;
  const int g = a.g, nrows = n * g;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int grp = lane >> 4, r16 = lane & 15;

  float qf[2][DL];
  int pos[2];
#pragma unroll
  for (int qb = 0; qb < 2; ++qb) {
    // rows past the last are clamped to it and not stored
    const int row = min(row0 + qb * 16 + r16, nrows - 1);
    pos[qb] = row / g;
    const float* qp = a.q + (int64_t(seq0 + pos[qb]) * a.hq + kvh * g + row % g) * D + grp * DL;
#pragma unroll
    for (int s = 0; s < DL; s += 4) {
      const f32x4u x = *reinterpret_cast<const f32x4u*>(qp + s);
#pragma unroll
      for (int i = 0; i < 4; ++i) qf[qb][s + i] = x[i];
    }
  }
  const int pos_hi = (min(row0 + F_ROWS, nrows) - 1) / g;
  const int t_begin = (row0 / g + (a.inclusive ? 0 : 1)) / F_BN;
  const int t_end = (n + F_BN - 1) / F_BN;
  const float* kb = static_cast<const float*>(a.k.base);
  const float* vb = static_cast<const float*>(a.v.base);

  float m[2] = {-INFINITY, -INFINITY}, l[2] = {0.f, 0.f};
  f32x4 acc[DB][2];
#pragma unroll
  for (int db = 0; db < DB; ++db) acc[db][0] = acc[db][1] = f32x4{};

  for (int t = t_begin + wave; t < t_end; t += W) {
    const int key0 = t * F_BN;
    // rows past the sequence end are clamped to its last key (their weights are 0)
    const float* kp = kb + kv_off<PAGED>(a.k, b, a.layer, kvh, min(key0 + r16, n - 1)) + grp * DL;
    float kf[DL], vf[4][DB];
#pragma unroll
    for (int i = 0; i < DL; i += 4) {
      const float4 x = *reinterpret_cast<const float4*>(kp + i);
      kf[i] = x.x; kf[i + 1] = x.y; kf[i + 2] = x.z; kf[i + 3] = x.w;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float* vp = vb + kv_off<PAGED>(a.v, b, a.layer, kvh, min(key0 + 4 * grp + e, n - 1)) + r16 * DB;
#pragma unroll
      for (int i = 0; i < DB; i += 4) {
        const float4 x = *reinterpret_cast<const float4*>(vp + i);
        vf[e][i] = x.x; vf[e][i + 1] = x.y; vf[e][i + 2] = x.z; vf[e][i + 3] = x.w;
      }
    }
    f32x4 sc[2] = {f32x4{}, f32x4{}};
#pragma unroll
    for (int s = 0; s < DL; ++s) {
      sc[0] = mfma4(kf[s], qf[0][s], sc[0]);
      sc[1] = mfma4(kf[s], qf[1][s], sc[1]);
    }
    const bool masked = key0 + F_BN > n || (a.inclusive ? key0 < pos_hi : key0 <= pos_hi);
    auto allowed = [&](int key, int qb) {
      return key < n && (a.inclusive ? key >= pos[qb] : key > pos[qb]);
    };
    float p[2][4];
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
      float mt = -INFINITY;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        p[qb][e] = sc[qb][e] * a.scale;
        if (masked && !allowed(key0 + 4 * grp + e, qb)) p[qb][e] = -INFINITY;
        mt = fmaxf(mt, p[qb][e]);
      }
      mt = fmaxf(mt, __shfl_xor(mt, 16));
      mt = fmaxf(mt, __shfl_xor(mt, 32));
      const float m_new = fmaxf(m[qb], mt);
      const float ref = m_new == -INFINITY ? 0.f : m_new;
      const float corr = expf(m[qb] - ref);   // 0 while nothing has been seen
      float sum = 0.f;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        p[qb][e] = expf(p[qb][e] - ref);
        sum += p[qb][e];
      }
      l[qb] = l[qb] * corr + sum;
      m[qb] = m_new;
      if (__any(corr != 1.f)) {
#pragma unroll
        for (int db = 0; db < DB; ++db) acc[db][qb] *= corr;
      }
    }
    // A key that a row may not see must not reach it even as 0 * inf: a masked tile that
    // holds a non-finite value is added key by key.
    bool odd = false;
    if (masked) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int db = 0; db < DB; ++db) odd |= non_finite(vf[e][db]);
    }
    if (__any(odd)) {
      for (int k = 0; k < F_BN; ++k) {
        const float* vp = vb + kv_off<PAGED>(a.v, b, a.layer, kvh, min(key0 + k, n - 1));
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) {
          const int e = k & 3;
          const float mine = e == 0 ? p[qb][0] : e == 1 ? p[qb][1] : e == 2 ? p[qb][2] : p[qb][3];
          const float pk = __shfl(mine, (k >> 2) * 16 + r16);
          if (!allowed(key0 + k, qb)) continue;
#pragma unroll
          for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[db][qb][i] += pk * vp[(4 * grp + i) * DB + db];
        }
      }
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int db = 0; db < DB; ++db) {
          acc[db][0] = mfma4(vf[e][db], p[0][e], acc[db][0]);
          acc[db][1] = mfma4(vf[e][db], p[1][e], acc[db][1]);
        }
    }
  }

  // merge the waves: lane element i of block db is dim (4 grp + i) * DB + db
#pragma unroll
  for (int qb = 0; qb < 2; ++qb) {
    l[qb] += __shfl_xor(l[qb], 16);
    l[qb] += __shfl_xor(l[qb], 32);
    const int r = qb * 16 + r16;
    if (grp == 0) {
      ms[wave][r] = m[qb];
      ls[wave][r] = l[qb];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int db = 0; db < DB; db += 4)
        *reinterpret_cast<float4*>(&os[wave][r][(4 * grp + i) * DB + db]) =
            make_float4(acc[db][qb][i], acc[db + 1][qb][i], acc[db + 2][qb][i], acc[db + 3][qb][i]);
  }
  __syncthreads();
  constexpr int TPR = 64 * W / F_ROWS;   // threads per row
  const int r = tid / TPR, row = row0 + r;
  if (row >= nrows) return;
  float M = -INFINITY, L = 0.f, wgt[W];
#pragma unroll
  for (int i = 0; i < W; ++i) M = fmaxf(M, ms[i][r]);
  const float ref = M == -INFINITY ? 0.f : M;
#pragma unroll
  for (int i = 0; i < W; ++i) {
    wgt[i] = expf(ms[i][r] - ref);
    L += wgt[i] * ls[i][r];
  }
  const float inv = L == 0.f ? 0.f : 1.f / L;   // no key allowed: the output is 0
  float* op = a.o + (int64_t(seq0 + row / g) * a.hq + kvh * g + row % g) * D;
#pragma unroll
  for (int c = 0; c < D / TPR; ++c) {
    const int e = c * TPR + tid % TPR;
    float x = 0.f;
#pragma unroll
    for (int i = 0; i < W; ++i) x += wgt[i] * os[i][r][e];
    op[e] = x * inv;
  }
}

template <int D, int W, class Items>
hipError_t launch_f32(const AttnLaunch& a, const Items& items, hipStream_t s) {
  AttnArgsF<Items> x;
  x.items = items;
  x.q = static_cast<const float*>(a.q);
  x.o = static_cast<float*>(a.o);
  x.k = a.k;
  x.v = a.v;
  x.layer = a.layer;
  x.hq = a.n_heads_q;
  x.g = a.n_heads_q / a.n_heads_kv;
  x.scale = a.scale;
  x.inclusive = a.inclusive;
  const dim3 grid(a.n_work), block(64 * W);
  if (a.paged)
    hipLaunchKernelGGL((attn_cc_f32<D, true, W, Items>), grid, block, 0, s, x);
  else
    hipLaunchKernelGGL((attn_cc_f32<D, false, W, Items>), grid, block, 0, s, x);
  return hipGetLastError();
}

// Eight waves an item where the launch leaves CUs idle and an item has tiles to share.  (At head dim
// 128 eight waves leave each too few registers.)
template <class Items>
hipError_t launch_f32(const AttnLaunch& a, const Items& items, hipStream_t s) {
  if (a.head_dim != 64) return launch_f32<128, 4>(a, items, s);
  const bool wide = a.n_work <= 256 && a.items.seqs[0].n >= 8 * F_BN;
  return wide ? launch_f32<64, 8>(a, items, s) : launch_f32<64, 4>(a, items, s);
}

}  // namespace

int attention_f32_rows() { return F_ROWS; }

hipError_t launch_attention_f32(const AttnLaunch& a, hipStream_t s) {
  if (a.table.table)   // more than ATTN_INLINE sequences: many items
    return a.head_dim != 64 ? launch_f32<128, 4>(a, a.table, s) : launch_f32<64, 4>(a, a.table, s);
  if (a.items.n_seqs == 1)
    return launch_f32(a, AttnOne{a.items.nkv, a.items.seqs[0].n}, s);
  return launch_f32(a, a.items, s);
}

}  // namespace cc
