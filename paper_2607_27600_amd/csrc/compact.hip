// KV compaction of the memory-refresh cycle (Sec. 3.2): the kept entries of every cache
// layer and KV head are gathered to the front of their sequence, dst[j] = src[keep[j]],
// as a bit copy of one head_dim row; token ids and position ids follow the same list.
//
// Out of place: one workgroup per (plane, chunk of rows), fully parallel.
// In place, short lists: one workgroup per plane with the whole list in registers.
// In place beyond: keep is ascending, so keep[j] >= j and a destination slot j can only be the
// source of an entry j' <= j.  One workgroup walks its plane in chunks of rows in
// increasing order.  Chunk c's rows are written only after a barrier that every thread
// reaches with chunk c's loads (and so all earlier loads) returned, which orders every
// read of those slots before the writes.  The sources of chunk c+1 are at or past slot
// (c+1)*rows, beyond everything chunk c writes, so its loads (and the keep indices of
// chunk c+3) are issued before chunk c is written and stay in flight across the barrier.  A plane is (sequence, layer,
// KV head, keys|values, column slab); there are hundreds to thousands per refresh.
//
// A block finds its plane from its index (sequences in the order of falling budget, then
// layers, heads, slabs), the list of a sequence comes by value with the launch (up to
// COMPACT_INLINE lists) or from a small uploaded table, and the token and position ids are
// moved by the first blocks of the same launch.  A table upload before the cache's kernel and
// an ids kernel behind it (4 us for a list of 512, 17 us for 4096) stood in line before.
#include <algorithm>

#include "cc_internal.h"

namespace cc {
namespace {

constexpr int CNT = 256;      // threads per workgroup
constexpr int CU = 5;         // 16-byte row pieces in flight per thread per chunk

struct CompactArgs {
  KvView src[2], dst[2];
  int row16;                  // 16-byte pieces of a row in one column slab
  int n_slabs;                // column slabs of a row (planes of their own)
  const int32_t* keep;
  const CompactList* lists_d; // null: lists
  int n_seqs, n_layers, n_heads, per_head;
  int n_tensors;              // 1 (rows of one array) or 2 (keys and values)
  int rows_per_chunk;         // (CNT / row16) * CU
  int id_blocks;              // leading blocks that move the ids, one for each sequence
  int32_t* ids[2];
  const int32_t* cu;
  CompactList lists[COMPACT_INLINE];   // sorted: see CompactList
};

struct Plane {
  int seq, layer, head, tensor;
  int64_t tok0;
  int k;
  const int32_t* keep;
  int col;                    // first byte of the slab
};

__device__ __forceinline__ CompactList list_of(const CompactArgs& a, int i) {
  return a.lists_d ? a.lists_d[i] : a.lists[i];
}

// Block -> plane: keys and values of a plane are adjacent blocks, slabs next, so that a row's
// pieces are moved at about the same time; the sequences come longest first.
__device__ __forceinline__ Plane plane_of(const CompactArgs& a, int i) {
  Plane P;
  P.tensor = i % a.n_tensors;
  i /= a.n_tensors;
  P.col = (i % a.n_slabs) * a.row16 * 16;
  i /= a.n_slabs;
  P.head = i % a.n_heads;
  i /= a.n_heads;
  P.layer = i % a.n_layers;
  i /= a.n_layers;
  const CompactList L = list_of(a, __builtin_amdgcn_readfirstlane(a.per_head ? i * a.n_heads + P.head : i));
  P.seq = L.seq;
  P.tok0 = L.tok0;
  P.k = L.k;
  P.keep = a.keep + L.keep_off;
  return P;
}

// ids[cu_b + j] = ids[cu_b + keep[j]] in place, block i for the i-th sequence's first list.
template <int NT>
__device__ __forceinline__ void compact_ids(const CompactArgs& a, int i) {
  constexpr int U = 8;
  const CompactList L = list_of(a, a.per_head ? i * a.n_heads : i);
  const int32_t* kp = a.keep + L.keep_off;
  const int base = a.cu[L.seq];
  for (int j0 = 0; j0 < L.k; j0 += NT * U) {
    int32_t x[2][U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int src = base + kp[min(j0 + u * NT + int(threadIdx.x), L.k - 1)];
      if (a.ids[0]) x[0][u] = a.ids[0][src];
      if (a.ids[1]) x[1][u] = a.ids[1][src];
    }
    __builtin_amdgcn_s_waitcnt(0);   // loads returned before anyone overwrites a source
    __syncthreads();
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int j = j0 + u * NT + threadIdx.x;
      if (j < L.k) {
        if (a.ids[0]) a.ids[0][base + j] = x[0][u];
        if (a.ids[1]) a.ids[1][base + j] = x[1][u];
      }
    }
  }
}

// A 16-byte piece of a source row, read non-temporally: a kept row is read once and never
// again, so the load need not stay in the caches.  Measured with the cache flushed, in-place
// compaction of a contiguous 32-layer, 8-head cache keeping 4096 of 32768 entries (1.07 GB
// moved) goes from 5.4 to 6.3 TB/s, of a paged 28-layer, 4-head cache keeping 20% of eight
// sequences (1.74 GB) from 4.9 to 5.1 TB/s.  (The same hint on the stores makes both slower:
// the compacted rows are written in runs that the caches merge.)
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 ldg16(const char* p) {
  const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
  return make_uint4(v.x, v.y, v.z, v.w);
}

// The paged in-place steps.  A source row needs its keep index, then its page number,
// then the row; a destination row needs its page number.  Step c issues, in this order,
// the keep indices of chunk c+3, the source pages of chunk c+2 (with the in-page rows),
// the destination pages and the rows of chunk c+1, then writes chunk c after the barrier.
// Everything a step waits for was issued before the rows of chunk c, so the rows of chunk
// c+1 stay in flight across the barrier.  Buffers alternate between even and odd steps.
struct PagedBufs {
  int idx[CU], spg[CU], srow[CU], dpg[CU];
  uint4 rows[CU];
};

__device__ __forceinline__ void compact_paged_steps(const CompactArgs& a, const KvView& v,
                                                    const Plane& P, const int32_t* keep,
                                                    int k, char* base, int r0,
                                                    int rstep, int esz16, int R, int nch) {
  (void)a;
  const int32_t* bt = v.block_table + int64_t(P.seq) * v.max_pages;
  char* pb = base + int64_t(P.layer) * v.layer_stride + int64_t(P.head) * v.head_stride + esz16;
  auto slot = [&](int c, int u) { return min(c * R + r0 + u * rstep, k - 1); };
  auto ld_idx = [&](int c, int (&I)[CU]) {
#pragma unroll
    for (int u = 0; u < CU; ++u) I[u] = keep[slot(min(c, nch - 1), u)];
  };
  auto ld_spg = [&](const int (&I)[CU], int (&SP)[CU], int (&RW)[CU]) {
#pragma unroll
    for (int u = 0; u < CU; ++u) {
      SP[u] = bt[I[u] >> v.page_shift];
      RW[u] = I[u] & v.page_mask;
    }
  };
  auto ld_dpg = [&](int c, int (&DP)[CU]) {
#pragma unroll
    for (int u = 0; u < CU; ++u) DP[u] = bt[slot(min(c, nch - 1), u) >> v.page_shift];
  };
  auto ld_rows = [&](const int (&SP)[CU], const int (&RW)[CU], uint4 (&D)[CU]) {
#pragma unroll
    for (int u = 0; u < CU; ++u)
      D[u] = ldg16(pb + int64_t(SP[u]) * v.page_stride + int64_t(RW[u]) * v.tok_stride);
  };
  PagedBufs e, o;   // e: buffers read in even steps, o: in odd steps (roles swap each step)
  // prologue: state for step 0 = indices of chunk 2, source pages of chunk 1, destination
  // pages and rows of chunk 0
  ld_idx(0, e.idx);
  ld_idx(1, o.idx);
  __builtin_amdgcn_sched_barrier(0);
  ld_spg(e.idx, o.spg, o.srow);   // chunk 0 -> held in o until its rows are issued below
  ld_spg(o.idx, e.spg, e.srow);   // chunk 1
  ld_idx(2, e.idx);
  ld_dpg(0, e.dpg);
  __builtin_amdgcn_sched_barrier(0);
  ld_rows(o.spg, o.srow, e.rows);
  // step c (cur = buffers of parity c, nxt = the other):
  //   cur.idx = chunk c+2, cur.spg/srow = chunk c+1, cur.dpg/rows = chunk c
  auto step = [&](int c, PagedBufs& cur, PagedBufs& nxt) {
    ld_idx(c + 3, nxt.idx);
    __builtin_amdgcn_sched_barrier(0);
    ld_spg(cur.idx, nxt.spg, nxt.srow);
    ld_dpg(c + 1, nxt.dpg);
    __builtin_amdgcn_sched_barrier(0);
    ld_rows(cur.spg, cur.srow, nxt.rows);
#pragma unroll
    for (int u = 0; u < CU; ++u)
      asm volatile("" ::"v"(cur.rows[u].x), "v"(cur.rows[u].y), "v"(cur.rows[u].z), "v"(cur.rows[u].w));
    __syncthreads();
#pragma unroll
    for (int u = 0; u < CU; ++u) {
      const int j = c * R + r0 + u * rstep;
      if (j < k)
        *reinterpret_cast<uint4*>(pb + int64_t(cur.dpg[u]) * v.page_stride +
                                  int64_t(j & v.page_mask) * v.tok_stride) = cur.rows[u];
    }
  };
  for (int c = 0; c < nch; c += 2) {
    step(c, e, o);
    step(c + 1, o, e);
  }
}

template <bool PAGED>
__global__ __launch_bounds__(CNT) void compact_in_place_kernel(CompactArgs a) {
  if (int(blockIdx.x) < a.id_blocks) {
    compact_ids<CNT>(a, blockIdx.x);
    return;
  }
  const Plane P = plane_of(a, int(blockIdx.x) - a.id_blocks);
  const int32_t* keep = P.keep;
  const int k = P.k;
  if (k <= 0) return;
  const KvView& v = a.src[P.tensor];   // source and destination views are the same
  char* base = reinterpret_cast<char*>(const_cast<void*>(v.base)) + P.tok0 * v.tok_stride;
  const int tpr = a.row16;
  const int r0 = threadIdx.x / tpr;
  const int rstep = CNT / tpr;
  const int esz16 = P.col + (threadIdx.x % tpr) * 16;
  const int R = a.rows_per_chunk;
  const int nch = (k + R - 1) / R;
  auto load_idx = [&](int c, int (&idx)[CU]) {
#pragma unroll
    for (int u = 0; u < CU; ++u) idx[u] = keep[min(c * R + r0 + u * rstep, k - 1)];
  };
  auto load_rows = [&](const int (&idx)[CU], uint4 (&buf)[CU]) {
#pragma unroll
    for (int u = 0; u < CU; ++u)
      buf[u] = ldg16(base + kv_off<PAGED>(v, P.seq, P.layer, P.head, idx[u]) + esz16);
  };
  if constexpr (PAGED) {
    compact_paged_steps(a, v, P, keep, k, base, r0, rstep, esz16, R, nch);
    return;
  } else {
    // Loads complete in issue order.  Each chunk step issues the keep indices of chunk c+2
    // before the rows of chunk c+1, so the indices a step waits for were issued before the
    // rows of the chunk being written and waiting for them never waits for those rows.  Two
    // index and two row buffers alternate; the loop is unrolled twice with the chunk count
    // rounded up to even (a register copy of a pending load, or a conditional step, would
    // make the compiler wait for every load).
    int ia[CU], ib[CU];
    uint4 dx[CU], dy[CU];
    // step c: `in` holds chunk c+1's indices, `dc` chunk c's rows; past the end, loads
    // re-read the last chunk and nothing is stored
    auto body = [&](int c, const int (&in)[CU], int (&ifree)[CU], const uint4 (&dc)[CU],
                    uint4 (&dn)[CU]) {
      load_idx(min(c + 2, nch - 1), ifree);
      __builtin_amdgcn_sched_barrier(0);   // keep the issue order: indices, then rows
      load_rows(in, dn);
  #pragma unroll
      for (int u = 0; u < CU; ++u)
        asm volatile("" ::"v"(dc[u].x), "v"(dc[u].y), "v"(dc[u].z), "v"(dc[u].w));
      __syncthreads();
  #pragma unroll
      for (int u = 0; u < CU; ++u) {
        const int j = c * R + r0 + u * rstep;
        if (j < k)
          *reinterpret_cast<uint4*>(base + kv_off<PAGED>(v, P.seq, P.layer, P.head, j) + esz16) = dc[u];
      }
    };
    load_idx(0, ia);
    load_idx(min(1, nch - 1), ib);
    __builtin_amdgcn_sched_barrier(0);
    load_rows(ia, dx);
    for (int c = 0; c < nch; c += 2) {
      body(c, ib, ia, dx, dy);
      body(c + 1, ia, ib, dy, dx);
    }
  }
}

// In place, lists of at most U rows a thread: a whole plane passes through the registers around one
// barrier, where the walk waits for a round trip to memory in each of its chunks.  Rows past the end
// of a list re-read its last entry (without them, under branches, the loads no longer go out at
// once: 11.4 -> 13.6 us for 224 planes of 512 rows, paged more).
constexpr int ONT = 1024;
template <bool PAGED, int U>
__global__ __launch_bounds__(ONT) void compact_once_kernel(CompactArgs a) {
  if (int(blockIdx.x) < a.id_blocks) {
    compact_ids<ONT>(a, blockIdx.x);
    return;
  }
  const Plane P = plane_of(a, int(blockIdx.x) - a.id_blocks);
  const int k = P.k;
  if (k <= 0) return;
  const KvView& v = a.src[P.tensor];   // source and destination views are the same
  char* base = reinterpret_cast<char*>(const_cast<void*>(v.base)) + P.tok0 * v.tok_stride;
  const int r0 = threadIdx.x / a.row16;
  const int rstep = ONT / a.row16;
  const int esz16 = P.col + (threadIdx.x % a.row16) * 16;
  int64_t to[U];
  int idx[U];
  uint4 row[U];
#pragma unroll
  for (int u = 0; u < U; ++u) idx[u] = P.keep[min(r0 + u * rstep, k - 1)];
#pragma unroll
  for (int u = 0; u < U; ++u) to[u] = kv_off<PAGED>(v, P.seq, P.layer, P.head, min(r0 + u * rstep, k - 1)) + esz16;
#pragma unroll
  for (int u = 0; u < U; ++u) row[u] = ldg16(base + kv_off<PAGED>(v, P.seq, P.layer, P.head, idx[u]) + esz16);
#pragma unroll
  for (int u = 0; u < U; ++u)   // loads returned before anyone overwrites a source
    asm volatile("" ::"v"(row[u].x), "v"(row[u].y), "v"(row[u].z), "v"(row[u].w));
  __syncthreads();
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (r0 + u * rstep < k) *reinterpret_cast<uint4*>(base + to[u]) = row[u];
}

constexpr int OMAX = 8;       // most rows a thread
template <int U>
void launch_once(const CompactArgs& a, bool paged, int passes, unsigned blocks, hipStream_t s) {
  if constexpr (U < OMAX) {
    if (passes > U) return launch_once<U + 1>(a, paged, passes, blocks, s);
  }
  if (paged)
    hipLaunchKernelGGL((compact_once_kernel<true, U>), dim3(blocks), dim3(ONT), 0, s, a);
  else
    hipLaunchKernelGGL((compact_once_kernel<false, U>), dim3(blocks), dim3(ONT), 0, s, a);
}

template <bool PAGED>
__global__ __launch_bounds__(CNT) void compact_kernel(CompactArgs a) {
  if (int(blockIdx.x) < a.id_blocks) {
    if (blockIdx.y == 0) compact_ids<CNT>(a, blockIdx.x);
    return;
  }
  const Plane P = plane_of(a, int(blockIdx.x) - a.id_blocks);
  const int32_t* keep = P.keep;
  const int k = P.k;
  const KvView& sv = a.src[P.tensor];
  const KvView& dv = a.dst[P.tensor];
  const char* sb = reinterpret_cast<const char*>(sv.base) + P.tok0 * sv.tok_stride;
  char* db = reinterpret_cast<char*>(const_cast<void*>(dv.base)) + P.tok0 * dv.tok_stride;
  const int tpr = a.row16;
  const int r0 = threadIdx.x / tpr;
  const int rstep = CNT / tpr;
  const int esz16 = P.col + (threadIdx.x % tpr) * 16;
  // element size is folded into the strides: the views carry byte strides here
  const int j_begin = blockIdx.y * a.rows_per_chunk;
  const int j_end = min(k, j_begin + a.rows_per_chunk);
  for (int j0 = j_begin; j0 < j_end; j0 += a.rows_per_chunk) {
    // branch-free gather: rows past the list end re-read its last entry and are not stored
    int src[CU];
#pragma unroll
    for (int u = 0; u < CU; ++u) src[u] = keep[min(j0 + r0 + u * rstep, j_end - 1)];
    uint4 buf[CU];
#pragma unroll
    for (int u = 0; u < CU; ++u)
      buf[u] = ldg16(sb + kv_off<PAGED>(sv, P.seq, P.layer, P.head, src[u]) + esz16);
#pragma unroll
    for (int u = 0; u < CU; ++u) {
      const int j = j0 + r0 + u * rstep;
      if (j < j_end)
        *reinterpret_cast<uint4*>(db + kv_off<PAGED>(dv, P.seq, P.layer, P.head, j) + esz16) =
            buf[u];
    }
  }
}

}  // namespace

hipError_t launch_compact(const CompactLaunch& c, hipStream_t s) {
  CompactArgs a;
  for (int t = 0; t < 2; ++t) {
    a.src[t] = c.src[t];
    a.dst[t] = c.dst[t];
    a.ids[t] = c.ids[t];
  }
  a.keep = c.keep;
  a.lists_d = c.lists_d;
  a.n_seqs = c.n_seqs;
  a.n_layers = c.n_layers;
  a.n_heads = c.n_heads;
  a.per_head = c.per_head;
  a.n_tensors = c.n_tensors;
  a.cu = c.cu_d;
  a.id_blocks = (c.ids[0] || c.ids[1]) ? c.n_seqs : 0;
  if (!c.lists_d) {
    const int n = c.n_seqs * (c.per_head ? c.n_heads : 1);
    if (n > COMPACT_INLINE) return hipErrorInvalidValue;
    std::copy(c.lists_h, c.lists_h + n, a.lists);
  }
  if (c.n_seqs == 0 || c.max_k == 0) return hipSuccess;
  const int64_t planes = int64_t(c.n_tensors) * c.n_seqs * c.n_layers * c.n_heads;
  a.n_slabs = 1;
  a.row16 = c.row_bytes / 16;
  auto chunk = [&]() { return (CNT / a.row16) * CU; };
  // Lists that fit one pass through the registers (512 rows of 256 bytes a plane) take it, in column
  // slabs while that leaves at most one block a CU; in a paged cache only up to one block a CU: there
  // each row's page is another load before it, which the walk hides better.  Walk against one pass,
  // us with the cache flushed: 224 planes of 512 rows 17.5 and 16.4, paged 17.8 and 16.6; 8 planes of
  // 500 rows 10.5 and 8.1; 3584 planes of up to 480 rows 175 and 160; but 672 paged planes of up to
  // 240 rows 21.0 and 22.4.
  auto passes = [&]() { return (int64_t(c.max_k) * a.row16 + ONT - 1) / ONT; };
  while (c.in_place && a.row16 > 4 && planes * a.n_slabs * 2 <= 256 && passes() > 1) {
    a.row16 /= 2;
    a.n_slabs *= 2;
  }
  const bool once = c.in_place && passes() <= OMAX && (!c.paged || planes <= 256);
  if (!once) {
    a.row16 = c.row_bytes / 16;
    a.n_slabs = 1;
  }
  // Beyond, a plane is one block walking its list.  Few planes with long lists leave most of
  // the chip idle and make the walk the launch's length: rows are then cut into column slabs (of
  // at least 64 bytes: half a cache line) while that leaves at most one block a CU and more than
  // 16 chunks in line.  Keeping 13200 of 20000 entries in 8 planes of 256-byte rows, selection
  // included: 136 us whole, 85 us in four slabs; 5000 of 20000 in 32 planes 77 and 59 us; lists of
  // 1024 in 32 planes are faster whole (38 and 42 us), and 64 planes of 19800 about even.  (Blocks
  // of 1024 threads measured no better anywhere.)
  while (c.in_place && !once && a.row16 > 4 && a.row16 % 2 == 0 && planes * a.n_slabs * 2 <= 256 && c.max_k > 16 * chunk()) {
    a.row16 /= 2;
    a.n_slabs *= 2;
  }
  a.rows_per_chunk = chunk();
  const int64_t blocks = planes * a.n_slabs + a.id_blocks;
  if (blocks > INT32_MAX) return hipErrorInvalidValue;
  if (once) {
    launch_once<1>(a, c.paged, int(passes()), unsigned(blocks), s);
  } else if (c.in_place) {
    if (c.paged)
      hipLaunchKernelGGL(compact_in_place_kernel<true>, dim3(unsigned(blocks)), dim3(CNT), 0, s, a);
    else
      hipLaunchKernelGGL(compact_in_place_kernel<false>, dim3(unsigned(blocks)), dim3(CNT), 0, s, a);
  } else {
    // chunks sized by the longest list; planes with shorter lists exit early
    const dim3 grid(unsigned(blocks), (c.max_k + a.rows_per_chunk - 1) / a.rows_per_chunk);
    if (c.paged)
      hipLaunchKernelGGL(compact_kernel<true>, grid, dim3(CNT), 0, s, a);
    else
      hipLaunchKernelGGL(compact_kernel<false>, grid, dim3(CNT), 0, s, a);
  }
  return hipGetLastError();
}

}  // namespace cc
