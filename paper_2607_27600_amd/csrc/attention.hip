// Counter-causal attention (Eq. (2) under the mask of Sec. 3.1): every cached entry i
// attends only to later entries j > i of its own sequence, reusing the stored keys and
// values.  Output o[i][h] = sum_j softmax_j(scale * q[i][h] . k[j][c]) v[j][c], c = h/g.
//
// bf16 path (head_dim 128 or 64): flash-style, one workgroup of 4 waves per (sequence, KV
// head, block of 128 "rows"), where a row is one (position, query head of the GQA group)
// pair, so the g query heads that share a KV head share every K/V tile staged in LDS.
//   S^T = K Q^T and O^T = V^T P^T on 32x32x16 bf16 MFMA.  Computing the transposed
//   products leaves each lane owning one query row (column of the MFMA output), so the
//   online-softmax statistics and rescaling stay in registers of that lane; the P tile
//   feeds the second MFMA straight from registers.
//   Key tiles entirely at or before the block's first row are never visited (they are
//   masked for every row), so the work per block shrinks towards the end of the
//   sequence; only tiles that straddle the diagonal or the sequence end are masked.
//   K and V tiles go from global memory straight into LDS (no register staging), both
//   row-major with XOR-swizzled 16-byte chunks; the V^T operand of the second product is
//   read with LDS transpose reads.  Both are double buffered with one barrier per tile.
// The fp32 path is in attention_f32.hip.
#include <type_traits>

#include "cc_internal.h"

namespace cc {
namespace {

constexpr int BN = 64;            // keys per tile
constexpr int ROWS_W = 32;        // rows per wave
constexpr int NWAVES = 4;
constexpr int ROWS = ROWS_W * NWAVES;
constexpr float kRescale = 8.f;   // log2 headroom before the softmax reference max moves

// Shape constants of the bf16 kernel for head dim HD (128 or 64).  A K or V tile is
// BN x HD bf16 in LDS, unpadded, rows of 2 HD bytes in 16-byte chunks whose positions are
// XOR-swizzled by bits of the row (key) index so that the fragment reads hit every bank
// once per 16 lanes:
//   HD = 128 (rows of 256 B = all 64 banks): K chunk c of row r at c ^ (r & 15); V chunk c
//     at c ^ ((r & 3) << 2) (the transpose reads take 4 rows at a time);
//   HD = 64 (rows of 128 B = half the banks, so rows r and r + 1 share no bank): K chunk c
//     at c ^ ((r >> 1) & 7); V chunk c at c ^ (((r >> 1) & 1) << 2).
template <int HD>
struct Shape {
  static_assert(HD == 128 || HD == 64, "head dim 128 or 64");
  static constexpr int TILE = BN * HD;      // elements of one K or V tile (16 or 8 KB)
  static constexpr int ROWB = HD * 2;       // bytes per tile row
  static constexpr int CPR = HD / 8;        // 16-byte chunks per row
  static constexpr int RPW = 64 / CPR;      // rows one wave-wide 1 KB load fills
  static constexpr int NI = BN / (NWAVES * RPW);   // load instructions per wave per tile
  static constexpr int NKS = HD / 16;       // k-steps of S^T = K Q^T
  static constexpr int NDB = HD / 32;       // 32-dim blocks of O^T
  static constexpr int NS = 2 * NKS;        // MFMAs of S^T per tile (two 32-key blocks)
  static constexpr int NPV = 4 * NDB;       // MFMAs of O^T per tile (four 16-key steps)
  __device__ static constexpr int kswz(int r) { return HD == 128 ? (r & 15) : ((r >> 1) & 7); }
  __device__ static constexpr int vswz(int r) {
    return HD == 128 ? ((r & 3) << 2) : (((r >> 1) & 1) << 2);
  }
};

typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(1))) const void global_void;
typedef short v4i16 __attribute__((ext_vector_type(4)));
typedef short v8i16 __attribute__((ext_vector_type(8)));

template <class Items>
struct AttnArgs {
  const u16* q;
  u16* o;
  Items items;
  KvView k, v;
  int layer;
  int hq, g;
  float c2;        // scale * log2(e)
  int inclusive;
};

__device__ __forceinline__ uint4 ld16(const u16* p) { return *reinterpret_cast<const uint4*>(p); }

// ds_read_b64_tr_b16: in each group of 16 lanes, lane i receives element i%4 of the 8-byte
// chunks addressed by lanes i/4, 4 + i/4, 8 + i/4 and 12 + i/4 of its group.  With lane
// 4e + c of a group addressing row r0 + e, columns c0 + 4c .. +3 of a row-major tile, lane i
// gets column c0 + i of rows r0 .. r0+3: a transposed 4x16 block.
__device__ __forceinline__ v4i16 ds_read_tr(const char* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4i16*)(p));
}

// A wave-uniform pointer held in scalar registers, so that pointer + 32-bit lane offset
// selects the scalar-base form of the load (no per-lane 64-bit address arithmetic).
__device__ __forceinline__ const char* uniform_ptr(const char* p) {
  const uint64_t u = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane(uint32_t(u));
  const uint32_t hi = __builtin_amdgcn_readfirstlane(uint32_t(u >> 32));
  return reinterpret_cast<const char*>((uint64_t(hi) << 32) | lo);
}

// One 16-byte-per-lane global -> LDS DMA: lane l's 16 bytes land at LDS byte address
// lds + 16 l.  Issued through inline asm rather than the builtin: with the builtin in the
// loop the compiler waits for all outstanding LDS reads (lgkmcnt(0)) wherever it waits for
// one, which defeats the fragment reads issued ahead of their MFMAs; through asm it counts
// the reads precisely.  The DMAs are ordered by the explicit waitcnt + barrier that ends
// every tile (and the asm's memory clobber keeps the compiler from moving it).
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
  return uint32_t(reinterpret_cast<uintptr_t>((lds_void*)(p)));
}
// scalar base + per-lane 32-bit offset
__device__ __forceinline__ void dma16(const char* sbase, uint32_t voff, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
               :: "v"(voff), "s"(sbase), "s"(lds) : "memory", "m0");
}
// per-lane 64-bit address
__device__ __forceinline__ void dma16(const char* vaddr, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off"
               :: "v"(vaddr), "s"(lds) : "memory", "m0");
}

// Page numbers of paged-cache slabs (16 keys, which lie in one page because pages hold a
// power of two >= 16 keys), fetched with scalar loads and waited for at once.  They are
// loaded where no LDS read is outstanding (the end of a step, or the prologue), so the wait
// covers only these loads, which hit the scalar cache (16 consecutive table entries per
// line).  Vector loads of the page numbers would be counted with the tile DMAs, which
// complete in order: waiting for a page number would wait for every DMA issued before it.
__device__ __forceinline__ void page_numbers(const int32_t* p0, const int32_t* p1, int& o0, int& o1) {
  asm volatile("s_load_dword %0, %2, 0x0\n\ts_load_dword %1, %3, 0x0\n\ts_waitcnt lgkmcnt(0)"
               : "=&s"(o0), "=&s"(o1) : "s"(p0), "s"(p1) : "memory");
}
__device__ __forceinline__ void page_numbers(const int32_t* p0, const int32_t* p1, const int32_t* p2,
                                             const int32_t* p3, int& o0, int& o1, int& o2, int& o3) {
  asm volatile("s_load_dword %0, %4, 0x0\n\ts_load_dword %1, %5, 0x0\n\t"
               "s_load_dword %2, %6, 0x0\n\ts_load_dword %3, %7, 0x0\n\ts_waitcnt lgkmcnt(0)"
               : "=&s"(o0), "=&s"(o1), "=&s"(o2), "=&s"(o3)
               : "s"(p0), "s"(p1), "s"(p2), "s"(p3) : "memory");
}

// KS key groups of four waves share an item's rows: group kg takes key tiles tb + kg, tb + kg +
// KS, ... through buffers of its own, and the groups' (max, sum, output) merge through LDS at
// the end.  KS = 1 is the kernel described above.  KS = 2 halves the serial chain of tiles of an
// item and is for launches of few items with tiles to share, whose length is that of one chain
// (launch_attention has the rule): one group against two, 8 heads of 128
// on one KV head: 1500 entries 29.7 and 26.6 us, 3000 entries 53 and 45; 8 heads of 64, 3000
// entries 45 and 34.5; 28 heads of 128 on four KV heads: 900 entries 23.3 and 22.1, 512 entries
// 15.2 and 15.6 (each tile costs a shared CU more, and the merge is a barrier).
template <int HD, bool PAGED, int KS, class Items>
__global__ __launch_bounds__(256 * KS, 2) void attn_cc_bf16(AttnArgs<Items> a) {
  using SH = Shape<HD>;
  constexpr int TILE = SH::TILE, ROWB = SH::ROWB, CPR = SH::CPR, RPW = SH::RPW, NI = SH::NI;
  constexpr int NKS = SH::NKS, NDB = SH::NDB, NS = SH::NS, NPV = SH::NPV;
  // Two K and two V buffers as distinct objects: the compiler can then tell the buffer a
  // DMA is filling from the one being read, and waits for the DMA only where asked.
  __shared__ __attribute__((aligned(1024))) u16 kb0[KS * TILE];
  __shared__ __attribute__((aligned(1024))) u16 kb1[KS * TILE];
  __shared__ __attribute__((aligned(1024))) u16 vb0[KS * TILE];
  __shared__ __attribute__((aligned(1024))) u16 vb1[KS * TILE];

  const AttnItem w = a.items.item(blockIdx.x);
  const int b = w.seq, kvh = w.kvh, rb = w.rb;
  const int seq0 = w.seq0, n = w.n;
  const int g = a.g;
  const int nrows = n * g;
  const int tid = threadIdx.x;
  const int wave = (tid >> 6) & (NWAVES - 1), lane = tid & 63;
  const int kg = KS == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid >> 8);
  u16* const kl0 = kb0 + kg * TILE;
  u16* const kl1 = kb1 + kg * TILE;
  u16* const vl0 = vb0 + kg * TILE;
  u16* const vl1 = vb1 + kg * TILE;
  const int hi = lane >> 5, col = lane & 31;

  const int row = rb * ROWS + wave * ROWS_W + col;
  const bool valid = row < nrows;
  const int pos = valid ? row / g : n;
  const int hq = kvh * g + (valid ? row % g : 0);

  // This lane's query row as the B operand of S^T = K Q^T: NKS k-steps of 16 dims,
  // lane half `hi` holds dims ks*16 + hi*8 .. +7.
  bf16x8 qf[NKS];
  {
    const u16* qp = a.q + (int64_t(seq0 + (valid ? pos : 0)) * a.hq + hq) * HD + hi * 8;
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
      uint4 v = valid ? ld16(qp + ks * 16) : make_uint4(0, 0, 0, 0);
      qf[ks] = as_bf16x8(v);
    }
  }

  const int row0 = rb * ROWS;
  const int pos_lo = row0 / g;
  const int wg_last = min(row0 + ROWS, nrows) - 1;
  const int pos_hi_wg = row0 + ROWS > nrows ? n : wg_last / g;   // partial blocks mask always
  const int first_key = pos_lo + (a.inclusive ? 0 : 1);
  const int tb0 = first_key / BN;
  const int te = (n + BN - 1) / BN;
  if (tb0 >= te) {
    // no key reachable from any row of the block: every output row is 0
    if (valid && kg == 0) {
      u16* op = a.o + (int64_t(seq0 + pos) * a.hq + hq) * HD + hi * 4;
#pragma unroll
      for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int jj = 0; jj < 4; ++jj)
          *reinterpret_cast<uint2*>(op + db * 32 + jj * 8) = make_uint2(0, 0);
    }
    return;
  }
  const int tb = tb0 + kg;   // this group's first tile (the last group may have none)
  // tiles [tb0, tm0) and [tm1, te) need the mask; [tm0, tm1) see every key of every row
  const int tm0 = min(te, max(tb0, (pos_hi_wg + 1 + BN - 1) / BN));
  const int tm1 = (n % BN == 0) ? te : te - 1;

  // ---- tile DMA (global -> LDS, no registers).  Wave w, instruction i fills the RPW tile
  // rows starting at R = 4 RPW i + RPW w (1 KB): lane l writes row R + l / CPR at 16-byte
  // position l % CPR, and loads the row's chunk (l % CPR) ^ swz(row) there (the swizzles of
  // Shape).  The rows of one instruction lie in one 16-key slab (keys 16 s .. 16 s + 15,
  // s = R / 16); drow = R % 16 + l / CPR is the lane's row within the slab.  Rows past the
  // sequence end are clamped to its last key (their weights are 0 and the clamped data is
  // finite).
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);
  const int drow = (RPW * NWAVES > 16 ? (wave * RPW) % 16 : wave * RPW) + lane / CPR;
  const int kch = (lane % CPR) ^ SH::kswz(drow);
  const int vch = (lane % CPR) ^ SH::vswz(drow);
  const char* kbase = reinterpret_cast<const char*>(a.k.base);
  const char* vbase = reinterpret_cast<const char*>(a.v.base);
  const int64_t kts = a.k.tok_stride * 2, vts = a.v.tok_stride * 2;   // bytes per key
  uint32_t klane = uint32_t(drow * kts + kch * 16);
  uint32_t vlane = uint32_t(drow * vts + vch * 16);
  // contiguous caches: the (sequence, layer, head) plane; paged: layer + head part
  const char* kplane = kbase + (PAGED ? int64_t(a.layer) * a.k.layer_stride + int64_t(kvh) * a.k.head_stride
                                      : kv_off<false>(a.k, b, a.layer, kvh, 0)) * 2;
  const char* vplane = vbase + (PAGED ? int64_t(a.layer) * a.v.layer_stride + int64_t(kvh) * a.v.head_stride
                                      : kv_off<false>(a.v, b, a.layer, kvh, 0)) * 2;
  const int32_t* btab = PAGED ? a.k.block_table + int64_t(b) * a.k.max_pages : nullptr;
  const int last_page = PAGED ? (n - 1) >> a.k.page_shift : 0;
  // The 16-key slab of load instruction i (wave-uniform): at HD = 128 the four waves' rows
  // of one instruction form slab i; at HD = 64 waves 0-1 fill slab 2i and waves 2-3 slab
  // 2i + 1.
  auto slab_of = [&](int i) {
    return RPW * NWAVES > 16 ? (RPW * NWAVES / 16) * i + (RPW * wave_u) / 16 : i;
  };
  // Page numbers of this wave's slabs of tile t (paged caches; K and V share the block
  // table): scalar loads, waited for at once.  Slabs past the sequence end take its last page.
  auto load_pages = [&](int t, int (&pg)[NI]) {
    if constexpr (PAGED) {
      const int32_t* pp[NI];
#pragma unroll
      for (int i = 0; i < NI; ++i) pp[i] = btab + min((t * BN + 16 * slab_of(i)) >> a.k.page_shift, last_page);
      if constexpr (NI == 4)
        page_numbers(pp[0], pp[1], pp[2], pp[3], pg[0], pg[1], pg[2], pg[3]);
      else
        page_numbers(pp[0], pp[1], pg[0], pg[1]);
    }
  };
  // Fill an LDS tile with tile t.  Full tiles of a contiguous cache: from a running tile
  // pointer (tile_ptr = plane + t * BN keys, advanced once per tile), a 64-bit scalar add per
  // 16-key slab and the lane's fixed offset.  Full tiles of a paged cache: a uniform base per
  // slab from its page, pg (loaded beforehand by load_pages).  The last, partial tile:
  // per-lane rows (clamped), per-lane page lookups.
  auto issue = [&](u16* dst, int t, const KvView& kv, const char* plane, const char* tile_ptr,
                   uint32_t lane_off, int ch, int64_t ts, const int (&pg)[NI]) {
    const int key0 = t * BN;
    u16* lds = dst + wave_u * RPW * HD;
    const uint32_t pstride = uint32_t(kv.page_stride * 2);   // bytes per page
    if (key0 + BN <= n) {
      // keep the 32-bit offset opaque here so that it is not widened outside the loop
      asm volatile("" : "+v"(lane_off));
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const int si = slab_of(i);
        const char* base;
        if constexpr (PAGED)   // a page spans < 4 GiB: 32 x 32 -> 64-bit page offset
          base = uniform_ptr(plane + (uint64_t(uint32_t(pg[i])) * pstride +
                                      uint32_t((key0 + 16 * si) & kv.page_mask) * uint32_t(ts)));
        else
          base = tile_ptr + int64_t(16 * si) * ts;
        dma16(base, lane_off, lds_addr(lds + i * NWAVES * RPW * HD));
      }
    } else {
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const int key = min(key0 + 16 * slab_of(i) + drow, n - 1);
        int64_t off;
        if constexpr (PAGED)
          off = int64_t(btab[key >> kv.page_shift]) * kv.page_stride + int64_t(key & kv.page_mask) * kv.tok_stride;
        else
          off = int64_t(key) * kv.tok_stride;
        dma16(plane + off * 2 + ch * 16, lds_addr(lds + i * NWAVES * RPW * HD));
      }
    }
  };

  // ---- fragment reads.  K (A operand of S^T = K Q^T): MFMA j reads row (j&1)*32 + col,
  // chunk 2*(j>>1) + hi.  V^T (A operand of O^T = V^T P^T): MFMA j = (k-step kk, d block db)
  // = (j / NDB, j % NDB) needs d = 32 db + col and keys 16kk + 4hi + {0..3},
  // 16kk + 8 + 4hi + {0..3} (the order of the P operand's k-slots): two transpose reads of
  // 4 keys x 16 dims.  Lane 4y + c of lane group G reads key row 4 (G >> 1) + y at dims
  // 32 db + 16 (G & 1) + 4 c .. +3, i.e. 8-byte half (c & 1) of chunk
  // 4 db + 2 (G & 1) + (c >> 1), at that chunk's swizzled position.
  uint32_t koff[NKS];
#pragma unroll
  for (int jj = 0; jj < NKS; ++jj) koff[jj] = col * ROWB + 16 * ((2 * jj + hi) ^ SH::kswz(col));
  uint32_t voff[NDB];
  {
    const int G = lane >> 4, L = lane & 15, y = L >> 2;
    const int r = 4 * (G >> 1) + y;
#pragma unroll
    for (int db = 0; db < NDB; ++db) {
      if constexpr (HD == 128)   // vswz(r) = 4 y: the swizzle moves whole 64-byte groups
        voff[db] = r * ROWB + 64 * (db ^ y) + 32 * (G & 1) + 8 * (L & 3);
      else
        voff[db] = r * ROWB + 16 * ((4 * db + 2 * (G & 1) + ((L & 3) >> 1)) ^ SH::vswz(r)) +
                   8 * (L & 1);
    }
  }
  auto kfrag = [&](const u16* Kl, int j) {
    return as_bf16x8(*reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(Kl) +
                                                     koff[j >> 1] + (j & 1) * (32 * ROWB)));
  };
  auto vfrag = [&](const u16* Vl, int j) {
    const char* p = reinterpret_cast<const char*>(Vl) + voff[j % NDB] + (j / NDB) * (16 * ROWB);
    const v4i16 lo = ds_read_tr(p), hi2 = ds_read_tr(p + 8 * ROWB);
    const v8i16 both = __builtin_shufflevector(lo, hi2, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, both);
  };

  // max over both lane halves (they hold the two 32-key blocks of one row)
  auto half_max = [](float x) {
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  };
  auto row_max = [&](const f32x16(&s)[2]) {
    float m = -INFINITY;
#pragma unroll
    for (int mb = 0; mb < 2; ++mb)
#pragma unroll
      for (int e = 0; e < 16; ++e) m = fmaxf(m, s[mb][e]);
    return half_max(m);
  };
  auto apply_mask = [&](f32x16(&s)[2], int t) {
    const int key0 = t * BN;
#pragma unroll
    for (int mb = 0; mb < 2; ++mb)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int key = key0 + mb * 32 + (e >> 2) * 8 + hi * 4 + (e & 3);
        const bool ok = key < n && (a.inclusive ? key >= pos : key > pos);
        s[mb][e] = ok ? s[mb][e] : -INFINITY;
      }
  };

  float m_run = -INFINITY, l_run = 0.f;
  f32x16 acc[NDB];
#pragma unroll
  for (int db = 0; db < NDB; ++db) acc[db] = f32x16{};

  // contiguous caches: tile pointers of the next K (t + 2 KS) and V (t + KS) DMAs, in bytes
  const int64_t kstep = int64_t(BN) * kts, vstep = int64_t(BN) * vts;
  const char* kptr = kplane + int64_t(tb + 2 * KS) * kstep;
  const char* vptr = vplane + int64_t(tb + KS) * vstep;
  // Paged caches: the page numbers of the tiles the next step loads are fetched at the end
  // of the step before (a tile's K pages are the next step's V pages), so no step waits for
  // a scalar load before its DMAs.  kpg: pages of the group's tile after next (K), vpg: of its next tile (V).
  int kpg[NI], vpg[NI];
  // prologue: K(tb), V(tb), K(tb+1) in LDS; S(tb) and its unmasked row max in registers.
  if (KS == 1 || tb < te) {
  load_pages(tb, kpg);
  issue(kl0, tb, a.k, kplane, kplane + int64_t(tb) * kstep, klane, kch, kts, kpg);
  issue(vl0, tb, a.v, vplane, vplane + int64_t(tb) * vstep, vlane, vch, vts, kpg);
  load_pages(tb + KS, vpg);
  if (tb + KS < te) issue(kl1, tb + KS, a.k, kplane, kplane + int64_t(tb + KS) * kstep, klane, kch, kts, vpg);
  if (tb + 2 * KS < te) load_pages(tb + 2 * KS, kpg);
  }
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  f32x16 sa[2], sb[2];
  sa[0] = f32x16{};
  sa[1] = f32x16{};
#pragma unroll
  for (int j = 0; j < NS; ++j) sa[j & 1] = mfma32(kfrag(kl0, j), qf[j >> 1], sa[j & 1]);
  // Every wave has read K(tb) before the first step's DMAs refill its buffer (if any group's do), as
  // the barrier at the end of a step has it for the tiles after.
  if (tb0 + 2 * KS < te) __syncthreads();
  float mx = row_max(sa);

  // Tile t with parity P = (t - tb) & 1.  S(t) is in sc with its unmasked row max in mx;
  // K(t+1) in kl[1-P], V(t) in vl[P].  The DMAs of K(t+2) -> kl[P] and V(t+1) -> vl[1-P]
  // refill buffers freed by the previous tile.  Issue order: the NS MFMAs of S(t+1) carry
  // the 32 exponentials of tile t; the NPV MFMAs of P V carry the bf16 packing of P, the row
  // sums and the row max of S(t+1).  sched_barrier fences keep the compiler from regrouping.
  auto step = [&](int t, auto par, bool masked) {
    constexpr int P = decltype(par)::value;
    f32x16(&sc)[2] = P ? sb : sa;
    f32x16(&sn)[2] = P ? sa : sb;
    const u16* Kn = P ? kl0 : kl1;
    u16* Kfree = P ? kl1 : kl0;
    const u16* Vc = P ? vl1 : vl0;
    u16* Vfree = P ? vl0 : vl1;
    // tiles past the last are never read: nothing to load
    if (t + 2 * KS < te) issue(Kfree, t + 2 * KS, a.k, kplane, kptr, klane, kch, kts, kpg);
    if (t + KS < te) issue(Vfree, t + KS, a.v, vplane, vptr, vlane, vch, vts, vpg);
    kptr += KS * kstep;
    vptr += KS * vstep;
    bf16x8 kf[4];
    kf[0] = kfrag(Kn, 0);
    kf[1] = kfrag(Kn, 1);
    kf[2] = kfrag(Kn, 2);
    if (masked) {
      apply_mask(sc, t);
      mx = row_max(sc);
    }
    // Lazy rescaling: the reference max only moves when the row max grows by more than
    // 2^8 in probability units (or on the first non-empty tile).  Numerator and
    // denominator always share the reference, so the result is unchanged; p stays <= 256.
    const bool up = mx > m_run + kRescale / a.c2;
    const float corr = up ? fast_exp2((m_run - mx) * a.c2) : 1.f;   // 0 when m_run = -inf
    m_run = up ? mx : m_run;
    const float mc = (m_run == -INFINITY ? 0.f : m_run) * a.c2;
    sn[0] = f32x16{};
    sn[1] = f32x16{};
    __builtin_amdgcn_sched_barrier(0);
    // The section that carries the exponentials issues at raised wave priority, so that on a
    // SIMD shared with a wave in another section its MFMAs and exponentials go first
    // (measured: 4-7% faster at n = 4096, 1.5% at 32768; the same priority over both
    // sections, or over the P V section, gains less or nothing).
    __builtin_amdgcn_s_setprio(1);
    constexpr int EPM = 32 / NS;   // exponentials per MFMA
#pragma unroll
    for (int j = 0; j < NS; ++j) {
      if (j + 3 < NS) kf[(j + 3) & 3] = kfrag(Kn, j + 3);
      sn[j & 1] = mfma32(kf[j & 3], qf[j >> 1], sn[j & 1]);
#pragma unroll
      for (int u = 0; u < EPM; ++u) {
        const int f = EPM * j + u, mb = f >> 4, e = f & 15;
        const float p = fast_exp2(fmaf(sc[mb][e], a.c2, -mc));
        // pin the exponential here, between the MFMAs, instead of next to its later uses
        asm volatile("" ::"v"(p));
        sc[mb][e] = p;
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    if (__any(corr != 1.f)) {
#pragma unroll
      for (int db = 0; db < NDB; ++db) acc[db] *= corr;
    }
    // P^T operand: k-step kk covers keys 16kk .. 16kk+15; lane half hi holds keys
    // {4hi..4hi+3, 8+4hi..8+4hi+3} of that step, i.e. S^T entries 8*(kk%2)..+7 of block kk/2
    bf16x8 pf[4];
    auto pack = [&](int kk) {
#pragma unroll
      for (int e = 0; e < 8; ++e) pf[kk][e] = (__bf16)sc[kk >> 1][(kk & 1) * 8 + e];
    };
    bf16x8 vf[4];
    vf[0] = vfrag(Vc, 0);
    vf[1] = vfrag(Vc, 1);
    vf[2] = vfrag(Vc, 2);
    __builtin_amdgcn_s_setprio(0);
    pack(0);
    float ls0 = 0.f, ls1 = 0.f, m0 = -INFINITY, m1 = -INFINITY;
    constexpr int SPM = 32 / NPV;   // row-sum terms per MFMA
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < NPV; ++j) {
      if (j + 3 < NPV) vf[(j + 3) & 3] = vfrag(Vc, j + 3);
      acc[j % NDB] = mfma32(vf[j & 3], pf[j / NDB], acc[j % NDB]);
      if (j % NDB == NDB - 1 && j < NPV - 1) pack(j / NDB + 1);
#pragma unroll
      for (int u = 0; u < SPM; u += 2) {
        ls0 += sc[(SPM * j + u) >> 4][(SPM * j + u) & 15];
        ls1 += sc[(SPM * j + u + 1) >> 4][(SPM * j + u + 1) & 15];
      }
      asm volatile("" : "+v"(ls0), "+v"(ls1));
      if constexpr (HD == 64) {
        // row max of S(t+1) over slots 2..7: six entries per slot (sn[0] then sn[1])
        if (j >= 2) {
#pragma unroll
          for (int u = 0; u < 6; ++u) {
            const int f = 6 * (j - 2) + u;
            if (f < 16) m0 = fmaxf(m0, sn[0][f]);
            else if (f < 32) m1 = fmaxf(m1, sn[1][f - 16]);
          }
          asm volatile("" : "+v"(m0), "+v"(m1));
        }
      } else if (j >= 2) {
        // row max of S(t+1), whose MFMAs were issued during the exponentials: 32 entries
        // over slots 2..12
        const int f = j - 2;
        if (f < 4) {
          m0 = fmaxf(m0, fmaxf(sn[0][3 * f], fmaxf(sn[0][3 * f + 1], sn[0][3 * f + 2])));
        } else if (f < 5) {
          m0 = fmaxf(m0, fmaxf(sn[0][12], fmaxf(sn[0][13], sn[0][14])));
          m1 = fmaxf(m1, sn[0][15]);
        } else if (f < 10) {
          const int e0 = 3 * (f - 5);
          m1 = fmaxf(m1, fmaxf(sn[1][e0], fmaxf(sn[1][e0 + 1], sn[1][e0 + 2])));
        } else if (f < 11) {
          m1 = fmaxf(m1, sn[1][15]);
        }
        asm volatile("" : "+v"(m0), "+v"(m1));
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    l_run = l_run * corr + (ls0 + ls1);
    mx = half_max(fmaxf(m0, m1));
    if constexpr (PAGED) {
      // pages of the next step's tiles; no LDS read is outstanding here, so the loads' wait
      // overlaps the DMA wait below
#pragma unroll
      for (int i = 0; i < NI; ++i) vpg[i] = kpg[i];
      if (t + 3 * KS < te) load_pages(t + 3 * KS, kpg);
    }
  };
  auto sync = [&]() {
    __builtin_amdgcn_s_waitcnt(0);   // this wave's DMAs have landed
    __syncthreads();                 // everyone's, and everyone is done with K(t+1), V(t)
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  // every group runs the barriers of the first one's tiles
  for (int t = tb; t - kg < te; t += 2 * KS) {
    if (KS == 1 || t < te) step(t, I0{}, t < tm0 || t >= tm1);
    sync();
    const int u = t + KS;
    if (u - kg < te) {
      if (KS == 1 || u < te) step(u, I1{}, u < tm0 || u >= tm1);
      sync();
    }
  }

  float l_all = l_run + __shfl_xor(l_run, 32);
  // the wave's output staging: its 32 rows in the K buffers
  char* stg = reinterpret_cast<char*>(wave < 2 ? kb0 : kb1) + (wave & 1) * (KS * ROWS_W * ROWB);
  if constexpr (KS == 2) {
    // group 1 leaves its output in the staging of the same wave of group 0 (32 rows of HD
    // floats, 16 bytes a lane at a time) and its row maxima and sums in the V buffers
    float* ml = reinterpret_cast<float*>(vb0) + wave * 128;
    if (kg == 1) {
#pragma unroll
      for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int jj = 0; jj < 4; ++jj)
          *reinterpret_cast<float4*>(stg + ((db * 4 + jj) * 64 + lane) * 16) =
              make_float4(acc[db][jj * 4], acc[db][jj * 4 + 1], acc[db][jj * 4 + 2], acc[db][jj * 4 + 3]);
      ml[lane] = m_run;
      ml[64 + lane] = l_all;
    }
    __syncthreads();
    if (kg == 1) return;
    const float m1 = ml[lane], M = fmaxf(m_run, m1), ref = M == -INFINITY ? 0.f : M;
    const float w0 = fast_exp2((m_run - ref) * a.c2), w1 = fast_exp2((m1 - ref) * a.c2);
    l_all = l_all * w0 + ml[64 + lane] * w1;
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) {
        const float4 x = *reinterpret_cast<const float4*>(stg + ((db * 4 + jj) * 64 + lane) * 16);
        acc[db][jj * 4] = acc[db][jj * 4] * w0 + x.x * w1;
        acc[db][jj * 4 + 1] = acc[db][jj * 4 + 1] * w0 + x.y * w1;
        acc[db][jj * 4 + 2] = acc[db][jj * 4 + 2] * w0 + x.z * w1;
        acc[db][jj * 4 + 3] = acc[db][jj * 4 + 3] * w0 + x.w * w1;
      }
  }
  const float l_tot = l_all;
  const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
  // The output goes out through LDS as whole rows.  The K buffers are free here (the last
  // step waited for every load and ended with a barrier); each wave stages its 32 rows x HD
  // dims (16-byte chunk c of row r at chunk c ^ kswz(r), so the 16-byte row reads hit every
  // bank once, and at HD = 128 the 8-byte writes of the lane halves too), then writes 16
  // bytes per lane along the rows.  The g rows of one position are adjacent in o
  // (head-major), so a wave instruction stores 1 KB of whole rows instead of 64 scattered
  // 8-byte pieces.  LDS operations of one wave complete in order, so the wave needs no
  // barrier of its own.
#pragma unroll
  for (int db = 0; db < NDB; ++db)
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) {
      bf16x4 o;
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = (__bf16)(acc[db][jj * 4 + e] * inv);
      const int c = db * 4 + jj;
      *reinterpret_cast<bf16x4*>(stg + col * ROWB + ((c ^ SH::kswz(col)) * 16) + hi * 8) = o;
    }
#pragma unroll
  for (int i = 0; i < ROWS_W * CPR / 64; ++i) {
    const int r = RPW * i + lane / CPR, c = lane % CPR;
    const uint4 v = *reinterpret_cast<const uint4*>(stg + r * ROWB + ((c ^ SH::kswz(r)) * 16));
    const int orow = rb * ROWS + wave * ROWS_W + r;
    if (orow < nrows) {
      const int opos = orow / g, ohq = kvh * g + orow % g;
      *reinterpret_cast<uint4*>(a.o + (int64_t(seq0 + opos) * a.hq + ohq) * HD + c * 8) = v;
    }
  }
}

template <int KS, class Items>
hipError_t launch_bf16(const AttnLaunch& a, const Items& items, hipStream_t s) {
  AttnArgs<Items> x;
  x.q = static_cast<const u16*>(a.q);
  x.o = static_cast<u16*>(a.o);
  x.items = items;
  x.k = a.k;
  x.v = a.v;
  x.layer = a.layer;
  x.hq = a.n_heads_q;
  x.g = a.n_heads_q / a.n_heads_kv;
  x.c2 = a.scale * kLog2e;
  x.inclusive = a.inclusive;
  const dim3 grid(a.n_work), block(256 * KS);
  if (a.head_dim == 64) {
    if (a.paged)
      hipLaunchKernelGGL((attn_cc_bf16<64, true, KS, Items>), grid, block, 0, s, x);
    else
      hipLaunchKernelGGL((attn_cc_bf16<64, false, KS, Items>), grid, block, 0, s, x);
  } else {
    if (a.paged)
      hipLaunchKernelGGL((attn_cc_bf16<128, true, KS, Items>), grid, block, 0, s, x);
    else
      hipLaunchKernelGGL((attn_cc_bf16<128, false, KS, Items>), grid, block, 0, s, x);
  }
  return hipGetLastError();
}

}  // namespace

int attention_rows_per_item(int dtype, int head_dim) {
  (void)head_dim;
  return dtype == CC_BF16 ? ROWS : attention_f32_rows();
}

hipError_t launch_attention(const AttnLaunch& a, hipStream_t s) {
  if (a.n_work == 0) return hipSuccess;
  if (a.dtype != CC_BF16) return launch_attention_f32(a, s);
  // a table stands for more than ATTN_INLINE sequences: many items
  if (a.table.table) return launch_bf16<1>(a, a.table, s);
  // Two key groups where the longest chain of tiles, not the sum of all, makes the launch's length:
  // up to one item a CU (two groups fill it) from 12 tiles on, up to two items a CU (one group each
  // would fill it, but the short ones leave early) from 12 to 28 tiles on.  One group against two:
  // 264 items of up to 66 tiles 57.4 and 45.3 us (64 wide), 288 of 36 49.6 and 41.5 (128 wide), 504
  // of 36 58.6 and 54.5, 512 of 64 66.9 and 52.0 (64 wide); but 440 of 16 32.3 and 35.3, 352 of 11
  // 16.1 and 18.5, and beyond: 552 of 24 45.3 and 49.7, 660 of 32 38.9 and 43.3.
  const int tiles = a.items.seqs[0].n / BN;
  const bool split = a.n_work <= 512 && 16 * tiles >= 16 * 12 + (a.n_work > 256 ? a.n_work - 256 : 0);
  if (a.items.n_seqs == 1) {
    const AttnOne one{a.items.nkv, a.items.seqs[0].n};
    return split ? launch_bf16<2>(a, one, s) : launch_bf16<1>(a, one, s);
  }
  return split ? launch_bf16<2>(a, a.items, s) : launch_bf16<1>(a, a.items, s);
}

}  // namespace cc
