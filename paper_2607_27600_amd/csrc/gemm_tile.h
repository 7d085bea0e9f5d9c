// The bf16 contraction of the scoring pass: C[m][n] = sum_k A[m][k] B[n][k], both operands
// K-contiguous, A the weights (features, vocabulary) and B the cached entries, on the 16x16x32
// bf16 MFMA with fp32 accumulators that an epilogue consumes in registers.
//
// Tile.  8 waves as 2 x 4, each 16 MB x 16 NB: a workgroup owns 32 MB features x 64 NB entries.
// The 256 x 256 tile (MB = 8, NB = 4) does the most work per byte brought into LDS; smaller
// ones exist for products whose 256 x 256 tiles fill the 256 CUs badly (plan_tiles below).
//
// Stages.  K advances 64 at a time (128-byte row pieces) through two rings of LDS buffers, SA
// for A and SB for B, loaded by direct global -> LDS instructions (1 KB per wave instruction)
// that are issued right after the barrier that frees their buffer, between MFMAs, so a load of
// A has SA - 1 k-tiles to land.  A comes from HBM and gets the deeper ring: at 256 x 256, three
// buffers of A and two of B fill the 160 KB exactly.  Against two buffers of each, the ring
// takes the LM head of 4096 entries (128256 x 4096) from 3215 to 2994 us (1.34 -> 1.44
// PFLOP/s).  There is one barrier per k-tile, in its middle: before it every wave waits for
// its own loads of the next tile (vmcnt counts them in issue order, and younger loads stay in
// flight) and has all fragments of the current tile in registers, so behind it the next tile
// may be read and the current buffers refilled.
//
// Fragments.  Rows are unpadded 128 bytes with the 16-byte chunk c of row r at c ^ ((r >> 1) & 7)
// (16 rows read at one chunk then cover all 64 banks once).  A fragments are refilled block by
// block behind their last MFMA, B fragments are double buffered.
//
// E4M3 codes (A_FP8) use the same tiles, rings and loads, a k-tile being 128 codes of every
// row, on the 16x16x128 MFMA with unit block scales (it multiplies the codes' values exactly
// and accumulates in fp32).  A fragment is the whole 128-byte row piece, 32 bytes a lane, so a
// k-tile is one k-step: both operands' fragments are refilled behind their last MFMA (the
// registers hold no second set) and the barrier stands in front of it.  128256 x 4096 codes
// at 4096 entries: 1630 us (2.64 PFLOP/s) against 1740 us on two buffers of each operand and
// the 32x32x64 MFMA.
//
// The loads are issued from inline assembly: the compiler cannot tell the buffers of a ring
// apart and would order every LDS read behind every pending load.
#pragma once

#include <type_traits>

#include "cc_internal.h"

namespace cc {

// How the rows of A lie in memory.
enum AMode {
  A_ROWS = 0,    // row-major [M][K]
  A_PACKED = 1,  // the layout of cc_pack_lmhead (256-row tiles of 32-column blocks); MB = 8
  A_GATED = 2,   // paired rows: feature f of A (gate) and of A2 (up)
  A_ROPE = 3,    // paired rows: elements e and e + 64 of one head of A (head_dim 128)
  A_FP8 = 4,     // rows of OCP E4M3 codes in both operands, K in 16-bit units (two codes)
};
// Paired modes interleave two sets of rows so that one lane holds both members of a pair:
// logical rows 16 i .. 16 i + 15 hold pairs 8 i .. 8 i + 7, and a lane of group grp holds
// pairs 8 i + 2 grp and + 1 (first members in accumulator elements 0 and 1, second in 2, 3).
// In LDS a 16-row block is 8 first rows, then 8 second rows (one load instruction each).

struct TileArgs {
  const u16* A;
  const u16* A2;
  const u16* B;
  int M, N, K;         // logical rows of A, rows of B, columns (a multiple of 64)
  int tiles_m, tiles_n;
  int slices;          // K is cut into this many slices of kt_slice k-tiles
  int kt_slice;
  int walk;            // 1: the supertile walk of tile_of; 0: dealt to the XCDs (no slices: either)
};

// Workgroup -> output tile.  The tile grid is cut into supertiles of ST_M x ST_N tiles (rows
// of supertiles first, each row walked left to right), and inside a supertile the workgroups
// walk groups of GROUP_M tile rows with the row index fastest.  Workgroups are dealt to the
// eight XCDs round robin, so each XCD's resident workgroups cover GROUP_M rows x 8 columns
// of tiles (few distinct k-slices per k-step in its L2), and the whole chip works inside one
// supertile at a time, whose operand rows (64 + 16 tiles of 256 rows, 147 MB at a 3584-wide
// K) stay in the Infinity Cache while the supertile row is swept: the wide operand is then
// re-read once per supertile row instead of once per GROUP_M tile rows.  A grid of at most 16
// tile columns is the plain GROUP_M walk.  (Partitioning the order by XCD explicitly measured
// no better; 64 supertile rows measured 1.4% faster than 32 on the 152064 x 75696 LM head,
// 96 and 128 no better than 64.)
constexpr int GROUP_M = 4;
constexpr int ST_M = 64, ST_N = 16;

__device__ __forceinline__ void tile_of(int bid, int tiles_m, int tiles_n, int& tm, int& tn) {
  const int sr = bid / (ST_M * tiles_n);
  const int rem = bid - sr * (ST_M * tiles_n);
  const int m0 = sr * ST_M;
  const int sm = min(ST_M, tiles_m - m0);        // tile rows in this supertile row
  const int sc = rem / (sm * ST_N);
  const int rem2 = rem - sc * (sm * ST_N);
  const int n0 = sc * ST_N;
  const int sn = min(ST_N, tiles_n - n0);        // tile columns in this supertile
  const int group = rem2 / (GROUP_M * sn);
  const int first = group * GROUP_M;
  const int gsize = min(GROUP_M, sm - first);
  const int within = rem2 - group * (GROUP_M * sn);
  tm = m0 + first + within % gsize;
  tn = n0 + within / gsize;
}

__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

typedef int i32x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ f32x4 mfma16(i32x8 a, i32x8 b, f32x4 c) {
  // operand formats 0 (E4M3), block scales 127 (2^0)
  return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a, b, c, 0, 0, 0, 127, 0, 127);
}

constexpr int TILE_NT = 512;   // threads: 8 waves, two per SIMD

template <int MB, int NB, int SA, int SB>
struct TileCfg {
  static constexpr int TM = 32 * MB, TN = 64 * NB;
  static constexpr int IA = TM / 8, IB = TN / 8;               // load instructions per k-tile
  static constexpr int LA = (IA + 7) / 8, LB = (IB + 7) / 8;   // the same per wave
  static constexpr int ASZ = TM * 128, BSZ = TN * 128;         // bytes of a buffer
  static constexpr int LDS = SA * ASZ + SB * BSZ;
  // loads of this wave that may be in flight when the next k-tile must have landed: those
  // issued after the next tile's (groups are issued B first, then A)
  static constexpr int W = SA > SB ? LA + (SB - 2) * (LA + LB) : (SB - 2) * (LA + LB);
  static_assert(SA >= SB && SB >= 2, "A has the deeper ring");
  static_assert(LDS <= 160 * 1024 && W < 64, "LDS, vmcnt");
};

// The row of A behind row l8 of load instruction idx (8 LDS rows) of the tile whose first
// logical row is m0; rows past the edge repeat the last one.
template <int AM>
__device__ __forceinline__ int a_row(const TileArgs& g, int m0, int idx, int l8) {
  if constexpr (AM == A_GATED) return min(m0 / 2 + (idx >> 1) * 8 + l8, g.M / 2 - 1);
  if constexpr (AM == A_ROPE) {
    const int p = min(m0 / 2 + (idx >> 1) * 8 + l8, g.M / 2 - 1);
    return (p >> 6) * 128 + (idx & 1) * 64 + (p & 63);
  }
  return min(m0 + idx * 8 + l8, g.M - 1);
}

// Rows shorter than this are addressed by a scalar base and 32-bit offsets within the tile
// (at most 384 rows apart in A_ROPE); longer ones (WIDE) by 64-bit addresses, which take twice
// the registers and leave no room for the widest tiles.
constexpr int kWideRow = 1 << 22;

template <int MB, int NB, int SA, int SB, int AM, bool WIDE, class Epi>
__global__ __launch_bounds__(TILE_NT, 1) void gemm_tile(TileArgs g, Epi epi) {
  using C = TileCfg<MB, NB, SA, SB>;
  constexpr bool PACK = AM == A_PACKED;
  constexpr bool PAIR = AM == A_GATED || AM == A_ROPE;
  constexpr bool F8 = AM == A_FP8;
  static_assert(!PACK || MB == 8, "packed tiles have 256 rows");
  __shared__ __attribute__((aligned(1024))) char lds[C::LDS];
  int tm, tn, sl = 0;
  if (g.walk) {
    tile_of(blockIdx.x, g.tiles_m, g.tiles_n, tm, tn);
  } else {
    // contiguous runs of (tile row, slice, tile column) to each XCD: the workgroups that share
    // rows of A share an L2, and no XCD has more than one workgroup above the others
    const int total = g.tiles_m * g.tiles_n * g.slices;
    const int lin = (blockIdx.x & 7) * ((total + 7) >> 3) + (blockIdx.x >> 3);
    if (int(blockIdx.x >> 3) >= ((total + 7) >> 3) || lin >= total) return;
    tn = lin % g.tiles_n;
    sl = (lin / g.tiles_n) % g.slices;
    tm = lin / g.tiles_n / g.slices;
  }
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 2, wn = wave & 3;
  const int grp = lane >> 4, r16 = lane & 15;
  const int m0 = tm * C::TM, n0 = tn * C::TN;
  const int kt0 = sl * g.kt_slice;
  const int nk = min(g.kt_slice, g.K / 64 - kt0);

  // Load instruction idx of a buffer covers its rows 8 idx .. 8 idx + 7: lane l fills 16-byte
  // position l % 8 of row l / 8.  Wave w issues idx = w, w + 8, ...; where a buffer has fewer
  // the spare waves repeat one (of the same parity: the same swizzle), so that every wave
  // counts the same number of loads.
  const int l8 = lane >> 3;
  const int chunk = (lane & 7) ^ ((4 * (wave & 1) + (l8 >> 1)) & 7);
  auto ia = [&](int j) { return min(j * 8 + wave, C::IA - 2 + (wave & 1)); };
  auto ib = [&](int j) { return min(j * 8 + wave, C::IB - 2 + (wave & 1)); };
  // the operands' first rows (A: the first that this wave loads) at this slice's first column
  const u16* a_mat = AM == A_GATED && (wave & 1) ? g.A2 : g.A;
  const int a_row0 = PACK ? 0 : a_row<AM>(g, m0, wave & 1, 0);
  const char* sa = PACK ? reinterpret_cast<const char*>(g.A) + (int64_t(tm) * (g.K / 64) + kt0) * C::ASZ
                        : reinterpret_cast<const char*>(a_mat + int64_t(a_row0) * g.K + int64_t(kt0) * 64);
  const char* sb = reinterpret_cast<const char*>(g.B + int64_t(n0) * g.K + int64_t(kt0) * 64);
  using Off = std::conditional_t<WIDE, int64_t, uint32_t>;
  Off va[C::LA], vb[C::LB];
#pragma unroll
  for (int j = 0; j < C::LA; ++j)   // packed: contiguous 1 KB runs, already swizzled
    va[j] = PACK ? Off(ia(j) * 1024 + lane * 16)
                 : Off(a_row<AM>(g, m0, ia(j), l8) - a_row0) * Off(g.K) * 2 + Off(chunk * 16);
#pragma unroll
  for (int j = 0; j < C::LB; ++j)
    vb[j] = Off(min(n0 + ib(j) * 8 + l8, g.N - 1) - n0) * Off(g.K) * 2 + Off(chunk * 16);
  const uint32_t lds0 = uint32_t(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) void*)(lds)));
  auto dma = [&](const char* base, Off off, uint32_t dst) {
    if constexpr (WIDE)
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(dst), "v"(base + off)
                   : "memory", "m0");
    else
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(dst), "v"(off), "s"(base)
                   : "memory", "m0");
  };
  // k-tile t (past the end: the last one again) into the buffer at byte offset `buf`
  auto load_a = [&](int t, uint32_t buf, int j) {
    dma(sa + int64_t(min(t, nk - 1)) * (PACK ? C::ASZ : 128), va[j], lds0 + buf + ia(j) * 1024);
  };
  auto load_b = [&](int t, uint32_t buf, int j) {
    dma(sb + int64_t(min(t, nk - 1)) * 128, vb[j], lds0 + SA * C::ASZ + buf + ib(j) * 1024);
  };

  // Fragment of a 16-row block for k-step ks (32 columns): lane (grp, r16) reads chunk 4 ks + grp
  // of its row.  In paired modes logical row 4 q + i is LDS row 8 (i >> 1) + 2 q + (i & 1).
  constexpr int ABLK = PACK ? 1024 : 2048;   // bytes from block to block
  const int ra = PAIR ? ((r16 >> 1) & 1) * 8 + (r16 >> 2) * 2 + (r16 & 1) : r16;
  // E4M3: lane (grp, r16) reads chunks 2 grp and 2 grp + 1, codes 32 grp .. 32 grp + 31.
  uint32_t fa_off[2], fb_off[2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
    const int c = F8 ? 2 * grp + ks : 4 * ks + grp;
    fa_off[ks] = PACK ? ks * 16384 + r16 * 64 + ((grp ^ ((r16 >> 1) & 3)) * 16)
                      : ra * 128 + ((c ^ ((ra >> 1) & 7)) * 16);
    fb_off[ks] = r16 * 128 + ((c ^ ((r16 >> 1) & 7)) * 16);
  }
  const uint32_t a_base = wm * MB * ABLK, b_base = SA * C::ASZ + wn * NB * 2048;

  f32x4 acc[MB][NB];
#pragma unroll
  for (int a = 0; a < MB; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[a][b] = f32x4{};

  // the load groups of "tiles" -SA .. -1, as the loop below would have issued them
#pragma unroll
  for (int q = -SA; q < -1; ++q) {
    if (q + SB >= 0) {
#pragma unroll
      for (int j = 0; j < C::LB; ++j) load_b(q + SB, (q + SB) * C::BSZ, j);
    }
#pragma unroll
    for (int j = 0; j < C::LA; ++j) load_a(q + SA, (q + SA) * C::ASZ, j);
  }
  constexpr int kWait = (C::W & 15) | ((C::W >> 4) << 14) | (7 << 4);   // vmcnt(W) lgkmcnt(0)
  __builtin_amdgcn_s_waitcnt(kWait);
  __syncthreads();
#pragma unroll
  for (int j = 0; j < C::LB; ++j) load_b(SB - 1, (SB - 1) * C::BSZ, j);
#pragma unroll
  for (int j = 0; j < C::LA; ++j) load_a(SA - 1, (SA - 1) * C::ASZ, j);

  constexpr int NM = MB * NB, NL = C::LA + C::LB, GAP = NM >= NL ? NM / NL : 1;
  uint32_t ca = 0, cb = 0;   // the current k-tile's buffers
  auto next_a = [&]() { return ca + C::ASZ == SA * C::ASZ ? 0u : ca + C::ASZ; };
  auto next_b = [&]() { return cb + C::BSZ == SB * C::BSZ ? 0u : cb + C::BSZ; };
  // the loads into the buffers that k-tile t has freed, spread over the MFMAs of a k-step
  // (small tiles: several at once)
  auto refill = [&](int t, int i) {
#pragma unroll
    for (int j = 0; j < NL; ++j) {
      if (i != (NM >= NL ? j * GAP : j * NM / NL)) continue;
      if (j < C::LB) load_b(t + SB, cb, j);
      else load_a(t + SA, ca, j - C::LB);
    }
  };
  if constexpr (F8) {
    auto frag8 = [&](uint32_t lo, uint32_t hi) {
      const uint4 x = *reinterpret_cast<const uint4*>(lds + lo), y = *reinterpret_cast<const uint4*>(lds + hi);
      return i32x8{int(x.x), int(x.y), int(x.z), int(x.w), int(y.x), int(y.y), int(y.z), int(y.w)};
    };
    i32x8 fa[MB], fb[NB];
#pragma unroll
    for (int a = 0; a < MB; ++a) fa[a] = frag8(a_base + fa_off[0] + a * ABLK, a_base + fa_off[1] + a * ABLK);
#pragma unroll
    for (int b = 0; b < NB; ++b) fb[b] = frag8(b_base + fb_off[0] + b * 2048, b_base + fb_off[1] + b * 2048);
    for (int t = 0; t < nk; ++t) {
      const uint32_t na = next_a(), nb = next_b();
      __builtin_amdgcn_s_waitcnt(kWait);
      __syncthreads();
      uint32_t qa0 = a_base + na + fa_off[0], qa1 = a_base + na + fa_off[1];
      uint32_t qb0 = b_base + nb + fb_off[0], qb1 = b_base + nb + fb_off[1];
      asm volatile("" : "+v"(qa0), "+v"(qa1), "+v"(qb0), "+v"(qb1));   // blocks as immediate offsets
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < NM; ++i) {
        const int a = i / NB, b = i % NB;
        acc[a][b] = mfma16(fa[a], fb[b], acc[a][b]);
        if (b == NB - 1) fa[a] = frag8(qa0 + a * ABLK, qa1 + a * ABLK);
        if (a == MB - 1) fb[b] = frag8(qb0 + b * 2048, qb1 + b * 2048);
        refill(t, i);
        __builtin_amdgcn_sched_barrier(0);
      }
      ca = na;
      cb = nb;
    }
  } else {
    auto frag = [&](uint32_t off) { return as_bf16x8(*reinterpret_cast<const uint4*>(lds + off)); };
    bf16x8 fa[MB], fb0[NB], fb1[NB];
#pragma unroll
    for (int a = 0; a < MB; ++a) fa[a] = frag(a_base + fa_off[0] + a * ABLK);
#pragma unroll
    for (int b = 0; b < NB; ++b) fb0[b] = frag(b_base + fb_off[0] + b * 2048);
    for (int t = 0; t < nk; ++t) {
      const uint32_t na = next_a(), nb = next_b();
      // one k-step: MFMAs on (fa, fbc); the next k-step's fragments from qa, qb
      auto kstep = [&](const bf16x8(&fbc)[NB], bf16x8(&fbn)[NB], uint32_t qa, uint32_t qb, auto loads) {
        asm volatile("" : "+v"(qa), "+v"(qb));   // one address each, blocks as immediate offsets
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < NM; ++i) {
          const int a = i / NB, b = i % NB;
          acc[a][b] = mfma16(fa[a], fbc[b], acc[a][b]);
          if (i < NB) fbn[i] = frag(qb + i * 2048);
          if (b == NB - 1) fa[a] = frag(qa + a * ABLK);
          loads(i);
          __builtin_amdgcn_sched_barrier(0);
        }
      };
      kstep(fb0, fb1, a_base + ca + fa_off[1], b_base + cb + fb_off[1], [](int) {});
      __builtin_amdgcn_s_waitcnt(kWait);
      __syncthreads();
      kstep(fb1, fb0, a_base + na + fa_off[0], b_base + nb + fb_off[0], [&](int i) { refill(t, i); });
      ca = na;
      cb = nb;
    }
  }
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  epi(acc, g, tm, sl, m0 + wm * 16 * MB, n0 + wn * 16 * NB, lane, lds);
}

template <int MB, int NB, int SA, int SB, int AM, bool WIDE = false, class Epi>
hipError_t launch_tile(TileArgs g, const Epi& e, int slices, hipStream_t s) {
  using C = TileCfg<MB, NB, SA, SB>;
  g.tiles_m = (g.M + C::TM - 1) / C::TM;
  g.tiles_n = (g.N + C::TN - 1) / C::TN;
  const int nk = g.K / 64;
  g.kt_slice = (nk + slices - 1) / slices;
  g.slices = (nk + g.kt_slice - 1) / g.kt_slice;
  // Few columns of tiles: every XCD keeps its own rows of A.  More: the supertile walk, which
  // re-reads less of B (walk against dealt: bf16, 152064 x 3584 at 3 columns 656 and 686 us,
  // 128256 x 4096 at 2 columns 447 and 443, at 16 columns 2994 and 3035; E4M3, at 3 columns
  // 386 and 375 us, at 16 columns 1630 and 1685).
  g.walk = slices == 1 && g.tiles_n > (AM == A_FP8 ? 4 : 2);
  const int64_t total = int64_t(g.tiles_m) * g.tiles_n * g.slices;
  const int64_t grid = g.walk ? total : (total + 7) / 8 * 8;
  if (grid > INT32_MAX) return hipErrorInvalidValue;
  hipLaunchKernelGGL((gemm_tile<MB, NB, SA, SB, AM, WIDE, Epi>), dim3(unsigned(grid)), dim3(TILE_NT), 0, s, g, e);
  return hipGetLastError();
}

}  // namespace cc
