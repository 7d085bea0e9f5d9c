// Keep selection of the memory-refresh cycle (Sec. 3.2): per segment, the k entries that
// come first under (score descending, ties to the lower index), emitted in ascending
// index order so the compacted cache keeps the original time order.  The order of the scores
// is that of order_key: -0 == +0, NaN below -inf.
//
// One workgroup per segment at a time.  A histogram whose bins cut the range of the segment's
// finite scores into equal parts finds the bin of the k-th largest score; the few scores of that
// bin are ranked among each other, which gives the threshold T and how many entries equal to T
// are kept; a last pass in index order emits every score above T and the lowest-index ties with
// batched prefix counts.  Rounding moves scores between bins, but never against their order, and
// everything behind the histogram compares exactly: the result is exact.
//
// Segments of up to 32768 scores are read once, into registers, by one of four sizes of the
// kernel; longer ones are read again by each pass.
#include <algorithm>

#include "cc_internal.h"

namespace cc {
namespace {

// Descriptor of segment b: computed for regular launches, else by value in the kernel
// arguments (the first SEL_INLINE) or from the uploaded table.
__device__ __forceinline__ SelSeg seg_desc(const SelInline& inl, const SelSeg* segs, int b) {
  if (inl.regular)
    return SelSeg{inl.start0 + int64_t(b) * inl.stride, inl.len, inl.k, int64_t(b) * inl.k};
  return b < inl.n ? inl.s[b] : segs[b];
}

// Wave-wide inclusive scans and reductions on DPP lane moves (VALU only, no LDS round
// trip): shifts of 1, 2, 4 and 8 lanes inside each row of 16 (lanes without a source keep
// the identity), then the last lane of row 0 (2) added into row 1 (3), then lane 31 into
// rows 2 and 3.  Lane i ends with op over lanes 0..i.
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_move(uint32_t x, uint32_t identity) {
  return uint32_t(__builtin_amdgcn_update_dpp(int(identity), int(x), CTRL, ROWS, 0xf, false));
}
template <class Op>
__device__ __forceinline__ uint32_t wave_scan(uint32_t x, uint32_t identity, Op op) {
  x = op(x, dpp_move<0x111, 0xf>(x, identity));   // row_shr:1
  x = op(x, dpp_move<0x112, 0xf>(x, identity));   // row_shr:2
  x = op(x, dpp_move<0x114, 0xf>(x, identity));   // row_shr:4
  x = op(x, dpp_move<0x118, 0xf>(x, identity));   // row_shr:8
  x = op(x, dpp_move<0x142, 0xa>(x, identity));   // row_bcast:15 into rows 1 and 3
  x = op(x, dpp_move<0x143, 0xc>(x, identity));   // row_bcast:31 into rows 2 and 3
  return x;
}
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t x, int lane) {
  (void)lane;
  return wave_scan(x, 0u, [](uint32_t a, uint32_t b) { return a + b; });
}
// the reduction over the whole wave, in every lane
template <class Op>
__device__ __forceinline__ uint32_t wave_reduce(uint32_t x, uint32_t identity, Op op) {
  return uint32_t(__builtin_amdgcn_readlane(int(wave_scan(x, identity, op)), 63));
}

__device__ __forceinline__ uint32_t order_key(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return 0u;   // NaN: lowest
  if ((u & 0x7fffffffu) == 0u) u = 0u;              // -0 == +0
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// ------------------------------------------------------------------ the kernel
// NT threads hold a tile of CH chunks of 4 NT scores: thread t holds scores 4t .. 4t+3 of every
// chunk (one 16-byte load per chunk, 1 KB per wave instruction), so index order is (chunk,
// thread, slot).  STREAM: a segment may span several tiles, and each pass reads them all again;
// otherwise the one tile stays in registers.  Bound by vector ALU issue and LDS atomics:
//  - Extremes of the finite scores, so that an infinite one (that of a sequence's last entry)
//    does not squeeze all others into one bin.
//  - bin = (f - min) * (NB - 2) / (max - min) by one fused multiply-add that also makes it a whole
//    number, clamped to 0 .. NB - 1: both are monotone, so a higher bin never holds a lower score,
//    whatever the rounding (a range that overflows or vanishes leaves one or two bins).  Digits of
//    the float's bits in its place put scores between 8 and 16 nats, where most lie, into 8 bins:
//    lanes of one instruction collide on them, and the threshold's bin holds thousands of scores.
//    4096 of 32768 scores in each of eight segments, digits and bins: 25.7 and 12.0 us; 16384 of
//    131072 scores 244 and 38 us (five passes of 4-byte loads before); 8192 of 32768 scores in each
//    of 4096 segments, caches flushed: 293 and 221 us for scores around 9 nats, 227 and 228 us for
//    exponential ones, which digits spread well.
//  - A far score (one entry pinned at 1e9) widens the range until all others share a bin.  Such a range
//    is cut beforehand where a few scores cause it, and the bins are made anew over the threshold's
//    bin where it holds more than the list does (half the entries masked with -1e30; two rounds
//    of that, then digits).  Bins at the ends of the range that many scores share are counted in
//    registers.  The eight segments and the 4096, digits, bins over the whole range, and now: one at 1e9
//    25.8 and 291, 54 and 887, 12.9 and 237 us; half at -1e30 25.7 and 426, 42 and 701, 19.9 and 345.
//  - A NaN counts in bin 0, where its key (0) is below all others.
//  - Up to CMAX scores of T's bin go to an LDS list (in any order).  Up to RANK of them are ranked
//    by comparing each with all, a wave a score (a thread a score: 2.0 us a segment against 0.7 at 41
//    scores); more are searched by block-wide digits of their offset from the bin's smallest, and
//    beyond CMAX that search runs over the tiles in place of the list.
//  - Bucket searches are two-level wave scans: lane sums over the lanes' bin ranges, then
//    the bins of the lane that holds the rank.
//  - Emission: a thread's flagged scores per chunk are counted, and one batched scan over
//    the workgroup (two chunk counts per word) gives every flagged score its rank in index
//    order: first for the ties (when not all of them are kept), then for the kept scores, which
//    each thread stores at their ranks through a buffer descriptor bounded by the segment's
//    budget.
constexpr int RNT = 1024;
constexpr int RCW = 4;                 // scores per thread per chunk
constexpr int CMAX = 4096;             // candidate list
constexpr uint32_t FIN_SHIFT = 0x00800000u;   // bits + FIN_SHIFT: of non-negative scores +inf alone turns negative
constexpr uint32_t RANK = 256;         // candidates ranked by comparison (a multiple of 64)
constexpr float ONE = 8388608.f;       // 2^23: floats from here on to 2^24 are whole numbers
constexpr uint32_t ONE_B = 0x4b000000u;

// The float of an order key.
__device__ __forceinline__ float key_float(uint32_t k) {
  return __uint_as_float((k & 0x80000000u) ? k ^ 0x80000000u : ~k);
}

// Inclusive scan inside each row of 16 lanes (row 0 holds lanes 0..15).
__device__ __forceinline__ uint32_t row_scan(uint32_t x) {
  x += dpp_move<0x111, 0xf>(x, 0u);
  x += dpp_move<0x112, 0xf>(x, 0u);
  x += dpp_move<0x114, 0xf>(x, 0u);
  x += dpp_move<0x118, 0xf>(x, 0u);
  return x;
}
// op over lanes 0..15, in every lane
template <class Op>
__device__ __forceinline__ uint32_t row0_reduce(uint32_t x, uint32_t identity, Op op) {
  x = op(x, dpp_move<0x111, 0xf>(x, identity));
  x = op(x, dpp_move<0x112, 0xf>(x, identity));
  x = op(x, dpp_move<0x114, 0xf>(x, identity));
  x = op(x, dpp_move<0x118, 0xf>(x, identity));
  return uint32_t(__builtin_amdgcn_readlane(int(x), 15));
}
constexpr auto fmin_bits = [](uint32_t a, uint32_t b) {
  return __float_as_uint(fminf(__uint_as_float(a), __uint_as_float(b)));
};
constexpr auto fmax_bits = [](uint32_t a, uint32_t b) {
  return __float_as_uint(fmaxf(__uint_as_float(a), __uint_as_float(b)));
};
constexpr auto imax_bits = [](uint32_t a, uint32_t b) { return uint32_t(max(int32_t(a), int32_t(b))); };
constexpr auto umin_bits = [](uint32_t a, uint32_t b) { return min(a, b); };
constexpr auto umax_bits = [](uint32_t a, uint32_t b) { return max(a, b); };
constexpr auto add_bits = [](uint32_t a, uint32_t b) { return a + b; };

// Of numbers (fminf and fmaxf would quiet each operand first: as many instructions again).
__device__ __forceinline__ float min3(float a, float b, float c) {
  float d;
  asm("v_min3_f32 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
  return d;
}
__device__ __forceinline__ float max3(float a, float b, float c) {
  float d;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
  return d;
}

struct Pick {
  uint32_t digit, rem, cnt;
};

// Run by one whole wave: in a histogram of 64 * BPL bins searched from the highest bin down,
// the bin holding the rem-th largest counted key (1 <= rem <= total), the rank left inside it and
// its count; every lane receives the result.  Level 1: lane l sums bins 64 BPL - BPL (l + 1) .. 64 BPL - 1 - BPL l and a wave scan
// finds the lane whose range holds the rank; level 2: lane j < BPL reads that range's j-th
// highest bin and a second scan finds the bin.
template <int BPL>
__device__ __forceinline__ Pick pick_bucket(const uint32_t* h, uint32_t rem, int lane) {
  constexpr int NB = 64 * BPL;
  static_assert(BPL % 4 == 0 && BPL <= 64, "16-byte reads, one bin a lane");
  const uint32_t* mine = h + NB - BPL * (lane + 1);
  uint32_t sum = 0u;
#pragma unroll
  for (int q = 0; q < BPL / 4; ++q) {
    const uint4 v = reinterpret_cast<const uint4*>(mine)[q];
    sum += (v.x + v.y) + (v.z + v.w);
  }
  const uint32_t incl = wave_incl_scan(sum, lane);
  const uint64_t over = __ballot(incl >= rem);
  const int owner = over ? int(__builtin_ctzll(over)) : 63;   // rem <= total: some lane does
  const uint32_t before = uint32_t(__builtin_amdgcn_readlane(int(incl - sum), owner));
  const int top = NB - BPL * owner - 1;              // the owner's highest bin
  const uint32_t c = lane < BPL ? h[top - lane] : 0u;
  const uint32_t incl2 = wave_incl_scan(c, lane);
  const uint64_t hit = __ballot(lane < BPL && before + incl2 >= rem);
  const int j = hit ? int(__builtin_ctzll(hit)) : BPL - 1;
  const uint32_t cj = uint32_t(__builtin_amdgcn_readlane(int(c), j));
  const uint32_t ij = uint32_t(__builtin_amdgcn_readlane(int(incl2), j));
  return {uint32_t(top - j), rem - before - (ij - cj), cj};
}

template <int NT, int CH>
struct KeepLds {
  static constexpr int NW = NT / 64, NQ = (CH + 1) / 2;
  static constexpr int DIGIT = NT < 1024 ? 9 : 11, NB = 1 << DIGIT;   // bins, and bits of a digit
  static constexpr int NC = NT * CH * RCW < CMAX ? NT * CH * RCW : CMAX;
  __attribute__((aligned(16))) uint32_t hist[NB];
  __attribute__((aligned(16))) uint32_t cand[NC];
  __attribute__((aligned(16))) uint32_t wtot[4][NW][NQ];
  uint32_t red[7][NW];
  uint32_t sh_key, sh_rem, sh_cnt, sh_ncand;
};

// Ranks in index order of flagged scores: base[c] = flagged scores before this thread's part of
// chunk c, from `run` on, which moves on to the end of the tile.  own[q]: this thread's flagged
// scores in chunks 2q (low half) and 2q + 1 (high half).  wtot: LDS owned by this call until the
// second barrier from here; wave: the wave's index, uniform.  Contains one barrier.  After it,
// lanes 0 .. NW - 1 of every wave scan the waves' totals.
template <int NW, int CH, int NQ>
__device__ __forceinline__ void chunk_offsets(const uint32_t (&own)[NQ], uint32_t (&base)[CH], uint32_t& run,
                                              uint32_t (*wtot)[NQ], int lane, int wave) {
  static_assert(NW <= 16, "the waves' totals are combined in one row of 16 lanes");
  uint32_t inc[NQ], tv[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    // inclusive scan over the wave, two chunks per word (a field stays below 4 * 64 + 1)
    inc[q] = wave_incl_scan(own[q], lane);
  }
  if (lane == 63) {
#pragma unroll
    for (int q = 0; q < NQ; ++q) wtot[wave][q] = inc[q];
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < NQ; ++q) tv[q] = lane < NW ? wtot[lane][q] : 0u;
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const uint32_t sc = row_scan(tv[q]);
    const uint32_t all = uint32_t(__builtin_amdgcn_readlane(int(sc), NW - 1));
    const uint32_t bef = uint32_t(__builtin_amdgcn_readlane(int(sc - tv[q]), wave));
    const uint32_t mine = bef + inc[q] - own[q];
    base[2 * q] = run + (mine & 0xffffu);
    run += all & 0xffffu;
    if (2 * q + 1 < CH) base[2 * q + 1 < CH ? 2 * q + 1 : 0] = run + (mine >> 16);
    run += all >> 16;
  }
}

// own[] of chunk_offsets from a mask (bit 4c + i: slot i of chunk c)
template <int NQ>
__device__ __forceinline__ void chunk_counts(uint32_t m, uint32_t (&own)[NQ]) {
#pragma unroll
  for (int q = 0; q < NQ; ++q)
    own[q] = uint32_t(__popc((m >> (8 * q)) & 0xfu)) | (uint32_t(__popc((m >> (8 * q + 4)) & 0xfu)) << 16);
}

// The descriptor's fields in scalar registers (a descriptor picked from the kernel
// arguments by the block index is otherwise not known to be uniform).
__device__ __forceinline__ int64_t uniform64(int64_t x) {
  const uint32_t lo = uint32_t(__builtin_amdgcn_readfirstlane(int(uint32_t(uint64_t(x)))));
  const uint32_t hi = uint32_t(__builtin_amdgcn_readfirstlane(int(uint32_t(uint64_t(x) >> 32))));
  return int64_t((uint64_t(hi) << 32) | lo);
}

// Four scores at any multiple of four bytes.
typedef float f32x4_u __attribute__((ext_vector_type(4), aligned(4)));

template <int NT, int CH, bool STREAM>
__global__ __launch_bounds__(NT, 1) void select_keep_kernel(const float* __restrict__ scores,
                                                            const SelSeg* __restrict__ segs, SelInline inl,
                                                            int n_segs, int32_t* __restrict__ keep) {
  typedef KeepLds<NT, CH> Lds;
  constexpr int NW = Lds::NW, NQ = Lds::NQ, NB = Lds::NB, NC = Lds::NC, DIGIT = Lds::DIGIT;
  constexpr int CHUNK = NT * RCW, TILE = CH * CHUNK, SPT = CH * RCW;
  // The list holds any bin: the range is taken as it is.  (Without the code for more, these kernels
  // stay below the 80 scalar registers at which a CU holds one workgroup of 1024 threads in place of
  // two: 2048 segments of 4096 scores 33 us with it, 21 without.)
  constexpr bool FITS = !STREAM && TILE <= NC;
  static_assert(SPT <= 32, "one bit per score in a 32-bit mask");
  __shared__ Lds L;
  // With more segments than workgroups each walks several: the stores of one segment drain
  // while the loads of the next are in flight.
  for (int sgi = blockIdx.x; sgi < n_segs; sgi += gridDim.x) {
    // thread indices opaque per iteration: nothing derived from them is hoisted out of the loop
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    SelSeg sg = seg_desc(inl, segs, sgi);
    sg.start = uniform64(sg.start);
    sg.out = uniform64(sg.out);
    const int n = __builtin_amdgcn_readfirstlane(sg.len), k = __builtin_amdgcn_readfirstlane(sg.k);
    int32_t* out = keep + sg.out;
    if (k <= 0) continue;
    if (k >= n) {
      for (int i = tid; i < n; i += NT) out[i] = i;
      continue;
    }
    const float* sp = scores + sg.start;
    float f[SPT];
    // Tile at score t0 into f; NaN past the end of the segment.  Loads stay inside the segment: a
    // thread whose four scores straddle the end reads the last four and shifts them down.
    auto load = [&](uint32_t t0) {
      if (n < 4) {
#pragma unroll
        for (int j = 0; j < SPT; ++j) f[j] = __uint_as_float(0x7fc00000u);
#pragma unroll
        for (int u = 0; u < RCW; ++u)
          if (RCW * tid + u < n) f[u] = sp[RCW * tid + u];
        return;
      }
      uint32_t t4 = t0 + RCW * tid;
#pragma unroll
      for (int c = 0; c < CH; ++c) {
        const f32x4_u v = *reinterpret_cast<const f32x4_u*>(sp + min(c * CHUNK + t4, uint32_t(n - 4)));
#pragma unroll
        for (int u = 0; u < RCW; ++u) f[RCW * c + u] = v[u];
      }
      asm volatile("" : "+v"(t4));
#pragma unroll
      for (int c = 0; c < CH; ++c) {
        if (t0 + (c + 1) * CHUNK <= uint32_t(n)) continue;   // uniform: the chunk is whole
        const int sh = int(c * CHUNK + t4 - uint32_t(n - 4));   // > 0: slot u holds the score of slot u - sh
        const float nan = __uint_as_float(0x7fc00000u);
        const float x1 = f[RCW * c + 1], x2 = f[RCW * c + 2], x3 = f[RCW * c + 3];
        f[RCW * c] = sh <= 0 ? f[RCW * c] : sh == 1 ? x1 : sh == 2 ? x2 : sh == 3 ? x3 : nan;
        f[RCW * c + 1] = sh <= 0 ? x1 : sh == 1 ? x2 : sh == 2 ? x3 : nan;
        f[RCW * c + 2] = sh <= 0 ? x2 : sh == 1 ? x3 : nan;
        f[RCW * c + 3] = sh <= 0 ? x3 : nan;
      }
    };
    // pass(t0) for every tile, its scores in f
    auto tiles = [&](auto&& pass) {
      if constexpr (STREAM) {
        for (uint32_t t0 = 0; t0 < uint32_t(n); t0 += TILE) {
          load(t0);
          pass(t0);
        }
      } else {
        pass(0);
      }
    };
    if constexpr (!STREAM) load(0);
    // fn(slot) for the scores of the tile at t0, without what lies past the end
    auto each_score = [&](uint32_t t0, auto&& fn) {
      uint32_t t4 = t0 + RCW * tid;
      asm volatile("" : "+v"(t4));
#pragma unroll
      for (int c = 0; c < CH; ++c) {
        if (t0 + (c + 1) * CHUNK <= uint32_t(n)) {   // uniform: the chunk is whole
#pragma unroll
          for (int u = 0; u < RCW; ++u) fn(RCW * c + u);
        } else if (t0 + c * CHUNK < uint32_t(n)) {
#pragma unroll
          for (int u = 0; u < RCW; ++u)
            if (c * CHUNK + t4 + u < uint32_t(n)) fn(RCW * c + u);
        }
      }
    };

    // The finite scores' extremes.  First taken for scores of language models, none negative and none
    // NaN: their bits compare as integers, and adding FIN_SHIFT takes +inf alone below all others
    // (2.5 instructions a score).  Bits above those of +inf (a sign, a NaN) or no finite score:
    // taken again, score by score.
    uint32_t lo_b = 0xffffffffu, hi_b = 0u;
    int32_t fin_b = int32_t(0x80000000u);
    tiles([&](uint32_t t0) {
      each_score(t0, [&](int j) {
        const uint32_t u = __float_as_uint(f[j]);
        lo_b = min(lo_b, u);
        hi_b = max(hi_b, u);
        fin_b = max(fin_b, int32_t(u + FIN_SHIFT));
      });
    });
    __syncthreads();   // the segment before is done with the LDS
    {
      const uint32_t r0 = wave_reduce(lo_b, 0xffffffffu, umin_bits);
      const uint32_t r1 = wave_reduce(hi_b, 0u, umax_bits);
      const uint32_t r2 = wave_reduce(uint32_t(fin_b), 0x80000000u, imax_bits);
      if (lane == 0) {
        L.red[0][wave] = r0;
        L.red[1][wave] = r1;
        L.red[2][wave] = r2;
      }
    }
    for (int i = tid; i < NB; i += NT) L.hist[i] = 0u;
    if (tid == 0) L.sh_ncand = 0u;
    __syncthreads();
    const uint32_t lo_w = lane < NW ? L.red[0][lane] : 0xffffffffu;
    const int32_t fin_w = lane < NW ? int32_t(L.red[2][lane]) : int32_t(0x80000000u);
    lo_b = row0_reduce(lo_w, 0xffffffffu, umin_bits);
    hi_b = row0_reduce(lane < NW ? L.red[1][lane] : 0u, 0u, umax_bits);
    fin_b = int32_t(row0_reduce(uint32_t(fin_w), 0x80000000u, imax_bits));
    if (lo_b == hi_b) {   // one value (or NaN): the first k
      for (int i = tid; i < k; i += NT) out[i] = i;
      continue;
    }
    uint32_t T = 0u;                // the threshold's order key,
    uint32_t rem = 0u, cnt = 0u;    // the rem-th largest of the cnt scores looked at last
    {
      constexpr uint32_t INF_B = 0x7f800000u, NINF_B = 0xff800000u;
      const bool clean = hi_b <= INF_B && fin_b >= int32_t(FIN_SHIFT);   // uniform
      float mn = __uint_as_float(lo_b), mx = __uint_as_float(uint32_t(fin_b) - FIN_SHIFT);
      // the finite extremes of wave `lane`'s scores (wlo > whi: it has none)
      const bool some = clean && fin_w >= int32_t(FIN_SHIFT);
      float wlo = some ? __uint_as_float(lo_w) : INFINITY;
      float whi = some ? __uint_as_float(uint32_t(fin_w) - FIN_SHIFT) : -INFINITY;
      // this thread's finite scores that are in (past the end: NaN)
      auto finite_extremes = [&](float& lo, float& hi, auto&& in) {
        tiles([&](uint32_t t0) {
#pragma unroll
          for (int c = 0; c < CH; ++c) {
            if (t0 + c * CHUNK >= uint32_t(n)) continue;   // uniform: nothing left
#pragma unroll
            for (int j = RCW * c; j < RCW * c + RCW; j += 2) {
              const bool a = fabsf(f[j]) < INFINITY && in(f[j]);
              const bool b = fabsf(f[j + 1]) < INFINITY && in(f[j + 1]);
              lo = min3(lo, a ? f[j] : INFINITY, b ? f[j + 1] : INFINITY);
              hi = max3(hi, a ? f[j] : -INFINITY, b ? f[j + 1] : -INFINITY);
            }
          }
        });
      };
      // the waves' extremes of those, to red[3] and red[4] and back
      auto leave_extremes = [&](float lo, float hi) {
        const uint32_t r0 = wave_reduce(__float_as_uint(lo), INF_B, fmin_bits);
        const uint32_t r1 = wave_reduce(__float_as_uint(hi), NINF_B, fmax_bits);
        if (lane == 0) {
          L.red[3][wave] = r0;
          L.red[4][wave] = r1;
        }
      };
      auto take_extremes = [&]() {
        wlo = __uint_as_float(lane < NW ? L.red[3][lane] : INF_B);
        whi = __uint_as_float(lane < NW ? L.red[4][lane] : NINF_B);
        mn = __uint_as_float(row0_reduce(__float_as_uint(wlo), INF_B, fmin_bits));
        mx = __uint_as_float(row0_reduce(__float_as_uint(whi), NINF_B, fmax_bits));
      };
      if (!clean) {
        float lo = INFINITY, hi = -INFINITY;
        finite_extremes(lo, hi, [](float) { return true; });
        leave_extremes(lo, hi);
        __syncthreads();
        take_extremes();
        if (mn > mx) mn = mx = 0.f;   // no finite score: -inf and NaN to bin 0, +inf to the last
      }
      // A few far scores (those of pinned or masked entries) would leave the others one bin: where the
      // whole range is many times what every wave's scores cover, the bins cut that, half as much again
      // to either side, and what lies beyond shares the first and the last bin.  (The first two waves'
      // say whether to look: one of them, for entries pinned in one run.)
      auto width = [&](int w) {
        return __uint_as_float(uint32_t(__builtin_amdgcn_readlane(int(__float_as_uint(whi)), w))) -
               __uint_as_float(uint32_t(__builtin_amdgcn_readlane(int(__float_as_uint(wlo)), w)));
      };
      if (!FITS && mx - mn > 8.f * fminf(width(0), width(1))) {
        const bool has = wlo <= whi;
        const float chi = __uint_as_float(row0_reduce(has ? __float_as_uint(whi) : INF_B, INF_B, fmin_bits));
        const float clo = __uint_as_float(row0_reduce(has ? __float_as_uint(wlo) : NINF_B, NINF_B, fmax_bits));
        const float w = chi - clo;
        if (w > 0.f && mx - mn > 8.f * w) {
          mn = fmaxf(mn, clo - w);
          mx = fminf(mx, chi + w);
        }
      }
      uint32_t bin = 0u;
      float inv, at;
      // Bits of ONE + the bin: the sum's unit is 1.  NaN goes to bin 0: that of a score, and that of
      // 0 times infinity or infinity less itself, which then takes every lower score with it.
      auto bin_of = [&](float x) {
        return __float_as_uint(__builtin_amdgcn_fmed3f(fmaf(x, inv, at), ONE, ONE + float(NB - 1)));
      };
      for (int level = 0;; ++level) {
        inv = mn < mx ? float(NB - 2) / (mx - mn) : 1.f;
        at = fmaf(-mn, inv, ONE);
        tiles([&](uint32_t t0) {
          // A bin that many scores share makes every lane's atomic wait for the others.  Such bins are
          // the outermost ones (equal scores, a far value and all others, what lies beyond the range):
          // where a wave's first scores show it, it adds them up in registers.
          const uint32_t s = bin_of(f[0]);
          const bool in = t0 + RCW * tid < uint32_t(n);
          if (__popcll(__ballot(in && s - (ONE_B + 1) >= uint32_t(NB - 3))) < 6) {
            each_score(t0, [&](int j) { atomicAdd(&L.hist[bin_of(f[j]) - ONE_B], 1u); });
          } else {
            const int n1 = __popcll(__ballot(in && s == ONE_B + NB - 2));
            const int n2 = __popcll(__ballot(in && s == ONE_B + NB - 1));
            const uint32_t top = n2 > n1 ? ONE_B + NB - 1 : ONE_B + NB - 2;
            uint32_t c0 = 0u, c1 = 0u;
            each_score(t0, [&](int j) {
              const uint32_t b = bin_of(f[j]);
              c0 += uint32_t(b == ONE_B);
              c1 += uint32_t(b == top);
              if (b != ONE_B && b != top) atomicAdd(&L.hist[b - ONE_B], 1u);
            });
            c0 = wave_reduce(c0, 0u, add_bits);
            c1 = wave_reduce(c1, 0u, add_bits);
            if (lane == 0) {
              atomicAdd(&L.hist[0], c0);
              atomicAdd(&L.hist[top - ONE_B], c1);
            }
          }
        });
        __syncthreads();
        if (wave == 0) {
          const Pick p = pick_bucket<NB / 64>(L.hist, uint32_t(k), lane);
          if (lane == 0) {
            L.sh_key = p.digit;
            L.sh_rem = p.rem;
            L.sh_cnt = p.cnt;
          }
        }
        __syncthreads();
        bin = ONE_B + L.sh_key;
        rem = L.sh_rem;   // T is the rem-th largest of the bin's cnt scores
        cnt = L.sh_cnt;
        if (FITS || cnt <= uint32_t(NC) || mn == mx || level == 2) break;
        // too many for the list (the range has a gap, or is that of a few scores): the bins anew, over
        // the finite scores of this one
        const float was = mx - mn;
        float lo = INFINITY, hi = -INFINITY;
        finite_extremes(lo, hi, [&](float x) { return bin_of(x) == bin; });
        leave_extremes(lo, hi);
        for (int i = tid; i < NB; i += NT) L.hist[i] = 0u;
        __syncthreads();
        take_extremes();
        if (!(mn < mx && mx - mn < was)) break;   // equal, none, or no narrower: the bins stay
      }
      auto here = [&](int j) { return bin_of(f[j]) == bin; };
      // T by block-wide digits of key - kmin (scores that are all equal leave no digit); each(visit)
      // visits this thread's keys of the bin
      auto search = [&](auto&& each) {
        uint32_t kmin = 0xffffffffu, kmax = 0u;
        each([&](uint32_t key) {
          kmin = min(kmin, key);
          kmax = max(kmax, key);
        });
        const uint32_t r0 = wave_reduce(kmin, 0xffffffffu, umin_bits);
        const uint32_t r1 = wave_reduce(kmax, 0u, umax_bits);
        if (lane == 0) {
          L.red[5][wave] = r0;
          L.red[6][wave] = r1;
        }
        __syncthreads();
        kmin = row0_reduce(lane < NW ? L.red[5][lane] : 0xffffffffu, 0xffffffffu, umin_bits);
        kmax = row0_reduce(lane < NW ? L.red[6][lane] : 0u, 0u, umax_bits);
        int hi = kmax > kmin ? 32 - __clz(kmax - kmin) : 0;   // offsets < 2^hi
        uint32_t prefix = 0u;                                 // offset >> hi of those in the running
        while (hi > 0) {
          // clear the histogram (the pick before read it before the barrier that ended it)
          for (int i = tid; i < NB; i += NT) L.hist[i] = 0u;
          __syncthreads();
          const int lo = hi > DIGIT ? hi - DIGIT : 0;
          const uint32_t dmask = (1u << (hi - lo)) - 1u;
          each([&](uint32_t key) {
            const uint32_t off = key - kmin;
            if ((hi == 32 ? 0u : off >> (hi & 31)) == prefix) atomicAdd(&L.hist[(off >> lo) & dmask], 1u);
          });
          __syncthreads();
          if (wave == 0) {
            const Pick p = pick_bucket<NB / 64>(L.hist, rem, lane);
            if (lane == 0) {
              L.sh_key = p.digit;
              L.sh_rem = p.rem;
              L.sh_cnt = p.cnt;
            }
          }
          __syncthreads();
          prefix = (prefix << (hi - lo)) | L.sh_key;
          rem = L.sh_rem;
          cnt = L.sh_cnt;
          hi = lo;
        }
        T = kmin + prefix;
      };
      if (FITS || cnt <= uint32_t(NC)) {
        tiles([&](uint32_t t0) {
          uint32_t t4 = t0 + RCW * tid;
          asm volatile("" : "+v"(t4));
#pragma unroll
          for (int c = 0; c < CH; ++c) {
            bool h[RCW], any = false;
#pragma unroll
            for (int u = 0; u < RCW; ++u) {
              h[u] = here(RCW * c + u);
              any |= h[u];
            }
            if (__any(any)) {
              // a score enters the list where it finds it (the search needs no order); the
              // increments of one instruction are combined by a single lane
#pragma unroll
              for (int u = 0; u < RCW; ++u)
                if (h[u] && c * CHUNK + t4 + u < uint32_t(n)) {
                  const uint32_t pos = atomicAdd(&L.sh_ncand, 1u);
                  if (pos < uint32_t(NC)) L.cand[pos] = order_key(f[RCW * c + u]);
                }
            }
            __builtin_amdgcn_sched_barrier(0);   // one chunk at a time: no 32 live masks
          }
        });
        __syncthreads();
        if (cnt <= RANK) {
          // one candidate a wave at a time: its rank is the count of lanes whose candidates compare so
          for (uint32_t c = wave; c < cnt; c += NW) {
            const uint32_t mine = L.cand[c];
            uint32_t above = 0u, same = 0u;
#pragma unroll 1
            for (uint32_t i = lane; i < ((cnt + 63u) & ~63u); i += 64) {   // inside cand (RANK)
              const uint32_t x = L.cand[i];
              above += uint32_t(__popcll(__ballot(i < cnt && x > mine)));
              same += uint32_t(__popcll(__ballot(i < cnt && x == mine)));
            }
            if (lane == 0 && above < rem && rem <= above + same) {   // one value; its holders write the same
              L.sh_key = mine;
              L.sh_rem = rem - above;
              L.sh_cnt = same;
            }
          }
          __syncthreads();
          T = L.sh_key;
          rem = L.sh_rem;
          cnt = L.sh_cnt;
        } else {
          const uint32_t nc = min(cnt, uint32_t(NC));
          search([&](auto&& visit) {
            for (uint32_t i = tid; i < nc; i += NT) visit(L.cand[i]);
          });
        }
      } else if constexpr (!FITS) {
        search([&](auto&& visit) {
          tiles([&](uint32_t t0) {
            each_score(t0, [&](int j) {
              if (here(j)) visit(order_key(f[j]));
              __builtin_amdgcn_sched_barrier(0);
            });
          });
        });
      }
    }
    // T == 0: the threshold is NaN; every other score is above it, and rem of the NaNs are kept
    // (the NaNs past the end come last in index order, and k < n leaves them out).
    const bool t_nan = T == 0u;
    const float tf = key_float(T);
    auto above = [&](float x) { return t_nan ? x == x : x > tf; };
    auto tie = [&](float x) { return t_nan ? x != x : x == tf; };
    const bool all_ties = !t_nan && cnt == rem;   // every tie is kept
    // stores go through a descriptor that drops any past the budget
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(out, 0, STREAM ? 0 : 4 * k, 0x00020000);
    uint32_t ties = 0u, kept = 0u;   // in the tiles before
    int par = 0;
    tiles([&](uint32_t t0) {
      uint32_t take = 0u, own[NQ], base[CH];
      if (all_ties) {
        // counted per chunk (no mask: the stores compare again)
        uint32_t n_c[2 * NQ] = {};
#pragma unroll
        for (int j = 0; j < SPT; ++j) n_c[j / RCW] += uint32_t(f[j] >= tf);
#pragma unroll
        for (int q = 0; q < NQ; ++q) own[q] = n_c[2 * q] | (n_c[2 * q + 1] << 16);
      } else {
        // ties ranked in index order; the first rem are kept
        uint32_t eq = 0u;
#pragma unroll
        for (int j = SPT - 1; j >= 0; --j) {
          take = (take << 1) | uint32_t(above(f[j]));
          eq = (eq << 1) | uint32_t(tie(f[j]));
        }
        chunk_counts(eq, own);
        chunk_offsets<NW, CH, NQ>(own, base, ties, L.wtot[2 + par], lane, wave);
#pragma unroll
        for (int j = 0; j < SPT; ++j) {
          const uint32_t below = uint32_t(__popc(eq & (((1u << (j & 3)) - 1u) << (j & ~3))));
          take |= uint32_t(((eq >> j) & 1u) && base[j >> 2] + below < rem) << j;
        }
        chunk_counts(take, own);
      }
      chunk_offsets<NW, CH, NQ>(own, base, kept, L.wtot[par], lane, wave);
      par ^= 1;
      uint32_t t4 = t0 + RCW * tid;
      asm volatile("" : "+v"(t4));
      // kept scores of chunk c at ranks base[c], base[c] + 1, ...
      auto emit = [&](auto&& is_kept) {
#pragma unroll
        for (int c = 0; c < CH; ++c) {
          uint32_t r = base[c];
#pragma unroll
          for (int u = 0; u < RCW; ++u) {
            if (is_kept(RCW * c + u)) {
              const uint32_t i = c * CHUNK + t4 + u;
              if constexpr (STREAM) {   // a budget may exceed a descriptor's 4 GB
                if (r < uint32_t(k)) out[r] = int32_t(i);
              } else {
                __builtin_amdgcn_raw_buffer_store_b32(i, rs, int(4u * r), 0, 0);
              }
              ++r;
            }
          }
        }
      };
      if (all_ties)
        emit([&](int j) { return f[j] >= tf; });
      else
        emit([&](int j) { return ((take >> j) & 1u) != 0u; });
    });
  }
}

template <int NT, int CH, bool STREAM>
void launch_keep(const float* scores, const SelSeg* segs, const SelInline& inl, int n_segs, int grid,
                 int32_t* keep, hipStream_t s) {
  hipLaunchKernelGGL((select_keep_kernel<NT, CH, STREAM>), dim3(grid), dim3(NT), 0, s, scores, segs, inl, n_segs,
                     keep);
}

}  // namespace

bool select_regular(const SelSeg* segs_h, int n_segs) {
  if (n_segs < 2) return n_segs == 1;
  const int64_t stride = segs_h[1].start - segs_h[0].start;
  for (int i = 1; i < n_segs; ++i)
    if (segs_h[i].len != segs_h[0].len || segs_h[i].k != segs_h[0].k ||
        segs_h[i].start - segs_h[i - 1].start != stride || segs_h[i].out != int64_t(i) * segs_h[0].k)
      return false;
  return segs_h[0].out == 0;
}

hipError_t launch_select(const float* scores, const SelSeg* segs_h, const SelSeg* segs_d,
                         int n_segs, int max_len, int32_t* keep, hipStream_t s) {
  if (n_segs == 0) return hipSuccess;
  SelInline inl{};
  if (n_segs <= SEL_INLINE) {
    for (int i = 0; i < n_segs; ++i) inl.s[i] = segs_h[i];
    inl.n = n_segs;
  } else if (select_regular(segs_h, n_segs)) {
    // equal segments at a fixed stride (one per KV head over the same scores, a batch of
    // equal-length sequences): the kernels compute each descriptor, nothing is uploaded
    inl.regular = 1;
    inl.start0 = segs_h[0].start;
    inl.stride = segs_h[1].start - segs_h[0].start;
    inl.len = segs_h[0].len;
    inl.k = segs_h[0].k;
  }
  // The smallest kernel that holds the longest segment in registers: each further chunk costs a
  // short segment instructions (8192 scores in two chunks take 3 us less than 9001 in eight).
  if (max_len <= 256 * RCW)
    launch_keep<256, 1, false>(scores, segs_d, inl, n_segs, n_segs, keep, s);
  else if (max_len <= RNT * RCW)
    launch_keep<RNT, 1, false>(scores, segs_d, inl, n_segs, n_segs, keep, s);
  else if (max_len <= 2 * RNT * RCW)
    launch_keep<RNT, 2, false>(scores, segs_d, inl, n_segs, n_segs, keep, s);
  else {
    // one workgroup per CU of the current device, each walking segments
    int dev = 0, cus = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return e;
    const int grid = std::min(n_segs, std::max(cus, 1));
    if (max_len <= 8 * RNT * RCW)
      launch_keep<RNT, 8, false>(scores, segs_d, inl, n_segs, grid, keep, s);
    else
      launch_keep<RNT, 8, true>(scores, segs_d, inl, n_segs, grid, keep, s);
  }
  return hipGetLastError();
}

}  // namespace cc
