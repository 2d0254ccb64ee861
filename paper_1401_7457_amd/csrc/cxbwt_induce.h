// cxbwt_induce.h -- the device side of the build by induced order: sort three
// tenths of the suffixes, derive the order of the others from them.
//
// A suffix is of type S when it is below the suffix that follows it in its
// read, else of type L (equal first bases: as its follower; the last suffix
// of a read, one base before its terminator, is L).  The *samples* are the
// S-type suffixes whose predecessor in the read is L-type: local minima, 29%
// of the suffixes of random reads and at most half of any.  The samples are
// sorted by the digit levels and chunks; then
//
//   left to right   the L-type suffixes of each first base, in order: walking
//                   the terminators and then the buckets A, C, G (the L part
//                   as far as it has grown, then the samples), an item whose
//                   preceding base d is above the bucket's base c makes its
//                   predecessor the next L-type suffix of bucket d;
//   right to left   the S-type suffixes, from the buckets T, G, C down: a
//                   preceding base d below c puts the predecessor before
//                   the S-type suffixes of bucket d found so far.
//
// Each step is a stable partition of a bucket by the preceding base: streams
// instead of 256-way scatters and random window loads, which is what a
// suffix costs in the sort (two to four level passes of 24 B and 1.1 random
// 16-byte loads for every suffix of 20x reads of 100 bases, at 51-57 G
// loads/s on this device whatever the table).  An item is 8 bytes, its
// position and the up to 15 bases before it, so a step reads no text.
// Suffixes c^(k+1) x with the same base run on both sides of the bucket
// border are all written by the step that finds the run's last member: the
// run's k = 0..14 land in regions of their own (their sizes are counted
// beforehand), so a bucket never feeds itself and the steps are few.
#pragma once

#include "cxbwt_kernels.h"

namespace {

// ---------------------------------------------------------------------------
// items: the bases before a position, and the key of a sample
// ---------------------------------------------------------------------------
// Preceding bases ("payload"): the nearest in bits 1..0, then the ones before
// it, then a marker: 01 when more bases precede than are held, 10 when the
// read begins there.  15 bases fit 32 bits.  A payload of 01 alone (nothing
// held, something there) is never stored; 10 alone is a read's first base.
constexpr uint32_t PL_UNKNOWN = 1u;
constexpr uint32_t PL_START = 2u;
constexpr uint32_t PL_BASES = 15;

__host__ __device__ __forceinline__ uint32_t pl_top(uint32_t pl) { return 31u - (uint32_t)__builtin_clz(pl); }
__host__ __device__ __forceinline__ uint32_t pl_len(uint32_t pl) { return pl_top(pl) >> 1; }
__host__ __device__ __forceinline__ bool pl_more(uint32_t pl) { return !(pl_top(pl) & 1u); }

// Payload of position p from the record before p's own (record p/16 - 1 holds
// the 16 bases before p and their start bits; for p < 16 record 0).  `end`:
// p is the end of a read of at least one base, whose own start bit belongs
// to the next read.
__host__ __device__ __forceinline__ uint32_t preceding_from(const TextRec &t, uint64_t p, bool end) {
  const uint32_t o = (uint32_t)(p & 15);
  const uint32_t at = p < 16 ? o : o + 16;  // p's offset in the record
  const uint32_t top = (uint32_t)(t.hi >> 32);
  const uint32_t x = p < 16 ? (o ? top >> (32 - 2 * o) : 0u) : funnel_left(top, (uint32_t)t.hi, 2 * o);
  const uint32_t st = (uint32_t)t.lo & ((end ? 1u << at : 2u << at) - 1u);  // starts at or before p
  const uint32_t dist = st ? at - (31u - (uint32_t)__builtin_clz(st)) : 32u;
  const uint32_t len = dist < PL_BASES ? dist : PL_BASES;
  return (x & ((1u << (2 * len)) - 1u)) | ((dist <= PL_BASES ? PL_START : PL_UNKNOWN) << (2 * len));
}
__host__ __device__ __forceinline__ uint32_t preceding(const TextRec *__restrict__ text, uint64_t p, bool end = false) {
  return preceding_from(text[p < 16 ? 0 : (p >> 4) - 1], p, end);
}

// The nearest seven of them in 15 bits (a start that does not fit becomes
// "more").
constexpr int KEY_PL_BITS = 15;
__host__ __device__ __forceinline__ uint32_t pl_trim(uint32_t pl) {
  const uint32_t len = pl_len(pl);
  if (len < 7 || (len == 7 && pl_more(pl))) return pl;
  if (len == 7) return (pl & 0xFFFu) | (PL_UNKNOWN << 12);
  return (pl & 0x3FFFu) | (PL_UNKNOWN << 14);
}

// Sample keys:  bits 63..20 22 bases, first highest, zero past the read's end
//               bits 19..15 min(bases left, 22)
//               bits 14..0  payload (not compared)
// 22 bases leave room for seven preceding ones: 4% of the samples of random
// reads are further than that from the sample before them and load their
// preceding bases again, against 20% with five (24 bases).
struct SampleKey {
  static constexpr int LAST = 6;
  static constexpr uint32_t FULL = 22;
  static constexpr uint64_t REST = (1ull << KEY_PL_BITS) - 1;
  static __host__ __device__ __forceinline__ uint32_t digit(uint64_t k, int j) {
    if (j >= ENDED) return GeneralKey::ended_digit(clamp(k), j);
    return j < 5 ? (uint32_t)(k >> (56 - 8 * j)) & 0xFFu : j == 5 ? (uint32_t)(k >> 20) & 0xFu : clamp(k);
  }
  static __host__ __device__ __forceinline__ uint32_t clamp(uint64_t k) { return (uint32_t)(k >> KEY_PL_BITS) & 31u; }
  static __host__ __device__ __forceinline__ int digit_of_bit(int top) {
    return top >= 24 ? (63 - top) >> 3 : top >= 20 ? 5 : 6;
  }
  static __device__ __forceinline__ TextRec load(const TextRec *__restrict__ text, uint64_t nb, uint64_t p, uint32_t r) {
    const uint64_t q = p + (uint64_t)FULL * r;
    return text[(q <= nb ? q : nb) >> 4];
  }
  static __device__ __forceinline__ uint64_t combine(const TextRec &t, uint64_t nb, uint64_t p, uint32_t r, uint64_t old);
};

// Bases of the window at q (inside record t) up to the read's end and at most
// `full` (<= 25) of them, first base highest; their number in `clamp`.
__host__ __device__ __forceinline__ uint64_t later_window(const TextRec &t, uint64_t q, uint32_t full, uint32_t &clamp) {
  const uint32_t o = (uint32_t)(q & 15);
  const uint32_t left = first_bit(starts_from(t, o));
  clamp = left < full ? left : full;
  return first_bases(window_at(t, o), clamp);
}

__device__ __forceinline__ uint64_t SampleKey::combine(const TextRec &t, uint64_t nb, uint64_t p, uint32_t r,
                                                       uint64_t old) {
  const uint64_t q = p + (uint64_t)FULL * r;
  if (q > nb) return old & REST;  // never taken for a live suffix
  uint32_t cl;
  const uint64_t x = later_window(t, q, FULL, cl);
  return x | ((uint64_t)cl << KEY_PL_BITS) | (old & REST);
}

// Type of the suffix at p (t its record): its first base, the bases equal to
// it that follow, and whether it is S.  left: bases to the read's end, as far
// as the record shows (64: beyond it).
struct SuffixType {
  uint32_t base, run, left;
  bool s;
  Window bases;
};
__host__ __device__ __forceinline__ SuffixType suffix_type(const TextRec *__restrict__ text, TextRec t, uint64_t p) {
  SuffixType r;
  r.run = 0;
  for (uint64_t q = p;;) {
    const uint32_t o = (uint32_t)(q & 15);
    const Window x = window_at(t, o);
    const uint32_t next = first_bit(starts_from(t, o + 1));
    const uint32_t left = next < 64 ? next + 1 : 64u;
    if (q == p) {
      r.base = x.hi >> 30;
      r.left = left;
      r.bases = x;
    }
    // a set pair: a base unlike the next
    const uint32_t yh = x.hi ^ ((x.hi << 2) | (x.lo >> 30)), yl = x.lo ^ (x.lo << 2);
    const uint32_t k = yh ? (uint32_t)__builtin_clz(yh) >> 1 : yl ? 16u + ((uint32_t)__builtin_clz(yl) >> 1) : 32u;
    if (left <= 27 && k + 1 >= left) {  // the run reaches the terminator
      r.run += left - 1;
      r.s = false;
      return r;
    }
    if (k < 26) {  // the base after the run is inside the 27 valid ones
      r.run += k;
      r.s = (((k < 15 ? x.hi : x.lo) >> (30 - 2 * ((k + 1) & 15))) & 3u) > r.base;
      return r;
    }
    r.run += 26;
    q += 26;  // the same base, in the same read
    t = text[q >> 4];
  }
}

// ---------------------------------------------------------------------------
// counting: what the regions of every bucket will hold, and the samples'
// first digits per tile
// ---------------------------------------------------------------------------
// Per collection: [type (L, S)][base][run 0..14, 15 = longer] suffix counts,
// the longest run per type and base, samples per first base.
constexpr int TC_MAXRUN = 128, TC_SAMPLES = 136, TC_WORDS = 160;
constexpr int RUN_REGIONS = 15;
// Tiles of the text are runs of records, from the one a collection starts in.
constexpr int SMP_NW = 8, SMP_TI = 8;
constexpr uint32_t SMP_RECS = 64u * SMP_NW;
constexpr uint32_t SMP_TILE = 16u * SMP_RECS;  // at most half of the positions are samples
static_assert(SMP_TILE / 2 == 64 * SMP_NW * SMP_TI, "a tile's samples fit the scatter's slots");

// The 16 positions of a record at once.  A mask has a bit per position in the
// position's pair of bits (the low one), first position highest.
constexpr uint32_t LANES = 0x55555555u;
__host__ __device__ __forceinline__ uint32_t reverse_bits(uint32_t x) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_bitreverse32(x);
#else
  uint32_t r = 0;
  for (int i = 0; i < 32; ++i) r |= ((x >> i) & 1u) << (31 - i);
  return r;
#endif
}
// bits 0..15 of x (first position lowest) as a mask
__host__ __device__ __forceinline__ uint32_t to_lanes(uint32_t x) {
  uint32_t y = reverse_bits(x) >> 16;
  y = (y | (y << 8)) & 0x00FF00FFu;
  y = (y | (y << 4)) & 0x0F0F0F0Fu;
  y = (y | (y << 2)) & 0x33333333u;
  return (y | (y << 1)) & LANES;
}
// pairs of a below those of b
__host__ __device__ __forceinline__ uint32_t below(uint32_t a, uint32_t b) {
  const uint32_t ah = a >> 1, bh = b >> 1;
  return ((~ah & bh) | (~(ah ^ bh) & ~a & b)) & LANES;
}
struct RecordTypes {
  uint32_t bases;    // the 16 bases
  uint32_t s;        // S-type positions
  uint32_t sample;
  uint32_t eq, eq2;  // the next base is the same and in the same read; of the 16 positions after these
  uint32_t cut;      // the read ends one or two positions on
  bool slow;         // a run reaches past the 32 positions: s and sample hold only with after_s
};
// after_s: of a slow record, whether the position after its 16 is S.
__host__ __device__ __forceinline__ RecordTypes record_types(const TextRec &t, bool after_s = false) {
  RecordTypes r;
  const uint32_t a = (uint32_t)(t.hi >> 32), b = (uint32_t)t.hi, c = (uint32_t)(t.lo >> 32);
  const uint32_t an = (a << 2) | (b >> 30), bn = (b << 2) | (c >> 30);
  const uint32_t ends = starts_from(t, 1);  // bit i: the read of position i ends with it
  const uint32_t ea = to_lanes(ends), eb = to_lanes(ends >> 16);
  const uint32_t xa = a ^ an, xb = b ^ bn;
  r.bases = a;
  r.eq = ~(xa | (xa >> 1)) & LANES & ~ea;
  r.eq2 = ~(xb | (xb >> 1)) & LANES & ~eb;
  r.slow = r.eq2 == LANES;
  r.cut = (ea << 2) | (eb >> 30) | (ea << 4) | (eb >> 28);
  // S of position 16: of the last position of its run
  const uint32_t last = ~r.eq2 & LANES;
  const uint32_t s16 = last ? (below(b, bn) & ~eb) >> (31 - (uint32_t)__builtin_clz(last)) & 1u : (uint32_t)after_s;
  // S: below the next, or equal to it and the next one S (runs of up to 16
  // here, by doubling)
  uint32_t g = (below(a, an) & ~ea) | (r.eq & s16), p = r.eq;
  g |= p & (g << 2);
  p &= p << 2;
  g |= p & (g << 4);
  p &= p << 4;
  g |= p & (g << 8);
  p &= p << 8;
  r.s = g | (p & (g << 16));
  const uint32_t before = (a >> 2) | ((uint32_t)(t.lo >> 42) << 30);
  r.sample = r.s & below(a, before) & ~to_lanes((uint32_t)t.lo);
  return r;
}
// Positions of the record at 16 w that lie in [a, e); a lies before the
// record's end.
__host__ __device__ __forceinline__ uint32_t lanes_within(uint64_t w, uint64_t a, uint64_t e) {
  const uint64_t p = 16 * w;
  uint32_t m = p < e ? LANES : 0u;
  if (p < a) m &= ~0u >> (2 * (uint32_t)(a - p));
  if (p + 16 > e && p < e) m &= ~(~0u >> (2 * (uint32_t)(e - p)));
  return m;
}
// A slow record's types, from one walk along the run that the 16 positions
// after it belong to; the run of the first of them.  (A walk for each of the
// record's positions, each with its own counter updates: 1.0 ms for 20 Mbases
// with runs of 90 bases in a tenth of the reads, and 0.55 so.)
__host__ __device__ __forceinline__ RecordTypes slow_types(const TextRec *__restrict__ text, const TextRec &t, uint64_t w,
                                                           uint32_t &after_run) {
  const SuffixType ty = suffix_type(text, text[w + 1], 16 * w + 16);
  after_run = ty.run;
  return record_types(t, ty.s);
}
__host__ __device__ __forceinline__ uint32_t slow_samples(const TextRec *__restrict__ text, const TextRec &t, uint64_t w,
                                                          uint32_t valid) {
  uint32_t run;
  return slow_types(text, t, w, run).sample & valid;
}

// Counts of every collection and first-digit counts of every tile's samples.
// A workgroup takes HIST_TILES neighbouring tiles and keeps the type counts in
// registers (one and, one count-and-add per record, class and run length up
// to 3; longer runs one by one).  The types of 16 positions cost about 80
// operations this way: 0.86 -> 0.30 ms per 400 Mbases against a position a lane.
constexpr uint32_t HIST_TILES = 8;
__global__ __launch_bounds__(BLOCK) void k_sample_hist(const Seg *__restrict__ segs, const uint32_t *__restrict__ tile_prefix,
                                                       uint32_t nsegs, uint32_t ntiles,
                                                       const TextRec *__restrict__ text,
                                                       uint32_t *__restrict__ tile_hist,
                                                       uint32_t *__restrict__ counts, uint32_t replicas) {
  constexpr int KR = 4;  // run lengths counted in registers
  __shared__ uint32_t hist[256];
  __shared__ uint32_t cls[TC_WORDS];
  uint32_t acc[KR][8];  // suffixes of a type and base with runs of at least k
  uint32_t smp[3];      // samples of a first base (none begins with T)
  const uint32_t tile0 = blockIdx.x * HIST_TILES, tile1 = min(tile0 + HIST_TILES, ntiles);
  uint32_t s = find_upper(tile_prefix, nsegs, tile0);
  auto clear = [&]() {
#pragma unroll
    for (int k = 0; k < KR; ++k)
#pragma unroll
      for (int j = 0; j < 8; ++j) acc[k][j] = 0;
#pragma unroll
    for (int j = 0; j < 3; ++j) smp[j] = 0;
    for (uint32_t i = threadIdx.x; i < TC_WORDS; i += BLOCK) cls[i] = 0;
  };
  // adds the counts to those of segment s
  auto flush = [&]() {
#pragma unroll
    for (int k = 0; k < KR; ++k)
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const uint32_t v = wave_incl_sum(acc[k][j]);
        if (lane_id() == 63 && v) {
          atomicAdd(&cls[j * 16 + k], v);
          if (k) atomicSub(&cls[j * 16 + k - 1], v);  // counted as at least k - 1 too
        }
      }
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      const uint32_t v = wave_incl_sum(smp[j]);
      if (lane_id() == 63 && v) atomicAdd(&cls[TC_SAMPLES + j], v);
    }
    __syncthreads();
    uint32_t *const out = counts + ((uint64_t)segs[s].coll * replicas + blockIdx.x % replicas) * TC_WORDS;
    for (uint32_t i = threadIdx.x; i < TC_WORDS; i += BLOCK) {
      const uint32_t v = cls[i];
      if (!v) continue;
      if (i >= TC_MAXRUN && i < TC_SAMPLES) atomicMax(&out[i], v);
      else atomicAdd(&out[i], v);
    }
    __syncthreads();
  };
  clear();
  for (uint32_t tile = tile0; tile < tile1; ++tile) {
    if (tile >= tile_prefix[s + 1]) {
      __syncthreads();
      flush();
      while (tile >= tile_prefix[s + 1]) ++s;
      clear();
    }
    const Seg sg = segs[s];
    const uint64_t start = sg.start, end = start + sg.len;
    const uint64_t w0 = start / 16 + (uint64_t)(tile - tile_prefix[s]) * SMP_RECS;
    hist[threadIdx.x] = 0;
    __syncthreads();
#pragma unroll
    for (uint32_t h = 0; h < SMP_RECS / BLOCK; ++h) {
      const uint64_t w = w0 + h * BLOCK + threadIdx.x;
      const uint32_t valid = lanes_within(w, start, end);
      if (!valid) continue;
      const TextRec t = text[w];
      RecordTypes ty = record_types(t);
      uint32_t counted = valid;
      if (ty.slow) {
        // the positions of the run that goes on past the record: one class
        uint32_t run;
        ty = slow_types(text, t, w, run);
        const uint32_t other = ~ty.eq & LANES;
        const uint32_t chain = (other ? (other & (0u - other)) - 1u : ~0u) & valid;
        if (chain) {
          const uint32_t j = ((ty.s & 1u) << 2) | (ty.bases & 3u);
          atomicAdd(&cls[j * 16 + RUN_REGIONS], (uint32_t)__popc(chain));
          atomicMax(&cls[TC_MAXRUN + j], run + 16u - ((uint32_t)__builtin_clz(chain) >> 1));
        }
        counted &= ~chain;
      }
      const uint32_t sample = ty.sample & valid;
      {
        const uint32_t bh = ty.bases >> 1, bl = ty.bases;
        uint32_t m[8];
#pragma unroll
        for (int j = 0; j < 8; ++j)
          m[j] = counted & ((j & 4) ? ty.s : ~ty.s) & ((j & 2) ? bh : ~bh) & ((j & 1) ? bl : ~bl);
        uint32_t e = ty.eq, f = ty.eq2, e1 = ty.eq;  // positions with runs of at least k; the rest shifted along
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[0][j] += (uint32_t)__popc(m[j]);
#pragma unroll
        for (int k = 1; k < KR; ++k) {
#pragma unroll
          for (int j = 0; j < 8; ++j) acc[k][j] += (uint32_t)__popc(m[j] & e);
          e1 = (e1 << 2) | (f >> 30);
          f <<= 2;
          e &= e1;
        }
        // runs of KR and more, one by one: moved from "at least k - 1" to k
        for (uint32_t k = KR; e & counted; ++k) {
          for (uint32_t left = e & counted; left;) {
            const uint32_t bit = 31u - (uint32_t)__builtin_clz(left);
            left &= ~(1u << bit);
            const uint32_t j = (((ty.s >> bit) & 1u) << 2) | ((ty.bases >> bit) & 3u);
            if (k <= RUN_REGIONS) {
              atomicAdd(&cls[j * 16 + k], 1u);
              atomicSub(&cls[j * 16 + k - 1], 1u);
            }
            if (k >= RUN_REGIONS) atomicMax(&cls[TC_MAXRUN + j], k);
          }
          e1 = (e1 << 2) | (f >> 30);
          f <<= 2;
          e &= e1;
        }
      }
#pragma unroll
      for (int j = 0; j < 3; ++j)
        smp[j] += (uint32_t)__popc(sample & ((j & 2) ? ty.bases >> 1 : ~(ty.bases >> 1)) &
                                   ((j & 1) ? ty.bases : ~ty.bases));
      // the digit: the four bases from the position on
      const uint32_t a4 = ty.bases, b4 = (uint32_t)t.hi;
#pragma unroll
      for (int o = 0; o < 16; ++o)
        if (sample & ~ty.cut & (1u << (30 - 2 * o)))
          atomicAdd(&hist[(o <= 12 ? a4 >> (24 - 2 * o) : (a4 << (2 * o - 24)) | (b4 >> (56 - 2 * o))) & 0xFFu], 1u);
      for (uint32_t left = sample & ty.cut; left;) {  // zero past the read's end
        const uint32_t o = (uint32_t)__builtin_clz(left) >> 1;
        left &= ~(1u << (30 - 2 * o));
        const uint32_t n = first_bit(starts_from(t, o + 1)) + 1u;
        atomicAdd(&hist[first_bases(window_at(t, o), min(n, 4u)) >> 56], 1u);
      }
    }
    __syncthreads();
    tile_hist[(uint64_t)tile * 256 + threadIdx.x] = hist[threadIdx.x];
  }
  __syncthreads();
  flush();
}

// Level 1 of the samples: found 16 positions at a time by a lane each, their
// places listed in text order, then a sample a lane: key, scatter by the
// first digit.  (With a pair of positions a lane and no list, 7 of 10 lanes
// made no key: 1.87 -> 0.85 ms per 400 Mbases.)
__global__ __launch_bounds__(64 * SMP_NW) void k_sample_scatter(
    const Seg *__restrict__ segs, const uint32_t *__restrict__ tile_prefix, const uint32_t *__restrict__ group_prefix,
    uint32_t nsegs, const TextRec *__restrict__ text, const uint32_t *__restrict__ tile_hist,
    const uint32_t *__restrict__ gsum, uint64_t *__restrict__ Ko, uint32_t *__restrict__ Ho) {
  __shared__ ScatterSmem<SMP_TI, SMP_NW> S;
  uint16_t *const list = reinterpret_cast<uint16_t *>(S.sh);  // read before the handles are staged
  const uint32_t tile = xcd_tile(blockIdx.x, gridDim.x);
  const uint32_t s = find_upper(tile_prefix, nsegs, tile);
  const Seg sg = segs[s];
  const uint32_t tl = tile - tile_prefix[s];
  const uint64_t start = sg.start, end = start + sg.len;
  const uint64_t w0 = start / 16 + (uint64_t)tl * SMP_RECS;
  uint32_t m = 0;
  {
    const uint64_t w = w0 + threadIdx.x;
    const uint32_t valid = lanes_within(w, start, end);
    uint32_t sample = 0;
    if (valid) {
      const TextRec t = text[w];
      const RecordTypes ty = record_types(t);
      sample = ty.slow ? slow_samples(text, t, w, valid) : ty.sample & valid;
    }
    uint32_t at = block_excl_sum<SMP_NW>((uint32_t)__popc(sample), S.tmp, &m);
    while (sample) {
      const uint32_t o = (uint32_t)__builtin_clz(sample) >> 1;
      sample &= ~(1u << (30 - 2 * o));
      list[at++] = (uint16_t)(16 * threadIdx.x + o);
    }
  }
  __syncthreads();
  // each wave takes an equal run of the list, a multiple of 64
  const uint32_t ni = (m + 64 * SMP_NW - 1) / (64 * SMP_NW);
  const uint32_t first = (threadIdx.x >> 6) * 64 * ni + lane_id();
  uint64_t kr[SMP_TI];
  uint32_t hr[SMP_TI], dig[SMP_TI];
#pragma unroll
  for (int i = 0; i < SMP_TI; ++i) {
    kr[i] = 0;
    hr[i] = 0;
    dig[i] = NODIGIT;
    const uint32_t li = first + i * 64;
    if ((uint32_t)i >= ni || li >= m) continue;
    const uint32_t o16 = list[li];
    const uint64_t w = w0 + (o16 >> 4);
    const uint32_t o = o16 & 15u;
    const TextRec t = text[w], before = text[w ? w - 1 : 0];
    const uint32_t left = first_bit(starts_from(t, o + 1)) + 1u;
    const uint32_t cl = left < SampleKey::FULL ? left : SampleKey::FULL;
    const uint64_t x = first_bases(window_at(t, o), cl), p = 16 * w + o;
    kr[i] = x | ((uint64_t)cl << KEY_PL_BITS) | pl_trim(preceding_from(before, p, false));
    hr[i] = (uint32_t)p;
    dig[i] = (uint32_t)(x >> 56);
  }
  const uint32_t g = group_prefix[s] + tl / GROUP_TILES;
  if (threadIdx.x < 256)
    S.goff[threadIdx.x] =
        (uint64_t)gsum[(uint64_t)g * 256 + threadIdx.x] + tile_hist[(uint64_t)tile * 256 + threadIdx.x];
  uint32_t pos[SMP_TI];
  block_multisplit<SMP_TI, SMP_NW>(dig, pos, S.wcount, S.dstart, S.tmp);
  __syncthreads();  // every wave has read its counters and the list before the stage is written
#pragma unroll
  for (int i = 0; i < SMP_TI; ++i) {
    if (dig[i] != NODIGIT) {
      S.sk[pos[i]] = kr[i];
      S.sh[pos[i]] = hr[i];
    }
  }
  __syncthreads();
  for (uint32_t q = threadIdx.x; q < m; q += 64 * SMP_NW) {
    const uint64_t k = S.sk[q];
    const uint32_t dd = (uint32_t)(k >> 56);
    const uint64_t at = S.goff[dd] + (q - S.dstart[dd]);
    Ko[at] = k;
    Ho[at] = S.sh[q];
  }
}

// ---------------------------------------------------------------------------
// rows: an item per suffix in its final place, and its code in its BWT byte
// until the byte itself is written: bits 1..0 the preceding base, bit 2 set
// for a read's first suffix, bits 6..3 the run of that base (1..15, 15 and
// more alike) when it will be carried on, else 0.
// ---------------------------------------------------------------------------
constexpr uint32_t CODE_START = 4u;
__host__ __device__ __forceinline__ uint32_t code_run(uint32_t code) { return code >> 3; }

// Run of the nearest base of a payload with at least one, as far as it is held.
__host__ __device__ __forceinline__ uint32_t pl_run(uint32_t pl) {
  const uint32_t x = pl ^ ((pl & 3u) * 0x55555555u);
  const uint32_t k = x ? (uint32_t)__builtin_ctz(x) >> 1 : 16u;
  const uint32_t len = pl_len(pl);
  return k < len ? k : len;
}

// Code of an item with payload pl in bucket c.  CODE_LOOK when the payload
// does not show enough: nothing held, or a run without its end in an item
// that a step will carry on (left to right any other base, then only a lower
// one); with the payload read from the text again it always does, so a stored
// item that is carried on has its whole run, up to 15, in its payload.
constexpr uint32_t CODE_LOOK = 0x80u;
template <bool LTR>
__host__ __device__ __forceinline__ uint32_t shown_code(uint32_t c, uint32_t pl) {
  if (pl == PL_UNKNOWN) return CODE_LOOK;
  if (pl == PL_START) return CODE_START;
  const uint32_t e = pl & 3u;
  if (LTR ? e == c : e >= c) return e;
  const uint32_t r = pl_run(pl), len = pl_len(pl);
  return r == len && r < PL_BASES && pl_more(pl) ? CODE_LOOK : e | (r << 3);
}
template <bool LTR>
__device__ __forceinline__ uint32_t item_code(const TextRec *__restrict__ text, uint32_t c, uint64_t p, uint32_t &pl) {
  uint32_t code = shown_code<LTR>(c, pl);
  if (code == CODE_LOOK) {
    pl = preceding(text, p);
    code = shown_code<LTR>(c, pl);
  }
  return code;
}

// The sorted samples.
struct SampleOut {
  uint32_t *pl, *h;
  uint8_t *code;
};
__device__ __forceinline__ void put_sample(const SampleOut &o, uint64_t at, uint64_t key, uint32_t first, uint32_t h,
                                           const TextRec *__restrict__ text) {
  uint32_t pl = (uint32_t)(key & SampleKey::REST);
  const uint32_t code = item_code<true>(text, first, h, pl);
  o.pl[at] = pl;
  o.h[at] = h;
  o.code[at] = (uint8_t)code;
}

// Groups of identical samples too large for one chunk, in place.
__global__ __launch_bounds__(BLOCK) void k_sample_final(const Seg *__restrict__ segs, const uint32_t *__restrict__ tile_prefix,
                                                        uint32_t nsegs, uint32_t tile_len, const uint64_t *__restrict__ keys0,
                                                        const uint64_t *__restrict__ keys1, const uint32_t *__restrict__ hdl0,
                                                        const uint32_t *__restrict__ hdl1, const TextRec *__restrict__ text,
                                                        SampleOut out) {
  const uint32_t tile = blockIdx.x;
  const uint32_t s = find_upper(tile_prefix, nsegs, tile);
  const Seg sg = segs[s];
  const uint64_t t0 = sg.start + (uint64_t)(tile - tile_prefix[s]) * tile_len;
  const uint64_t t1 = min(t0 + (uint64_t)tile_len, (uint64_t)sg.start + sg.len);
  const uint64_t *K = sg.buf ? keys1 : keys0;
  const uint32_t *H = sg.buf ? hdl1 : hdl0;
  for (uint64_t j = t0 + threadIdx.x; j < t1; j += BLOCK) {
    const uint32_t h = H[j];
    const uint64_t k = K[j];
    // a key of a later window does not hold the first base
    put_sample(out, j, k, sg.r ? base_in(text[h >> 4], h & 15u) : (uint32_t)(k >> 62), h, text);
  }
}

// ---------------------------------------------------------------------------
// the chunk kernel of the samples: one wave sorts a chunk in LDS, as k_local
// does, with keys of its own: bits 63..14 up to 25 bases, 13..9 the clamped
// length, 8..0 the sample's place in the chunk as loaded.  The place is the
// stable order among equal ordering bits, so keys are distinct and a rank is
// one count of smaller keys; only keys move, the handle and what else is
// known of a sample stay at its place.  A tied sample loads a record for a
// window of 25 bases.  PAIR: it loads the record after it too, which is in the
// same request three times of four, for a window of 18 more that waits at its
// place, while the handles, read once in two windows now, are not held.
//
// What bounds it is latency and requests: half of the issue slots are empty,
// and the waves of a CU are as many as its LDS holds (17 or 21 bytes a
// sample).  With PAIR, buckets are packed into chunks of at most 256, 28
// waves a CU, and only one above that takes a chunk of up to 512 (15 waves)
// before it is worth a level.
//
// PAIR is for a mean read length of 150 bases and more, whose ties pass more
// windows (the mean, which the sizes give, and not the caller's bound: a bound of
// 250 on reads of 100 says nothing of them).  Single records and pairs, 250
// Mbases at 20x: reads of 100 bases 7.15 and 7.15 ms, 125 7.53 and 7.47, 150 7.90
// and 7.63, 200 8.59 and 8.03, 400 10.5 and 9.38; 1 Gbase 25.7 and 25.7, 26.7 and
// 26.0, 28.7 and 27.0, 31.5 and 28.0, 39.5 and 34.0; 2 Gbases of 100 bases with
// repeats are 3% slower by pairs, and 60 Mbases 4% (100 bases) to 1% (400).
// (Text lines of 64 bytes, three windows each: equal at 200 Mbases, 3% slower at
// 2 G.  Chunks of 256 alone, without those of 512: 2 Gbases 54 -> 66 ms.)
// ---------------------------------------------------------------------------
constexpr uint32_t SAMPLE_CHUNK = 512, PAIR_PACK = 256;
constexpr uint64_t PAIR_MEAN_READ = 150;
constexpr uint64_t PLACE = 511ull;
constexpr uint32_t WINDOW_0 = 25, WINDOW_1 = 18;  // of a pair of records: 59 bases and 58 starts, less an offset

__device__ __forceinline__ uint32_t place_digit(uint64_t k, int j) {
  return j < 5 ? (uint32_t)(k >> (56 - 8 * j)) & 0xFFu : j == 5 ? (uint32_t)(k >> 20) & 0xFu : (uint32_t)(k >> 9) & 31u;
}
__device__ __forceinline__ uint64_t place_mask(int j) {
  return j < 5 ? 0xFFull << (56 - 8 * j) : j == 5 ? 0xFull << 20 : 31ull << 9;
}

// The windows of q (offset o in its record t; u the record after it): bases
// and clamped length as in a chunk key, place zero.
__device__ __forceinline__ void pair_windows(const TextRec &t, const TextRec &u, uint32_t o, uint64_t &w0, uint64_t &w1) {
  const uint32_t near = first_bit(starts_from(t, o)), far = 16u + first_bit(starts_from(u, o));
  const uint32_t left = near < 16 ? near : far;  // to the read's end
  const uint32_t n0 = min(left, WINDOW_0), n1 = min(left - n0, WINDOW_1);
  w0 = first_bases(window_at(t, o), n0) | ((uint64_t)n0 << 9);
  const uint32_t r = o + WINDOW_0 - 16;  // in u
  const uint32_t a = (uint32_t)(u.hi >> 32), b = (uint32_t)u.hi, c = (uint32_t)(u.lo >> 32);
  const uint32_t x = r < 16 ? a : b, y = r < 16 ? b : c, z = r < 16 ? c : 0u;
  w1 = first_bases(Window{funnel_left(x, y, 2 * (r & 15u)), funnel_left(y, z, 2 * (r & 15u))}, n1) | ((uint64_t)n1 << 9);
}

template <int LI, bool PAIR>
struct SampleSmem {
  static constexpr int CHUNK = LOCAL_WG * LI;
  uint64_t K[CHUNK];     // key of each position
  uint64_t W[PAIR ? CHUNK : 1];  // by place: the window after the current one
  uint32_t H[PAIR ? 1 : CHUNK];  // by place: handle
  union {
    struct {  // as in LocalSmem
      uint16_t live[CHUNK];
      uint16_t gr[CHUNK];
      uint16_t hp[CHUNK / 2 + 1];
    };
    struct {
      uint16_t cnt[256];
      uint16_t dstart[256];
    };
  };
  uint32_t headw[CHUNK / 32];
};
template <int LI, bool PAIR>
__device__ __forceinline__ bool sample_head(const SampleSmem<LI, PAIR> &S, uint32_t j) {
  return (S.headw[j >> 5] >> (j & 31u)) & 1u;
}

// wave_split on keys alone.
template <int LI, bool PAIR>
__device__ __forceinline__ void split_places(SampleSmem<LI, PAIR> &S, uint32_t m, int sel, uint32_t lane, uint64_t lt) {
  for (uint32_t x = lane; x < 256; x += LOCAL_WG) S.cnt[x] = 0;
  __syncthreads();
  uint64_t kr[LI];
  uint32_t dig[LI], pos[LI];
#pragma unroll
  for (int i = 0; i < LI; ++i) {
    const uint32_t j = i * LOCAL_WG + lane;
    const bool valid = j < m;
    dig[i] = NODIGIT;
    if (valid) {
      kr[i] = S.K[j];
      dig[i] = place_digit(kr[i], sel);
    }
    if (i * LOCAL_WG >= (int)m) continue;
    const uint64_t peers = wave_match8(dig[i], __ballot(valid));
    if (valid) {
      const uint32_t before = S.cnt[dig[i]];
      pos[i] = before + (uint32_t)__popcll(peers & lt);
      if ((peers & lt) == 0) S.cnt[dig[i]] = before + (uint32_t)__popcll(peers);
    }
    __syncthreads();
  }
  const uint32_t c0 = S.cnt[4 * lane], c1 = S.cnt[4 * lane + 1], c2 = S.cnt[4 * lane + 2], c3 = S.cnt[4 * lane + 3];
  const uint32_t tot = c0 + c1 + c2 + c3;
  const uint32_t ex = wave_incl_sum(tot) - tot;
  S.dstart[4 * lane] = ex;
  S.dstart[4 * lane + 1] = ex + c0;
  S.dstart[4 * lane + 2] = ex + c0 + c1;
  S.dstart[4 * lane + 3] = ex + c0 + c1 + c2;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < LI; ++i)
    if (dig[i] != NODIGIT) S.K[S.dstart[dig[i]] + pos[i]] = kr[i];
  __syncthreads();
}

// The bitonic network of bitonic_group on keys that are distinct.
template <int LI, bool PAIR>
__device__ __forceinline__ void bitonic_places(SampleSmem<LI, PAIR> &S, uint32_t a, uint32_t m, uint32_t lane) {
  uint32_t P = 2;
  while (P < m) P <<= 1;
  for (uint32_t k = 2; k <= P; k <<= 1) {
    for (uint32_t d = k >> 1; d > 0; d >>= 1) {
      for (uint32_t q = lane; q < P / 2; q += LOCAL_WG) {
        uint32_t i, l;
        if (d == k >> 1) {  // mirrored pairs of a block of k
          const uint32_t blk = q / d, off = q % d;
          i = blk * k + off;
          l = blk * k + (k - 1 - off);
        } else {
          i = (q / d) * 2 * d + (q % d);
          l = i + d;
        }
        if (l < m) {
          const uint64_t ki = S.K[a + i], kl = S.K[a + l];
          if (ki > kl) {
            S.K[a + i] = kl;
            S.K[a + l] = ki;
          }
        }
      }
      __syncthreads();
    }
  }
}

template <int LI, bool PAIR>
__device__ __forceinline__ void sort_big_places(SampleSmem<LI, PAIR> &S, uint32_t ngroups, uint32_t lane) {
  for (uint32_t g0 = 0; g0 < ngroups; g0 += LOCAL_WG) {
    const uint32_t g = g0 + lane;
    const bool big = g < ngroups && (uint32_t)S.hp[g + 1] - S.hp[g] > BIG_GROUP;
    uint64_t todo = __ballot(big);
    while (todo) {
      const uint32_t b = g0 + (uint32_t)__builtin_ctzll(todo);
      todo &= todo - 1;
      const uint32_t x0 = S.hp[b];
      bitonic_places(S, (uint32_t)S.live[x0], (uint32_t)S.hp[b + 1] - x0, lane);
    }
  }
}

// #{t in [a, e) : k_t < v} by the keys' low words (T = uint32_t) or whole, four
// reads a step.
template <typename T>
__device__ __forceinline__ uint32_t count_smaller(const uint64_t *k, uint32_t a, uint32_t e, T v) {
  uint32_t c = 0;
  const uint64_t *p = k + a;
  const uint64_t *const pe = k + e, *const pe3 = k + (e >= 3 ? e - 3 : 0);
  for (; p < pe3; p += 4)
    c += (uint32_t)((T)p[0] < v) + (uint32_t)((T)p[1] < v) + (uint32_t)((T)p[2] < v) + (uint32_t)((T)p[3] < v);
  for (; p < pe; ++p) c += (uint32_t)((T)*p < v);
  return c;
}

template <int LI, int OCC, bool PAIR>
__global__ __launch_bounds__(LOCAL_WG, OCC) void k_sample_chunk(
    const Seg *__restrict__ chunks, const uint64_t *__restrict__ keys0, const uint64_t *__restrict__ keys1,
    const uint32_t *__restrict__ hdl0, const uint32_t *__restrict__ hdl1, const TextRec *__restrict__ text,
    uint32_t maxlen, uint32_t above, SampleOut out, uint32_t *status, unsigned long long *fetches) {
  static_assert(LI * LOCAL_WG <= 512, "a place in a chunk is 9 bits");
  __shared__ SampleSmem<LI, PAIR> S;
  const uint32_t lane = threadIdx.x;
  const uint64_t le = lanemask_lt() | (1ull << lane);
  uint32_t nfetch = 0;
  const Seg ch = chunks[blockIdx.x];
  const uint32_t m = ch.len;
  if (m <= above || m > LI * LOCAL_WG) return;  // the other kernel's
  const uint64_t *Kg = (ch.buf ? keys1 : keys0) + ch.start;
  const uint32_t *Hg = (ch.buf ? hdl1 : hdl0) + ch.start;
  auto handle = [&](uint32_t place) { return PAIR ? Hg[place] : S.H[PAIR ? 0 : place]; };
  {
    uint64_t lk[LI];
    uint32_t lh[LI];
#pragma unroll
    for (int i = 0; i < LI; ++i) {
      const uint32_t j = i * LOCAL_WG + lane;
      lk[i] = Kg[j < m ? j : m - 1];
      if (!PAIR) lh[i] = Hg[j < m ? j : m - 1];
    }
#pragma unroll
    for (int i = 0; i < LI; ++i) {
      const uint32_t j = i * LOCAL_WG + lane;
      if (j < m) {
        S.K[j] = (lk[i] & (~0ull << 20)) | ((uint64_t)SampleKey::clamp(lk[i]) << 9) | j;
        if (!PAIR) S.H[PAIR ? 0 : j] = lh[i];
      }
    }
  }
  __syncthreads();
  // as k_local: ordered by digits d and d + 1 first (one bucket: d + 1 is
  // enough), then groups of equal digits
  const int d0 = ch.d;
  const bool two = d0 < SampleKey::LAST;
  if (two) {
    const bool one_bucket = !ch.unsplit && place_digit(S.K[0], d0) == place_digit(S.K[m - 1], d0);
    split_places(S, m, d0 + 1, lane, le & ~(1ull << lane));
    if (!one_bucket) split_places(S, m, d0, lane, le & ~(1ull << lane));
  }
  const uint64_t hmask = two ? (place_mask(d0) | place_mask(d0 + 1)) : place_mask(d0);
  uint32_t n = 0, ngroups = 0;
  {
    uint32_t run = 0;
#pragma unroll
    for (int i = 0; i < LI; ++i) {
      if (i * LOCAL_WG >= (int)m) break;
      const uint32_t j = i * LOCAL_WG + lane;
      bool keep = false, h = false;
      if (j < m) {
        const uint64_t kj = S.K[j];
        h = j == 0 || ((kj ^ S.K[j - 1]) & hmask) != 0;
        const bool hn = j + 1 >= m || ((S.K[j + 1] ^ kj) & hmask) != 0;
        keep = !(h && hn);
      }
      const uint64_t hm = __ballot(h);
      if (lane == 0) {
        S.headw[2 * i] = (uint32_t)hm;
        S.headw[2 * i + 1] = (uint32_t)(hm >> 32);
      }
      const uint64_t kb = __ballot(keep);
      const uint64_t hb = __ballot(keep && h);
      if (keep) {
        const uint32_t xn = n + (uint32_t)__popcll(kb & (le >> 1));
        const uint32_t g = run + (uint32_t)__popcll(hb & le) - 1u;
        S.live[xn] = (uint16_t)j;
        S.gr[xn] = (uint16_t)g;
        if (h) S.hp[g] = (uint16_t)xn;
      }
      n += (uint32_t)__popcll(kb);
      run += (uint32_t)__popcll(hb);
    }
    if (lane == 0) S.hp[run] = (uint16_t)n;
    ngroups = run;
  }
  __syncthreads();
  uint32_t depth = SampleKey::FULL * ((uint32_t)ch.r + 1);  // bases compared once the current window is sorted
  uint32_t full = SampleKey::FULL;
  bool held = false;  // the next window has come with the current one
  bool fetch_round = false;
  for (;;) {
    if (!fetch_round) {
      if (n == 0) break;
    } else {
      // drop single samples and runs of equal keys that end inside the
      // window; see k_local
      uint32_t kept = 0, run = 0;
#pragma unroll
      for (int i = 0; i < LI; ++i) {
        if (i * LOCAL_WG >= (int)n) break;
        const uint32_t x = i * LOCAL_WG + lane;
        bool keep = false, hd = false, fresh = false;
        uint16_t pos = 0;
        if (x < n) {
          pos = S.live[x];
          const uint64_t kp = S.K[pos];
          hd = sample_head(S, pos);
          if (!hd) fresh = hd = ((kp ^ S.K[pos - 1]) & ~PLACE) != 0;
          bool next_hd = true;
          if (x + 1 < n) {
            const uint32_t p1 = S.live[x + 1];
            next_hd = sample_head(S, p1);
            if (!next_hd) next_hd = ((S.K[p1] ^ kp) & ~PLACE) != 0;
          }
          keep = !(hd && next_hd) && ((uint32_t)(kp >> 9) & 31u) == full;
        }
        const uint64_t kb = __ballot(keep);
        const uint64_t hb = __ballot(keep && hd);
        if (keep) {
          const uint32_t xn = kept + (uint32_t)__popcll(kb & (le >> 1));
          const uint32_t g = run + (uint32_t)__popcll(hb & le) - 1u;
          S.live[xn] = pos;
          S.gr[xn] = (uint16_t)g;
          if (hd) S.hp[g] = (uint16_t)xn;
          if (fresh) atomicOr(&S.headw[pos >> 5], 1u << (pos & 31u));
        }
        kept += (uint32_t)__popcll(kb);
        run += (uint32_t)__popcll(hb);
      }
      n = kept;
      ngroups = run;
      if (n == 0) break;
      if (lane == 0) S.hp[run] = (uint16_t)n;
      __syncthreads();
      if (depth > maxlen) {  // a suffix this deep does not exist
        if (lane == 0) atomicOr(status, ST_WINDOW_BOUND);
        break;
      }
      // the next window of every live sample: all of them hold `depth` bases,
      // so it starts inside the read or at its end, and all have loaded the
      // same windows
      if (!PAIR || !held) {
        for (uint32_t x0 = 0; x0 < n; x0 += FETCH_BATCH * LOCAL_WG) {
          TextRec t[FETCH_BATCH], u[FETCH_BATCH];
          uint32_t tp[FETCH_BATCH], at[FETCH_BATCH], o[FETCH_BATCH];
#pragma unroll
          for (int i = 0; i < FETCH_BATCH; ++i) {
            const uint32_t x = x0 + i * LOCAL_WG + lane;
            tp[i] = S.live[x < n ? x : 0];
            at[i] = (uint32_t)(S.K[tp[i]] & PLACE);
            const uint64_t q = (uint64_t)handle(at[i]) + depth;
            o[i] = (uint32_t)(q & 15);
            t[i] = text[q >> 4];
            if (PAIR) u[i] = text[(q >> 4) + 1];
          }
#pragma unroll
          for (int i = 0; i < FETCH_BATCH; ++i) {
            const uint32_t x = x0 + i * LOCAL_WG + lane;
            if (x < n) {
              if constexpr (PAIR) {
                uint64_t w0, w1;
                pair_windows(t[i], u[i], o[i], w0, w1);
                S.K[tp[i]] = w0 | at[i];
                S.W[at[i]] = w1;
              } else {
                const uint32_t n0 = min(first_bit(starts_from(t[i], o[i])), WINDOW_0);
                S.K[tp[i]] = first_bases(window_at(t[i], o[i]), n0) | ((uint64_t)n0 << 9) | at[i];
              }
            }
          }
        }
        if (lane == 0) nfetch += n;
        full = WINDOW_0;
      } else {
        for (uint32_t x = lane; x < n; x += LOCAL_WG) {
          const uint32_t j = S.live[x];
          const uint32_t at = (uint32_t)(S.K[j] & PLACE);
          S.K[j] = S.W[PAIR ? at : 0] | at;
        }
        full = WINDOW_1;
      }
      held = !held;
      depth += full;
      __syncthreads();
    }
    // rank inside each live group (a run of positions): every rank is taken
    // before any entry moves.  After two splits from digit d >= 2 a group
    // agrees in its keys' high words.
    bool big_groups = false;
    const bool low_words = !fetch_round && two && d0 >= 2;
    for (uint32_t x = lane; x < n; x += LOCAL_WG) {
      const uint32_t j = S.live[x];
      const uint32_t g = S.gr[x];
      const uint32_t x0 = S.hp[g];
      const uint32_t a = S.live[x0];
      const uint32_t e = a + ((uint32_t)S.hp[g + 1] - x0);
      if (e - a > BIG_GROUP) {
        S.gr[x] = (uint16_t)j;
        big_groups = true;
        continue;
      }
      const uint64_t kj = S.K[j];
      const uint32_t c = low_words ? count_smaller<uint32_t>(S.K, a, e, (uint32_t)kj) : count_smaller<uint64_t>(S.K, a, e, kj);
      S.gr[x] = (uint16_t)(a + c);
    }
    __syncthreads();
    {
      uint64_t sk[LI];
      uint32_t sd[LI];
#pragma unroll
      for (int i = 0; i < LI; ++i) {
        const uint32_t x = i * LOCAL_WG + lane;
        if (x < n) {
          sk[i] = S.K[S.live[x]];
          sd[i] = S.gr[x];
        }
      }
      __syncthreads();
#pragma unroll
      for (int i = 0; i < LI; ++i) {
        const uint32_t x = i * LOCAL_WG + lane;
        if (x < n) S.K[sd[i]] = sk[i];
      }
    }
    __syncthreads();
    if (__ballot(big_groups)) sort_big_places(S, ngroups, lane);
    fetch_round = true;
  }
  {
    uint64_t g[LI];
    uint32_t hh[LI];
#pragma unroll
    for (int i = 0; i < LI; ++i) {
      const uint32_t j = i * LOCAL_WG + lane;
      const uint32_t at = j < m ? (uint32_t)(S.K[j] & PLACE) : 0u;
      g[i] = Kg[at];
      hh[i] = handle(at);
    }
#pragma unroll
    for (int i = 0; i < LI; ++i) {
      const uint32_t j = i * LOCAL_WG + lane;
      if (j >= m) continue;
      const uint32_t h = hh[i];
      // a key of a later window does not hold the first base
      const uint32_t first = ch.r ? base_in(text[h >> 4], h & 15u) : (uint32_t)(g[i] >> 62);
      put_sample(out, (uint64_t)ch.start + j, g[i], first, h, text);
    }
  }
  if (lane == 0 && nfetch) atomicAdd(stat_slot(fetches), (unsigned long long)nfetch);
}

// ---------------------------------------------------------------------------
// the steps: stable partitions of a bucket by the preceding base
// ---------------------------------------------------------------------------
// A step's sources, in order: runs of rows, of samples or (the first step) of
// reads, a wave tile at a time; tiles in groups of GROUP_TILES within a
// collection.  Classes: (base d, run index k) at d * 16 + k, one per lane.
// A tile is what a wave loads at once: a build of 20 Mbases fills the device
// only so, and larger ones have fewer waves at work on their last tiles (512
// rows instead of 2048, with the scan of the groups' totals shared by a
// workgroup: 20 Mbases 1.25 -> 1.06 ms, 20 at 2000x 5.0 -> 4.6, 400 11.3 -> 10.9,
// 2 Gbases 53.8 -> 51.3).
constexpr uint32_t IND_SLOTS = 8;
constexpr uint32_t IND_TILE = 64 * IND_SLOTS;
constexpr uint32_t IND_BATCH = 8;  // slots whose loads are in flight together
enum { SRC_ROWS = 0, SRC_SAMPLES = 1, SRC_READS = 2 };
struct IndSeg {
  uint32_t start, len, coll, src;
};
struct IndStep {
  const IndSeg *segs;
  const uint32_t *tile_prefix;                 // nsegs + 1
  const uint32_t *coll_tiles, *coll_groups;    // ncoll + 1 each
  uint32_t nsegs, ntiles, ncoll, base;         // base: the bucket's (4: the terminators)
};
struct IndData {
  uint2 *rows;  // {position, payload}
  uint8_t *bwt;
  const CollMap *cmap;
  SampleOut smp;
  const TextRec *text;
  const uint32_t *srank;
  const uint64_t *offsets;
  uint64_t *start_row;
  uint32_t *hist;    // per tile and class
  uint32_t *gtot;    // per group and class
  uint32_t *cursor;  // per collection, direction and class: where the next item goes (S: ends)
  uint32_t *status;
  uint64_t nb;
};

// Entry x of a segment: position, payload, code.
__device__ __forceinline__ void ind_read_end(const IndData &D, uint64_t i, uint32_t &p, uint32_t &pl, uint32_t &code) {
  const uint64_t a = D.offsets[i], e = D.offsets[i + 1];
  p = 0;
  pl = PL_START;
  code = CODE_START;
  if (e > a) {
    pl = preceding(D.text, e, true);
    p = (uint32_t)e;
    code = (pl & 3u) | (pl_run(pl) << 3);
  }
}

template <bool LTR>
__device__ __forceinline__ bool ind_taken(uint32_t code, uint32_t c) {
  return !(code & CODE_START) && (LTR ? c == 4 || (code & 3u) > c : (code & 3u) < c);
}

// Class counts of every wave tile.
template <bool LTR>
__global__ __launch_bounds__(BLOCK) void k_ind_count(IndStep P, IndData D) {
  constexpr uint32_t REP = 8;  // counter copies per wave, against conflicts on the hot classes
  __shared__ uint32_t cnt[WAVES][REP][65];
  const uint32_t w = threadIdx.x >> 6, l = lane_id();
  const uint32_t tile = (uint32_t)__builtin_amdgcn_readfirstlane((int)(blockIdx.x * WAVES + w));
  for (uint32_t r = 0; r < REP; ++r) cnt[w][r][l] = 0;
  __syncthreads();
  if (tile < P.ntiles) {
    const uint32_t s = find_upper(P.tile_prefix, P.nsegs, tile);
    const IndSeg sg = P.segs[s];
    const uint32_t t0 = (tile - P.tile_prefix[s]) * IND_TILE;
    const uint32_t m = min(IND_TILE, sg.len - t0);
    const uint64_t at0 = (uint64_t)sg.start + t0;
    const uint8_t *codes = sg.src == SRC_SAMPLES ? D.smp.code + at0 : D.bwt + D.cmap[sg.coll].out_shift + at0;
    for (uint32_t x0 = 0; x0 < m; x0 += IND_BATCH * 64) {
      uint32_t code[IND_BATCH];
#pragma unroll
      for (uint32_t i = 0; i < IND_BATCH; ++i) {
        const uint32_t x = x0 + i * 64 + l;
        code[i] = CODE_START;
        if (x < m) {
          uint32_t p, pl;
          if (LTR && sg.src == SRC_READS) ind_read_end(D, at0 + x, p, pl, code[i]);
          else code[i] = codes[x];
        }
      }
#pragma unroll
      for (uint32_t i = 0; i < IND_BATCH; ++i)
        if (ind_taken<LTR>(code[i], P.base))
          atomicAdd(&cnt[w][l % REP][(code[i] & 3u) * 16 + code_run(code[i])], 1u);
    }
  }
  __syncthreads();
  if (tile < P.ntiles) {
    uint32_t v = 0;
    for (uint32_t r = 0; r < REP; ++r) v += cnt[w][r][l];
    // runs longer than k: sum over the classes above, within the 16 of a base
    uint32_t sum = v;
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) {
      const uint32_t t = __shfl_down(sum, o, 16);
      if ((l & 15u) + o < 16) sum += t;
    }
    D.hist[(uint64_t)tile * 64 + l] = sum - v;
  }
}

// Tile counts to exclusive prefixes inside a group, and the group's totals.
__global__ __launch_bounds__(BLOCK) void k_ind_group(IndStep P, IndData D) {
  constexpr uint32_t PER = GROUP_TILES / WAVES;
  __shared__ uint32_t tot[WAVES][64];
  const uint32_t g = blockIdx.x;
  const uint32_t c = find_upper(P.coll_groups, P.ncoll, g);
  const uint32_t tb = P.coll_tiles[c] + (g - P.coll_groups[c]) * GROUP_TILES;
  const uint32_t te = min(tb + (uint32_t)GROUP_TILES, P.coll_tiles[c + 1]);
  const uint32_t w = threadIdx.x >> 6, l = lane_id();
  const uint32_t t0 = tb + w * PER;
  uint32_t x[PER], sum = 0;
#pragma unroll
  for (uint32_t i = 0; i < PER; ++i) x[i] = t0 + i < te ? D.hist[(uint64_t)(t0 + i) * 64 + l] : 0u;
#pragma unroll
  for (uint32_t i = 0; i < PER; ++i) sum += x[i];
  tot[w][l] = sum;
  __syncthreads();
  uint32_t run = 0;
  for (uint32_t ww = 0; ww < w; ++ww) run += tot[ww][l];
#pragma unroll
  for (uint32_t i = 0; i < PER; ++i) {
    if (t0 + i < te) D.hist[(uint64_t)(t0 + i) * 64 + l] = run;
    run += x[i];
  }
  if (w == WAVES - 1) D.gtot[(uint64_t)g * 64 + l] = run;
}

// Group totals to first places, from the collection's cursors; one workgroup
// a collection, its waves a run of groups each (one wave alone took 0.83 ms of
// the 52 of 2 Gbases).  Right to left a step's items go in front of the
// earlier ones.
constexpr int TOP_WAVES = 16;
template <bool LTR>
__global__ __launch_bounds__(64 * TOP_WAVES) void k_ind_top(IndStep P, IndData D) {
  constexpr uint32_t NB = 8;
  __shared__ uint32_t tot[TOP_WAVES][64];
  const uint32_t c = blockIdx.x, w = threadIdx.x >> 6, l = lane_id();
  const uint32_t g0 = P.coll_groups[c], g1 = P.coll_groups[c + 1];
  const uint32_t per = (g1 - g0 + TOP_WAVES - 1) / TOP_WAVES;
  const uint32_t b = min(g0 + w * per, g1), e = min(b + per, g1);
  uint32_t *cur = D.cursor + ((uint64_t)c * 2 + (LTR ? 0 : 1)) * 64 + l;
  const uint32_t from = *cur;
  uint32_t sum = 0;
  for (uint32_t g = b; g < e; g += NB) {
    uint32_t x[NB];
#pragma unroll
    for (uint32_t i = 0; i < NB; ++i) x[i] = g + i < e ? D.gtot[(uint64_t)(g + i) * 64 + l] : 0u;
#pragma unroll
    for (uint32_t i = 0; i < NB; ++i) sum += x[i];
  }
  tot[w][l] = sum;
  __syncthreads();  // (and every wave has read the cursors)
  uint32_t before = 0, total = 0;
  for (uint32_t ww = 0; ww < (uint32_t)TOP_WAVES; ++ww) {
    before += ww < w ? tot[ww][l] : 0u;
    total += tot[ww][l];
  }
  uint32_t run = (LTR ? from : from - total) + before;
  if (w == 0) *cur = LTR ? from + total : from - total;
  for (uint32_t g = b; g < e; g += NB) {
    uint32_t x[NB];
#pragma unroll
    for (uint32_t i = 0; i < NB; ++i) x[i] = g + i < e ? D.gtot[(uint64_t)(g + i) * 64 + l] : 0u;
#pragma unroll
    for (uint32_t i = 0; i < NB; ++i) {
      if (g + i < e) D.gtot[(uint64_t)(g + i) * 64 + l] = run;
      run += x[i];
    }
  }
}

// Work that waits for a load, put off until a wave's worth of it is there: a
// lane in sixty needs one (a payload that has run out, a read's first
// suffix), and one lane's load would hold up its wave for as long as sixty
// four's.  Entries are (a, b, c) as the user of the list defines.
struct WaveList {
  uint32_t a[64], b[64];
  uint8_t c[64];
};
// Appends the entries of the lanes with `on` (n: entries held, the same in
// every lane); true when the list must be worked off first.
__device__ __forceinline__ bool list_full(uint32_t n, uint64_t on) { return n + (uint32_t)__popcll(on) > 64; }
__device__ __forceinline__ void list_append(WaveList &L, uint32_t &n, bool on, uint64_t mask, uint32_t a, uint32_t b,
                                            uint32_t c) {
  if (on) {
    const uint32_t at = n + bits_below_lane(mask);
    L.a[at] = a;
    L.b[at] = b;
    L.c[at] = (uint8_t)c;
  }
  n += (uint32_t)__popcll(mask);
}
__device__ __forceinline__ void wave_lds_fence() {  // LDS written by some lanes is read by others
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ void put_row(const IndData &D, const CollMap &cm, uint64_t g, uint32_t q, uint32_t pl,
                                        uint32_t code, bool read = true) {
  if (g >= D.nb) {
    atomicOr(D.status, ST_LIST_OVERFLOW);
    return;
  }
  if (read) D.rows[g] = make_uint2(q, pl);
  D.bwt[g + cm.out_shift] = (uint8_t)code;
}

// Rows (a: row, b: position, c: bucket) whose payload comes from the text.
template <bool LTR>
__device__ __forceinline__ void put_looked_up(const IndData &D, const CollMap &cm, WaveList &L, uint32_t &n) {
  wave_lds_fence();
  const uint32_t l = lane_id();
  if (l < n) {
    const uint32_t q = L.b[l];
    const uint32_t pl = preceding(D.text, q);
    put_row(D, cm, L.a[l], q, pl, shown_code<LTR>(L.c[l], pl));
  }
  n = 0;
  wave_lds_fence();
}

// Copy k of the run that precedes item (p, pl), r long: the suffix k + 1 bases
// earlier, in bucket d at row g, for the lanes with `on`.
template <bool LTR>
__device__ __forceinline__ void ind_put(const IndData &D, const CollMap &cm, WaveList &L, uint32_t &n, bool on,
                                        uint32_t g, uint32_t d, uint32_t k, uint32_t r, uint32_t p, uint32_t pl) {
  const uint32_t q = p - 1 - k;
  const uint32_t x = pl >> (2 * (k + 1));
  const uint32_t code = k + 1 < r ? d : shown_code<LTR>(d, x);
  const bool look = on && code == CODE_LOOK;
  // Right to left nothing reads a row of A but for a read's first suffix and
  // the runs beyond the regions: half of the rows written, whole lines (400
  // Mbases 1.76 -> 1.61 ms with tiles of 2048).  Left out one by one, the other rows that nothing
  // reads save nothing.
  const bool read = LTR || d != 0 || (code & CODE_START) || k + 1 >= (uint32_t)RUN_REGIONS;
  if (on && !look) put_row(D, cm, g, q, x, code, read);
  const uint64_t m = __ballot(look);
  if (m) {
    if (list_full(n, m)) put_looked_up<LTR>(D, cm, L, n);
    list_append(L, n, look, m, g, q, d);
  }
}

__device__ __forceinline__ uint32_t bwt_symbol(uint32_t code) {
  const uint32_t lut = 'A' | ('C' << 8) | ('G' << 16) | ('T' << 24);
  return code & CODE_START ? (uint32_t)'$' : (lut >> (8 * (code & 3u))) & 0xFFu;
}
// Rows of reads' first suffixes (a: row, b: position).
__device__ __forceinline__ void put_first_rows(const IndData &D, const CollMap &cm, WaveList &L, uint32_t &n) {
  wave_lds_fence();
  const uint32_t l = lane_id();
  if (l < n) D.start_row[start_rank(D.text, D.srank, L.b[l])] = (uint64_t)((int64_t)L.a[l] + cm.row_shift);
  n = 0;
  wave_lds_fence();
}
__device__ __forceinline__ void note_first_rows(const IndData &D, const CollMap &cm, WaveList &L, uint32_t &n, bool on,
                                                uint32_t j, uint32_t p) {
  const uint64_t m = __ballot(on);
  if (m) {
    if (list_full(n, m)) put_first_rows(D, cm, L, n);
    list_append(L, n, on, m, j, p, 0);
  }
}

// Class ranks of one slot: this lane's place, from the places the wave's
// classes (base, k) have come to in nxt; advances them.
__device__ __forceinline__ uint32_t ind_place(bool ok, uint32_t d, uint32_t (&nxt)[4], uint32_t lo, uint32_t hi) {
  uint32_t g = 0;
#pragma unroll
  for (uint32_t dd = 0; dd < 4; ++dd) {
    if (dd < lo || dd >= hi) continue;
    const bool is = ok && d == dd;
    const uint64_t mk = __ballot(is);
    if (is) g = nxt[dd] + bits_below_lane(mk);
    nxt[dd] += (uint32_t)__popcll(mk);
  }
  return g;
}

// The partition itself, a wave a tile, IND_BATCH slots at a time.  Copy 0 of
// every item first; the items whose run is longer (a quarter of them) are
// kept in LDS, and their further copies written k by k, so that full waves
// write them.  (Listed per tile by place and loaded again they cost a second
// read of a quarter of the rows: 2.46 instead of 1.90 GB counted in the
// right-to-left steps of 400 Mbases.)  Bound by its traffic: 10.1 GB read and
// written in both directions in 2.42 ms (1.35 right to left), 4.2 TB/s where a
// copy reaches 4.5.
template <bool LTR>
__global__ __launch_bounds__(BLOCK) void k_ind_scatter(IndStep P, IndData D) {
  __shared__ uint2 lists[WAVES][64 * IND_BATCH];
  __shared__ WaveList looks[WAVES], firsts[LTR ? 1 : WAVES];
  const uint32_t w = threadIdx.x >> 6, l = lane_id();
  uint32_t n_look = 0, n_first = 0;
  const uint32_t tile =
      (uint32_t)__builtin_amdgcn_readfirstlane((int)(xcd_tile(blockIdx.x, gridDim.x) * WAVES + w));
  if (tile >= P.ntiles) return;
  uint2 *const list = lists[w];
  const uint32_t s = find_upper(P.tile_prefix, P.nsegs, tile);
  const IndSeg sg = P.segs[s];
  const CollMap cm = D.cmap[sg.coll];
  const uint32_t t0 = (tile - P.tile_prefix[s]) * IND_TILE;
  const uint32_t m = min(IND_TILE, sg.len - t0);
  const uint64_t at0 = (uint64_t)sg.start + t0;
  const uint32_t g = P.coll_groups[sg.coll] + (tile - P.coll_tiles[sg.coll]) / GROUP_TILES;
  // the place of class l's next item
  uint32_t place = D.gtot[(uint64_t)g * 64 + l] + D.hist[(uint64_t)tile * 64 + l];
  // bases the step's items can go to
  const uint32_t lo = LTR ? (P.base == 4 ? 0u : P.base + 1) : 0u, hi = LTR ? 4u : P.base;
  uint32_t nxt[4];
  auto take_places = [&](uint32_t k) {
#pragma unroll
    for (uint32_t dd = 0; dd < 4; ++dd) nxt[dd] = (uint32_t)__builtin_amdgcn_readlane((int)place, (int)(dd * 16 + k));
  };
  auto keep_places = [&](uint32_t k) {
#pragma unroll
    for (uint32_t dd = 0; dd < 4; ++dd)
      if (l == dd * 16 + k) place = nxt[dd];
  };
  const uint8_t *codes = sg.src == SRC_SAMPLES ? D.smp.code + at0 : D.bwt + cm.out_shift + at0;
  for (uint32_t x0 = 0; x0 < m; x0 += IND_BATCH * 64) {
    uint32_t code[IND_BATCH], p[IND_BATCH], pl[IND_BATCH];
#pragma unroll
    for (uint32_t i = 0; i < IND_BATCH; ++i) {
      const uint32_t x = x0 + i * 64 + l;
      code[i] = CODE_START;
      p[i] = 0;
      pl[i] = PL_START;
      if (x < m) {
        if (LTR && sg.src == SRC_READS) {
          ind_read_end(D, at0 + x, p[i], pl[i], code[i]);
        } else if (LTR && sg.src == SRC_SAMPLES) {
          code[i] = codes[x];
          p[i] = D.smp.h[at0 + x];
          pl[i] = D.smp.pl[at0 + x];
        } else {
          code[i] = codes[x];
          const uint2 v = D.rows[at0 + x];
          p[i] = v.x;
          pl[i] = v.y;
        }
      }
    }
    uint32_t n1 = 0;
    take_places(0);
#pragma unroll
    for (uint32_t i = 0; i < IND_BATCH; ++i) {
      const uint32_t x = x0 + i * 64 + l;
      const bool ok = ind_taken<LTR>(code[i], P.base);
      const uint32_t d = code[i] & 3u, r = code_run(code[i]);
      const uint32_t to = ind_place(ok, d, nxt, lo, hi);
      ind_put<LTR>(D, cm, looks[w], n_look, ok, to, d, 0, r, p[i], pl[i]);
      const uint64_t more = __ballot(ok && r > 1);
      if (ok && r > 1) list[n1 + bits_below_lane(more)] = make_uint2(p[i], pl[i]);
      n1 += (uint32_t)__popcll(more);
      if (!LTR) {  // the last step to read this row's code
        if (x < m) D.bwt[at0 + x + cm.out_shift] = (uint8_t)bwt_symbol(code[i]);
        note_first_rows(D, cm, firsts[w], n_first, x < m && (code[i] & CODE_START), (uint32_t)(at0 + x), p[i]);
      }
    }
    keep_places(0);
    for (uint32_t k = 1; n1 && k < (uint32_t)RUN_REGIONS; ++k) {
      wave_lds_fence();
      take_places(k);
      uint32_t n2 = 0;
      for (uint32_t y0 = 0; y0 < n1; y0 += 64) {
        const uint32_t y = y0 + l;
        const bool in = y < n1;
        const uint2 e = in ? list[y] : make_uint2(0, PL_START);
        const uint32_t d = e.y & 3u;  // the preceding base is the payload's first
        const uint32_t r = in ? pl_run(e.y) : 0u;
        const uint32_t to = ind_place(in, d, nxt, lo, hi);
        ind_put<LTR>(D, cm, looks[w], n_look, in, to, d, k, r, e.x, e.y);
        const uint64_t more = __ballot(in && r > k + 1);
        __builtin_amdgcn_wave_barrier();  // this slot's entries are read before any is overwritten
        if (in && r > k + 1) list[n2 + bits_below_lane(more)] = e;
        n2 += (uint32_t)__popcll(more);
      }
      keep_places(k);
      n1 = n2;
    }
    wave_lds_fence();
  }
  if (n_look) put_looked_up<LTR>(D, cm, looks[w], n_look);
  if (!LTR && n_first) put_first_rows(D, cm, firsts[w], n_first);
}

// Runs beyond the regions: the members of region 14 (and of every later one)
// whose preceding base is still the bucket's, one base further, until there
// is none.  One workgroup a collection; rare and short (runs of 16 and more).
constexpr int TAIL_WG = 1024;
struct IndTail {
  uint32_t start, len, limit;  // region 14; the end (L) or start (S) of the bucket's part
};
template <bool LTR>
__global__ __launch_bounds__(TAIL_WG) void k_ind_tail(const IndTail *__restrict__ tails, uint32_t c, IndData D) {
  constexpr int NW = TAIL_WG / 64;
  __shared__ uint32_t tmp[NW];
  const IndTail t = tails[blockIdx.x];
  const CollMap cm = D.cmap[blockIdx.x];
  uint64_t s = t.start, e = s + t.len;
  auto goes_on = [&](uint64_t j) {
    return j < e && D.bwt[j + cm.out_shift] == (uint8_t)c;  // the bucket's base, no run
  };
  for (;;) {
    uint32_t mine = 0, total = 0;
    for (uint64_t j = s + threadIdx.x; j < e; j += TAIL_WG) mine += goes_on(j);
    (void)block_excl_sum<NW>(mine, tmp, &total);
    if (!total) return;
    if (LTR ? e + total > t.limit : s < (uint64_t)t.limit + total) {
      if (threadIdx.x == 0) atomicOr(D.status, ST_LIST_OVERFLOW);
      return;
    }
    uint64_t to = LTR ? e : s - total;
    const uint64_t first = to;
    for (uint64_t j0 = s; j0 < e; j0 += TAIL_WG) {
      const uint64_t j = j0 + threadIdx.x;
      const bool on = goes_on(j);
      uint32_t cnt = 0;
      const uint32_t at = block_excl_sum<NW>(on ? 1u : 0u, tmp, &cnt);
      if (on) {
        const uint2 v = D.rows[j];
        uint32_t x = v.y >> 2;
        const uint32_t code = item_code<LTR>(D.text, c, v.x - 1, x);
        D.rows[to + at] = make_uint2(v.x - 1, x);
        D.bwt[to + at + cm.out_shift] = (uint8_t)code;
      }
      to += cnt;
    }
    __syncthreads();
    s = first;
    e = first + total;
  }
}

// BWT bytes of the rows that no step reads (bucket A), four a lane.
__global__ __launch_bounds__(BLOCK) void k_ind_emit(IndStep P, IndData D) {
  __shared__ WaveList firsts[WAVES];
  const uint32_t w = threadIdx.x >> 6;
  const uint32_t tile = (uint32_t)__builtin_amdgcn_readfirstlane((int)(blockIdx.x * WAVES + w));
  if (tile >= P.ntiles) return;
  const uint32_t s = find_upper(P.tile_prefix, P.nsegs, tile);
  const IndSeg sg = P.segs[s];
  const CollMap cm = D.cmap[sg.coll];
  const uint32_t t0 = (tile - P.tile_prefix[s]) * IND_TILE;
  const int64_t j0 = (int64_t)sg.start + t0, j1 = j0 + min(IND_TILE, sg.len - t0);
  uint32_t n_first = 0;
  // whole words of the output, the rows at both ends of the tile by byte
  const int64_t word0 = (int64_t)((uintptr_t)(D.bwt + cm.out_shift + j0) & 3u);
  for (int64_t jj = j0 - word0; jj < j1; jj += 4 * 64) {
    const int64_t j = jj + 4 * (int64_t)lane_id();
    uint8_t *const at = D.bwt + cm.out_shift + j;
    uint32_t c = 0;
    const bool whole = j >= j0 && j + 4 <= j1;
    if (whole) {
      c = *reinterpret_cast<const uint32_t *>(at);
    } else {
      for (int i = 0; i < 4; ++i)
        if (j + i >= j0 && j + i < j1) c |= (uint32_t)at[i] << (8 * i);
    }
    uint32_t out = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) out |= bwt_symbol((c >> (8 * i)) & 0xFFu) << (8 * i);
    if (whole) {
      *reinterpret_cast<uint32_t *>(at) = out;
    } else {
      for (int i = 0; i < 4; ++i)
        if (j + i >= j0 && j + i < j1) at[i] = (uint8_t)(out >> (8 * i));
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const bool first = ((c >> (8 * i)) & CODE_START) != 0;  // (only rows of the tile have a code)
      const uint32_t p = first ? D.rows[j + i].x : 0u;
      note_first_rows(D, cm, firsts[w], n_first, first, (uint32_t)(j + i), p);
    }
  }
  if (n_first) put_first_rows(D, cm, firsts[w], n_first);
}

}  // namespace
