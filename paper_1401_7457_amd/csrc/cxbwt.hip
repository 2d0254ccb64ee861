// cxbwt.hip -- multi-string BWT of a read collection on MI355X (gfx950).
//
// Liu, Luo & Lam, "GPU-Accelerated BWT Construction for Large Collection of
// Short Reads": Section 2 defines the transform (sort every suffix of every
// S_i = r_i $_i, terminators below the bases and ordered by read index, emit
// the preceding symbol); Section 3.2 sorts suffixes with LSD radix passes over
// packed 2-bit "stringwords" gathered by index, with '$' padding and stable
// passes giving the read-index tie-break.
//
// This implementation keeps the idea of sorting suffix handles by packed
// multi-base keys gathered from the 2-bit reads, but organises the sort for a
// 256-CU, 8 TB/s device:
//
//   * handle  = the 32-bit global base position p of a suffix's first base;
//               the n empty suffixes ($_i alone) are not sorted at all: they
//               are rows 0..n-1 in read order.
//   * key     = one 27-base window of the suffix (layout in device_common.h):
//               bases zero-padded past the read end, then min(remaining, 27).
//               Comparing (bases, clamped length) is the order of Section 2
//               inside one window: a suffix that ends in the window is a
//               proper prefix of, hence below, one that goes on; equal keys
//               with a clamped length below 27 are identical suffixes, which
//               stable passes keep in read order.
//   * sort    = most-significant digit first.  Level 1 computes window-0 keys
//               from the 2-bit reads and scatters them by their top 8 bits
//               (keys are never stored unsorted); further 8-bit levels split
//               every bucket larger than one chunk (64 x 3, 6 or 8 suffixes,
//               the tuning's choice).  Runs of small buckets are then sorted
//               on their remaining digits, tie-refined window by window and
//               emitted by one wave, in LDS.  A tie on a full window (clamped
//               length 27) fetches the next window of the tied suffixes only,
//               one aligned 16-byte text record each.
//   * levels  = each level's scan hands on the next level's segment list and
//               its tile totals; the lists and their prefixes are built on the
//               device, so the host reads one small counter block per level,
//               and a build whose level kernels read their sizes on the
//               device can be captured whole in a hipGraph.
//
// Every pass is stable and the initial order is read-major, so suffixes that
// are equal through their terminators stay in read-index order (the stability
// argument of Section 3.2).

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <atomic>
#include <mutex>
#include <new>
#include <thread>
#include <vector>

#include "cxbwt.h"
#include "cxbwt_induce.h"
#include "cxbwt_kernels.h"

namespace {

using namespace cxk;

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
thread_local cxbwt_stats g_stats;
thread_local int g_timing = 0;

// The instantiation a build uses (see the tuning constants).
struct Tuning {
  uint32_t tile_items;   // 6, 8 or 16 suffixes per 256 threads' thread in a level tile (16: 8 waves x 8)
  uint32_t chunk_items;  // 3, 6 or 8 suffixes per lane in a chunk
  uint32_t schedule = CXBWT_SCHEDULE_MSD;  // sort schedule of single-collection builds
  uint32_t tile_len() const { return BLOCK * tile_items; }
  uint32_t chunk() const { return LOCAL_WG * chunk_items; }
};

// What a build of n_coll collections that sorts n_sort suffixes at once takes.  The default pair
// leaves it to the library (so that the pair is all there is to a choice, and
// cxbwt_set_tuning with what cxbwt_get_tuning gave restores a thread): from
// LARGE_SORT suffixes on 16 x 8 (8 x 6 and 16 x 8: 8 Mbases of 100-base reads
// 0.576 and 0.550 ms, 8.75 of 100 to 250 bases 0.622 and 0.644, 16 Mbases 1.18
// and 0.93, 200 Mbases in four ranges 13.9 and 13.0).  Collections that do not
// fill the narrow tile (2048 suffixes) keep it, and take the long chunk only:
// each has a tile of its own (30 Mbases in collections of 1 kbase, 8 x 6, 8 x 8
// and 16 x 8: 1.10, 1.11 and 1.21 ms, of 2 kbases 0.86, 0.84 and 0.88, of 3
// kbases 0.82, 0.82 and 0.80; of 500 bases, which fit the long chunk, 1.69, 1.00
// and 1.00).
constexpr uint64_t LARGE_SORT = 12000000;
constexpr uint32_t DEFAULT_TILE = 8, DEFAULT_CHUNK = 6;
thread_local Tuning g_tuning{DEFAULT_TILE, DEFAULT_CHUNK};
Tuning tuning_for(Tuning t, uint64_t n_sort, uint64_t n_coll) {
  if (t.tile_items == DEFAULT_TILE && t.chunk_items == DEFAULT_CHUNK && n_sort >= LARGE_SORT) {
    t.tile_items = n_sort / n_coll > BLOCK * MAX_TILE_ITEMS ? 16 : 8;
    t.chunk_items = 8;
  }
  return t;
}

// tile_items 16 is the wide tile: 8 waves x 8 items (4096 suffixes); the
// histogram kernels take it as two sub-tiles of BLOCK * MAX_TILE_ITEMS
static_assert(BLOCK * MAX_TILE_ITEMS * 2 == 4096, "a wide tile is two histogram sub-tiles");
bool tuning_ok(uint32_t tile_items, uint32_t chunk_items) {
  return (tile_items == 6 || tile_items == 8 || tile_items == 16) &&
         (chunk_items == 3 || chunk_items == 6 || chunk_items == 8);
}

inline uint64_t ceil_div(uint64_t a, uint64_t b) { return (a + b - 1) / b; }
inline uint64_t align_up(uint64_t x) { return (x + 255) & ~255ull; }


struct Layout {
  uint64_t keys0, keys1, hdl0, hdl1, text, srank, rank_blocks, start_row, tile_hist, gsum, segs, tile_prefix,
      group_prefix, seg_or, seg_and, seg_split, big_next, chunks, finals, coll_reads, coll_bases, cmap, counters,
      stats, list_tiles, list_blocks, ph_counts, ph_prefixes, pos64, total;
  uint64_t cap_big, cap_chunks, cap_finals, seg_slots, max_tiles, max_groups, n_rec, n_rank_words, n_rank_blocks;
  uint64_t sort_cap, n_cmap, n_list_tiles, n_list_blocks, tile_hist_bytes;
};

bool sizes_ok(uint64_t n_reads, uint64_t n_bases, uint32_t max_read_len) {
  return n_reads >= 1 && n_reads < (1ull << 32) && n_bases <= CXBWT_MAX_BASES && max_read_len <= CXBWT_MAX_READ_LEN;
}
// A build in ranges: the handles of one range are 32-bit (sort positions of
// at most max_range_suffixes suffixes), so the collection may exceed 32-bit
// base positions when they are kept in a 64-bit table.
bool range_wide(uint64_t n_bases, uint32_t flags) {
  return n_bases > CXBWT_MAX_BASES || (flags & CXBWT_RANGE_WIDE) != 0;
}
bool range_sizes_ok(uint64_t n_reads, uint64_t n_bases, uint32_t max_read_len, uint64_t m, uint32_t flags) {
  (void)flags;
  return n_reads >= 1 && n_reads < (1ull << 32) && n_bases <= CXBWT_MAX_RANGE_BASES &&
         max_read_len <= CXBWT_MAX_READ_LEN && m >= 1 && m <= CXBWT_MAX_BASES;
}

// Workspace of a build of nb bases in n_reads reads and n_coll collections
// whose sort buffers hold at most m_sort suffixes at once (all nb of them,
// or one range of a build in ranges).
Layout make_layout(uint64_t n_reads, uint64_t nb_text, uint32_t n_coll, uint64_t m_sort = ~0ull, bool wide = false) {
  Layout L{};
  const uint64_t nb = std::min(nb_text, m_sort);  // suffixes sorted at once
  L.sort_cap = nb;
  L.n_cmap = n_coll;  // a build in ranges rewrites its one entry per range
  // segments of one level are disjoint and each holds more than a chunk
  // (at least MIN_CHUNK) suffixes; level 1 starts with one segment per
  // collection
  L.cap_big = nb / (MIN_CHUNK + 1) + 2;
  L.cap_finals = L.cap_big;
  // chunks of one level: two neighbouring chunks of a run hold more than
  // a chunk's suffixes together, and a run ends at an oversized bucket or at the
  // end of its parent (both at most cap_big per level); level 1 adds one
  // chunk per collection that fits a chunk
  L.cap_chunks = 2 * ceil_div(nb, MIN_CHUNK) + 2 * L.cap_big + n_coll + 2;
  // segments split in one batch of a level: the per-segment and per-tile
  // scratch is sized for segments of more than SEG_BATCH_MIN suffixes; a
  // level with more segments runs in several batches.  Level 1 (one segment
  // per collection) always fits one batch, and so do the 256 segments that level
  // 1 of one collection can leave (of 100 to 525 kbases: fewer than 2048 suffixes
  // each, so that builds of these sizes, whose levels are listed, were finished
  // by the host: 400 kbases 0.63 ms, and 0.25 so; 0.5 MB of scratch).
  L.seg_slots = std::max<uint64_t>({nb / (SEG_BATCH_MIN + 1) + 2, (uint64_t)n_coll + 1, 256 + 2});
  L.max_tiles = ceil_div(nb, MIN_TILE) + L.seg_slots + 1;
  L.max_groups = ceil_div(nb, (uint64_t)MIN_TILE * GROUP_TILES) + L.seg_slots + 1;
  L.n_rec = nb_text / 16 + 2;
  L.n_list_tiles = ceil_div(nb_text, LIST_TILE) + 1;
  L.n_list_blocks = ceil_div(L.n_list_tiles, RANK_BLOCK_WORDS) + 1;
  L.n_rank_words = ceil_div(L.n_rec, 2);  // bitmap words covering the records
  L.n_rank_blocks = ceil_div(L.n_rank_words, RANK_BLOCK_WORDS);
  uint64_t off = 0;
  auto take = [&](uint64_t bytes) {
    uint64_t at = off;
    off = align_up(off + bytes);
    return at;
  };
  const uint64_t seg_slots = L.seg_slots;
  L.keys0 = take(8 * nb);
  L.keys1 = take(8 * nb);
  L.hdl0 = take(4 * nb);
  L.hdl1 = take(4 * nb);
  L.text = take(sizeof(TextRec) * L.n_rec);
  L.srank = take(4 * L.n_rec);
  L.rank_blocks = take(4 * L.n_rank_blocks);
  L.start_row = take(8 * n_reads);
  // the read-start bitmap (one bit per base) lives here before level 1
  // and a range's level 1 counts here per RANGE_TILE positions
  L.tile_hist_bytes = std::max<uint64_t>(4 * 256 * L.max_tiles, 4 * (nb_text / 32 + 4));
  if (nb_text > nb) L.tile_hist_bytes = std::max<uint64_t>(L.tile_hist_bytes, 4 * 256 * ceil_div(nb_text, RANGE_TILE));
  L.tile_hist = take(L.tile_hist_bytes);
  L.gsum = take(4 * 256 * L.max_groups);
  L.segs = take(sizeof(Seg) * seg_slots);
  // tile prefixes serve a batch of segments and, after it, the final groups
  // of the batch (each more than a chunk's suffixes: at most cap_finals)
  L.tile_prefix = take(4 * (std::max(seg_slots, L.cap_finals) + 1));
  L.group_prefix = take(4 * (seg_slots + 1));
  L.seg_or = take(8 * seg_slots);
  L.seg_and = take(8 * seg_slots);
  L.seg_split = take(seg_slots);
  L.big_next = take(sizeof(Seg) * L.cap_big);
  L.chunks = take(sizeof(Seg) * L.cap_chunks);
  L.finals = take(sizeof(Seg) * L.cap_finals);
  L.coll_reads = take(8 * ((uint64_t)n_coll + 1));
  L.coll_bases = take(8 * ((uint64_t)n_coll + 1));
  L.cmap = take(sizeof(CollMap) * L.n_cmap);
  L.counters = take(4 * C_COUNT);
  L.stats = take(8 * STAT_WORDS);
  L.list_tiles = take(4 * L.n_list_tiles);
  L.list_blocks = take(4 * L.n_list_blocks);
  L.ph_counts = take(8 * 256 * PH_MAX_PREFIXES);
  L.ph_prefixes = take(8 * PH_MAX_PREFIXES);
  // wide positions: a 64-bit position per listed suffix; 0 = no table (the
  // layout starts with keys0 at offset 0, so no other region sits there)
  L.pos64 = wide ? take(8 * nb) : 0;
  L.total = off;
  return L;
}

// The text behind the calling thread's last CXBWT_EDEVICE or CXBWT_EDATA
// (cxbwt_last_error).
thread_local char g_last_error[256] = "";
int fail_hip(hipError_t e, const char *what) {
  snprintf(g_last_error, sizeof(g_last_error), "%s: %s", what, hipGetErrorString(e));
  return CXBWT_EDEVICE;
}
// An internal size check that failed (a list or scratch area smaller than
// the work handed to it).
int fail_internal(const char *what) {
  snprintf(g_last_error, sizeof(g_last_error), "internal check failed: %s", what);
  return CXBWT_EDEVICE;
}

// A failure the device reported in its status word.
int fail_status(uint32_t status) {
  snprintf(g_last_error, sizeof(g_last_error), "device status 0x%x:%s%s%s%s%s%s", status,
           (status & ST_BAD_OFFSETS) ? " offsets are not a non-decreasing partition of the bases;" : "",
           (status & ST_TOO_LONG) ? " a read is longer than max_read_len;" : "",
           (status & ST_BAD_CHAR) ? " a byte is not A/C/G/T;" : "",
           (status & ST_LIST_OVERFLOW) ? " a work list overflowed its capacity;" : "",
           (status & ST_WINDOW_BOUND) ? " a tie outlived the windows of max_read_len;" : "",
           (status & ST_PLAN_MISMATCH) ? " collection bases differ from the captured plan;" : "");
  if (status & (ST_BAD_OFFSETS | ST_TOO_LONG)) return CXBWT_EDATA;
  if (status & ST_PLAN_MISMATCH) return CXBWT_EINVAL;
  return CXBWT_EDEVICE;
}

// A C entry's work: no C++ exception (host memory that has run out) leaves it,
// and the device is through with the caller's buffers when it returns.
template <class Work>
int guarded(hipStream_t st, Work work) {
  try {
    return work();
  } catch (...) {
    (void)hipStreamSynchronize(st);
    snprintf(g_last_error, sizeof(g_last_error), "out of host memory");
    return CXBWT_EDEVICE;
  }
}

#define CX_CHECK(x)                                                        \
  do {                                                                     \
    const hipError_t cx_e_ = (x);                                          \
    if (cx_e_ != hipSuccess) return fail_hip(cx_e_, "HIP runtime call");   \
  } while (0)
#define CX_LAUNCHED()                                                      \
  do {                                                                     \
    const hipError_t cx_e_ = hipGetLastError();                            \
    if (cx_e_ != hipSuccess) return fail_hip(cx_e_, "kernel launch");      \
  } while (0)

unsigned grid_for(uint64_t n, unsigned block) {
  uint64_t g = ceil_div(n, block);
  if (g == 0) g = 1;
  if (g > 0x7FFFFFFFull) g = 0x7FFFFFFFull;
  return (unsigned)g;
}

int fill_u64(uint64_t *p, uint64_t n, uint64_t v, hipStream_t st) {
  if (!n) return CXBWT_OK;
  unsigned g = grid_for(n, 256);
  if (g > 65536) g = 65536;
  k_fill_u64<<<g, 256, 0, st>>>(p, n, v);
  CX_LAUNCHED();
  return CXBWT_OK;
}
int fill_u32(uint32_t *p, uint64_t n, uint32_t v, hipStream_t st) {
  if (!n) return CXBWT_OK;
  unsigned g = grid_for(n, 256);
  if (g > 65536) g = 65536;
  k_fill_u32<<<g, 256, 0, st>>>(p, n, v);
  CX_LAUNCHED();
  return CXBWT_OK;
}

// Kernel classes timed by PhaseTimer (indices of cxbwt_stats.ms).
enum Phase { PH_PREP = 0, PH_GEN, PH_HIST, PH_SCAN, PH_SCATTER, PH_LOCAL, PH_FINAL, PH_INDUCE };

// Brackets kernel launches with HIP events on the build's stream when timing
// is on; durations are summed at the host synchronisation points.
struct PhaseTimer {
  hipStream_t st;
  bool on;
  struct Pending {
    int phase;
    hipEvent_t a, b;
  };
  std::vector<Pending> pending;
  hipEvent_t open_ev = nullptr;
  static std::vector<hipEvent_t> &pool() {
    thread_local std::vector<hipEvent_t> p;
    return p;
  }
  hipEvent_t get() {
    auto &p = pool();
    if (!p.empty()) {
      hipEvent_t e = p.back();
      p.pop_back();
      return e;
    }
    hipEvent_t e = nullptr;
    if (hipEventCreate(&e) != hipSuccess) return nullptr;
    return e;
  }
  void begin() {
    if (!on) return;
    open_ev = get();
    if (open_ev) (void)hipEventRecord(open_ev, st);
  }
  void end(int phase) {
    if (!on || !open_ev) return;
    hipEvent_t b = get();
    if (!b) return;
    (void)hipEventRecord(b, st);
    pending.push_back({phase, open_ev, b});
    open_ev = nullptr;
  }
  // call only after the stream has been synchronised
  void collect() {
    for (auto &q : pending) {
      float ms = 0.f;
      if (hipEventElapsedTime(&ms, q.a, q.b) == hipSuccess) g_stats.ms[q.phase] += ms;
      g_stats.launches[q.phase]++;
      pool().push_back(q.a);
      pool().push_back(q.b);
    }
    pending.clear();
  }
  ~PhaseTimer() {
    for (auto &q : pending) {
      pool().push_back(q.a);
      pool().push_back(q.b);
    }
    if (open_ev) pool().push_back(open_ev);
  }
};


struct Buffers {
  uint64_t *keys0, *keys1, *start_row, *coll_reads, *coll_bases, *ph_prefixes;
  uint64_t *pos64;  // 64-bit positions of the listed range (wide builds in ranges), else null
  uint32_t *list_tiles, *list_blocks;
  unsigned long long *ph_counts;
  TextRec *text;
  uint32_t *hdl0, *hdl1, *srank, *rank_blocks, *tile_hist, *gsum, *tile_prefix, *group_prefix, *counters;
  Seg *segs, *big_next, *chunks, *finals;
  CollMap *cmap;
  unsigned long long *seg_or, *seg_and, *stats;
  uint8_t *seg_split;
  // a build by induced order: the sort buffers above hold its samples, in
  // SampleKey's format, and finished ones go to smp
  bool sample = false, pair = false;  // pair: two windows a load (k_sample_chunk)
  SampleOut smp{};
};

// End of the batch of segments starting at b0 that fits the per-segment and
// per-tile scratch (at least one segment: a single segment always fits).
size_t batch_end(const std::vector<Seg> &segs, size_t b0, const Layout &Lo, uint32_t tile_len) {
  uint64_t tiles = 0, groups = 0;
  size_t b1 = b0;
  while (b1 < segs.size() && b1 - b0 < Lo.seg_slots) {
    const uint64_t nt = ceil_div(segs[b1].len, tile_len);
    const uint64_t ng = ceil_div(nt, GROUP_TILES);
    if (b1 > b0 && (tiles + nt > Lo.max_tiles || groups + ng > Lo.max_groups)) break;
    tiles += nt;
    groups += ng;
    ++b1;
  }
  return b1;
}

// Upload a segment list with its tile and group prefixes; returns the tile
// and group totals.
int upload_segments(const Buffers &B, const Layout &Lo, const std::vector<Seg> &segs, uint32_t tile_len,
                    std::vector<uint32_t> &tprefix, std::vector<uint32_t> &gprefix, uint32_t &ntiles,
                    uint32_t &ngroups, hipStream_t st) {
  const uint32_t ns = (uint32_t)segs.size();
  if (ns > Lo.seg_slots) return fail_internal("work exceeds a workspace list or scratch area");
  tprefix.assign(ns + 1, 0);
  gprefix.assign(ns + 1, 0);
  for (uint32_t i = 0; i < ns; ++i) {
    const uint32_t nt = (uint32_t)ceil_div(segs[i].len, tile_len);
    tprefix[i + 1] = tprefix[i] + nt;
    gprefix[i + 1] = gprefix[i] + (uint32_t)ceil_div(nt, GROUP_TILES);
  }
  ntiles = tprefix[ns];
  ngroups = gprefix[ns];
  if (ntiles > Lo.max_tiles || ngroups > Lo.max_groups) return fail_internal("work exceeds a workspace list or scratch area");
  CX_CHECK(hipMemcpyAsync(B.segs, segs.data(), sizeof(Seg) * ns, hipMemcpyHostToDevice, st));
  CX_CHECK(hipMemcpyAsync(B.tile_prefix, tprefix.data(), 4 * (ns + 1), hipMemcpyHostToDevice, st));
  CX_CHECK(hipMemcpyAsync(B.group_prefix, gprefix.data(), 4 * (ns + 1), hipMemcpyHostToDevice, st));
  return CXBWT_OK;
}

// Workgroups of the launches whose size is fixed before their work count is
// known (the work count is read on the device; see the kernels): a few per
// CU, multiples of the XCD count.
constexpr unsigned PG_HIST = 256 * 8;
constexpr unsigned PG_GROUP = 256 * 4;
constexpr unsigned PG_SCAN = 256 * 4;
constexpr unsigned PG_SCATTER = 256 * 5;
constexpr unsigned PG_SCATTER_WIDE = 256 * 2;
constexpr unsigned PG_EMIT = 256 * 4;
constexpr unsigned PG_FILL = 256 * 2;

// Second scan stage launch: a workgroup per segment when the segments span
// many groups each (the first levels), else a wave per segment.  With
// dev_ns the count is on the device and the launch is the fixed one of a
// wave per segment.
void launch_level_scan(const Buffers &B, uint32_t ns, uint32_t ngroups, const Lists &Ls, int force_split,
                       hipStream_t st, const uint32_t *dev_ns = nullptr, unsigned dev_grid = PG_SCAN) {
#define CX_SCAN(F, COOP, GRID)                                                                                  \
  k_level_scan<F, COOP, false><<<GRID, BLOCK, 0, st>>>(B.segs, B.group_prefix, ns, B.gsum, B.seg_or, B.seg_and, \
                                                       B.seg_split, Ls, force_split, nullptr)
  const unsigned waves_grid = (unsigned)ceil_div(ns, WAVES);
  if (dev_ns)
    k_level_scan<GeneralKey, false, true><<<dev_grid, BLOCK, 0, st>>>(B.segs, B.group_prefix, 0, B.gsum, B.seg_or,
                                                                      B.seg_and, B.seg_split, Ls, force_split, dev_ns);
  else if (ngroups > 8u * ns) {
    if (B.sample) CX_SCAN(SampleKey, true, ns);
    else CX_SCAN(GeneralKey, true, ns);
  } else {
    if (B.sample) CX_SCAN(SampleKey, false, waves_grid);
    else CX_SCAN(GeneralKey, false, waves_grid);
  }
#undef CX_SCAN
}

// Tile prefixes (and group prefixes, and a copy of the list, when given) of
// the first n entries of a segment list, computed on the device.  Uses the
// scan-group totals area as scratch.  With dev_n the count is on the device
// and n is only its bound.
int prefix_list(const Buffers &B, const Seg *list, uint32_t n, uint32_t tile_len, Seg *copy, uint32_t *tprefix,
                uint32_t *gprefix, hipStream_t st, const uint32_t *dev_n = nullptr, bool begin = false) {
  if (!n) return CXBWT_OK;
  const unsigned nwg = (unsigned)ceil_div(n, SEGP_WG);
  if (nwg > 1) {
    k_seg_count<<<nwg, BLOCK, 0, st>>>(list, n, dev_n, tile_len, B.gsum);
    CX_LAUNCHED();
  }
  k_seg_scan<<<nwg, BLOCK, 0, st>>>(list, n, dev_n, tile_len, B.gsum, copy, tprefix, gprefix,
                                    begin ? B.counters : nullptr, B.seg_or, B.seg_and);
  CX_LAUNCHED();
  return CXBWT_OK;
}

// What one scan of a level handed on, from the counters block after the
// fold.
struct LevelOut {
  uint32_t status, n_chunks, n_finals, n_big;  // n_big: all batches of the level so far
  uint64_t next_len, next_regather, next_maxr, next_tiles, next_groups, final_len, final_tiles;
};

LevelOut level_out(const uint32_t *hc) {
  LevelOut o{};
  uint64_t f[K_LEVEL_KINDS];
  memcpy(f, hc + C_FOLD, sizeof(f));
  o.status = hc[C_STATUS];
  o.n_chunks = hc[C_NCHUNK];
  o.n_finals = hc[C_NFINAL];
  o.n_big = hc[C_NBIG];
  o.next_len = f[K_NEXT_LEN - K_LEVEL_FIRST];
  o.next_regather = f[K_NEXT_REGATHER - K_LEVEL_FIRST];
  o.next_maxr = f[K_NEXT_MAXR - K_LEVEL_FIRST];
  o.next_tiles = f[K_NEXT_TILES - K_LEVEL_FIRST];
  o.next_groups = f[K_NEXT_GROUPS - K_LEVEL_FIRST];
  o.final_len = f[K_FINAL_LEN - K_LEVEL_FIRST];
  o.final_tiles = f[K_FINAL_TILES - K_LEVEL_FIRST];
  return o;
}

// Fold the level statistics, read the counters back and wait for everything.
int read_level(const Buffers &B, LevelOut &o, PhaseTimer &T, hipStream_t st) {
  uint32_t hc[C_COUNT];
  k_level_fold<<<1, 64, 0, st>>>(B.stats, B.counters, nullptr, nullptr);
  CX_LAUNCHED();
  CX_CHECK(hipMemcpyAsync(hc, B.counters, sizeof(hc), hipMemcpyDeviceToHost, st));
  CX_CHECK(hipStreamSynchronize(st));
  T.collect();
  o = level_out(hc);
  return o.status ? CXBWT_EDEVICE : CXBWT_OK;
}

// While it lives, calls of this thread that allocate or free do not disturb a
// capture on another one: nothing here is part of it.
struct BesideCaptures {
  hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
  const bool on = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
  ~BesideCaptures() {
    if (on) (void)hipThreadExchangeStreamCaptureMode(&mode);
  }
};

// Counters blocks in host memory that the device writes: one a build while
// its levels run, kept for the builds that follow (at most MOST of them).
struct HostBlocks {
  static constexpr size_t MOST = 16;
  std::mutex m;
  std::vector<uint32_t *> idle;
  HostBlocks() { idle.reserve(MOST); }  // (a block is given back by a destructor, which must not throw)
  uint32_t *take() {
    {
      std::lock_guard<std::mutex> g(m);
      if (!idle.empty()) {
        uint32_t *p = idle.back();
        idle.pop_back();
        return p;
      }
    }
    BesideCaptures beside;
    uint32_t *p = nullptr;
    if (hipHostMalloc((void **)&p, 4 * C_COUNT, hipHostMallocPortable) != hipSuccess) {
      (void)hipGetLastError();
      p = nullptr;
    }
    return p;
  }
  void give(uint32_t *p) {
    {
      std::lock_guard<std::mutex> g(m);
      if (idle.size() < MOST) {
        idle.push_back(p);
        return;
      }
    }
    BesideCaptures beside;
    (void)hipHostFree(p);
  }
};
HostBlocks g_host_blocks;

// A level's counters without a wait for what was enqueued after it: post()
// behind the level's kernels, wait() when they are needed.
struct LevelWait {
  uint32_t *block = nullptr;
  hipEvent_t ev = nullptr;
  bool posted = false, recorded = false;
  bool open() {
    if (hipEventCreateWithFlags(&ev, hipEventDisableTiming) != hipSuccess) {
      (void)hipGetLastError();
      ev = nullptr;
      return false;
    }
    return (block = g_host_blocks.take()) != nullptr;
  }
  int post(const Buffers &B, hipStream_t st) {
    k_level_fold<<<1, 64, 0, st>>>(B.stats, B.counters, nullptr, block);
    CX_LAUNCHED();
    posted = true;
    recorded = hipEventRecord(ev, st) == hipSuccess;
    if (!recorded) (void)hipGetLastError();  // (an event of another device than the stream's)
    return CXBWT_OK;
  }
  int wait(LevelOut &o, hipStream_t st) {
    if (recorded) CX_CHECK(hipEventSynchronize(ev));
    else CX_CHECK(hipStreamSynchronize(st));
    posted = false;
    o = level_out(block);
    return o.status ? CXBWT_EDEVICE : CXBWT_OK;
  }
  ~LevelWait() {
    // (after an error the device may still write the block: it stays out)
    if (block && !posted) g_host_blocks.give(block);
    if (ev) (void)hipEventDestroy(ev);
  }
};

// Work counts of one level as an eager build saw them (level 1 at index 0).
// A captured build sizes its launches from them, so that each workgroup
// usually takes one item as in an eager launch (the looping kernels stay
// correct for larger counts).
struct LevelShape {
  uint32_t nsegs = 0, ntiles = 0, ngroups = 0, nchunks = 0, nfinals = 0, ftiles = 0;
};
thread_local std::vector<LevelShape> *g_shapes = nullptr;  // recorder of an eager build, when set
struct ShapeScope {
  explicit ShapeScope(std::vector<LevelShape> *to) { g_shapes = to; }
  ~ShapeScope() { g_shapes = nullptr; }
};

void record_shape(uint32_t level, const LevelShape &x) {
  if (!g_shapes) return;
  if (g_shapes->size() <= level) g_shapes->resize(level + 1);
  LevelShape &y = (*g_shapes)[level];
  y.nsegs = std::max(y.nsegs, x.nsegs);
  y.ntiles = std::max(y.ntiles, x.ntiles);
  y.ngroups = std::max(y.ngroups, x.ngroups);
  y.nchunks = std::max(y.nchunks, x.nchunks);
  y.nfinals = std::max(y.nfinals, x.nfinals);
  y.ftiles = std::max(y.ftiles, x.ftiles);
}

// Launch size for an item count seen before: a quarter more, a multiple of
// the XCD count, or the fixed size when nothing was seen.
unsigned grid_from(uint32_t seen, unsigned fixed) {
  if (!seen) return fixed;
  const uint64_t g = ((uint64_t)seen + seen / 4 + 64 + 7) & ~7ull;
  return (unsigned)std::min<uint64_t>(g, 0x7FFFFFF8ull);
}

// The chunk kernel for the selected chunk size: one workgroup per chunk, or
// with dev_nchunks a launch of `grid` workgroups (0: a few waves per SIMD)
// looping over a count on the device.
int launch_local(const Buffers &B, const Tuning &tu, uint64_t nb, uint32_t rmax, uint8_t *bwt, uint32_t n_chunks,
                 const uint32_t *dev_nchunks, hipStream_t st, unsigned grid = 0, unsigned most = ~0u) {
  // the looping form holds a few more registers: one wave per SIMD fewer
  // for the smallest chunk keeps it from spilling
  // with a device count and no grid: the looping form, of at most `most`
  // workgroups;
  // with a device count and a grid: the one-chunk form over the first
  // `grid` chunks, then the looping form over any beyond them
#define CX_LOCAL(LI, OCC, OCCP)                                                                                  \
  do {                                                                                                           \
    if (dev_nchunks && grid) {                                                                                   \
      k_local<LI, OCC, false><<<grid, LOCAL_WG, 0, st>>>(B.chunks, B.keys0, B.keys1, B.hdl0, B.hdl1, B.pos64, B.text,\
                                                        B.srank, B.cmap, nb, rmax, bwt, B.start_row,             \
                                                        B.counters + C_STATUS, B.stats, 0, dev_nchunks, 0);      \
      k_local<LI, OCCP, true><<<256u, LOCAL_WG, 0, st>>>(B.chunks, B.keys0, B.keys1, B.hdl0, B.hdl1, B.pos64, B.text,\
                                                        B.srank, B.cmap, nb, rmax, bwt, B.start_row,             \
                                                        B.counters + C_STATUS, B.stats, 0, dev_nchunks, grid);   \
    } else if (dev_nchunks) {                                                                                    \
      k_local<LI, OCCP, true><<<std::min(256u * 4u * OCCP, most), LOCAL_WG, 0, st>>>(                            \
          B.chunks, B.keys0, B.keys1, B.hdl0, B.hdl1, B.pos64, B.text, B.srank, B.cmap, nb, rmax, bwt, B.start_row,\
          B.counters + C_STATUS, B.stats, 0, dev_nchunks, 0);                                                    \
    } else {                                                                                                     \
      k_local<LI, OCC, false><<<n_chunks, LOCAL_WG, 0, st>>>(B.chunks, B.keys0, B.keys1, B.hdl0, B.hdl1, B.pos64, B.text,\
                                                            B.srank, B.cmap, nb, rmax, bwt, B.start_row,         \
                                                            B.counters + C_STATUS, B.stats, n_chunks, nullptr,   \
                                                            0);                                                  \
    }                                                                                                            \
  } while (0)
  // waves per SIMD the register allocation is held to: 8 per lane at 4, 6 per
  // lane at 6 (70 registers; the LDS of a 384-suffix chunk, 6.4 KB, also
  // allows six), 3 per lane at 7 (8 spills and is slower)
  if (tu.chunk_items == 8) CX_LOCAL(8, 4, 3);
  else if (tu.chunk_items == 6) CX_LOCAL(6, 6, 4);
  else CX_LOCAL(3, 7, 5);
#undef CX_LOCAL
  CX_LAUNCHED();
  return CXBWT_OK;
}

// Finish the chunks and final groups a level produced.
int finish_level(const Buffers &B, const Layout &Lo, const Tuning &tu, uint64_t nb, uint32_t rmax, uint32_t maxlen,
                 uint8_t *bwt, uint32_t n_chunks, uint32_t n_finals, uint64_t final_tiles, uint64_t final_len, PhaseTimer &T,
                 hipStream_t st) {
  if (n_chunks > Lo.cap_chunks || n_finals > Lo.cap_finals) return fail_internal("work exceeds a workspace list or scratch area");
  int rc;
  if (n_chunks) {
    T.begin();
    if (B.sample) {
#define CX_CHUNK(LI, OCC, PAIR, ABOVE)                                                                             \
  k_sample_chunk<LI, OCC, PAIR><<<n_chunks, LOCAL_WG, 0, st>>>(B.chunks, B.keys0, B.keys1, B.hdl0, B.hdl1, B.text, \
                                                               maxlen, ABOVE, B.smp, B.counters + C_STATUS, B.stats)
      if (B.pair) {
        CX_CHUNK(4, 6, true, 0);
        CX_LAUNCHED();
        CX_CHUNK(8, 4, true, PAIR_PACK);
      } else {
        CX_CHUNK(8, 4, false, 0);
      }
#undef CX_CHUNK
      CX_LAUNCHED();
    } else if ((rc = launch_local(B, tu, nb, rmax, bwt, n_chunks, nullptr, st))) {
      return rc;
    }
    T.end(PH_LOCAL);
    g_stats.chunks += n_chunks;
  }
  if (n_finals) {
    if (final_tiles == 0 || final_tiles > 0xFFFFFFFFull) return fail_internal("work exceeds a workspace list or scratch area");
    if ((rc = prefix_list(B, B.finals, n_finals, tu.tile_len(), nullptr, B.tile_prefix, nullptr, st))) return rc;
    T.begin();
    if (B.sample)
      k_sample_final<<<(unsigned)final_tiles, BLOCK, 0, st>>>(B.finals, B.tile_prefix, n_finals, tu.tile_len(), B.keys0,
                                                              B.keys1, B.hdl0, B.hdl1, B.text, B.smp);
    else
      k_emit_final<false><<<(unsigned)final_tiles, BLOCK, 0, st>>>(B.finals, B.tile_prefix, n_finals, nullptr,
                                                                   tu.tile_len(), B.keys0, B.keys1, B.hdl0, B.hdl1,
                                                                   B.pos64, B.text, B.srank, B.cmap, bwt, B.start_row);
    CX_LAUNCHED();
    T.end(PH_FINAL);
    g_stats.final_big += n_finals;
    g_stats.chunk_suffixes -= final_len;
  }
  return CXBWT_OK;
}

// Histogram, two scan stages and scatter of a level 2.. over nsg segments
// (ntiles tiles, ngroups groups), or with dev_nsg over a segment count on
// the device in launches of fixed size.
int launch_level_kernels(const Buffers &B, const Tuning &tu, const Lists &Ls, uint64_t nb, uint32_t nsg,
                         uint32_t ntiles, uint32_t ngroups, const uint32_t *dev_nsg, PhaseTimer &T, hipStream_t st,
                         const LevelShape *seen = nullptr) {
  const bool dev = dev_nsg != nullptr;
  // device mode: launch sizes from the counts seen, else fixed
  const LevelShape none;
  const LevelShape &sh = seen ? *seen : none;
  const unsigned g_hist = grid_from(sh.ntiles, PG_HIST), g_group = grid_from(sh.ngroups, PG_GROUP),
                 g_scan = grid_from((sh.nsegs + WAVES - 1) / WAVES, PG_SCAN),
                 g_scatter = grid_from(sh.ntiles, tu.tile_items == 16 ? PG_SCATTER_WIDE : PG_SCATTER);
  T.begin();
#define CX_HIST(F, P, SUBT)                                                                                      \
  k_level_hist<F, P, SUBT><<<P ? g_hist : ntiles, BLOCK, 0, st>>>(B.segs, B.tile_prefix, nsg, dev_nsg, tu.tile_len(), \
                                                                B.keys0, B.keys1, B.hdl0, B.hdl1, B.text, nb,        \
                                                                B.pos64, B.tile_hist, B.seg_or, B.seg_and)
  if (B.sample) {
    CX_HIST(SampleKey, false, 2);  // always the wide tile
  } else if (tu.tile_items == 16) {
    if (dev) CX_HIST(GeneralKey, true, 2);
    else CX_HIST(GeneralKey, false, 2);
  } else {
    if (dev) CX_HIST(GeneralKey, true, 1);
    else CX_HIST(GeneralKey, false, 1);
  }
#undef CX_HIST
  CX_LAUNCHED();
  T.end(PH_HIST);
  T.begin();
  if (dev)
    k_group_scan<true><<<g_group, BLOCK, 0, st>>>(B.tile_prefix, B.group_prefix, nsg, dev_nsg, B.tile_hist, B.gsum);
  else
    k_group_scan<false><<<ngroups, BLOCK, 0, st>>>(B.tile_prefix, B.group_prefix, nsg, nullptr, B.tile_hist, B.gsum);
  CX_LAUNCHED();
  launch_level_scan(B, nsg, ngroups, Ls, 0, st, dev_nsg, g_scan);
  CX_LAUNCHED();
  T.end(PH_SCAN);
  T.begin();
#define CX_SCATTER(F, TI, NW, P)                                                                                \
  k_level_scatter<F, TI, NW, P><<<P ? g_scatter : ntiles, 64 * NW, 0, st>>>(                                    \
      B.segs, B.tile_prefix, B.group_prefix, nsg, dev_nsg, B.seg_split, B.tile_hist, B.gsum, B.keys0, B.keys1,    \
      B.hdl0, B.hdl1)
  if (B.sample) {
    CX_SCATTER(SampleKey, 8, 8, false);
  } else if (tu.tile_items == 16) {
    if (dev) CX_SCATTER(GeneralKey, 8, 8, true);
    else CX_SCATTER(GeneralKey, 8, 8, false);
  } else if (tu.tile_items == 8) {
    if (dev) CX_SCATTER(GeneralKey, 8, 4, true);
    else CX_SCATTER(GeneralKey, 8, 4, false);
  } else {
    if (dev) CX_SCATTER(GeneralKey, 6, 4, true);
    else CX_SCATTER(GeneralKey, 6, 4, false);
  }
#undef CX_SCATTER
  CX_LAUNCHED();
  T.end(PH_SCATTER);
  return CXBWT_OK;
}

// One batch of a level 2..: nsg segments in B.segs with their tile and group
// prefixes in place.  Counts, splits, scatters, then finishes the chunks and
// final groups the batch produced.
int run_level_batch(const Buffers &B, const Layout &Lo, const Tuning &tu, const Lists &Ls, uint64_t nb,
                    uint32_t rmax, uint32_t maxlen, uint8_t *bwt, uint32_t nsg, uint32_t ntiles, uint32_t ngroups, LevelOut &o,
                    PhaseTimer &T, hipStream_t st) {
  int rc;
  if ((rc = fill_u64((uint64_t *)B.seg_or, nsg, 0, st))) return rc;
  if ((rc = fill_u64((uint64_t *)B.seg_and, nsg, ~0ull, st))) return rc;
  if ((rc = fill_u32(B.counters + C_NFINAL, 2, 0, st))) return rc;  // final and chunk counts
  if ((rc = launch_level_kernels(B, tu, Ls, nb, nsg, ntiles, ngroups, nullptr, T, st))) return rc;
  g_stats.level_batches++;
  if ((rc = read_level(B, o, T, st))) return rc;
  return finish_level(B, Lo, tu, nb, rmax, maxlen, bwt, o.n_chunks, o.n_finals, o.final_tiles, o.final_len, T, st);
}

// Everything one build needs: its sizes, the caller's buffers, the workspace
// layout and the level-1 plan made from the collection bases.
struct Build {
  const uint64_t *packed, *offsets;
  uint64_t n, nb;
  uint32_t maxlen, ncoll;
  uint8_t *bwt;
  uint64_t *term_pos;
  Layout Lo;
  Buffers B;
  Tuning tu;
  uint32_t rmax, tile_len;
  Lists Ls;
  std::vector<uint64_t> coll_reads, cbase;
  std::vector<CollMap> cm;
  std::vector<Seg> big, small;  // level-1 segments; collections that fit one chunk
  bool planned = false;         // k_begin's plan of one collection is in place on the device
};

Buffers buffers_of(unsigned char *ws, const Layout &Lo) {
  Buffers B;
  B.keys0 = (uint64_t *)(ws + Lo.keys0);
  B.keys1 = (uint64_t *)(ws + Lo.keys1);
  B.hdl0 = (uint32_t *)(ws + Lo.hdl0);
  B.hdl1 = (uint32_t *)(ws + Lo.hdl1);
  B.text = (TextRec *)(ws + Lo.text);
  B.srank = (uint32_t *)(ws + Lo.srank);
  B.rank_blocks = (uint32_t *)(ws + Lo.rank_blocks);
  B.start_row = (uint64_t *)(ws + Lo.start_row);
  B.tile_hist = (uint32_t *)(ws + Lo.tile_hist);
  B.gsum = (uint32_t *)(ws + Lo.gsum);
  B.segs = (Seg *)(ws + Lo.segs);
  B.tile_prefix = (uint32_t *)(ws + Lo.tile_prefix);
  B.group_prefix = (uint32_t *)(ws + Lo.group_prefix);
  B.seg_or = (unsigned long long *)(ws + Lo.seg_or);
  B.seg_and = (unsigned long long *)(ws + Lo.seg_and);
  B.seg_split = (uint8_t *)(ws + Lo.seg_split);
  B.big_next = (Seg *)(ws + Lo.big_next);
  B.chunks = (Seg *)(ws + Lo.chunks);
  B.finals = (Seg *)(ws + Lo.finals);
  B.coll_reads = (uint64_t *)(ws + Lo.coll_reads);
  B.coll_bases = (uint64_t *)(ws + Lo.coll_bases);
  B.cmap = (CollMap *)(ws + Lo.cmap);
  B.counters = (uint32_t *)(ws + Lo.counters);
  B.stats = (unsigned long long *)(ws + Lo.stats);
  B.list_tiles = (uint32_t *)(ws + Lo.list_tiles);
  B.list_blocks = (uint32_t *)(ws + Lo.list_blocks);
  B.ph_counts = (unsigned long long *)(ws + Lo.ph_counts);
  B.ph_prefixes = (uint64_t *)(ws + Lo.ph_prefixes);
  B.pos64 = Lo.pos64 ? (uint64_t *)(ws + Lo.pos64) : nullptr;
  return B;
}

void build_init(Build &b, const uint64_t *packed, const uint64_t *offsets, uint64_t n, uint64_t nb, uint32_t maxlen,
                const uint64_t *coll_reads, uint32_t ncoll, uint8_t *bwt, uint64_t *term_pos, unsigned char *ws,
                uint64_t m_sort = ~0ull, bool wide = false) {
  b.packed = packed;
  b.offsets = offsets;
  b.n = n;
  b.nb = nb;
  b.maxlen = maxlen;
  b.ncoll = ncoll;
  b.bwt = bwt;
  b.term_pos = term_pos;
  b.Lo = make_layout(n, nb, ncoll, m_sort, wide);
  b.B = buffers_of(ws, b.Lo);
  b.tu = tuning_for(g_tuning, b.Lo.sort_cap, ncoll);
  b.rmax = maxlen / W + 1;
  b.tile_len = b.tu.tile_len();
  uint32_t *c = b.B.counters;
  b.Ls = Lists{b.B.big_next, c + C_NBIG, (uint32_t)b.Lo.cap_big, b.B.chunks, (unsigned long long *)(c + C_NCHUNK),
               (uint32_t)b.Lo.cap_chunks, b.B.finals, c + C_NFINAL, (uint32_t)b.Lo.cap_finals, c + C_STATUS, b.rmax,
               b.B.stats, b.tu.chunk(), b.tu.chunk(), b.tile_len, 1};
  b.coll_reads.assign(coll_reads, coll_reads + ncoll + 1);
  b.planned = ncoll == 1;
}

// The level-1 plan of one collection, which its sizes give: one segment, or
// one unsplit chunk.
void plan_single(Build &b) {
  b.cbase = {0, b.nb};
  b.cm.assign(1, CollMap{b.n, (int64_t)b.n});
  b.big.clear();
  b.small.clear();
  if (b.nb > (uint64_t)b.tu.chunk()) b.big.push_back(Seg{0, (uint32_t)b.nb, 0, 0, 0, 0, 0, 0, 0});
  else if (b.nb > 0) b.small.push_back(Seg{0, (uint32_t)b.nb, 0, 0, 0, 0, 1, 0, 0});
}

// Clears the counters, statistics and read-start bitmap, validates the
// offsets and marks the read starts.  For one collection the level-1 plan is
// in place after it; for several, with bases_src, the collection bases are
// compared with the planned ones (staged in the scan-group area).
int enqueue_prep(const Build &b, const uint64_t *coll_reads_src, const uint64_t *bases_src, PhaseTimer &T,
                 hipStream_t st) {
  const Buffers &B = b.B;
  uint32_t *sbits = B.tile_hist;  // the tile histograms are not used before level 1
  const uint64_t n_sbits = b.nb / 32 + 4;
  if (4 * n_sbits > b.Lo.tile_hist_bytes) return fail_internal("work exceeds a workspace list or scratch area");
  int rc;
  if (b.ncoll == 1) {
    OnePlan P{};
    P.n = b.n;
    P.nb = b.nb;
    P.cm = CollMap{b.n, (int64_t)b.n};
    P.seg = Seg{0, (uint32_t)b.nb, 0, 0, 0, 0, (uint8_t)(b.nb <= (uint64_t)b.tu.chunk()), 0, 0};
    P.ntiles = (uint32_t)ceil_div(b.nb, b.tile_len);
    P.ngroups = (uint32_t)ceil_div(P.ntiles, GROUP_TILES);
    k_begin<<<std::min(grid_for(std::max<uint64_t>(n_sbits, STAT_WORDS), 256), 4096u), 256, 0, st>>>(
        P, B.counters, (uint64_t *)B.stats, STAT_WORDS, sbits, n_sbits, B.coll_reads, B.coll_bases, B.cmap, B.segs,
        B.chunks, B.tile_prefix, B.group_prefix);
    CX_LAUNCHED();
  } else {
    if ((rc = fill_u32(B.counters, C_COUNT, 0, st))) return rc;
    if ((rc = fill_u64((uint64_t *)B.stats, STAT_WORDS, 0, st))) return rc;
    if ((rc = fill_u32(sbits, n_sbits, 0, st))) return rc;
    CX_CHECK(hipMemcpyAsync(B.coll_reads, coll_reads_src, 8 * ((uint64_t)b.ncoll + 1), hipMemcpyHostToDevice, st));
  }
  T.begin();
  k_prep<<<grid_for(b.n, 256), 256, 0, st>>>(b.packed, b.offsets, b.n, b.nb, b.maxlen, B.coll_reads, b.ncoll, sbits,
                                            b.bwt, b.term_pos, B.counters + C_STATUS);
  CX_LAUNCHED();
  T.end(PH_PREP);
  if (b.ncoll == 1) return CXBWT_OK;
  k_coll_bases<<<grid_for((uint64_t)b.ncoll + 1, 256), 256, 0, st>>>(b.offsets, B.coll_reads, b.ncoll,
                                                                     B.coll_bases);
  CX_LAUNCHED();
  if (bases_src) {
    uint64_t *want = (uint64_t *)B.gsum;
    CX_CHECK(hipMemcpyAsync(want, bases_src, 8 * ((uint64_t)b.ncoll + 1), hipMemcpyHostToDevice, st));
    k_check_bases<<<grid_for((uint64_t)b.ncoll + 1, 256), 256, 0, st>>>(B.coll_bases, want, b.ncoll + 1,
                                                                        B.counters + C_STATUS);
    CX_LAUNCHED();
  }
  return CXBWT_OK;
}

// The last kernel of every build: term_pos, and the statistics' totals.
int launch_term(const Build &b, hipStream_t st) {
  k_term<<<grid_for(b.n, BLOCK), BLOCK, 0, st>>>(b.offsets, b.n, b.nb, b.B.text, b.B.srank, b.B.start_row, b.term_pos,
                                                 b.B.stats, b.B.counters);
  CX_LAUNCHED();
  return CXBWT_OK;
}

// Text records and the read-start ranks: they need the read-start bitmap
// only, so they are enqueued before the host waits for the level-1 plan.
int enqueue_records(const Build &b, PhaseTimer &T, hipStream_t st) {
  const Buffers &B = b.B;
  const Layout &Lo = b.Lo;
  if (b.nb == 0) return CXBWT_OK;
  uint32_t *sbits = B.tile_hist;
  T.begin();
  k_text_records<<<grid_for(Lo.n_rec, 256), 256, 0, st>>>(b.packed, cxbwt_packed_words(b.nb), sbits, B.text,
                                                           Lo.n_rec);
  CX_LAUNCHED();
  k_rank_count<<<(unsigned)Lo.n_rank_blocks, BLOCK, 0, st>>>(sbits, Lo.n_rank_words, B.rank_blocks);
  CX_LAUNCHED();
  if (Lo.n_rank_blocks <= RANK_SUM_BLOCKS) {
    k_rank_words<true><<<(unsigned)Lo.n_rank_blocks, BLOCK, 0, st>>>(sbits, Lo.n_rank_words, B.rank_blocks, B.srank,
                                                                     Lo.n_rec);
  } else {
    k_rank_top<<<1, BLOCK, 0, st>>>(B.rank_blocks, (uint32_t)Lo.n_rank_blocks);
    CX_LAUNCHED();
    k_rank_words<false><<<(unsigned)Lo.n_rank_blocks, BLOCK, 0, st>>>(sbits, Lo.n_rank_words, B.rank_blocks, B.srank,
                                                                      Lo.n_rec);
  }
  CX_LAUNCHED();
  T.end(PH_PREP);
  return CXBWT_OK;
}

// Reads the collection bases back and plans level 1: the collections above
// one chunk are its segments, the others one unsplit chunk each.
int plan_level1(Build &b, PhaseTimer &T, hipStream_t st) {
  uint32_t hc[C_COUNT];
  b.cbase.assign((size_t)b.ncoll + 1, 0);
  CX_CHECK(hipMemcpyAsync(hc, b.B.counters, sizeof(hc), hipMemcpyDeviceToHost, st));
  CX_CHECK(hipMemcpyAsync(b.cbase.data(), b.B.coll_bases, 8 * ((uint64_t)b.ncoll + 1), hipMemcpyDeviceToHost, st));
  CX_CHECK(hipStreamSynchronize(st));
  T.collect();
  if (hc[C_STATUS] & (ST_BAD_OFFSETS | ST_TOO_LONG)) return fail_status(hc[C_STATUS]);
  // offsets are valid, so the collection bases are non-decreasing and end at nb
  b.cm.assign(b.ncoll, CollMap{});
  b.big.clear();
  b.small.clear();
  for (uint32_t c = 0; c < b.ncoll; ++c) {
    const uint64_t nc = b.coll_reads[c + 1] - b.coll_reads[c];
    const uint64_t bc = b.cbase[c + 1] - b.cbase[c];
    b.cm[c].out_shift = b.coll_reads[c + 1];
    b.cm[c].row_shift = (int64_t)nc - (int64_t)b.cbase[c];
    if (bc > (uint64_t)b.tu.chunk()) b.big.push_back(Seg{(uint32_t)b.cbase[c], (uint32_t)bc, 0, 0, 0, 0, 0, 0, c});
    else if (bc > 0) b.small.push_back(Seg{(uint32_t)b.cbase[c], (uint32_t)bc, 0, 0, 0, 0, 1, 0, c});
  }
  return CXBWT_OK;
}

// Host sources of the level-1 copies: the segment lists with their tile
// and group prefixes.  An eager build points them at vectors; a captured
// build at pinned memory that lives as long as its graph.
struct SegSrc {
  const Seg *segs = nullptr;
  const uint32_t *tprefix = nullptr, *gprefix = nullptr;
  uint32_t ns = 0, ntiles = 0, ngroups = 0;
};
struct Level1Src {
  const CollMap *cm = nullptr;
  SegSrc big, small;
  const uint32_t *nsmall = nullptr;
};

void seg_prefixes(const std::vector<Seg> &segs, uint32_t tile_len, std::vector<uint32_t> &tp,
                  std::vector<uint32_t> &gp) {
  const size_t ns = segs.size();
  tp.assign(ns + 1, 0);
  gp.assign(ns + 1, 0);
  for (size_t i = 0; i < ns; ++i) {
    const uint32_t nt = (uint32_t)ceil_div(segs[i].len, tile_len);
    tp[i + 1] = tp[i] + nt;
    gp[i + 1] = gp[i] + (uint32_t)ceil_div(nt, GROUP_TILES);
  }
}

int upload_src(const Buffers &B, const Layout &Lo, const SegSrc &s, hipStream_t st) {
  if (s.ns > Lo.seg_slots || s.ntiles > Lo.max_tiles || s.ngroups > Lo.max_groups) return fail_internal("work exceeds a workspace list or scratch area");
  CX_CHECK(hipMemcpyAsync(B.segs, s.segs, sizeof(Seg) * s.ns, hipMemcpyHostToDevice, st));
  CX_CHECK(hipMemcpyAsync(B.tile_prefix, s.tprefix, 4 * ((uint64_t)s.ns + 1), hipMemcpyHostToDevice, st));
  CX_CHECK(hipMemcpyAsync(B.group_prefix, s.gprefix, 4 * ((uint64_t)s.ns + 1), hipMemcpyHostToDevice, st));
  return CXBWT_OK;
}

// The final groups of the current level, with their count on the device.
int finish_finals_dev(const Build &b, hipStream_t st, unsigned emit_grid = PG_EMIT) {
  const Buffers &B = b.B;
  int rc;
  if ((rc = prefix_list(B, B.finals, (uint32_t)b.Lo.cap_finals, b.tile_len, nullptr, B.tile_prefix, nullptr, st,
                        B.counters + C_NFINAL)))
    return rc;
  k_emit_final<true><<<emit_grid, BLOCK, 0, st>>>(B.finals, B.tile_prefix, 0, B.counters + C_NFINAL, b.tile_len, B.keys0,
                                          B.keys1, B.hdl0, B.hdl1, B.pos64, B.text, B.srank, B.cmap, b.bwt, B.start_row);
  CX_LAUNCHED();
  return CXBWT_OK;
}

// What a level left in the lists for chunks and final groups, still to be
// finished.
struct LevelRest {
  LevelOut o{};
  int half = 0;  // of the lists; the other is free
  bool open = false;
};
int finish_rest(const Build &b, LevelRest &rest, PhaseTimer &T, hipStream_t st) {
  if (!rest.open) return CXBWT_OK;
  rest.open = false;
  Buffers B = b.B;
  if (rest.half) {
    B.chunks += b.Lo.cap_chunks / 2;
    B.finals += b.Lo.cap_finals / 2;
  }
  const LevelOut &o = rest.o;
  return finish_level(B, b.Lo, b.tu, b.nb, b.rmax, b.maxlen, b.bwt, o.n_chunks, o.n_finals, o.final_tiles, o.final_len, T,
                      st);
}

// Levels 2.. on the host's schedule, after a level 1 (or a range's list, or
// what the device left) that handed on acc: every segment of a level is split
// by one digit.  A level that fits the per-segment and per-tile scratch runs
// as one batch whose segment list is prepared on the device; a larger one
// is cut into batches on the host.
//
// The chunks and final groups of a level (of level 1 too: `first`) are
// launched behind the next level's kernels, so that the host reads that
// level's counts and plans the one after while they run, and the device does
// not wait for it (with the segment list's kernels, six of which became one or
// two: 20 Mbases at 2000x, 17 levels, 5.65 -> 5.07 ms; 200 Mbases in four
// ranges 13.0 -> 12.6; 400 Mbases, 5 levels, 11.6 -> 11.4).  Two levels then share the lists: with chunks of 512 a
// level makes at most nb / 128 chunks and nb / 513 groups (four lists' worth of
// S / C as for LISTED_LEVELS, and the samples, packed by 256, are at most half
// of nb), and half of the lists holds nb / 96 and nb / 386.  Smaller chunks are
// finished at once.
int run_levels(const Build &b, LevelOut acc, bool first, PhaseTimer &T, hipStream_t st) {
  const Buffers &B = b.B;
  const Layout &Lo = b.Lo;
  std::vector<Seg> big;
  std::vector<uint32_t> tprefix, gprefix;
  uint32_t ntiles = 0, ngroups = 0;
  uint32_t nbig = acc.n_big;
  int rc;
  LevelWait behind;
  const uint32_t half_chunks = (uint32_t)(Lo.cap_chunks / 2), half_finals = (uint32_t)(Lo.cap_finals / 2);
  const bool halves = b.Ls.chunk >= 512 && nbig && behind.open();
  LevelRest rest;
  if (first) {
    rest.o = acc;
    rest.open = true;
    if (!halves || acc.n_chunks > half_chunks || acc.n_finals > half_finals) {
      if ((rc = finish_rest(b, rest, T, st))) return rc;
    }
  }
  LevelOut o{};
  while (nbig) {
    if (nbig > Lo.cap_big) return fail_internal("work exceeds a workspace list or scratch area");
    g_stats.levels++;
    g_stats.host_levels++;
    g_stats.big_segments += nbig;
    g_stats.level_suffixes += acc.next_len;
    g_stats.regathered += acc.next_regather;
    g_stats.max_window = std::max<uint32_t>(g_stats.max_window, (uint32_t)acc.next_maxr);
    const uint64_t lt = acc.next_tiles, lg = acc.next_groups;
    acc = LevelOut{};
    if (nbig <= Lo.seg_slots && lt <= Lo.max_tiles && lg <= Lo.max_groups) {
      Lists Ls = b.Ls;
      LevelRest made;
      if (halves) {
        made.half = rest.open ? !rest.half : 0;
        Ls.chunks += made.half * half_chunks;
        Ls.finals += made.half * half_finals;
        Ls.cap_chunks = half_chunks;
        Ls.cap_finals = half_finals;
      }
      if ((rc = prefix_list(B, B.big_next, nbig, b.tile_len, B.segs, B.tile_prefix, B.group_prefix, st, nullptr, true)))
        return rc;
      if ((rc = launch_level_kernels(B, b.tu, Ls, b.nb, nbig, (uint32_t)lt, (uint32_t)lg, nullptr, T, st))) return rc;
      g_stats.level_batches++;
      if (halves) {
        if ((rc = behind.post(B, st))) return rc;
        if ((rc = finish_rest(b, rest, T, st))) return rc;
        if ((rc = behind.wait(o, st))) return rc;
      } else if ((rc = read_level(B, o, T, st))) {
        return rc;
      }
      record_shape(g_stats.levels - 1, LevelShape{nbig, (uint32_t)lt, (uint32_t)lg, o.n_chunks, o.n_finals,
                                                  (uint32_t)o.final_tiles});
      made.o = o;
      made.open = true;
      rest = made;
      if (!halves && (rc = finish_rest(b, rest, T, st))) return rc;
      acc = o;
    } else {
      if ((rc = finish_rest(b, rest, T, st))) return rc;
      if ((rc = fill_u32(B.counters + C_NBIG, 1, 0, st))) return rc;
      big.resize(nbig);
      CX_CHECK(hipMemcpyAsync(big.data(), B.big_next, sizeof(Seg) * nbig, hipMemcpyDeviceToHost, st));
      CX_CHECK(hipStreamSynchronize(st));
      for (size_t b0 = 0; b0 < big.size();) {
        const size_t b1 = batch_end(big, b0, Lo, b.tile_len);
        const std::vector<Seg> part(big.begin() + b0, big.begin() + b1);
        if ((rc = upload_segments(B, Lo, part, b.tile_len, tprefix, gprefix, ntiles, ngroups, st))) return rc;
        if ((rc = run_level_batch(B, Lo, b.tu, b.Ls, b.nb, b.rmax, b.maxlen, b.bwt, (uint32_t)part.size(), ntiles, ngroups, o,
                                  T, st)))
          return rc;
        record_shape(g_stats.levels - 1, LevelShape{(uint32_t)part.size(), ntiles, ngroups, o.n_chunks, o.n_finals,
                                                    (uint32_t)o.final_tiles});
        acc.next_len += o.next_len;
        acc.next_regather += o.next_regather;
        acc.next_maxr = std::max(acc.next_maxr, o.next_maxr);
        acc.next_tiles += o.next_tiles;
        acc.next_groups += o.next_groups;
        b0 = b1;
      }
    }
    nbig = o.n_big;
  }
  return finish_rest(b, rest, T, st);
}

// Levels whose chunks and final groups stay in their lists together: those of
// any three in a row fit.  A level makes at most 2 S / C chunks of the S
// suffixes that leave it in chunks of up to C, plus one for every segment it
// splits and every large bucket (each of more than C suffixes) it makes: over
// three levels at most 7 nb / C, which for C = 384 is less than the 4 nb / 192
// that the list holds for one level of the smallest chunks.  Final groups are
// disjoint.
constexpr uint32_t LISTED_LEVELS = 3;
// Most levels of a build that splits by the windows' own digits alone: eight a
// window, and in the last one, of which reads hold rem bases, those of its
// bases, one that finds the digits after them constant, and the length.
uint32_t most_levels(uint32_t maxlen) {
  const uint32_t d = (maxlen % W + 3) / 4;
  return 8 * (maxlen / W) + d + (d < 7 ? 1 : 0) + 1;
}
// Whether a build's levels can be listed.
bool levels_listed(const Build &b) {
  return b.tu.chunk_items >= 6 && b.Lo.seg_slots <= NEXT_SEGS &&
         b.Lo.cap_finals + 1 <= 256 * b.Lo.max_groups &&      // the groups' tile prefixes
         sizeof(Seg) * b.Lo.cap_big <= b.Lo.tile_hist_bytes;  // k_rest_level's second list
}

// Whether the segments that level 1 leaves of several collections fit the
// scratch of one batch: up to 256 of each that does not fall into chunks.  (Else
// level 2 stalls and the host finishes the build: not worth listing.)
bool level2_fits(const Build &b) {
  uint64_t segs = 0;
  for (const Seg &g : b.big) segs += g.len > 230ull * b.tu.chunk() ? 256 : 0;
  return b.ncoll == 1 || segs <= b.Lo.seg_slots;
}

// Levels scheduled at once for a build that the host will only look at when
// they are through (it finishes the build if that is not all): one level of
// 256 buckets, two of 65536, and the split of their ended suffixes.
uint32_t levels_ahead(const Build &b) {
  return b.nb <= 16ull * b.tu.chunk() ? 1u : b.nb <= 256ull * b.tu.chunk() ? 2u : 3u;
}

// The lists of a level whose number is `level` among `ended`: the segments it
// makes are those of level + 1.
Lists lists_for(const Build &b, uint32_t level, uint32_t ended) {
  Lists Ls = b.Ls;
  Ls.ended = level < ended;
  return Ls;
}

// After level 1's scan and scatter: the rest of `levels` levels sized on the
// device, five launches each, and every LISTED_LEVELS of them the chunks and
// final groups they listed.  Grids cover the counts seen (or the most that
// level 2 can have; later levels of a small build hold little); every kernel
// loops.  Then `rest` levels of a launch each, for inputs that need them.
int enqueue_listed_levels(const Build &b, uint32_t levels, uint32_t rest, uint32_t ended, PhaseTimer &T, hipStream_t st,
                          const std::vector<LevelShape> *shapes) {
  const Buffers &B = b.B;
  const Layout &Lo = b.Lo;
  const uint64_t nb = b.nb, chunk = b.tu.chunk();
  auto seen = [&](uint32_t lv) { return shapes && lv < shapes->size(); };
  int rc;
  uint32_t seen_chunks = 0;
  for (uint32_t lv = 0;; ++lv) {
    if (seen(lv)) seen_chunks += (*shapes)[lv].nchunks;
    const int last = lv + 1 == levels, flush = last || (lv + 1) % LISTED_LEVELS == 0;
    k_next_level<<<1, NEXT_WG, 0, st>>>(B.counters, B.stats, B.big_next, B.segs, B.tile_prefix, B.group_prefix, B.seg_or,
                                        B.seg_and, b.tile_len, Lo.seg_slots, Lo.max_tiles, Lo.max_groups, B.finals,
                                        (uint32_t)Lo.cap_finals, B.gsum, (uint32_t)Lo.cap_chunks, flush,
                                        !last ? NEXT_NOT_LAST : rest ? NEXT_REST : NEXT_LAST);
    CX_LAUNCHED();
    if (flush) {
      T.begin();
      // chunks hold two thirds of a chunk's suffixes and more on average; a small
      // build takes the looping kernel alone
      const uint64_t expect = std::max<uint64_t>(seen_chunks, 3 * nb / (2 * chunk) + 1);
      if ((rc = launch_local(B, b.tu, nb, b.rmax, b.bwt, (uint32_t)Lo.cap_chunks, B.counters + C_LCHUNK, st,
                             nb <= 1u << 20 ? 0u : grid_from((uint32_t)expect, 0), (unsigned)expect)))
        return rc;
      T.end(PH_LOCAL);
      T.begin();
      const uint64_t groups = std::min<uint64_t>(PG_EMIT, nb / (2 * chunk) + 16);
      k_emit_final<true><<<(unsigned)groups, BLOCK, 0, st>>>(B.finals, B.gsum, 0, B.counters + C_LFINAL, b.tile_len,
                                                            B.keys0, B.keys1, B.hdl0, B.hdl1, B.pos64, B.text, B.srank,
                                                            B.cmap, b.bwt, B.start_row);
      CX_LAUNCHED();
      T.end(PH_FINAL);
      seen_chunks = 0;
    }
    if (last) break;
    LevelShape sh;
    if (seen(lv + 1)) {
      sh = (*shapes)[lv + 1];
    } else {
      const uint64_t segs = std::min<uint64_t>(256ull * b.big.size(), nb / (chunk + 1) + 1);
      sh.nsegs = (uint32_t)(lv == 0 ? segs : segs / 8 + 1);
      sh.ntiles = (uint32_t)((lv == 0 ? nb : nb / 8) / b.tile_len + sh.nsegs);
      sh.ngroups = (uint32_t)(sh.ntiles / GROUP_TILES + sh.nsegs);
    }
    if ((rc = launch_level_kernels(B, b.tu, lists_for(b, lv + 2, ended), nb, 0, 0, 0, B.counters + C_NCUR, T, st, &sh)))
      return rc;
  }
  // the two lists in turn: the level's own, and the histograms' area
  constexpr unsigned REST_GRID = 256;
  Seg *const lists[2] = {B.big_next, (Seg *)B.tile_hist};
  for (uint32_t k = 0; k < rest; ++k) {
    uint32_t *const c = B.counters, *const nchunk = c + C_RCHUNK + k / LISTED_LEVELS % 2;
    const bool last = k + 1 == rest, opens = k % LISTED_LEVELS == 0;
    k_rest_level<<<REST_GRID, 64 * REST_NW, 0, st>>>(
        lists[k % 2], k ? c + C_REST + (k - 1) % 3 : c + C_NBIG, lists[1 - k % 2], last ? nullptr : c + C_REST + k % 3,
        (uint32_t)Lo.cap_big, c + C_REST + (k + 1) % 3, B.chunks, nchunk, (uint32_t)Lo.cap_chunks,
        opens ? c + C_RCHUNK + (k / LISTED_LEVELS + 1) % 2 : nullptr, (uint32_t)chunk, b.rmax, B.keys0, B.keys1, B.hdl0,
        B.hdl1, B.text, nb, B.srank, B.cmap, b.bwt, B.start_row, c, B.stats);
    CX_LAUNCHED();
    if (last || (k + 1) % LISTED_LEVELS == 0)
      if ((rc = launch_local(B, b.tu, nb, b.rmax, b.bwt, (uint32_t)Lo.cap_chunks, nchunk, st, 0, 2 * REST_GRID))) return rc;
  }
  return CXBWT_OK;
}

// Text records, read-end ranks, the collections that fit one chunk, and
// level 1.  Then either (device_levels = 0) the host schedules levels 2..
// with a counter readback per level, or the next device_levels levels are
// enqueued with their sizes read on the device (no host wait: the whole
// sequence can be captured), followed by a last step that flags segments
// left over.  The first `ended` levels split off ended suffixes first; the listed
// form takes a launch each for those after them.  Ends with term_pos.
int enqueue_body(const Build &b, const Level1Src &src, uint32_t device_levels, PhaseTimer &T, hipStream_t st,
                 const std::vector<LevelShape> *shapes = nullptr, uint32_t ended = ~0u) {
  const Buffers &B = b.B;
  const Layout &Lo = b.Lo;
  uint32_t *counters = B.counters;
  const uint64_t nb = b.nb;
  int rc;
  const bool planned = b.planned;
  if (!planned) CX_CHECK(hipMemcpyAsync(B.cmap, src.cm, sizeof(CollMap) * b.ncoll, hipMemcpyHostToDevice, st));
  if (nb == 0) return CXBWT_OK;

  // collections that fit one chunk: keys in read order, one unsplit chunk each
  if (src.small.ns) {
    if (!planned && (rc = upload_src(B, Lo, src.small, st))) return rc;
    T.begin();
    k_gen<<<src.small.ntiles, BLOCK, 0, st>>>(B.segs, B.tile_prefix, src.small.ns, b.tile_len, B.text, nb, B.keys0,
                                              B.hdl0);
    CX_LAUNCHED();
    T.end(PH_GEN);
    if (!planned)
      CX_CHECK(hipMemcpyAsync(B.chunks, src.small.segs, sizeof(Seg) * src.small.ns, hipMemcpyHostToDevice, st));
    if (!src.big.ns) {
      if ((rc = finish_level(B, Lo, b.tu, nb, b.rmax, b.maxlen, b.bwt, src.small.ns, 0, 0, 0, T, st))) return rc;
    } else {
      // level 1 appends its chunks after these
      CX_CHECK(hipMemcpyAsync(counters + C_NCHUNK, src.nsmall, 4, hipMemcpyHostToDevice, st));
    }
  }
  if (src.big.ns) {
    // level 1: keys computed from the 2-bit reads, counted, recomputed, scattered
    const uint32_t ns = src.big.ns, ntiles = src.big.ntiles, ngroups = src.big.ngroups;
    if (!planned && (rc = upload_src(B, Lo, src.big, st))) return rc;
    T.begin();
    if (b.tu.tile_items == 16)
      k_gen_hist<2><<<ntiles, BLOCK, 0, st>>>(B.segs, B.tile_prefix, ns, b.tile_len, B.text, nb, B.tile_hist);
    else
      k_gen_hist<1><<<ntiles, BLOCK, 0, st>>>(B.segs, B.tile_prefix, ns, b.tile_len, B.text, nb, B.tile_hist);
    CX_LAUNCHED();
    T.end(PH_GEN);
    T.begin();
    k_group_scan<false><<<ngroups, BLOCK, 0, st>>>(B.tile_prefix, B.group_prefix, ns, nullptr, B.tile_hist, B.gsum);
    CX_LAUNCHED();
    launch_level_scan(B, ns, ngroups, lists_for(b, 1, ended), 1, st);
    CX_LAUNCHED();
    T.end(PH_SCAN);
    T.begin();
#define CX_GEN_SCATTER(TI, NW)                                                                                    \
  k_gen_scatter<TI, NW><<<ntiles, 64 * NW, 0, st>>>(B.segs, B.tile_prefix, B.group_prefix, ns, B.text, nb,         \
                                                    B.tile_hist, B.gsum, B.keys1, B.hdl1)
    if (b.tu.tile_items == 16) CX_GEN_SCATTER(8, 8);
    else if (b.tu.tile_items == 8) CX_GEN_SCATTER(8, 4);
    else CX_GEN_SCATTER(6, 4);
#undef CX_GEN_SCATTER
    CX_LAUNCHED();
    T.end(PH_SCATTER);
    if (device_levels == 0) {
      LevelOut o{};
      if ((rc = read_level(B, o, T, st))) return rc;
      record_shape(0, LevelShape{ns, ntiles, ngroups, o.n_chunks, o.n_finals, (uint32_t)o.final_tiles});
      if ((rc = run_levels(b, o, true, T, st))) return rc;
    } else if (levels_listed(b)) {
      const uint32_t levels = std::min(device_levels, ended);
      if ((rc = enqueue_listed_levels(b, levels, device_levels - levels, ended, T, st, shapes))) return rc;
    } else {
      const uint32_t *ncur = counters + C_NCUR;
      const LevelShape none;
      auto seen = [&](uint32_t lv) -> const LevelShape & {
        return shapes && lv < shapes->size() ? (*shapes)[lv] : none;
      };
      for (uint32_t lv = 0;; ++lv) {
        // the level just scanned: fold, finish its chunks and final groups
        k_level_fold<<<1, 64, 0, st>>>(B.stats, counters, counters + C_FLAGS, nullptr);
        CX_LAUNCHED();
        T.begin();
        if ((rc = launch_local(B, b.tu, nb, b.rmax, b.bwt, (uint32_t)Lo.cap_chunks, counters + C_NCHUNK, st,
                               grid_from(seen(lv).nchunks, 0))))
          return rc;
        T.end(PH_LOCAL);
        T.begin();
        if ((rc = finish_finals_dev(b, st, grid_from(seen(lv).ftiles, PG_EMIT)))) return rc;
        T.end(PH_FINAL);
        const int last = lv == device_levels - 1;
        k_level_step<<<1, 64, 0, st>>>(counters, Lo.seg_slots, Lo.max_tiles, Lo.max_groups, last);
        CX_LAUNCHED();
        if (last) break;
        // the next level, sized on the device
        if ((rc = prefix_list(B, B.big_next, (uint32_t)Lo.seg_slots, b.tile_len, B.segs, B.tile_prefix,
                              B.group_prefix, st, ncur)))
          return rc;
        k_fill_seg<<<PG_FILL, 256, 0, st>>>(B.seg_or, B.seg_and, ncur);
        CX_LAUNCHED();
        if ((rc = launch_level_kernels(B, b.tu, lists_for(b, lv + 2, ended), nb, 0, 0, 0, ncur, T, st, &seen(lv + 1))))
          return rc;
      }
    }
  }
  T.begin();
  if ((rc = launch_term(b, st))) return rc;
  T.end(PH_FINAL);
  return CXBWT_OK;
}

// The counters of a build whose last kernel (launch_term) is enqueued: the
// device status, and the statistics' totals.
int read_totals(const Build &b, PhaseTimer &T, hipStream_t st, uint32_t (&hc)[C_COUNT]) {
  CX_CHECK(hipMemcpyAsync(hc, b.B.counters, sizeof(hc), hipMemcpyDeviceToHost, st));
  CX_CHECK(hipStreamSynchronize(st));
  T.collect();
  uint64_t t[2];
  memcpy(t, hc + C_TOTALS, sizeof(t));
  g_stats.window_fetches += t[0];
  g_stats.scattered_suffixes += t[1];
  return CXBWT_OK;
}

// Level-1 sources taken from the plan's vectors (an eager build).
struct Level1Vectors {
  std::vector<uint32_t> btp, bgp, stp, sgp;
  uint32_t nsmall = 0;
  Level1Src src;
  void make(const Build &b) {
    seg_prefixes(b.big, b.tile_len, btp, bgp);
    seg_prefixes(b.small, b.tile_len, stp, sgp);
    nsmall = (uint32_t)b.small.size();
    src.cm = b.cm.data();
    src.big = SegSrc{b.big.data(), btp.data(), bgp.data(), (uint32_t)b.big.size(), btp.back(), bgp.back()};
    src.small = SegSrc{b.small.data(), stp.data(), sgp.data(), nsmall, stp.back(), sgp.back()};
    src.nsmall = &nsmall;
  }
};

// Adds the level 1 of b's collections.
void level1_stats(const Build &b) {
  for (const Seg &g : b.small) g_stats.chunk_suffixes += g.len;
  if (!b.big.empty()) {
    g_stats.levels++;
    g_stats.big_segments += b.big.size();
    for (const Seg &g : b.big) {
      g_stats.chunk_suffixes += g.len;
      g_stats.level_suffixes += g.len;
    }
  }
}

// The stringword schedule (Section 3.2) over one collection: for every
// window from the last to the first, its keys in position order, permuted
// into the current order, then one stable pass per varying digit, least
// significant first; finally the rows and term_pos.
int run_stringword(const Build &b, PhaseTimer &T, hipStream_t st) {
  constexpr int TI = 8, NW = 4;
  constexpr uint32_t TL = 64 * NW * TI;
  const Buffers &B = b.B;
  const Layout &Lo = b.Lo;
  const uint64_t nb = b.nb;
  int rc;
  g_stats.schedule = CXBWT_SCHEDULE_STRINGWORD;
  if (b.ncoll) CX_CHECK(hipMemcpyAsync(B.cmap, b.cm.data(), sizeof(CollMap), hipMemcpyHostToDevice, st));
  if (nb) {
    const uint64_t ntiles = ceil_div(nb, TL), ngroups = ceil_div(ntiles, GROUP_TILES);
    if (ntiles > Lo.max_tiles || ngroups > Lo.max_groups || ntiles > 0x7FFFFFFFull) return fail_internal("work exceeds a workspace list or scratch area");
    const uint32_t tp[2] = {0, (uint32_t)ntiles}, gp[2] = {0, (uint32_t)ngroups};
    CX_CHECK(hipMemcpyAsync(B.tile_prefix, tp, sizeof(tp), hipMemcpyHostToDevice, st));
    CX_CHECK(hipMemcpyAsync(B.group_prefix, gp, sizeof(gp), hipMemcpyHostToDevice, st));
    uint64_t *K[2] = {B.keys0, B.keys1};
    uint32_t *H[2] = {B.hdl0, B.hdl1};
    unsigned long long *orand = B.seg_or;  // OR and AND of a window's ordering bits
    const unsigned grid = (unsigned)std::min<uint64_t>(ceil_div(nb, BLOCK), 65536);
    int cur = 0;
    for (int w = (int)b.rmax - 1; w >= 0; --w) {
      if ((rc = fill_u64((uint64_t *)orand, 1, 0, st))) return rc;
      if ((rc = fill_u64((uint64_t *)orand + 1, 1, ~0ull, st))) return rc;
      T.begin();
      k_sched_window<<<grid, BLOCK, 0, st>>>(B.text, B.srank, nb, (uint32_t)w, K[1 - cur], orand);
      CX_LAUNCHED();
      k_sched_gather<<<grid, BLOCK, 0, st>>>(K[1 - cur], nb, w == (int)b.rmax - 1, K[cur], H[cur]);
      CX_LAUNCHED();
      T.end(PH_GEN);
      uint64_t oa[2];
      CX_CHECK(hipMemcpyAsync(oa, orand, sizeof(oa), hipMemcpyDeviceToHost, st));
      CX_CHECK(hipStreamSynchronize(st));
      T.collect();
      g_stats.window_fetches += nb;
      for (int d = 7; d >= 0; --d) {
        if (((oa[0] ^ oa[1]) & digit_mask(d)) == 0) continue;  // constant digit: the pass would not move anything
        T.begin();
        k_sched_hist<TL><<<(unsigned)ntiles, BLOCK, 0, st>>>(K[cur], nb, d, B.tile_hist);
        CX_LAUNCHED();
        T.end(PH_HIST);
        T.begin();
        k_group_scan<false><<<(unsigned)ngroups, BLOCK, 0, st>>>(B.tile_prefix, B.group_prefix, 1, nullptr,
                                                                 B.tile_hist, B.gsum);
        CX_LAUNCHED();
        k_sched_top<<<1, 64, 0, st>>>(B.gsum, (uint32_t)ngroups);
        CX_LAUNCHED();
        T.end(PH_SCAN);
        T.begin();
        k_sched_scatter<TI, NW><<<(unsigned)ntiles, 64 * NW, 0, st>>>(K[cur], H[cur], nb, d, B.tile_hist, B.gsum,
                                                                      K[1 - cur], H[1 - cur]);
        CX_LAUNCHED();
        T.end(PH_SCATTER);
        cur = 1 - cur;
        g_stats.levels++;
        g_stats.scattered_suffixes += nb;
        g_stats.level_suffixes += nb;
      }
      g_stats.max_window = std::max<uint32_t>(g_stats.max_window, (uint32_t)w);
    }
    T.begin();
    k_sched_emit<<<grid, BLOCK, 0, st>>>(K[cur], H[cur], nb, B.cmap, B.text, B.srank, b.bwt, B.start_row);
    CX_LAUNCHED();
    T.end(PH_FINAL);
  }
  T.begin();
  if ((rc = launch_term(b, st))) return rc;
  T.end(PH_FINAL);
  return CXBWT_OK;
}

// After a run of levels the device scheduled (a graph replay): the status,
// the statistics the device counted, and the levels it left to the host.
// hc0 holds the counters read after the run.
int finish_device_levels(const Build &b, const uint32_t (&hc0)[C_COUNT], PhaseTimer &T, hipStream_t st) {
  uint32_t hc[C_COUNT];
  memcpy(hc, hc0, sizeof(hc));
  int rc;
  if (hc[C_STATUS] & (ST_BAD_OFFSETS | ST_TOO_LONG)) return fail_status(hc[C_STATUS]);
  if (hc[C_STATUS]) return fail_status(hc[C_STATUS]);
  uint64_t g[G_COUNT], f[K_LEVEL_KINDS];
  memcpy(g, hc + C_CUM, sizeof(g));
  memcpy(f, hc + C_FOLD, sizeof(f));
  g_stats.levels += (uint32_t)g[G_LEVELS];
  g_stats.big_segments += g[G_BIGSEG];
  g_stats.level_suffixes += g[G_LEVSUF];
  g_stats.regathered += g[G_REGATH];
  g_stats.max_window = std::max<uint32_t>(g_stats.max_window, (uint32_t)g[G_MAXWIN]);
  g_stats.chunks += g[G_CHUNKS];
  g_stats.final_big += g[G_FINALS];
  g_stats.chunk_suffixes -= g[G_FINLEN];
  g_stats.level_batches += (uint32_t)g[G_BATCHES];
  if (!(hc[C_FLAGS] & (FL_STALLED | FL_INCOMPLETE))) return CXBWT_OK;
  // the device schedule did not cover the build: the host finishes it
  LevelOut acc{};
  acc.next_len = f[K_NEXT_LEN - K_LEVEL_FIRST];
  acc.next_regather = f[K_NEXT_REGATHER - K_LEVEL_FIRST];
  acc.next_maxr = f[K_NEXT_MAXR - K_LEVEL_FIRST];
  acc.next_tiles = f[K_NEXT_TILES - K_LEVEL_FIRST];
  acc.next_groups = f[K_NEXT_GROUPS - K_LEVEL_FIRST];
  acc.n_big = hc[C_NBIG];
  if ((rc = run_levels(b, acc, false, T, st))) return rc;
  if ((rc = launch_term(b, st))) return rc;
  // the statistics block still holds the device levels' counts: take the rest only
  g_stats.window_fetches = 0;
  g_stats.scattered_suffixes = 0;
  if ((rc = read_totals(b, T, st, hc))) return rc;
  if (hc[C_STATUS]) return fail_status(hc[C_STATUS]);
  return CXBWT_OK;
}

// ---- the build by induced order ------------------------------------------
// Taken from this many bases on: the steps are about thirty launches of their
// own, and up to 16.7 Mbases the sort lists its levels: 16 Mbases of 100-base
// reads at 20x take 0.97 ms here and 0.95 by the sort, 17 Mbases 0.99 and 1.08,
// 18 of 250 bases 1.21 and 1.41 (deeper reads gain from less on: at 2000x, 10
// Mbases take 3.8 ms here and 9.2 by the sort, but the depth is not known
// before).
#ifndef CXBWT_INDUCE_MIN_BASES
#define CXBWT_INDUCE_MIN_BASES 16500000ull
#endif
// Time that the runs beyond the regions may take besides a hundredth of the
// nanoseconds of the bases (run_induced).
#ifndef CXBWT_INDUCE_TAIL_NS
#define CXBWT_INDUCE_TAIL_NS 50000ull
#endif
// Not where all reads are shorter.  They would be faster this way too (47 Mbases
// of 30-base reads 3.5 ms by the sort, 1.7 by samples; 20 Mbases the same), but
// nearly all of their suffixes are in large groups of identical ones, which
// cxbwt_stats.final_big counts for the callers of such builds, and of which the
// samples are a third.
constexpr uint32_t INDUCE_MIN_READ = 33;

// One collection's plan: the buckets' parts from the counted types.
struct InduceColl {
  uint32_t n[2][4][RUN_REGIONS + 1];  // [L, S][base][run]
  uint32_t samples[4], maxrun[8];
  uint64_t l0[4], s1[4];  // the L part's first row, the S part's end
  uint64_t nl[4], ns[4], first_sample;
};

// Host image of everything the steps read: descriptors of every step, laid
// out in one block for one copy.
struct StepBlob {
  std::vector<unsigned char> bytes;
  size_t put(const void *p, size_t n) {
    const size_t at = (bytes.size() + 15) & ~(size_t)15;
    bytes.resize(at + n);
    if (n) memcpy(bytes.data() + at, p, n);
    return at;
  }
};
struct StepPlan {
  size_t segs = 0, tiles = 0, coll_tiles = 0, coll_groups = 0;
  uint32_t nsegs = 0, ntiles = 0, ngroups = 0;
};

// src: the step's sources of every collection, in order.
StepPlan plan_step(StepBlob &blob, const std::vector<std::vector<IndSeg>> &src) {
  std::vector<IndSeg> segs;
  std::vector<uint32_t> tiles{0}, ct{0}, cg{0};
  for (const auto &list : src) {
    for (const IndSeg &g : list) {
      if (!g.len) continue;
      segs.push_back(g);
      tiles.push_back(tiles.back() + (uint32_t)ceil_div(g.len, IND_TILE));
    }
    cg.push_back(cg.back() + (uint32_t)ceil_div(tiles.back() - ct.back(), GROUP_TILES));
    ct.push_back(tiles.back());
  }
  StepPlan p;
  p.segs = blob.put(segs.data(), sizeof(IndSeg) * segs.size());
  p.tiles = blob.put(tiles.data(), 4 * tiles.size());
  p.coll_tiles = blob.put(ct.data(), 4 * ct.size());
  p.coll_groups = blob.put(cg.data(), 4 * cg.size());
  p.nsegs = (uint32_t)segs.size();
  p.ntiles = tiles.back();
  p.ngroups = cg.back();
  return p;
}

// The collections of b to be built by induced order (`large`) and those to be
// sorted in any case (`rest`); false when too few bases are in large ones.
// A collection of up to about 256 chunks is sorted by one level: cheaper than
// its samples and their steps, whose host plan and descriptors cost half a
// microsecond a collection besides (by the sort and by samples, 200 Mbases in
// collections of 30, 65, 100, 130 and 200 kbases: 3.5 and 6.6, 3.8 and 4.7, 3.9
// and 4.3, 6.7 and 4.1, 9.7 and 5.3 ms; the level's buckets are uneven, so some
// are above a chunk from 200 chunks on).  A few small ones are carried along:
// a sort of their own is a dozen launches and two waits.
#ifndef CXBWT_INDUCE_COLL_CHUNKS
#define CXBWT_INDUCE_COLL_CHUNKS 215ull
#endif
constexpr size_t INDUCE_CARRIED = 400;
bool pick_induced(const Build &b, std::vector<Seg> &large, std::vector<Seg> &rest) {
  const uint64_t least = CXBWT_INDUCE_COLL_CHUNKS * b.tu.chunk();
  auto is_large = [&](const Seg &g) { return b.ncoll == 1 || g.len >= least; };
  uint64_t bases = 0;
  size_t small = 0;
  for (const Seg &g : b.big) {
    if (is_large(g)) bases += g.len;
    else ++small;
  }
  if (bases < CXBWT_INDUCE_MIN_BASES) return false;
  for (const Seg &g : b.big) (small <= INDUCE_CARRIED || is_large(g) ? large : rest).push_back(g);
  return true;
}

// Plans and runs the build by induced order of b's collections above one
// chunk (the others have been built).  *taken stays false, and nothing has
// been written, where it does not apply.
// blob: the host image of the steps, which the caller keeps until it has waited
// for the stream.
int run_induced(const Build &b, StepBlob &blob, bool *taken, PhaseTimer &T, hipStream_t st) {
  *taken = false;
  const Layout &Lo = b.Lo;
  const uint64_t nb = b.nb;
  const uint32_t nc = (uint32_t)b.big.size();
  int rc;
  // the text of every collection in tiles, counted
  std::vector<uint32_t> tp, gp;
  {
    std::vector<Seg> whole(b.big);  // tiles begin at the record a collection begins in
    for (Seg &g : whole) g.len = (uint32_t)std::min<uint64_t>((uint64_t)g.len + g.start % 16, 0xFFFFFFFFull);
    seg_prefixes(whole, SMP_TILE, tp, gp);
  }
  const uint32_t ntiles = tp.back(), ngroups = gp.back();
  const uint32_t replicas = std::max<uint32_t>(1, 64 / nc);
  const uint64_t n_counts = (uint64_t)nc * replicas * TC_WORDS;
  if (nc > Lo.seg_slots || nc > Lo.cap_finals || ntiles > Lo.max_tiles || ngroups > Lo.max_groups ||
      4 * n_counts > 4 * 256 * Lo.max_groups)
    return CXBWT_OK;
  std::vector<Seg> text(b.big);
  for (uint32_t c = 0; c < nc; ++c) text[c].coll = c;  // collections are numbered among those built here
  Seg *d_text = b.B.finals;  // level 1 has no final groups
  uint32_t *d_counts = b.B.gsum;
  CX_CHECK(hipMemcpyAsync(d_text, text.data(), sizeof(Seg) * nc, hipMemcpyHostToDevice, st));
  CX_CHECK(hipMemcpyAsync(b.B.tile_prefix, tp.data(), 4 * ((uint64_t)nc + 1), hipMemcpyHostToDevice, st));
  CX_CHECK(hipMemcpyAsync(b.B.group_prefix, gp.data(), 4 * ((uint64_t)nc + 1), hipMemcpyHostToDevice, st));
  if ((rc = fill_u32(d_counts, n_counts, 0, st))) return rc;
  T.begin();
  k_sample_hist<<<(unsigned)ceil_div(ntiles, HIST_TILES), BLOCK, 0, st>>>(
      d_text, b.B.tile_prefix, nc, ntiles, b.B.text, b.B.tile_hist, d_counts, replicas);
  CX_LAUNCHED();
  T.end(PH_GEN);
  std::vector<uint32_t> hc(n_counts);
  CX_CHECK(hipMemcpyAsync(hc.data(), d_counts, 4 * n_counts, hipMemcpyDeviceToHost, st));
  CX_CHECK(hipStreamSynchronize(st));
  T.collect();

  // the buckets' parts
  std::vector<InduceColl> cs(nc);
  uint64_t M = 0, tail = 0, tail_steps = 0;
  for (uint32_t c = 0; c < nc; ++c) {
    InduceColl &q = cs[c];
    memset(&q, 0, sizeof(q));
    for (uint32_t r = 0; r < replicas; ++r) {
      const uint32_t *w = hc.data() + ((uint64_t)c * replicas + r) * TC_WORDS;
      for (int i = 0; i < 128; ++i) (&q.n[0][0][0])[i] += w[i];
      for (int i = 0; i < 8; ++i) q.maxrun[i] = std::max(q.maxrun[i], w[TC_MAXRUN + i]);
      for (int i = 0; i < 4; ++i) q.samples[i] += w[TC_SAMPLES + i];
    }
    uint64_t at = text[c].start;
    for (int d = 0; d < 4; ++d) {
      for (int k = 0; k <= RUN_REGIONS; ++k) {
        q.nl[d] += q.n[0][d][k];
        q.ns[d] += q.n[1][d][k];
      }
      q.l0[d] = at;
      at += q.nl[d] + q.ns[d];
      q.s1[d] = at;
      tail += (uint64_t)q.n[0][d][RUN_REGIONS] + q.n[1][d][RUN_REGIONS];
    }
    if (at != (uint64_t)text[c].start + text[c].len) return fail_internal("suffix types do not add up");
    q.first_sample = M;
    for (int d = 0; d < 4; ++d) M += q.samples[d];
  }
  for (int i = 0; i < 8; ++i) {
    uint32_t longest = 0;
    for (const InduceColl &q : cs) longest = std::max(longest, q.maxrun[i]);
    tail_steps += longest > (uint32_t)RUN_REGIONS ? longest - RUN_REGIONS + 1 : 0;
  }
  // runs beyond the regions are followed a base at a time by one workgroup
  // (about 5 us a base, 1 ns a suffix): left to the sort where they could
  // cost half of what this saves (20 ns per 1000 bases) and more
  if (tail_steps * 5000 + tail > nb / 100 + CXBWT_INDUCE_TAIL_NS) return CXBWT_OK;

  // the samples' sort buffers, the sorted samples and the rows, in the space
  // of the general sort buffers
  Build s = b;
  s.B.sample = true;
  s.B.pair = nb >= PAIR_MEAN_READ * b.n;
  unsigned char *const arena = (unsigned char *)b.B.keys0;
  const uint64_t room = (uint64_t)((unsigned char *)(b.B.hdl1 + nb) - arena);
  uint64_t off = 0;
  auto take = [&](uint64_t bytes) {
    unsigned char *p = arena + off;
    off = align_up(off + bytes);
    return p;
  };
  s.B.keys0 = (uint64_t *)take(8 * M);
  s.B.keys1 = (uint64_t *)take(8 * M);
  s.B.hdl0 = (uint32_t *)take(4 * M);
  s.B.hdl1 = (uint32_t *)take(4 * M);
  s.B.smp.pl = (uint32_t *)take(4 * M);
  s.B.smp.h = (uint32_t *)take(4 * M);
  s.B.smp.code = (uint8_t *)take(M);
  uint2 *rows = (uint2 *)take(8 * nb);
  if (off > room) return CXBWT_OK;

  // the steps: terminators; L of A, C, G; S of T, G, C; the rows of A
  std::vector<CollMap> cm(nc);
  std::vector<uint32_t> cur((size_t)nc * 128, 0);
  std::vector<IndTail> tails[2][4];
  for (uint32_t c = 0; c < nc; ++c) {
    cm[c] = b.cm[b.big[c].coll];
    const InduceColl &q = cs[c];
    for (int d = 0; d < 4; ++d) {
      uint64_t l = q.l0[d], e = q.s1[d];
      for (int k = 0; k < RUN_REGIONS; ++k) {
        cur[(size_t)c * 128 + d * 16 + k] = (uint32_t)l;
        cur[(size_t)c * 128 + 64 + d * 16 + k] = (uint32_t)e;
        if (k == RUN_REGIONS - 1) {
          tails[0][d].push_back(IndTail{(uint32_t)l, q.n[0][d][k], (uint32_t)(q.l0[d] + q.nl[d])});
          tails[1][d].push_back(IndTail{(uint32_t)(e - q.n[1][d][k]), q.n[1][d][k], (uint32_t)(q.l0[d] + q.nl[d])});
        }
        l += q.n[0][d][k];
        e -= q.n[1][d][k];
      }
    }
  }
  StepPlan seeds, left[3], right[4];
  {
    std::vector<std::vector<IndSeg>> src(nc);
    for (uint32_t c = 0; c < nc; ++c) {
      const uint64_t r0 = b.coll_reads[b.big[c].coll], r1 = b.coll_reads[b.big[c].coll + 1];
      src[c] = {IndSeg{(uint32_t)r0, (uint32_t)(r1 - r0), c, SRC_READS}};
    }
    seeds = plan_step(blob, src);
    for (int d = 0; d < 3; ++d) {
      for (uint32_t c = 0; c < nc; ++c) {
        uint64_t at = cs[c].first_sample;
        for (int x = 0; x < d; ++x) at += cs[c].samples[x];
        src[c] = {IndSeg{(uint32_t)cs[c].l0[d], (uint32_t)cs[c].nl[d], c, SRC_ROWS},
                  IndSeg{(uint32_t)at, cs[c].samples[d], c, SRC_SAMPLES}};
      }
      left[d] = plan_step(blob, src);
    }
    for (int d = 0; d < 4; ++d) {
      for (uint32_t c = 0; c < nc; ++c)
        src[c] = {IndSeg{(uint32_t)cs[c].l0[d], (uint32_t)(cs[c].s1[d] - cs[c].l0[d]), c, SRC_ROWS}};
      right[d] = plan_step(blob, src);
    }
  }
  const size_t o_cm = blob.put(cm.data(), sizeof(CollMap) * nc);
  const size_t o_cur = blob.put(cur.data(), 4 * cur.size());
  size_t o_tail[2][4];
  bool has_tail[2][4];
  for (int t = 0; t < 2; ++t)
    for (int d = 0; d < 4; ++d) {
      o_tail[t][d] = blob.put(tails[t][d].data(), sizeof(IndTail) * nc);
      has_tail[t][d] = false;
      for (const InduceColl &q : cs) has_tail[t][d] |= q.n[t][d][RUN_REGIONS] != 0;
    }
  // (the descriptors take the place of the chunk list, which the sort is done with)
  uint32_t most_tiles = seeds.ntiles, most_groups = seeds.ngroups;
  for (const StepPlan &p : left) most_tiles = std::max(most_tiles, p.ntiles), most_groups = std::max(most_groups, p.ngroups);
  for (const StepPlan &p : right) most_tiles = std::max(most_tiles, p.ntiles), most_groups = std::max(most_groups, p.ngroups);
  if (blob.bytes.size() > sizeof(Seg) * Lo.cap_chunks || 256ull * most_tiles > Lo.tile_hist_bytes ||
      256ull * most_groups > 4ull * 256 * Lo.max_groups)
    return CXBWT_OK;
  *taken = true;

  // sort the samples: level 1 from the text, then levels and chunks
  s.tu = Tuning{16, 8, CXBWT_SCHEDULE_MSD};
  s.tile_len = s.tu.tile_len();
  s.rmax = b.maxlen / SampleKey::FULL + 1;
  s.Ls.rmax = s.rmax;
  s.Ls.chunk = SAMPLE_CHUNK;
  s.Ls.pack = s.B.pair ? PAIR_PACK : SAMPLE_CHUNK;
  s.Ls.tile_len = s.tile_len;
  std::vector<Seg> seg(nc);
  g_stats.chunk_suffixes += M;
  g_stats.levels++;
  g_stats.big_segments += nc;
  g_stats.level_suffixes += M;
  for (uint32_t c = 0; c < nc; ++c) {
    uint64_t len = 0;
    for (int d = 0; d < 4; ++d) len += cs[c].samples[d];
    seg[c] = Seg{(uint32_t)cs[c].first_sample, (uint32_t)len, 0, 0, 0, 0, 0, 0, c};
  }
  if (M) {
    CX_CHECK(hipMemcpyAsync(s.B.segs, seg.data(), sizeof(Seg) * nc, hipMemcpyHostToDevice, st));
    if ((rc = fill_u32(s.B.counters + C_NFINAL, 3, 0, st))) return rc;
    T.begin();
    k_group_scan<false><<<ngroups, BLOCK, 0, st>>>(s.B.tile_prefix, s.B.group_prefix, nc, nullptr, s.B.tile_hist,
                                                   s.B.gsum);
    CX_LAUNCHED();
    launch_level_scan(s.B, nc, ngroups, s.Ls, 1, st);
    CX_LAUNCHED();
    T.end(PH_SCAN);
    T.begin();
    k_sample_scatter<<<ntiles, 64 * SMP_NW, 0, st>>>(d_text, s.B.tile_prefix, s.B.group_prefix, nc, s.B.text,
                                                     s.B.tile_hist, s.B.gsum, s.B.keys1, s.B.hdl1);
    CX_LAUNCHED();
    T.end(PH_SCATTER);
    LevelOut o{};
    if ((rc = read_level(s.B, o, T, st))) return rc;
    if ((rc = run_levels(s, o, true, T, st))) return rc;
  }

  // the steps, with every size known
  unsigned char *const dev = (unsigned char *)b.B.chunks;
  CX_CHECK(hipMemcpyAsync(dev, blob.bytes.data(), blob.bytes.size(), hipMemcpyHostToDevice, st));
  IndData D;
  D.rows = rows;
  D.bwt = b.bwt;
  D.cmap = (const CollMap *)(dev + o_cm);
  D.smp = s.B.smp;
  D.text = b.B.text;
  D.srank = b.B.srank;
  D.offsets = b.offsets;
  D.start_row = b.B.start_row;
  D.hist = b.B.tile_hist;
  D.gtot = b.B.gsum;
  D.cursor = (uint32_t *)(dev + o_cur);
  D.status = b.B.counters + C_STATUS;
  D.nb = nb;
  auto step = [&](const StepPlan &p, uint32_t base) {
    return IndStep{(const IndSeg *)(dev + p.segs), (const uint32_t *)(dev + p.tiles),
                   (const uint32_t *)(dev + p.coll_tiles), (const uint32_t *)(dev + p.coll_groups), p.nsegs, p.ntiles,
                   nc, base};
  };
#define CX_STEP(LTR, PLAN, BASE)                                              \
  do {                                                                        \
    if ((PLAN).ntiles) {                                                      \
      const IndStep P = step(PLAN, BASE);                                     \
      const unsigned grid = (unsigned)ceil_div(P.ntiles, WAVES);              \
      k_ind_count<LTR><<<grid, BLOCK, 0, st>>>(P, D);                         \
      CX_LAUNCHED();                                                          \
      k_ind_group<<<(PLAN).ngroups, BLOCK, 0, st>>>(P, D);                    \
      CX_LAUNCHED();                                                          \
      k_ind_top<LTR><<<nc, 64 * TOP_WAVES, 0, st>>>(P, D);                    \
      CX_LAUNCHED();                                                          \
      k_ind_scatter<LTR><<<grid, BLOCK, 0, st>>>(P, D);                       \
      CX_LAUNCHED();                                                          \
    }                                                                         \
  } while (0)
#define CX_TAIL(LTR, DIR, BASE)                                                                          \
  do {                                                                                                   \
    if (has_tail[DIR][BASE]) {                                                                           \
      k_ind_tail<LTR><<<nc, TAIL_WG, 0, st>>>((const IndTail *)(dev + o_tail[DIR][BASE]), BASE, D);      \
      CX_LAUNCHED();                                                                                     \
    }                                                                                                    \
  } while (0)
  T.begin();
  CX_STEP(true, seeds, 4u);
  for (uint32_t d = 0; d < 4; ++d) {
    CX_TAIL(true, 0, d);
    if (d < 3) CX_STEP(true, left[d], d);
  }
  for (uint32_t d = 4; d-- > 0;) {
    CX_TAIL(false, 1, d);
    if (d) CX_STEP(false, right[d], d);
  }
  if (right[0].ntiles) {
    const IndStep P = step(right[0], 0);
    k_ind_emit<<<(unsigned)ceil_div(P.ntiles, WAVES), BLOCK, 0, st>>>(P, D);
    CX_LAUNCHED();
  }
#undef CX_STEP
#undef CX_TAIL
  T.end(PH_INDUCE);
  T.begin();
  if ((rc = launch_term(b, st))) return rc;
  T.end(PH_FINAL);
  return CXBWT_OK;
}

// The whole build for ncoll collections laid end to end (a single build is
// one collection).  coll_reads (host) holds ncoll + 1 read boundaries.
int run_build(const uint64_t *packed, const uint64_t *offsets, uint64_t n, uint64_t nb, uint32_t maxlen,
              const uint64_t *coll_reads, uint32_t ncoll, uint8_t *bwt, uint64_t *term_pos, unsigned char *ws,
              hipStream_t st, bool allow_timing = true) {
  g_stats = cxbwt_stats{};
  g_last_error[0] = 0;
  PhaseTimer T{st, allow_timing && g_timing != 0, {}};
  Build b;
  build_init(b, packed, offsets, n, nb, maxlen, coll_reads, ncoll, bwt, term_pos, ws);
  const bool msd = !(ncoll == 1 && b.tu.schedule == CXBWT_SCHEDULE_STRINGWORD);
  const bool induce = msd && nb >= CXBWT_INDUCE_MIN_BASES && maxlen >= INDUCE_MIN_READ;
  // small builds run their levels without a look from the host in between;
  // for one collection it need not look at the offsets' verdict either
  // (kernels stay in bounds on invalid offsets, as in a replayed graph)
  const bool ahead = msd && !induce && levels_listed(b);
  int rc;
  if ((rc = enqueue_prep(b, b.coll_reads.data(), nullptr, T, st))) return rc;
  if ((rc = enqueue_records(b, T, st))) return rc;
  if (ahead && ncoll == 1) plan_single(b);
  else if ((rc = plan_level1(b, T, st))) return rc;
  uint32_t hc[C_COUNT];
  Build apart;           // collections sorted beside a build by induced order
  Level1Vectors v, va;   // sources of copies, kept until the last wait
  StepBlob blob;         // the same
  if (!msd) {
    if ((rc = run_stringword(b, T, st))) return rc;
  } else {
    bool done = false;
    std::vector<Seg> large, rest;
    if (induce && pick_induced(b, large, rest)) {
      if (!rest.empty() || !b.small.empty()) {
        apart = b;
        apart.big.swap(rest);
        va.make(apart);
        level1_stats(apart);
        if ((rc = enqueue_body(apart, va.src, 0, T, st))) return rc;
        if ((rc = fill_u32(b.B.counters + C_NFINAL, 3, 0, st))) return rc;  // the lists, as level 1 finds them
      }
      b.big.swap(large);
      b.small.clear();
      if ((rc = run_induced(b, blob, &done, T, st))) return rc;
      b.planned = false;  // its tiles have taken the plan's place
    }
    if (!done) {
      v.make(b);
      level1_stats(b);
      const bool listed = ahead && !b.big.empty() && level2_fits(b);
      if ((rc = enqueue_body(b, v.src, listed ? levels_ahead(b) : 0, T, st))) return rc;
      if (listed) {
        if ((rc = read_totals(b, T, st, hc))) return rc;
        return finish_device_levels(b, hc, T, st);
      }
    }
  }
  if ((rc = read_totals(b, T, st, hc))) return rc;
  if (hc[C_STATUS]) return fail_status(hc[C_STATUS]);
  return CXBWT_OK;
}

// ---- the build in ranges of window-0 key prefixes -------------------------

// A class of suffixes whose window-0 keys share their top `depth` digits
// (`prefix`, ordering bits only), and its size.
struct PrefixClass {
  uint64_t prefix;
  uint32_t depth;
  uint64_t count;
};
// A range: consecutive classes, keys lo..hi (ordering bits, inclusive), the
// rows after `before` suffixes of earlier ranges; its keys agree on their
// first `common` digits.
struct Range {
  uint64_t lo, hi, count, before;
  uint32_t common;
  uint64_t skip = 0;  // a piece of one class of identical suffixes: its first member in read order
  bool piece = false;
};

// Ordering bits of the smallest and largest key with this prefix.
uint64_t class_lo(const PrefixClass &c) { return c.prefix; }
uint64_t class_hi(const PrefixClass &c) {
  if (c.depth >= 8) return c.prefix;
  if (c.depth == 0) return ~7ull;
  return (c.prefix | ((1ull << (64 - 8 * c.depth)) - 1)) & ~7ull;
}

// Counts the next digit of every class in `parents` (all of one depth, at
// most PH_MAX_PREFIXES, ascending) on the device; returns the child classes.
int count_children(const Build &b, const std::vector<PrefixClass> &parents, std::vector<PrefixClass> &children,
                   hipStream_t st) {
  const Buffers &B = b.B;
  const uint32_t np = (uint32_t)parents.size();
  const uint32_t depth = parents[0].depth;
  std::vector<uint64_t> pf(np);
  for (uint32_t i = 0; i < np; ++i) pf[i] = parents[i].prefix;
  std::vector<unsigned long long> cnt((size_t)np * 256);
  int rc;
  if ((rc = fill_u64((uint64_t *)B.ph_counts, (uint64_t)np * 256, 0, st))) return rc;
  CX_CHECK(hipMemcpyAsync(B.ph_prefixes, pf.data(), 8 * np, hipMemcpyHostToDevice, st));
  const uint64_t nrec = ceil_div(b.nb, 16);
  const unsigned grid = (unsigned)std::min<uint64_t>(ceil_div(nrec, BLOCK), 2048);
  const size_t lds = (size_t)np * 256 * 4 + (size_t)np * 8;
  k_prefix_hist<<<grid, BLOCK, lds, st>>>(B.text, b.nb, B.ph_prefixes, np, depth, B.ph_counts);
  CX_LAUNCHED();
  CX_CHECK(hipMemcpyAsync(cnt.data(), B.ph_counts, 8 * cnt.size(), hipMemcpyDeviceToHost, st));
  CX_CHECK(hipStreamSynchronize(st));
  const uint32_t nd = depth == 7 ? 32u : 256u;  // digit 7 is the 5-bit clamped length
  for (uint32_t i = 0; i < np; ++i)
    for (uint32_t v = 0; v < nd; ++v) {
      const uint64_t c = cnt[(size_t)i * 256 + v];
      if (!c) continue;
      const uint64_t bits = depth < 7 ? (uint64_t)v << (56 - 8 * depth) : (uint64_t)v << 3;
      children.push_back(PrefixClass{parents[i].prefix | bits, depth + 1, c});
    }
  return CXBWT_OK;
}

// Section 3.1's partitioning on the device: classes of window-0 key
// prefixes, refined one digit at a time while larger than m, packed in key
// order into ranges of at most m suffixes.  CXBWT_ERANGE when a class of
// identical window-0 keys alone exceeds m.
int plan_ranges(const Build &b, uint64_t m, std::vector<Range> &ranges, hipStream_t st) {
  std::vector<PrefixClass> leaves, todo{PrefixClass{0, 0, b.nb}};
  int rc;
  while (!todo.empty()) {
    // the shallowest classes first, up to PH_MAX_PREFIXES per counting pass
    std::sort(todo.begin(), todo.end(), [](const PrefixClass &x, const PrefixClass &y) {
      return x.depth != y.depth ? x.depth < y.depth : x.prefix < y.prefix;
    });
    size_t k = 1;
    while (k < todo.size() && k < (size_t)PH_MAX_PREFIXES && todo[k].depth == todo[0].depth) ++k;
    const std::vector<PrefixClass> parents(todo.begin(), todo.begin() + k);
    todo.erase(todo.begin(), todo.begin() + k);
    std::vector<PrefixClass> kids;
    if ((rc = count_children(b, parents, kids, st))) return rc;
    for (const PrefixClass &c : kids) {
      if (c.count <= m) leaves.push_back(c);
      else if (c.depth < 8) todo.push_back(c);
      else if (clamp_of(c.prefix) < (uint32_t)W) leaves.push_back(c);  // identical suffixes: cut by read order below
      else return CXBWT_ERANGE;  // equal whole first windows whose order depends on later windows
    }
  }
  std::sort(leaves.begin(), leaves.end(),
            [](const PrefixClass &x, const PrefixClass &y) { return x.prefix < y.prefix; });
  ranges.clear();
  uint64_t before = 0;
  bool open = false;  // the last range takes more classes
  for (const PrefixClass &c : leaves) {
    if (c.count > m) {
      // a class of identical suffixes (one whole first-window key that ends
      // inside the window) above the budget: their order is the read order,
      // so it is cut into pieces of m in that order, each a range of its own
      for (uint64_t k = 0; k < c.count; k += m) {
        Range r{c.prefix, c.prefix, std::min<uint64_t>(m, c.count - k), before, 0};
        r.skip = k;
        r.piece = true;
        ranges.push_back(r);
        before += r.count;
      }
      open = false;
      continue;
    }
    if (!open || ranges.back().count + c.count > m) {
      ranges.push_back(Range{class_lo(c), class_hi(c), 0, before, 0});
      open = true;
    }
    Range &r = ranges.back();
    r.hi = class_hi(c);
    r.count += c.count;
    before += c.count;
  }
  for (Range &r : ranges) {
    uint32_t j = 0;
    while (j < 8 && digit_of(r.lo, (int)j) == digit_of(r.hi, (int)j)) ++j;
    r.common = j;
  }
  return CXBWT_OK;
}

// Lists the suffixes of range `r` into keys0 / hdl0 [0, count), in position
// order.
int list_range(const Build &b, const Range &r, PhaseTimer &T, hipStream_t st) {
  const Buffers &B = b.B;
  const Layout &Lo = b.Lo;
  const uint64_t ntl = ceil_div(b.nb, LIST_TILE);
  const uint64_t nlb = ceil_div(ntl, RANK_BLOCK_WORDS);
  if (ntl + 1 > Lo.n_list_tiles || nlb + 1 > Lo.n_list_blocks || r.count > Lo.sort_cap) return fail_internal("work exceeds a workspace list or scratch area");
  T.begin();
  k_range_count<<<(unsigned)ntl, BLOCK, 0, st>>>(B.text, b.nb, r.lo, r.hi, B.list_tiles);
  CX_LAUNCHED();
  k_count_blocks<<<(unsigned)nlb, BLOCK, 0, st>>>(B.list_tiles, ntl, B.list_blocks);
  CX_LAUNCHED();
  k_rank_top<<<1, BLOCK, 0, st>>>(B.list_blocks, (uint32_t)nlb);
  CX_LAUNCHED();
  k_count_prefix<<<(unsigned)nlb, BLOCK, 0, st>>>(B.list_tiles, ntl, B.list_blocks);
  CX_LAUNCHED();
  k_range_list<<<(unsigned)ntl, BLOCK, 0, st>>>(B.text, b.nb, r.lo, r.hi, B.list_tiles, r.skip, r.count, B.keys0,
                                                 B.hdl0, B.pos64);
  CX_LAUNCHED();
  T.end(PH_GEN);
  return CXBWT_OK;
}

// Level 1 of range `r` as seg (of digit seg.d), and what it makes; *fits
// false, and nothing done, where the scratch is too small for the counts.
int range_level1(const Build &b, const Range &r, const Seg &seg, bool *fits, LevelOut &o, PhaseTimer &T,
                 hipStream_t st) {
  const Buffers &B = b.B;
  const Layout &Lo = b.Lo;
  const uint64_t ntiles = ceil_div(b.nb, RANGE_TILE), ngroups = ceil_div(ntiles, GROUP_TILES);
  *fits = 4 * 256 * ntiles <= Lo.tile_hist_bytes && ngroups <= Lo.max_groups && ntiles <= 0x7FFFFFFFull;
  if (!*fits) return CXBWT_OK;
  int rc;
  const uint32_t tp[2] = {0, (uint32_t)ntiles}, gp[2] = {0, (uint32_t)ngroups};
  CX_CHECK(hipMemcpyAsync(B.segs, &seg, sizeof(Seg), hipMemcpyHostToDevice, st));
  CX_CHECK(hipMemcpyAsync(B.tile_prefix, tp, sizeof(tp), hipMemcpyHostToDevice, st));
  CX_CHECK(hipMemcpyAsync(B.group_prefix, gp, sizeof(gp), hipMemcpyHostToDevice, st));
  if ((rc = fill_u32(B.counters + C_NFINAL, 3, 0, st))) return rc;  // final, chunk and segment counts
  const bool fast = (uint32_t)r.lo == 0 && (uint32_t)r.hi == ~7u && seg.d <= 3;
  T.begin();
  if (fast) k_range_hist<true><<<(unsigned)ntiles, BLOCK, 0, st>>>(B.text, b.nb, r.lo, r.hi, seg.d, B.tile_hist);
  else k_range_hist<false><<<(unsigned)ntiles, BLOCK, 0, st>>>(B.text, b.nb, r.lo, r.hi, seg.d, B.tile_hist);
  CX_LAUNCHED();
  T.end(PH_GEN);
  T.begin();
  k_group_scan<false><<<(unsigned)ngroups, BLOCK, 0, st>>>(B.tile_prefix, B.group_prefix, 1, nullptr, B.tile_hist,
                                                           B.gsum);
  CX_LAUNCHED();
  launch_level_scan(B, 1, (uint32_t)ngroups, b.Ls, 1, st);
  CX_LAUNCHED();
  T.end(PH_SCAN);
  T.begin();
#define CX_RANGE_SCATTER(FAST)                                                                                     \
  k_range_scatter<FAST><<<(unsigned)ntiles, 64 * RANGE_NW, 0, st>>>(B.text, b.nb, r.lo, r.hi, seg.d, B.tile_hist, B.gsum, \
                                                                    B.keys1, B.hdl1, B.pos64)
  if (fast) CX_RANGE_SCATTER(true);
  else CX_RANGE_SCATTER(false);
#undef CX_RANGE_SCATTER
  CX_LAUNCHED();
  T.end(PH_SCATTER);
  g_stats.levels++;
  g_stats.host_levels++;
  g_stats.big_segments++;
  g_stats.level_suffixes += r.count;
  g_stats.level_batches++;
  return read_level(B, o, T, st);
}

// One collection built in ranges of at most m suffixes: the bare
// terminators and text records as for a whole build, the ranges planned
// from prefix counts, then each range listed, sorted (levels and chunks) and
// emitted at its rows; term_pos at the end.
int run_range_build(const uint64_t *packed, const uint64_t *offsets, uint64_t n, uint64_t nb, uint32_t maxlen,
                    uint64_t m, bool wide, uint8_t *bwt, uint64_t *term_pos, unsigned char *ws, hipStream_t st) {
  g_stats = cxbwt_stats{};
  g_last_error[0] = 0;
  PhaseTimer T{st, g_timing != 0, {}};
  Build b;
  const uint64_t one[2] = {0, n};
  build_init(b, packed, offsets, n, nb, maxlen, one, 1, bwt, term_pos, ws, m, wide);
  int rc;
  if ((rc = enqueue_prep(b, b.coll_reads.data(), nullptr, T, st))) return rc;
  if ((rc = enqueue_records(b, T, st))) return rc;
  {  // the offsets are checked on the device before anything is listed
    uint32_t hc[C_COUNT];
    CX_CHECK(hipMemcpyAsync(hc, b.B.counters, sizeof(hc), hipMemcpyDeviceToHost, st));
    CX_CHECK(hipStreamSynchronize(st));
    T.collect();
    if (hc[C_STATUS] & (ST_BAD_OFFSETS | ST_TOO_LONG)) return fail_status(hc[C_STATUS]);
  }
  g_stats.chunk_suffixes = nb;
  std::vector<Range> ranges;
  if (nb) {
    if ((rc = plan_ranges(b, m, ranges, st))) return rc;
  }
  g_stats.ranges = (uint32_t)ranges.size();
  // every range's rows follow the n bare-terminator rows and the earlier ranges
  std::vector<CollMap> cm(ranges.size());
  std::vector<Seg> seg(ranges.size());
  for (size_t i = 0; i < ranges.size(); ++i) {
    cm[i].out_shift = n + ranges[i].before;
    cm[i].row_shift = (int64_t)(n + ranges[i].before);
  }
  for (size_t i = 0; i < ranges.size(); ++i) {
    const Range &r = ranges[i];
    // the row map of this range, in the one collection slot (stream order:
    // after the previous range's kernels have read theirs)
    CX_CHECK(hipMemcpyAsync(b.B.cmap, &cm[i], sizeof(CollMap), hipMemcpyHostToDevice, st));
    const bool small = r.count <= (uint64_t)b.tu.chunk();
    // a range that fits a chunk: one unsplit chunk; else one segment whose
    // keys agree on their first `common` digits
    seg[i] = Seg{0, (uint32_t)r.count, 0, (uint8_t)std::min<uint32_t>(r.common, small ? 6 : 7), 0, 0,
                 (uint8_t)(small ? 1 : 0), 0, 0};
    if (!small && !r.piece) {
      bool fits = false;
      LevelOut o{};
      if ((rc = range_level1(b, r, seg[i], &fits, o, T, st))) return rc;
      if (fits) {
        if ((rc = run_levels(b, o, true, T, st))) return rc;
        continue;
      }
    }
    if ((rc = list_range(b, r, T, st))) return rc;
    if (small) {
      CX_CHECK(hipMemcpyAsync(b.B.chunks, &seg[i], sizeof(Seg), hipMemcpyHostToDevice, st));
      if ((rc = finish_level(b.B, b.Lo, b.tu, nb, b.rmax, b.maxlen, bwt, 1, 0, 0, 0, T, st))) return rc;
      continue;
    }
    CX_CHECK(hipMemcpyAsync(b.B.big_next, &seg[i], sizeof(Seg), hipMemcpyHostToDevice, st));
    LevelOut acc{};
    acc.next_len = r.count;
    acc.next_tiles = ceil_div(r.count, b.tile_len);
    acc.next_groups = ceil_div(acc.next_tiles, GROUP_TILES);
    acc.n_big = 1;
    if ((rc = run_levels(b, acc, false, T, st))) return rc;
  }
  T.begin();
  if ((rc = launch_term(b, st))) return rc;
  T.end(PH_FINAL);
  uint32_t hc[C_COUNT];
  if ((rc = read_totals(b, T, st, hc))) return rc;
  if (hc[C_STATUS]) return fail_status(hc[C_STATUS]);
  return CXBWT_OK;
}

// A build captured once in a hipGraph for fixed sizes and buffers, replayed
// on new contents of the same buffers.
struct GraphPlan {
  Build b;
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
  unsigned char *pinned = nullptr;  // host sources of the captured copies
  uint32_t levels = 0;              // levels scheduled on the device, level 1 included
  cxbwt_stats base{};               // statistics of level 1 (known on the host)
  std::vector<LevelShape> shapes;   // per-level counts of the eager build made at creation
  ~GraphPlan() {
    if (exec) (void)hipGraphExecDestroy(exec);
    if (graph) (void)hipGraphDestroy(graph);
    if (pinned) (void)hipHostFree(pinned);
  }
};

int graph_capture(GraphPlan &P, hipStream_t st) {
  Build &b = P.b;
  PhaseTimer T{st, false, {}};
  // eager build: validates the offsets, learns the collection bases and
  // records every level's counts, which size the captured launches
  int rc;
  if ((rc = enqueue_prep(b, b.coll_reads.data(), nullptr, T, st))) return rc;
  if ((rc = enqueue_records(b, T, st))) return rc;
  if ((rc = plan_level1(b, T, st))) return rc;
  Level1Vectors v;
  v.make(b);
  g_stats = cxbwt_stats{};
  level1_stats(b);
  P.base = g_stats;
  P.shapes.clear();
  {
    ShapeScope record(&P.shapes);
    rc = enqueue_body(b, v.src, 0, T, st);
  }
  uint32_t hc[C_COUNT];
  if (!rc) rc = read_totals(b, T, st, hc);
  if (rc) return rc;
  if (hc[C_STATUS]) return fail_status(hc[C_STATUS]);
  // pinned copies of everything the captured copies read
  const size_t nc1 = (size_t)b.ncoll + 1;
  const size_t nbg = b.big.size(), nsm = b.small.size();
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t at = off;
    off = (off + bytes + 255) & ~(size_t)255;
    return at;
  };
  const size_t o_cr = take(8 * nc1), o_cb = take(8 * nc1), o_cm = take(sizeof(CollMap) * b.ncoll),
               o_bs = take(sizeof(Seg) * nbg), o_btp = take(4 * (nbg + 1)), o_bgp = take(4 * (nbg + 1)),
               o_ss = take(sizeof(Seg) * nsm), o_stp = take(4 * (nsm + 1)), o_sgp = take(4 * (nsm + 1)),
               o_ns = take(4);
  CX_CHECK(hipHostMalloc((void **)&P.pinned, off, hipHostMallocDefault));
  unsigned char *h = P.pinned;
  memcpy(h + o_cr, b.coll_reads.data(), 8 * nc1);
  memcpy(h + o_cb, b.cbase.data(), 8 * nc1);
  if (b.ncoll) memcpy(h + o_cm, b.cm.data(), sizeof(CollMap) * b.ncoll);
  if (nbg) memcpy(h + o_bs, b.big.data(), sizeof(Seg) * nbg);
  memcpy(h + o_btp, v.btp.data(), 4 * (nbg + 1));
  memcpy(h + o_bgp, v.bgp.data(), 4 * (nbg + 1));
  if (nsm) memcpy(h + o_ss, b.small.data(), sizeof(Seg) * nsm);
  memcpy(h + o_stp, v.stp.data(), 4 * (nsm + 1));
  memcpy(h + o_sgp, v.sgp.data(), 4 * (nsm + 1));
  memcpy(h + o_ns, &v.nsmall, 4);
  Level1Src src;
  src.cm = (const CollMap *)(h + o_cm);
  src.big = SegSrc{(const Seg *)(h + o_bs), (const uint32_t *)(h + o_btp), (const uint32_t *)(h + o_bgp),
                   (uint32_t)nbg, v.btp.back(), v.bgp.back()};
  src.small = SegSrc{(const Seg *)(h + o_ss), (const uint32_t *)(h + o_stp), (const uint32_t *)(h + o_sgp),
                     (uint32_t)nsm, v.stp.back(), v.sgp.back()};
  src.nsmall = (const uint32_t *)(h + o_ns);
  // levels by default: enough for any input, and those that are spent on ended
  // suffixes, every other one at most of the first ones.  These are as many as
  // this build took (three where that is the form anyway): past them ended
  // suffixes are not split off.  (1 Mbase of 100-base reads, which takes 3: 32
  // scheduled, 301 us a replay, where 3 take 227.)
  uint32_t ended = ~0u;
  const uint32_t full = most_levels(b.maxlen);
  if (!P.levels || P.levels >= full) {
    ended = std::min(std::max((uint32_t)P.shapes.size(), LISTED_LEVELS), full);
    P.levels = std::max(P.levels, full + ended / 2);
  }
  // capture: every size below is fixed now or read on the device
  CX_CHECK(hipStreamBeginCapture(st, hipStreamCaptureModeThreadLocal));
  rc = enqueue_prep(b, (const uint64_t *)(h + o_cr), (const uint64_t *)(h + o_cb), T, st);
  if (!rc) rc = enqueue_records(b, T, st);
  if (!rc) rc = enqueue_body(b, src, P.levels, T, st, &P.shapes, ended);
  hipGraph_t g = nullptr;
  const hipError_t ec = hipStreamEndCapture(st, &g);
  if (rc) {
    if (g) (void)hipGraphDestroy(g);
    return rc;
  }
  if (ec != hipSuccess || !g) return fail_hip(ec, "graph capture");
  P.graph = g;
  CX_CHECK(hipGraphInstantiate(&P.exec, P.graph, nullptr, nullptr, 0));
  return CXBWT_OK;
}

// After a replay: status, statistics, and the levels left to the host.
int graph_finish(GraphPlan &P, hipStream_t st) {
  PhaseTimer T{st, false, {}};
  g_stats = P.base;
  uint32_t hc[C_COUNT];
  int rc;
  if ((rc = read_totals(P.b, T, st, hc))) return rc;
  return finish_device_levels(P.b, hc, T, st);
}

}  // namespace

struct cxbwt_graph {
  GraphPlan p;
};

// A build started by cxbwt_build_start / cxbwt_build_batch_start: a worker
// thread enqueues it on the caller's stream and waits on that stream between
// levels; the caller waits for the job instead of for the call.
struct cxbwt_job {
  std::thread worker;
  std::atomic<int> done{0};
  int status = CXBWT_OK;
  cxbwt_stats stats{};
  char error[256] = "";
};

namespace {

struct JobArgs {
  const uint64_t *packed, *offsets;
  uint64_t n, nb;
  uint32_t maxlen;
  std::vector<uint64_t> coll_reads;  // copied at the call: the caller's array may go away
  uint8_t *bwt;
  uint64_t *term_pos;
  unsigned char *ws;
  hipStream_t st;
  int device;
  Tuning tu;   // the calling thread's choices at the call
  int timing;
};

void job_main(cxbwt_job *job, JobArgs a) {
  int rc = CXBWT_OK;
  try {
    if (hipSetDevice(a.device) != hipSuccess) {
      rc = CXBWT_EDEVICE;
    } else {
      g_tuning = a.tu;
      g_timing = a.timing;
      rc = run_build(a.packed, a.offsets, a.n, a.nb, a.maxlen, a.coll_reads.data(),
                     (uint32_t)(a.coll_reads.size() - 1), a.bwt, a.term_pos, a.ws, a.st);
      // a failed build may leave work in flight: the job ends when the stream has drained
      if (rc && hipStreamSynchronize(a.st) != hipSuccess) rc = CXBWT_EDEVICE;
    }
  } catch (...) {
    rc = CXBWT_EDEVICE;
    (void)hipStreamSynchronize(a.st);
  }
  job->stats = g_stats;
  job->status = rc;
  memcpy(job->error, g_last_error, sizeof(job->error));
  job->done.store(1, std::memory_order_release);
}

// The choices a started build runs with: opts, or the calling thread's.
bool job_choices(const cxbwt_opts *opts, Tuning &tu, int &timing) {
  if (!opts) {
    tu = g_tuning;
    timing = g_timing;
    return true;
  }
  if (!tuning_ok(opts->tile_items, opts->chunk_items)) return false;
  if (opts->schedule != CXBWT_SCHEDULE_MSD && opts->schedule != CXBWT_SCHEDULE_STRINGWORD) return false;
  tu.tile_items = opts->tile_items;
  tu.chunk_items = opts->chunk_items;
  tu.schedule = opts->schedule;
  timing = opts->timing ? 1 : 0;
  return true;
}

// A blocking build's choices: set for the call, the thread's restored after.
struct ChoiceScope {
  Tuning saved_tu;
  int saved_timing;
  ChoiceScope(const Tuning &tu, int timing) : saved_tu(g_tuning), saved_timing(g_timing) {
    g_tuning = tu;
    g_timing = timing;
  }
  ~ChoiceScope() {
    g_tuning = saved_tu;
    g_timing = saved_timing;
  }
};

int start_job(JobArgs &&a, cxbwt_job **out) {
  if (hipGetDevice(&a.device) != hipSuccess) return CXBWT_EDEVICE;
  cxbwt_job *job = new (std::nothrow) cxbwt_job;
  if (!job) return CXBWT_ENOMEM;
  try {
    job->worker = std::thread(job_main, job, std::move(a));
  } catch (...) {
    delete job;
    return CXBWT_EDEVICE;
  }
  *out = job;
  return CXBWT_OK;
}

}  // namespace

// Workspace of cxbwt_build_noalloc: a fixed array in the code object, one
// copy per device the library runs on, held until the process ends.  Host
// code never passes the array's name to a kernel or a copy (on the host it
// names a stand-in, not device memory): it uses the device address
// hipGetSymbolAddress returns, taken once per device with that device
// current and kept in g_scratch_addr.
static __device__ __align__(256) unsigned char scratch[CXBWT_NOALLOC_WORKSPACE_BYTES];

namespace {
constexpr int SCRATCH_MAX_DEVICES = 64;
std::mutex g_scratch_mu;
unsigned char *g_scratch_addr[SCRATCH_MAX_DEVICES] = {};

// Device address of the current device's copy of `scratch`.
int scratch_address(unsigned char **out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= SCRATCH_MAX_DEVICES) return CXBWT_EDEVICE;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_addr[dev]) {
    void *p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return CXBWT_EDEVICE;
    if (((uintptr_t)p & 255u) != 0) return fail_internal("work exceeds a workspace list or scratch area");
    g_scratch_addr[dev] = (unsigned char *)p;
  }
  *out = g_scratch_addr[dev];
  return CXBWT_OK;
}
}  // namespace

// ---------------------------------------------------------------------------
// C ABI
// ---------------------------------------------------------------------------
extern "C" {

uint64_t cxbwt_packed_words(uint64_t n_bases) { return (n_bases + 31) / 32 + 1; }

int cxbwt_pack(const uint8_t *ascii, uint64_t n_bases, uint64_t *packed, uint32_t *d_status, void *stream) {
  if (n_bases > CXBWT_MAX_RANGE_BASES) return CXBWT_ERANGE;
  if (!packed || (n_bases && !ascii)) return CXBWT_EINVAL;
  hipStream_t st = (hipStream_t)stream;
  const uint64_t nw = cxbwt_packed_words(n_bases);
  if (nw <= PACK_SMALL_WORDS) {
    k_pack_small<<<1, PACK_WG, 0, st>>>(ascii, n_bases, packed, nw, d_status);
    CX_LAUNCHED();
    return CXBWT_OK;
  }
  if (d_status) {
    int rc = fill_u32(d_status, 1, 0, st);
    if (rc) return rc;
  }
  k_pack<<<grid_for(nw, 256), 256, 0, st>>>(ascii, n_bases, packed, nw, d_status);
  CX_LAUNCHED();
  return CXBWT_OK;
}

size_t cxbwt_workspace_bytes(uint64_t n_reads, uint64_t n_bases, uint32_t max_read_len) {
  if (!sizes_ok(n_reads, n_bases, max_read_len)) return 0;
  return (size_t)make_layout(n_reads, n_bases, 1).total;
}

size_t cxbwt_batch_workspace_bytes(uint64_t n_reads, uint64_t n_bases, uint32_t max_read_len, uint32_t n_coll) {
  if (!sizes_ok(n_reads, n_bases, max_read_len) || n_coll == 0 || n_coll > n_reads) return 0;
  return (size_t)make_layout(n_reads, n_bases, n_coll).total;
}

int cxbwt_build(const uint64_t *packed, const uint64_t *offsets, uint64_t n_reads, uint64_t n_bases,
                uint32_t max_read_len, uint8_t *bwt, uint64_t *term_pos, void *workspace, size_t workspace_bytes,
                const cxbwt_opts *opts, void *stream) {
  if (!packed || !offsets || !bwt || !term_pos || !workspace || n_reads == 0) return CXBWT_EINVAL;
  if (!sizes_ok(n_reads, n_bases, max_read_len)) return CXBWT_ERANGE;
  if (workspace_bytes < cxbwt_workspace_bytes(n_reads, n_bases, max_read_len)) return CXBWT_ENOMEM;
  if (((uintptr_t)workspace & 255u) != 0) return CXBWT_EINVAL;
  Tuning tu;
  int timing = 0;
  if (!job_choices(opts, tu, timing)) return CXBWT_EINVAL;
  ChoiceScope scope(tu, timing);
  const uint64_t one[2] = {0, n_reads};
  return guarded((hipStream_t)stream, [&] {
    return run_build(packed, offsets, n_reads, n_bases, max_read_len, one, 1, bwt, term_pos, (unsigned char *)workspace,
                     (hipStream_t)stream);
  });
}

int cxbwt_build_noalloc(const uint64_t *packed, const uint64_t *offsets, uint64_t n_reads, uint64_t n_bases,
                        uint32_t max_read_len, uint8_t *bwt, uint64_t *term_pos, void *stream) {
  if (!packed || !offsets || !bwt || !term_pos || n_reads == 0) return CXBWT_EINVAL;
  if (!sizes_ok(n_reads, n_bases, max_read_len)) return CXBWT_ERANGE;
  if (cxbwt_workspace_bytes(n_reads, n_bases, max_read_len) > CXBWT_NOALLOC_WORKSPACE_BYTES) return CXBWT_ESCRATCH;
  unsigned char *ws = nullptr;
  int rc = scratch_address(&ws);
  if (rc) return rc;
  const uint64_t one[2] = {0, n_reads};
  // no kernel timing here: it would create HIP events
  return guarded((hipStream_t)stream, [&] {
    return run_build(packed, offsets, n_reads, n_bases, max_read_len, one, 1, bwt, term_pos, ws, (hipStream_t)stream,
                     false);
  });
}

size_t cxbwt_range_workspace_bytes(uint64_t n_reads, uint64_t n_bases, uint32_t max_read_len,
                                   uint64_t max_range_suffixes, uint32_t flags) {
  if (!range_sizes_ok(n_reads, n_bases, max_read_len, max_range_suffixes, flags)) return 0;
  return (size_t)make_layout(n_reads, n_bases, 1, max_range_suffixes, range_wide(n_bases, flags)).total;
}

int cxbwt_build_ranges(const uint64_t *packed, const uint64_t *offsets, uint64_t n_reads, uint64_t n_bases,
                       uint32_t max_read_len, uint64_t max_range_suffixes, uint32_t flags, uint8_t *bwt,
                       uint64_t *term_pos, void *workspace, size_t workspace_bytes, void *stream) {
  if (!packed || !offsets || !bwt || !term_pos || !workspace || n_reads == 0 || max_range_suffixes == 0 ||
      (flags & ~(uint32_t)CXBWT_RANGE_WIDE))
    return CXBWT_EINVAL;
  if (!range_sizes_ok(n_reads, n_bases, max_read_len, max_range_suffixes, flags)) return CXBWT_ERANGE;
  if (workspace_bytes < cxbwt_range_workspace_bytes(n_reads, n_bases, max_read_len, max_range_suffixes, flags))
    return CXBWT_ENOMEM;
  if (((uintptr_t)workspace & 255u) != 0) return CXBWT_EINVAL;
  return guarded((hipStream_t)stream, [&] {
    return run_range_build(packed, offsets, n_reads, n_bases, max_read_len, max_range_suffixes,
                           range_wide(n_bases, flags), bwt, term_pos, (unsigned char *)workspace, (hipStream_t)stream);
  });
}

int cxbwt_build_start(const uint64_t *packed, const uint64_t *offsets, uint64_t n_reads, uint64_t n_bases,
                      uint32_t max_read_len, uint8_t *bwt, uint64_t *term_pos, void *workspace,
                      size_t workspace_bytes, const cxbwt_opts *opts, void *stream, cxbwt_job **job) {
  if (!job) return CXBWT_EINVAL;
  *job = nullptr;
  if (!packed || !offsets || !bwt || !term_pos || !workspace || n_reads == 0) return CXBWT_EINVAL;
  if (!sizes_ok(n_reads, n_bases, max_read_len)) return CXBWT_ERANGE;
  if (workspace_bytes < cxbwt_workspace_bytes(n_reads, n_bases, max_read_len)) return CXBWT_ENOMEM;
  if (((uintptr_t)workspace & 255u) != 0) return CXBWT_EINVAL;
  JobArgs a{packed, offsets, n_reads, n_bases, max_read_len, {0, n_reads}, bwt, term_pos,
            (unsigned char *)workspace, (hipStream_t)stream, 0, Tuning{8, 6}, 0};
  if (!job_choices(opts, a.tu, a.timing)) return CXBWT_EINVAL;
  return start_job(std::move(a), job);
}

int cxbwt_build_batch_start(const uint64_t *packed, const uint64_t *offsets, uint64_t n_reads, uint64_t n_bases,
                            uint32_t max_read_len, const uint64_t *coll_reads, uint32_t n_coll, uint8_t *bwt,
                            uint64_t *term_pos, void *workspace, size_t workspace_bytes,
                            const cxbwt_opts *opts, void *stream, cxbwt_job **job) {
  if (!job) return CXBWT_EINVAL;
  *job = nullptr;
  if (!packed || !offsets || !bwt || !term_pos || !workspace || !coll_reads || n_reads == 0 || n_coll == 0)
    return CXBWT_EINVAL;
  if (!sizes_ok(n_reads, n_bases, max_read_len)) return CXBWT_ERANGE;
  if (n_coll > n_reads) return CXBWT_EINVAL;
  if (coll_reads[0] != 0 || coll_reads[n_coll] != n_reads) return CXBWT_EINVAL;
  for (uint32_t c = 0; c < n_coll; ++c)
    if (coll_reads[c + 1] <= coll_reads[c]) return CXBWT_EINVAL;
  if (workspace_bytes < cxbwt_batch_workspace_bytes(n_reads, n_bases, max_read_len, n_coll)) return CXBWT_ENOMEM;
  if (((uintptr_t)workspace & 255u) != 0) return CXBWT_EINVAL;
  return guarded((hipStream_t)stream, [&] {
    JobArgs a{packed, offsets, n_reads, n_bases, max_read_len,
              std::vector<uint64_t>(coll_reads, coll_reads + n_coll + 1), bwt, term_pos,
              (unsigned char *)workspace, (hipStream_t)stream, 0, Tuning{8, 6}, 0};
    if (!job_choices(opts, a.tu, a.timing)) return (int)CXBWT_EINVAL;
    return start_job(std::move(a), job);
  });
}

int cxbwt_job_done(const cxbwt_job *job) { return job && job->done.load(std::memory_order_acquire) ? 1 : 0; }

int cxbwt_job_wait(cxbwt_job *job, cxbwt_stats *stats) {
  if (!job) return CXBWT_EINVAL;
  if (job->worker.joinable()) job->worker.join();
  const int rc = job->status;
  if (stats) *stats = job->stats;
  g_stats = job->stats;  // cxbwt_last_stats and cxbwt_last_error on the waiting thread
  memcpy(g_last_error, job->error, sizeof(g_last_error));
  delete job;
  return rc;
}

int cxbwt_build_batch(const uint64_t *packed, const uint64_t *offsets, uint64_t n_reads, uint64_t n_bases,
                      uint32_t max_read_len, const uint64_t *coll_reads, uint32_t n_coll, uint8_t *bwt,
                      uint64_t *term_pos, void *workspace, size_t workspace_bytes, const cxbwt_opts *opts,
                      void *stream) {
  if (!packed || !offsets || !bwt || !term_pos || !workspace || !coll_reads || n_reads == 0 || n_coll == 0)
    return CXBWT_EINVAL;
  if (!sizes_ok(n_reads, n_bases, max_read_len)) return CXBWT_ERANGE;
  if (n_coll > n_reads) return CXBWT_EINVAL;
  if (coll_reads[0] != 0 || coll_reads[n_coll] != n_reads) return CXBWT_EINVAL;
  for (uint32_t c = 0; c < n_coll; ++c)
    if (coll_reads[c + 1] <= coll_reads[c]) return CXBWT_EINVAL;  // every collection holds a read
  if (workspace_bytes < cxbwt_batch_workspace_bytes(n_reads, n_bases, max_read_len, n_coll)) return CXBWT_ENOMEM;
  if (((uintptr_t)workspace & 255u) != 0) return CXBWT_EINVAL;
  Tuning tu;
  int timing = 0;
  if (!job_choices(opts, tu, timing)) return CXBWT_EINVAL;
  ChoiceScope scope(tu, timing);
  return guarded((hipStream_t)stream, [&] {
    return run_build(packed, offsets, n_reads, n_bases, max_read_len, coll_reads, n_coll, bwt, term_pos,
                     (unsigned char *)workspace, (hipStream_t)stream);
  });
}

int cxbwt_graph_create(const uint64_t *packed, const uint64_t *offsets, uint64_t n_reads, uint64_t n_bases,
                       uint32_t max_read_len, const uint64_t *coll_reads, uint32_t n_coll, uint8_t *bwt,
                       uint64_t *term_pos, void *workspace, size_t workspace_bytes, uint32_t levels, void *stream,
                       cxbwt_graph **out) {
  if (!out) return CXBWT_EINVAL;
  *out = nullptr;
  if (!packed || !offsets || !bwt || !term_pos || !workspace || n_reads == 0 || n_coll == 0) return CXBWT_EINVAL;
  if (!sizes_ok(n_reads, n_bases, max_read_len)) return CXBWT_ERANGE;
  const uint64_t one[2] = {0, n_reads};
  if (!coll_reads) {
    if (n_coll != 1) return CXBWT_EINVAL;
    coll_reads = one;
  }
  if (n_coll > n_reads || coll_reads[0] != 0 || coll_reads[n_coll] != n_reads) return CXBWT_EINVAL;
  for (uint32_t c = 0; c < n_coll; ++c)
    if (coll_reads[c + 1] <= coll_reads[c]) return CXBWT_EINVAL;
  if (workspace_bytes < cxbwt_batch_workspace_bytes(n_reads, n_bases, max_read_len, n_coll)) return CXBWT_ENOMEM;
  if (((uintptr_t)workspace & 255u) != 0) return CXBWT_EINVAL;
  cxbwt_graph *g = new (std::nothrow) cxbwt_graph;
  if (!g) return CXBWT_ENOMEM;
  g->p.levels = levels;
  // the eager pass runs on the caller's stream; the capture on a stream of
  // its own (a capture needs a non-default stream)
  hipStream_t cs = nullptr;
  int rc = CXBWT_OK;
  if (hipStreamCreateWithFlags(&cs, hipStreamNonBlocking) != hipSuccess) rc = CXBWT_EDEVICE;
  if (!rc && hipStreamSynchronize((hipStream_t)stream) != hipSuccess) rc = CXBWT_EDEVICE;
  if (!rc)
    rc = guarded(cs, [&] {
      build_init(g->p.b, packed, offsets, n_reads, n_bases, max_read_len, coll_reads, n_coll, bwt, term_pos,
                 (unsigned char *)workspace);
      return graph_capture(g->p, cs);
    });
  if (cs) (void)hipStreamDestroy(cs);
  if (rc) {
    delete g;
    return rc;
  }
  *out = g;
  return CXBWT_OK;
}

int cxbwt_graph_launch(cxbwt_graph *g, void *stream) {
  if (!g || !g->p.exec) return CXBWT_EINVAL;
  return hipGraphLaunch(g->p.exec, (hipStream_t)stream) == hipSuccess ? CXBWT_OK : CXBWT_EDEVICE;
}

int cxbwt_graph_finish(cxbwt_graph *g, void *stream) {
  if (!g || !g->p.exec) return CXBWT_EINVAL;
  return guarded((hipStream_t)stream, [&] { return graph_finish(g->p, (hipStream_t)stream); });
}

void cxbwt_graph_destroy(cxbwt_graph *g) { delete g; }

int cxbwt_last_stats(cxbwt_stats *out) {
  if (!out) return CXBWT_EINVAL;
  *out = g_stats;
  return CXBWT_OK;
}

int cxbwt_set_tuning(uint32_t tile_items, uint32_t chunk_items) {
  if (!tuning_ok(tile_items, chunk_items)) return CXBWT_EINVAL;
  g_tuning.tile_items = tile_items;
  g_tuning.chunk_items = chunk_items;
  return CXBWT_OK;
}

int cxbwt_set_schedule(uint32_t schedule) {
  if (schedule != CXBWT_SCHEDULE_MSD && schedule != CXBWT_SCHEDULE_STRINGWORD) return CXBWT_EINVAL;
  g_tuning.schedule = schedule;
  return CXBWT_OK;
}

int cxbwt_get_schedule(uint32_t *schedule) {
  if (!schedule) return CXBWT_EINVAL;
  *schedule = g_tuning.schedule;
  return CXBWT_OK;
}

int cxbwt_get_tuning(uint32_t *tile_items, uint32_t *chunk_items) {
  if (!tile_items || !chunk_items) return CXBWT_EINVAL;
  *tile_items = g_tuning.tile_items;
  *chunk_items = g_tuning.chunk_items;
  return CXBWT_OK;
}

int cxbwt_build_tuning(uint64_t n_sort, uint32_t n_coll, uint32_t *tile_items, uint32_t *chunk_items) {
  if (!n_coll || !tile_items || !chunk_items) return CXBWT_EINVAL;
  const Tuning t = tuning_for(g_tuning, n_sort, n_coll);
  *tile_items = t.tile_items;
  *chunk_items = t.chunk_items;
  return CXBWT_OK;
}

int cxbwt_set_timing(int enable) {
  const int prev = g_timing;
  g_timing = enable ? 1 : 0;
  return prev;
}

const char *cxbwt_last_error(void) { return g_last_error; }

const char *cxbwt_status_str(int status) {
  switch (status) {
    case CXBWT_OK: return "ok";
    case CXBWT_EINVAL: return "invalid argument (null pointer or inconsistent sizes)";
    case CXBWT_ERANGE: return "size out of the supported range";
    case CXBWT_ENOMEM: return "workspace smaller than cxbwt_workspace_bytes()";
    case CXBWT_EDEVICE: return "HIP launch/runtime failure or internal device check failed";
    case CXBWT_EDATA: return "invalid input data found on the device (offsets, read length or bases)";
    case CXBWT_ESCRATCH:
      return "input needs more workspace than cxbwt_build_noalloc's fixed device array holds "
             "(CXBWT_NOALLOC_WORKSPACE_BYTES); use cxbwt_build with a caller workspace";
    default: return "unknown status";
  }
}

}  // extern "C"
