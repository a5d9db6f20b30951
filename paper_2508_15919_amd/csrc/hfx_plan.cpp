// Host planner: turns the scheduler's statement of a step (HFX Section 3.3.1: which requests
// run and how many new tokens each contributes) into the batch descriptor one persistent launch
// drains.  Integer work only; no device calls in this file.
#include "hfx_plan.h"

#include <algorithm>
#include <cmath>
#include <cstring>

namespace hfx {

// Relative cost model, in nanoseconds of one resident workgroup when the whole chip runs that
// kind of work: decode streams KV bytes (about 6 TB/s over HFX_PLAN_WGS workgroups), prefill
// does MFMA flops (about 1 PFLOP/s over HFX_PLAN_WGS workgroups).  Only ratios matter: they
// order the queue and size the splits.
static const double kDecodeBytesPerNs = 12.0;
static const double kPrefillFlopsPerNs = 2000.0;
static const double kPrefillFlopsPerNs64 = 1400.0;   // 64-wide heads: twice the exponentials per MFMA
static const double kMinItemNs = 32000.0;
static const double kItemNs = 3000.0;      // of a prefill item, besides its keys
static const int kMinDecodeTokens = 128;
static const int kMinPrefillKeys = 256;
static const int kMaxSplits = 64;
static const int kDecodeItemsPerWg = 4;    // decode partials are small (rows of D + 2 floats per q-head)
// Which prefill-dominated steps have their items laid out die by die (see the queue order in plan_step), by items per
// workgroup of the planning width and by the time of the step.  What it buys is HBM traffic: 0.6 instead of 1.06 GB on the
// prefill-heavy mixed step, in the same time (822 us, one queue 826).  The lines were drawn when the counters shared a cache line, which cost such a step 40 to
// 80 us.  With the present counters, over one queue for all and, second, over the order table that queue_per_die would make of the same steps: 14 steps of one to six
// prompts of the first kind 0.999 (0.985 to 1.02) and 1.002; 14 of the second, more than 1 GB of keys (the last-level cache holds 256 MB), each read by two items
// or more, in long items (kMinItemNs, by the (row, key) pairs they work on), 1.049 (1.005 to 1.3) and 0.998 (105 chunks of 64 rows behind 8500 to 34009 on 64-wide 24/8 heads
// 1586 us, 1631 and 1587); 14 of the third kind, below, 1.236 and 1.000.  So the order table would do as well in all three.
static const int kClassRoundsMin = 4;
static const double kClassStepNs = 800000.0;
static const double kClassStreamBytes = 1e9;
// Steps of requests with one row tile of few rows behind long contexts are another matter.  Where several head
// blocks read the same keys, each on a die of its own, the step lasts as long as the blocks take to stream them apart
// (apart_ns), unless the tiles keep the matrix cores busy for about as long (beside_ns): 134 chunks of 2 rows behind 5734 to
// 22937 tokens on 24/8 heads 2422 us from one queue, 1950 with classes and with an order table; 97 of one row behind 12208, 1489, 1221 and 1224.  The ratio is
// 1.9 with one busy wavefront of four, 1.65 with two, 1.3 with four, where two head blocks still find each other's keys in
// the cache.  Below three rounds and about 2100 keys an item queue_per_die takes over.
static const int kClassRoundsMinApart = 3;
static const double kClassApart = 1.5;
static const double kClassItemNsApart = 70000.0;
static const double kLongStepNs = 400000.0; // steps of less time than this are cut by trying what the cut leads to ...
// Time of an item alone on its CU over its time beside another, steps of 256 equal items over steps of 512: 0.54 to 0.55 behind 2048 to
// 16384 earlier tokens, 0.59 behind 1024, 0.65 behind 512; on 64-wide heads 0.58 to 0.63, 0.69 and 0.75.  (Counted in clocks of the stage loop it
// is 0.68 to 0.73, but the clock falls when all CUs have two.)
static const double kLoneShare = 0.575;
static const int64_t kCutMaxTiles = 8192;   // ... if they have no more row tiles (the host time of the trial)
static const int kClassRoundsMax = 8;
static const int kFitRounds = 6;           // steps with fewer rounds of prefill items than this get whole rounds
static const int kPrefillItemsPerWg = 2;   // prefill partials are 128 rows: split only where balance needs it
static const uint32_t kNoUnit = 0x0fffffffu;   // items that share keys with no other item

static int kv_heads_per_item(int Hkv) { return (Hkv % 4 == 0) ? 4 : (Hkv % 2 == 0 ? 2 : 1); }
static int q_heads_per_item(int G) { return (G % 4 == 0) ? 4 : (G % 2 == 0 ? 2 : 1); }

hfx_status check_shape(const hfx_shape* s) {
  if (!s) return HFX_ERR_NULL;
  if (s->num_q_heads <= 0 || s->num_kv_heads <= 0) return HFX_ERR_SHAPE;
  if (s->num_q_heads % s->num_kv_heads != 0) return HFX_ERR_SHAPE;
  if (s->num_q_heads / s->num_kv_heads > 16) return HFX_ERR_SHAPE;
  if (s->num_kv_heads > 2 && s->num_kv_heads % 4 != 0) return HFX_ERR_SHAPE;
  if (s->head_dim != 64 && s->head_dim != 128) return HFX_ERR_SHAPE;
  if (s->page_size != HFX_PAGE) return HFX_ERR_SHAPE;
  if (s->num_pages < 1) return HFX_ERR_SHAPE;
  if (!(s->softmax_scale == s->softmax_scale)) return HFX_ERR_SHAPE;
  return HFX_OK;
}

// visible (row, key) pairs of chunk rows [r0, r1) against keys [kb, ke); row i sees keys <= p+i.
// Rows below i_lo see nothing of the range, rows from i_hi on see all of it, the rows between
// see p+i+1-kb keys (an arithmetic series).
static int64_t pairs_in(int64_t p, int64_t r0, int64_t r1, int64_t kb, int64_t ke) {
  if (ke <= kb || r1 <= r0) return 0;
  const int64_t i_lo = std::min(r1, std::max(r0, kb - p));
  const int64_t i_hi = std::min(r1, std::max(i_lo, ke - p - 1));
  const int64_t n = i_hi - i_lo;
  return n * (p + 1 - kb) + (i_lo + i_hi - 1) * n / 2 + (r1 - i_hi) * (ke - kb);
}

// Time of a row tile that sees `keys` keys.  What counts is the time a workgroup spends, which is that of
// four full wavefronts however few rows the tile has.  Cuts and the queue go by it alike: the ragged last tile
// of a prompt sees the most keys and has to start first.  (Ordered by the (row, key) pairs of the tile it started
// among the last: 2500 tokens 74 us instead of 55, 4097 tokens 155 instead of 126; 45 steps of one to four prompts of 32 k + 1..5 tokens took 1.16
// times as long on average with the prefill loop before its whole pairs, up to 1.48.)
static double tile_ns(int D, int64_t keys) {
  return 4.0 * D * 4 * HFX_WAVE_ROWS * (double)keys / (D == 64 ? kPrefillFlopsPerNs64 : kPrefillFlopsPerNs);
}

// Share of a row tile's four wavefronts that have rows to work on: `rows` chunk rows of hpw q-heads, a wavefront 32 rows
// of one head.
static double tile_busy(int hpw, int64_t rows) {
  return 0.25 * hpw * (double)((rows + HFX_WAVE_ROWS - 1) / HFX_WAVE_ROWS);
}

// How the kmax keys a row tile of ns_all sees are cut into items of at most about cap_ns each: nsplit pieces
// of tiles_per key tiles (the last may be shorter).
static void prefill_splits(int64_t kmax, double ns_all, double cap_ns, int64_t* nsplit_out, int64_t* tiles_per_out) {
  const int64_t ntiles = (kmax + HFX_KEY_TILE - 1) / HFX_KEY_TILE;
  if (ns_all <= cap_ns) {             // most tiles, without a division
    *nsplit_out = 1;
    *tiles_per_out = std::max<int64_t>(ntiles, kMinPrefillKeys / HFX_KEY_TILE);
    return;
  }
  int64_t nsplit = (int64_t)std::min(std::ceil(ns_all / cap_ns), (double)kMaxSplits);
  nsplit = std::max<int64_t>(1, nsplit);
  int64_t tiles_per = (ntiles + nsplit - 1) / nsplit;
  tiles_per = std::max<int64_t>(tiles_per, kMinPrefillKeys / HFX_KEY_TILE);
  *nsplit_out = (ntiles + tiles_per - 1) / tiles_per;
  *tiles_per_out = tiles_per;
}

static int32_t clamp_cost(double ns) {
  if (ns < 1.0) return 1;
  if (ns > 2.0e9) return 2000000000;
  return (int32_t)ns;
}

// Sorts positive floats, largest first: their bit patterns order like the values.  Four passes of 8 bits.
static void sort_descending(std::vector<float>& v, std::vector<float>& scratch) {
  scratch.resize(v.size());
  const size_t n = v.size();
  float* a = v.data();
  float* b = scratch.data();
  uint32_t count[4][256];
  std::memset(count, 0, sizeof count);
  auto bits = [](float x) {
    uint32_t u;
    std::memcpy(&u, &x, sizeof u);
    return ~u;
  };
  for (size_t i = 0; i < n; ++i) {
    const uint32_t u = bits(a[i]);
    for (int pass = 0; pass < 4; ++pass) ++count[pass][(u >> (8 * pass)) & 255u];
  }
  for (int pass = 0; pass < 4; ++pass) {
    const int shift = 8 * pass;
    uint32_t* c = count[pass];
    if (n == 0 || c[(bits(a[0]) >> shift) & 255u] == n) continue;      // all alike in these bits
    uint32_t at = 0;
    for (int d = 0; d < 256; ++d) {
      const uint32_t k = c[d];
      c[d] = at;
      at += k;
    }
    for (size_t i = 0; i < n; ++i) b[c[(bits(a[i]) >> shift) & 255u]++] = a[i];
    std::swap(a, b);
  }
  if (a != v.data()) v.swap(scratch);
}

// When the last bin ends that items of `cost` * `scale` (sorted, largest first; each comes `copies` times) keep busy, if every
// item goes to the least loaded bin.  Beyond two rounds the placing is left out for its bound, if not asked for (exact): an
// item starts no later than when the items before it, perfectly spread, are done.  Beyond eight rounds all but the last
// four are taken as perfectly spread.
static double last_end(const std::vector<float>& cost, int copies, float scale, size_t bins, bool exact, std::vector<float>& load) {
  const size_t n = cost.size() * (size_t)copies;
  double end = 0.0;
  if (!exact && n > 2 * bins && n > 1024) {
    double before = 0.0;
    for (const float c : cost) {
      end = std::max(end, before + (double)c * (double)(copies - 1) / (double)bins + c);
      before += (double)c * copies / (double)bins;
    }
    return end * scale;
  }
  load.assign(bins, 0.f);         // from the point on where all bins have an item: a heap, least loaded on top
  size_t first = 0;
  if (n > 8 * bins) {
    first = (n / bins - 4) * bins;
    double before = 0.0;
    for (size_t i = 0; i < first / (size_t)copies; ++i) before += cost[i];
    load.assign(bins, (float)(before * copies * scale / (double)bins));
  }
  for (size_t i = first; i < n; ++i) {
    const float c = scale * cost[i / (size_t)copies];
    if (i < bins) {               // the first of each bin; they descend, so the reverse order is a heap
      load[bins - 1 - i] = c;
      continue;
    }
    const float x = load[0] + c;
    size_t at = 0;
    for (;;) {
      size_t child = 2 * at + 1;
      if (child >= bins) break;
      if (child + 1 < bins && load[child + 1] < load[child]) ++child;
      if (load[child] >= x) break;
      load[at] = load[child];
      at = child;
    }
    load[at] = x;
  }
  for (const float x : load) end = std::max(end, (double)x);
  return end;
}

// The cap on an item's time by which the row tiles of a step are cut along the keys.  Tiles come `mult` at
// a time, one per head block, all alike.  `share` is the step's time when perfectly spread; no cap is
// smaller than about half of it.  What the cut needs of workspace is bounded afterwards (cap_within_workspace).
//
// In a decode-dominated step the prefill items run beside the decode stream on CUs of their own (see the
// queue order in plan_step) and only have to be done when it is: pieces of up to 0.75 of a share save
// partials and merge work (64 decodes and two chunks of 512: 108 us at 0.6, where the later chunk's tiles
// are cut in two, 99 at 0.75, where they are not).
//
// Prefill-dominated steps:
// In short steps the cap is chosen by what it leads to: largest first, items go to where there is the least
// work, an item alone on its CU runs at 1.74 times its rate, and every cut adds partials (64 KB a piece,
// written and read: 26 ns) and the merge launch (4 us).  Not cutting at all is the common answer: whole tiles
// fill the CUs (1500 tokens on 32/8 heads: 33.6 us cut at half a share, 27.8 whole; 2500 tokens 77 and 57; 4096 tokens 149 and
// 126; 1000 behind 3000 beside 16 decodes 95 and 79).  Cuts pay where there are fewer tiles than CUs (128 tokens behind
// 8000: 94 us whole, 36 in 4 pieces, 30 in 8, 42 in 9; 8 chunks of one row behind 4000: 57 whole, 33 in 4) and where a few tiles
// outlast the rest (300 behind 5000 and 200 behind 6000: 83 and 63).  The estimate dates from a slower loop, so that the line lies
// a little early: 8 chunks of one row behind 1000 take 18.2 in 3 pieces and 16.8 whole (20.6 and 21.6 with that loop).
// Tiles of few rows in layouts of few q-heads per kv-head leave wavefronts without rows.  Where all such tiles start at
// once, whole, they slow their neighbours on the CU the less; and no cut makes a step shorter than its keys take to
// stream from memory (stream_ns, once per kv-head).  36 chunks of 4 rows behind 17273 on 8/8 heads: 468 us whole, 489 in
// three pieces each; 42 behind 5321 on 8/8 heads of 64 90 and 112 in four.  (Several head blocks that share their keys on a die are no longer bound by that stream:
// 23 behind 8015 on 12/4 heads, 166 and 178 when they did not, take 141 whole and 131 in three pieces, which the estimate does not see.)
// Long steps are cut by half a share of the step and then into whole rounds: a step of few, about equally
// expensive items per workgroup lasts a whole number of items, so a partly filled last round is closed by
// raising the cap by up to a half.
//
// Planning has to stay short next to the step: a trial is a pass over the row tiles, a radix sort and, up to two rounds or in
// long steps, the placing itself (last_end).  With a general sort and heap, 120 prompt chunks on 8/1 heads (8000 items; tiles of one
// kv-head are all different) took 1390 us to plan, 390 without any trial; 500 so.
static const double kWhole = 1e18;
static double prefill_cap(const int32_t* kind, const int32_t* q_len, const int32_t* ctx_len, int R, int mult, int D,
                          int hpw, int rows_wg, double dec_ns, double stream_ns, bool decode_dominated, Plan* P) {
  std::vector<float>& cost = P->cut_cost;
  double longest = 0.0, sum = 0.0, piece = 0.0;     // of the tiles; time of the longest item
  int64_t pieces = 0;          // of tiles that are cut
  bool idle_waves = false;     // count the wavefronts that have rows
  auto cut = [&](double cap, bool list) {      // returns the number of items
    int64_t count = 0;
    cost.clear();
    sum = piece = 0.0;
    pieces = 0;
    for (int r = 0; r < R; ++r) {
      if (kind[r] != HFX_PREFILL) continue;
      const int64_t p = ctx_len[r] - q_len[r];
      const int n_rt = (q_len[r] + rows_wg - 1) / rows_wg;
      for (int rt = 0; rt < n_rt; ++rt) {
        const int64_t r1 = std::min<int64_t>(q_len[r], (int64_t)(rt + 1) * rows_wg);
        int64_t nsplit, tiles_per;
        const double ns = tile_ns(D, p + r1);
        prefill_splits(p + r1, ns, cap, &nsplit, &tiles_per);
        longest = std::max(longest, ns);
        sum += ns * mult;
        count += nsplit * mult;
        if (nsplit > 1) pieces += nsplit * mult;
        if (list) {
          const double one = ns / (double)nsplit + kItemNs;
          const double busy = idle_waves ? tile_busy(hpw, r1 - (int64_t)rt * rows_wg) : 1.0;
          piece = std::max(piece, one);
          cost.insert(cost.end(), (size_t)nsplit, (float)(one * (kLoneShare + (1.0 - kLoneShare) * busy)));
        }
      }
    }
    return count;
  };
  const int64_t whole_tiles = cut(kWhole, false);
  const double share = (sum + dec_ns) / HFX_PLAN_WGS;
  const double least = std::max(share, (dec_ns + stream_ns) / HFX_PLAN_WGS);
  double cap = std::max(share / kPrefillItemsPerWg, kMinItemNs);
  if (decode_dominated) return std::max(cap, 0.75 * share);
  if (longest <= cap || whole_tiles > kCutMaxTiles) return cap;
  // The time a cap leads to.  Workgroups and CUs are taken in sets that get the same items: as many as the
  // common divisor of their number and `mult`.
  int set = 1;
  while (mult % (2 * set) == 0 && 2 * set <= HFX_PLAN_WGS / 2) set *= 2;
  const double merge_ns = 4000.0, piece_ns = 26.0 * (D / 128.0);
  // In a long step the bound of last_end, in the place of either side of its one comparison, would cut, and take workspace
  // for it, where whole tiles are as good.
  const bool exact = share >= kLongStepNs;
  auto time_of = [&](double cap, double limit) {      // ... or `limit`, if it is no less
    const bool queue = cut(cap, true) > HFX_PLAN_WGS;
    const double extra = pieces > 0 ? merge_ns + piece_ns * (double)pieces : 0.0;
    if (least + extra >= limit) return limit;
    sort_descending(cost, P->cut_sort);
    // up to one round: a CU's workgroups get items that fit; more: workgroups come back for the next item
    const size_t bins = (size_t)(HFX_PLAN_WGS / (queue ? 1 : 2) / set);
    double t = std::max(last_end(cost, mult / set, queue ? 1.f : 0.5f, bins, exact, P->cut_load), least);
    if (queue) t = least + kLoneShare * (t - least);       // what is left at the end has its CU to itself
    else t = std::max(t, kLoneShare * piece);
    return std::min(t + extra, limit);
  };
  idle_waves = whole_tiles <= HFX_PLAN_WGS;
  double best_cap = kWhole, best = time_of(best_cap, kWhole);
  idle_waves = false;
  if (share < kLongStepNs) {
    for (const double f : {2.1, 1.45, 1.0, 0.7, 0.52}) {
      const double c = std::max(f * share, 0.5 * kMinItemNs);
      if (c >= longest) continue;
      const double limit = 0.9 * best;
      if (least + merge_ns >= limit) break;
      const double t = time_of(c, limit);
      // a cut has to promise a tenth, which is about what the estimate is worth, and costs workspace
      // (the fixed workspace keeps room for the partials, and a quarter of it for those of decodes)
      if (t < limit && (double)pieces * 4 * HFX_WAVE_ROWS * (4.0 * D + 8.0) <= 0.75 * HFX_STATIC_WS_BYTES) {
        best = t;
        best_cap = c;
      }
      if (c <= 0.5 * kMinItemNs) break;
    }
    return best_cap;
  }
  const int64_t n0 = cut(cap, false), whole = n0 / HFX_PLAN_WGS * HFX_PLAN_WGS;
  if (whole >= HFX_PLAN_WGS && n0 > whole && n0 < (int64_t)kFitRounds * HFX_PLAN_WGS && cut(1.5 * cap, false) <= whole) {
    double lo = cap, hi = 1.5 * cap;
    for (int it = 0; it < 12; ++it) {
      const double mid = 0.5 * (lo + hi);
      (cut(mid, false) <= whole ? hi : lo) = mid;
    }
    cap = hi;
  }
  return best <= time_of(cap, best) ? best_cap : cap;
}

// Partial rows of a cut of the step's row tiles by cap: 4 * HFX_WAVE_ROWS for every piece of a tile that is cut.
// tile_time(p, r0, r1) is the time of the tile of chunk rows [r0, r1) behind p earlier tokens.
template <typename F>
static int64_t cut_rows(const int32_t* kind, const int32_t* q_len, const int32_t* ctx_len, int R, int mult, int rows_wg,
                        double cap, F tile_time, int64_t* n_items = nullptr) {
  int64_t pieces = 0, count = 0;
  for (int r = 0; r < R; ++r) {
    if (kind[r] != HFX_PREFILL) continue;
    const int64_t p = ctx_len[r] - q_len[r];
    for (int64_t r0 = 0; r0 < q_len[r]; r0 += rows_wg) {
      const int64_t r1 = std::min<int64_t>(q_len[r], r0 + rows_wg);
      int64_t nsplit, tiles_per;
      prefill_splits(p + r1, tile_time(p, r0, r1), cap, &nsplit, &tiles_per);
      count += nsplit * mult;
      if (nsplit > 1) pieces += nsplit * mult;
    }
  }
  if (n_items) *n_items = count;
  return pieces * 4 * HFX_WAVE_ROWS;
}

// A cap >= `cap` whose partial rows, with the dec_rows of the decode items, stay inside the fixed workspace
// (HFX_STATIC_WS_BYTES): a caller that has no other must not be refused because tiles of few rows, which take the time of
// full ones, are cut like full ones and write as many partial rows.  More than the fixed workspace is taken only
// where the work itself asks for it: as many rows as half a share of the step, counted in visible
// (row, key) pairs, cuts the tiles into, in whole rounds.  (A 4096-token chunk behind 61440 on one kv-head: 72 MB,
// two rounds of equal pieces.  40 chunks of 40 rows behind 19960 tokens beside four of 2048, with the prefill loop before its whole
// pairs: 85 MB and 1349 us by time, 64 MB by pairs, 43 MB and 1264 us so bounded; 1186 us now, 1163 uncut.)
static double cap_within_workspace(const int32_t* kind, const int32_t* q_len, const int32_t* ctx_len, int R, int mult, int D,
                                   int hpw, int rows_wg, double dec_ns, double pre_ns, int64_t dec_rows, double cap) {
  auto by_pairs = [&](int64_t p, int64_t r0, int64_t r1) {
    return 4.0 * D * hpw * (double)pairs_in(p, r0, r1, 0, p + r1) / kPrefillFlopsPerNs;
  };
  auto by_time = [&](int64_t p, int64_t, int64_t r1) { return tile_ns(D, p + r1); };
  const double total = dec_ns + pre_ns;
  double pair_cap = std::max(total / (HFX_PLAN_WGS * kPrefillItemsPerWg), kMinItemNs);
  if (dec_ns > pre_ns) pair_cap = std::max(pair_cap, 0.6 * total / HFX_PLAN_WGS);
  int64_t n = 0;
  int64_t pair_rows = cut_rows(kind, q_len, ctx_len, R, mult, rows_wg, pair_cap, by_pairs, &n);
  const int64_t whole = n / HFX_PLAN_WGS * HFX_PLAN_WGS;
  if (pre_ns > dec_ns && whole >= HFX_PLAN_WGS && n > whole && n < (int64_t)kFitRounds * HFX_PLAN_WGS) {
    double lo = pair_cap, hi = 1.5 * pair_cap;
    cut_rows(kind, q_len, ctx_len, R, mult, rows_wg, hi, by_pairs, &n);
    for (int it = 0; it < 12 && n <= whole; ++it) {
      const double mid = 0.5 * (lo + hi);
      int64_t n_mid = 0;
      cut_rows(kind, q_len, ctx_len, R, mult, rows_wg, mid, by_pairs, &n_mid);
      (n_mid <= whole ? hi : lo) = mid;
    }
    if (n <= whole) pair_rows = cut_rows(kind, q_len, ctx_len, R, mult, rows_wg, hi, by_pairs);
  }
  const int64_t fixed_rows = (int64_t)((HFX_STATIC_WS_BYTES - 512) / (4 * D + 8));     // 512: both parts start on 256 bytes
  const int64_t allowed = std::max(fixed_rows - dec_rows, pair_rows);
  double longest = 0.0;
  for (int r = 0; r < R; ++r)
    if (kind[r] == HFX_PREFILL) longest = std::max(longest, tile_ns(D, ctx_len[r]));
  double lo = cap, hi = std::max(cap, longest);        // uncut tiles need no partials
  if (cut_rows(kind, q_len, ctx_len, R, mult, rows_wg, cap, by_time) <= allowed) return cap;
  for (int it = 0; it < 20; ++it) {
    const double mid = 0.5 * (lo + hi);
    (cut_rows(kind, q_len, ctx_len, R, mult, rows_wg, mid, by_time) <= allowed ? hi : lo) = mid;
  }
  return hi;
}

// How the contexts of decode requests are cut: kv-heads of an item, and tokens of a piece at most.
struct DecodeCut {
  int heads;
  int64_t tokens;
};

// By default an item has up to four kv-heads, one for each wavefront, and takes about cap_ns.  Steps whose items all have a place on the
// chip at once do better with fewer heads an item: its wavefronts then walk a quarter or half of the pages each, so that pieces
// can be longer and partials fewer, or there is nothing to merge.  `n_pre`: prefill items of the step.
// Decodes alone take up to two items a CU (all on 32/8 heads of 128 unless named): 4 of 100 to 2000 tokens 12.4 us by default, 10.4 so;
// 12 of 200 to 400 11.3 and 7.5; 16 of 2000 29.5 and 25.3; 64 of 1000 53.9 and 49.7; 128 of 500 to 2000 133 and 118 (two heads);
// 100 of 500 to 5000 on 64-wide heads 115 and 108; 8 of 20000 to 60000 on one kv-head 32.4 and 31.6; at worst 64 of 1000 to 4000 there,
// 18.3 and 18.9.  A context is left whole if that saves the merge launch (3.3 us) for at most 1024 more tokens of one head (4 us): 500 tokens
// 10.1 us in pieces, 7.9 whole; with 2048 more, the 4 decodes above 14.0.  Pieces have 256 tokens of one head at least (128, 512: the same within
// 3 % where they differ).
// Beside prefill items decodes keep to CUs of their own, or the longer piece beside a prefill item ends last, and to pieces no
// longer than the default: 3 of 200 to 900 beside a prompt of 100 10.6 us and 8.3; where up to 512 items were allowed, 6 of 500 to 5000 beside 777
// 23.0 and 26.2, and 10 of 200 to 3000 on 8/8 heads beside 192 rows 15.1 and 16.8 (14.8 so); with longer pieces the first of these 32.2.
//
// Beside prefill items that a decode stream outweighs, a step of up to kRoundsOver times the 1024 items of two rounds has its pieces
// lengthened to that, if pieces four times as long are enough: all items are then dealt, and no round has a few items in it.  150 steps of 1.0 to
// 2.0 times 1024 items on seven head layouts: 1.007 to 1.044 times as fast on average in each tenth, the slowest 0.965, the fastest 1.112; six
// steps of 2.0 to 2.4 times 1.020, six of 2.4 to 2.6 times 0.991.
// Decodes alone gain as well, up to four rounds of pieces by time: a piece that is dealt asks for no ticket, and there are fewer partials.  165 random steps
// of up to 600 us on eight head layouts with such plans 1.03 times as fast on average (0.998 to 1.10; 249 decodes on 64-wide 32/4 heads 189 us and 175, 143
// on 32/8 heads 261 and 252).  Beyond kRoundsAloneNs a workgroup the pieces get so long that the dies' different rates show: 17 steps of
// 700 to 1270 us 1.004, 0.97 to 1.04.  Where the two rounds would not be two thirds full, few long contexts are left whole (288 on 64-wide 32/8 heads
// in 602 pieces 133 us and 143).
static const double kRoundsOver = 2.0;
static const double kRoundsOverAlone = 4.0;
static const double kRoundsAloneNs = 600000.0;
static const double kRoundsFilled = 2.0 / 3;
static const int64_t kHeadTokensMin = 256;
static const int64_t kHeadTokensWhole = 1024;
static const int64_t kHeadTokensBeside = 700;
// One round has to come out even: no piece may be longer than kLongestPiece times an even share, or what is left of a long context when
// there is room for one piece of each ends last (64 contexts spread evenly over the logarithm from 16 to 8192: 62.1 us by default, 85.9 in
// one round of one-head items, 60.6 of two-head items; 20 such families 1.05 on average, none slower; at 2 times 1.045, at 1.5 1.037).  Only in
// steps of at most kHeadShareWhole tokens of a head for each item is the longer piece bound by latency and not by the stream.
static const double kLongestPiece = 3.0;
static const int64_t kHeadShareWhole = 512;
static DecodeCut decode_cut(const int32_t* kind, const int32_t* ctx_len, int R, int Hkv, int D, double cap_ns, int64_t n_dec, int64_t dec_tokens,
                            int64_t n_pre, bool decode_dominated) {
  const int most = kv_heads_per_item(Hkv);
  const DecodeCut by_time = {most, std::max<int64_t>((int64_t)(cap_ns / ((double)most * D * 4.0 / kDecodeBytesPerNs)), kMinDecodeTokens)};
  constexpr uint32_t kPair = 2 * HFX_PAGE;    // tokens of a page pair
  auto items = [&](uint32_t pairs, int heads) {          // with pieces of that many page pairs
    int64_t n = 0;
    for (int r = 0; r < R; ++r) {
      if (kind[r] != HFX_DECODE) continue;
      const uint32_t all = ((uint32_t)ctx_len[r] + kPair - 1) / kPair;
      const uint32_t piece = std::max(pairs, (all + kMaxSplits - 1) / kMaxSplits);
      n += (all + piece - 1) / piece;
    }
    return n * (Hkv / heads);
  };
  auto shortest = [&](uint32_t lo, uint32_t hi, int heads, int64_t most_items) {    // pieces in [lo, hi] that make no more items
    while (lo < hi) {
      const uint32_t mid = lo + (hi - lo) / 2;
      if (items(mid, heads) <= most_items) hi = mid;
      else lo = mid + 1;
    }
    return lo;
  };
  auto by_rounds = [&]() -> DecodeCut {      // by time, but lengthened to two rounds if that is close
    const bool alone = n_pre == 0;
    const int64_t two_rounds = 2 * HFX_PLAN_WGS - n_pre;
    if (alone && (double)dec_tokens * Hkv * D * 4.0 > kRoundsAloneNs * HFX_PLAN_WGS * kDecodeBytesPerNs) return by_time;
    if (!alone && (!decode_dominated || n_pre >= HFX_PLAN_WGS || n_dec * (Hkv / most) > HFX_PLAN_WGS)) return by_time;
    const uint32_t piece = (uint32_t)(by_time.tokens + kPair - 1) / kPair;
    const int64_t now = items(piece, most);
    if (now <= two_rounds || (double)(now + n_pre) > (alone ? kRoundsOverAlone : kRoundsOver) * (double)(2 * HFX_PLAN_WGS)) return by_time;
    const uint32_t longer = shortest(piece, 4 * piece, most, two_rounds);
    const int64_t then = items(longer, most);
    if (then > two_rounds || (alone && (double)then < kRoundsFilled * (double)two_rounds)) return by_time;
    return {most, (int64_t)longer * kPair};
  };
  const int64_t room = n_pre == 0 ? HFX_PLAN_WGS : HFX_PLAN_WGS / 2 - n_pre;
  int h = 1;
  while (h < most && n_dec * (Hkv / h) > room) h *= 2;
  if (n_dec == 0) return by_time;
  if (h > 2 || n_dec * (Hkv / h) > room || (n_pre > 0 && h == most)) return by_rounds();
  int32_t longest = 0;
  for (int r = 0; r < R; ++r)
    if (kind[r] == HFX_DECODE) longest = std::max(longest, ctx_len[r]);
  for (; h <= std::min(2, most); h *= 2) {
    const int64_t share = dec_tokens * (Hkv / h) / room;
    const uint32_t least = (uint32_t)std::max<int64_t>(std::max(kHeadTokensMin / h, share) / kPair, 1);
    const uint32_t lo = shortest(least, (uint32_t)longest / kPair + 1, h, room);
    const int64_t tokens = (int64_t)lo * kPair;
    if (tokens > kLongestPiece * (double)(least * kPair)) continue;
    if (n_pre > 0 && (tokens * h > kHeadTokensBeside || h == most)) break;
    const bool whole = longest <= tokens + kHeadTokensWhole / h && share * h <= kHeadShareWhole;
    return {h, whole ? std::max<int64_t>(longest, tokens) : tokens};
  }
  return by_rounds();
}

// The work items of the step's requests (P.reqs), decode requests cut by dec_cut and prefill tiles
// by cap_prefill_ns, with their merge groups; *rows: partial rows of all of them, *dec_rows: those of decode items,
// *pre_ord: prefill requests.
static hfx_status make_items(const hfx_shape* shape, int32_t R, const DecodeCut& dec_cut, double cap_prefill_ns, Plan* out,
                             int64_t* rows_out, int64_t* dec_rows_out, int64_t* pre_ord_out) {
  const int Hkv = shape->num_kv_heads, D = shape->head_dim, G = shape->num_q_heads / Hkv;
  const int ngc = dec_cut.heads;
  const int hpw = q_heads_per_item(G);
  const int rows_wg = HFX_WAVE_ROWS * (4 / hpw);
  Plan& P = *out;
  P.items.clear();
  P.groups.clear();
  P.notes.clear();
  P.n_decode_items = 0;
  int64_t rows = 0, dec_rows = 0;
  std::vector<int32_t>& split_cost = P.split_cost;
  int64_t pre_ord = 0;              // prefill requests seen so far
  for (int r = 0; r < R; ++r) {
    const HfxReq& q = P.reqs[(size_t)r];
    if (q.kind == HFX_DECODE) {
      const double ns_per_token = (double)ngc * D * 4.0 / kDecodeBytesPerNs;
      const int64_t L = std::max<int64_t>(dec_cut.tokens, ((int64_t)q.ctx_len + kMaxSplits - 1) / kMaxSplits);
      int64_t pages_per = (L + HFX_PAGE - 1) / HFX_PAGE;
      pages_per += pages_per & 1;                     // page pairs stay aligned across splits
      int nsplit = (int)((q.n_pages + pages_per - 1) / pages_per);
      // even out the pieces
      pages_per = (q.n_pages + nsplit - 1) / nsplit;
      pages_per += pages_per & 1;
      nsplit = (int)((q.n_pages + pages_per - 1) / pages_per);
      HfxItem proto;                  // what all items of the request share
      std::memset(&proto, 0, sizeof proto);
      proto.type = HFX_ITEM_DECODE;
      proto.req = r;
      proto.hn = ngc;
      proto.rq = q;
      for (int g0 = 0; g0 < Hkv; g0 += ngc) {
        int group = -1;
        if (nsplit > 1) {
          group = (int)P.groups.size();
          HfxGroup gr = {nsplit, (int32_t)rows, ngc * G, HFX_ITEM_DECODE, r, g0, ngc, 0, q.q_start, q.q_len};
          P.groups.push_back(gr);
        }
        P.n_decode_items += nsplit;
        for (int s = 0; s < nsplit; ++s) {
          HfxItem it = proto;
          it.group = group;
          it.slot_row = (nsplit > 1) ? (int32_t)(rows + (int64_t)s * ngc * G) : -1;
          it.h0 = g0;
          it.kb = (int32_t)(s * pages_per);
          it.ke = (int32_t)std::min<int64_t>(q.n_pages, (int64_t)(s + 1) * pages_per);
          int64_t toks = std::min<int64_t>(q.ctx_len, (int64_t)it.ke * HFX_PAGE) - (int64_t)it.kb * HFX_PAGE;
          it.cost = clamp_cost((double)toks * ns_per_token + 2000.0);
          it.home = -1;
          P.items.push_back(it);
          P.notes.push_back(ItemNote{(uint32_t)it.cost, kNoUnit, 0.f});
        }
        if (nsplit > 1) {
          rows += (int64_t)nsplit * ngc * G;
          dec_rows += (int64_t)nsplit * ngc * G;
        }
      }
    } else {
      const int64_t p = q.ctx_len - q.q_len;
      const int n_rt = (q.q_len + rows_wg - 1) / rows_wg;
      for (int rt = 0; rt < n_rt; ++rt) {
        const int64_t r0 = (int64_t)rt * rows_wg, r1 = std::min<int64_t>(q.q_len, r0 + rows_wg);
        const int64_t kmax = p + r1;
        int64_t nsplit, tiles_per;
        prefill_splits(kmax, tile_ns(D, kmax), cap_prefill_ns, &nsplit, &tiles_per);
        split_cost.resize((size_t)nsplit);
        for (int64_t s = 0; s < nsplit; ++s) {
          const int64_t kb = s * tiles_per * HFX_KEY_TILE, ke = std::min<int64_t>(kmax, (s + 1) * tiles_per * HFX_KEY_TILE);
          split_cost[(size_t)s] = clamp_cost(tile_ns(D, ke - kb) + kItemNs);
        }
        const float frac = (float)rt / (float)n_rt;
        HfxItem proto;                // what all items of the row tile share
        std::memset(&proto, 0, sizeof proto);
        proto.type = HFX_ITEM_PREFILL;
        proto.req = r;
        proto.hn = hpw;
        proto.row0 = (int32_t)r0;
        proto.nrows = rows_wg;
        proto.rq = q;
        // All items of a row tile cost the same and stay in this order, in which dealt positions go round the dies: with the kv-heads innermost, the head blocks
        // that read one kv-head's keys come 8 positions apart, on one die, where there are 8 kv-heads.  (24/8 heads: 36 chunks of 7 rows behind 550 to
        // 760 tokens 46.4 us with the head blocks innermost, 28.0 so; 39 of 2 rows behind 5000 to 9000 464 and 261.  40 random steps of a few rows and of prompts on layouts
        // with several head blocks 1.09 times as fast on average, 40 of one to three prompts, some beside decodes, 1.009, 0.97 to 1.05; one chunk of 698 behind
        // 2749 beside 20 decodes is slower, 56 us and 60.)
        for (int hb = 0; hb < G / hpw; ++hb)
          for (int g = 0; g < Hkv; ++g) {
            int group = -1;
            if (nsplit > 1) {
              group = (int)P.groups.size();
              HfxGroup gr = {(int32_t)nsplit, (int32_t)rows, 4 * HFX_WAVE_ROWS, HFX_ITEM_PREFILL, r, g * G + hb * hpw, hpw, (int32_t)r0, q.q_start, q.q_len};
              P.groups.push_back(gr);
            }
            for (int64_t s = 0; s < nsplit; ++s) {
              HfxItem it = proto;
              it.group = group;
              it.slot_row = (nsplit > 1) ? (int32_t)(rows + s * 4 * HFX_WAVE_ROWS) : -1;
              it.h0 = g * G + hb * hpw;
              it.kb = (int32_t)(s * tiles_per * HFX_KEY_TILE);
              it.ke = (int32_t)std::min<int64_t>(kmax, (s + 1) * tiles_per * HFX_KEY_TILE);
              it.cost = split_cost[(size_t)s];
              it.home = -1;
              P.items.push_back(it);
              // the row tiles and head blocks that read the s-th piece of the keys of (request, kv-head)
              const int64_t unit = (pre_ord * Hkv + g) * kMaxSplits + s;
              P.notes.push_back(ItemNote{(uint32_t)it.cost, unit < (int64_t)kNoUnit ? (uint32_t)unit : kNoUnit, frac});
            }
            if (nsplit > 1) rows += nsplit * 4 * HFX_WAVE_ROWS;
          }
      }
      ++pre_ord;
    }
    if (rows > 0x7fffffff / 2 || P.items.size() > 0x3fffffffu) return HFX_ERR_LEN;
  }
  P.n_prefill_items = (int32_t)P.items.size() - P.n_decode_items;
  *rows_out = rows;
  *dec_rows_out = dec_rows;
  *pre_ord_out = pre_ord;
  return HFX_OK;
}

// The order in which the items of a step of many prompts are taken, where that is not their own (descending cost).
//
// Row tiles and head blocks of one (request, kv-head) read the same keys.  In a step of many prompts the 64 workgroups of a die work on as many different ones
// at a time, the tiles of one meet on a die by chance only, and every tile fetches its keys again: 1.79 GB fetched for 0.65 GB of keys, Q and
// decodes in a step of 384 short requests, 6.9 TB/s with the results, at a matrix rate of a third and at any core clock the same time.
// So the items of a unit go to one die, one behind the other, units in the order of their largest item: 0.73 GB, 304 -> 272 us.  The
// last prompts of the queue are the shortest ones, so that the dies end close to each other, and what is left is for all (kSharedTail).
//
// Measured on random steps, over one queue for all.  A workgroup's share at least 1.5 times the longest item: 50 steps of 80 streams
// ((request, kv-head) pairs) or more 1.06 times as fast on average, the slowest 1.00; of 128-wide heads with 32 to 79 streams 1.018 (41 steps, 0.98 to 1.06); 12 of
// fewer streams 1.00 (0.985 to 1.03: one prompt's tiles on all dies share their keys as it is).  64-wide heads have half the bytes a key and less to save:
// 0.990 with 32 to 79 streams (26 steps, 0.96 to 1.02), 1.007 with 104 to 176 (5, 0.99 to 1.03), 1.017 with 200 to 400 (9, 1.00 to 1.04).
// A share of 0.75 to 1.5 of the longest item and at least 160 streams 1.02 (0.97 to 1.07; 0.94 to 1.0 where decodes are more than a fifth of the
// step).  Chunks of a few rows whose head blocks share keys gain most: 14 of them behind 1800 to 30000 on 24/8 and 12/4 heads 1.24 (1.08 to 1.32).
//
// Where the kv-heads are a multiple of 8, the dealt positions keep a stream on one die as it is, and the order has something to give only behind them.  Random
// steps, by items: a share of 1.5 and more from 1025 items on 0.995 times as fast (17 steps, 0.98 to 1.02), from 1408 on 1.024 (11, 0.99 to 1.06), 1536 1.02, 1664
// 1.03; a smaller share from 1025 on 0.993 (49, 0.93 to 1.05), 1408 0.996 (11), 1536 1.007 (15), 1664 1.013, 1792 and more 1.02
// (40, 0.99 to 1.065).  With 1, 2 or 4 kv-heads all sizes gain: 1.02 from 1025 items on (18, 0.985 to 1.076), 1.03 from 1408 on.
static const int64_t kDieStreams = 32, kDieStreams64 = 80, kDieStreamsShort = 160;
static const double kDieShare = 1.5, kDieShareShort = 0.75, kDieDecodes = 0.2;
static const size_t kDieItems = HFX_PLAN_WGS * 11 / 4, kDieItemsShort = HFX_PLAN_WGS * 3;
// A unit is at most this part of a die's share of the step: a longer one is cut into consecutive row tiles.  (2: 1.026 over the steps that 16 to 128 take 1.039 to
// 1.044 over.)
static const int kDieUnits = 32;
// The share of a step's cost at the end of the queue that is handed out to all dies.  (3, 6, 12 and 25 %: 1.075, 1.064, 1.067 and 1.061 over 21 steps of
// short prompts; 384 of them 294.0, 293.6, 295.4 and 297.4 us; the prefill-heavy mixed step the same within 1 %.)
static const double kSharedTail = 0.06;

// `sorted`: the n items in descending cost, as keys of plan_step's sort (max_cost minus cost, index); P.stream_ns: time of the items of each stream
// of each request with a prompt; all: that of all items.
static void queue_per_die(const uint64_t* sorted, size_t n, int Hkv, double all, Plan* out) {
  Plan& P = *out;
  const double most = all / (kDieUnits * HFX_QUEUE_CLASSES);
  std::vector<Stream>& streams = P.streams;
  streams.resize(P.stream_ns.size() * (size_t)Hkv);
  uint32_t n_pieces = 0;
  for (size_t r = 0, st = 0; r < P.stream_ns.size(); ++r) {
    const double pieces = std::min(std::max(std::ceil(P.stream_ns[r] / most), 1.0), 1024.0);
    for (int g = 0; g < Hkv; ++g, ++st, n_pieces += (uint32_t)pieces) streams[st] = Stream{n_pieces, (uint32_t)pieces, P.stream_ns[r] / pieces};
  }
  // In the order of the items: a piece that is met for the first time goes to the die with the least work so far, behind that die's
  // other pieces.  A decode item is a piece of its own.
  std::vector<uint32_t>& count = P.unit_fill;            // items of a piece
  std::vector<uint32_t>& place = P.unit_start;           // die of a piece; then the position of its next item
  std::vector<uint32_t>& piece_of = P.order_pre;         // of the i-th item
  count.assign(n_pieces + n, 0);
  place.resize(n_pieces + n);
  piece_of.resize(n);
  static_assert(HFX_QUEUE_CLASSES == 8, "loads compared below");
  double load[HFX_QUEUE_CLASSES] = {0.0};
  std::vector<uint32_t>* lists = P.die_lists;            // pieces of each die
  for (int c = 0; c < HFX_QUEUE_CLASSES; ++c) lists[c].clear();
  for (size_t i = 0; i < n; ++i) {
    const ItemNote& note = P.notes[(uint32_t)sorted[i]];
    uint32_t piece;
    double work;
    if (note.unit != kNoUnit) {
      const Stream& st = streams[note.unit / kMaxSplits];
      piece = st.first;
      if (st.pieces > 1) piece += std::min(st.pieces - 1, (uint32_t)(note.frac * (float)st.pieces));
      work = st.work;
    } else {
      piece = n_pieces++;
      work = note.cost;
    }
    piece_of[i] = piece;
    if (count[piece]++) continue;
    // (a chain of eight comparisons, each waiting for the one before, was two thirds of this function's time)
    const double least = std::min(std::min(std::min(load[0], load[1]), std::min(load[2], load[3])),
                                  std::min(std::min(load[4], load[5]), std::min(load[6], load[7])));
    unsigned mask = 0;
    for (int c = 0; c < HFX_QUEUE_CLASSES; ++c) mask |= (unsigned)(load[c] == least) << c;
    const int home = __builtin_ctz(mask);
    load[home] += work;
    lists[home].push_back(piece);
  }
  size_t end[HFX_QUEUE_CLASSES];
  for (int c = 0; c < HFX_QUEUE_CLASSES; ++c) {
    size_t at = (size_t)c;
    for (const uint32_t piece : lists[c]) {
      place[piece] = (uint32_t)at;
      at += (size_t)HFX_QUEUE_CLASSES * count[piece];
    }
    end[c] = at;
  }
  // position p is for die p % HFX_QUEUE_CLASSES; when a die's list ends, its positions take what is left of the longer ones
  std::vector<uint32_t>& left = P.order_dec;
  left.clear();
  for (size_t i = 0; i < n; ++i) {
    const uint32_t at = place[piece_of[i]];
    place[piece_of[i]] = at + HFX_QUEUE_CLASSES;
    if (at < n) P.queue[at] = (int32_t)i;
    else left.push_back((uint32_t)i);
  }
  for (int c = 0; c < HFX_QUEUE_CLASSES; ++c)
    for (size_t at = end[c]; at < n; at += HFX_QUEUE_CLASSES) {
      P.queue[at] = (int32_t)left.back();
      left.pop_back();
    }
}

// How many of the positions of a queue per die are handed out by die; cost(p) is that of position p, all that of all n.
template <typename F>
static int32_t positions_by_die(size_t n, double all, F cost) {
  double behind = 0.0;
  size_t at = n;
  while (at > 0 && behind + cost(at - 1) <= kSharedTail * all) behind += cost(--at);
  return (int32_t)(at / HFX_QUEUE_CLASSES * HFX_QUEUE_CLASSES);
}

hfx_status plan_step(const hfx_shape* shape, int32_t R, const int32_t* kind, const int32_t* q_len,
                     const int32_t* ctx_len, Plan* out, bool sizes_only) {
  hfx_status st = check_shape(shape);
  if (st != HFX_OK) return st;
  if (!kind || !q_len || !ctx_len || !out) return HFX_ERR_NULL;
  if (R < 1) return HFX_ERR_SHAPE;
  const int Hq = shape->num_q_heads, Hkv = shape->num_kv_heads, D = shape->head_dim;
  const int G = Hq / Hkv;
  const int hpw = q_heads_per_item(G);
  const int rows_wg = HFX_WAVE_ROWS * (4 / hpw);
  const int mult = Hkv * (G / hpw);      // prefill items of a row tile, when it is not cut

  Plan& P = *out;
  P.reqs.assign((size_t)R, HfxReq());
  P.stream_ns.clear();
  int64_t T = 0, nbt = 0, n_dec = 0, dec_tokens = 0;
  double dec_ns = 0.0, pre_ns = 0.0;   // modelled time of each kind of work, prefill by (row, key) pairs
  double stream_ns = 0.0;              // the prefills' keys streamed once, at the rate of decodes ...
  double apart_ns = 0.0;               // ... or by every row tile and head block of a request that has one row tile
  double tiles_ns = 0.0, beside_ns = 0.0;   // the row tiles: time of full ones, and counting the wavefronts that have rows
  int64_t streams = 0, readers = 0;    // (request, kv-head) pairs of prefills, and the uncut items that read their keys
  for (int r = 0; r < R; ++r) {
    if (kind[r] != HFX_DECODE && kind[r] != HFX_PREFILL) return HFX_ERR_KIND;
    if (q_len[r] < 1 || ctx_len[r] < q_len[r]) return HFX_ERR_LEN;
    if (kind[r] == HFX_DECODE && q_len[r] != 1) return HFX_ERR_LEN;
    HfxReq& q = P.reqs[(size_t)r];
    q.kind = kind[r];
    q.q_len = q_len[r];
    q.ctx_len = ctx_len[r];
    q.n_pages = (int32_t)(((int64_t)ctx_len[r] + HFX_PAGE - 1) / HFX_PAGE);
    q.bt_len = ((q.n_pages + 3) & ~3) + HFX_BT_PAD;
    if (T > 0x7fffffff - q_len[r] || nbt > 0x7fffffff - q.bt_len) return HFX_ERR_LEN;
    q.q_start = (int32_t)T;
    q.bt_start = (int32_t)nbt;
    T += q_len[r];
    nbt += q.bt_len;
    if (kind[r] == HFX_DECODE) {
      dec_ns += (double)ctx_len[r] * Hkv * D * 4.0 / kDecodeBytesPerNs;
      ++n_dec;
      dec_tokens += ctx_len[r];
    } else {
      double ql = q_len[r], p = ctx_len[r] - q_len[r];
      pre_ns += 4.0 * D * Hq * (ql * p + ql * (ql + 1) / 2) / kPrefillFlopsPerNs;
      const double keys_ns = (double)ctx_len[r] * D * 4.0 / kDecodeBytesPerNs;
      stream_ns += keys_ns * Hkv;
      apart_ns += keys_ns * (q_len[r] <= rows_wg ? mult : Hkv);
      // full row tiles see p + rows_wg, p + 2 rows_wg, ... keys; a last one that is not full sees all
      const int64_t full = q_len[r] / rows_wg, rest = q_len[r] % rows_wg;
      const double full_ns = tile_ns(D, 1) * mult * ((double)full * p + 0.5 * rows_wg * (double)full * (double)(full + 1));
      const double rest_ns = rest ? tile_ns(D, ctx_len[r]) * mult : 0.0;
      streams += Hkv;
      readers += (full + (rest ? 1 : 0)) * mult;
      tiles_ns += full_ns + rest_ns;
      P.stream_ns.push_back((full_ns + rest_ns + kItemNs * (double)((full + (rest ? 1 : 0)) * mult)) / Hkv);
      beside_ns += full_ns + rest_ns * (kLoneShare + (1.0 - kLoneShare) * tile_busy(hpw, rest));
    }
  }
  P.total_q = (int32_t)T;
  P.n_bt = (int32_t)nbt;
  int64_t n_runs = 0;   // pages touched by each request's new tokens
  for (int r = 0; r < R; ++r)
    n_runs += (ctx_len[r] - 1) / HFX_PAGE - (ctx_len[r] - q_len[r]) / HFX_PAGE + 1;
  P.n_runs = (int32_t)n_runs;
  const double total_ns = dec_ns + pre_ns;
  // Which kind of work outweighs the other goes by the time the items take, as cuts and queue do.  (By pairs, four decodes of
  // 2000 tokens outweighed 48 chunks of one row behind 3269 that take twenty times as long: all tiles were cut for a decode
  // stream that is not there, and the step took 84 us instead of 70.)
  const bool decode_dominated = dec_ns > tiles_ns;
  // Decode pieces are sized against the decode work alone (in a step dominated by prefill they stay
  // small and fill the gaps between the large prefill items), for a whole number of rounds of the
  // planning width: as many rounds as fit pieces of at least the minimum size, at most
  // kDecodeItemsPerWg.  A step with work for 2.4 rounds of minimum-size pieces is better served by
  // two rounds of larger ones than by a third, half-empty round.
  double rounds = std::floor(dec_ns / (HFX_PLAN_WGS * kMinItemNs));
  rounds = std::min<double>(std::max(rounds, 1.0), kDecodeItemsPerWg);
  const double cap_ns = std::max(dec_ns / (HFX_PLAN_WGS * rounds), kMinItemNs);
  const double cap_prefill_ns =
      pre_ns > 0.0 ? prefill_cap(kind, q_len, ctx_len, R, mult, D, hpw, rows_wg, dec_ns, stream_ns, decode_dominated, &P) : kMinItemNs;

  int64_t n_pre = 0;                   // prefill items
  if (pre_ns > 0.0 && n_dec > 0 && (decode_dominated || n_dec * (Hkv / kv_heads_per_item(Hkv)) < HFX_PLAN_WGS / 2))
    cut_rows(kind, q_len, ctx_len, R, mult, rows_wg, cap_prefill_ns, [&](int64_t p, int64_t, int64_t r1) { return tile_ns(D, p + r1); }, &n_pre);
  else if (pre_ns > 0.0)
    n_pre = HFX_PLAN_WGS;
  const DecodeCut dec_cut = decode_cut(kind, ctx_len, R, Hkv, D, cap_ns, n_dec, dec_tokens, n_pre, decode_dominated);

  int64_t rows = 0, dec_rows = 0, pre_ord = 0;
  st = make_items(shape, R, dec_cut, cap_prefill_ns, &P, &rows, &dec_rows, &pre_ord);
  if (st != HFX_OK) return st;
  if (rows * (4ll * D + 8) + 512 > (int64_t)HFX_STATIC_WS_BYTES && rows > dec_rows) {
    const double c = cap_within_workspace(kind, q_len, ctx_len, R, mult, D, hpw, rows_wg, dec_ns, pre_ns, dec_rows, cap_prefill_ns);
    if (c > cap_prefill_ns) {
      st = make_items(shape, R, dec_cut, c, &P, &rows, &dec_rows, &pre_ord);
      if (st != HFX_OK) return st;
    }
  }
  P.n_partial_rows = (int32_t)rows;
  const size_t n = P.items.size();
  uint32_t max_cost = 0;
  for (size_t i = 0; i < n; ++i) max_cost = std::max(max_cost, P.notes[i].cost);
  // Which of the queue orders below the step gets.
  const bool beside = decode_dominated && pre_ns > 0.0;
  const bool units_fit = pre_ord * Hkv * kMaxSplits < (int64_t)kNoUnit;
  const bool classes = !beside && pre_ns > 0.0 && units_fit && n <= (size_t)kClassRoundsMax * HFX_PLAN_WGS &&
                       ((n >= (size_t)kClassRoundsMin * HFX_PLAN_WGS &&
                         ((D == 128 && total_ns >= kClassStepNs * HFX_PLAN_WGS) ||
                          (stream_ns >= kClassStreamBytes / kDecodeBytesPerNs && readers >= 2 * streams && total_ns >= kMinItemNs * (double)n))) ||
                        (n >= (size_t)kClassRoundsMinApart * HFX_PLAN_WGS && dec_ns + tiles_ns >= kClassItemNsApart * (double)n &&
                         mult > Hkv && apart_ns >= kClassApart * beside_ns));
  const double all_ns = dec_ns + tiles_ns + kItemNs * (double)n, even_ns = (double)HFX_PLAN_WGS * max_cost;
  const size_t from = Hkv % HFX_QUEUE_CLASSES == 0 ? kDieItems : 0, from_short = Hkv % HFX_QUEUE_CLASSES == 0 ? kDieItemsShort : 0;
  const bool per_die = !beside && !classes && pre_ns > 0.0 && units_fit && n > 2 * (size_t)HFX_PLAN_WGS && readers >= 2 * streams &&
                       ((all_ns >= kDieShare * even_ns && n >= from && streams >= (D == 64 ? kDieStreams64 : kDieStreams)) ||
                        (all_ns >= kDieShareShort * even_ns && n >= from_short && dec_ns <= kDieDecodes * all_ns && streams >= kDieStreamsShort));
  P.queue.resize(per_die ? n : 0);
  // queue order: descending cost, ties in creation order: a stable radix sort (11-bit digits) of
  // (inverted cost, index) keys, then one permutation of the item records.
  if (!sizes_only) {
    std::vector<uint64_t>& key = P.sort_keys;
    key.resize(2 * n);
    uint64_t* a = key.data();
    uint64_t* b = a + n;
    // keys count down from the largest cost, so that the number of digit passes follows the range
    // of costs in the step and not the width of the field
    uint32_t top = 0;
    for (size_t i = 0; i < n; ++i) {
      const uint32_t inv = max_cost - P.notes[i].cost;
      a[i] = ((uint64_t)inv << 32) | (uint64_t)i;
      top |= inv;
    }
    for (int shift = 0; shift < 31 && (top >> shift) != 0; shift += 11) {
      uint32_t count[2048] = {0};
      for (size_t i = 0; i < n; ++i) count[(a[i] >> (32 + shift)) & 2047u]++;
      uint32_t sum = 0;
      for (int d = 0; d < 2048; ++d) {
        const uint32_t c = count[d];
        count[d] = sum;
        sum += c;
      }
      for (size_t i = 0; i < n; ++i) b[count[(a[i] >> (32 + shift)) & 2047u]++] = a[i];
      std::swap(a, b);
    }
    // the queue order is kept as a permutation; the records are put in that order when the blob is written
    std::vector<uint32_t>& order = P.order;
    order.resize(n);
    P.queue_classes = 1;
    P.die_items = 0;
    P.deal_balanced = !beside;   // the layout below is by workgroup
    if (beside) {
      // A step whose decode work outweighs its prefill work.  The first two items of workgroup b
      // are queue positions b and b + HFX_PLAN_WGS, and workgroups b and b + HFX_PLAN_WGS/2 share a
      // CU.  Over those two rounds the prefill items (largest first) go to the workgroups of the
      // first `pair_cus` CUs, both workgroups of a CU, and the decode items to all the others:
      // the matrix work then runs in the shadow of the memory-bound stream without sharing a
      // CU's memory path with it (a prefill workgroup next to a decode workgroup on one CU saw its
      // tiles take 2.5 times as long; measured on the Llama-8B-shaped mixed step, this layout takes
      // 6 % less time than one workgroup of each kind per CU, which in turn took 5 % less than plain
      // descending order).  pair_cus is sized so that the two rounds hold all prefill items, up to
      // half the CUs.  Behind the two rounds the kinds alternate in blocks of half the planning
      // width, decode first, each kind still in descending cost.  On prefill-dominated steps any
      // such interleave costs 2-13 %, so they keep the plain order.
      constexpr size_t kBlockItems = HFX_PLAN_WGS / 2;
      std::vector<uint32_t>& dec = P.order_dec;
      std::vector<uint32_t>& pre = P.order_pre;
      dec.clear();
      pre.clear();
      for (size_t i = 0; i < n; ++i) {
        const uint32_t idx = (uint32_t)(a[i] & 0xffffffffu);
        (P.items[idx].type == HFX_ITEM_DECODE ? dec : pre).push_back(idx);
      }
      const size_t pair_cus = std::min<size_t>((pre.size() + 3) / 4, kBlockItems / 2);
      size_t di = 0, pi = 0, o = 0;
      for (int round = 0; round < 2; ++round)
        for (size_t b = 0; b < (size_t)HFX_PLAN_WGS && o < n; ++b) {
          const bool prefill_slot = (b % kBlockItems) < pair_cus;
          if ((prefill_slot && pi < pre.size()) || di >= dec.size()) order[o++] = pre[pi++];
          else order[o++] = dec[di++];
        }
      while (di < dec.size() || pi < pre.size()) {
        for (size_t k = 0; k < kBlockItems && di < dec.size(); ++k) order[o++] = dec[di++];
        for (size_t k = 0; k < kBlockItems && pi < pre.size(); ++k) order[o++] = pre[pi++];
      }
    } else if (classes) {
      // A step whose prefill work outweighs its decode work.  Many prefill items read the same
      // keys: all row tiles (and q-head blocks) of one request and kv-head that hold the same
      // piece of the key range.  Call that set a unit.  The chip has HFX_QUEUE_CLASSES dies, each
      // with an L2 of its own, and workgroup b runs on die b % HFX_QUEUE_CLASSES; the kernel hands
      // queue position p to a workgroup of die p % HFX_QUEUE_CLASSES (as long as that die has work).
      // So the queue is built per class: every unit gets a home class (largest total cost first,
      // each to the class with the least cost so far), a class lists the items homed there in
      // descending cost, and the classes are interleaved position by position.  Items of a unit
      // that cost about the same then run side by side on one die and fetch their keys from
      // memory once instead of once per die and round, while the queue as a whole still goes
      // from the most to the least expensive items.  A decode item is a unit of its own.  When
      // a class runs out of items before the others, its positions are filled from the tail of
      // the class that has most left.
      const size_t n_slots = (size_t)(pre_ord * Hkv * kMaxSplits);
      std::vector<int64_t>& ucost = P.unit_cost;
      std::vector<uint32_t>& ufill = P.unit_fill;
      std::vector<uint32_t>& ustart = P.unit_start;
      std::vector<uint64_t>& ukeys = P.unit_keys;
      // A unit that would be a large share of a class's work is cut into sub-units of consecutive
      // row tiles, each at most about half of one class's share of the step, so that there is
      // something to balance with (a long prompt on one kv-head has as few units as it has splits).
      ucost.assign(n_slots, 0);
      int64_t all_cost = 0;
      for (size_t i = 0; i < n; ++i) {
        all_cost += P.notes[i].cost;
        if (P.notes[i].unit != kNoUnit) ucost[P.notes[i].unit] += P.notes[i].cost;
      }
      const int64_t sub_cost = std::max<int64_t>(1, all_cost / (2 * HFX_QUEUE_CLASSES));
      ufill.assign(n_slots, 0);     // sub-units of the slot
      ustart.assign(n_slots, 0);    // index of its first sub-unit
      size_t n_units = 0;
      for (size_t u = 0; u < n_slots; ++u)
        if (ucost[u] > 0) {
          ufill[u] = (uint32_t)std::min<int64_t>((ucost[u] + sub_cost - 1) / sub_cost, 4 * HFX_QUEUE_CLASSES);
          ustart[u] = (uint32_t)n_units;
          n_units += ufill[u];
        }
      // decode items (and anything else without a unit) get singleton units behind those
      for (size_t i = 0; i < n; ++i) {
        const uint32_t u = P.notes[i].unit;
        if (u == kNoUnit) P.notes[i].unit = (uint32_t)n_units++;
        else P.notes[i].unit = ustart[u] + std::min<uint32_t>(ufill[u] - 1, (uint32_t)(P.notes[i].frac * (float)ufill[u]));
      }
      ucost.assign(n_units, 0);     // total cost of the unit; once it has a home, the home
      ustart.assign(n_units, 0);    // items in the unit
      for (size_t i = 0; i < n; ++i) {
        const uint32_t u = P.notes[i].unit;
        ucost[u] += P.notes[i].cost;
        ustart[u]++;
      }
      // home classes: units by descending total cost (36 bits of it, saturating; the low 28 bits
      // of a key hold the unit's index)
      ukeys.clear();
      const int64_t kCostTop = (1ll << 36) - 1;
      for (size_t u = 0; u < n_units; ++u)
        if (ustart[u]) ukeys.push_back(((uint64_t)(kCostTop - std::min(ucost[u], kCostTop)) << 28) | (uint64_t)u);
      std::sort(ukeys.begin(), ukeys.end());
      int64_t load[HFX_QUEUE_CLASSES] = {0};
      for (uint64_t& k : ukeys) {
        const uint32_t u = (uint32_t)(k & 0x0fffffffu);
        int home = 0;
        for (int c = 1; c < HFX_QUEUE_CLASSES; ++c)
          if (load[c] < load[home]) home = c;
        load[home] += ucost[u];
        ucost[u] = home;
      }
      // The items are in descending cost (a[]); a class's list is those of them that are homed
      // there, in that order (a stable counting sort by class into b[]).
      size_t head[HFX_QUEUE_CLASSES], tail[HFX_QUEUE_CLASSES];
      for (int c = 0; c < HFX_QUEUE_CLASSES; ++c) tail[c] = 0;
      for (size_t i = 0; i < n; ++i) {
        const uint32_t idx = (uint32_t)(a[i] & 0xffffffffu);
        const int home = (int)ucost[P.notes[idx].unit];
        P.items[idx].home = home;
        tail[home]++;
      }
      for (int c = 0, at = 0; c < HFX_QUEUE_CLASSES; ++c) {
        head[c] = (size_t)at;
        at += (int)tail[c];
        tail[c] = head[c];          // fill cursor; ends up one past the class's last item
      }
      for (size_t i = 0; i < n; ++i) b[tail[P.items[(uint32_t)(a[i] & 0xffffffffu)].home]++] = a[i];
      std::swap(a, b);
      P.queue_classes = HFX_QUEUE_CLASSES;
      for (size_t o = 0; o < n; ++o) {
        const int c = (int)(o % HFX_QUEUE_CLASSES);
        if (head[c] < tail[c]) {
          order[o] = (uint32_t)(a[head[c]++] & 0xffffffffu);
        } else {
          int from = 0;
          for (int y = 1; y < HFX_QUEUE_CLASSES; ++y)
            if (tail[y] - head[y] > tail[from] - head[from]) from = y;
          order[o] = (uint32_t)(a[--tail[from]] & 0xffffffffu);
        }
      }
      P.die_items = positions_by_die(n, (double)all_cost, [&](size_t p) { return (double)P.items[order[p]].cost; });
    } else {
      for (size_t i = 0; i < n; ++i) order[i] = (uint32_t)(a[i] & 0xffffffffu);
      if (per_die) {
        queue_per_die(a, n, Hkv, all_ns, &P);
        P.die_items = positions_by_die(n, all_ns, [&](size_t p) { return (double)(max_cost - (uint32_t)(a[P.queue[p]] >> 32)); });
      }
    }
  }
  // merge work units: groups with many splits get 8 threads per (row, column) and one row per
  // workgroup, groups with few splits one thread per (row, column) and 8 rows per workgroup
  P.units.clear();
  for (size_t gi = 0; gi < P.groups.size(); ++gi) {
    const int rows_per_unit = P.groups[gi].nsplit > 8 ? 1 : 8;
    for (int c = 0; c * rows_per_unit < P.groups[gi].rows_per_split; ++c) {
      HfxUnit u = {(int32_t)gi, c};
      P.units.push_back(u);
    }
  }
  return HFX_OK;
}

static uint64_t align_up(uint64_t x, uint64_t a) { return (x + a - 1) / a * a; }

void layout_blob(const hfx_shape* shape, const Plan& P, HfxHeader* h) {
  std::memset(h, 0, sizeof *h);
  h->magic = HFX_DESC_MAGIC;
  h->version = HFX_DESC_VERSION;
  h->num_requests = (int32_t)P.reqs.size();
  h->total_q = P.total_q;
  h->num_q_heads = shape->num_q_heads;
  h->num_kv_heads = shape->num_kv_heads;
  h->head_dim = shape->head_dim;
  h->page_size = shape->page_size;
  h->num_pages = shape->num_pages;
  h->softmax_scale = shape->softmax_scale > 0.f ? shape->softmax_scale : 1.0f / std::sqrt((float)shape->head_dim);
  h->n_items = (int32_t)P.items.size();
  h->n_decode_items = P.n_decode_items;
  h->n_prefill_items = P.n_prefill_items;
  h->n_groups = (int32_t)P.groups.size();
  h->n_partial_rows = P.n_partial_rows;
  h->n_bt = P.n_bt;
  h->n_ctrl = HFX_CTRL_WORDS;
  h->queue_classes = (uint32_t)P.queue_classes;
  h->deal_balanced = (uint32_t)P.deal_balanced;
  h->die_items = (uint32_t)P.die_items;
  h->max_group_rows = 0;
  for (const HfxGroup& g : P.groups) h->max_group_rows = std::max(h->max_group_rows, g.rows_per_split);
  uint64_t off = align_up(sizeof(HfxHeader), 256);
  h->off_ctrl = (uint32_t)off;
  off = align_up(off + 4ull * h->n_ctrl, 64);
  h->off_req = (uint32_t)off;
  off = align_up(off + sizeof(HfxReq) * P.reqs.size(), 64);
  h->off_bt = (uint32_t)off;
  off = align_up(off + 4ull * (uint64_t)P.n_bt, 64);
  h->off_items = (uint32_t)off;
  off = align_up(off + sizeof(HfxItem) * P.items.size(), 64);
  h->off_queue = P.queue.empty() ? 0u : (uint32_t)off;
  off = align_up(off + 4ull * P.queue.size(), 64);
  h->off_groups = (uint32_t)off;
  off = align_up(off + sizeof(HfxGroup) * P.groups.size(), 64);
  h->off_units = (uint32_t)off;
  h->n_units = (int32_t)P.units.size();
  off = align_up(off + sizeof(HfxUnit) * P.units.size(), 64);
  h->off_runs = (uint32_t)off;
  h->n_runs = P.n_runs;
  off = align_up(off + sizeof(HfxRun) * (uint64_t)P.n_runs, 256);
  h->total_bytes = off;
  uint64_t acc_bytes = align_up((uint64_t)P.n_partial_rows * shape->head_dim * 4ull, 256);
  h->ws_off_ml = acc_bytes;
  h->workspace_bytes = P.n_partial_rows ? acc_bytes + align_up((uint64_t)P.n_partial_rows * 8ull, 256) : 0;
}

hfx_status fill_blob(const hfx_shape* shape, Plan& P, const int32_t* bt_indptr, const int32_t* bt_pages,
                     void* host_desc, size_t host_desc_bytes) {
  if (!bt_indptr || !bt_pages || !host_desc) return HFX_ERR_NULL;
  HfxHeader h;
  layout_blob(shape, P, &h);
  if (h.total_bytes > 0xffffffffull) return HFX_ERR_LEN;
  if (host_desc_bytes < h.total_bytes) return HFX_ERR_BUFSIZE;
  const int R = (int)P.reqs.size();
  if (bt_indptr[0] != 0) return HFX_ERR_PAGES;
  for (int r = 0; r < R; ++r) {
    if (bt_indptr[r + 1] < bt_indptr[r]) return HFX_ERR_PAGES;
    if ((int64_t)bt_indptr[r + 1] - bt_indptr[r] < P.reqs[(size_t)r].n_pages) return HFX_ERR_PAGES;
  }
  for (int r = 0; r < R; ++r) {
    const int32_t* src = bt_pages + bt_indptr[r];
    for (int i = 0; i < P.reqs[(size_t)r].n_pages; ++i)
      if (src[i] < 0 || src[i] >= shape->num_pages) return HFX_ERR_PAGE_ID;
  }
  char* base = (char*)host_desc;
  // every byte of the blob is written: sections by copy, the padding between them with zeros
  auto put = [base](uint64_t off, const void* src, uint64_t bytes, uint64_t next_off) {
    if (bytes) std::memcpy(base + off, src, (size_t)bytes);
    std::memset(base + off + bytes, 0, (size_t)(next_off - off - bytes));
  };
  put(0, &h, sizeof h, h.off_ctrl);
  put(h.off_ctrl, nullptr, 0, h.off_req);
  put(h.off_req, P.reqs.data(), sizeof(HfxReq) * P.reqs.size(), h.off_bt);
  int32_t* bt = (int32_t*)(base + h.off_bt);
  for (int r = 0; r < R; ++r) {
    const HfxReq& q = P.reqs[(size_t)r];
    int32_t* dst = bt + q.bt_start;
    // (looked at again on the way: the caller's list may have changed since)
    const int32_t* src = bt_pages + bt_indptr[r];
    bool outside = false;
    for (int i = 0; i < q.n_pages; ++i) {
      const int32_t page = src[i];
      outside |= (uint32_t)page >= (uint32_t)shape->num_pages;
      dst[i] = page;
    }
    if (outside) {
      std::memset(base, 0, sizeof h);       // half a descriptor is none
      return HFX_ERR_PAGE_ID;
    }
    for (int i = q.n_pages; i < q.bt_len; ++i) dst[i] = dst[q.n_pages - 1];
  }
  put(h.off_bt + 4ull * (uint64_t)P.n_bt, nullptr, 0, h.off_items);
  HfxItem* queue = (HfxItem*)(base + h.off_items);
  for (size_t i = 0; i < P.items.size(); ++i) queue[i] = P.items[P.order[i]];
  const uint64_t items_end = h.off_items + sizeof(HfxItem) * P.items.size();
  if (h.off_queue) {
    put(items_end, nullptr, 0, h.off_queue);
    put(h.off_queue, P.queue.data(), 4ull * P.queue.size(), h.off_groups);
  } else {
    put(items_end, nullptr, 0, h.off_groups);
  }
  put(h.off_groups, P.groups.data(), sizeof(HfxGroup) * P.groups.size(), h.off_units);
  put(h.off_units, P.units.data(), sizeof(HfxUnit) * P.units.size(), h.off_runs);
  // append runs: each request's new tokens, cut at page boundaries
  HfxRun* run = (HfxRun*)(base + h.off_runs);
  for (int r = 0; r < R; ++r) {
    const HfxReq& q = P.reqs[(size_t)r];
    const int32_t* pages = bt + q.bt_start;
    int32_t t = q.ctx_len - q.q_len;
    while (t < q.ctx_len) {
      const int32_t slot0 = t % HFX_PAGE;
      const int32_t n = std::min<int32_t>(HFX_PAGE - slot0, q.ctx_len - t);
      *run++ = HfxRun{q.q_start + (t - (q.ctx_len - q.q_len)), n, pages[t / HFX_PAGE], slot0};
      t += n;
    }
  }
  put(h.off_runs + sizeof(HfxRun) * (uint64_t)P.n_runs, nullptr, 0, h.total_bytes);
  return HFX_OK;
}

}  // namespace hfx
