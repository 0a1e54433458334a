// Host planner: turns the per-request (prefix, suffix) lengths of a wave into
// the work lists the kernels consume.  Integer work only.
//
// The wave is the set of requests launched together for prefill (Sec. 2.4);
// request r contributes S_r uncached rows that attend over P_r + S_r keys
// (Eq. 3-4).  Work per (request, kv head, row tile) grows with the visible key
// count, which varies by two orders of magnitude inside one wave, so the
// planner cuts long key ranges into chunks (split-KV) and orders workgroups
// longest first.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <map>
#include <set>
#include <tuple>

#include "prism_internal.h"

namespace prism {

int check_shape(const prism_shape_t &s) {
  if (s.batch <= 0 || s.num_q_heads <= 0 || s.num_kv_heads <= 0 || s.num_pages <= 0 ||
      s.max_blocks_per_req <= 0)
    return PRISM_ERR_INVALID_ARG;
  if (s.num_q_heads % s.num_kv_heads != 0) return PRISM_ERR_INVALID_ARG;
  if (!(s.softmax_scale > 0.0f) || !std::isfinite(s.softmax_scale)) return PRISM_ERR_INVALID_ARG;
  if (s.page_size != kPage) return PRISM_ERR_UNSUPPORTED;
  if (s.head_dim != 64 && s.head_dim != 128) return PRISM_ERR_UNSUPPORTED;
  return PRISM_OK;
}

namespace {

int key_tiles(int keys) { return (keys + kTileKeys - 1) / kTileKeys; }

// How the key range of a row tile is cut: into pieces of about `chunk` key tiles,
// a range that exceeds it by no more than `slack` staying whole, and so many that
// none need be shorter than `least`.
struct SplitRule {
  int chunk = 0, slack = 0, least = 1;             // chunk 0: never cut
  int pieces(int cost) const {
    return chunk ? std::max(1, std::min(cost / least, (cost - slack + chunk - 1) / chunk)) : 1;
  }
};

// Row tiles of one kv head by their key tiles, descending.
struct Cost {
  int tiles;
  int64_t count, rows;                             // how many, and the packed rows of all of them
};
using Costs = std::vector<Cost>;

// Time, in key tiles, until `slots` workers have done all pieces, longest first.
int64_t makespan(const Costs &costs, int heads, const SplitRule &rule, int slots) {
  std::vector<std::pair<int, int64_t>> pieces;     // length, how many
  int64_t total = 0;
  for (const auto &c : costs) {
    const int n = rule.pieces(c.tiles), len = (c.tiles + n - 1) / n;
    const int64_t count = c.count * n * heads;
    pieces.push_back({len, count});
    total += count * len;
  }
  std::sort(pieces.rbegin(), pieces.rend());
  std::vector<int64_t> at(total / slots + 2 * (int64_t)pieces[0].first + 2, 0);   // workers by load so far
  at[0] = slots;
  int64_t low = 0, high = 0;
  for (auto &p : pieces)
    while (p.second > 0) {
      while (at[low] == 0) ++low;
      const int64_t k = std::min(at[low], p.second);
      at[low] -= k;
      at[low + p.first] += k;
      p.second -= k;
      high = std::max(high, low + p.first);
    }
  return high;
}

// The smallest chunk >= min_chunk whose pieces number at most `items`.
SplitRule fit(const Costs &costs, int heads, int min_chunk, int slack, int64_t items) {
  int lo = min_chunk, hi = std::max(min_chunk, costs[0].tiles);
  while (lo < hi) {
    const SplitRule mid{(lo + hi) / 2, slack, min_chunk};
    int64_t n = 0;
    for (const auto &c : costs) n += c.count * mid.pieces(c.tiles);
    if (n * heads <= items) hi = mid.chunk;
    else lo = mid.chunk + 1;
  }
  return SplitRule{lo, slack, min_chunk};
}

// The same rule with the smallest larger chunk that leaves at most `slots` pieces
// of cut ranges.
SplitRule coarser(const Costs &costs, int heads, const SplitRule &rule, int64_t slots) {
  const bool follows = rule.slack == rule.chunk;
  auto with = [&](int chunk) { return SplitRule{chunk, follows ? chunk : rule.slack, rule.least}; };
  int lo = rule.chunk + 1, hi = std::max(lo, costs[0].tiles);   // the largest cuts nothing
  while (lo < hi) {
    const SplitRule mid = with((lo + hi) / 2);
    int64_t n = 0;
    for (const auto &c : costs)
      if (mid.pieces(c.tiles) > 1) n += c.count * mid.pieces(c.tiles);
    if (n * heads <= slots) hi = mid.chunk;
    else lo = mid.chunk + 1;
  }
  return with(lo);
}

// `dies`: how many the row tiles go to.  `asked`: min_chunk is the caller's.
SplitRule choose_split(const Costs &costs, int heads, int dies, int min_chunk, bool asked, bool stream, bool in_tiles, int d) {
  int64_t total = 0, n = 0;
  for (const auto &c : costs) {
    total += c.count * c.tiles * heads;
    n += c.count * heads;
  }
  if (stream) {
    // One workgroup per CU (two at d = 64: LDS) and bound by bytes: cut to fill
    // the chip once, and not at all when it is full anyway - then only ranges
    // far above a CU's share.  A merge costs about 4 us, a workgroup's time for
    // 8 key tiles alone.  16 requests x 300..4100 keys x 8 heads: uncut 45.9 us,
    // 2 pieces each 35.6, 4 pieces 33.7, cut to 256 items 31.5; 320 ranges of
    // 1000..4000 keys: uncut 72.6 us, cut to two rounds 77.9.
    // Ranges of a CU's time for 12 tiles and less end sooner whole: decode steps of 10
    // tiles x 8 heads, d = 128, in two or three pieces -> whole: 8 ranges 8.6 -> 7.9, 32
    // 10.3 -> 8.0; d = 64: 36 of up to 9 tiles 6.6 -> 5.6, 192 of 10 10.8 -> 8.1; of 16
    // tiles and more 6.8 -> 7.5 and, at d = 128, 9.3 -> 11.0.  Nor are row tiles of 16
    // cut, which are chosen for what they take whole.  A caller who names the
    // smallest piece gets pieces.
    if (!asked && (in_tiles || costs[0].tiles <= 12)) return SplitRule{};
    const int64_t slots = (d == 64 ? 2 : 1) * kNumCU;
    if (n <= slots) return fit(costs, heads, min_chunk, 4, slots);
    const int chunk = (int)std::max<int64_t>(min_chunk, total / slots);
    return SplitRule{chunk, chunk, min_chunk};
  }
  // Waves that fill the chip several times are left alone but for extreme ranges.
  if (n > 4 * kNumCU) {
    const int chunk = (int)std::max<int64_t>(min_chunk, (total + 3 * kNumCU - 1) / (3 * kNumCU));
    return SplitRule{chunk, chunk, min_chunk};
  }
  // For the others the least estimate decides, of no cuts and of those into at
  // most one to four workgroups per CU, of the chip and of the dies that the row tiles
  // go to, where those are fewer (a few more would wait for a round of their own).  In us: the
  // longest piece takes `alone` per key tile, a CU that is never idle `busy`;
  // cutting adds the launch of the merge, the serial reads of the group with the
  // most pieces and, for 128 rows of partials, `partials` to write and read them.
  // (At d = 64, with more workgroups on a CU, the time on all CUs was closer than
  // that on those reached.)  Constants from 149 waves of 3 to 1000 row tiles of 8
  // to 470 key tiles, each timed with up to 20 chunks.  Against one set of constants
  // for both head dims without the terms for the merge, of 206 waves of 10 us and
  // more 18 take 3 to 25 % less and two 4 % more.  (34 rows x 15.9k keys, 8/1 heads,
  // d = 64: 50 pieces a group 38.8 us, 21 pieces 27.8, 4 pieces 44.8; 140 row tiles
  // of 15 key tiles on two dies, d = 128: cut 58.1 us, uncut 45.5; dealt out to eight, cut
  // 22.6, uncut 25.8.)
  const double alone = d == 64 ? 0.7 : 1.2, busy = d == 64 ? 0.47 : 0.95, partials = d == 64 ? 0.015 : 0.04;
  const int64_t reached = (int64_t)dies * (kNumCU / kNumXCD);
  const int cus = d == 64 ? kNumCU : (int)reached;
  auto longest_piece = [&](const SplitRule &r) {
    int longest = 0;
    for (const auto &c : costs) {
      const int k = r.pieces(c.tiles);
      longest = std::max(longest, (c.tiles + k - 1) / k);
    }
    return longest;
  };
  auto estimate = [&](const SplitRule &r) {
    int64_t rows = 0;
    int most = 1;
    for (const auto &c : costs) {
      const int k = r.pieces(c.tiles);
      if (k > 1) rows += c.rows * k * heads;
      most = std::max(most, k);
    }
    return std::max(alone * longest_piece(r), busy * (double)makespan(costs, heads, r, cus)) +
           (most > 1 ? 3.5 + 0.5 * most + partials * rows / 128 : 0.0);
  };
  SplitRule best;
  double best_time = estimate(best);
  for (int64_t items : {reached, 2 * reached, (int64_t)kNumCU, (int64_t)2 * kNumCU, (int64_t)3 * kNumCU, (int64_t)4 * kNumCU}) {
    const SplitRule r = fit(costs, heads, min_chunk, 6, items);
    const double t = estimate(r);
    if (t < best_time) {
      best_time = t;
      best = r;
    }
  }
  return best;
}

// Whether a wave with at most `rows` packed rows per (request, kv head), on
// `ranges` key ranges of `tiles` key tiles on average, goes to the kernel whose
// waves split the keys.  Up to 32 rows - decode steps, short suffixes - its work
// is bound by bytes or latency, not by the matrix cores, and that kernel keeps
// every wave busy.  But it holds a CU alone (half of one at d = 64), so ranges
// beyond those places wait for the first to end, which the prefill kernel's two
// and three workgroups per CU take better unless the ranges are long.  Time of
// that kernel over the prefill kernel's on waves of 1.9 to 10 times as many ranges
// as places (357 waves in all), by the mean length of the ranges:
//   key tiles                 1         2         3         6         15        41
//   d = 128, 1..16 rows    1.4..1.7  1.2..1.5  1.1..1.3  1.0..1.2  .95..1.0  .90..1.0
//            17..32 rows   1.7..2.0  1.6..1.8  1.4..1.5  1.1..1.3  1.0..1.1  .92..1.0
//   d = 64,  1..16 rows    1.1..1.2  1.1       1.0       .93..1.0  .97..1.0  .98
//            17..32 rows   1.5       1.3..1.4  1.1       .97..1.1  1.0       1.0
// With no more ranges than places: 0.63..1.0 up to 16 rows, 0.82..1.3 and 1.0 on
// average above.  (27 requests of 1..18 rows x 12..89 keys, 40 heads,
// d = 128: 25.4 -> 14.9 us.)  With 33..64 rows the prefill kernel is ahead (160
// ranges of up to 300 keys, 40 heads: 11.2 us against 13.3).
bool splits_keys(int64_t rows, int64_t ranges, int64_t tiles, int d) {
  if (rows > kStreamRows) return false;
  if (ranges <= (d == 64 ? 2 : 1) * kNumCU) return true;
  return tiles >= (rows <= 16 ? (d == 64 ? 4 : 11) : (d == 64 ? 16 : 32));
}

// Whether a wave of more rows goes to that kernel in row tiles of 16: if they all find
// a place at once, on the die of their (cluster, kv head) set, and the longest range is
// short enough to be read by four waves alone.  `sets` has the costs of the tiles of
// one kv head by cluster, `longest` the most key tiles.  Time of that kernel over the
// prefill kernel's, with its cuts, on 300 waves of 2 to 1400 such tiles:
//   key tiles               1     2     3..4   5..8   9..12  13..16  17..20  21..26
//   d = 128, with a place  .97   .81    .76    .72     .70   .73..97  .75..82  .96..1.3
//            2 to 4 a place 1.8  2.2    1.5    1.4     1.5    1.5     1.8     1.5
//   d = 64,  with a place 1.00   .99    .86    .69     .61    .68     .77     .74..1.0
//            1.5 a place          -     1.05  .83..1.2 .76..97 -      .94      -
// (Sets that a die has no room for, 668 rows x 2 heads: 1.5.)  With 17 to 32 rows it
// is ahead of a workgroup for all of them too: 4 ranges of 26 rows x 10 tiles, d = 64,
// 9.9 -> 5.7, 24 of 24 rows x 6 tiles, d = 128, 9.1 -> 6.6.
bool fits_in_row_tiles(std::vector<std::pair<int64_t, int64_t>> sets, int heads, int longest, int d) {
  if (longest > (d == 64 ? 22 : 20)) return false;
  const int64_t places = (d == 64 ? 2 : 1) * kNumCU / kNumXCD;
  std::sort(sets.rbegin(), sets.rend());             // dealt as build_schedule deals them
  int64_t load[kNumXCD] = {0}, taken[kNumXCD] = {0};
  for (const auto &set : sets)
    for (int h = 0; h < heads; ++h) {
      int die = 0;
      for (int x = 1; x < kNumXCD; ++x)
        if (load[x] < load[die]) die = x;
      load[die] += set.first;
      taken[die] += set.second;
      if (taken[die] > places) return false;
    }
  return true;
}

// Deals workgroups to the dies, set by set: a set begins on the die with the least so
// far, and one that is dealt out goes on on another whenever its die is full.  us per
// pass, a dozen whole row tiles on every die it reaches -> this: 8/1 heads, d = 64, one
// request of 800 new over 30000 cached tokens (50 row tiles: five dies -> eight) 111.0 -> 62.6,
// of 1300 126.7 -> 107.0, 1000 over 8192 43.7 -> 32.8; d = 128, 800 over 8192 59.3 -> 44.9, 960
// over 16384 116.9 -> 72.0, 900 over none 16.12 -> 16.25.
struct Dealer {
  int64_t wave;                                      // key tiles of all row tiles and kv heads
  int die = 0;
  int64_t load[kNumXCD] = {0};
  int64_t run = 0, run_cost = 0;                     // row tiles begun on this die since, and key tiles dealt to it
  void open() {
    die = 0;
    for (int x = 1; x < kNumXCD; ++x)
      if (load[x] < load[die]) die = x;
    run = run_cost = 0;
  }
  // It has an eighth of the wave, and of this set a dozen row tiles, which share what
  // they read, or half of that eighth, where that is less.
  bool full() const { return load[die] * kNumXCD >= wave && (run >= 12 || run_cost * 2 * kNumXCD >= wave); }
  void take(int cost) {
    load[die] += cost;
    run_cost += cost;
  }
};

// Whether some request's cached prefix lies in pages that the same wave appends
// to (pages published to later requests of the wave before they are written), or
// a page is appended to through two table entries.  Attention then has to run
// after the whole append.  Looks at the wave's own pages only: the appended ones
// form an open-addressing set, and a bitmap over the same hashes answers for
// nearly all of the cached ones.  (An array over the whole pool made this the
// larger part of a plan: 16 decode requests in a pool of 1 Mi pages took 192 us,
// now 21.)
bool reads_pages_of_this_wave(const prism_shape_t &s, const int32_t *prefix, const int32_t *suffix,
                              const int32_t *table) {
  auto row = [&](int r) { return table + (size_t)r * s.max_blocks_per_req; };
  auto in_pool = [&](int32_t page) { return page >= 0 && page < s.num_pages; };
  size_t entries = 0;
  for (int r = 0; r < s.batch; ++r)
    if (suffix[r] > 0) entries += (prefix[r] % kPage + suffix[r] + kPage - 1) / kPage;
  int bits = 4;                                    // the set has 2^bits places, the bitmap 4 bits for each
  while (((size_t)1 << bits) < 4 * entries) ++bits;
  std::vector<int32_t> appended((size_t)1 << bits, -1);
  std::vector<uint64_t> marked((size_t)1 << (bits - 4), 0);
  auto hash = [&](int32_t page) { return (uint32_t)page * 0x9E3779B1u >> (30 - bits); };
  auto place_of = [&](int32_t page) {              // where the page is, or where it would go
    size_t i = hash(page) >> 2;
    while (appended[i] != -1 && appended[i] != page) i = (i + 1) & (appended.size() - 1);
    return i;
  };
  for (int r = 0; r < s.batch; ++r) {
    if (suffix[r] == 0) continue;
    for (int b = prefix[r] / kPage; b <= (prefix[r] + suffix[r] - 1) / kPage; ++b) {
      const int32_t page = row(r)[b];
      if (!in_pool(page)) return true;
      int32_t &place = appended[place_of(page)];
      if (place == page) return true;
      place = page;
      marked[hash(page) >> 6] |= (uint64_t)1 << (hash(page) & 63);
    }
  }
  for (int r = 0; r < s.batch; ++r) {
    if (suffix[r] == 0) continue;
    for (int b = 0; b < prefix[r] / kPage; ++b) {
      const int32_t page = row(r)[b];
      if (!in_pool(page)) return true;
      if ((marked[hash(page) >> 6] >> (hash(page) & 63) & 1) && appended[place_of(page)] == page) return true;
    }
  }
  return false;
}

// Whether the tables of `requests` name more than `limit` different pages.  Stops
// looking there: the set, open addressing again, stays at most half full.  What a
// request's table has in common with the first of its cluster, which is one of them
// too, is compared and not looked up (a plan of 63 requests sharing 1000 pages:
// 226 us, now 154, without the count 133).
bool distinct_pages_exceed(const prism_shape_t &s, const std::vector<int> &requests, const std::vector<int> &cluster,
                           const int32_t *prefix, const int32_t *suffix, const int32_t *table, int64_t limit) {
  auto row = [&](int r) { return table + (size_t)r * s.max_blocks_per_req; };
  auto pages = [&](int r) { return (prefix[r] + suffix[r] + kPage - 1) / kPage; };
  int64_t entries = 0, distinct = 0;
  for (int r : requests) entries += pages(r);
  if (entries <= limit) return false;
  int bits = 4;
  while (((int64_t)1 << bits) < 2 * (limit + 1)) ++bits;
  std::vector<int32_t> seen((size_t)1 << bits, -1);
  for (int r : requests) {
    const int first = cluster[r];
    const int32_t *page = row(r), *end = page + pages(r);
    if (r != first) {
      constexpr int kRun = 16;
      const int common = std::min(pages(r), pages(first));
      for (int b = 0; b + kRun <= common && !std::memcmp(row(r) + b, row(first) + b, kRun * sizeof *page); b += kRun) page += kRun;
    }
    for (; page < end; ++page) {
      if (*page < 0) continue;
      size_t i = (uint32_t)*page * 0x9E3779B1u >> (32 - bits);
      while (seen[i] != -1 && seen[i] != *page) i = (i + 1) & (seen.size() - 1);
      if (seen[i] == *page) continue;
      if (++distinct > limit) return true;
      seen[i] = *page;
    }
  }
  return false;
}

}  // namespace

int build_schedule(const prism_shape_t &s, const int32_t *prefix, const int32_t *suffix,
                   const prism_plan_options_t &opt, Schedule *out) {
  int rc = check_shape(s);
  if (rc != PRISM_OK) return rc;
  const int G = s.num_q_heads / s.num_kv_heads;
  int tile_rows = opt.tile_rows ? opt.tile_rows : 128;
  if (tile_rows != 64 && tile_rows != 128 && tile_rows != 256) return PRISM_ERR_UNSUPPORTED;
  const int rows_per_wave = opt.rows_per_wave ? opt.rows_per_wave : 32;
  if (rows_per_wave != 32 && rows_per_wave != 64) return PRISM_ERR_UNSUPPORTED;
  if (rows_per_wave == 64 && tile_rows == 64) return PRISM_ERR_UNSUPPORTED;
  if (opt.split_kv < 0 || opt.min_split_keys < 0 || opt.min_split_keys % kTileKeys != 0)
    return PRISM_ERR_UNSUPPORTED;
  const int d = s.head_dim;
  const int64_t token_bytes = 2LL * 2 * d * s.num_kv_heads;   // K and V

  Schedule sch;
  std::vector<int32_t> q_off(s.batch);
  int64_t total = 0;
  int64_t most_rows = 0;       // packed rows of the largest request, per kv head
  int64_t ranges = 0, range_tiles = 0;   // requests with rows, and the key tiles of their sequences
  int64_t row_tiles = 0;       // of 16 packed rows, per kv head
  for (int r = 0; r < s.batch; ++r) {
    const int64_t P = prefix[r], S = suffix[r];
    if (P < 0 || S < 0) return PRISM_ERR_INVALID_ARG;
    if (P + S > (int64_t)kPage * s.max_blocks_per_req) return PRISM_ERR_INVALID_ARG;
    if (total + S > INT32_MAX / 2) return PRISM_ERR_INVALID_ARG;
    if (S * s.num_kv_heads * (d / 8) > INT32_MAX / 2) return PRISM_ERR_INVALID_ARG;   // 16-byte units of one request
    q_off[r] = (int32_t)total;
    total += S;
    sch.flops += 4LL * d * s.num_q_heads * (S * P + S * (S + 1) / 2);
    if (S > 0) {
      sch.kv_bytes += token_bytes * (P + S);
      most_rows = std::max(most_rows, S * G);
      row_tiles += (S * G + 15) / 16;
      ++ranges;
      range_tiles += (P + S + kTileKeys - 1) / kTileKeys;
    }
  }
  sch.total_suffix = total;

  // Requests that share a cached prefix start with the same page: give them
  // one cluster id (the smallest request index of the cluster).
  std::vector<int> cluster(s.batch);
  for (int r = 0; r < s.batch; ++r) cluster[r] = r;
  if (opt.block_table_host) {
    std::map<int32_t, int> first_page_owner;
    for (int r = 0; r < s.batch; ++r) {
      if (prefix[r] < kPage || suffix[r] == 0) continue;       // no whole cached page
      const int32_t pg = opt.block_table_host[(size_t)r * s.max_blocks_per_req];
      auto ins = first_page_owner.insert({pg, r});
      cluster[r] = ins.first->second;
    }
  }

  // More than 16 rows, in tiles of 16 rows each.
  bool in_tiles = false;
  const int64_t places = (d == 64 ? 2 : 1) * kNumCU;
  if (!opt.tile_rows && !opt.rows_per_wave && most_rows > 16 && row_tiles * s.num_kv_heads <= places) {
    std::map<int, std::pair<int64_t, int64_t>> by_cluster;
    int longest = 0;
    for (int r = 0; r < s.batch; ++r)
      for (int rows = suffix[r] * G, row0 = 0; row0 < rows; row0 += 16) {
        const int cost = key_tiles(prefix[r] + (std::min(rows, row0 + 16) - 1) / G + 1);
        auto &set = by_cluster[cluster[r]];
        set.first += cost;
        ++set.second;
        longest = std::max(longest, cost);
      }
    std::vector<std::pair<int64_t, int64_t>> sets;
    for (const auto &c : by_cluster) sets.push_back(c.second);
    in_tiles = fits_in_row_tiles(std::move(sets), s.num_kv_heads, longest, d);
  }
  const bool stream = in_tiles || (!opt.tile_rows && !opt.rows_per_wave &&
                                   splits_keys(most_rows, ranges * s.num_kv_heads, ranges ? range_tiles / ranges : 0, d));
  if (stream) tile_rows = in_tiles || most_rows <= 16 ? 16 : 32;
  sch.stream = stream;
  sch.tile_rows = tile_rows;
  sch.rows_per_wave = stream ? tile_rows : rows_per_wave;
  // Both kernels that do it take 32 rows a wave at most.
  sch.fused_append = (stream || rows_per_wave == 32) && opt.block_table_host && opt.table_is_final &&
                     !reads_pages_of_this_wave(s, prefix, suffix, opt.block_table_host);

  sch.q_off = q_off;

  // Row tiles, the same for every kv head: the keys that each one sees, by request.
  // (Everything up to the items is done once for all kv heads: with a list of all
  // (request, kv head, row tile) sorted as a whole, the plan of 32 requests x 40
  // heads took 441 us, now 108.)
  std::vector<int> first_tile(s.batch + 1, 0), tile_keys;
  std::vector<int64_t> cluster_cost(s.batch, 0);       // key tiles of the cluster, of one kv head
  std::vector<int> live, sharers(s.batch, 0);          // requests with rows; how many of them are in the cluster
  int most_cost = 0;
  int64_t clusters = 0;
  for (int r = 0; r < s.batch; ++r) {
    const int P = prefix[r], S = suffix[r];
    const int rows = S * G;
    if (S > 0) {
      live.push_back(r);
      ++sharers[cluster[r]];
    }
    clusters += S > 0 && cluster[r] == r;
    for (int row0 = 0; row0 < rows; row0 += tile_rows) {
      const int kv_len = P + (std::min(rows, row0 + tile_rows) - 1) / G + 1;
      tile_keys.push_back(kv_len);
      cluster_cost[cluster[r]] += key_tiles(kv_len);
      most_cost = std::max(most_cost, key_tiles(kv_len));
    }
    first_tile[r + 1] = (int)tile_keys.size();
  }

  // Heaviest cluster first, and of equal ones, where fits_in_row_tiles has counted on
  // that, the one of more row tiles; inside a (cluster, kv head) set the requests, the
  // longest first, and inside a request the row tiles, stay adjacent so that they
  // run at the same time and find each other's K/V pages in cache.
  std::vector<int64_t> set_tiles(s.batch, 0);          // row tiles of a cluster, of one kv head
  for (int r : live) set_tiles[cluster[r]] += first_tile[r + 1] - first_tile[r];
  std::sort(live.begin(), live.end(), [&](int a, int b) {
    const int ca = cluster[a], cb = cluster[b];
    if (ca != cb) {
      if (cluster_cost[ca] != cluster_cost[cb]) return cluster_cost[ca] > cluster_cost[cb];
      return in_tiles && set_tiles[ca] != set_tiles[cb] ? set_tiles[ca] > set_tiles[cb] : ca < cb;
    }
    const int ka = key_tiles(prefix[a] + suffix[a]), kb = key_tiles(prefix[b] + suffix[b]);
    return ka != kb ? ka > kb : a < b;
  });

  // A (cluster, kv head) set of more row tiles than one and a half for each CU of a die
  // is dealt to as many dies as it takes to give each an eighth of the wave: with
  // fewer sets than dies, or a few more, most of the chip waited for those that had
  // them, and what the others read again is little beside that.  us per pass, whole ->
  // dealt out: 8/1 heads, d = 64, one request of 4096 new 126.6 -> 33.0, 3 of 1648..3297 over
  // 18612 cached tokens 916 -> 354, 9 of 2500..3000 over 100..3000 199 -> 173, 12 of 1300 over
  // 500 61.2 -> 47.6; 8/2 heads, d = 128, 3 of 2685 over 373 80.3 -> 63.6, one of 1800 34.0 -> 21.9,
  // one of 1700 over 8000 228 -> 83.  Smaller sets keep their die, as most waves have
  // many (33 to 44 tiles would gain 1.05 to 1.5 where they are alone, 17 to 32 up to 1.7).
  const int64_t die_tiles = kNumCU / kNumXCD * 3 / 2;
  int64_t wave_cost = 0;                               // key tiles of all kv heads
  for (int c = 0; c < s.batch; ++c) wave_cost += cluster_cost[c] * s.num_kv_heads;
  auto dealt_out = [&](int c) { return !stream && set_tiles[c] > die_tiles; };
  // The dies that the wave reaches, for the cuts: as many as it has sets, and those that
  // the row tiles of sets dealt out go to, of one request or of several that share a
  // prefix.  us per pass of the latter, cut as if each set had one die -> this: 8/1 heads,
  // d = 128, 8 of 120 new over 16384 shared tokens 192.9 -> 69.1; 8/2 heads, 8 of 200 over 8192
  // 103.0 -> 61.6, two of 1000 114.4 -> 91.7, 4 of 500 over 2000 36.1 -> 29.7, two of 1500 over
  // 1000 38.4 -> 39.7.
  auto dies_reached = [&]() -> int {
    if (clusters * s.num_kv_heads >= kNumXCD) return kNumXCD;
    Dealer to{wave_cost};
    for (size_t i = 0, j; i < live.size(); i = j) {
      for (j = i; j < live.size() && cluster[live[j]] == cluster[live[i]];) ++j;
      for (int h = 0; h < s.num_kv_heads; ++h) {
        to.open();
        for (size_t m = i; m < j; ++m)
          for (int tile = first_tile[live[m] + 1] - 1; tile >= first_tile[live[m]]; --tile) {
            if (dealt_out(cluster[live[i]]) && to.full()) to.open();
            ++to.run;
            to.take(key_tiles(tile_keys[tile]));
          }
      }
    }
    return kNumXCD - (int)std::count(to.load, to.load + kNumXCD, 0);
  };

  // Split-KV: no piece of the automatic cuts has fewer key tiles than a caller's
  // min_split_keys; without one, all but the last of a range have four.
  const int min_chunk = std::max(1, (opt.min_split_keys ? opt.min_split_keys : 256) / kTileKeys);
  SplitRule rule;
  Costs costs;
  if (opt.split_kv == 0 && !tile_keys.empty()) {
    std::vector<int64_t> count(most_cost + 1, 0), rows(most_cost + 1, 0);
    for (int r : live)
      for (int t = first_tile[r]; t < first_tile[r + 1]; ++t) {
        const int c = key_tiles(tile_keys[t]);
        ++count[c];
        rows[c] += std::min(tile_rows, suffix[r] * G - (t - first_tile[r]) * tile_rows);
      }
    for (int c = most_cost; c > 0; --c)
      if (count[c]) costs.push_back({c, count[c], rows[c]});
    rule = choose_split(costs, s.num_kv_heads, dies_reached(), min_chunk, opt.min_split_keys != 0, stream, in_tiles, d);
  }

  // The key-splitting kernel reads every key of an item once: pages of one request
  // alone, whose rows are one tile, can pass the caches by, if the wave is more than those of the dies hold
  // (8 x 4 MB), a page counting once however many requests share it.  us per pass,
  // kept -> passed by, with more pools in rotation than the 256 MB memory-side cache
  // holds, as in a model whose layers have a pool each | on one pool again and again;
  // one new token a request, d = 128 but where said:
  //   20 MB (16 x 300 keys, 8 heads)     8.10 ->  7.98 |  6.26 ->  6.37
  //   34 MB (16 x 500)                   9.96 ->  9.60 |  7.48 ->  8.16
  //   46 MB (16 x 700)                  13.65 -> 12.63 | 11.95 -> 10.57
  //   66 MB (16 x 1000)                 16.82 -> 15.46 | 14.95 -> 13.13
  //   155 MB (16 x 300..4100)           32.31 -> 29.49 | 26.76 -> 27.39
  //   5.4 GB (64 x 4096, 40 heads)     897 -> 808
  //   33 MB (16 x 1000, d = 64)         11.24 -> 10.84 |  8.02 ->  8.62
  // Below the line the gain on pools in rotation (2 %) is no more than the cost on
  // one that the step before left in the caches (8 new tokens a request would gain
  // there already: 21 MB 11.13 -> 10.42 | 9.27 -> 9.08).  Pages that several share
  // are kept: passed by, 32 requests x 4096 keys x 40 heads that share by two, eight
  // and 32 took 258 -> 270, 168 -> 190 and 156 -> 162.
  bool reads_once = stream && opt.block_table_host && sch.kv_bytes > kCacheBytes;
  if (reads_once) {
    int64_t own = 0;                                 // bytes of requests that share no prefix
    for (int r : live)
      if (sharers[cluster[r]] == 1) own += (int64_t)(prefix[r] + suffix[r]) * token_bytes;
    if (own <= kCacheBytes) {
      std::vector<int> sharing;
      for (int r : live)
        if (sharers[cluster[r]] > 1) sharing.push_back(r);
      const int64_t room = (kCacheBytes - own) / (kPage * token_bytes);
      reads_once = own > 0 && distinct_pages_exceed(s, sharing, cluster, prefix, suffix, opt.block_table_host, room);
    }
  }

  auto deal = [&](const SplitRule &rule) {
    sch.items.clear();
    sch.groups.clear();
    sch.num_split_items = 0;
    sch.read_once = false;
    sch.most_pieces = 0;
    // Workgroup b runs on accelerator die b % 8, and each die has its own L2.
    // Row tiles (and key chunks) of one (request, kv head), and of requests with
    // a common cached prefix, read the same K/V pages, so each (cluster, kv
    // head) set is dealt to one die, or to several where it is larger than one -
    // the least loaded so far, heaviest sets first - and the per-die lists are then
    // interleaved so that list position k of die x becomes workgroup 8k + x.
    struct ItemSet {                 // the workgroups of one (cluster, kv head) on one die
      int longest;                   // keys of the longest
      size_t begin, end;
    };
    std::vector<ItemSet> die_sets[kNumXCD];
    std::vector<AttnItem> die_items[kNumXCD];
    Dealer to{wave_cost};
    int next_slot = 0;
    for (size_t i = 0, j; i < live.size(); i = j) {
      j = i;
      while (j < live.size() && cluster[live[j]] == cluster[live[i]]) ++j;
      for (int h = 0; h < s.num_kv_heads; ++h) {
        ItemSet set{};
        std::vector<AttnItem> *items = nullptr;
        // (calls of their own would make the plan of 32 requests x 40 heads 13 % longer)
        auto open = [&]() __attribute__((always_inline)) {
          to.open();
          items = &die_items[to.die];
          set = ItemSet{0, items->size(), 0};
        };
        auto close = [&]() __attribute__((always_inline)) {
          set.end = items->size();
          die_sets[to.die].push_back(set);
        };
        const bool out = dealt_out(cluster[live[i]]);
        auto add = [&](const AttnItem &it) __attribute__((always_inline)) {
          if (out) {
            if (to.full()) {
              close();
              open();
            }
            to.run += it.kv_begin == 0;
            to.take(key_tiles(it.kv_end - it.kv_begin));
          }
          set.longest = std::max(set.longest, it.kv_end - it.kv_begin);
          items->push_back(it);
        };
        open();
        for (size_t m = i; m < j; ++m)
          for (int tile = first_tile[live[m] + 1] - 1; tile >= first_tile[live[m]]; --tile) {
            const int req = live[m], kv_len = tile_keys[tile], cost = key_tiles(kv_len);
            if (!out) to.take(cost);
            int nsplit = 1;
            if (opt.split_kv > 1) nsplit = std::min(opt.split_kv, cost);
            else if (opt.split_kv == 0) nsplit = rule.pieces(cost);
            AttnItem it{};
            it.req = req;
            it.kv_head = h;
            it.row0 = (tile - first_tile[req]) * tile_rows;
            it.prefix = prefix[req];
            it.suffix = suffix[req];
            it.q_off = q_off[req];
            it.read_once = reads_once && j - i == 1 && first_tile[req + 1] - first_tile[req] == 1;
            sch.read_once |= it.read_once != 0;
            if (nsplit <= 1) {
              it.kv_begin = 0;
              it.kv_end = kv_len;
              it.part_slot = -1;
              add(it);
              continue;
            }
            // Pieces of one length and a last one with what they leave: it also has the
            // causal diagonal and the append (3 requests of 1200 to 2100 new over 112
            // cached tokens, d = 64: 21.0 us, with a last piece of at least 4 tiles 22.1),
            // and groups that end at different times share the merging.  Where the
            // caller's limit forbids that, pieces that differ by one key tile at most.
            const int per = (cost + nsplit - 1) / nsplit;
            nsplit = (cost + per - 1) / per;
            const bool even = opt.min_split_keys && cost - (nsplit - 1) * per < rule.least;
            auto tile_of = [&](int piece) {
              return even ? cost / nsplit * piece + std::min(piece, cost % nsplit) : std::min(cost, piece * per);
            };
            ReduceGroup g{};
            g.req = req;
            g.kv_head = h;
            g.row0 = it.row0;
            g.nsplit = nsplit;
            sch.most_pieces = std::max(sch.most_pieces, nsplit);
            g.first_slot = next_slot;
            g.suffix = suffix[req];
            g.q_off = q_off[req];
            it.group = (int32_t)sch.groups.size();
            sch.groups.push_back(g);
            for (int c = 0; c < nsplit; ++c) {
              it.kv_begin = tile_of(c) * kTileKeys;
              it.kv_end = std::min(kv_len, tile_of(c + 1) * kTileKeys);
              it.part_slot = next_slot++;
              add(it);
              ++sch.num_split_items;
            }
          }
        close();
      }
    }
    // The sets of a die start in the order of their longest workgroup: a long one
    // that starts late runs on alone.  (In the order of total work, in which they
    // are dealt, a request of few rows over a long prefix comes last.)  For the
    // same reason the last two workgroups per CU go strictly longest first; the
    // ones before them keep the order of the sets, whose pages they share.
    // (12 requests of 200..512 rows x 130..3000 keys, 32/8 heads, d = 64: 95.7 ->
    // 90.0 us; the 4B-class wave 145.7 -> 139.4; waves of many rounds unchanged.)
    std::vector<uint32_t> per_die[kNumXCD];           // positions in die_items
    std::vector<std::pair<int, uint32_t>> keys;        // (-keys, position): longest first, else in order
    size_t longest = 0;
    for (int x = 0; x < kNumXCD; ++x) {
      std::vector<uint32_t> &order = per_die[x];
      order.reserve(die_items[x].size());
      std::stable_sort(die_sets[x].begin(), die_sets[x].end(),
                       [](const ItemSet &a, const ItemSet &b) { return a.longest > b.longest; });
      for (const ItemSet &set : die_sets[x])
        for (size_t k = set.begin; k < set.end; ++k) order.push_back((uint32_t)k);
      const size_t tail = std::min(order.size(), (size_t)2 * kNumCU / kNumXCD), head = order.size() - tail;
      keys.clear();
      for (size_t k = 0; k < tail; ++k) {
        const AttnItem &it = die_items[x][order[head + k]];
        keys.push_back({it.kv_begin - it.kv_end, (uint32_t)k});
      }
      std::sort(keys.begin(), keys.end());
      const std::vector<uint32_t> last(order.begin() + head, order.end());
      for (size_t k = 0; k < tail; ++k) order[head + k] = last[keys[k].second];
      longest = std::max(longest, order.size());
    }
    AttnItem idle{};
    idle.req = -1;                 // the kernel returns at once on such an entry
    idle.part_slot = -1;
    sch.items.reserve(longest * kNumXCD);
    for (size_t k = 0; k < longest; ++k)
      for (int x = 0; x < kNumXCD; ++x)
        sch.items.push_back(k < per_die[x].size() ? die_items[x][per_die[x][k]] : idle);
    // drop idle entries at the very end of the list
    while (!sch.items.empty() && sch.items.back().req < 0) sch.items.pop_back();
    sch.num_slots = next_slot;
    sch.workspace_bytes = (size_t)next_slot * partial_slot_bytes(tile_rows, d);
  };
  deal(rule);
  // A plan of the library's own choosing fits the scratch of the entry that takes
  // no workspace whenever its uncut form does: it is cut less until it fits.
  // (Four rounds of 128-row pieces at d = 128, the most that the rule above
  // chooses, are 65 MiB of partials.)
  while (rule.chunk && sch.num_slots) {
    const size_t lists = lists_bytes(sch);
    if (lists + sch.workspace_bytes <= PRISM_STATIC_SCRATCH_BYTES) break;
    const size_t room = lists < PRISM_STATIC_SCRATCH_BYTES ? PRISM_STATIC_SCRATCH_BYTES - lists : 0;
    rule = coarser(costs, s.num_kv_heads, rule, (int64_t)(room / partial_slot_bytes(tile_rows, d)));
    deal(rule);
  }
  *out = std::move(sch);
  return PRISM_OK;
}

int validate_table(const prism_shape_t &s, const int32_t *prefix, const int32_t *suffix,
                   const int32_t *table) {
  int rc = check_shape(s);
  if (rc != PRISM_OK) return rc;
  if (!prefix || !suffix || !table) return PRISM_ERR_INVALID_ARG;
  std::set<int32_t> cached_pages;       // pages that hold some request's whole-page prefix
  std::map<int32_t, int> suffix_owner;  // page -> request writing into it
  std::set<std::pair<int32_t, int>> slots;
  for (int r = 0; r < s.batch; ++r) {
    const int64_t P = prefix[r], S = suffix[r];
    if (P < 0 || S < 0 || P + S > (int64_t)kPage * s.max_blocks_per_req) return PRISM_ERR_INVALID_ARG;
    const int nb = (int)((P + S + kPage - 1) / kPage);
    for (int b = 0; b < nb; ++b) {
      const int32_t pg = table[(size_t)r * s.max_blocks_per_req + b];
      if (pg < 0 || pg >= s.num_pages) return PRISM_ERR_TABLE;
    }
  }
  for (int r = 0; r < s.batch; ++r) {
    const int P = prefix[r], S = suffix[r];
    // Pages read by r that r does not write: every block wholly below P, and a
    // partial last prefix block only when r appends nothing.
    const int read_only = S > 0 ? P / kPage : (P + kPage - 1) / kPage;
    for (int b = 0; b < read_only; ++b) cached_pages.insert(table[(size_t)r * s.max_blocks_per_req + b]);
  }
  for (int r = 0; r < s.batch; ++r) {
    const int P = prefix[r], S = suffix[r];
    for (int i = 0; i < S; ++i) {
      const int pos = P + i;
      const int32_t pg = table[(size_t)r * s.max_blocks_per_req + pos / kPage];
      if (!slots.insert({pg, pos % kPage}).second) return PRISM_ERR_TABLE;
      auto it = suffix_owner.find(pg);
      if (it != suffix_owner.end() && it->second != r) return PRISM_ERR_TABLE;
      suffix_owner[pg] = r;
      if (cached_pages.count(pg)) return PRISM_ERR_TABLE;
    }
  }
  return PRISM_OK;
}

}  // namespace prism
