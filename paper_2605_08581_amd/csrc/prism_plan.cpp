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

struct RowTile {
  int req, kv_head, row0;
  int kv_len;      // keys visible to the tile's last row
  int cost;        // key tiles
  int group_cost;  // cost of the heaviest row tile of the same (request, kv head)
  int cluster;     // requests with a common cached prefix share a cluster
  int64_t cluster_cost;   // all key tiles of the (cluster, kv head) set
};

// How the key range of a row tile is cut: into pieces of about `chunk` key tiles,
// a range that exceeds it by no more than `slack` staying whole.
struct SplitRule {
  int chunk = 0, slack = 0;                        // chunk 0: never cut
  int pieces(int cost) const {
    return chunk ? std::max(1, std::min(cost, (cost - slack + chunk - 1) / chunk)) : 1;
  }
};

// Time, in key tiles, until `slots` workers have done all pieces, longest first.
int64_t makespan(const std::vector<int> &costs, int heads, const SplitRule &rule, int slots) {
  std::vector<std::pair<int, int64_t>> pieces;     // length, how many
  int64_t total = 0;
  for (int c : costs) {
    const int n = rule.pieces(c), len = (c + n - 1) / n;
    pieces.push_back({len, (int64_t)n * heads});
    total += (int64_t)n * heads * len;
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
SplitRule fit(const std::vector<int> &costs, int heads, int min_chunk, int slack, int64_t items) {
  int lo = min_chunk, hi = std::max(min_chunk, costs[0]);
  while (lo < hi) {
    const SplitRule mid{(lo + hi) / 2, slack};
    int64_t n = 0;
    for (int c : costs) n += mid.pieces(c);
    if (n * heads <= items) hi = mid.chunk;
    else lo = mid.chunk + 1;
  }
  return SplitRule{lo, slack};
}

SplitRule choose_split(const std::vector<int> &costs, int heads, int min_chunk, bool stream, int d) {
  int64_t total = 0;
  for (int c : costs) total += c;
  total *= heads;
  const int64_t n = (int64_t)costs.size() * heads;
  if (stream) {
    // One workgroup per CU (two at d = 64: LDS) and bound by bytes: cut to fill
    // the chip once, and not at all when it is full anyway - then only ranges
    // far above a CU's share.  A merge costs about 4 us, a workgroup's time for
    // 8 key tiles alone.  16 requests x 300..4100 keys x 8 heads: uncut 45.9 us,
    // 2 pieces each 35.6, 4 pieces 33.7, cut to 256 items 31.5; 320 ranges of
    // 1000..4000 keys: uncut 72.6 us, cut to two rounds 77.9.
    const int64_t slots = (d == 64 ? 2 : 1) * kNumCU;
    if (n <= slots) return fit(costs, heads, min_chunk, 4, slots);
    const int chunk = (int)std::max<int64_t>(min_chunk, total / slots);
    return SplitRule{chunk, chunk};
  }
  // The prefill kernel takes about 1.1 us per key tile alone on a CU and 1.9 us
  // beside a second workgroup; cutting costs another launch (5 us) and 0.02 us
  // of partials per piece.  Waves that fill the chip several times are left
  // alone but for extreme ranges; for the others the least estimate decides.
  // (148 rows x 1040 keys x 8 heads: 16 workgroups 20.0 us, 64 of them 14.8;
  // 3 requests of 100..300 rows x 1000..3300 keys, 8/2 heads: 31.4 -> 21.2 us.)
  if (n > 4 * kNumCU) {
    const int chunk = (int)std::max<int64_t>(min_chunk, (total + 3 * kNumCU - 1) / (3 * kNumCU));
    return SplitRule{chunk, chunk};
  }
  auto estimate = [&](const SplitRule &r) {
    int64_t cut = 0;
    int longest = 0;
    for (int c : costs) {
      const int k = r.pieces(c);
      longest = std::max(longest, (c + k - 1) / k);
      if (k > 1) cut += (int64_t)k * heads;
    }
    return std::max(1.1 * longest, 0.95 * (double)makespan(costs, heads, r, kNumCU)) + (cut ? 5.0 + 0.02 * cut : 0.0);
  };
  SplitRule best;
  double best_time = estimate(best);
  for (int64_t items : {1, 2, 3, 4}) {
    const SplitRule r = fit(costs, heads, min_chunk, 6, items * kNumCU);
    const double t = estimate(r);
    if (t < best_time) {
      best_time = t;
      best = r;
    }
  }
  return best;
}

// Whether some request's cached prefix lies in pages that the same wave appends
// to (pages published to later requests of the wave before they are written).
// Attention then has to run after the whole append.
bool reads_pages_of_this_wave(const prism_shape_t &s, const int32_t *prefix, const int32_t *suffix,
                              const int32_t *table) {
  std::vector<int32_t> writer(s.num_pages, -1);    // request that appends to the page, -2: several
  for (int pass = 0; pass < 2; ++pass)
    for (int r = 0; r < s.batch; ++r) {
      if (suffix[r] == 0) continue;
      const int32_t *row = table + (size_t)r * s.max_blocks_per_req;
      const int whole = prefix[r] / kPage, last = (prefix[r] + suffix[r] - 1) / kPage;
      for (int b = pass == 0 ? whole : 0; b <= (pass == 0 ? last : whole); ++b) {
        if (row[b] < 0 || row[b] >= s.num_pages) return true;
        int32_t &w = writer[row[b]];
        if (pass == 0) w = w == -1 || w == r ? r : -2;
        else if (b < whole ? w != -1 : w != r) return true;
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

  Schedule sch;
  std::vector<int32_t> q_off(s.batch);
  int64_t total = 0;
  int64_t most_rows = 0;       // packed rows of the largest request, per kv head
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
      sch.kv_bytes += 2LL * 2 * d * s.num_kv_heads * (P + S);
      most_rows = std::max(most_rows, S * G);
    }
  }
  sch.total_suffix = total;

  // Up to 32 packed rows per (request, kv head) - decode steps, short suffixes -
  // a wave's work is bound by bytes or latency, not by the matrix cores: the
  // kernel whose waves split the keys then keeps every wave busy.  With 33..64
  // rows the prefill kernel is ahead (40 heads x 160 ranges of up to 300 keys:
  // 11.2 us against 13.3; 17..32 rows: 9.9 against 9.0).
  const bool stream = !opt.tile_rows && !opt.rows_per_wave && most_rows <= kStreamRows;
  if (stream) tile_rows = most_rows <= 16 ? 16 : 32;
  sch.stream = stream;
  sch.tile_rows = tile_rows;
  sch.rows_per_wave = stream ? tile_rows : rows_per_wave;
  sch.fused_append = opt.block_table_host && !reads_pages_of_this_wave(s, prefix, suffix, opt.block_table_host);

  sch.q_off = q_off;

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

  // Row tiles of every (request, kv head).
  std::vector<RowTile> tiles;
  for (int r = 0; r < s.batch; ++r) {
    const int P = prefix[r], S = suffix[r];
    if (S == 0) continue;
    const int rows = S * G;
    const int ntile = (rows + tile_rows - 1) / tile_rows;
    for (int h = 0; h < s.num_kv_heads; ++h) {
      for (int t = 0; t < ntile; ++t) {
        const int last_row = std::min(rows, (t + 1) * tile_rows) - 1;
        const int kv_len = P + last_row / G + 1;
        const int cost = (kv_len + kTileKeys - 1) / kTileKeys;
        const int gmax = (P + S + kTileKeys - 1) / kTileKeys;
        tiles.push_back(RowTile{r, h, t * tile_rows, kv_len, cost, gmax, cluster[r], 0});
      }
    }
  }

  // Split-KV: never below min_split_keys.
  std::vector<int> costs;      // key tiles of each row tile of one kv head, descending
  for (const RowTile &t : tiles)
    if (t.kv_head == 0) costs.push_back(t.cost);
  std::sort(costs.rbegin(), costs.rend());
  const int min_chunk = std::max(1, (opt.min_split_keys ? opt.min_split_keys : 256) / kTileKeys);
  const SplitRule rule = opt.split_kv == 0 && !costs.empty()
                             ? choose_split(costs, s.num_kv_heads, min_chunk, stream, d)
                             : SplitRule{};

  // Heaviest (cluster, kv head) set first; inside a set the requests, and
  // inside a request the row tiles, stay adjacent so that they run at the same
  // time and find each other's K/V pages in cache.
  {
    std::map<std::pair<int, int>, int64_t> set_cost;
    for (const RowTile &t : tiles) set_cost[{t.cluster, t.kv_head}] += t.cost;
    for (RowTile &t : tiles) t.cluster_cost = set_cost[{t.cluster, t.kv_head}];
  }
  std::stable_sort(tiles.begin(), tiles.end(), [](const RowTile &a, const RowTile &b) {
    if (a.cluster_cost != b.cluster_cost) return a.cluster_cost > b.cluster_cost;
    if (a.cluster != b.cluster) return a.cluster < b.cluster;
    if (a.kv_head != b.kv_head) return a.kv_head < b.kv_head;
    if (a.group_cost != b.group_cost) return a.group_cost > b.group_cost;
    if (a.req != b.req) return a.req < b.req;
    return a.row0 > b.row0;
  });

  // Workgroup b runs on accelerator die b % 8, and each die has its own L2.
  // Row tiles (and key chunks) of one (request, kv head), and of requests with
  // a common cached prefix, read the same K/V pages, so each (cluster, kv
  // head) set is dealt whole to one die - the least loaded so far, heaviest
  // sets first - and the per-die lists are then interleaved so that list
  // position k of die x becomes workgroup 8k + x.
  struct ItemSet {                 // the workgroups of one (cluster, kv head)
    int longest = 0;               // keys of the longest
    std::vector<AttnItem> items;
  };
  std::vector<ItemSet> die_sets[kNumXCD];
  int64_t die_load[kNumXCD] = {0};
  int next_slot = 0;
  size_t i = 0;
  while (i < tiles.size()) {
    size_t j = i;
    int64_t group_cost = 0;
    while (j < tiles.size() && tiles[j].cluster == tiles[i].cluster && tiles[j].kv_head == tiles[i].kv_head)
      group_cost += tiles[j++].cost;
    int die = 0;
    for (int x = 1; x < kNumXCD; ++x)
      if (die_load[x] < die_load[die]) die = x;
    die_load[die] += group_cost;
    die_sets[die].emplace_back();
    ItemSet &set = die_sets[die].back();
    auto add = [&](const AttnItem &it) {
      set.longest = std::max(set.longest, it.kv_end - it.kv_begin);
      set.items.push_back(it);
    };
    for (; i < j; ++i) {
      const RowTile &t = tiles[i];
      int nsplit = 1;
      if (opt.split_kv > 1) nsplit = std::min(opt.split_kv, t.cost);
      else if (opt.split_kv == 0) nsplit = rule.pieces(t.cost);
      AttnItem it{};
      it.req = t.req;
      it.kv_head = t.kv_head;
      it.row0 = t.row0;
      it.prefix = prefix[t.req];
      it.suffix = suffix[t.req];
      it.q_off = q_off[t.req];
      if (nsplit <= 1) {
        it.kv_begin = 0;
        it.kv_end = t.kv_len;
        it.part_slot = -1;
        add(it);
        continue;
      }
      const int per = (t.cost + nsplit - 1) / nsplit;   // key tiles per chunk
      nsplit = (t.cost + per - 1) / per;
      ReduceGroup g{};
      g.req = t.req;
      g.kv_head = t.kv_head;
      g.row0 = t.row0;
      g.nsplit = nsplit;
      g.first_slot = next_slot;
      g.suffix = suffix[t.req];
      g.q_off = q_off[t.req];
      it.group = (int32_t)sch.groups.size();
      sch.groups.push_back(g);
      for (int c = 0; c < nsplit; ++c) {
        it.kv_begin = c * per * kTileKeys;
        it.kv_end = std::min(t.kv_len, (c + 1) * per * kTileKeys);
        it.part_slot = next_slot++;
        add(it);
        ++sch.num_split_items;
      }
    }
  }
  // The sets of a die start in the order of their longest workgroup: a long one
  // that starts late runs on alone.  (In the order of total work, in which they
  // are dealt, a request of few rows over a long prefix comes last.)  For the
  // same reason the last two workgroups per CU go strictly longest first; the
  // ones before them keep the order of the sets, whose pages they share.
  // (12 requests of 200..512 rows x 130..3000 keys, 32/8 heads, d = 64: 95.7 ->
  // 90.0 us; the 4B-class wave 145.7 -> 139.4; waves of many rounds unchanged.)
  std::vector<AttnItem> per_die[kNumXCD];
  for (int x = 0; x < kNumXCD; ++x) {
    std::stable_sort(die_sets[x].begin(), die_sets[x].end(),
                     [](const ItemSet &a, const ItemSet &b) { return a.longest > b.longest; });
    for (const ItemSet &set : die_sets[x]) per_die[x].insert(per_die[x].end(), set.items.begin(), set.items.end());
    const size_t tail = std::min(per_die[x].size(), (size_t)2 * kNumCU / kNumXCD);
    std::stable_sort(per_die[x].end() - tail, per_die[x].end(), [](const AttnItem &a, const AttnItem &b) {
      return a.kv_end - a.kv_begin > b.kv_end - b.kv_begin;
    });
  }
  size_t longest = 0;
  for (int x = 0; x < kNumXCD; ++x) longest = std::max(longest, per_die[x].size());
  AttnItem idle{};
  idle.req = -1;                 // the kernel returns at once on such an entry
  idle.part_slot = -1;
  for (size_t k = 0; k < longest; ++k)
    for (int x = 0; x < kNumXCD; ++x) {
      sch.items.push_back(k < per_die[x].size() ? per_die[x][k] : idle);
    }
  // drop idle entries at the very end of the list
  while (!sch.items.empty() && sch.items.back().req < 0) sch.items.pop_back();
  sch.num_slots = next_slot;
  sch.workspace_bytes = (size_t)next_slot * partial_slot_bytes(tile_rows, d);
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
