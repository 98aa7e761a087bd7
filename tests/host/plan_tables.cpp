// The tables of ob_plan.h over random tensor lists: what the kernels take for granted about the order of their workgroups
// and the numbering of their arrivals.  One check per argument.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <numeric>
#include <random>

#include "ob_plan.h"

using namespace obk;

#define CHECK(x) do { if (!(x)) { printf("%s:%d: %s\n", __FILE__, __LINE__, #x); exit(1); } } while (0)

namespace {
std::mt19937_64 rng(2024);
int64_t pick(int64_t a, int64_t b) { return a + (int64_t)(rng() % (uint64_t)(b - a + 1)); }

struct List {
  int64_t W, L, n_c;
  std::vector<int64_t> off;   // [L + 2], the padding last
  Tiling tm, tl;
};
constexpr int TILE = 8 * SPAN;
List random_list() {
  const int64_t kinds[] = {0, 1, 2, 255, 256, 1023, 1024, 1025, 4097, TILE - 1, TILE, TILE + 1, 3 * TILE, 63 * TILE, 64 * TILE,
                           65 * TILE + 77, 70 * TILE + 1, 100 * TILE, 300 * TILE + 5};
  List s;
  s.W = (const int64_t[]){1, 2, 3, 7, 16, 61}[rng() % 6];
  s.L = pick(1, 14);
  s.off.assign(1, 0);
  for (int64_t l = 0; l < s.L; ++l) s.off.push_back(s.off.back() + kinds[rng() % (sizeof(kinds) / sizeof(kinds[0]))]);
  if (s.off.back() == 0) s.off.back() = pick(1, 5000);
  const int64_t unit = 256 * s.W;
  s.n_c = (s.off.back() + unit - 1) / unit * 256;
  s.off.push_back(s.n_c * s.W);
  CHECK(build_tiling(SPAN, s.n_c, s.W, s.L, s.off, &s.tm) && build_tiling(TILE, s.n_c, s.W, s.L, s.off, &s.tl));
  return s;
}

// Moments and updates take turns: behind every TRAIL_BATCH moments parts (on all XCDs alike) a batch of the updates that are due, one for
// each `spread` of them, and none elsewhere, but for those up to a layer of more than `keep` parts that are due at once (at_once).  What is
// left of them stands behind the moments of the list, or of the launch.  update, launch: of each item.
void check_turns(const std::vector<char>& update, const std::vector<int64_t>& launch, const std::vector<int>& n, const std::vector<int>& begin,
                 int64_t lag, int64_t keep, int64_t spread, bool at_once) {
  CHECK(TRAIL_BATCH % 8 == 0);
  std::vector<int64_t> left(launch.empty() ? 0 : (size_t)launch.back() + 1, 0);   // moments parts of each launch
  for (size_t i = 0; i < update.size(); ++i) left[(size_t)launch[i]] += !update[i];
  int64_t pos = 0, due = 0, once = 0, taken = 0, launch_start = 0, in_launch = -1;
  size_t next = 0;   // the next layer to become due
  for (size_t i = 0; i < update.size();) {
    if (update[i]) {   // (behind a launch's moments)
      CHECK(left[(size_t)launch[i]] == 0);
      ++taken, ++i;
      continue;
    }
    if (launch[i] != in_launch) in_launch = launch[i], launch_start = pos;
    ++pos;
    const int64_t left_now = --left[(size_t)launch[i]];
    for (; next < n.size(); ++next) {
      if (n[next] == 0) continue;
      if (begin[next] + n[next] + lag > (lag > 0 ? pos : launch_start)) break;
      due += n[next];
      if (at_once && n[next] > keep) once = due;
    }
    int64_t run = 0;
    for (++i; i < update.size() && update[i] && launch[i] == in_launch; ++i) ++run;
    const int64_t pending = due - taken;
    const int64_t want = once > taken ? once - taken : pos % TRAIL_BATCH ? 0 : std::min(pending, (pending + spread - 1) / spread * TRAIL_BATCH);
    if (left_now > 0) CHECK(run == want);
    taken += run;
  }
  CHECK(taken == pos);
}

// Every part once as moments and once as update, the update after all moments of its layer (no later workgroup is waited
// for), `lag` moments parts behind them while there are any, in a later launch where nothing waits; what is kept is at most what the cache holds, and updated first.
void check_trail(const std::vector<int>& n, const std::vector<int>& begin, int64_t lag, int64_t group) {
  std::vector<unsigned int> items;
  std::vector<int64_t> end;
  trail_items(n, begin, lag, group, &items, &end);
  const int64_t parts = std::accumulate(n.begin(), n.end(), (int64_t)0);
  CHECK((int64_t)items.size() == 2 * parts);
  if (parts == 0) return;
  CHECK(end.back() == (int64_t)items.size() && std::is_sorted(end.begin(), end.end()));
  if (lag > 0) CHECK(end.size() == 1);
  std::vector<int64_t> at_moments((size_t)parts, -1), at_update((size_t)parts, -1);
  std::vector<char> kept((size_t)parts, 0);
  for (size_t i = 0; i < items.size(); ++i) {
    const int64_t p = items[i] & (TRAIL_KEEP - 1u);
    CHECK(p < parts);
    std::vector<int64_t>& at = (items[i] & TRAIL_UPDATE) ? at_update : at_moments;
    CHECK(at[(size_t)p] < 0);
    at[(size_t)p] = (int64_t)i;
    if (!(items[i] & TRAIL_UPDATE)) kept[(size_t)p] = (items[i] & TRAIL_KEEP) != 0;
  }
  std::vector<char> update;
  std::vector<int64_t> launch;
  for (size_t i = 0; i < items.size(); ++i) {
    update.push_back((items[i] & TRAIL_UPDATE) != 0);
    launch.push_back(std::upper_bound(end.begin(), end.end(), (int64_t)i) - end.begin());
  }
  check_turns(update, launch, n, begin, lag, TRAIL_KEEP_PARTS, TRAIL_SPREAD, true);
  auto launch_of = [&](int64_t i) { return std::upper_bound(end.begin(), end.end(), i) - end.begin(); };
  for (size_t l = 0; l < n.size(); ++l) {
    if (n[l] == 0) continue;
    int64_t last_moments = -1, first_update = (int64_t)items.size(), first_kept_update = -1, n_kept = 0;
    for (int64_t p = begin[l]; p < begin[l] + n[l]; ++p) {
      last_moments = std::max(last_moments, at_moments[(size_t)p]);
      first_update = std::min(first_update, at_update[(size_t)p]);
      n_kept += kept[(size_t)p];
      if (kept[(size_t)p] && first_kept_update < 0) first_kept_update = at_update[(size_t)p];
    }
    CHECK(last_moments >= 0 && last_moments < first_update);
    int64_t between = 0, left = 0;
    for (int64_t at : at_moments) {
      between += at > last_moments && at < first_update;
      left += at > first_update;
    }
    if (lag > 0) CHECK(between >= lag || left == 0);
    if (lag == 0) CHECK(launch_of(last_moments) < launch_of(first_update));
    CHECK(n_kept == std::min<int64_t>(n[l], TRAIL_KEEP_PARTS) && first_kept_update == first_update);
  }
}

void trail() {
  for (int it = 0; it < 300; ++it) {
    std::vector<int> n, begin;
    int at = 0;
    const int L = (int)pick(1, 9);
    for (int l = 0; l < L; ++l) {
      const int64_t kinds[] = {0, 0, 64 * TRAIL_PARTS, pick(1, 300), pick(256, 4000), pick(8000, 9000)};
      n.push_back((int)kinds[rng() % 6]);
      begin.push_back(n.back() ? at : 0);
      at += n.back();
    }
    for (int64_t lag : {trail_lag(256), (int64_t)pick(1, 6000), (int64_t)0}) check_trail(n, begin, lag, it % 2 ? TRAIL_GROUP : pick(1, 9000));
  }
}

// k_ratios_trail: every tile once for the ratio pass and in all its parts for the update, those of a layer after its last tile
// and some way behind it; the turns; and its rule.
void ratios_trail_order() {
  for (int it = 0; it < 200; ++it) {
    std::vector<int> n, begin;
    int at = 0;
    const int L = (int)pick(1, 9);
    for (int l = 0; l < L; ++l) {
      const int64_t kinds[] = {0, pick(64, 300), pick(1017, 2100), pick(6000, 7000)};
      n.push_back((int)kinds[rng() % 4]);
      begin.push_back(n.back() ? at : 0);
      at += n.back();
    }
    std::vector<unsigned int> items;
    ratios_trail_items(n, begin, 256, &items);
    const int parts = 8 / RATIOS_TRAIL_U;
    CHECK((int64_t)items.size() == (int64_t)at * (1 + parts));
    std::vector<int64_t> ratio((size_t)at, -1), first((size_t)at, -1);
    std::vector<int> seen((size_t)at, 0);
    std::vector<char> update;   // by tile
    int64_t n_ratio = 0;
    unsigned int before = 0;
    for (unsigned int i : items) {
      const unsigned int pos = i & (RATIOS_TRAIL_PART - 1u), part = (i & ~TRAIL_UPDATE) / RATIOS_TRAIL_PART;
      CHECK((int)pos < at && (int)part < parts);
      if (part == 0) update.push_back((i & TRAIL_UPDATE) != 0);
      else CHECK(i == before + RATIOS_TRAIL_PART);   // the parts of a tile stand together
      before = i;
      if (i & TRAIL_UPDATE) {
        CHECK(seen[pos] == (1 << part) - 1);
        seen[pos] |= 1 << part;
        if (first[pos] < 0) first[pos] = n_ratio;
      } else {
        CHECK(part == 0 && ratio[pos] < 0);
        ratio[pos] = n_ratio++;
      }
    }
    for (size_t l = 0; l < n.size(); ++l)
      for (int p = begin[l]; p < begin[l] + n[l]; ++p) {
        CHECK(seen[(size_t)p] == (1 << parts) - 1);
        CHECK(first[(size_t)p] >= std::min<int64_t>(ratio[(size_t)(begin[l] + n[l] - 1)] + 1 + 6 * 256, at));
      }
    check_turns(update, std::vector<int64_t>(update.size(), 0), n, begin, 6 * 256, RATIOS_TRAIL_KEEP, RATIOS_TRAIL_SPREAD, false);
    const int64_t most = *std::max_element(n.begin(), n.end());
    CHECK(ratios_trail(n, 256) == (at >= 1024 && 8 * (at - most) >= at));
  }
  const int line = (int)RATIOS_TRAIL_LARGE;   // at most 15/16 in layers above it, with a copy three quarters
  CHECK(ratios_trail_pays({line, line, 0}, true) && !ratios_trail_pays({line + 1, line + 1}, false) && !ratios_trail_pays({0, line + 1, line / 3}, true));
  CHECK(ratios_trail_pays({line + 1, line / 3 + 1}, true) && ratios_trail_pays({3 * line, line}, true) && !ratios_trail_pays({3 * line, line - 1}, true));
  CHECK(ratios_trail_each_step({8192, 8192, 8192, 8192}) && !ratios_trail_each_step({8193, 8193, 8193, 8193}) && !ratios_trail_each_step({4000, 4000, 3999}));
  CHECK(ratios_trail_each_step({9000, 9000, 8192, 8192, 1616}) && !ratios_trail_each_step({9000, 9000, 8192, 8192, 1615}));
  CHECK(ratios_trail_pays({3 * line, line - 1}, false) && ratios_trail_pays({15 * line, line}, false) && !ratios_trail_pays({15 * line, line - 1}, false));
}

// Which layers that rule takes: all those with enough whole tiles and not too many, or none at all below the total.
void big_rule() {
  for (int it = 0; it < 150; ++it) {
    const List s = random_list();
    const int64_t max_tiles = (const int64_t[]){0, 5, 66, 1000}[rng() % 4];
    BigRule rule;
    rule.max_tiles = (const int64_t[]){64, 99, rule.max_tiles}[rng() % 3];
    rule.min_total = (const int64_t[]){0, 65, 200, 500}[rng() % 4];
    SplitPlan pl;
    plan_split(s.tl, TILE, s.tm, s.off, s.n_c, s.L, max_tiles, rule, &pl);
    std::vector<int> inside((size_t)s.L, 0);
    for (int64_t t = 0; t < s.tl.n_tiles; ++t) {
      const int64_t a = t / s.tl.tpc * s.n_c + t % s.tl.tpc * TILE, e = std::min(a + TILE, (t / s.tl.tpc + 1) * s.n_c);
      const int l = s.tl.first[(size_t)t];
      if (l < s.L && e <= s.off[(size_t)l + 1]) ++inside[(size_t)l];
    }
    int64_t total = 0, got = 0;
    for (int64_t l = 0; l < s.L; ++l) {
      const bool fits = !pl.has_listed[(size_t)l] && inside[(size_t)l] >= rule.min_tiles && inside[(size_t)l] <= rule.max_tiles;
      if (fits) total += inside[(size_t)l];
      CHECK(pl.big_n[(size_t)l] == 0 || fits);
      got += pl.big_n[(size_t)l];
    }
    CHECK(got == (total >= rule.min_total ? total : 0) && got == (int64_t)pl.big_tiles.size());
  }
  // by the device's size: without waits from 20 tiles a CU on, with them from 7; a lowered limit takes lists of any size
  for (int cus : {256, 64}) {
    CHECK(trail_rule(true, 0, cus).min_total == 7 * cus && trail_rule(false, 0, cus).min_total == 20 * cus);
    CHECK(trail_rule(true, 8, cus).min_total == 0 && trail_rule(false, 8, cus).min_total == 0);
    CHECK(rest_in_launch(5 * cus, 20 * cus, 0, cus) && !rest_in_launch(5 * cus + 1, 1, 0, cus) && !rest_in_launch(1, cus, 19 * cus + 1, cus));
    // layers of at most two tiles a CU on average and no large ones: up to 40 tiles a CU
    CHECK(rest_in_launch(1, 40 * cus, 0, cus, 20) && !rest_in_launch(1, 40 * cus + 1, 0, cus, 99) && rest_in_launch(5 * cus, 30 * cus, 0, cus, 15));
    CHECK(!rest_in_launch(1, 30 * cus, 0, cus, 14) && rest_in_launch(1, 20 * cus, 0, cus, 1) && !rest_in_launch(1, 20 * cus + 1, 0, cus, 10));
    CHECK(!rest_in_launch(1, 20 * cus, 1, cus, 99) && !rest_in_launch(5 * cus + 1, 30 * cus, 0, cus, 99) && !rest_in_launch(1, 0, 0, cus, 9));
    CHECK(server_spans(2, 16 * cus, cus) == 4 && server_spans(3, 16 * cus, cus) == 2 && server_spans(1, 16 * cus - 1, cus) == 2);
    CHECK(server_spans(32, 8 * cus, cus) == 2 && server_spans(32, 8 * cus - 1, cus) == 1 && server_spans(33, 99 * cus, cus) == 1);
    CHECK(worker_sum_lds(80 * cus, cus) && !worker_sum_lds(80 * cus - 1, cus));
    CHECK(arrivals_one_level(40 * cus, cus) == 256 && arrivals_one_level(40 * cus + 1, cus) == 512);
  }
}

// Every arrival of a layer has a number of its own below the layer's count, whoever arrives for it (k_ratios_apply_hist's
// listed tiles, the first and the last segment of a rest tile); segments between them are layers of their own; the
// layers' group counters lie apart and inside their allocation.
void arrivals() {
  for (int it = 0; it < 300; ++it) {
    const List s = random_list();
    SplitPlan pl;
    plan_split(s.tl, TILE, s.tm, s.off, s.n_c, s.L, (const int64_t[]){0, 5, 66, 1000}[rng() % 4], BigRule(), &pl);
    ArrivalPlan ap;
    plan_arrivals(pl, s.tm, s.L, &ap);
    std::vector<std::vector<char>> seen((size_t)s.L);
    std::vector<int> finished((size_t)s.L, 0);
    auto seg0 = [&](int l) { return s.tm.layer_seg0[(size_t)l]; };
    for (int l = 0; l < s.L; ++l) {
      const size_t i = (size_t)l;
      const int n = layer_arrivals(pl.n_listed[i], seg0(l), ap.skip_first[i], ap.skip_end[i], seg0(l + 1));
      CHECK(n >= 0 && (n == 0) == (std::count(ap.alone.begin(), ap.alone.end(), l) == 1));
      seen[i].assign((size_t)n, 0);
      // a listed tile's own count, from what it has at hand
      if (pl.n_listed[i]) CHECK(n == layer_arrivals(pl.n_listed[i], seg0(l), pl.seg_first[i], pl.seg_end[i], seg0(l + 1)));
      for (int j = 0; j < pl.n_listed[i]; ++j) seen[i][(size_t)j] = 1;
    }
    for (int tile : pl.rest_ratio_tiles) {
      const int s0 = s.tm.tile_seg0[(size_t)tile], s1 = s.tm.tile_seg0[(size_t)tile + 1];
      CHECK(s1 > s0);
      for (int sg = s0; sg < s1; ++sg) {
        const int l = s.tm.seg_layer[(size_t)sg];
        const size_t i = (size_t)l;
        const int j = rest_arrival(sg, pl.n_listed[i], seg0(l), ap.skip_first[i], ap.skip_end[i]);
        CHECK(sg < ap.skip_first[i] || sg >= ap.skip_end[i]);
        CHECK(j >= 0 && j < (int)seen[i].size() && !seen[i][(size_t)j]);
        seen[i][(size_t)j] = 1;
        if (sg > s0 && sg < s1 - 1) CHECK(seen[i].size() == 1);
      }
    }
    int64_t next = 0, line_end = 0;
    for (int l = 0; l < s.L; ++l) {
      const size_t i = (size_t)l;
      CHECK(std::count(seen[i].begin(), seen[i].end(), 1) == (int64_t)seen[i].size());
      CHECK(ap.arr0[i] == next);
      const int64_t line = group_line(ap.arr0[i], l) / CTR_STRIDE;
      CHECK(line >= line_end);
      line_end = line + (int64_t)arrival_groups((int64_t)seen[i].size());
      next += (int64_t)seen[i].size();
    }
    CHECK(next == ap.n_arrivals && line_end <= (int64_t)group_lines(ap.n_arrivals, s.L));
    // what the last workgroups wait for, event by event: the arrivals in any order
    std::vector<int> left((size_t)s.L);
    for (int l = 0; l < s.L; ++l) left[(size_t)l] = (int)seen[(size_t)l].size() - pl.n_listed[(size_t)l];
    int64_t events = (int64_t)ap.alone.size();
    for (int l = 0; l < s.L; ++l) events += pl.n_listed[(size_t)l] > 0 && left[(size_t)l] == 0;
    for (int tile : pl.rest_ratio_tiles) {
      const int s0 = s.tm.tile_seg0[(size_t)tile], s1 = s.tm.tile_seg0[(size_t)tile + 1];
      events += --left[(size_t)s.tm.seg_layer[(size_t)s0]] == 0;
      if (s1 - s0 > 1) events += --left[(size_t)s.tm.seg_layer[(size_t)s1 - 1]] == 0;
      events += s1 - s0 > 2;
    }
    CHECK(events == coefficient_events(pl, s.tm, s.L, ap));
  }
}

// A launch from the last tile to the first takes every tile once, later ones first, each on its own XCD; the second
// reads of a list stay in the caches only where the server's words don't need them (64 tiles a chunk, or 8e6 elements).
void second_reads() {
  for (unsigned int n = 1; n <= 2100; n += n < 40 ? 1 : 97) {
    std::vector<char> seen(n, 0);
    for (unsigned int b = 0; b < n; ++b) {
      const int t = tile_from_end(b, n);
      CHECK(t >= 0 && t < (int)n && !seen[(size_t)t]);
      seen[(size_t)t] = 1;
      CHECK((unsigned int)t % 8 == b % 8);
      CHECK(b < 8 || t == tile_from_end(b - 8, n) - 8);
    }
  }
  CHECK(!keeps_second_reads(2 * 909 * 909, 147) && !keeps_second_reads(64 * 65536 - 1, 64) && keeps_second_reads(64 * 65536, 64));
  CHECK(keeps_second_reads(8000000, 256) && !keeps_second_reads(7999999, 256) && keeps_second_reads(65536, 1));
}

// Tile sizes of the one-launch kernels where another one measures 4 % or more slower (256 CUs; 80 % of the slots), and what the rule takes for the
// LAMB step of six tensors, where one span measures 5 % faster.
void small_lists() {
  struct Want { int64_t W; std::vector<int64_t> sizes; int u_apply, u_lamb; };
  const int64_t k = 1024;
  const Want wants[] = {
      {4, {400 * k}, 1, 1},          {4, {625 * k}, 1, 1},             {2, {784 * k}, 1, 1},
      {4, {900601}, 1, 1},           {4, std::vector<int64_t>(4, 256 * k), 2, 1},
      {4, std::vector<int64_t>(4, 225 * k), 2, 1}, {6, std::vector<int64_t>(6, 256 * k), 2, 2},
      {4, {1600225}, 1, 2},          {4, {1600 * k}, 1, 2},            {4, std::vector<int64_t>(4, 354 * 354), 1, 2},
      {4, std::vector<int64_t>(8, 352 * 352), 1, 1}, {4, std::vector<int64_t>(100, 10000), 1, 1},
      {4, {2304 * k}, 4, 4},         {8, std::vector<int64_t>(30, 130 * k), 0, 0},
  };
  for (const Want& w : wants) {
    std::vector<int64_t> off(1, 0);
    for (int64_t s : w.sizes) off.push_back(off.back() + s);
    const int64_t L = (int64_t)w.sizes.size(), n_c = (off.back() + 256 * w.W - 1) / (256 * w.W) * 256;
    off.push_back(n_c * w.W);
    SmallShape sh[3];
    bool fits[3];
    for (int i = 0; i < 3; ++i) {
      sh[i] = small_shape(1 << i, off, n_c, w.W, L);
      fits[i] = 5 * (sh[i].n_tiles + 8) <= 4 * 256 * (i == 0 ? 8 : i == 1 ? 5 : 4);
    }
    for (bool by_slots : {true, false}) {
      const int c = small_choice(sh, fits, by_slots, 256), got = c < 0 ? 0 : 1 << c, want = by_slots ? w.u_apply : w.u_lamb;
      if (got != want) printf("%d tensors of %ld, slots %d: U = %d\n", (int)L, (long)w.sizes[0], by_slots, got);
      CHECK(got == want);
    }
  }
}
}  // namespace

int main(int argc, char** argv) {
  const struct { const char* name; void (*f)(); } checks[] = {{"trail", trail}, {"ratios_trail", ratios_trail_order}, {"big_rule", big_rule}, {"arrivals", arrivals}, {"second_reads", second_reads},
                                                              {"small_lists", small_lists}};
  for (const auto& c : checks)
    if (argc == 2 && !strcmp(argv[1], c.name)) {
      c.f();
      printf("ok\n");
      return 0;
    }
  return 2;
}
