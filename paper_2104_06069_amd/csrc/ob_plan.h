// Host planning of libonebitlamb, without any HIP call or device type: the tables that say which tile of which tensor
// list each kernel takes and in what order, and the constants and index functions that the kernels share with them.  Plain
// C++, so that the plans can be checked on their own.
#pragma once

#include <algorithm>
#include <cstdint>
#include <limits>
#include <numeric>
#include <vector>

#ifndef OB_BIG_MIN_TILES
#define OB_BIG_MIN_TILES 64   // a layer outside the barrier kernel with at least that many whole 8192-element tiles
#endif

namespace obk {

constexpr int BLOCK = 256;       // threads per workgroup (4 wavefronts of 64)
constexpr int WAVE = 64;
constexpr int SPAN = BLOCK * 4;  // elements one workgroup-wide 128-bit access covers
// Arrival counters of different chunks / layers sit 128 bytes apart: read-modify-write atomics on one
// cache line are served one at a time (12 ns each, measured), whichever word of it they address,
// and several chunks or layers are always in flight together.
constexpr int CTR_STRIDE = 16;   // in 8-byte words
constexpr int TICKET_SUB = 64;   // tiles of a first-level group of chunk_ticket
constexpr int ARRIVE_ONE_LEVEL = 256, ARRIVE_SUB = 32;   // (barrier_arrive)

// Where the group counters of layer l begin (in 8-byte words), whose arrivals are first, first + 1, ... in a numbering
// that runs on from layer to layer: no two layers' groups overlap, and no table is needed.
constexpr int64_t group_line(int first, int l) { return (int64_t)(first / ARRIVE_SUB + l) * CTR_STRIDE; }

// Workgroup b's tile in a launch of n that goes from the last tile to the first.  Workgroups go round the XCDs, each with an L2
// of its own: every tile stays on the XCD that it has in a launch from the first to the last (b mod 8).
constexpr unsigned int XCDS = 8;
constexpr int tile_from_end(unsigned int b, unsigned int n) {
  const unsigned int x = b % XCDS;
  return (int)(((n - x + XCDS - 1) / XCDS - 1 - b / XCDS) * XCDS + x);
}

// Whether the plain form leaves what its next kernel reads again in the caches (ld4_keep): where each worker's chunk has
// at least 64 tiles, or the buffer 8 M elements.  Below, with many workers and so a short served chunk, the server's few
// workgroups are bound by the latency of their W rows of words, which the lines kept for the other kernels push out.  A step of two equal
// tensors in plain form, us, kept / not, by workers:
//   elements   32           64           96           128          192          256
//   1.7 M      41.1 / 41.1  42.7 / 41.8  44.6 / 42.8  43.8 / 41.7  45.1 / 41.4  47.9 / 42.9
//   2.9 M      49.1 / 49.0  50.2 / 49.2  51.4 / 49.6  53.2 / 51.0  56.8 / 52.7  59.4 / 53.3
//   4.2 M      56.0 / 57.3  56.9 / 57.4  59.2 / 58.7  60.8 / 59.1  65.4 / 62.9  68.9 / 63.8
//   5.8 M      66.1 / 68.8  66.8 / 68.3  68.8 / 69.4  69.7 / 70.3  72.9 / 71.9  78.4 / 78.5
//   8.4 M      82.4 / 86.6  81.5 / 85.6  84.2 / 88.3  85.2 / 87.7  90.1 / 93.6  92.9 / 91.7
//   11.5 M    101.5 / 108.1 104.6 / 111.3 105.8 / 113.1 106.9 / 112.4 113.9 / 119.1 115.0 / 119.5
// (1448x1448 twice with 16 workers 56.9 / 58.4, with 147 63.8 / 60.4.)
constexpr int64_t KEEP_MIN_CHUNK = 64 * SPAN, KEEP_MIN = 8000000;
constexpr bool keeps_second_reads(int64_t n, int64_t W) { return n >= (W * KEEP_MIN_CHUNK < KEEP_MIN ? W * KEEP_MIN_CHUNK : KEEP_MIN); }

// Whether the worker's pass with a 16-bit gradient and no momentum scaling sums its tile's squares and forms its sign words through LDS
// instead of by register moves: the code before is the same, and so are registers and occupancy; what differs is when the workgroups leave, and so how
// the next ones' loads meet the stores.  The call on the same buffers, us, register moves / LDS (8 workers): 6 M elements 13.8 / 14.6, 12 M 23.8 / 24.3, 18 M
// 34.2 / 33.9, 27 M 50.6 / 49.4, 36 M 68.0 / 65.3, 50 M 94.2 / 89.7, 110 M 194.4 / 187, 336 M 591 / 554, 700 M 1218 / 1152; 780 lists of 13 to 73 M with 1 to 256
// workers, mean of moves over LDS by tiles a CU: 50 to 60 0.989, 60 to 80 1.000, 80 to 100 1.016, 120 to 240 1.028, 240 to 256 1.031.  (The sum alone through
// LDS: 336 M 574, 700 M 1177.)  With momentum scaling the moves are faster everywhere (336 M 566 / 581), and in fp32 not slower (18 M 38.8 / 38.8, 50 M 98.3 /
// 98.8, 336 M 660 / 659).
inline bool worker_sum_lds(int64_t n_tiles, int cus) { return n_tiles >= 80 * (int64_t)cus; }

// Arrivals at a layer's barrier with nl listed tiles, whose segments are seg0 .. seg1-1 and of which those from skip_first to
// skip_end-1 lie in listed or big tiles; the number of the arrival of one of the others, sg (the listed tiles come first).
constexpr int layer_arrivals(int nl, int seg0, int skip_first, int skip_end, int seg1) {
  return nl + (skip_first - seg0) + (seg1 - skip_end);
}
constexpr int rest_arrival(int sg, int nl, int seg0, int skip_first, int skip_end) {
  return nl + (sg < skip_first ? sg - seg0 : (skip_first - seg0) + (sg - skip_end));
}

// k_warmup_trail's workgroups
constexpr unsigned int TRAIL_UPDATE = 1u << 31;   // update (else: moments)
constexpr unsigned int TRAIL_KEEP = 1u << 30;     // moments: m and v read again soon
constexpr int TRAIL_U = 2;                        // spans per part
constexpr int TRAIL_PARTS = 8 / TRAIL_U;          // parts per tile
struct SmallTile {
  int l0;          // layer of the first element
  int seg0;        // first segment
  int nseg;        // segments (0: padding)
  int chunk_kind;  // chunk << 2 | (1: wholly inside one layer) | (2: lagging)
  int l_last;      // layer of the last segment
  int n_first;     // segments of the first segment's layer, over all tiles
  int n_last;      // ... of the last segment's
  int pad;
};

// Tables of one tiling of the padded buffer (tiles of `tile` elements inside each chunk): the layer
// of each tile's first element (L = padding), the (tile, layer) segments in position order and
// their grouping by layer.
struct Tiling {
  int64_t tpc = 0, n_tiles = 0;
  std::vector<int> first, tile_seg0, seg_layer, layer_seg0;
};

inline bool build_tiling(int64_t tile, int64_t n_c, int64_t W, int64_t L, const std::vector<int64_t>& h_off,
                  Tiling* out) {
  out->tpc = (n_c + tile - 1) / tile;
  out->n_tiles = out->tpc * W;
  if (out->n_tiles > 0x7fffffff) return false;
  out->first.resize((size_t)out->n_tiles);
  out->tile_seg0.resize((size_t)out->n_tiles + 1);
  out->seg_layer.clear();
  out->layer_seg0.assign((size_t)L + 1, 0);
  for (int64_t t = 0; t < out->n_tiles; ++t) {
    const int64_t c = t / out->tpc, b = t % out->tpc;
    const int64_t tile0 = c * n_c + b * tile;
    const int64_t tile1 = std::min(tile0 + tile, (c + 1) * n_c);
    // first layer: the non-empty layer that holds tile0 (binary search on the offsets)
    int64_t lo = 0, hi = L + 1;  // h_off[lo] <= tile0 < h_off[hi]
    while (hi - lo > 1) {
      const int64_t mid = (lo + hi) / 2;
      if (h_off[(size_t)mid] <= tile0) lo = mid; else hi = mid;
    }
    out->first[(size_t)t] = (int)lo;  // lo == L when tile0 >= N
    out->tile_seg0[(size_t)t] = (int)out->seg_layer.size();
    for (int64_t l = lo; l < L && h_off[(size_t)l] < tile1; ++l) {
      const int64_t a = std::max(h_off[(size_t)l], tile0), e = std::min(h_off[(size_t)l + 1], tile1);
      if (e > a) out->seg_layer.push_back((int)l);
    }
  }
  out->tile_seg0[(size_t)out->n_tiles] = (int)out->seg_layer.size();
  std::vector<int> count((size_t)L, 0);  // segments are ordered by position, hence grouped by layer
  for (int l : out->seg_layer) ++count[(size_t)l];
  for (int64_t l = 0; l < L; ++l)
    out->layer_seg0[(size_t)l + 1] = out->layer_seg0[(size_t)l] + count[(size_t)l];
  return true;
}

// The host side of one LayerSplit: which tiles the barrier kernel takes and what is left.
struct SplitPlan {
  std::vector<unsigned char> has_listed;   // [L] 1 for layers that the barrier kernel finishes
  std::vector<int> fused_tiles, rest_tiles, n_listed, list_begin, seg_first, seg_end;
  std::vector<unsigned char> covered;      // [SPAN tiles] 1 inside a listed tile
  std::vector<int> big_tiles, rest_ratio_tiles;
  std::vector<int> big_n, big_begin, big_seg_first, big_seg_end;   // [L]
  std::vector<unsigned char> covered_big;  // [SPAN tiles] 1 inside a big tile
  int64_t n_layers = 0, n_params = 0, n_big_params = 0;
};

// Which layers outside the barrier kernel have big tiles: those with enough whole tiles and not too many,
// and only if they hold enough together.
struct BigRule {
  int64_t min_tiles = OB_BIG_MIN_TILES, max_tiles = std::numeric_limits<int64_t>::max(), min_total = 0;
};

// tl / tm: the barrier kernel's tiling (tiles of tile_lb elements) and the SPAN tiling;
// max_tiles: the largest number of tiles of one layer the barrier kernel may hold (0: it is not
// used).  No HIP call.
inline void plan_split(const Tiling& tl, int64_t tile_lb, const Tiling& tm, const std::vector<int64_t>& h_off,
                int64_t n_c, int64_t L, int64_t max_tiles, const BigRule& rule, SplitPlan* pl) {
  pl->has_listed.assign((size_t)L, 0);
  pl->n_listed.assign((size_t)L, 0);
  pl->list_begin.assign((size_t)L, 0);
  pl->seg_first.assign(tm.layer_seg0.begin(), tm.layer_seg0.begin() + L);   // (no listed tile: nothing skipped)
  pl->seg_end = pl->seg_first;
  pl->covered.assign((size_t)tm.n_tiles, 0);
  auto tile_range = [&](int64_t t, int64_t* tile0, int64_t* tile1) {
    const int64_t c = t / tl.tpc, b = t % tl.tpc;
    *tile0 = c * n_c + b * tile_lb;
    *tile1 = std::min(*tile0 + tile_lb, (c + 1) * n_c);
  };
  // tiles inside one layer, per layer in position order
  std::vector<std::vector<int>> inside((size_t)L);
  for (int64_t t = 0; t < tl.n_tiles; ++t) {
    int64_t tile0, tile1;
    tile_range(t, &tile0, &tile1);
    const int l = tl.first[(size_t)t];
    if (l < L && tile1 <= h_off[(size_t)l + 1]) inside[(size_t)l].push_back((int)t);
  }
  for (int64_t l = 0; l < L; ++l) {
    const std::vector<int>& in = inside[(size_t)l];
    const size_t n = in.size();
    if (n == 0 || n > (size_t)max_tiles) continue;   // (max_tiles = 0: no layer is listed)
    pl->has_listed[(size_t)l] = 1;
    pl->n_listed[(size_t)l] = (int)n;
    pl->list_begin[(size_t)l] = (int)pl->fused_tiles.size();
    pl->n_layers += 1;
    for (size_t j = 0; j < n; ++j) {
      const int64_t t = in[j];
      int64_t tile0, tile1;
      tile_range(t, &tile0, &tile1);
      pl->fused_tiles.push_back((int)t);
      pl->n_params += tile1 - tile0;
      const int64_t c = t / tl.tpc, b = t % tl.tpc;
      const int64_t span0 = c * tm.tpc + b * (tile_lb / SPAN);
      const int64_t nspan = (tile1 - tile0 + SPAN - 1) / SPAN;
      for (int64_t j2 = 0; j2 < nspan; ++j2) pl->covered[(size_t)(span0 + j2)] = 1;
      // each of these spans lies inside the layer: one segment each, consecutive
      if (j == 0) pl->seg_first[(size_t)l] = tm.tile_seg0[(size_t)span0];
      pl->seg_end[(size_t)l] = tm.tile_seg0[(size_t)(span0 + nspan)];
    }
  }
  // big tiles: the whole tiles of the layers that hold many of them but are not listed
  pl->covered_big.assign((size_t)tm.n_tiles, 0);
  for (std::vector<int>* v : {&pl->big_n, &pl->big_begin, &pl->big_seg_first, &pl->big_seg_end}) v->assign((size_t)L, 0);
  auto is_big = [&](int64_t l) {
    const int64_t n = (int64_t)inside[(size_t)l].size();
    return !pl->has_listed[(size_t)l] && n >= rule.min_tiles && n <= rule.max_tiles;
  };
  int64_t n_big = 0;
  for (int64_t l = 0; l < L; ++l) n_big += is_big(l) ? (int64_t)inside[(size_t)l].size() : 0;
  for (int64_t l = 0; l < L; ++l) {   // (also when no layer is listed: the pass needs no barrier)
    if (!is_big(l) || n_big < rule.min_total) continue;
    const std::vector<int>& in = inside[(size_t)l];
    pl->big_n[(size_t)l] = (int)in.size();
    pl->big_begin[(size_t)l] = (int)pl->big_tiles.size();
    for (int t : in) {
      int64_t tile0, tile1;
      tile_range(t, &tile0, &tile1);
      pl->big_tiles.push_back(t);
      pl->n_big_params += tile1 - tile0;
      const int64_t c = t / tl.tpc, b = t % tl.tpc;
      const int64_t span0 = c * tm.tpc + b * (tile_lb / SPAN);
      const int64_t nspan = (tile1 - tile0 + SPAN - 1) / SPAN;
      for (int64_t j2 = 0; j2 < nspan; ++j2) pl->covered_big[(size_t)(span0 + j2)] = 1;
      if (t == in.front()) pl->big_seg_first[(size_t)l] = tm.tile_seg0[(size_t)span0];
      pl->big_seg_end[(size_t)l] = tm.tile_seg0[(size_t)(span0 + nspan)];
    }
  }
  for (int64_t t = 0; t < tm.n_tiles; ++t)
    if (!pl->covered[(size_t)t] && tm.tile_seg0[(size_t)t + 1] > tm.tile_seg0[(size_t)t]) {
      pl->rest_tiles.push_back((int)t);
      if (!pl->covered_big[(size_t)t]) pl->rest_ratio_tiles.push_back((int)t);
    }
}

// Which layers k_warmup_trail takes, and how.  A LAMB step, us, in two passes over everything outside the barrier
// kernel / with k_warmup_trail (256 CUs; fp32 gradient except gpt, 16-bit there):
//   in one launch: squares of 3300 x 1 75.7 / 78.2, 4000 x 1 115 / 109, 3400 x 2 156 / 151, 5000 x 1 173 / 160, 4000 x 3 313 / 286,
//     5000 x 8 1335 / 1175, 7000 x 6 1930 / 1838, 20000 x 2 5400 / 5520; the GPT list of 1.3e9 parameters 8490 / 7400
//   in several launches (no kernel may wait): BERT and GPT lists of 11 M 80 / 87, 25 M 152 / 160, 40 M 273 / 275,
//     50 M 353 / 332, 60 M 400 / 386, 110 M 733 / 681, 336 M 2218 / 2056, 1.3e9 8800 / 8010
// so that it is taken from 7 and 20 tiles a CU on (14.7 M and 42 M elements), and not for layers of which the cache holds next to nothing.
// A configuration that lowers the barrier kernels' limit (cap) takes it for lists of any size.
constexpr int64_t TRAIL_MAX_LAYER_TILES = 16384;
inline BigRule trail_rule(bool wait, int32_t cap, int cus) {
  BigRule r;
  r.max_tiles = TRAIL_MAX_LAYER_TILES;
  r.min_total = cap > 0 ? 0 : (wait ? 7 : 20) * (int64_t)cus;
  return r;
}

// The workgroups of k_warmup_trail in order (no HIP call).  n, begin: parts of each layer.  lag > 0: one launch, the
// update of a layer from `lag` moments parts after the layer's last one on: what is in flight on the device then (8 workgroups a
// CU; trail_lag: 10) lies between them, so that no update waits for long (half of that 2 % slower, twice no difference).  lag = 0: no update
// waits; the layers are taken in groups of at least `group` parts (16.8 M elements; 33 M no difference), and a launch updates one
// group and forms the moments of the next.
// Updates and moments take turns, TRAIL_BATCH of each at a time (of the updates the more, the more are due: one batch for
// every `spread` of them), so that at any time the device reads and writes alike; batches are a multiple of the 8 XCDs,
// to which consecutive workgroups go in turn: one by one, all updates would be half of the XCDs'.
// A layer of more than TRAIL_KEEP_PARTS parts (16.8 M elements, 200 MB of m, v and x) does not fit the cache: its last
// parts are updated first, and only they are kept; the moments of the next layer wait for all of its updates (spread_large: they do not).
// A LAMB step, us, a layer's updates all at once / in batches of 32, one for every 2048 (of 8: 7360 to 7560; every 4096, 8192, 16384 in batches of 8:
// 7430, 7670, 9030): the GPT list of 1.3e9 parameters 7350-7416 / 7240-7315, 5000 x 8 1156 / 1142, 3600 x 3 236.4 / 233.4, 3300 x 2
// 141.2 / 139.8; layers beyond the cache, spread too: 7000 x 6 1825 / 1843, 10000 x 4 2631 / 2653.
constexpr int64_t TRAIL_GROUP = 8192, TRAIL_KEEP_PARTS = 8192, TRAIL_SPREAD = 2048, TRAIL_BATCH = 32;
inline int64_t trail_lag(int cus) { return 10 * (int64_t)cus; }
inline void trail_items(const std::vector<int>& n, const std::vector<int>& begin, int64_t lag, int64_t group,
                 std::vector<unsigned int>* items, std::vector<int64_t>* item_end, int64_t keep_parts = TRAIL_KEEP_PARTS,
                 int64_t spread = TRAIL_SPREAD, bool spread_large = false) {
  items->clear();
  item_end->clear();
  std::vector<unsigned int> due;   // the updates that may run, in order; due[0 .. at) are in the list
  size_t at = 0, at_once = 0;      // due[at .. at_once): not spread
  auto kept_from = [&](int64_t l) { return n[(size_t)l] - std::min<int64_t>(n[(size_t)l], keep_parts); };
  auto update = [&](int64_t l) {
    const int64_t keep = kept_from(l);
    for (int64_t j = keep; j < n[(size_t)l]; ++j) due.push_back((unsigned int)(begin[(size_t)l] + j) | TRAIL_UPDATE);
    for (int64_t j = 0; j < keep; ++j) due.push_back((unsigned int)(begin[(size_t)l] + j) | TRAIL_UPDATE);
    if (keep > 0 && !spread_large) at_once = due.size();
  };
  auto take = [&](int64_t k) {
    for (; k > 0 && at < due.size(); --k) items->push_back(due[at++]);
  };
  std::vector<int64_t> layers;
  for (size_t l = 0; l < n.size(); ++l)
    if (n[l] > 0) layers.push_back((int64_t)l);
  if (layers.empty()) return;
  size_t done = 0, launched = 0;   // layers whose update is due; whose moments lie in earlier launches
  int64_t pos = 0, in_group = 0;   // moments parts in the list; of the present group
  for (size_t i = 0; i < layers.size(); ++i) {
    const int64_t l = layers[i], keep = kept_from(l);
    if (lag == 0 && in_group >= group) {
      take((int64_t)due.size());
      item_end->push_back((int64_t)items->size());
      launched = i;
      in_group = 0;
    }
    in_group += n[(size_t)l];
    for (int64_t j = 0; j < n[(size_t)l]; ++j) {
      items->push_back((unsigned int)(begin[(size_t)l] + j) | (j >= keep ? TRAIL_KEEP : 0u));
      ++pos;
      while (done < (lag > 0 ? layers.size() : launched) &&
             (lag == 0 || begin[(size_t)layers[done]] + n[(size_t)layers[done]] + lag <= pos))
        update(layers[done++]);
      const int64_t pending = (int64_t)(due.size() - at);
      if (at < at_once) take((int64_t)(at_once - at));
      else if (pos % TRAIL_BATCH == 0) take((pending + spread - 1) / spread * TRAIL_BATCH);
    }
  }
  if (lag == 0) {
    take((int64_t)due.size());
    item_end->push_back((int64_t)items->size());
  }
  while (done < layers.size()) update(layers[done++]);
  take((int64_t)due.size());
  item_end->push_back((int64_t)items->size());
}

// k_ratios_trail: whole tiles for the ratio pass, in parts of RATIOS_TRAIL_U spans for the update, in the same order (what the cache is to
// hold is v_frozen alone).  Four steps, us, k_ratios_big_hist and k_decompress_apply / k_ratios_trail (256 CUs): squares of
// 3300 x 2 571 / 557, 3600 x 3 933 / 908, 5000 x 2 1179 / 1137, 5000 x 8 4400 / 4228, 7000 x 6 6438 / 6335, the
// GPT list of 1.3e9 parameters 27900 / 26400, lists of its shape with one block, three quarters of their large layers one word embedding,
// 2749 / 2715, 3225 / 3175, 3608 / 3555; but with no other large layer, in which to spread the embedding's update, 110 M 2301 / 2310,
// 336 M 6728 / 6761.  So it is taken where an eighth of the large layers' tiles lies outside the largest of them (and there are more
// than a lowered limit of the barrier kernel may leave).
// GPT list, by the order: a layer's updates all at once 27590, parts of 2 spans in that 28160; one by one in turn with the ratio pass 28380 (the XCDs; see
// above), in batches 26550, 26470, 26660 with parts of 8, 4 and 2 spans; batches of 64, one for every 1024 or 4096, lag of 1 to 12, and
// 4096 to 8192 kept: 26440 to 26760.
constexpr int64_t RATIOS_TRAIL_KEEP = 6144, RATIOS_TRAIL_SPREAD = 2048;
constexpr int RATIOS_TRAIL_U = 4;
constexpr unsigned int RATIOS_TRAIL_PART = 1u << 27;   // the part, above the tile's position
inline bool ratios_trail(const std::vector<int>& n, int cus) {
  const int64_t total = std::accumulate(n.begin(), n.end(), (int64_t)0), most = n.empty() ? 0 : *std::max_element(n.begin(), n.end());
  return total >= 4 * (int64_t)cus && total < (int64_t)RATIOS_TRAIL_PART && 8 * (total - most) >= total;
}
// With a history, not where most of the elements lie in layers far beyond the cache: the two passes over one do not meet in it, and beside the ratio pass's reads
// the update's, with a 16-bit copy above all, are only more streams at a time.  The call, us, period 4, two kernels / k_ratios_trail, squares (tiles of a layer):
//   with a copy: 7500 x 10 (6867) 2054 / 1996, 8500 x 8 (8820) 2136 / 2122, 9500 x 6 (11017) 1983 / 2010 (but the step 3020 / 3015), 10000 x 8 (12208) 2907 /
//   2964 (4456 / 4430), 10500 x 5 (13459) 2023 / 2063 (3072 / 3084), 11500 x 4 1925 / 1995 (2930 / 2971), 13000 x 3 1841 / 1927, 20000 x 2 2977 / 3134;
//   without: 9500 x 6 1795 / 1788, 10500 x 5 1830 / 1842 (2996 / 2975), 11500 x 4 1738 / 1765 (2861 / 2864), 13000 x 3 1675 / 1704 (2759 / 2769),
//   20000 x 2 2678 / 2715 (4406 / 4373), 20000 x 3 3977 / 4063 (6502 / 6522); period 2 as period 4; the array written at every step: no difference.
// Lists by the share in layers above the line: with a copy 0.66 4201 / 4317 (6389 / 6434), 0.68 4087 / 4115 (6208 / 6174) and 4315 / 4322 (6573 / 6500), 0.81 2237 /
// 2260 (3371 / 3361), 0.89 2564 / 2625 (3892 / 3904), 0.93 4040 / 4110 (6105 / 6128); without 0.81 2031 / 1994, 0.89 2314 / 2307, 0.93 3640 / 3631.
constexpr int64_t RATIOS_TRAIL_LARGE = 2 * RATIOS_TRAIL_KEEP;
inline int64_t tiles_in_layers_above(const std::vector<int>& n, int64_t line) {
  return std::accumulate(n.begin(), n.end(), (int64_t)0, [=](int64_t a, int q) { return a + (q > line ? q : 0); });
}
inline bool ratios_trail_pays(const std::vector<int>& n, bool copy) {
  const int64_t total = tiles_in_layers_above(n, 0), large = tiles_in_layers_above(n, RATIOS_TRAIL_LARGE);
  return copy ? 4 * large <= 3 * total : 16 * large <= 15 * total;
}
// ... and where the array is written at every step: the largest layer at most a quarter of the tiles, and at most half of them in layers of more than 8192.
// A step / the call, us, plain kernels around k_ratios_apply_resident / k_ratios_trail beside k_ratios_apply_hist, by that half's share: 0.11 6725 / 6698, 4361 / 4315; 0.17
// 5819 / 5769, 3784 / 3755; 0.68 7021 / 7071, 4478 / 4571; 0.88 7510 / 7672, 4877 / 5024; 0.90 5314 / 5434, 3394 / 3526; with a copy 0.11 6970 / 6873, 4762 /
// 4775; 0.17 5992 / 5876, 4111 / 4068; 0.68 7223 / 7216, 4962 / 5048; 0.88 7738 / 7852, 5281 / 5531; 0.90 5517 / 5537, 3789 / 3886.
inline bool ratios_trail_each_step(const std::vector<int>& n) {
  const int64_t total = tiles_in_layers_above(n, 0), most = n.empty() ? 0 : *std::max_element(n.begin(), n.end());
  return 4 * most <= total && 2 * tiles_in_layers_above(n, 8192) <= total;
}
inline void ratios_trail_items(const std::vector<int>& n, const std::vector<int>& begin, int cus, std::vector<unsigned int>* items) {
  std::vector<unsigned int> tiles;
  std::vector<int64_t> end;
  trail_items(n, begin, 6 * (int64_t)cus, 0, &tiles, &end, RATIOS_TRAIL_KEEP, RATIOS_TRAIL_SPREAD, true);
  items->clear();
  for (unsigned int i : tiles)
    for (unsigned int part = 0; part < ((i & TRAIL_UPDATE) ? 8u / RATIOS_TRAIL_U : 1u); ++part)
      items->push_back((i & ~TRAIL_KEEP) | part * RATIOS_TRAIL_PART);
}

// Group counters of a barrier with n arrivals, and of the barriers of L layers with n together (group_line).
inline size_t arrival_groups(int64_t n) { return (size_t)((n + ARRIVE_SUB - 1) / ARRIVE_SUB); }
inline size_t group_lines(int64_t n, int64_t L) { return arrival_groups(n) + (size_t)L; }

// Whether the plain ratio pass runs in k_ratios_apply_hist's launch instead of its own, which saves that launch (5.6 us and
// a gap) and costs its tiles the occupancy of their own kernel and every wavefront the values of StepTerms.  A step, us, in a
// launch of its own / in that one, rest tiles and 8192-element tiles: 240, 1424 86.4 / 83.6; 1209, 2232 131.3 / 128.8; 468,
// 2580 140.6 / 138.8; 433, 1713 110.1 / 109.3; 286, 3920 188.4 / 188.7; 1600, 4800 236.9 / 241.7; 647, 5135 242 / 239.7; 1297, 9677
// 448 / 445; 710, 11239 501 / 511; 997, 25803 1134 / 1140; 1430, 40908 1716 / 1728.
// (The line: 5 rest tiles and 20 tiles a CU.)
// Since the rest tiles' update is in that launch too, where there are no large tiles (four steps, us, a launch of its own / in that one: 11 M 319.5 / 309.8,
// 30 M 692 / 681, 18 M with a 16-bit copy 507.5 / 500, 27 M 683.6 / 668.6, 4.2 M 187.0 / 180.4, five of 2800x2800 950.6 / 945.5), that line lies at
// 40 tiles a CU for layers that leave room for others beside them (of at most 2 tiles a CU on average), us: 26 and 40 of 1300x1300 946.5 /
// 930, 1388.6 / 1375.6; BERT shapes of 49 to 59 M 1068 / 1058, 1274 / 1262, with a 16-bit copy 1287 / 1263; a GPT shape of 75 M 1608 / 1602; but
// eight of 2801x2801 1464 / 1479.
inline bool rest_in_launch(int n_rest_tiles, int n_listed, int n_big, int cus, int64_t n_layers = 0 /* listed */) {
  const int line = (n_big == 0 && n_listed <= 2 * cus * n_layers) ? 40 : 20;
  return n_listed > 0 && n_rest_tiles <= 5 * cus && n_listed + n_big <= line * cus;
}

// Arrivals of a layer of the barrier kernels that are counted in one level, by their listed tiles.  (Figures at
// barrier_arrive.  The lists that gain in layers of up to 512 tiles have at most 24 tiles a CU, those that lose 70.)
inline int arrivals_one_level(int n_listed_tiles, int cus) { return n_listed_tiles > 40 * cus ? 512 : ARRIVE_ONE_LEVEL; }


// Spans per tile of the server kernel without a barrier (k_server_unpack_avg).  With few workers a tile of 1024 elements is a
// chain of latencies (scales, LDS, words) around a few additions: larger ones where the chunk still makes rounds of
// the device; with many workers the additions bind, and more, smaller workgroups hide them better.  The call, us, 1 / 2 / 4 spans
// (above 1 with chunk_ticket, which costs less than a launch by then), workers, tiles of 1024 elements:
//   1, 107520 202 / 157 / 151; 2, 53760 111 / 86.7 / 78.6; 2, 5504 16.0 / 13.4 / 12.8; 4, 26880 67.3 / 43.6 / 43.7; 4, 2752 11.4 /
//   9.4 / 9.9; 8, 13440 31.3 / 26.2 / 26.6; 8, 4096 13.1 / 11.4 / 12.6; 8, 2048 10.5 / 8.9 / 9.2; 8, 1376 10.2 / 7.9 / 9.1; 16, 6720 21.3 / 19.8 / 20.3;
//   16, 2048 10.0 / 10.5 / 11.1; 16, 688 10.2 / 8.1 / 9.3; 32, 3360 17.2 / 17.2 / 21.0; 32, 2048 12.3 / 13.3 / 13.9; 64, 5254 33.7 / 34.4 / 39.9; 64, 1680
//   15.7 / 18.1 / 19.2; 128, 840 15.2 / 17.7 / 30.0
// with one span and the ticket: 8, 2048 8.9; 8, 1376 8.0; 16, 2048 9.6; 16, 688 7.7; 32, 2048 12.2; 64, 1680 15.5 (single calls in a row: a second launch
// costs what it does not in a step, whose kernels follow each other).
// (The line: 16 and 8 tiles a CU, one or two rounds of the device.)
inline int server_spans(int64_t W, int tpc, int cus) {
  if (W <= 2 && tpc >= 16 * cus) return 4;
  return (W <= 32 && tpc >= 8 * cus) ? 2 : 1;
}

// Arrivals at the layers' barriers in k_ratios_apply_hist with the plain ratio pass in its launch: the listed tiles of each
// layer, then its segments outside listed and big tiles (those in position order).
struct ArrivalPlan {
  std::vector<int> arr0;                   // [L] arrivals of the layers before
  std::vector<int> alone;                  // layers without arrivals
  std::vector<int> skip_first, skip_end;   // [L] first / one past the last of the layer's segments that no rest tile forms
  int64_t n_arrivals = 0;
};
inline void plan_arrivals(const SplitPlan& pl, const Tiling& tm, int64_t L, ArrivalPlan* ap) {
  ap->arr0.resize((size_t)L);
  ap->skip_first = pl.seg_first;
  ap->skip_end = pl.seg_end;
  for (int64_t l = 0; l < L; ++l) {
    const size_t i = (size_t)l;
    if (pl.big_n[i]) {
      ap->skip_first[i] = pl.big_seg_first[i];
      ap->skip_end[i] = pl.big_seg_end[i];
    }
    ap->arr0[i] = (int)ap->n_arrivals;
    const int n = layer_arrivals(pl.n_listed[i], tm.layer_seg0[i], ap->skip_first[i], ap->skip_end[i], tm.layer_seg0[i + 1]);
    if (n == 0) ap->alone.push_back((int)l);
    ap->n_arrivals += n;
  }
}

// The update of the rest tiles in that launch too: its last workgroups wait until every c_t is there.  How many events that takes: a
// layer without arrivals; a layer that its last arrival finishes; a rest tile that finishes layers of its own between
// its first and its last segment.
inline int64_t coefficient_events(const SplitPlan& pl, const Tiling& tm, int64_t L, const ArrivalPlan& ap) {
  std::vector<char> finished(pl.has_listed.begin(), pl.has_listed.end());   // by its last arrival
  int64_t n = (int64_t)ap.alone.size();
  for (int t : pl.rest_ratio_tiles) {
    const int s0 = tm.tile_seg0[(size_t)t], s1 = tm.tile_seg0[(size_t)t + 1];
    finished[(size_t)tm.seg_layer[(size_t)s0]] = finished[(size_t)tm.seg_layer[(size_t)s1 - 1]] = 1;
    n += (s1 - s0 > 2);
  }
  for (int64_t l = 0; l < L; ++l) n += finished[(size_t)l];
  return n;
}

// The tiles and segments of one SmallPlan (no HIP call).  lagging: per 1024-element span (tm's tiling).
inline void small_tiles(const Tiling& t, int U, const Tiling& tm, const std::vector<int64_t>& h_off, int64_t n_c, int64_t L,
                 const std::vector<unsigned char>& lagging, std::vector<SmallTile>* tiles) {
  tiles->resize((size_t)t.n_tiles);
  for (int64_t i = 0; i < t.n_tiles; ++i) {
    const int64_t c = i / t.tpc, b = i % t.tpc;
    const int64_t tile0 = c * n_c + b * (int64_t)SPAN * U, tile1 = std::min(tile0 + (int64_t)SPAN * U, (c + 1) * n_c);
    SmallTile& st = (*tiles)[(size_t)i];
    st.l0 = t.first[(size_t)i];
    st.seg0 = t.tile_seg0[(size_t)i];
    st.nseg = t.tile_seg0[(size_t)i + 1] - st.seg0;
    const bool inside = st.l0 < L && tile1 <= h_off[(size_t)st.l0 + 1];
    const bool lag = inside && lagging[(size_t)(c * tm.tpc + b * U)];   // (a lagging span's 8192-element tile lags as a whole)
    st.chunk_kind = (int)(c << 2) | (inside ? 1 : 0) | (lag ? 2 : 0);
    st.l_last = st.nseg > 0 ? t.seg_layer[(size_t)(st.seg0 + st.nseg - 1)] : st.l0;
    auto total = [&](int l) { return l < L ? t.layer_seg0[(size_t)l + 1] - t.layer_seg0[(size_t)l] : 0; };
    st.n_first = total(st.l0);
    st.n_last = total(st.l_last);
    st.pad = 0;
  }
}

// What the choice of a tile size rests on, without its tables.
struct SmallShape {
  int64_t tpc = 0, n_tiles = 0;
  int max_seg = 1;        // most layers that meet one tile
  int max_arrivals = 0;   // most tiles that one layer meets
  int mixed_spans = 0;    // 1024-element spans of the longest tile that is not wholly inside one layer
};
inline SmallShape small_shape(int U, const std::vector<int64_t>& h_off, int64_t n_c, int64_t W, int64_t L) {
  const int64_t tile = (int64_t)SPAN * U;
  SmallShape sh;
  sh.tpc = (n_c + tile - 1) / tile;
  sh.n_tiles = sh.tpc * W;
  int64_t cur = -1;
  int seg = 0;
  for (int64_t l = 0; l < L; ++l) {
    const int64_t a = h_off[(size_t)l], e = h_off[(size_t)l + 1];
    if (e == a) continue;
    const int64_t c = (e - 1) / n_c, b = (e - 1) % n_c / tile;
    const int64_t t0 = a / n_c * sh.tpc + a % n_c / tile, t1 = c * sh.tpc + b;
    seg = (t0 == cur) ? seg + 1 : 1;
    sh.max_seg = std::max(sh.max_seg, seg);
    if (t1 > t0) seg = 1;
    cur = t1;
    sh.max_arrivals = (int)std::max<int64_t>(sh.max_arrivals, t1 - t0 + 1);
    const int64_t in_chunk = b * tile, len = std::min(tile, n_c - in_chunk);
    if (e < c * n_c + in_chunk + len) sh.mixed_spans = (int)std::max<int64_t>(sh.mixed_spans, (len + SPAN - 1) / SPAN);
  }
  return sh;
}
// What sets the tile sizes apart, in ns: a workgroup's own chain of loads and divisions, the look-ups with which the threads
// of a tile that meets several layers (or the padding) go through its spans, the segments of such a tile, which its wavefronts
// finish in turn, and many workgroups.  k_ratios_apply_small reads a slot for every tile of its layer, which costs next to nothing; only
// workgroups of several layers side by side cost it time (those of one layer, up to 1600, do not).  k_warmup_small's arrivals queue
// at a counter, in two levels from SMALL_ONE_LEVEL on.
// Compression steps and LAMB steps at U = 1 / 2 / 4, us (256 CUs; -: does not fit; those below 20 us are bound by the host):
//   elements, tensors      steps with the variance's history       steps without             LAMB steps
//   0.18 M, 46 tensors     18.8 / 19.1 / 23.5                      17.6 / 18.8 / 23.8        9.2 / 11.3 / 16.9
//   0.41 M, one            18.5 / 18.7 / 20.2                      17.5 / 18.7 / 20.0        7.2 / 7.2 / 9.0
//   0.50 M, four, shared   19.4 / 19.4 / 23.4                      19.0 / 19.4 / 23.7        8.8 / 7.6 / 13.5
//   0.52 M, eight          18.7 / 18.8 / 20.9                      18.0 / 18.5 / 20.8        6.8 / 7.0 / 8.6
//   0.64 M, one            19.3 / 20.1 / 21.8                      19.1 / 19.8 / 21.2        8.3 / 8.3 / 9.7
//   0.90 M, one, padded    20.5 / 22.2 / 26.4                      20.2 / 22.2 / 27.0        9.3 / 10.6 / 14.6
//   0.92 M, four           21.8 / 21.7 / 22.7                      22.6 / 21.1 / 21.8        8.0 / 8.5 / 9.2
//   0.99 M, eight, shared  22.1 / 23.1 / 27.9                      22.3 / 23.2 / 27.7        8.1 / 11.1 / 16.3
//   1.00 M, hundred        21.6 / 24.0 / 28.8                      21.5 / 23.9 / 28.9        10.5 / 12.8 / 17.4
//   1.05 M, four           21.1 / 21.0 / 23.2                      20.9 / 20.2 / 22.3        7.9 / 8.6 / 9.1
//   1.2 M, three           22.9 / 23.4 / 23.8                      23.6 / 23.4 / 22.9        8.9 / 9.1 / 10.5
//   1.31 M, five           23.7 / 23.4 / 25.0                      23.9 / 22.7 / 24.1        8.8 / 9.5 / 10.9
//   1.5 M, 110 tensors     25.5 / 26.8 / 31.5                      25.6 / 26.4 / 31.4        12.3 / 14.2 / 19.6
//   1.57 M, six            25.7 / 24.1 / 25.0                      26.8 / 23.3 / 24.1        9.5 / 10.0 / 11.3
//   1.60 M, one, padded    25.6 / 25.6 / 27.3                      24.7 / 24.4 / 27.5        12.4 / 11.0 / 15.0
//   1.64 M, one            25.0 / 25.4 / 25.4                      24.3 / 24.4 / 24.3        11.5 / 11.1 / 12.1
//   1.64 M, sixteen        26.4 / 24.8 / 24.8                      26.7 / 23.9 / 24.0        9.8 / 9.7 / 11.2
//   1.84 M, seven          - / 25.6 / 25.7                         - / 24.6 / 24.6           - / 10.8 / 11.5
//   2.4 M, one             - / - / 30.9                            - / - / 29.7              - / - / 14.2
// The choice is the fastest of these and of six lists like them or within 3.4 %, on average within half a per cent, but for the LAMB step of 1.57 M in six
// tensors (two spans, 5 % behind one).
constexpr int SMALL_ONE_LEVEL = 128;   // (figures at k_warmup_small)
inline int64_t small_cost(int U, const SmallShape& sh, bool by_slots, int cus) {
  int64_t c = (U == 1 ? 0 : U == 2 ? 500 : 2000) + 2500 * std::max(sh.mixed_spans - 1, 0) + 100 * sh.max_seg +
              3 * std::max<int64_t>(by_slots ? sh.n_tiles - sh.max_arrivals - 11 * cus / 8 : sh.n_tiles - 4 * cus, 0);
  if (!by_slots)
    c += 13 * (sh.max_arrivals <= SMALL_ONE_LEVEL ? sh.max_arrivals : ARRIVE_SUB + sh.max_arrivals / ARRIVE_SUB + 46 /* another trip */);
  return c;
}
// The index in U = 1, 2, 4 (fits[i]: the tiles of sh[i] fit on the device; the smallest of equals), -1 if none fits.
inline int small_choice(const SmallShape (&sh)[3], const bool (&fits)[3], bool by_slots, int cus) {
  int best = -1;
  for (int i = 0; i < 3; ++i)
    if (fits[i] && (best < 0 || small_cost(1 << i, sh[i], by_slots, cus) < small_cost(1 << best, sh[best], by_slots, cus))) best = i;
  return best;
}
// A list all of whose parameters lie in 8192-element tiles of layers that the barrier kernels take keeps those where one layer
// has more than this many 1024-element spans.  Steps of one tensor, or two, us, in one launch / in the barrier kernel, with the
// variance's history, without, LAMB: 1.6 M (1600 spans) 25.5 / 28.8, 24.8 / 29.4, 11.3 / 16.3; two of 1.6 M 36.8 / 36.7, 35.9 /
// 37.3, 16.7 / 19.4; 2.4 M (2304) 31.2 / 33.0, 30.4 / 34.2, 15.3 / 18.9; 2.9 M (2880) 33.4 / 34.8, 32.9 / 36.3, 15.6 / 19.8; 3.2 M (3136) 36.4 / 36.0, 35.5 /
// 37.8, 17.2 / 20.4.  (One limit for all calls; compression steps with the history are what runs most.  By these figures it could lie at 3000 spans, and
// nowhere for the LAMB step.)
constexpr int64_t SMALL_MAX_SPANS = 2800;

// Tilings of the tile sizes that a SmallPlan may take, formed when first asked for, and their shapes.
struct SmallTilings {
  const Tiling& tm;       // U = 1
  SmallShape sh[3];       // U = 1, 2, 4 (n_tiles = 0: more tiles than any device holds)
  Tiling t2, t4;
  SmallTilings(const Tiling& t, int64_t n_c, int64_t W, int64_t L, const std::vector<int64_t>& h_off) : tm(t) {
    for (int i = 0; i < 3; ++i)
      if ((n_c + ((int64_t)SPAN << i) - 1) / ((int64_t)SPAN << i) * W <= 4096) sh[i] = small_shape(1 << i, h_off, n_c, W, L);
  }
  const Tiling* get(int U, int64_t n_c, int64_t W, int64_t L, const std::vector<int64_t>& h_off) {
    if (U == 1) return &tm;
    Tiling* t = (U == 2) ? &t2 : &t4;
    if (t->n_tiles == 0 && !build_tiling((int64_t)SPAN * U, n_c, W, L, h_off, t)) return nullptr;
    return t;
  }
};

}  // namespace obk
