// Host-side work list of the persistent prefill kernel: items, and one chain of items per workgroup.
#pragma once

#include <algorithm>
#include <vector>

#include "internal.h"

namespace spd {

// One workgroup per compute unit walks a chain of work items.  Workgroup b runs on XCD b % xcds
// (round-robin dispatch), and each XCD has its own L2, so all items that read the same K, V - the
// query tiles and head groups of one (request, KV head) "unit" - go to chains of the same XCD.
// Units are spread over the XCDs longest-first; inside an XCD the items are dealt longest-first onto
// the least-loaded chain (weight = KV tiles to visit + a fixed per-item cost: measured, an item costs what
// four tiles cost beyond its own, in query loads, output stores and a first tile that sets the softmax
// reference), and every chain is
// ordered by unit, so that the chains of an XCD work on the same unit at about the same time.
// With fewer units than XCDs the items themselves are dealt round-robin.
// Without `persistent` there is one workgroup per item (or part of one, below) instead (chains of length one, handed out by the
// hardware in launch order: the XCDs' queues interleaved, each queue heaviest unit first): for
// partitions on which a launch of exactly one workgroup per compute unit does not get one compute
// unit each.
constexpr long ITEM_COST_TILES = 4;

// (kept small: large batches sort many of them)
struct PrefillItem {
  int32_t row0, len, q_tile, head0, kv_row0, q_off, tiles, unit;
  int32_t weight() const { return tiles + (int32_t)ITEM_COST_TILES; }
  PrefillWork part(int32_t kt0, int32_t kt1, int32_t number) const { return PrefillWork{row0, len, q_tile, head0, kv_row0, q_off, kt0, kt1, number}; }
  PrefillWork whole() const { return part(0, tiles, -1); }
};

// ---- Sharing items out by keys.  A step with few items, or with a few long ones (short pieces of prompts behind long cached
// prefixes), leaves most compute units idle while the longest item runs.  Then the chains get about the same weight, and an
// item that none of them has room for is cut: each part leaves its sums in memory, and a second launch adds them up.  Whole step, 32
// heads: 2 pieces of up to 14 tokens behind 2805 on 256 CUs 63.9 -> 38 us; 512 tokens behind 8000 on 128 CUs 193 -> 121; one token behind
// 8000, 64 heads on 64 CUs 186 -> 61; 4 pieces of 355 .. 867 behind up to 5023 on 256 CUs (312 items of up to 89 tiles, mean load 57, now
// at most 61; with all compute units busy the clock is lower) 159 -> 139.
// A part pays its item's fixed cost again and one tile for writing its sums; the second launch costs what six tiles do.  Parts are no
// shorter than eight tiles.  No part begins behind the item's first row, so that every row has keys in every part.
constexpr long PART_COST_TILES = 1, MERGE_COST_TILES = 6, LEAST_PART_TILES = 8;

struct PrefillPlace { PrefillWork w; int chain; };

// Deals the items of one XCD, longest first, to n_chains chains of weight `cap`: whole into the chain whose room they fill best, else in
// parts, from the chain with most room on.  `places` (in the order of the items and of their parts, which are not numbered yet: -2) null:
// only asks.  false: they do not fit.
inline bool deal_parts(const std::vector<PrefillItem>& items, int n_chains, long cap, int block_m, std::vector<PrefillPlace>* places) {
  std::vector<long> room((size_t)n_chains, cap);
  for (const PrefillItem& item : items) {
    const int32_t last_cut = (item.q_off + item.q_tile * block_m) / 64;   // the tile of the item's first row
    int32_t k0 = 0;
    while (k0 < item.tiles) {
      const long rest = item.tiles - k0 + ITEM_COST_TILES + (k0 > 0 ? PART_COST_TILES : 0);
      int best = -1, widest = 0;
      for (int c = 0; c < n_chains; ++c) {
        if (room[(size_t)c] >= rest && (best < 0 || room[(size_t)c] < room[(size_t)best])) best = c;
        if (room[(size_t)c] > room[(size_t)widest]) widest = c;
      }
      int32_t k1 = item.tiles;
      if (best >= 0) {
        room[(size_t)best] -= rest;
      } else {
        best = widest;
        long take = std::min<long>(room[(size_t)best] - ITEM_COST_TILES - PART_COST_TILES, item.tiles - k0 - LEAST_PART_TILES);
        take = std::min<long>(take, last_cut - k0);
        if (take < LEAST_PART_TILES) return false;
        k1 = k0 + (int32_t)take;
        room[(size_t)best] -= take + ITEM_COST_TILES + PART_COST_TILES;
      }
      if (places) places->push_back(PrefillPlace{item.part(k0, k1, k0 > 0 || k1 < item.tiles ? -2 : -1), best});
      k0 = k1;
    }
  }
  return true;
}

// The work list and the merge list, if every chain can be that much shorter than the longest load `longest` of whole items; else nothing.
// xq: every XCD's items.  `persistent`: workgroup c xcds + x takes chain c of XCD x.  Without, the chains only say where to cut, and every
// item and part is a workgroup of its own, each XCD's longest first: where the phases' masks overlap, the other phase's
// workgroups then get a compute unit whenever a part ends, not with the kernel.  (The four pieces above on 256 CUs, both phases there: as
// chains 136 us, as workgroups 137, in the order of the chains 147.  A decode step of 16 requests of 1000 tokens that comes in the
// middle of it ends 111 us later beside chains, 105 beside workgroups, and 79 beside whole items, which leave it compute units of
// their own; pairs of both steps, queued, 148, 146 and 159 us.)
inline bool share_out(std::vector<std::vector<PrefillItem>>& xq, int per_xcd, bool persistent, long longest, int block_m, std::vector<PrefillWork>& work,
                      std::vector<int32_t>& chain, std::vector<PrefillMerge>& merge) {
  const long most = longest * 9 / 10 - MERGE_COST_TILES;   // a tenth ahead, or it is not worth another launch
  long cap = LEAST_PART_TILES + ITEM_COST_TILES + PART_COST_TILES;
  for (const auto& items : xq) {
    long sum = 0;
    for (const PrefillItem& item : items) sum += item.weight();
    cap = std::max(cap, (sum + per_xcd - 1) / per_xcd);
  }
  if (cap > most) return false;
  const size_t xcds = xq.size();
  for (auto& items : xq) std::stable_sort(items.begin(), items.end(), [](const PrefillItem& a, const PrefillItem& b) { return a.tiles > b.tiles; });
  for (size_t x = 0; x < xcds;) {                 // the least that the items of all XCDs fit into
    if (deal_parts(xq[x], per_xcd, cap, block_m, nullptr)) {
      ++x;
    } else {
      cap += 1 + cap / 24;
      if (cap > most) return false;
      x = 0;                                      // (what fitted into less need not fit into more)
    }
  }
  merge.clear();
  std::vector<std::vector<PrefillPlace>> places(xcds);
  int32_t n_parts = 0;
  size_t most_places = 0, n_places = 0;
  for (size_t x = 0; x < xcds; ++x) {
    (void)deal_parts(xq[x], per_xcd, cap, block_m, &places[x]);
    for (PrefillPlace& p : places[x]) {
      if (p.w.part == -1) continue;
      if (p.w.kt0 == 0) merge.push_back(PrefillMerge{p.w.row0, p.w.len, p.w.q_tile, p.w.head0, n_parts, 0});
      p.w.part = n_parts++;
      ++merge.back().n_parts;
    }
    n_places += places[x].size();
    most_places = std::max(most_places, places[x].size());
  }
  if (!persistent) {
    for (auto& of_xcd : places)
      std::stable_sort(of_xcd.begin(), of_xcd.end(), [](const PrefillPlace& a, const PrefillPlace& b) { return a.w.kt1 - a.w.kt0 > b.w.kt1 - b.w.kt0; });
    work.clear();
    work.reserve(n_places);
    chain.clear();
    for (size_t i = 0; i < most_places; ++i)
      for (size_t x = 0; x < xcds; ++x) {
        chain.push_back((int32_t)work.size());
        if (i < places[x].size()) work.push_back(places[x][i].w);
      }
    chain.push_back((int32_t)work.size());
    return true;
  }
  chain.assign(xcds * (size_t)per_xcd + 1, 0);
  for (size_t x = 0; x < xcds; ++x)
    for (const PrefillPlace& p : places[x]) ++chain[(size_t)p.chain * xcds + x + 1];
  for (size_t c = 0; c + 1 < chain.size(); ++c) chain[c + 1] += chain[c];
  std::vector<int32_t> at(chain.begin(), chain.end() - 1);
  work.resize(n_places);
  for (size_t x = 0; x < xcds; ++x)
    for (const PrefillPlace& p : places[x]) work[(size_t)at[(size_t)p.chain * xcds + x]++] = p.w;
  return true;
}

// `persistent`: a chain per compute unit; `merge` null: no item is shared out.
// (Lists in a few flat arrays: with a vector per unit, per XCD and per chain this took 13 of the 20 us of a step of 8 short prompts.)
inline void build_prefill_chains(const int32_t* cu_seqlens, const int32_t* prefix_lens, const int32_t* kv_cu, int n_req,
                                 int H, int Hkv, int xcds, int share, bool persistent, std::vector<PrefillWork>& work,
                                 std::vector<int32_t>& chain, std::vector<PrefillMerge>* merge) {
  const int G = H / Hkv, hb = prefill_heads_per_block(G), bm = prefill_block_m(G), groups = G / hb;
  // items, unit after unit, each unit's longest first
  const size_t n_units = (size_t)n_req * (size_t)Hkv;
  size_t n_items = 0;
  for (int r = 0; r < n_req; ++r) n_items += (size_t)((cu_seqlens[r + 1] - cu_seqlens[r] + bm - 1) / bm) * (size_t)(groups * Hkv);
  std::vector<PrefillItem> items;
  items.reserve(n_items);
  std::vector<long> unit_weight(n_units);
  std::vector<uint32_t> unit_first(n_units + 1);
  long heaviest = 0;
  for (int r = 0; r < n_req; ++r) {
    const int32_t row0 = cu_seqlens[r], len = cu_seqlens[r + 1] - row0;
    const int32_t q_off = prefix_lens ? prefix_lens[r] : 0, kv_row0 = prefix_lens ? kv_cu[r] : row0;
    const int tiles = (len + bm - 1) / bm;
    heaviest = std::max(heaviest, (long)((int64_t)q_off + len + 63) / 64 + ITEM_COST_TILES);
    for (int g = 0; g < Hkv; ++g) {
      const size_t u = (size_t)r * (size_t)Hkv + (size_t)g;
      unit_first[u] = (uint32_t)items.size();
      long weight = 0;
      for (int t = tiles - 1; t >= 0; --t)
        for (int hg = 0; hg < groups; ++hg) {
          const long kv_tiles = (q_off + std::min<long>(len, (long)(t + 1) * bm) + 63) / 64;
          items.push_back(PrefillItem{row0, len, t, g * G + hg * hb, kv_row0, q_off, (int32_t)kv_tiles, (int32_t)u});
          weight += kv_tiles + ITEM_COST_TILES;
        }
      unit_weight[u] = weight;
    }
  }
  unit_first[n_units] = (uint32_t)items.size();
  if (merge) merge->clear();
  const bool even = share >= xcds && share % xcds == 0;
  if (persistent && !even) xcds = 1;
  const int per_xcd = std::max(1, share / xcds);  // chains per XCD, or workgroups that run there at a time
  // xq: every XCD's items, one XCD after the other from xq_first[x] on; units heaviest first, with fewer units than XCDs item by item
  std::vector<uint32_t> xq(n_items), xq_first((size_t)xcds + 1, 0);
  if (n_units >= (size_t)xcds) {
    std::vector<uint32_t> order(n_units), xcd_of(n_units);
    for (size_t i = 0; i < n_units; ++i) order[i] = (uint32_t)i;
    std::stable_sort(order.begin(), order.end(), [&](uint32_t a, uint32_t b) { return unit_weight[a] > unit_weight[b]; });
    std::vector<long> load((size_t)xcds, 0);
    for (uint32_t u : order) {
      const size_t x = (size_t)(std::min_element(load.begin(), load.end()) - load.begin());
      load[x] += unit_weight[u];
      xcd_of[u] = (uint32_t)x;
      xq_first[x + 1] += unit_first[u + 1] - unit_first[u];
    }
    for (int x = 0; x < xcds; ++x) xq_first[(size_t)x + 1] += xq_first[(size_t)x];
    std::vector<uint32_t> at(xq_first.begin(), xq_first.end() - 1);
    for (uint32_t u : order)
      for (uint32_t i = unit_first[u]; i < unit_first[u + 1]; ++i) xq[at[xcd_of[u]]++] = i;
  } else {
    for (int x = 0; x < xcds; ++x) xq_first[(size_t)x + 1] = xq_first[(size_t)x] + (uint32_t)((n_items + (size_t)(xcds - 1 - x)) / (size_t)xcds);
    for (size_t i = 0; i < n_items; ++i) xq[xq_first[i % (size_t)xcds] + i / (size_t)xcds] = (uint32_t)i;
  }
  auto share_items = [&](long longest) -> bool {
    std::vector<std::vector<PrefillItem>> lists((size_t)xcds);
    for (int x = 0; x < xcds; ++x)
      for (uint32_t i = xq_first[(size_t)x]; i < xq_first[(size_t)x + 1]; ++i) lists[(size_t)x].push_back(items[xq[i]]);
    return share_out(lists, per_xcd, persistent, longest, bm, work, chain, *merge);
  };
  // (at most the heaviest item's weight is to be gained, and with many items per compute unit whole ones balance well enough)
  const bool may_share = merge && even && n_items <= 8 * (size_t)share && heaviest > 2 * LEAST_PART_TILES;
  std::vector<long> load((size_t)per_xcd);
  long longest = 0;                               // load of the chain, or of the compute unit, that is done last
  if (!persistent) {
    if (may_share) {
      for (int x = 0; x < xcds; ++x) {
        std::fill(load.begin(), load.end(), 0);
        for (uint32_t i = xq_first[(size_t)x]; i < xq_first[(size_t)x + 1]; ++i) *std::min_element(load.begin(), load.end()) += items[xq[i]].weight();
        longest = std::max(longest, *std::max_element(load.begin(), load.end()));
      }
      if (share_items(longest)) return;
    }
    uint32_t most = 0;
    for (int x = 0; x < xcds; ++x) most = std::max(most, xq_first[(size_t)x + 1] - xq_first[(size_t)x]);
    work.clear();
    work.reserve(n_items);
    chain.clear();
    chain.reserve((size_t)most * (size_t)xcds + 1);
    for (uint32_t i = 0; i < most; ++i)
      for (int x = 0; x < xcds; ++x) {            // workgroup i * xcds + x runs on XCD x
        chain.push_back((int32_t)work.size());
        if (xq_first[(size_t)x] + i < xq_first[(size_t)x + 1]) work.push_back(items[xq[xq_first[(size_t)x] + i]].whole());
      }
    chain.push_back((int32_t)work.size());
    return;
  }
  // Unit after unit (in the order the XCD took them), each unit's items longest-first onto the chain
  // with the least load so far: every chain then holds about the same weight of EVERY unit, so the
  // chains of an XCD pass from one unit to the next at about the same time and the XCD's L2 has to
  // hold one or two units' K, V, not all of them.  (Dealt over all units at once the chains were as
  // well balanced in total, but drifted apart unit by unit, and K, V crossed HBM four times.)
  std::vector<uint32_t> chain_of(n_items);
  chain.assign((size_t)share + 1, 0);
  for (int x = 0; x < xcds; ++x) {
    std::fill(load.begin(), load.end(), 0);
    for (uint32_t i = xq_first[(size_t)x]; i < xq_first[(size_t)x + 1]; ++i) {
      const size_t c = (size_t)(std::min_element(load.begin(), load.end()) - load.begin());
      load[c] += items[xq[i]].weight();
      chain_of[xq[i]] = (uint32_t)(c * (size_t)xcds) + (uint32_t)x;   // workgroup id = chain slot * xcds + xcd
      ++chain[c * (size_t)xcds + (size_t)x + 1];
    }
    longest = std::max(longest, *std::max_element(load.begin(), load.end()));
  }
  if (may_share && share_items(longest)) return;
  // every chain in the order of the units
  for (int c = 0; c < share; ++c) chain[(size_t)c + 1] += chain[(size_t)c];
  std::vector<int32_t> at(chain.begin(), chain.end() - 1);
  work.resize(n_items);
  for (size_t i = 0; i < n_items; ++i) work[(size_t)at[chain_of[i]]++] = items[i].whole();
}

// Tiles of 64 keys that the longest item visits.
inline int longest_item(const int32_t* cu_seqlens, const int32_t* prefix_lens, int n_req) {
  int most = 0;
  for (int r = 0; r < n_req; ++r) most = std::max(most, (cu_seqlens[r + 1] - cu_seqlens[r] - 1 + (prefix_lens ? prefix_lens[r] : 0)) / 64 + 1);
  return most;
}

}  // namespace spd
