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
  PrefillWork work() const { return PrefillWork{row0, len, q_tile, head0, kv_row0, q_off}; }
};

// ---- Sharing items out by keys.  A step with few items, or with a few long ones (short pieces of prompts behind long cached
// prefixes), leaves most compute units idle while the longest item runs.  Then the chains get about the same weight, and an
// item that none of them has room for is cut: each part leaves its sums in memory, and a second launch adds them up.  Whole step, 32
// heads: 2 pieces of up to 14 tokens behind 2805 on 256 CUs 63.9 -> 38 us; 512 tokens behind 8000 on 128 CUs 193 -> 121; one token behind
// 8000, 64 heads on 64 CUs 186 -> 61; 4 pieces of 355 .. 867 behind up to 5023 on 256 CUs (312 items of up to 89 tiles, mean load 57, now
// at most 65; with all compute units busy the clock is lower) 155 -> 137.
// A part pays its item's fixed cost again and one tile for writing its sums; the second launch costs what six tiles do.  Parts are no
// shorter than eight tiles.  No part begins behind the item's first row, so that every row has keys in every part.
constexpr long PART_COST_TILES = 1, MERGE_COST_TILES = 6, LEAST_PART_TILES = 8;
// With more than MANY_PIECES items and parts the host takes so much longer to deal and stage them that MANY_PIECES_TILES more have to be
// won: 1500 tokens on 256 CUs (192 items of up to 28 tiles, 264 pieces of up to 19) 45.7 -> 47.3 us, waited for 58 -> 68, 1659 behind 519 (39 tiles,
// 28) 66.3 -> 63.6 and 78.5 -> 87.3; where more is won both fall (100 tokens behind 2000, four times: 256 pieces, 37 -> 14 tiles, 68 -> 51
// and 80 -> 73).
constexpr size_t MANY_PIECES = 192;
constexpr long MANY_PIECES_TILES = 5;
// Where the parts have to end for whole items that end at `longest`: a tenth ahead, or it is not worth another launch; with a chain per compute
// unit ten tiles do (pieces of 893, 207 and 547 tokens behind 4118, 3798 and 7358 on 128 CUs, 188 tiles -> 167: 266.6 -> 246.9 us, waited for 303 ->
// 284; 20 batches of 119 to 315 tiles won 5 to 10 % queued and 2 to 9 waited for; as workgroups of their own 3 to 6, and waited for up to 4
// were lost).
inline long shared_end(long longest, size_t n_pieces, bool persistent) {
  const long ahead = persistent ? std::min((longest + 9) / 10, 10l) : (longest + 9) / 10;
  return longest - ahead - MERGE_COST_TILES - (n_pieces > MANY_PIECES ? MANY_PIECES_TILES : 0);
}
// The same ahead of the search: every item that is longer than that will be two pieces at least.
inline long shared_end(long longest, const std::vector<PrefillItem>& items, bool persistent) {
  const long end = shared_end(longest, 0, persistent);
  size_t n = items.size();
  for (const PrefillItem& item : items) n += item.weight() > end;
  return shared_end(longest, n, persistent);
}

struct PrefillPiece { uint32_t item; int32_t kt0, kt1; uint32_t chain; };

// The whole items as they were dealt (`load` of every chain, XCD after XCD) and what has to move for no chain to exceed a `cap`: a chain
// with too much cuts its longest item so that it ends at the cap, and what is left over goes where it fits best, in further parts
// where it fits nowhere.  So the search looks at the chains with too much and at what they give away, not at every item.  Host time of
// dealing a batch, against dealing all items anew for every cap that is tried: 4 pieces of 355 .. 867 behind up to 5023 on 256 CUs
// 23 -> 10 us (dealt whole: 3); of random batches of 6 to 16 pieces, nearly none of which is cut, 31 -> 13 on average, 127 -> 38
// at most.  A step that is waited for has it ahead of everything else: those 4 pieces 168 -> 159 us.
class PrefillShares {
 public:
  PrefillShares(const std::vector<PrefillItem>& items, const std::vector<uint32_t>& chain_of, const std::vector<long>& load, int per_xcd, int block_m,
                bool persistent)
      : items_(items), chain_of_(chain_of), load_(load), per_xcd_((size_t)per_xcd), block_m_(block_m), persistent_(persistent) {}
  // The pieces that take the place of some whole items, ordered by item and keys, if every chain can be that much shorter than the longest.
  bool find(std::vector<PrefillPiece>& pieces) {
    const long longest = *std::max_element(load_.begin(), load_.end());
    long hi = shared_end(longest, items_, persistent_);
    long lo = LEAST_PART_TILES + ITEM_COST_TILES + PART_COST_TILES;
    for (size_t x = 0; x < load_.size(); x += per_xcd_) {
      long sum = 0;
      for (size_t c = x; c < x + per_xcd_; ++c) sum += load_[c];
      lo = std::max(lo, (sum + (long)per_xcd_ - 1) / (long)per_xcd_);
    }
    if (lo > hi) return false;
    first_.assign(load_.size() + 1, 0);
    for (uint32_t c : chain_of_) ++first_[c + 1];
    for (size_t c = 0; c < load_.size(); ++c) first_[c + 1] += first_[c];
    std::vector<uint32_t> at(first_.begin(), first_.end() - 1);
    of_chain_.resize(items_.size());
    for (size_t i = 0; i < items_.size(); ++i) {  // (each in its place by length: chains are short here)
      const uint32_t c = chain_of_[i];
      uint32_t to = at[c]++;
      for (; to > first_[c] && items_[of_chain_[to - 1]].tiles < items_[i].tiles; --to) of_chain_[to] = of_chain_[to - 1];
      of_chain_[to] = (uint32_t)i;
    }
    by_load_.resize(load_.size());
    for (size_t c = 0; c < load_.size(); ++c) by_load_[c] = (uint32_t)c;
    for (size_t x = 0; x < load_.size(); x += per_xcd_)
      std::sort(by_load_.begin() + (long)x, by_load_.begin() + (long)(x + per_xcd_),
                [&](uint32_t a, uint32_t b) { return load_[a] != load_[b] ? load_[a] < load_[b] : a < b; });
    // About the least cap that they fit into: mostly near the mean with what the parts themselves cost; else halfway between what does
    // not fit and what does.
    long near = lo;
    for (size_t x = 0; x < load_.size(); x += per_xcd_) {
      long sum = 0;
      for (size_t c = x; c < x + per_xcd_; ++c) {
        const long over = load_[c] - lo, part = lo - ITEM_COST_TILES - PART_COST_TILES;
        sum += load_[c] + (over > 0 ? PART_COST_TILES + (over + part - 1) / part * (ITEM_COST_TILES + PART_COST_TILES) : 0);
      }
      near = std::max(near, sum / (long)per_xcd_);
    }
    near = std::min(hi, near + near / 32 + 1);
    if (!fits(near, pieces)) {
      if (near == hi || !fits(hi, pieces)) return false;
      std::vector<PrefillPiece> fewer;
      for (lo = near; hi - lo > hi / 16;) {
        const long mid = (lo + hi) / 2;
        if (fits(mid, fewer)) {
          hi = mid;
          pieces.swap(fewer);
        } else {
          lo = mid;
        }
        if (hi - lo == 1) break;
      }
    }
    std::sort(pieces.begin(), pieces.end(), [](const PrefillPiece& a, const PrefillPiece& b) { return a.item != b.item ? a.item < b.item : a.kt0 < b.kt0; });
    return true;
  }
  long looked_at() const { return looked_at_; }   // items, parts and chains, over the whole search

 private:
  const std::vector<PrefillItem>& items_;
  const std::vector<uint32_t>& chain_of_;
  const std::vector<long>& load_;
  const size_t per_xcd_;
  const int block_m_;
  const bool persistent_;
  std::vector<uint32_t> first_, of_chain_;        // every chain's items, the longest first
  std::vector<uint32_t> by_load_;                 // every XCD's chains, the least loaded first
  struct Room { long room; uint32_t chain; };
  std::vector<Room> rooms_;                       // of one XCD, the widest first
  struct Rest { int32_t tiles; uint32_t item; };  // the last `tiles` of an item, which its chain gives away
  std::vector<Rest> rest_;
  size_t doubtful_ = 0;                           // the XCD that did not fit the last time is asked first
  long looked_at_ = 0;

  bool fits(long cap, std::vector<PrefillPiece>& pieces) {
    pieces.clear();
    const size_t xcds = load_.size() / per_xcd_, start = doubtful_;
    for (size_t i = 0; i < xcds; ++i) {
      const size_t x = (start + i) % xcds;
      if (!fits_xcd(x * per_xcd_, cap, pieces)) {
        doubtful_ = x;
        return false;
      }
    }
    return true;
  }
  int32_t last_cut(uint32_t i) const { return (items_[i].q_off + items_[i].q_tile * block_m_) / 64; }   // the tile of the item's first row
  bool fits_xcd(size_t c0, long cap, std::vector<PrefillPiece>& pieces) {
    rooms_.clear();
    rest_.clear();
    ++looked_at_;
    if (load_[by_load_[c0 + per_xcd_ - 1]] <= cap) return true;
    looked_at_ += (long)per_xcd_;
    size_t n_within = per_xcd_;
    while (n_within > 0 && load_[by_load_[c0 + n_within - 1]] > cap) --n_within;
    for (size_t i = 0; i < n_within; ++i) rooms_.push_back(Room{cap - load_[by_load_[c0 + i]], by_load_[c0 + i]});
    for (size_t i = per_xcd_; i > n_within; --i) {  // the most loaded first: what they give away is about in order then
      const uint32_t c = by_load_[c0 + i - 1];
      long room = cap - load_[c];
      for (uint32_t n = first_[c]; room < 0; ++n) {
        const uint32_t item = of_chain_[n];
        ++looked_at_;
        room += items_[item].weight();
        int32_t keep = (int32_t)std::min<long>(room - ITEM_COST_TILES - PART_COST_TILES, items_[item].tiles - LEAST_PART_TILES);
        keep = std::min(keep, last_cut(item));
        if (keep < LEAST_PART_TILES) keep = 0;    // all of it goes
        if (keep) {
          pieces.push_back(PrefillPiece{item, 0, keep, c});
          room -= keep + ITEM_COST_TILES + PART_COST_TILES;
        }
        const Rest r{items_[item].tiles - keep, item};
        rest_.push_back(r);
        size_t to = rest_.size() - 1;
        for (; to > 0 && rest_[to - 1].tiles < r.tiles; --to) rest_[to] = rest_[to - 1];
        rest_[to] = r;
      }
      const Room r{room, c};
      rooms_.push_back(r);
      size_t to = rooms_.size() - 1;
      for (; to > 0 && rooms_[to - 1].room < room; --to) rooms_[to] = rooms_[to - 1];
      rooms_[to] = r;
    }
    for (const Rest& r : rest_) {
      const int32_t tiles = items_[r.item].tiles;
      for (int32_t kt0 = tiles - r.tiles; kt0 < tiles;) {
        ++looked_at_;
        long need = tiles - kt0 + ITEM_COST_TILES + (kt0 > 0 ? PART_COST_TILES : 0);
        int32_t kt1 = tiles;
        // the narrowest that takes all of it, else a part into the widest
        auto at = std::partition_point(rooms_.begin(), rooms_.end(), [&](const Room& a) { return a.room >= need; });
        if (at != rooms_.begin()) {
          --at;
        } else {
          const long rest = tiles - kt0, most = std::max<long>(1, at->room - ITEM_COST_TILES - PART_COST_TILES), n = (rest + most - 1) / most;
          const long even = (rest + n - 1) / n;   // n parts of a length, where there are n chains for them
          long take = std::min(most, rest - LEAST_PART_TILES);
          if ((size_t)n <= rooms_.size() && rooms_[(size_t)n - 1].room >= even + ITEM_COST_TILES + PART_COST_TILES) take = even;
          take = std::min({take, rest - LEAST_PART_TILES, (long)last_cut(r.item) - kt0});
          if (take < LEAST_PART_TILES) return false;
          kt1 = kt0 + (int32_t)take;
          need = take + ITEM_COST_TILES + PART_COST_TILES;
        }
        pieces.push_back(PrefillPiece{r.item, kt0, kt1, at->chain});
        kt0 = kt1;
        const Room left{at->room - need, at->chain};
        for (; at + 1 != rooms_.end() && at[1].room > left.room; ++at) *at = at[1];
        *at = left;
      }
    }
    return true;
  }
};

// When the last of an XCD's workgroups ends, of these weights in the order in which they are launched, one per compute unit.  The XCD deals
// them to its four shader arrays in turn, each as soon as its array has a compute unit free, and not before the one ahead of it has begun.
inline long dealt_end(const std::vector<int32_t>& weights, int per_xcd) {
  const size_t arrays = per_xcd % 4 == 0 ? 4 : 1, cus = (size_t)per_xcd / arrays;
  std::vector<long> free(arrays * cus, 0);        // when every compute unit is free, array after array
  long begun = 0, end = 0;
  for (size_t i = 0; i < weights.size(); ++i) {
    const auto array = free.begin() + (long)(i % arrays * cus), cu = std::min_element(array, array + (long)cus);
    begun = std::max(begun, *cu);
    *cu = begun + weights[i];
    end = std::max(end, *cu);
  }
  return end;
}

// The work list and the merge list of items some of which are shared out.  `persistent`: workgroup c xcds + x takes chain c of XCD x, each in
// the order of its items.  Without, the chains only say where to cut, and every
// item and part is a workgroup of its own, each XCD's longest first: where the phases' masks overlap, the other phase's
// workgroups then get a compute unit whenever a part ends, not with the kernel.  Of every four, one per shader array, the shortest goes
// first, so that the array whose turn it is when all compute units have one is the one that comes free.  (Longest first throughout
// leaves the next one waiting behind the longest: 300 tokens behind 4000, 5 items a head on 8 compute units, cut into 46 + 21 tiles: the
// last parts began when the first ones ended, 97.5 us, whole 88.9.)  `whole_end`: when the whole items would end; false, and nothing
// written, if no item is cut or the parts do not end early enough after all.  (The four pieces above on 256 CUs, both phases there: as
// chains 136 us, as workgroups 137, in the order of the chains 147.  A decode step of 16 requests of 1000 tokens that comes in the
// middle of it ends 111 us later beside chains, 105 beside workgroups, and 79 beside whole items, which leave it compute units of
// their own; pairs of both steps, queued, 148, 146 and 159 us.)
inline bool write_shares(const std::vector<PrefillItem>& items, const std::vector<uint32_t>& chain_of, const std::vector<PrefillPiece>& pieces, size_t xcds,
                         size_t per_xcd, bool persistent, long whole_end, std::vector<PrefillWork>& work, std::vector<PrefillRange>& range, std::vector<int32_t>& chain,
                         std::vector<PrefillMerge>& merge) {
  // what goes where, in the order of the items: a piece (its number), or the whole item
  struct Entry { uint32_t item, chain; int32_t tiles, piece; };
  std::vector<Entry> all;
  all.reserve(items.size() + pieces.size());
  std::vector<int32_t> part(pieces.size(), -1);   // numbers of the pieces that are not whole
  int32_t n_parts = 0;
  for (size_t i = 0, p = 0; i < items.size(); ++i) {
    if (p == pieces.size() || pieces[p].item != i) {
      all.push_back(Entry{(uint32_t)i, chain_of[i], items[i].tiles, -1});
      continue;
    }
    const bool cut = pieces[p].kt1 < items[i].tiles;
    if (cut) merge.push_back(PrefillMerge{items[i].row0, items[i].len, items[i].q_tile, items[i].head0, n_parts, 0});
    for (; p < pieces.size() && pieces[p].item == i; ++p) {
      all.push_back(Entry{(uint32_t)i, pieces[p].chain, pieces[p].kt1 - pieces[p].kt0, (int32_t)p});
      if (!cut) continue;
      part[p] = n_parts++;
      ++merge.back().n_parts;
    }
  }
  if (n_parts == 0) return false;
  const size_t n = all.size();
  auto write = [&](size_t to, const Entry& e) {
    work[to] = items[e.item].work();
    range[to] = e.piece < 0 ? PrefillRange{0, e.tiles, -1} : PrefillRange{pieces[(size_t)e.piece].kt0, pieces[(size_t)e.piece].kt1, part[(size_t)e.piece]};
  };
  auto weight = [&](const Entry& e) -> int32_t { return e.tiles + (int32_t)(ITEM_COST_TILES + (e.piece >= 0 && part[(size_t)e.piece] >= 0 ? PART_COST_TILES : 0)); };
  const long latest = shared_end(whole_end, n, persistent);
  long end = 0;
  if (persistent) {
    std::vector<long> load(xcds * per_xcd, 0);
    for (const Entry& e : all) end = std::max(end, load[e.chain] += weight(e));
    if (end > latest) {
      merge.clear();
      return false;
    }
    work.resize(n);
    range.resize(n);
    auto slot = [&](uint32_t c) -> size_t { return c % (uint32_t)per_xcd * (uint32_t)xcds + c / (uint32_t)per_xcd; };
    chain.assign(xcds * per_xcd + 1, 0);
    for (const Entry& e : all) ++chain[slot(e.chain) + 1];
    for (size_t c = 0; c + 1 < chain.size(); ++c) chain[c + 1] += chain[c];
    std::vector<int32_t> at(chain.begin(), chain.end() - 1);
    for (const Entry& e : all) write((size_t)at[slot(e.chain)]++, e);
    return true;
  }
  std::vector<uint64_t> order(n);                 // XCD, longest first (an item has fewer than 2^26 tiles of 64 keys), place
  std::vector<size_t> first(xcds + 1, 0);
  for (size_t i = 0; i < n; ++i) {
    const uint64_t x = all[i].chain / (uint32_t)per_xcd;
    order[i] = x << 58 | (uint64_t)((1 << 26) - all[i].tiles) << 32 | i;
    ++first[x + 1];
  }
  std::sort(order.begin(), order.end());
  size_t most = 0, at = 0;
  std::vector<int32_t> weights;
  for (size_t x = 0; x < xcds; ++x) {
    most = std::max(most, first[x + 1]);
    first[x + 1] += first[x];
    weights.clear();
    for (size_t i = first[x]; i < first[x + 1]; ++i) {
      if (i % 4 == first[x] % 4 && i + 4 <= first[x + 1]) std::reverse(order.begin() + (long)i, order.begin() + (long)i + 4);
      weights.push_back(weight(all[(uint32_t)order[i]]));
    }
    end = std::max(end, dealt_end(weights, (int)per_xcd));
  }
  if (end > latest) {
    merge.clear();
    return false;
  }
  work.resize(n);
  range.resize(n);
  chain.clear();
  chain.reserve(most * xcds + 1);
  for (size_t i = 0; i < most; ++i)
    for (size_t x = 0; x < xcds; ++x) {           // workgroup i * xcds + x runs on XCD x
      chain.push_back((int32_t)at);
      if (first[x] + i < first[x + 1]) write(at++, all[(uint32_t)order[first[x] + i]]);
    }
  chain.push_back((int32_t)at);
  return true;
}

// What a step's items that were shared out need besides `work` and `chain`; both empty where all items are whole.
struct PrefillParts {
  std::vector<PrefillRange> range;                // one per item of `work`
  std::vector<PrefillMerge> merge;
};

// `persistent`: a chain per compute unit; `parts` null: no item is shared out.
// (Lists in a few flat arrays: with a vector per unit, per XCD and per chain this took 13 of the 20 us of a step of 8 short prompts.)
inline void build_prefill_chains(const int32_t* cu_seqlens, const int32_t* prefix_lens, const int32_t* kv_cu, int n_req,
                                 int H, int Hkv, int xcds, int share, bool persistent, std::vector<PrefillWork>& work,
                                 std::vector<int32_t>& chain, PrefillParts* parts, long* looked_at = nullptr) {
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
    const int32_t q_off = prefix_lens ? prefix_lens[r] : 0, kv_row0 = kv_cu ? kv_cu[r] : row0;
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
  if (parts) {
    parts->range.clear();
    parts->merge.clear();
  }
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
  // At most the heaviest item's weight is to be gained, and with many items per compute unit whole ones balance well enough: of random
  // batches with more than three per compute unit one in twelve can be a sixth shorter, and all of them would pay for the search.
  bool may_share = parts && even && n_items <= 3 * (size_t)share && heaviest > 2 * LEAST_PART_TILES;
  if (may_share && !persistent) {
    // Before the items are dealt only for the search: one begins no later than when those ahead of it fill all compute units, and those
    // that have to be cut cost more.  (Near the border the search finds nothing, mostly: one prompt of 2500 tokens on 256 CUs.)
    long end = 0;
    for (int x = 0; x < xcds; ++x) {
      long ahead = 0;
      for (uint32_t i = xq_first[(size_t)x]; i < xq_first[(size_t)x + 1]; ++i) {
        const long w = items[xq[i]].weight();
        end = std::max(end, (i - xq_first[(size_t)x] < (uint32_t)per_xcd ? 0 : ahead / per_xcd) + w);
        ahead += w;
      }
    }
    const long cap = shared_end(end, items, false);
    for (int x = 0; x < xcds; ++x) {
      long sum = 0;
      for (uint32_t i = xq_first[(size_t)x]; i < xq_first[(size_t)x + 1]; ++i) {
        const long w = items[xq[i]].weight();
        sum += w + (w > cap ? ITEM_COST_TILES + 2 * PART_COST_TILES : 0);
      }
      may_share = may_share && sum * 16 <= cap * per_xcd * 15;
    }
  }
  std::vector<uint32_t> chain_of(n_items);        // chain c of XCD x: x * per_xcd + c
  std::vector<long> load((size_t)xcds * (size_t)per_xcd, 0);
  // Unit after unit (in the order the XCD took them), each unit's items longest-first onto the chain
  // with the least load so far: every chain then holds about the same weight of EVERY unit, so the
  // chains of an XCD pass from one unit to the next at about the same time and the XCD's L2 has to
  // hold one or two units' K, V, not all of them.  (Dealt over all units at once the chains were as
  // well balanced in total, but drifted apart unit by unit, and K, V crossed HBM four times.)
  // Workgroups of one item each land on the compute units in the same way.
  if (persistent || may_share)
    for (int x = 0; x < xcds; ++x) {
      const auto of_xcd = load.begin() + (long)x * per_xcd;
      for (uint32_t i = xq_first[(size_t)x]; i < xq_first[(size_t)x + 1]; ++i) {
        const auto least = std::min_element(of_xcd, of_xcd + per_xcd);
        *least += items[xq[i]].weight();
        chain_of[xq[i]] = (uint32_t)(least - load.begin());
      }
    }
  if (may_share) {
    PrefillShares shares(items, chain_of, load, per_xcd, bm, persistent);
    std::vector<PrefillPiece> pieces;
    const bool found = shares.find(pieces);
    if (looked_at) *looked_at = shares.looked_at();
    long end = persistent ? *std::max_element(load.begin(), load.end()) : 0;
    if (found && !persistent) {
      std::vector<int32_t> weights;
      for (int x = 0; x < xcds; ++x) {
        weights.clear();
        for (uint32_t i = xq_first[(size_t)x]; i < xq_first[(size_t)x + 1]; ++i) weights.push_back(items[xq[i]].weight());
        end = std::max(end, dealt_end(weights, per_xcd));
      }
    }
    if (found && write_shares(items, chain_of, pieces, (size_t)xcds, (size_t)per_xcd, persistent, end, work, parts->range, chain, parts->merge)) return;
  }
  if (!persistent) {
    uint32_t most = 0;
    for (int x = 0; x < xcds; ++x) most = std::max(most, xq_first[(size_t)x + 1] - xq_first[(size_t)x]);
    work.clear();
    work.reserve(n_items);
    chain.clear();
    chain.reserve((size_t)most * (size_t)xcds + 1);
    for (uint32_t i = 0; i < most; ++i)
      for (int x = 0; x < xcds; ++x) {            // workgroup i * xcds + x runs on XCD x
        chain.push_back((int32_t)work.size());
        if (xq_first[(size_t)x] + i < xq_first[(size_t)x + 1]) work.push_back(items[xq[xq_first[(size_t)x] + i]].work());
      }
    chain.push_back((int32_t)work.size());
    return;
  }
  // every chain in the order of the units
  auto slot = [&](uint32_t c) -> size_t { return (size_t)(c % (uint32_t)per_xcd) * (size_t)xcds + c / (uint32_t)per_xcd; };   // workgroup id = chain slot * xcds + xcd
  chain.assign((size_t)share + 1, 0);
  for (uint32_t c : chain_of) ++chain[slot(c) + 1];
  for (int c = 0; c < share; ++c) chain[(size_t)c + 1] += chain[(size_t)c];
  std::vector<int32_t> at(chain.begin(), chain.end() - 1);
  work.resize(n_items);
  for (size_t i = 0; i < n_items; ++i) work[(size_t)at[slot(chain_of[i])]++] = items[i].work();
}

// A step with cached tokens: are its keys and values as dense rows, brought together ahead of the attention kernel, the faster way, or
// the pages?  Out of the pages the kernel takes up to 4 % longer (operands of V come in smaller reads) and 1 to 2 us longer to begin (the list of
// units is one more round trip); dense rows cost a pass over the cached ones and, in the page write's launch, a second store of the new ones.
// So the pairs of query and key per cached row decide, and the pass is free where it is short, or runs beside the rotation of the step's
// queries (`rotates`: 64 query heads, 12 pieces of 128 behind 100 on 256 CUs 45 / 41 us, 4 of 256 on 64 69 / 66).  Whole step, pages / dense rows, 8 KV heads of 128 dims on 128
// CUs: 32 query heads, 4 pieces of 2048 behind 100 tokens 289 / 277 us, 1 of 4096 behind 1500 335 / 325, 4 of 1024 behind 6000 569 / 594, 4 of
// 256 behind 1500 55 / 65, 1 of 128 behind one 19.3 / 17.7; 64 query heads, 1 of 1024 behind 6000 290 / 286, 4 of 256 behind 6000 278 / 307.  With a query
// head per KV head the pages cost the kernel 1 % at most: 16 heads, 1 of 4096 behind 1500 180 / 183.  One KV head has a launch of its own for
// the rows, the new ones among them: 32 query heads, 1 of 4096 behind 100 203 / 199, 4 of 700 behind 400 72 / 74.  Over 1207 steps (32 to 16000 cached tokens, 1
// to 12 pieces of 40 to 4096, eleven layers, 64 to 256 CUs) 0.2 % over the faster one of the two on average, always pages 1.5 %, always rows 10 %.
inline bool dense_rows_pay(const int32_t* cu_seqlens, const int32_t* prefix_lens, int n_req, int H, int Hkv, int dim, int share, bool rotates) {
  double pairs = 0, cached = 0;                   // of query and key, over all heads; rows of all KV heads
  for (int r = 0; r < n_req; ++r) {
    const double len = cu_seqlens[r + 1] - cu_seqlens[r];
    pairs += len * (prefix_lens[r] + len / 2) * H;
    cached += (double)prefix_lens[r] * Hkv;
  }
  if (Hkv == 1) return pairs * dim > 1.2e6 * 128 * share;
  if (rotates) pairs += 400. * cu_seqlens[n_req] * H;
  return pairs * dim + 1e5 * 128 * share > (H > Hkv ? 8e3 : 3e4) * cached * dim;
}

// 192 / 128 dims: is prefill_192_kernel the faster one for the step?  It gains about three times per tile ahead of an item's diagonal what it
// loses per item, and nothing where only one group of waves has rows (up to 128), so the sum over the step's items decides.  (Not the share:
// a batch has the same bits on all of them.)  One prompt of 400 .. 4000 tokens of 16 heads with 8 .. 60 of 1 .. 300, equal prompts of 1 .. 1024 and
// random ones of up to 200 .. 1500, on 64, 128 and 256 CUs (549 steps, kernel alone): 0.16, 0.26 and 0.33 % over the better one of the two on average,
// at most 7 % over prefill_kernel (24 -> 26 us); with "longest prompt over six tiles" as the rule 0.71, 0.77 and 0.26 %.  prefill_kernel /
// prefill_192_kernel on 64 CUs: a prompt of 400 tokens and 60 of 64 tokens 91 / 96 us, of 1000 and 24 of 64 70 / 67, of 4000 and 8 of 64 333 / 263;
// 32 of 384 tokens 217 / 220, of 448 303 / 279.
inline bool two_groups_pay(const int32_t* cu_seqlens, int n_req) {
  int64_t gain = 0;
  for (int r = 0; r < n_req; ++r) {
    const int64_t len = cu_seqlens[r + 1] - cu_seqlens[r], items = (len + 255) / 256, full = len - 256 * (items - 1) > 128 ? items : items - 1;
    gain += 6 * full * (full - 1) - items;        // 3 x (0 + 4 + 8 ..) tiles ahead of the full items' diagonals
  }
  return gain > 0;
}

}  // namespace spd
