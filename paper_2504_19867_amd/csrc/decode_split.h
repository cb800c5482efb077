// How a decode step's contexts are split over workgroups: the work items of the GQA and of the latent kernel (host only).
#pragma once

#include <algorithm>
#include <functional>

#include "internal.h"

namespace spd {

// How the step's contexts are split over workgroups, in units of 16 tokens.
struct DecodeSplit {
  int n_wgs = 0, max_chunks = 1;
  int32_t chunk_units = 0;       // largest chunk
  int64_t dealt = 0;             // latent: units that a workgroup was dealt, its chunks' cost included
};

// The step's metadata as the kernels read it: a record per item (header and page ids; a chunk that starts inside a page
// touches one more than it holds), then the requests' chunk counts.
struct DecodeRecords {
  size_t stride = 0, off_chunks = 0, bytes = 0;
};
inline DecodeRecords decode_records(const DecodeSplit& sp, int n_items, int B, int max_pages, int units_per_page) {
  DecodeRecords d;
  const size_t chunk_pages = (size_t)std::min<int64_t>(max_pages, ((int64_t)sp.chunk_units + units_per_page - 2) / units_per_page + 1);
  d.stride = (sizeof(DecodeItem) + sizeof(int32_t) * chunk_pages + 63) & ~(size_t)63;
  d.off_chunks = d.stride * (size_t)n_items;
  d.bytes = (d.off_chunks + sizeof(int32_t) * (size_t)B + 15) & ~(size_t)15;
  return d;
}
// What the metadata limit of the entry point that allocates nothing counts: one block table row per request, the items, the
// appends, the RoPE frequencies.  Any batch within it fits a staging slot of NOALLOC_RING_BYTES in the form above.
inline size_t noalloc_metadata(int n_items, int B, int max_pages, bool append, size_t w_bytes) {
  return sizeof(int32_t) * (size_t)B * (1 + (size_t)max_pages) + 8 * (size_t)n_items + (append ? sizeof(TileDesc) * (size_t)B : 0) + w_bytes;
}
// Split-K partials: O of every (request, head, chunk), then its maximum and sum.
inline size_t partial_o_bytes(int B, int H, int max_chunks, int dv) {
  return max_chunks > 1 ? (sizeof(float) * (size_t)B * H * max_chunks * dv + 15) & ~(size_t)15 : 0;
}
inline size_t partial_ml_bytes(int B, int H, int max_chunks) {
  return max_chunks > 1 ? (sizeof(float) * (size_t)B * H * max_chunks * 2 + 15) & ~(size_t)15 : 0;
}

inline void push_chunk(std::vector<DecodeItem>& items, int r, int32_t chunk, int32_t n, int32_t u0, int32_t nu) {
  items.push_back(DecodeItem{r, chunk, 0, n, u0, nu, -1, 0});
}

// Chunks of c units, handed out longest first: the full chunks, request by request, then the requests' remainders by length.
inline void cut_chunks(spd_phase_state& ps, const int32_t* ctx_lens, int B, int max_units, int64_t c, int32_t* n_chunks, DecodeSplit& out) {
  out.chunk_units = (int32_t)c;
  out.max_chunks = (int)((max_units + c - 1) / c);
  std::vector<DecodeItem>& items = ps.tmp_items;
  std::vector<uint64_t>& rest = ps.tmp_set;                      // (units << 32 | request)
  items.clear();
  rest.clear();
  for (int r = 0; r < B; ++r) {
    const int32_t units = (ctx_lens[r] + TILE_T - 1) / TILE_T, full = units / (int32_t)c;
    n_chunks[r] = (int32_t)((units + c - 1) / c);
    for (int32_t ck = 0; ck < full; ++ck) push_chunk(items, r, ck, ctx_lens[r], ck * (int32_t)c, (int32_t)c);
    if (units % c) rest.push_back((uint64_t)(units % c) << 32 | (uint32_t)(B - 1 - r));   // equal lengths: request order
  }
  std::sort(rest.begin(), rest.end(), std::greater<uint64_t>());
  for (uint64_t k : rest) {
    const int r = B - 1 - (int)(uint32_t)k;
    push_chunk(items, r, n_chunks[r] - 1, ctx_lens[r], (n_chunks[r] - 1) * (int32_t)c, (int32_t)(k >> 32));
  }
  out.n_wgs = (int)items.size();
}

// GQA: about 6 workgroups per CU of the decode share: enough to balance unequal contexts, few enough to keep the split-K
// partials small.
inline void split_gqa(spd_phase_state& ps, const int32_t* ctx_lens, int B, int64_t sum_units, int max_units, int Hkv, int cus, int override_tiles,
                      int32_t* n_chunks, DecodeSplit& out) {
  const int64_t round = 8;                       // 4 waves x 2 tiles per step
  int64_t c;
  if (override_tiles > 0) {                      // tuning override
    c = (override_tiles + round - 1) / round * round;
  } else {
    const int64_t per_head_chunks = std::max<int64_t>(1, (int64_t)cus * 6 / std::max(1, Hkv));
    c = (sum_units + per_head_chunks - 1) / per_head_chunks;
    c = std::min<int64_t>(std::max<int64_t>((c + round - 1) / round * round, 16), 1 << 20);
  }
  cut_chunks(ps, ctx_lens, B, max_units, std::min<int64_t>(c, (max_units + round - 1) / round * round), n_chunks, out);
}

// What a latent chunk costs beside its tiles, in tiles.  FP8 tiles take less time and the cost is the same: 128 requests of
// 1024 .. 8192 tokens on 128 CUs 97.6 us with 20, 96.0 with 30 (bf16 148.8, 151.0; with 12 both are 2 to 3 us slower).
constexpr int64_t CHUNK_COST = 20, CHUNK_COST_FP8 = 30;
// Whole requests dealt to `slots` workgroups (B >= slots): true, with the batch so split, if none gets `worst` units or more and
// no request has more than `most`.
inline bool deal_whole(spd_phase_state& ps, const int32_t* ctx_lens, int B, int64_t slots, int64_t most, int64_t worst, int32_t* n_chunks, DecodeSplit& out, int64_t cost) {
  std::vector<uint64_t>&by_length = ps.tmp_set, &loads = ps.tmp_heap;     // (units << 32 | request, counted from the end), (load << 32 | workgroup)
  by_length.clear();
  for (int r = 0; r < B; ++r) {
    const uint64_t units = (uint64_t)(((int64_t)ctx_lens[r] + TILE_T - 1) / TILE_T);
    if ((int64_t)units > most || (int64_t)units + cost >= worst) return false;
    by_length.push_back(units << 32 | (uint32_t)(B - 1 - r));
  }
  std::sort(by_length.begin(), by_length.end(), std::greater<uint64_t>());
  loads.clear();
  for (int64_t w = 0; w < slots; ++w) loads.push_back((uint64_t)w);       // (in order: a heap already)
  std::vector<int32_t>& owner = ps.tmp_owner;
  owner.clear();
  for (uint64_t k : by_length) {
    std::pop_heap(loads.begin(), loads.end(), std::greater<uint64_t>());
    owner.push_back((int32_t)(uint32_t)loads.back());
    loads.back() += ((k >> 32) + cost) << 32;
    if ((int64_t)(loads.back() >> 32) >= worst) return false;
    std::push_heap(loads.begin(), loads.end(), std::greater<uint64_t>());
  }
  // the first `slots` items, one per workgroup in order, are where the workgroups start
  std::vector<DecodeItem>& items = ps.tmp_items;
  std::vector<int32_t>& last = ps.tmp_last;
  items.clear();
  last.assign((size_t)slots, -1);
  for (int i = 0; i < B; ++i) {
    const uint64_t k = by_length[(size_t)i];
    const int r = B - 1 - (int)(uint32_t)k, wg = owner[(size_t)i];
    push_chunk(items, r, 0, ctx_lens[r], 0, (int32_t)(k >> 32));
    if (last[(size_t)wg] >= 0) items[(size_t)last[(size_t)wg]].next = i;
    last[(size_t)wg] = i;
    n_chunks[r] = 1;
  }
  out.n_wgs = (int)slots;
  out.max_chunks = 1;
  out.chunk_units = (int32_t)(by_length[0] >> 32);
  return true;
}

// Latent decode: two workgroups per CU are resident, and the batch's units are dealt to them evenly, in request order, a
// workgroup going on from one request's end to the next one's beginning.  (Chunks of one length, handed out longest first, left
// a quarter of the slots idle at the end.)  A chunk costs its pipeline fill and its merge beside its tiles, about as
// much as `cost` tiles; chunks are whole rounds of the four waves, except at a request's end.  `least`: deal a workgroup no
// fewer units than this.
inline void split_latent(spd_phase_state& ps, const int32_t* ctx_lens, int B, int64_t sum_units, int cus, int units_per_page, int override_units,
                         int64_t least, int32_t* n_chunks, DecodeSplit& out, int64_t cost = CHUNK_COST) {
  constexpr int64_t ROUND = 4;
  const int64_t slots = std::max(1, 2 * cus), most = (int64_t)(MLA_CHUNK_PAGES - 1) * units_per_page / ROUND * ROUND;
  std::vector<DecodeItem>& items = ps.tmp_items;
  std::vector<int32_t>& owner = ps.tmp_sizes;                    // workgroup of each chunk
  // at least two tiles per wave
  int64_t quota = cost + std::max(least, override_units > 0 ? override_units : std::max<int64_t>(2 * ROUND, (sum_units + B * cost) / slots));
  for (;; quota += std::max<int64_t>(1, quota / 64)) {
    const int64_t sliver = std::min<int64_t>((quota - cost) / 4, 4);
    items.clear();
    owner.clear();
    int wg = 0;
    int64_t room = quota;
    out.chunk_units = 0;
    out.max_chunks = 1;
    for (int r = 0; r < B; ++r) {
      const int32_t units = (ctx_lens[r] + TILE_T - 1) / TILE_T;
      int32_t u0 = 0, chunk = 0;
      while (u0 < units) {
        const int64_t left = units - u0;
        if (room < quota && room - cost <= sliver && left > room - cost) { ++wg; room = quota; }   // too little room to start here
        int64_t take = std::min<int64_t>(left, std::max<int64_t>(ROUND, (room - cost) / ROUND * ROUND));
        if (left > take && left - take <= sliver) take = left;                  // too little left to start elsewhere
        take = std::min(take, most);
        push_chunk(items, r, chunk++, ctx_lens[r], u0, (int32_t)take);
        owner.push_back(wg);
        out.chunk_units = std::max(out.chunk_units, (int32_t)take);
        u0 += (int32_t)take;
        room -= cost + take;
        if (room < cost + ROUND) { ++wg; room = quota; }
      }
      n_chunks[r] = chunk;
      out.max_chunks = std::max(out.max_chunks, (int)chunk);
    }
    out.n_wgs = owner.back() + 1;
    if (out.n_wgs <= slots || override_units > 0) break;
  }
  out.dealt = quota;
  // With at least a request per workgroup, dealt whole instead, the longest first to whoever has least, where the most that a
  // workgroup then has is less: nothing is cut, and no workgroup stands idle.  (256 requests of 150 .. 450 tokens on 64 CUs: 100 -> 79
  // units at most; the step 74 -> 58 us.)
  if (B >= slots && least == 0 && override_units <= 0) {
    int64_t load = 0, worst = 0;
    for (size_t i = 0; i < items.size(); ++i) {
      if (i > 0 && owner[i] != owner[i - 1]) load = 0;
      load += cost + items[i].n_units;
      worst = std::max(worst, load);
    }
    if (deal_whole(ps, ctx_lens, B, slots, most, worst, n_chunks, out, cost)) return;
  }
  // workgroup i starts with record i: first chunks to the front, the others behind them, linked
  const int n = (int)items.size();
  std::vector<DecodeItem>& sorted = ps.tmp_items2;
  sorted.resize((size_t)n);
  int behind = out.n_wgs, prev = 0;
  for (int i = 0; i < n; ++i) {
    const bool first = i == 0 || owner[(size_t)i] != owner[(size_t)i - 1];
    const int at = first ? owner[(size_t)i] : behind++;
    sorted[(size_t)at] = items[(size_t)i];
    if (!first) sorted[(size_t)prev].next = at;
    prev = at;
  }
  items.swap(sorted);
}

// The same for the entry point that allocates nothing: where the even deal's records or partials would not fit, workgroups
// are dealt more, in fewer and longer chunks, until they do (or until there is nothing left to lengthen).
inline void split_latent_within_limits(spd_phase_state& ps, const int32_t* ctx_lens, int B, int H, int dv, int64_t sum_units, int max_pages, int cus,
                                       int units_per_page, int override_units, bool append, size_t w_bytes, int32_t* n_chunks, DecodeSplit& out,
                                       int64_t cost = CHUNK_COST) {
  for (int64_t least = 0;; least = out.dealt + out.dealt / 4) {
    split_latent(ps, ctx_lens, B, sum_units, cus, units_per_page, override_units, least, n_chunks, out, cost);
    if (noalloc_metadata((int)ps.tmp_items.size(), B, max_pages, append, w_bytes) <= NOALLOC_STAGE_BYTES &&
        partial_o_bytes(B, H, out.max_chunks, dv) + partial_ml_bytes(B, H, out.max_chunks) <= NOALLOC_WS_BYTES)
      return;
    if (out.dealt >= sum_units + B * cost) return;
  }
}

}  // namespace spd
