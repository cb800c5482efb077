// Prints how a decode batch is split over workgroups (csrc/decode_split.h), one batch per input line:
//   latent|noalloc|latent_fp8|noalloc_fp8|gqa page_tokens cus n_kv_heads n_q_heads append override_units B length...
// (noalloc: the latent split of the entry point that allocates nothing; fp8: with what a chunk costs there, as steps.cpp passes it.)
// Answer: "n_wgs max_chunks chunk_units n_items", the bytes of its records, of its metadata as the limit counts it and of its
// partials, then a line "req chunk unit0 n_units next" per item.
// First line of all: the page ids that a latent record's copy in LDS holds, the words of the record's header, the bytes
// of a staging slot, and what a latent chunk costs beside its tiles, in tiles, over bf16 and over FP8 pages.
#include <iostream>
#include <sstream>
#include <string>

#include "decode_split.h"

int main() {
  using namespace spd;
  std::printf("%d %d %zu %d %d\n", MLA_CHUNK_PAGES, DECODE_ITEM_WORDS, NOALLOC_RING_BYTES, (int)CHUNK_COST, (int)CHUNK_COST_FP8);
  std::string line, kind;
  while (std::getline(std::cin, line)) {
    std::istringstream in(line);
    int P, cus, Hkv, H, append, override_units, B;
    in >> kind >> P >> cus >> Hkv >> H >> append >> override_units >> B;
    std::vector<int32_t> lens((size_t)B), n_chunks((size_t)B);
    int64_t sum = 0;
    int most = 0, pages = 0;
    for (int32_t& n : lens) {
      in >> n;
      const int units = (n + TILE_T - 1) / TILE_T;
      sum += units;
      most = std::max(most, units);
      pages = std::max(pages, (n + P - 1) / P);
    }
    spd_phase_state ps;
    DecodeSplit sp;
    const int dv = kind == "gqa" ? 128 : 512, upp = P / TILE_T;
    const int64_t cost = kind == "latent_fp8" || kind == "noalloc_fp8" ? CHUNK_COST_FP8 : CHUNK_COST;
    if (kind == "latent" || kind == "latent_fp8") split_latent(ps, lens.data(), B, sum, cus, upp, override_units, 0, n_chunks.data(), sp, cost);
    else if (kind == "noalloc" || kind == "noalloc_fp8")
      split_latent_within_limits(ps, lens.data(), B, H, dv, sum, pages, cus, upp, override_units, append != 0, 0, n_chunks.data(), sp, cost);
    else split_gqa(ps, lens.data(), B, sum, most, Hkv, cus, override_units, n_chunks.data(), sp);
    const int n_items = (int)ps.tmp_items.size();
    std::printf("%d %d %d %d %zu %zu %zu\n", sp.n_wgs, sp.max_chunks, sp.chunk_units, n_items, decode_records(sp, n_items, B, pages, upp).bytes,
                noalloc_metadata(n_items, B, pages, append != 0, 0), partial_o_bytes(B, H, sp.max_chunks, dv) + partial_ml_bytes(B, H, sp.max_chunks));
    for (const DecodeItem& it : ps.tmp_items) std::printf("%d %d %d %d %d\n", it.req, it.chunk, it.unit0, it.n_units, it.next);
  }
}
