// Prints how a decode batch is split over workgroups (csrc/decode_split.h), one batch per input line:
//   latent|gqa page_tokens cus n_kv_heads override_units B length...
// Answer: "n_wgs max_chunks chunk_units n_items", then a line "req chunk unit0 n_units next" per item.
// First line of all: the page ids that a latent record's copy in LDS holds, the words of the record's header.
#include <iostream>
#include <sstream>
#include <string>

#include "decode_split.h"

int main() {
  using namespace spd;
  std::printf("%d %d\n", MLA_CHUNK_PAGES, DECODE_ITEM_WORDS);
  std::string line, kind;
  while (std::getline(std::cin, line)) {
    std::istringstream in(line);
    int P, cus, Hkv, override_units, B;
    in >> kind >> P >> cus >> Hkv >> override_units >> B;
    std::vector<int32_t> lens((size_t)B), n_chunks((size_t)B);
    int64_t sum = 0;
    int most = 0;
    for (int32_t& n : lens) {
      in >> n;
      const int units = (n + TILE_T - 1) / TILE_T;
      sum += units;
      most = std::max(most, units);
    }
    spd_phase_state ps;
    DecodeSplit sp;
    if (kind == "latent") split_latent(ps, lens.data(), B, sum, cus, P / TILE_T, override_units, n_chunks.data(), sp);
    else split_gqa(ps, lens.data(), B, sum, most, Hkv, cus, override_units, n_chunks.data(), sp);
    std::printf("%d %d %d %zu\n", sp.n_wgs, sp.max_chunks, sp.chunk_units, ps.tmp_items.size());
    for (const DecodeItem& it : ps.tmp_items) std::printf("%d %d %d %d %d\n", it.req, it.chunk, it.unit0, it.n_units, it.next);
  }
}
