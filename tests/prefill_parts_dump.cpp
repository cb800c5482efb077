// Prints how a prefill batch is dealt to chains (csrc/prefill_work.h), one batch per input line:
//   share persistent whole_items n_q_heads n_kv_heads n_req (len prefix)...
// Answer: "n_chains n_work n_merge looked_at two_groups" (what the search for the cuts looked at; which kernel 192 / 128 dims take), the chains' bounds, a line "row0 len q_tile head0 kv_row0 q_off kt0 kt1 part" per item and a line
// "row0 len q_tile head0 part0 n_parts" per merged one.
// Called as "rows": whether a chunked step has its keys as dense rows (dense_rows_pay), 0 or 1 per line "share H Hkv dim rope n (len prefix)..".
// Called as "uncut": what comes of sharing out two whole items (write_shares), as chains and as workgroups: "shared_out n_work n_ranges n_merge" each.
#include <iostream>
#include <sstream>
#include <string>

#include "prefill_work.h"

namespace spd {
// (as the kernels' file has them: eight waves, HB query heads of a KV head each)
int prefill_heads_per_block(int group) {
  for (int hb = 8; hb > 1; hb >>= 1)
    if (group % hb == 0) return hb;
  return 1;
}
int prefill_block_m(int group) { return 32 * (8 / prefill_heads_per_block(group)); }
}  // namespace spd

int main(int argc, char** argv) {
  using namespace spd;
  if (argc > 1 && std::string(argv[1]) == "rows") {
    int share, H, Hkv, dim, rope, n;
    while (std::cin >> share >> H >> Hkv >> dim >> rope >> n) {
      std::vector<int32_t> cu(1, 0), pre((size_t)n);
      for (int i = 0, len; i < n; ++i) {
        std::cin >> len >> pre[(size_t)i];
        cu.push_back(cu.back() + len);
      }
      std::printf("%d\n", (int)dense_rows_pay(cu.data(), pre.data(), n, H, Hkv, dim, share, rope != 0));
    }
    return 0;
  }
  if (argc > 1) {
    const std::vector<PrefillItem> items(2, PrefillItem{0, 128, 0, 0, 0, 0, 2, 0});
    for (bool persistent : {false, true}) {
      std::vector<PrefillWork> work;
      std::vector<int32_t> chain;
      PrefillParts parts;
      const bool shared = write_shares(items, {0, 0}, {PrefillPiece{0, 0, 2, 1}}, 1, 2, persistent, 1000, work, parts.range, chain, parts.merge);
      std::printf("%d %zu %zu %zu\n", (int)shared, work.size(), parts.range.size(), parts.merge.size());
    }
    return 0;
  }
  std::string line;
  while (std::getline(std::cin, line)) {
    std::istringstream in(line);
    int share, persistent, whole, H, Hkv, n;
    in >> share >> persistent >> whole >> H >> Hkv >> n;
    std::vector<int32_t> cu(1, 0), pre, kv(1, 0);
    for (int i = 0; i < n; ++i) {
      int len, p;
      in >> len >> p;
      cu.push_back(cu.back() + len);
      pre.push_back(p);
      kv.push_back(kv.back() + len + p);
    }
    std::vector<PrefillWork> work;
    std::vector<int32_t> chain;
    PrefillParts parts;
    const std::vector<PrefillMerge>& merge = parts.merge;
    long looked_at = 0;
    build_prefill_chains(cu.data(), pre.data(), kv.data(), n, H, Hkv, 8, share, persistent != 0, work, chain, whole ? nullptr : &parts, &looked_at);
    std::printf("%zu %zu %zu %ld %d\n", chain.size() - 1, work.size(), merge.size(), looked_at, (int)two_groups_pay(cu.data(), n));
    for (int32_t c : chain) std::printf("%d ", c);
    std::printf("\n");
    const int bm = prefill_block_m(H / Hkv);
    for (size_t i = 0; i < work.size(); ++i) {
      const PrefillWork& w = work[i];
      const int end = w.q_off + std::min(w.len, (w.q_tile + 1) * bm);   // behind the last key that a whole item visits
      const PrefillRange r = parts.range.empty() ? PrefillRange{0, (end + 63) / 64, -1} : parts.range[i];
      std::printf("%d %d %d %d %d %d %d %d %d\n", w.row0, w.len, w.q_tile, w.head0, w.kv_row0, w.q_off, r.kt0, r.kt1, r.part);
    }
    for (const PrefillMerge& m : merge) std::printf("%d %d %d %d %d %d\n", m.row0, m.len, m.q_tile, m.head0, m.part0, m.n_parts);
  }
}
