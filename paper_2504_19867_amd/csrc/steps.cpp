// Host side of the two steps and of the page write / gather: validation, atomic block
// reservation, block-table staging, launch geometry.  All arithmetic of the method runs in
// the kernels (kernels_*.hip).
#include "internal.h"
#include "decode_split.h"
#include "prefill_work.h"

#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <atomic>
#include <new>
#include <thread>
#include <cmath>

using namespace spd;

namespace spd {
int64_t blocks_missing_locked(spd_pool* pool, uint64_t req, int64_t n_tokens);
uint64_t reserve_locked(spd_pool* pool, uint64_t req, int64_t n_tokens);
uint64_t reserve_entry_locked(spd_pool* pool, spd_req_table& table, int64_t n_tokens);
}  // namespace spd

static inline size_t align16(size_t x) { return (x + 15) & ~(size_t)15; }
static inline size_t align4k(size_t x) { return (x + 4095) & ~(size_t)4095; }

// Tile descriptors covering logical positions [start, start + n) of a request whose block
// table is `bt`, written at `out`; dense row src_row0 maps to position `start`.  Returns how many.
static int build_tile_descs(const PoolGeom& g, const int32_t* bt, int32_t start, int32_t n, int32_t src_row0, TileDesc* out) {
  int32_t tile = start / TILE_T, t_begin = start % TILE_T, row = src_row0, left = n;
  int32_t page = tile / g.tiles_per_page, sub = tile % g.tiles_per_page;
  int count = 0;
  for (; left > 0; ++count) {
    const int32_t t_end = std::min<int32_t>(TILE_T, t_begin + left);
    out[count] = TileDesc{row, bt[page], sub, t_begin, t_end, {tile * TILE_T, 0, 0}};
    row += t_end - t_begin;
    left -= t_end - t_begin;
    t_begin = 0;
    ++tile;
    if (++sub == g.tiles_per_page) { sub = 0; ++page; }
  }
  return count;
}
static size_t tile_desc_count(int32_t start, int32_t n) { return ((size_t)(start % TILE_T) + (size_t)n + TILE_T - 1) / TILE_T; }

// Does a request id occur twice?  Small batches pair by pair, larger ones through an open-addressing table.
static bool has_duplicates(const uint64_t* ids, int n, std::vector<uint64_t>& set) {
  if (n <= 24) {
    for (int i = 1; i < n; ++i)
      for (int j = 0; j < i; ++j)
        if (ids[i] == ids[j]) return true;
    return false;
  }
  size_t cap = 64;
  while (cap < (size_t)n * 2) cap *= 2;
  set.assign(cap, 0);                       // holds index + 1
  for (int i = 0; i < n; ++i) {
    size_t h = (size_t)((ids[i] * 0x9e3779b97f4a7c15ull) >> 20) & (cap - 1);
    for (; set[h]; h = (h + 1) & (cap - 1))
      if (ids[set[h] - 1] == ids[i]) return true;
    set[h] = (uint64_t)i + 1;
  }
  return false;
}

// The kernels move 16 bytes per lane: every tensor a step is given must start on a 16-byte boundary.
static bool misaligned16(const void* a, const void* b = nullptr, const void* c = nullptr, const void* d = nullptr,
                         const void* e = nullptr) {
  return (((uintptr_t)a | (uintptr_t)b | (uintptr_t)c | (uintptr_t)d | (uintptr_t)e) & 15) != 0;
}

// The number the phase's step now being prepared will carry (its staging slot's commit assigns it).
static uint64_t next_step_number(spd_ctx* ctx, int phase) {
  return ctx->phase[phase].issue_seq.load(std::memory_order_relaxed) + 1;
}

static int kv_copy(spd_ctx* ctx, spd_pool* pool, int phase, uint64_t req_id, int32_t start_pos, int32_t n_tokens,
                   const void* k, const void* v, bool write) {
  if (!ctx || !pool || pool->ctx != ctx || phase < 0 || phase > 1 || start_pos < 0 || n_tokens <= 0 || !k)
    return SPD_EINVAL;
  const PoolGeom& g = pool->geom;
  if ((g.kind == SPD_KV_GQA) != (v != nullptr)) return SPD_EINVAL;
  if (misaligned16(k, v)) return SPD_EINVAL;
  if (ctx->device < 0) return SPD_ESTATE;
  // the request's table, if it holds the positions named (caller holds pool->mu)
  auto find_locked = [&](spd_req_table** out) -> int {
    auto it = pool->tables.find(req_id);
    if (it == pool->tables.end()) return SPD_ENOENT;
    const int64_t need = ((int64_t)start_pos + n_tokens + g.P - 1) / g.P;
    if ((int64_t)it->second.size() < need) return SPD_EINVAL;
    *out = &it->second;
    return SPD_OK;
  };
  // asked before anything is allocated for n_tokens, and again once there is a slot to write to (the wait for it is not under
  // the lock)
  spd_req_table* table = nullptr;
  spd_stage* st;
  int rc, n_descs;
  {
    std::lock_guard<std::mutex> lk(pool->mu);
    if ((rc = find_locked(&table)) != SPD_OK) return rc;
  }
  if ((rc = stage_acquire(ctx, phase, tile_desc_count(start_pos, n_tokens) * sizeof(TileDesc), &st)) != SPD_OK) return rc;
  {
    std::lock_guard<std::mutex> lk(pool->mu);
    if ((rc = find_locked(&table)) != SPD_OK) return rc;
    n_descs = build_tile_descs(g, table->data(), start_pos, n_tokens, 0, (TileDesc*)st->host);
    table->last_use[phase] = next_step_number(ctx, phase);
  }
  hipStream_t stream;
  if ((rc = phase_enter(ctx, phase, &stream)) != SPD_OK) return rc;
  StepScope step{ctx, phase, st, stream};
  const TileDesc* descs = (const TileDesc*)st->dev;              // read over PCIe, once per workgroup
  const StepMark mark = step_mark(ctx, phase, step.capturing);
  const bool fp8 = g.kind == SPD_KV_MLA_LATENT_FP8;
  KvRows rows;
  phase_exclusive(ctx, phase, &rows.cus);                         // (its share)
  if (write && fp8) SPD_HIP(launch_kv_write_fp8(g, pool->base, descs, n_descs, k, mark, stream));
  else if (write && kv_rows_supported(g)) SPD_HIP(launch_kv_rows(g, pool->base, descs, n_descs, k, v, rows, mark, stream));
  else if (write) SPD_HIP(launch_kv_write(g, pool->base, descs, n_descs, k, v, mark, stream));
  else if (fp8) SPD_HIP(launch_kv_gather_fp8(g, pool->base, descs, n_descs, (void*)k, mark, stream));
  else SPD_HIP(launch_kv_gather(g, pool->base, descs, n_descs, (void*)k, (void*)v, mark, stream));
  return step.commit();
}

extern "C" int spd_kv_write(spd_ctx* ctx, spd_pool* pool, int phase, uint64_t req_id, int32_t start_pos,
                            int32_t n_tokens, const void* k, const void* v) {
  return kv_copy(ctx, pool, phase, req_id, start_pos, n_tokens, k, v, true);
}

extern "C" int spd_kv_gather(spd_ctx* ctx, spd_pool* pool, int phase, uint64_t req_id, int32_t n_tokens,
                             void* k_out, void* v_out) {
  return kv_copy(ctx, pool, phase, req_id, 0, n_tokens, k_out, v_out, false);
}

// ------------------------------------------------------------------------------------------ prefill
constexpr int64_t Q_IN_ONE_LAUNCH = 32ll << 20;   // bytes of query rows that are rotated by the page write's launch
constexpr size_t MOST_DENSE_BYTES = 1ull << 30;   // of a chunked step's dense rows, a buffer that the context keeps

extern "C" int spd_prefill_step(spd_ctx* ctx, spd_pool* pool, const spd_prefill_batch* b) {
  if (!ctx || !pool || pool->ctx != ctx || !b || b->n_req <= 0 || !b->req_ids || !b->cu_seqlens) return SPD_EINVAL;
  if (!b->q || !b->k || !b->v || !b->out || b->n_q_heads <= 0 || b->n_kv_heads <= 0) return SPD_EINVAL;
  const PoolGeom& g = pool->geom;
  if (b->n_q_heads % b->n_kv_heads != 0 || b->cu_seqlens[0] != 0) return SPD_EINVAL;
  if (!(b->scale > 0.f) || !std::isfinite(b->scale)) return SPD_EINVAL;
  if (g.kind == SPD_KV_GQA) {
    if (b->latent || b->n_kv_heads != g.Hkv || b->dim_qk != g.dk || b->dim_v != g.dv) return SPD_EINVAL;
  } else {
    if (!b->latent || b->n_kv_heads != b->n_q_heads) return SPD_EINVAL;
  }
  if (!prefill_shape_supported(b->dim_qk, b->dim_v)) return SPD_EINVAL;
  if (misaligned16(b->q, b->k, b->v, b->out, b->latent)) return SPD_EINVAL;
  if (b->rope) {
    if (g.kind != SPD_KV_GQA) return SPD_EINVAL;
    int rrc = rope_config_check(b->rope);
    if (rrc != SPD_OK) return rrc;
    if (b->rope->rotary_dim % 16 || b->rope->rotary_offset % 8 || b->rope->rotary_offset + b->rope->rotary_dim > b->dim_qk)
      return SPD_EINVAL;
  }
  spd_phase_state& ps = ctx->phase[SPD_PHASE_PREFILL];
  for (int r = 0; r < b->n_req; ++r)
    if (b->cu_seqlens[r + 1] <= b->cu_seqlens[r]) return SPD_EINVAL;     // zero-length prompt
  if (has_duplicates(b->req_ids, b->n_req, ps.tmp_set)) return SPD_EINVAL;
  if (ctx->device < 0) return SPD_ESTATE;

  // chunked prefill: some request continues a prompt whose first prefix_lens[r] tokens are cached
  bool chunked = false;
  if (b->prefix_lens) {
    if (g.kind != SPD_KV_GQA) return SPD_EINVAL;
    for (int r = 0; r < b->n_req; ++r) {
      if (b->prefix_lens[r] < 0) return SPD_EINVAL;
      chunked = chunked || b->prefix_lens[r] > 0;
    }
  }
  int64_t n_keys = 0;
  if (chunked) {
    for (int r = 0; r < b->n_req; ++r) n_keys += (int64_t)b->prefix_lens[r] + (b->cu_seqlens[r + 1] - b->cu_seqlens[r]);
    if (n_keys > INT32_MAX) return SPD_EINVAL;
  }

  int rc;
  // One persistent workgroup per compute unit of the prefill share, each with its chain of work items, where phase_exclusive says
  // so; elsewhere one workgroup per item or part of one, handed out by the hardware as compute units free up.
  // The share is the one this step will run on: a staged partition is adopted below, once nothing but a HIP
  // call can fail any more, so a step that returns an error of its own leaves the partition as it was.
  int share;
  bool persistent = phase_exclusive(ctx, SPD_PHASE_PREFILL, &share);
  if (ctx->env_prefill_persistent >= 0) persistent = ctx->env_prefill_persistent != 0;   // experiment switch
  // Chunked: the attention kernel's keys and values as dense rows, brought together for it where that pays and there is memory for them
  // (K whole pages of 4 KiB: the kernel loads rows in 1 KiB pieces, which should not straddle cache lines) ...
  char *rows_k = nullptr, *rows_v = nullptr;
  const size_t k_bytes = align4k((size_t)n_keys * g.Hkv * g.dk * 2), v_bytes = (size_t)n_keys * g.Hkv * g.dv * 2;
  if (chunked && k_bytes + v_bytes <= MOST_DENSE_BYTES &&
      dense_rows_pay(b->cu_seqlens, b->prefix_lens, b->n_req, b->n_q_heads, b->n_kv_heads, g.dk, share, b->rope != nullptr)) {
    rows_k = rows_reserve(ctx, k_bytes + v_bytes);
    if (rows_k) rows_v = rows_k + k_bytes;
  }
  // ... else out of the pages.  kv_cu: where each request's begin, its first dense row or its first unit of 16 tokens in the list that the
  // kernel finds them with
  const bool paged = chunked && !rows_k;
  std::vector<int32_t> kv_cu;
  if (chunked) {
    kv_cu.resize((size_t)b->n_req + 1, 0);
    for (int r = 0; r < b->n_req; ++r) {
      const int32_t len = b->prefix_lens[r] + (b->cu_seqlens[r + 1] - b->cu_seqlens[r]);
      kv_cu[(size_t)r + 1] = kv_cu[(size_t)r] + (paged ? (len + TILE_T - 1) / TILE_T : len);
    }
  }
  std::vector<PrefillWork> work;
  std::vector<int32_t> chain;
  PrefillParts shared;
  const std::vector<PrefillMerge>& merge = shared.merge;
  float* parts = nullptr;
  auto deal = [&](PrefillParts* p) {
    build_prefill_chains(b->cu_seqlens, chunked ? b->prefix_lens : nullptr, chunked ? kv_cu.data() : nullptr, b->n_req,
                         b->n_q_heads, b->n_kv_heads, ctx->xcds, share, persistent, work, chain, p);
  };
  deal(b->dim_qk <= 128 ? &shared : nullptr);     // (the kernel for 192 dims takes whole items)
  if (!merge.empty()) {
    size_t n_parts = 0;
    for (const PrefillMerge& m : merge) n_parts += (size_t)m.n_parts;
    parts = parts_reserve(ctx, n_parts * prefill_part_floats(b->dim_v) * sizeof(float));
    if (!parts) {
      shared = PrefillParts();
      deal(nullptr);
    }
  }

  // page write, RoPE and dense rows in one launch, where that kernel takes the pool's shape (elsewhere the rows, the new ones included, are
  // gathered out of the pages by a launch of its own)
  const bool one_launch = kv_rows_supported(g);
  size_t n_descs = 0, n_gather = 0;
  for (int r = 0; r < b->n_req; ++r) {
    const int32_t len = b->cu_seqlens[r + 1] - b->cu_seqlens[r], pre = chunked ? b->prefix_lens[r] : 0;
    n_descs += tile_desc_count(pre, len);
    if (rows_k) n_gather += tile_desc_count(0, one_launch ? pre : pre + len);
  }
  size_t off_chain = align16(work.size() * sizeof(PrefillWork));
  size_t off_range = align16(off_chain + chain.size() * sizeof(int32_t));
  size_t off_merge = align16(off_range + shared.range.size() * sizeof(PrefillRange));
  size_t off_desc = align16(off_merge + merge.size() * sizeof(PrefillMerge));
  size_t off_units = align16(off_desc + n_descs * sizeof(TileDesc)), off_gather = off_units;
  // RoPE inside the step: every row's position where the queries have a launch of their own, and room for the frequency
  // table.  A launch of its own has eight waves per SIMD instead of the four that the page write leaves; short batches gain what
  // a launch and its gap cost.  Step with the queries in the same launch / in their own, 256-token prompts of 64 heads: 8 MiB of
  // queries 28 / 35 us on 128 CUs, 16 MiB 42 / 50, 32 MiB 65 / 70, 64 MiB 118 / 119, 128 MiB 239 / 230; on 96 CUs level at 64 MiB
  // too (147 / 144), 320 MiB 785 / 762.  On 256 CUs one launch stays 3 to 6 % ahead up to 320 MiB, which this line leaves.
  const int32_t n_rows = b->cu_seqlens[b->n_req];
  const bool own_rope = b->rope && (!one_launch || (int64_t)n_rows * b->n_q_heads * b->dim_qk * 2 > Q_IN_ONE_LAUNCH);
  size_t off_pos = align16(off_units + (paged ? (size_t)kv_cu.back() * sizeof(int32_t) : n_gather * sizeof(TileDesc)));
  size_t bytes = align16(off_pos + (own_rope ? sizeof(int32_t) * (size_t)n_rows : 0));
  const size_t off_w = bytes, w_bytes = b->rope ? sizeof(double) * (size_t)(b->rope->rotary_dim / 2) : 0;
  spd_stage* st;
  if ((rc = stage_acquire(ctx, SPD_PHASE_PREFILL, bytes + w_bytes, &st)) != SPD_OK) return rc;
  char* ws = nullptr;                                               // the metadata's device twin
  if ((rc = workspace_reserve(ctx, SPD_PHASE_PREFILL, bytes, &ws)) != SPD_OK) return rc;
  TileDesc *h_desc = (TileDesc*)(st->host + off_desc), *h_gather = (TileDesc*)(st->host + off_gather);
  int32_t* h_units = (int32_t*)(st->host + off_units);
  {
    std::lock_guard<std::mutex> lk(pool->mu);                       // atomic: query, get, update
    int64_t need = 0;
    for (int r = 0; r < b->n_req; ++r) {
      const int32_t len = b->cu_seqlens[r + 1] - b->cu_seqlens[r], pre = chunked ? b->prefix_lens[r] : 0;
      if (pre > 0) {                                                // the cached prefix must be there
        auto it = pool->tables.find(b->req_ids[r]);
        if (it == pool->tables.end()) return SPD_ENOENT;
        if ((int64_t)it->second.size() * g.P < pre) return SPD_EINVAL;
      }
      need += blocks_missing_locked(pool, b->req_ids[r], pre + len);
    }
    if (need > (int64_t)pool->free_stack.size()) return SPD_ENOMEM;
    for (int r = 0; r < b->n_req; ++r) {
      const int32_t row0 = b->cu_seqlens[r], len = b->cu_seqlens[r + 1] - row0, pre = chunked ? b->prefix_lens[r] : 0;
      reserve_locked(pool, b->req_ids[r], pre + len);
      spd_req_table& entry = pool->tables[b->req_ids[r]];
      entry.last_use[SPD_PHASE_PREFILL] = next_step_number(ctx, SPD_PHASE_PREFILL);
      const int n_new = build_tile_descs(g, entry.data(), pre, len, row0, h_desc);
      if (rows_k) {
        for (int i = 0; i < n_new; ++i) h_desc[i].pad[1] = kv_cu[(size_t)r] + pre + (h_desc[i].src_row - row0);
        h_gather += build_tile_descs(g, entry.data(), 0, one_launch ? pre : pre + len, kv_cu[(size_t)r], h_gather);
      }
      h_desc += n_new;
      if (paged) {
        const int n = kv_cu[(size_t)r + 1] - kv_cu[(size_t)r], tpp = g.tiles_per_page;
        for (int i = 0, page = 0; i < n; ++page)
          for (int sub = 0; sub < tpp && i < n; ++sub) h_units[i++] = entry[(size_t)page] * g.Hkv * tpp + sub;
        h_units += n;
      }
    }
  }
  hipStream_t stream;
  if ((rc = phase_enter(ctx, SPD_PHASE_PREFILL, &stream)) != SPD_OK) return rc;
  StepScope step{ctx, SPD_PHASE_PREFILL, st, stream};
  memcpy(st->host, work.data(), work.size() * sizeof(PrefillWork));
  memcpy(st->host + off_chain, chain.data(), chain.size() * sizeof(int32_t));
  if (!shared.range.empty()) memcpy(st->host + off_range, shared.range.data(), shared.range.size() * sizeof(PrefillRange));
  if (!merge.empty()) memcpy(st->host + off_merge, merge.data(), merge.size() * sizeof(PrefillMerge));
  StepMark mark = step_mark(ctx, SPD_PHASE_PREFILL, step.capturing);
  const double* rope_w = nullptr;
  if (ctx->kernel_timing) SPD_HIP(hipEventRecord(ps.ev_start, stream));
  if (b->rope) {
    if (own_rope) {
      int32_t* pos = (int32_t*)(st->host + off_pos);
      for (int r = 0; r < b->n_req; ++r)
        for (int32_t i = b->cu_seqlens[r]; i < b->cu_seqlens[r + 1]; ++i)
          pos[i] = (chunked ? b->prefix_lens[r] : 0) + (i - b->cu_seqlens[r]);
    }
    if ((rc = rope_table(step, b->rope, st->host + off_w, st->dev + off_w, &mark, &rope_w)) != SPD_OK) return rc;
  }
  const void* page_src_k = g.kind == SPD_KV_GQA ? b->k : b->latent;
  const void* page_src_v = g.kind == SPD_KV_GQA ? b->v : nullptr;
  // the page write reads its descriptors straight out of the pinned staging buffer, and extra workgroups of the
  // same kernel copy the whole staging buffer to its device twin, where the attention kernel finds its lists
  const spd_rope_config* rc_ = b->rope;
  const TileDesc *d_desc = (const TileDesc*)(st->dev + off_desc);
  if (one_launch) {
    KvRows x;
    x.cus = share;
    x.copy_dst = ws; x.copy_src = st->dev; x.copy_bytes = bytes;
    if (rc_) {
      x.rope_w = rope_w; x.rot = rc_->rotary_dim; x.off = rc_->rotary_offset; x.interleaved = rc_->interleaved != 0;
      if (!own_rope) { x.q = (void*)b->q; x.n_q_heads = b->n_q_heads; }
    }
    if (rows_k) {
      x.d_cached = (const TileDesc*)(st->dev + off_gather); x.n_cached = (int)n_gather;
      x.k_all = rows_k; x.v_all = rows_v;
    }
    SPD_HIP(launch_kv_rows(g, pool->base, d_desc, (int)n_descs, page_src_k, page_src_v, x, mark, stream));
    if (own_rope)
      SPD_HIP(launch_rope((void*)b->q, b->n_q_heads, nullptr, 0, b->dim_qk, rc_->rotary_dim, rc_->rotary_offset,
                          rc_->interleaved != 0, n_rows, (const int32_t*)(ws + off_pos), rope_w, StepMark{}, stream));
  } else {
    if (rc_) {
      SPD_HIP(launch_rope((void*)b->q, b->n_q_heads, (void*)b->k, b->n_kv_heads, b->dim_qk, rc_->rotary_dim, rc_->rotary_offset,
                          rc_->interleaved != 0, n_rows, (const int32_t*)(st->dev + off_pos), rope_w, mark, stream));
      mark.flag = nullptr;
    }
    if (g.kind == SPD_KV_MLA_LATENT_FP8)
      SPD_HIP(launch_kv_write_fp8(g, pool->base, d_desc, (int)n_descs, page_src_k, mark, stream, ws, st->dev, bytes));
    else
      SPD_HIP(launch_kv_write(g, pool->base, d_desc, (int)n_descs, page_src_k, page_src_v, mark, stream, ws, st->dev, bytes));
    if (rows_k) SPD_HIP(launch_kv_gather(g, pool->base, (const TileDesc*)(ws + off_gather), (int)n_gather, rows_k, rows_v, StepMark{}, stream));
  }
  if ((rc = kernel_timing_mark(ctx, SPD_PHASE_PREFILL, 0, stream)) != SPD_OK) return rc;
  const PrefillLists lists{(const PrefillWork*)ws, (const int32_t*)(ws + off_chain), (int)chain.size() - 1,
                           shared.range.empty() ? nullptr : (const PrefillRange*)(ws + off_range), (const PrefillMerge*)(ws + off_merge), (int)merge.size(), parts,
                           paged ? pool->base : nullptr, (const int32_t*)(ws + off_units), g.tiles_per_page};
  const bool two_groups = b->dim_qk == 192 && two_groups_pay(b->cu_seqlens, b->n_req);
  SPD_HIP(launch_prefill(b->q, rows_k ? rows_k : b->k, rows_k ? rows_v : b->v, b->out, lists, two_groups, b->n_q_heads, b->n_kv_heads, b->dim_qk,
                         b->dim_v, b->scale, stream));
  if ((rc = kernel_timing_mark(ctx, SPD_PHASE_PREFILL, 1, stream)) != SPD_OK) return rc;
  if ((rc = step.commit()) != SPD_OK) return rc;
  if (ctx->kernel_timing) {
    SPD_HIP(hipEventRecord(ps.ev_end, stream));
    ps.timed = true;
  }
  return SPD_OK;
}

// ------------------------------------------------------------------------------------------ decode
// A compute unit holds two workgroups of the GQA kernel (64-dim heads: three).  From the third (fifth) on, what each of them does
// before its first tile is waited for in turn.
// Then the records are copied to the device first: with 30-token contexts on 64 .. 256 CUs reading them there takes 0.81 .. 0.98 of
// the step's time with the reads over the host link, 3 to 24 workgroups per compute unit; 1.02 .. 1.15 below 3.
static bool gqa_many(int n_wgs, int share, int dim) { return dim > 64 ? n_wgs >= 3 * share : n_wgs > 4 * share; }
// And where HBM does not hide it, a launch rotates and appends for all of them.  It does where the workgroups' rows, at the rate
// of all the share's compute units, take longer: line at 32 MiB (no rotation: 24) of mean bytes per workgroup times compute units.
// Step without the launch ahead / with it, 8 KV heads of 128 dims with RoPE, tokens per workgroup: 64 CUs 200 1.35 .. 1.51,
// 590 1.12, 1000 1.05, 1729 1.01; 128 CUs 200 1.23, 365 1.09, 600 1.02, 914 0.99; 256 CUs 164 1.03 .. 1.05, 274 0.99, 579 0.96.  Append
// alone: 64 CUs 590 1.03, 914 0.99; 128 CUs 300 1.00 .. 1.02, 450 0.96; 256 CUs 200 0.99.
static bool gqa_prepares(int64_t bytes, int n_wgs, int share, bool rope) { return bytes / n_wgs * share <= (rope ? 32 << 20 : 24 << 20); }

// noalloc: the variant that allocates nothing.  The metadata's device twin and the workspace lie in the static scratch
// array, the staging ring is used as spd_ctx_create made it, no timing events are recorded.
static int decode_step_impl(spd_ctx* ctx, spd_pool* pool, const spd_decode_batch* b, bool noalloc) {
  if (!ctx || !pool || pool->ctx != ctx || !b || b->n_req <= 0 || !b->req_ids || !b->ctx_lens) return SPD_EINVAL;
  if (!b->q || !b->out || b->n_q_heads <= 0) return SPD_EINVAL;
  const PoolGeom& g = pool->geom;
  if (b->n_q_heads % g.Hkv != 0 || b->n_q_heads / g.Hkv > 16) return SPD_EINVAL;
  if (!(b->scale > 0.f) || !std::isfinite(b->scale)) return SPD_EINVAL;
  const bool append = b->k_new != nullptr;
  if (append && (g.kind == SPD_KV_GQA) != (b->v_new != nullptr)) return SPD_EINVAL;
  if (!append && b->v_new) return SPD_EINVAL;
  if (misaligned16(b->q, b->out, b->k_new, b->v_new)) return SPD_EINVAL;
  spd_phase_state& ds = ctx->phase[SPD_PHASE_DECODE];
  for (int r = 0; r < b->n_req; ++r)
    if (b->ctx_lens[r] <= 0) return SPD_EINVAL;                            // empty context
  if (append && has_duplicates(b->req_ids, b->n_req, ds.tmp_set)) return SPD_EINVAL;
  if (b->rope) {
    if (g.kind == SPD_KV_MLA_LATENT_FP8) return SPD_EINVAL;
    int rrc = rope_config_check(b->rope);
    if (rrc != SPD_OK) return rrc;
    if (b->rope->rotary_dim % 16 || b->rope->rotary_dim > 256 || b->rope->rotary_offset % 8 ||
        b->rope->rotary_offset + b->rope->rotary_dim > g.dk)
      return SPD_EINVAL;
  }
  if (ctx->device < 0) return SPD_ESTATE;

  const int B = b->n_req;
  const bool mla = g.kind != SPD_KV_GQA;
  const int units_per_page = g.P / TILE_T;
  int64_t sum_units = 0;
  int32_t max_units = 0, max_pages = 0;
  for (int r = 0; r < B; ++r) {
    const int32_t units = (b->ctx_lens[r] + TILE_T - 1) / TILE_T;
    sum_units += units;
    max_units = std::max(max_units, units);
    max_pages = std::max(max_pages, (b->ctx_lens[r] + g.P - 1) / g.P);
  }

  // the share this step will run on: a staged partition is adopted further down, once nothing but a HIP call can
  // fail any more, so a step that returns an error of its own leaves the partition as it was
  int rc;
  int share;
  {
    std::lock_guard<std::mutex> lk(ctx->part_mu);
    share = ds.has_pending ? ds.pending_cus : ds.active_cus;
  }
  std::vector<int32_t>& n_chunks = ds.tmp_chunks;
  n_chunks.resize((size_t)B);
  DecodeSplit sp;
  const size_t w_bytes = b->rope ? sizeof(double) * (size_t)(b->rope->rotary_dim / 2) : 0;
  const int cut = ctx->env_decode_chunk_tiles;
  const int64_t cost = g.kind == SPD_KV_MLA_LATENT_FP8 ? CHUNK_COST_FP8 : CHUNK_COST;
  if (!mla) split_gqa(ds, b->ctx_lens, B, sum_units, max_units, g.Hkv, share, cut, n_chunks.data(), sp);
  else if (!noalloc) split_latent(ds, b->ctx_lens, B, sum_units, share, units_per_page, cut, 0, n_chunks.data(), sp, cost);
  else
    split_latent_within_limits(ds, b->ctx_lens, B, b->n_q_heads, g.dv, sum_units, max_pages, share, units_per_page, cut, append, w_bytes,
                               n_chunks.data(), sp, cost);
  const std::vector<DecodeItem>& items = ds.tmp_items;
  const int n_items = (int)items.size(), max_chunks = sp.max_chunks;
  const DecodeRecords rec_layout = decode_records(sp, n_items, B, max_pages, units_per_page);
  const size_t stride = rec_layout.stride, off_chunks = rec_layout.off_chunks, bytes = rec_layout.bytes;
  if (stride > INT32_MAX) return SPD_EINVAL;
  if (noalloc && noalloc_metadata(n_items, B, max_pages, append, w_bytes) > NOALLOC_STAGE_BYTES) return SPD_ETOOBIG;
  spd_stage* st;
  if ((rc = stage_acquire(ctx, SPD_PHASE_DECODE, bytes + w_bytes, &st, !noalloc)) != SPD_OK) return rc;
  const bool timing = ctx->kernel_timing && !noalloc;
  const int n_wgs = sp.n_wgs * g.Hkv;
  // Few workgroups read their records straight out of the pinned staging buffer: a launch less.  Above 128 KiB, as the
  // workgroups read them, they are copied too (a latent pool's workgroups, at most two per compute unit, are served as well from
  // pinned memory up to there: 2048 records on 128 CUs 155 us, 159 copied).
  const bool many = !mla && gqa_many(n_wgs, share, g.dk);
  bool twin = many || (size_t)n_items * g.Hkv * stride > 131072;
  bool prepare = many && (append || b->rope) &&
                 gqa_prepares(sum_units * TILE_T * g.Hkv * (g.dk + g.dv) * (int64_t)sizeof(uint16_t), n_wgs, share, b->rope != nullptr);
  if (noalloc && bytes > NOALLOC_TWIN_BYTES) twin = prepare = false;
  // Split-K partials of a GQA launch of few workgroups are merged by that launch, where a request has few chunks; else by a
  // launch of its own.  Whole step over 128-dim heads, in the launch / on its own: 24 workgroups, 3 chunks 9.1 / 10.9 us; 192, 9
  // chunks 11.4 / 12.2 on 128 CUs; 400, 9 chunks 14.1 / 15.1 on 256; level from 500 to 1100 workgroups; 1392, 16 chunks 51.0 / 48.0
  // (each workgroup pays for going past the L2).  Never for latent pools: their partials are four times as long, and the one
  // workgroup that merges a request's 16 heads was 7 to 19 us at it (1 request of 4000 tokens in 16 chunks 39.6 / 20.4 us, 16 of 300
  // tokens 22.7 / 19.4).
  const bool inline_merge = !mla && n_wgs <= 512 && max_chunks <= MERGE_IN_LAUNCH_CHUNKS && (size_t)B * g.Hkv <= MERGE_COUNTERS;
  char* ws = nullptr;
  const size_t ws_o_bytes = partial_o_bytes(B, b->n_q_heads, max_chunks, g.dv), ws_ml_bytes = partial_ml_bytes(B, b->n_q_heads, max_chunks);
  size_t ws_q_bytes = prepare && b->rope ? sizeof(uint16_t) * (size_t)B * b->n_q_heads * g.dk : 0;   // rotated queries
  if (noalloc && ws_q_bytes && ws_o_bytes + ws_ml_bytes + ws_q_bytes > NOALLOC_WS_BYTES) {
    prepare = false;
    ws_q_bytes = 0;
  }
  // A merge launch reads the requests' chunk counts first of all: out of device memory, where the records have them in pinned memory.
  const bool put_chunks = !twin && !inline_merge && max_chunks > 1;
  const size_t ws_bytes = ws_o_bytes + ws_ml_bytes + ws_q_bytes + (noalloc ? 0 : twin ? bytes : put_chunks ? sizeof(int32_t) * (size_t)B : 0);
  if (noalloc) {
    if (ws_bytes > NOALLOC_WS_BYTES) return SPD_ETOOBIG;
    ws = ctx->scratch + NOALLOC_TWIN_BYTES;
  } else if (ws_bytes > 0 && (rc = workspace_reserve(ctx, SPD_PHASE_DECODE, ws_bytes, &ws)) != SPD_OK) {
    return rc;
  }

  int32_t* h_chunks = (int32_t*)(st->host + off_chunks);
  std::vector<spd_req_table*>& tables = ds.tmp_tables;
  tables.assign((size_t)B, nullptr);
  {
    std::lock_guard<std::mutex> lk(pool->mu);                       // atomic: query, get, update
    int64_t need = 0;
    for (int r = 0; r < B; ++r) {
      auto it = pool->tables.find(b->req_ids[r]);
      if (it != pool->tables.end()) tables[(size_t)r] = &it->second;
      const int64_t have = it == pool->tables.end() ? 0 : (int64_t)it->second.size();
      if (append) {
        need += std::max<int64_t>(0, (b->ctx_lens[r] + (int64_t)g.P - 1) / g.P - have);
      } else {
        if (it == pool->tables.end()) return SPD_ENOENT;
        if (have * g.P < b->ctx_lens[r]) return SPD_EINVAL;
      }
    }
    if (need > (int64_t)pool->free_stack.size()) return SPD_ENOMEM;
    const uint64_t number = next_step_number(ctx, SPD_PHASE_DECODE);
    for (int r = 0; r < B; ++r) {
      if (append) {
        if (!tables[(size_t)r]) tables[(size_t)r] = &pool->tables[b->req_ids[r]];
        reserve_entry_locked(pool, *tables[(size_t)r], b->ctx_lens[r]);
      }
      tables[(size_t)r]->last_use[SPD_PHASE_DECODE] = number;
    }
    const int words = (int)((stride - sizeof(DecodeItem)) / sizeof(int32_t));
    char* rec = st->host;
    for (int i = 0; i < n_items; ++i, rec += stride) {
      DecodeItem it = items[(size_t)i];
      it.n_chunks = n_chunks[(size_t)it.req];
      *(DecodeItem*)rec = it;
      const int32_t p0 = it.unit0 / units_per_page, p1 = (it.unit0 + it.n_units - 1) / units_per_page + 1;
      const int32_t* src = tables[(size_t)it.req]->data();
      int32_t* dst = (int32_t*)(rec + sizeof(DecodeItem));
      memcpy(dst, src + p0, sizeof(int32_t) * (size_t)(p1 - p0));
      for (int32_t j = p1 - p0; j < words; ++j) dst[j] = src[p1 - 1];
    }
    memcpy(h_chunks, n_chunks.data(), sizeof(int32_t) * (size_t)B);
  }
  hipStream_t stream;
  if ((rc = phase_enter(ctx, SPD_PHASE_DECODE, &stream)) != SPD_OK) return rc;
  StepScope step{ctx, SPD_PHASE_DECODE, st, stream};
  if (timing) SPD_HIP(hipEventRecord(ds.ev_start, stream));
  StepMark mark = step_mark(ctx, SPD_PHASE_DECODE, step.capturing);
  DecodeLaunch d{};
  if (b->rope && (rc = rope_table(step, b->rope, st->host + bytes, st->dev + bytes, &mark, &d.w)) != SPD_OK) return rc;
  d.q = b->q; d.k_new = b->k_new; d.v_new = b->v_new; d.out = b->out;
  d.items = st->dev; d.n_chunks = (const int32_t*)(st->dev + off_chunks);
  d.item_stride = (int)stride; d.n_wgs = sp.n_wgs; d.B = B; d.H = b->n_q_heads; d.scale = b->scale;
  d.max_chunks = max_chunks;
  if (b->rope) { d.rot = b->rope->rotary_dim; d.off = b->rope->rotary_offset; d.interleaved = b->rope->interleaved != 0; }
  d.ws_o = (float*)ws; d.ws_ml = (float*)(ws + ws_o_bytes);
  d.counters = inline_merge ? ds.merge_counters : nullptr;
  d.mark = mark;
  if (put_chunks) {
    static_assert(NOALLOC_STAGE_BYTES <= NOALLOC_TWIN_BYTES, "room for a count per request");
    d.put_chunks = (int32_t*)(noalloc ? ctx->scratch : ws + ws_o_bytes + ws_ml_bytes + ws_q_bytes);
    d.n_chunks = d.put_chunks;
  }
  if (twin) {
    char* q_rot = ws + ws_o_bytes + ws_ml_bytes;
    char* to = noalloc ? ctx->scratch : q_rot + ws_q_bytes;
    SPD_HIP(launch_meta_copy(to, st->dev, bytes, mark, stream));
    d.mark.flag = nullptr;
    d.items = to;
    d.n_chunks = (const int32_t*)(to + off_chunks);
    if (prepare) {
      SPD_HIP(launch_decode_prepare(g, pool->base, d, n_items, q_rot, stream));
      if (b->rope) d.q = q_rot;
      d.prepared = true;
    }
  }
  if (timing && (rc = kernel_timing_mark(ctx, SPD_PHASE_DECODE, 0, stream)) != SPD_OK) return rc;
  if (mla) SPD_HIP(launch_decode_mla(g, pool->base, d, stream));
  else SPD_HIP(launch_decode_gqa(g, pool->base, d, stream));
  if (timing && (rc = kernel_timing_mark(ctx, SPD_PHASE_DECODE, 1, stream)) != SPD_OK) return rc;
  if ((rc = step.commit()) != SPD_OK) return rc;
  if (timing) {
    SPD_HIP(hipEventRecord(ds.ev_end, stream));
    ds.timed = true;
  }
  return SPD_OK;
}

extern "C" int spd_decode_step(spd_ctx* ctx, spd_pool* pool, const spd_decode_batch* b) {
  return decode_step_impl(ctx, pool, b, false);
}

extern "C" int spd_decode_step_noalloc(spd_ctx* ctx, spd_pool* pool, const spd_decode_batch* b) {
  return decode_step_impl(ctx, pool, b, true);
}

extern "C" int spd_noalloc_limits(uint64_t* metadata_bytes, uint64_t* workspace_bytes) {
  if (metadata_bytes) *metadata_bytes = NOALLOC_STAGE_BYTES;
  if (workspace_bytes) *workspace_bytes = NOALLOC_WS_BYTES;
  return SPD_OK;
}


// ------------------------------------------------------------------------------------------ decode worker
struct spd_worker {
  std::thread th;
  std::atomic<bool> stop{false};
  std::atomic<int64_t> issued{0};
  std::atomic<int> status{SPD_OK};
};

extern "C" int spd_decode_worker_start(spd_ctx* ctx, spd_pool* pool, const spd_decode_batch* const* batches,
                                       int32_t n_batches, spd_worker** out) {
  if (!ctx || !pool || pool->ctx != ctx || !batches || n_batches <= 0 || !out) return SPD_EINVAL;
  for (int i = 0; i < n_batches; ++i)
    if (!batches[i]) return SPD_EINVAL;
  if (ctx->device < 0) return SPD_ESTATE;
  spd_worker* w = new (std::nothrow) spd_worker();
  if (!w) return SPD_EINVAL;
  std::vector<const spd_decode_batch*> list(batches, batches + n_batches);
  w->th = std::thread([w, ctx, pool, list]() {
    if (hipSetDevice(ctx->device) != hipSuccess) {
      w->status.store(SPD_EHIP);
      return;
    }
    size_t i = 0;
    do {                                          // at least one step, however early the stop comes
      const int rc = spd_decode_step(ctx, pool, list[i]);
      if (rc != SPD_OK) {
        w->status.store(rc);
        return;
      }
      w->issued.fetch_add(1, std::memory_order_relaxed);
      i = (i + 1) % list.size();
    } while (!w->stop.load(std::memory_order_relaxed));
  });
  *out = w;
  return SPD_OK;
}

extern "C" int spd_decode_worker_steps(spd_worker* w, int64_t* steps_issued) {
  if (!w || !steps_issued) return SPD_EINVAL;
  *steps_issued = w->issued.load(std::memory_order_relaxed);
  return SPD_OK;
}

extern "C" int spd_decode_worker_stop(spd_worker* w, int64_t* steps_issued, int* status) {
  if (!w) return SPD_EINVAL;
  w->stop.store(true);
  if (w->th.joinable()) w->th.join();
  if (steps_issued) *steps_issued = w->issued.load();
  if (status) *status = w->status.load();
  delete w;
  return SPD_OK;
}
