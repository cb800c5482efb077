// Internal declarations shared by the host side and the kernels of libsemipd.
// Not part of the public ABI (see include/semipd.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <map>
#include <atomic>
#include <mutex>
#include <unordered_map>
#include <vector>

#include "semipd.h"

namespace spd {

// ---------------------------------------------------------------------------------------------
// Page layout in HBM.
//
// Tokens are grouped in tiles of 16 (TILE_T).  A GQA page holds, for every KV head g, a
// contiguous "head region" of P/16 tiles; each tile is a K part followed by a V part:
//
//   K part (16 tokens x dk):  [chunk c = d/8][token t][8 dims]
//       A wave that loads "chunk 4s + lane/16, token lane%16" with one 16-byte load per lane
//       reads 1 KiB contiguous and gets exactly the A operand of v_mfma_f32_16x16x32_bf16
//       (row = token, 8 consecutive contraction elements per lane) for k-step s.
//   V part (16 tokens x dv):  [d/32][token quad t/4][d%16][(d/16)%2][t%4]
//       One 16-byte load per lane at "(blk2*4 + lane/16)*16 + lane%16" is again 1 KiB
//       contiguous and holds the A operands (row = d, 4 consecutive tokens per lane) of two
//       v_mfma_f32_16x16x16_bf16 for the value blocks 2*blk2 and 2*blk2 + 1.
//
// An MLA latent page keeps the natural order: P rows of 576 dims.  Its decode kernel stages rows
// through LDS and reads them back in both operand orders (kernels_decode_mla.hip).
// ---------------------------------------------------------------------------------------------
constexpr int TILE_T = 16;
// FP8 latent pages: a cached row is 512 E4M3 codes, 4 fp32 scales (one per 128 entries) and 64 bf16 rope entries
constexpr int FP8_ROW_BYTES = 512 + 16 + 128;

struct PoolGeom {
  int kind, P, Hkv, dk, dv;
  int tiles_per_page;
  uint32_t tile_k_bytes, tile_v_bytes, tile_bytes, head_bytes;
  uint64_t page_bytes;
};

__host__ __device__ inline uint32_t k_elem_offset(int t16, int d) { return ((d >> 3) * 16 + t16) * 8 + (d & 7); }
__host__ __device__ inline uint32_t v_elem_offset(int t16, int d) {
  return (((((d >> 5) * 4 + (t16 >> 2)) * 16 + (d & 15)) * 2 + ((d >> 4) & 1)) * 4) + (t16 & 3);
}

inline PoolGeom make_geom(const spd_pool_desc& d) {
  PoolGeom g{};
  g.kind = d.kind; g.P = d.page_tokens; g.Hkv = d.n_kv_heads; g.dk = d.dim_k; g.dv = d.dim_v;
  g.tiles_per_page = d.page_tokens / TILE_T;
  g.tile_k_bytes = d.kind == SPD_KV_MLA_LATENT_FP8 ? TILE_T * FP8_ROW_BYTES : TILE_T * d.dim_k * 2;
  g.tile_v_bytes = d.kind == SPD_KV_GQA ? TILE_T * d.dim_v * 2 : 0;
  g.tile_bytes = g.tile_k_bytes + g.tile_v_bytes;
  g.head_bytes = g.tiles_per_page * g.tile_bytes;
  g.page_bytes = (uint64_t)g.head_bytes * d.n_kv_heads;
  return g;
}

// One 16-token tile's worth of rows to copy between a dense [rows, heads, dim] tensor and a page.
struct TileDesc {
  int32_t src_row;   // row of the dense tensor that maps to token t_begin of the tile
  int32_t page;      // physical page id
  int32_t sub;       // tile index inside the page
  int32_t t_begin;   // first token slot (0..15) touched
  int32_t t_end;     // one past the last token slot touched
  int32_t pad[3];    // [0]: logical position of the tile's token slot 0 in its request; [1]: row of KvRows::k_all that t_begin maps to
};

// A step's first kernel stores `seq`, the number of the phase's step before it, at `flag`: that step has finished.
struct StepMark {
  uint64_t* flag;
  uint64_t seq;
};
#if defined(__HIPCC__)
__device__ inline void store_mark(const StepMark& m) {
  if (m.flag) __hip_atomic_store(m.flag, m.seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
#endif

// Decode work item = one chunk of one request's context: this header, then the ids of the pages the chunk touches (the
// first one is the page of the chunk's first token), the last id repeated up to the record's end.  Everything a
// workgroup needs sits at an address it knows from its own number, so that it is had in one round trip, which counts
// where the records are read over PCIe out of the staging buffer.
struct DecodeItem {
  int32_t req, chunk, n_chunks;
  int32_t n;         // attended tokens of the request
  int32_t unit0, n_units;   // the chunk, in units of 16 tokens
  int32_t next;      // the record the workgroup goes on with, or -1 (latent decode)
  int32_t pad;
};
constexpr int DECODE_ITEM_WORDS = sizeof(DecodeItem) / 4;

// What a decode attention launch is given.
struct DecodeLaunch {
  const void *q, *k_new, *v_new;      // k_new: null without append
  void* out;
  const char* items;                  // n_items records of item_stride bytes
  const int32_t* n_chunks;            // [B], for the merge launch
  int32_t* put_chunks;                // where the attention launch puts them, for a merge launch that would find them in pinned memory; or null
  const double* w;                    // rot / 2 frequencies
  int item_stride, n_wgs, B, H;       // n_wgs: workgroups (GQA: per KV head), each starts with the record of its number
  float scale;
  int max_chunks;
  int rot, off, interleaved;          // rot = 0: no rotation
  float *ws_o, *ws_ml;
  bool prepared;                      // GQA: launch_decode_prepare has rotated and appended
  uint32_t* counters;                 // [B * Hkv] zeros: the chunks are merged by the last workgroup (GQA); null: by a launch of its own
  StepMark mark;
};

// Prefill work item = one workgroup: one tile of query rows of one request, for a group of query
// heads that share a KV head.  len == 0 marks a padding item (the workgroup exits at once).
struct PrefillWork {
  int32_t row0;      // first packed row of the request's queries (and outputs)
  int32_t len;       // number of query rows of the request in this step
  int32_t q_tile;    // tile index inside those rows (tile height depends on the head grouping)
  int32_t head0;     // first query head of the workgroup's head group
  int32_t kv_row0;   // where the request's keys and values begin in what the kernel reads: its first unit in PrefillLists::units, or row of k, v
  int32_t q_off;     // position of query row 0 in the request = number of cached tokens before it
};
// What an item of a step with shared-out items visits (a list beside the items': the others, of more items, have nothing to stage for it).
struct PrefillRange {
  int32_t kt0, kt1;  // the tiles of 64 keys: all that the rows can see, or a part of them
  int32_t part;      // number of the part, where its sums go; -1: the item is whole
};
// An item that was shared out: its parts are part0 .. part0 + n_parts - 1.
struct PrefillMerge {
  int32_t row0, len, q_tile, head0, part0, n_parts;
};
// floats that a part leaves: 8 waves x (32 rows x dv sums, reference and row sum of 32 rows)
constexpr __host__ __device__ inline size_t prefill_part_floats(int dv) { return 8 * (size_t)(dv * 32 + 64); }
// What launch_prefill reads on the device.
// A step with cached tokens has all its keys and values, its own rows among them, as dense rows, request after request (dense_rows_pay),
// or out of the pages, where its own are written ahead:
// `units` holds for each request the numbers of its units (16 tokens of one head: K part, V part, consecutive in a page) for KV head 0,
// in the order of the tokens; head g's are g * head_units further.
struct PrefillLists {
  const PrefillWork* work;
  const int32_t* chain;
  int n_blocks;
  const PrefillRange* range;   // null: all items are whole
  const PrefillMerge* merge;
  int n_merge;
  float* parts;
  const char* pages;           // null: k, v are dense rows
  const int32_t* units;
  int head_units;
};

// The entry point that allocates nothing keeps its device-side working memory in one static device
// array (noalloc.hip): the metadata's device twin (one, written and read in stream order), then the
// split-K partials.
constexpr size_t NOALLOC_STAGE_BYTES = 256u << 10;   // limit of a step's metadata as noalloc_metadata counts it
constexpr size_t NOALLOC_WS_BYTES = 32u << 20;
constexpr size_t NOALLOC_TWIN_BYTES = 4 * NOALLOC_STAGE_BYTES;   // a longer batch's records are read from pinned memory
// Pinned bytes of a staging slot of the decode phase: any batch within NOALLOC_STAGE_BYTES in the form the kernels read.
// A record is at least 64 bytes, where the limit counts 16 (one page, nothing appended: 16384 requests, 1.06 MiB) or, of a
// long context cut into many items, 8 (32768 of them, 2 MiB; only with SPD_DECODE_CHUNK_TILES).
constexpr size_t NOALLOC_RING_BYTES = 9 * NOALLOC_STAGE_BYTES;
constexpr size_t MERGE_COUNTERS = 4096;
constexpr int MERGE_IN_LAUNCH_CHUNKS = 16; // most chunks of a request that a workgroup of the attention launch merges on the side
constexpr int STAGE_SLOTS = 8;             // staging slots of a phase (captured steps keep theirs)
constexpr int STEPS_IN_FLIGHT = 4;         // steps of a phase in flight before a new one waits for the oldest
constexpr size_t SCRATCH_BYTES = NOALLOC_TWIN_BYTES + NOALLOC_WS_BYTES;

extern thread_local int g_last_hip_error;
inline int hip_fail(hipError_t e) { g_last_hip_error = (int)e; return SPD_EHIP; }
#define SPD_HIP(expr) do { hipError_t _e = (expr); if (_e != hipSuccess) return ::spd::hip_fail(_e); } while (0)

}  // namespace spd

// ------------------------------------------------------------------------------------------ objects
// A request's block table, and for each phase the number of the last step of that phase that took the table
// (0: none): spd_kv_free refuses while such a step may still be running on the GPU.
struct spd_req_table : std::vector<int32_t> {
  uint64_t last_use[2] = {0, 0};
};

struct spd_pool {
  spd_ctx* ctx;
  spd_pool_desc desc;
  spd::PoolGeom geom;
  char* base;
  uint64_t bytes;
  std::mutex mu;                                  // the "lock on memory utilisation"
  std::vector<int32_t> free_stack;                // top = back()
  int64_t used = 0;
  uint64_t op_seq = 0;
  std::unordered_map<uint64_t, spd_req_table> tables;
};

struct spd_stage {          // pinned host buffer a step's metadata is read from, reused round-robin per phase
  char* host = nullptr;
  char* dev = nullptr;      // the same buffer as the device addresses it
  size_t cap = 0;
  uint64_t seq = 0;         // number of the last step that used the slot (0: none)
  bool captured = false;    // a graph's replays read the buffer: not handed round any more
};

// An event recorded behind a step, for the steps whose end no later step of the phase reports (see phase_seal).
struct spd_seal {
  hipEvent_t ev = nullptr;
  std::atomic<uint64_t> seq{0};       // that step's number (stored after the event has been recorded)
};

struct spd_phase_state {
  hipStream_t stream = nullptr;        // active
  int active_cus = 0;
  hipStream_t pending_stream = nullptr;
  int pending_cus = 0;
  bool has_pending = false;
  std::vector<uint32_t> active_mask, pending_mask;
  spd_stage ring[spd::STAGE_SLOTS];
  int ring_pos = 0;
  uint64_t recent[spd::STEPS_IN_FLIGHT] = {};   // numbers of the last steps that were issued, not captured; oldest at recent_pos
  int recent_pos = 0;
  std::vector<char*> kept;             // buffers of captured steps whose slots have got new ones
  // One word of pinned memory per phase: the first kernel of every step stores the number of the step before it, which
  // the stream has finished by then.  Steps cost no event this way (an event record is 2 us of host time and 4 to 6 us
  // of the stream's).
  uint64_t* flag = nullptr;            // host address
  uint64_t* flag_dev = nullptr;        // the same word as the device addresses it
  spd_seal seals[spd::STAGE_SLOTS];
  int seal_pos = 0;
  std::mutex seal_mu;
  uint64_t sealed_seq = 0;             // latest step with a seal of its own
  std::atomic<bool> stream_lent{false};            // spd_phase_stream has handed the stream out: the caller's own work may follow any step
  std::atomic<uint64_t> issue_seq{0};  // steps (ring commits) of this phase so far; the next step's number is this + 1
  std::atomic<uint64_t> done_seq{0};   // a step number known to have finished on the GPU (steps of a phase finish in order)
  hipEvent_t ev_start = nullptr, ev_end = nullptr, ev_switch = nullptr, ev_cross = nullptr;
  bool timed = false;
  // RoPE frequencies of the configuration the phase's steps used last, in device memory (rope_table)
  double* rope_dev = nullptr;
  spd_rope_config rope_key{};
  bool rope_valid = false;
  uint32_t* merge_counters = nullptr;  // decode phase: MERGE_COUNTERS zeros (split_merge.h), zero again after every step
  // a step's working lists, kept from step to step (one thread drives a phase)
  std::vector<uint64_t> tmp_set, tmp_heap;
  std::vector<spd::DecodeItem> tmp_items, tmp_items2;
  std::vector<spd_req_table*> tmp_tables;
  std::vector<int32_t> tmp_sizes, tmp_chunks, tmp_owner, tmp_last;
  char* workspace = nullptr;           // split-K partials (decode)
  size_t ws_cap = 0;
  char* parts = nullptr;               // sums of items that were shared out (prefill)
  size_t parts_cap = 0;
  char* rows = nullptr;                // keys and values of a chunked step as dense rows (prefill)
  size_t rows_cap = 0;
  // workspaces outgrown, with the number of the last step that may still read them: freed once that step has
  // finished (looked at when the workspace grows again, in spd_phase_sync and when the context goes)
  std::vector<std::pair<char*, uint64_t>> ws_retired;
  std::mutex ws_mu;                    // the list above (a step's thread against another thread's spd_phase_sync)
  hipEvent_t kev[256][2] = {};         // kernel timing ring (measurement aid)
  uint64_t kev_count = 0, kev_read = 0;
};

struct spd_ctx {
  int device = -1;                     // -1: host only
  int total_cus = 256, xcds = 8, granularity = 32;
  std::mutex part_mu;                  // partition state (set_partition vs step entry)
  std::map<std::vector<uint32_t>, hipStream_t> stream_cache;
  spd_phase_state phase[2];
  bool kernel_timing = false;
  int env_prefill_persistent = -1;     // SPD_PREFILL_PERSISTENT as read by spd_ctx_create (-1: not set)
  int env_decode_chunk_tiles = 0;      // SPD_DECODE_CHUNK_TILES as read by spd_ctx_create (0: not set)
  char* scratch = nullptr;             // this device's copy of the static scratch array (noalloc.hip)
};

namespace spd {
// host helpers (ctx.cpp)
int phase_enter(spd_ctx* ctx, int phase, hipStream_t* stream_out);   // adopt pending stream
// May the phase's next launch be one workgroup per compute unit of its share (the staged one, where one is)?  `share`: its size.
bool phase_exclusive(spd_ctx* ctx, int phase, int* share);
// may_alloc = false: SPD_ETOOBIG instead of growing the slot's buffers
int stage_acquire(spd_ctx* ctx, int phase, size_t bytes, spd_stage** out, bool may_alloc = true);
int scratch_resolve(int device, char** out);   // noalloc.hip: address of `device`'s copy of the scratch array
// behind the step's last launch: the step has its number
int stage_commit(spd_ctx* ctx, int phase, spd_stage* st, hipStream_t stream, bool capturing);
// Is a graph being captured on the phase's stream?  (Only where the caller has been given a phase's stream.)
bool stream_capturing(spd_ctx* ctx, hipStream_t stream);
// A step from its first launch on.  One that returns before its commit may have launches in the queue that read the staging slot,
// and its batch's requests carry its number: it counts as issued all the same, and what it left on the device (the
// RoPE table) as unknown.
// While a graph is captured on the stream the step's launches are only noted, to run at every replay: they then store no mark
// and take nothing from the device that a later step may overwrite.
struct StepScope {
  spd_ctx* ctx;
  int phase;
  spd_stage* st;
  hipStream_t stream;
  bool capturing, open = true;
  StepScope(spd_ctx* c, int ph, spd_stage* s, hipStream_t str) : ctx(c), phase(ph), st(s), stream(str), capturing(stream_capturing(c, str)) {}
  int commit() {
    open = false;
    return stage_commit(ctx, phase, st, stream, capturing);
  }
  ~StepScope() {
    if (!open) return;
    const int error = g_last_hip_error;
    ctx->phase[phase].rope_valid = false;
    (void)commit();
    g_last_hip_error = error;
  }
};
// what the first kernel enqueued behind the phase's last step stores (see spd_phase_state::flag)
StepMark step_mark(spd_ctx* ctx, int phase, bool capturing);
// Before anything but a step's first kernel goes onto the phase's stream: an event behind the last step, unless that
// step is known to have finished or has one.
int phase_seal(spd_ctx* ctx, int phase, hipStream_t stream);
// true if step number `seq` of `phase` has finished on the GPU (any thread may ask)
bool phase_step_done(spd_ctx* ctx, int phase, uint64_t seq);
int workspace_reserve(spd_ctx* ctx, int phase, size_t bytes, char** out);
// Memory for the parts of a prefill step's items, of its own, so that the workspace grows as ever; null: there is none, or the
// phase's stream, or the staged one, is being captured (the captured launches would outlive the buffer).
float* parts_reserve(spd_ctx* ctx, size_t bytes);
// The same for the dense rows of a chunked step.
char* rows_reserve(spd_ctx* ctx, size_t bytes);
int kernel_timing_mark(spd_ctx* ctx, int phase, int which, hipStream_t stream);   // which: 0 begin, 1 end
// rope.cpp: SPD_OK if the configuration is well-formed; the frequency table (rotary_dim / 2 doubles)
int rope_config_check(const spd_rope_config* c);
void rope_frequencies(const spd_rope_config* c, double* out);
// The frequency table of `c` in device memory, valid for the phase's work enqueued from here on.  A configuration the
// phase has not just used is written to a staging slot and copied by a launch of its own (rotary_dim <= ROPE_TABLE_DIM);
// a captured step reads it there.
constexpr int ROPE_TABLE_DIM = 1024;
int rope_table(const StepScope& step, const spd_rope_config* c, char* host, const char* host_dev, StepMark* mark, const double** out);

// kernel launchers (kernels_*.hip); all enqueue on `stream` and return the launch status; `mark` is stored by the launch
// where it is the first one behind a step (flag null: it is not)
// d_tiles may be device-readable pinned host memory.  With copy_dst non-null the same launch also
// copies copy_bytes (rounded up to 16) from copy_src to copy_dst.
hipError_t launch_kv_write(const PoolGeom& g, char* pool_base, const TileDesc* d_tiles, int n_tiles,
                           const void* k, const void* v, const StepMark& mark, hipStream_t stream, void* copy_dst = nullptr,
                           const void* copy_src = nullptr, uint64_t copy_bytes = 0);
// What a prefill step does besides the page write, in the same launch (only where kv_rows_supported).
struct KvRows {
  void* copy_dst = nullptr;             // metadata copy, as above
  const void* copy_src = nullptr;
  uint64_t copy_bytes = 0;
  const double* rope_w = nullptr;       // non-null: key rows are rotated, in the pages and in k (position = TileDesc.pad[0] + token slot)
  int rot = 0, off = 0;
  bool interleaved = false;
  void* q = nullptr;                    // with rope_w: the tiles' query rows [rows, n_q_heads, dk], rotated in place
  int n_q_heads = 0;
  const TileDesc* d_cached = nullptr;   // tiles of cached rows that go to k_all, v_all, as do the new rows (at TileDesc.pad[1])
  int n_cached = 0;
  void *k_all = nullptr, *v_all = nullptr;
  int cus = 0;                          // compute units that the launch will run on
};
bool kv_rows_supported(const PoolGeom& g);
hipError_t launch_kv_rows(const PoolGeom& g, char* pool_base, const TileDesc* d_tiles, int n_tiles, const void* k, const void* v,
                          const KvRows& x, const StepMark& mark, hipStream_t stream);
hipError_t launch_kv_gather(const PoolGeom& g, const char* pool_base, const TileDesc* d_tiles, int n_tiles,
                            void* k_out, void* v_out, const StepMark& mark, hipStream_t stream);
// FP8 latent pools (kernels_kv_fp8.hip): quantising page write of dense [rows, 576] bf16 latent rows (with the same
// optional metadata copy as launch_kv_write), and the gather that hands back the dequantised rows
hipError_t launch_kv_write_fp8(const PoolGeom& g, char* pool_base, const TileDesc* d_tiles, int n_tiles, const void* latent,
                               const StepMark& mark, hipStream_t stream, void* copy_dst = nullptr, const void* copy_src = nullptr,
                               uint64_t copy_bytes = 0);
hipError_t launch_kv_gather_fp8(const PoolGeom& g, const char* pool_base, const TileDesc* d_tiles, int n_tiles, void* out,
                                const StepMark& mark, hipStream_t stream);
hipError_t launch_meta_copy(void* dst, const void* src, uint64_t bytes, const StepMark& mark, hipStream_t stream);
// What `d` rotates and appends, ahead of the attention launch: its queries are rotated to q_rot (with d.rot), the new tokens go into
// their pages (with d.k_new).  d.items: n_items records in device memory.
hipError_t launch_decode_prepare(const PoolGeom& g, char* pool_base, const DecodeLaunch& d, int n_items, void* q_rot, hipStream_t stream);
hipError_t launch_decode_gqa(const PoolGeom& g, char* pool_base, const DecodeLaunch& d, hipStream_t stream);
hipError_t launch_decode_mla(const PoolGeom& g, char* pool_base, const DecodeLaunch& d, hipStream_t stream);
// The latent decode's workgroup fetches a record one word per thread and keeps it in LDS: as many pages as that leaves a chunk
// may touch, and no record may be longer (checked again at the launch).
constexpr int MLA_THREADS = 256;
constexpr int MLA_CHUNK_PAGES = MLA_THREADS - DECODE_ITEM_WORDS;
// one workgroup per chain: workgroup b computes the items work[chain[b]] .. work[chain[b + 1] - 1].  two_groups: 192 / 128 dims only, as
// two_groups_pay says
// (k, v are not read where lists.pages is there)
hipError_t launch_prefill(const void* q, const void* k, const void* v, void* out, const PrefillLists& lists, bool two_groups, int H, int Hkv, int dqk, int dv,
                          float scale, hipStream_t stream);
// x [T, K], w_gu [2 I, K] (joint gate/up rows in blocks of 32 + 32), out [T, I], all bf16 in device memory;
// K a multiple of 32, I a multiple of 128
// exclusive: as phase_exclusive says
hipError_t launch_ffn_gate_up(const void* x, const void* w_gu, void* out, int T, int K, int I, int xcds, int cus, bool exclusive,
                              const StepMark& mark, hipStream_t stream);
hipError_t launch_ffn_pack(const void* w_gate, const void* w_up, void* w_gu, int K, int I, hipStream_t stream);
// d_pos, d_w may be device-readable pinned host memory
hipError_t launch_rope(void* q, int n_q_heads, void* k, int n_kv_heads, int dim, int rot, int off, bool interleaved,
                       int n_tokens, const int32_t* d_pos, const double* d_w, const StepMark& mark, hipStream_t stream);
hipError_t launch_probe(int32_t* d_ids, int n_blocks, hipStream_t stream);
hipError_t launch_copy(void* dst, const void* src, uint64_t bytes, int cus, hipStream_t stream);
hipError_t launch_read(const void* src, uint64_t bytes, int cus, uint32_t* sink, hipStream_t stream);
hipError_t launch_read_lds(const void* src, uint64_t bytes, int cus, uint32_t* sink, hipStream_t stream);
hipError_t launch_clock_probe(uint64_t iters, uint64_t* d_out, hipStream_t stream);
hipError_t launch_issue_probe(uint64_t* d_out, hipStream_t stream);
bool prefill_shape_supported(int dqk, int dv);
int prefill_heads_per_block(int group);   // query heads of one KV head that share a workgroup
int prefill_block_m(int group);           // query rows per workgroup
}  // namespace spd
