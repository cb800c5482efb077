// The steps' host side (ctx.cpp, steps.cpp, pool.cpp, rope.cpp) over a stand-in for the HIP runtime, on the CPU: memory is
// host memory, a stream is a queue of closures that run when the test lets them, and a launch stores the step mark it was
// given and logs what it reads.  host_steps NAME runs one scenario.
#include <hip/hip_runtime.h>

#include <climits>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <deque>
#include <functional>
#include <set>
#include <string>
#include <vector>

#include "internal.h"

using namespace spd;

#define CHECK(x) do { if (!(x)) { fprintf(stderr, "check failed: %s (line %d)\n", #x, __LINE__); exit(1); } } while (0)

// ------------------------------------------------------------------------------------------ the runtime's stand-in
struct Stream {
  std::deque<std::function<void()>> queue;      // not yet run
  std::vector<std::function<void()>>* graph = nullptr;   // being captured
};
struct Event {
  bool recorded = false, done = false;
  std::vector<std::function<void()>>* graph = nullptr;   // recorded into a graph: who waits for it joins the capture
};
static std::vector<Stream*> streams;
static long n_pinned = 0, pinned_bytes = 0, n_device = 0;   // allocations so far
static int device = 0;                          // the calling thread's current one
static std::set<int> allocated_on;
static bool fail_malloc = false;                // the next allocation of device memory fails
static std::set<void*> freed;                   // device memory that was given back
static int fail_launch = -1;                    // the launch of this number fails
static int n_launches = 0;
static std::vector<PrefillLists> seen_lists;     // what every attention launch of a prefill step was given
static std::vector<const void*> seen_keys;       // ... and where it finds its keys, if not in the pages
static std::vector<int> seen_cus;                // compute units that every page write was told of
static uint64_t staged_bytes = 0;                // of the last prefill step: what its launch copies to the device
static std::vector<bool> seen_counters;         // may the decode launch merge its own chunks?
static std::vector<double> seen_w;              // sum of the RoPE frequencies that each decode launch found when it ran

static void put(hipStream_t s, std::function<void()> f) {
  Stream* st = (Stream*)s;
  if (st->graph) st->graph->push_back(f);
  else st->queue.push_back(f);
}
static void run(Stream* s, size_t n = SIZE_MAX) {
  for (; n && !s->queue.empty(); --n) {
    auto f = s->queue.front();
    s->queue.pop_front();
    f();
  }
}
extern "C" {
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) {
  memset(p, 0, sizeof *p);
  strcpy(p->gcnArchName, "gfx950");
  p->multiProcessorCount = 256;
  return hipSuccess;
}
hipError_t hipSetDevice(int d) { device = d; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipMalloc(void** p, size_t n) {
  if (fail_malloc) {
    fail_malloc = false;
    return hipErrorOutOfMemory;
  }
  ++n_device;
  allocated_on.insert(device);
  *p = calloc(1, n);
  return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void* p) { freed.insert(p); return hipSuccess; }   // (kept, so that no address comes twice)
hipError_t hipMemset(void* p, int v, size_t n) { memset(p, v, n); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  ++n_pinned;
  allocated_on.insert(device);
  pinned_bytes += (long)n;
  *p = aligned_alloc(4096, (n + 4095) / 4096 * 4096);
  return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipHostFree(void* p) { free(p); return hipSuccess; }
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned) { *d = h; return hipSuccess; }
hipError_t hipExtStreamCreateWithCUMask(hipStream_t* s, uint32_t, const uint32_t*) {
  streams.push_back(new Stream);
  *s = (hipStream_t)streams.back();
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) {
  if (((Stream*)s)->graph) return hipErrorStreamCaptureUnsupported;
  run((Stream*)s);
  return hipSuccess;
}
hipError_t hipStreamQuery(hipStream_t s) {      // whoever asks lets the stream go on by one
  if (((Stream*)s)->graph) return hipErrorStreamCaptureUnsupported;
  run((Stream*)s, 1);
  return ((Stream*)s)->queue.empty() ? hipSuccess : hipErrorNotReady;
}
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* st) {
  *st = ((Stream*)s)->graph ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) { *e = (hipEvent_t)new Event; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { delete (Event*)e; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  Event* ev = (Event*)e;
  ev->recorded = true;
  ev->done = false;
  ev->graph = ((Stream*)s)->graph;
  put(s, [ev] { ev->done = true; });
  return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t e) {
  Event* ev = (Event*)e;
  if (ev->graph) return hipErrorCapturedEvent;
  return !ev->recorded || ev->done ? hipSuccess : hipErrorNotReady;
}
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 0; return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
  if (((Event*)e)->graph) ((Stream*)s)->graph = ((Event*)e)->graph;
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t) { return hipErrorUnknown; }
}

// ------------------------------------------------------------------------------------------ the launchers' stand-ins
namespace spd {
static hipError_t launch(hipStream_t s, const StepMark& m, std::function<void()> f = [] {}) {
  if (n_launches++ == fail_launch) return hipErrorLaunchFailure;
  put(s, [m, f] {
    if (m.flag) *m.flag = m.seq;
    f();
  });
  return hipSuccess;
}
hipError_t launch_kv_write(const PoolGeom&, char*, const TileDesc*, int, const void*, const void*, const StepMark& m, hipStream_t s, void*,
                           const void*, uint64_t) { return launch(s, m); }
bool kv_rows_supported(const PoolGeom& g) { return g.kind == SPD_KV_GQA && g.Hkv >= 2; }
hipError_t launch_kv_rows(const PoolGeom&, char*, const TileDesc*, int, const void*, const void*, const KvRows& x, const StepMark& m, hipStream_t s) {
  staged_bytes = x.copy_bytes;
  seen_cus.push_back(x.cus);
  return launch(s, m);
}
hipError_t launch_kv_gather(const PoolGeom&, const char*, const TileDesc*, int, void*, void*, const StepMark& m, hipStream_t s) { return launch(s, m); }
hipError_t launch_kv_write_fp8(const PoolGeom&, char*, const TileDesc*, int, const void*, const StepMark& m, hipStream_t s, void*, const void*,
                               uint64_t) { return launch(s, m); }
hipError_t launch_kv_gather_fp8(const PoolGeom&, const char*, const TileDesc*, int, void*, const StepMark& m, hipStream_t s) { return launch(s, m); }
hipError_t launch_meta_copy(void* dst, const void* src, uint64_t bytes, const StepMark& m, hipStream_t s) {
  return launch(s, m, [=] { memcpy(dst, src, bytes); });
}
hipError_t launch_decode_gqa(const PoolGeom&, char*, const DecodeLaunch& d, hipStream_t s) {
  seen_counters.push_back(d.counters != nullptr);
  return launch(s, d.mark, [d] {
    double sum = 0;
    for (int i = 0; i < d.rot / 2; ++i) sum += d.w[i];
    seen_w.push_back(sum);
  });
}
hipError_t launch_decode_prepare(const PoolGeom&, char*, const DecodeLaunch& d, int, void*, hipStream_t s) { return launch(s, d.mark); }
hipError_t launch_decode_mla(const PoolGeom& g, char* b, const DecodeLaunch& d, hipStream_t s) { return launch_decode_gqa(g, b, d, s); }
hipError_t launch_prefill(const void*, const void* k, const void*, void*, const PrefillLists& d, bool, int, int, int, int, float, hipStream_t s) {
  seen_lists.push_back(d);
  seen_keys.push_back(d.pages ? nullptr : k);
  return launch(s, StepMark{});
}
hipError_t launch_rope(void*, int, void*, int, int, int, int, bool, int, const int32_t*, const double*, const StepMark& m, hipStream_t s) { return launch(s, m); }
hipError_t launch_probe(int32_t*, int, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_copy(void*, const void*, uint64_t, int, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_read(const void*, uint64_t, int, uint32_t*, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_read_lds(const void*, uint64_t, int, uint32_t*, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_clock_probe(uint64_t, uint64_t*, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_issue_probe(uint64_t*, hipStream_t) { return hipErrorUnknown; }
bool prefill_shape_supported(int dqk, int dv) { return dqk == dv; }
int prefill_heads_per_block(int group) { return group; }
int prefill_block_m(int) { return 128; }
int scratch_resolve(int, char** out) {
  *out = (char*)aligned_alloc(4096, SCRATCH_BYTES);
  return SPD_OK;
}
}  // namespace spd

// ------------------------------------------------------------------------------------------ what the scenarios share
static spd_ctx* ctx;
static spd_pool* pool;
alignas(16) static char tensor[1 << 16];

static spd_rope_config rope(double theta) { return spd_rope_config{theta, 1.0, 1.0, 4.0, 8192, 128, 0, 0}; }

static void setup() {
  CHECK(spd_ctx_create(0, &ctx) == SPD_OK);
  const spd_pool_desc desc = {SPD_KV_GQA, 16, 2, 128, 128, 64};
  uint64_t bytes;
  CHECK(spd_pool_bytes(&desc, &bytes) == SPD_OK);
  CHECK(spd_pool_create(ctx, aligned_alloc(4096, bytes), bytes, &desc, &pool) == SPD_OK);
  for (uint64_t r = 1; r <= 4; ++r) CHECK(spd_kv_reserve(pool, r, 40, nullptr) == SPD_OK);
}
static Stream* decode_stream() { return (Stream*)ctx->phase[SPD_PHASE_DECODE].stream; }

static int decode(uint64_t req, const spd_rope_config* r = nullptr, bool noalloc = false) {
  const int32_t len = 40;
  const spd_decode_batch b = {1, &req, &len, tensor, nullptr, nullptr, tensor, 8, 0.1f, r};
  return noalloc ? spd_decode_step_noalloc(ctx, pool, &b) : spd_decode_step(ctx, pool, &b);
}

// A pool of its own with requests that have `n_tokens` cached tokens, and the prefill step of the next five of each: two items a request, whose
// keys are shared out.
static spd_pool* long_pool(uint64_t req, int32_t n_tokens, int n_req = 1) {
  spd_pool* p;
  uint64_t bytes;
  const spd_pool_desc desc = {SPD_KV_GQA, 16, 2, 128, 128, ((n_tokens + 5) / 16 + 1) * n_req};
  CHECK(spd_pool_bytes(&desc, &bytes) == SPD_OK);
  CHECK(spd_pool_create(ctx, aligned_alloc(4096, bytes), bytes, &desc, &p) == SPD_OK);
  for (int r = 0; r < n_req; ++r) CHECK(spd_kv_reserve(p, req + (uint64_t)r, n_tokens, nullptr) == SPD_OK);
  return p;
}
static int prefill(spd_pool* p, uint64_t req, int32_t n_cached, int n_req = 1) {
  std::vector<uint64_t> ids;
  std::vector<int32_t> cu(1, 0), cached((size_t)n_req, n_cached);
  for (int r = 0; r < n_req; ++r) {
    ids.push_back(req + (uint64_t)r);
    cu.push_back(cu.back() + 5);
  }
  const spd_prefill_batch b = {n_req, ids.data(), cu.data(), tensor, tensor, tensor, nullptr, tensor, 8, 2, 128, 128, 0.1f, cached.data(), nullptr};
  return spd_prefill_step(ctx, p, &b);
}

static double sum_w(const spd_rope_config& c) {
  double w[64], sum = 0;
  CHECK(spd_rope_inv_freq(&c, w, 64) == SPD_OK);
  for (double x : w) sum += x;
  return sum;
}

// ------------------------------------------------------------------------------------------ scenarios
// A page write or gather that is refused allocates nothing, however many tokens it names.
static void refused_copies() {
  spd_ctx* c = ctx;
  const int P = SPD_PHASE_PREFILL;
  const long pinned = n_pinned;
  for (const int32_t n : {INT32_MAX, INT32_MAX - 7, 100000000, 49}) {
    CHECK(spd_kv_write(c, pool, P, 1, 0, n, tensor, tensor) == SPD_EINVAL);       // longer than the request's pages
    CHECK(spd_kv_write(c, pool, P, 1, 8, n, tensor, tensor) == SPD_EINVAL);
    CHECK(spd_kv_gather(c, pool, P, 1, n, tensor, tensor) == SPD_EINVAL);
    CHECK(spd_kv_write(c, pool, P, 99, 0, n, tensor, tensor) == SPD_ENOENT);
    CHECK(spd_kv_gather(c, pool, P, 99, n, tensor, tensor) == SPD_ENOENT);
  }
  CHECK(n_pinned == pinned && n_launches == 0);
  CHECK(spd_kv_write(c, pool, P, 1, 8, 40, tensor, tensor) == SPD_OK && n_launches == 1);
}

// A step whose attention launch fails: its staging slot, which the launch before it reads, stays untouched until that has run,
// the frequency table that was on its way is not taken for granted, and nothing of it keeps its request's pages.
static void failed_launch() {
  const spd_rope_config a = rope(10000.0), b = rope(500000.0);
  CHECK(decode(1, &a) == SPD_OK);
  run(decode_stream());
  fail_launch = n_launches + 1;                      // the frequencies' copy goes out, the attention does not
  CHECK(decode(2, &b) == SPD_EHIP);
  CHECK(spd_kv_write(ctx, pool, SPD_PHASE_DECODE, 3, 0, 40, tensor, tensor) == SPD_OK);      // the next user of a slot
  CHECK(decode(4, &b) == SPD_OK);
  CHECK(decode(1, &a) == SPD_OK);
  fail_launch = n_launches;                          // nothing goes out
  CHECK(decode(2, &b) == SPD_EHIP);
  CHECK(decode(4, &b) == SPD_OK);
  run(decode_stream());
  CHECK(seen_w.size() == 4 && seen_w[0] == sum_w(a) && seen_w[1] == sum_w(b) && seen_w[2] == sum_w(a) && seen_w[3] == sum_w(b));
  for (uint64_t r = 1; r <= 4; ++r) CHECK(spd_kv_free(pool, r, nullptr) == SPD_OK);
}

// The step that allocates nothing, under graph capture on the phase's stream, which the caller has asked for: a replay reads what
// the captured call was given, whatever steps and configurations have come in between, and reports no step's end.
static void captured() {
  const spd_rope_config a = rope(10000.0), b = rope(500000.0), c = rope(20000.0);
  spd_phase_state& ps = ctx->phase[SPD_PHASE_DECODE];
  void* handle;
  CHECK(spd_phase_stream(ctx, SPD_PHASE_DECODE, &handle) == SPD_OK && handle == decode_stream());
  std::vector<std::function<void()>> graph, graph2;
  auto capture = [&](std::vector<std::function<void()>>* g, const spd_rope_config* r) -> int {
    decode_stream()->graph = g;
    const int rc = decode(2, r, true);
    decode_stream()->graph = nullptr;
    return rc;
  };
  auto last = [&](const spd_rope_config& r) { run(decode_stream()); return seen_w.back() == sum_w(r); };
  CHECK(decode(1, &a) == SPD_OK && last(a));
  CHECK(capture(&graph, &b) == SPD_OK);              // the first call with this configuration: nothing has run yet
  CHECK(decode(3, &b) == SPD_OK && last(b));
  CHECK(capture(&graph2, &b) == SPD_OK);             // and one whose frequencies are on the device
  for (int round = 0; round < 3; ++round) {
    for (int i = 0; i < 20; ++i) CHECK(decode(4, i % 2 ? &a : &c) == SPD_OK);
    CHECK(last(a));
    const uint64_t flag = *ps.flag;
    for (auto* g : {&graph, &graph2}) {
      for (auto& node : *g) put((hipStream_t)decode_stream(), node);
      CHECK(last(b));
    }
    CHECK(*ps.flag == flag);
  }
  // as many captured calls as there are staging slots; then steps that may allocate go on, the others are refused
  int more = 0, rc;
  std::vector<std::function<void()>> rest;
  while ((rc = capture(&rest, &a)) == SPD_OK) CHECK(++more < STAGE_SLOTS);
  CHECK(rc == SPD_ESTATE && more + 2 == STAGE_SLOTS);
  for (int i = 0; i < 20; ++i) CHECK(decode(4, &c) == SPD_OK && last(c));
  CHECK(decode(4, &c, true) == SPD_OK);              // (the slots that the steps in between have brought)
  for (auto& node : graph) put((hipStream_t)decode_stream(), node);
  CHECK(last(b));
  for (uint64_t r = 1; r <= 4; ++r) CHECK(spd_kv_free(pool, r, nullptr) == SPD_OK);
}

// A call blocks while four steps of its phase are in flight: what has been issued runs on the share of its time, and a new
// partition waits for no more than that.
static void in_flight() {
  for (int i = 0; i < 4; ++i) {
    CHECK(decode(1) == SPD_OK);
    CHECK((int)decode_stream()->queue.size() == i + 1);
  }
  for (int i = 0; i < 20; ++i) {
    CHECK(decode(1) == SPD_OK);
    CHECK(decode_stream()->queue.size() <= 4);       // (the wait lets the stream go on)
  }
}

// A few chunks of a GQA launch are merged by the launch, those of a latent one (16 heads, one merging workgroup per request) never.
static void merges() {
  const spd_pool_desc desc = {SPD_KV_MLA_LATENT, 64, 1, 576, 512, 64};
  spd_pool* latent;
  uint64_t bytes, req = 9;
  CHECK(spd_pool_bytes(&desc, &bytes) == SPD_OK);
  CHECK(spd_pool_create(ctx, aligned_alloc(4096, bytes), bytes, &desc, &latent) == SPD_OK);
  CHECK(spd_kv_reserve(latent, req, 4000, nullptr) == SPD_OK && spd_kv_reserve(pool, req, 700, nullptr) == SPD_OK);
  for (const int32_t n : {100, 600, 1500, 4000}) {
    const spd_decode_batch b = {1, &req, &n, tensor, nullptr, nullptr, tensor, 16, 0.1f, nullptr};
    CHECK(spd_decode_step(ctx, latent, &b) == SPD_OK && !seen_counters.back());
    CHECK(spd_decode_step_noalloc(ctx, latent, &b) == SPD_OK && !seen_counters.back());
  }
  const int32_t n = 700;
  const spd_decode_batch b = {1, &req, &n, tensor, nullptr, nullptr, tensor, 16, 0.1f, nullptr};
  CHECK(spd_decode_step(ctx, pool, &b) == SPD_OK && seen_counters.back());
}

// One launch where a compute unit has few workgroups; records copied, rows prepared and attention where it has many with short
// contexts; without the preparation where the contexts are long or there is nothing to prepare.
static void launches() {
  const spd_rope_config r = rope(10000.0);
  uint64_t req = 9;
  CHECK(spd_kv_reserve(pool, req, 800, nullptr) == SPD_OK);
  auto count = [&](int B, int32_t n, const spd_rope_config* rp, bool noalloc = false) -> int {
    std::vector<uint64_t> ids((size_t)B, req);
    std::vector<int32_t> lens((size_t)B, n);
    const spd_decode_batch b = {B, ids.data(), lens.data(), tensor, nullptr, nullptr, tensor, 8, 0.1f, rp};
    run(decode_stream());
    const int before = n_launches;
    CHECK((noalloc ? spd_decode_step_noalloc(ctx, pool, &b) : spd_decode_step(ctx, pool, &b)) == SPD_OK);
    run(decode_stream());
    return n_launches - before;
  };
  CHECK(count(1, 30, &r) == 2);                      // (the frequency table's copy)
  for (bool noalloc : {false, true}) {
    CHECK(count(1, 30, &r, noalloc) == 1 && count(380, 30, &r, noalloc) == 1);     // two KV heads, 256 compute units: 760 workgroups
    CHECK(count(390, 30, &r, noalloc) == 3);
    CHECK(count(390, 30, nullptr, noalloc) == 2);    // nothing to rotate or append
    CHECK(count(800, 800, &r, noalloc) == 2);
  }
}

// Under graph capture a prefill step takes whole items: the launches would outlive the buffer of the parts' sums.  Also where the step adopts
// a staged partition, whose stream joins the capture only then.
static void captured_prefill() {
  spd_pool* p = long_pool(9, 3000);
  CHECK(prefill(p, 9, 3000) == SPD_OK && seen_lists.back().n_merge == 2 && seen_lists.back().parts);
  void* handle;
  CHECK(spd_phase_stream(ctx, SPD_PHASE_PREFILL, &handle) == SPD_OK);
  run((Stream*)handle);
  std::vector<std::function<void()>> graph;
  auto whole = [] { return seen_lists.back().n_merge == 0 && !seen_lists.back().parts; };
  ((Stream*)handle)->graph = &graph;
  CHECK(prefill(p, 9, 3000) == SPD_OK && whole());
  CHECK(spd_set_partition(ctx, 128, 128) == SPD_OK);
  CHECK(prefill(p, 9, 3000) == SPD_OK && whole());
  Stream* staged = (Stream*)ctx->phase[SPD_PHASE_PREFILL].stream;
  CHECK(staged != handle && staged->graph == &graph);
  staged->graph = ((Stream*)handle)->graph = nullptr;
  CHECK(prefill(p, 9, 3000) == SPD_OK && seen_lists.back().n_merge == 2 && seen_lists.back().parts);
}

// The buffer of the parts' sums: where there is no memory for it the step takes whole items; one that is outgrown stays until the steps
// that were given it have finished.
static void parts() {
  spd_pool *p = long_pool(9, 3000), *many = long_pool(20, 6000, 8);
  CHECK(prefill(p, 9, 3000) == SPD_OK && seen_lists.back().n_merge == 2);
  char* const first = (char*)seen_lists.back().parts;
  CHECK(first && first == ctx->phase[SPD_PHASE_PREFILL].parts);
  fail_malloc = true;
  CHECK(prefill(many, 20, 6000, 8) == SPD_OK && !fail_malloc && spd_last_hip_error() == 0);
  CHECK(seen_lists.back().n_merge == 0 && !seen_lists.back().parts);
  CHECK(prefill(many, 20, 6000, 8) == SPD_OK && seen_lists.back().n_merge == 16);
  char* const second = (char*)seen_lists.back().parts;
  CHECK(second && second != first);
  CHECK(prefill(p, 9, 3000) == SPD_OK && (char*)seen_lists.back().parts == second);
  CHECK(!freed.count(first));                        // the first step has not run yet
  CHECK(spd_phase_sync(ctx, SPD_PHASE_PREFILL) == SPD_OK);
  CHECK(freed.count(first) && !freed.count(second));
}

// Long pieces behind few cached tokens have their keys as dense rows: not where there is no memory for them, nor under capture; a buffer that
// is outgrown stays until the steps that were given it have finished.  Short ones behind many read the pages.
static void dense_rows() {
  spd_pool *few = long_pool(9, 40), *more = long_pool(20, 40, 32), *many = long_pool(9, 3000);
  spd_phase_state& ps = ctx->phase[SPD_PHASE_PREFILL];
  CHECK(prefill(many, 9, 3000) == SPD_OK && !seen_keys.back() && seen_lists.back().units && !ps.rows);
  void* handle;
  CHECK(spd_phase_stream(ctx, SPD_PHASE_PREFILL, &handle) == SPD_OK);
  std::vector<std::function<void()>> graph;
  run((Stream*)handle);
  ((Stream*)handle)->graph = &graph;
  CHECK(prefill(few, 9, 40) == SPD_OK && !seen_keys.back() && !ps.rows);
  ((Stream*)handle)->graph = nullptr;
  fail_malloc = true;
  CHECK(prefill(few, 9, 40) == SPD_OK && !fail_malloc && spd_last_hip_error() == 0 && !seen_keys.back() && !ps.rows);
  CHECK(prefill(few, 9, 40) == SPD_OK && seen_keys.back() && seen_keys.back() == ps.rows);
  char* const first = ps.rows;
  ps.rows_cap = 1 << 10;                             // (as if it were a small one)
  CHECK(prefill(more, 20, 40, 32) == SPD_OK && seen_keys.back() == ps.rows && ps.rows != first);
  CHECK(!freed.count(first));
  CHECK(spd_phase_sync(ctx, SPD_PHASE_PREFILL) == SPD_OK);
  CHECK(freed.count(first) && !freed.count(ps.rows));
}

// Lists cross the host link ahead of the attention: a step of whole items stages 24 bytes for each, and no ranges of keys.
static void staged() {
  constexpr int N = 64;
  spd_pool* p = long_pool(100, 1, N);
  CHECK(prefill(p, 100, 0, N) == SPD_OK && seen_lists.back().n_merge == 0 && !seen_lists.back().range);
  const uint64_t items = 2 * N, chains = (uint64_t)seen_lists.back().n_blocks + 1;
  CHECK(staged_bytes >= items * 24 && staged_bytes < items * 24 + chains * 4 + N * sizeof(TileDesc) + 5 * 16);
}

// A page write is laid out for the compute units that it runs on: those of its phase's share, a staged one among them.
static void shares() {
  CHECK(spd_kv_write(ctx, pool, SPD_PHASE_DECODE, 1, 0, 40, tensor, tensor) == SPD_OK && seen_cus == std::vector<int>{256});
  CHECK(spd_set_partition(ctx, 192, 64) == SPD_OK);
  for (const int phase : {SPD_PHASE_PREFILL, SPD_PHASE_DECODE}) CHECK(spd_kv_write(ctx, pool, phase, 1, 0, 40, tensor, tensor) == SPD_OK);
  CHECK(prefill(long_pool(9, 40), 9, 40) == SPD_OK);
  CHECK(seen_cus == (std::vector<int>{256, 192, 64, 192}));
}

// Whatever GPU the calling thread's last call was for, a step's buffers lie on the context's own.
static void devices() {
  spd_pool* p = long_pool(9, 3000);
  allocated_on.clear();
  const long pinned = n_pinned, before = n_device;
  CHECK(hipSetDevice(1) == hipSuccess);
  CHECK(prefill(p, 9, 3000) == SPD_OK && seen_lists.back().n_merge == 2 && seen_lists.back().parts);
  CHECK(n_pinned > pinned && n_device == before + 2);      // the staging slot; the workspace and the parts' sums
  CHECK(hipSetDevice(1) == hipSuccess);
  CHECK(spd_kv_write(ctx, p, SPD_PHASE_DECODE, 9, 0, 3000, tensor, tensor) == SPD_OK);
  CHECK(allocated_on == std::set<int>{0});
}

int main(int argc, char** argv) {
  CHECK(argc == 2);
  const std::string name = argv[1];
  setup();
  if (name == "refused_copies") refused_copies();
  else if (name == "failed_launch") failed_launch();
  else if (name == "captured") captured();
  else if (name == "in_flight") in_flight();
  else if (name == "merges") merges();
  else if (name == "launches") launches();
  else if (name == "captured_prefill") captured_prefill();
  else if (name == "parts") parts();
  else if (name == "staged") staged();
  else if (name == "devices") devices();
  else if (name == "shares") shares();
  else if (name == "dense_rows") dense_rows();
  else CHECK(!"a scenario of that name");
  puts("ok");
}
