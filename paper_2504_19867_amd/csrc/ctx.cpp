// Context, CU partition controller, per-phase streams, staging buffers.
//
// Paper, "Computational Resource Controller": the (x, y) split is realised with MPS and can
// only change by replacing the worker processes; the cost is hidden by (1) keeping weights and
// KV cache in a resident owner, (2) preparing the new workers first and switching late, and
// (3) letting each worker switch at its own iteration boundary.  On this GPU a stream's CU
// mask is likewise fixed at creation, so the same three ideas apply to streams: the pool is
// owned outside any stream, spd_set_partition prepares (or re-uses) the new masked streams and
// only stages them, and each phase adopts its staged stream at its next step entry.
#include "internal.h"

#include <string.h>

#include <algorithm>
#include <new>
#include <chrono>
#include <set>
#include <thread>

using namespace spd;

static int round_cus(int x, int gran, int total) {
  if (x < gran) x = gran;
  int r = (x + gran / 2) / gran * gran;
  if (r > total) r = total / gran * gran;
  if (r < gran) r = gran;
  return r;
}

extern "C" int spd_partition_masks(int total_cus, int granularity, int prefill_cus, int decode_cus,
                                   uint32_t* prefill_words, uint32_t* decode_words, int* p_out, int* d_out) {
  if (total_cus <= 0 || granularity <= 0 || total_cus % granularity != 0 || total_cus > 1024) return SPD_EINVAL;
  if (prefill_cus <= 0 || decode_cus <= 0 || !prefill_words || !decode_words) return SPD_EINVAL;
  int p = round_cus(prefill_cus, granularity, total_cus);
  int d = round_cus(decode_cus, granularity, total_cus);
  // a request for disjoint shares stays disjoint after the rounding
  if ((int64_t)prefill_cus + decode_cus <= total_cus && p + d > total_cus) {
    if (p > total_cus - granularity) p = total_cus - granularity;
    d = total_cus - p;
  }
  int words = (total_cus + 31) / 32;
  memset(prefill_words, 0, sizeof(uint32_t) * words);
  memset(decode_words, 0, sizeof(uint32_t) * words);
  for (int i = 0; i < p; ++i) prefill_words[i / 32] |= 1u << (i % 32);
  for (int i = total_cus - d; i < total_cus; ++i) decode_words[i / 32] |= 1u << (i % 32);
  if (p_out) *p_out = p;
  if (d_out) *d_out = d;
  return SPD_OK;
}

static int get_masked_stream(spd_ctx* ctx, int phase, const std::vector<uint32_t>& mask, hipStream_t* out) {
  std::vector<uint32_t> key = mask;
  key.push_back((uint32_t)phase);   // the two phases never share a stream, even with equal masks
  auto it = ctx->stream_cache.find(key);
  if (it != ctx->stream_cache.end()) { *out = it->second; return SPD_OK; }
  hipStream_t s = nullptr;
  SPD_HIP(hipExtStreamCreateWithCUMask(&s, (uint32_t)mask.size(), mask.data()));
  ctx->stream_cache[key] = s;
  *out = s;
  return SPD_OK;
}

static int stage_alloc(spd_stage* st, size_t cap) {
  char *h = nullptr, *d = nullptr;
  SPD_HIP(hipHostMalloc((void**)&h, cap, hipHostMallocDefault));
  hipError_t e = hipHostGetDevicePointer((void**)&d, h, 0);
  if (e != hipSuccess) { (void)hipHostFree(h); return hip_fail(e); }
  if (st->host) (void)hipHostFree(st->host);
  st->host = h; st->dev = d; st->cap = cap;
  return SPD_OK;
}

extern "C" int spd_ctx_create(int device, spd_ctx** out) {
  if (!out || device < -1) return SPD_EINVAL;
  spd_ctx* c = new (std::nothrow) spd_ctx();
  if (!c) return SPD_EINVAL;
  c->device = device;
  // the two measurement overrides are read here, once: the steps never touch the environment
  if (const char* env = getenv("SPD_PREFILL_PERSISTENT")) c->env_prefill_persistent = atoi(env) != 0;
  if (const char* env = getenv("SPD_DECODE_CHUNK_TILES")) c->env_decode_chunk_tiles = std::max(0, atoi(env));
  if (device >= 0) {
    hipDeviceProp_t prop;
    hipError_t e = hipGetDeviceProperties(&prop, device);
    if (e != hipSuccess) { delete c; return hip_fail(e); }
    if (strncmp(prop.gcnArchName, "gfx950", 6) != 0) { delete c; return SPD_ESTATE; }
    c->total_cus = prop.multiProcessorCount;
    c->xcds = 8;
    if (c->total_cus % c->xcds != 0) c->xcds = 1;
    // An XCD hands its workgroups to its four shader arrays in turn, whatever each array has left of
    // the mask, so a share is only as fast as four times its smallest per-array count (measured: 64, 72
    // and 80 compute units give the same prefill time, 96 and 112 too): whole rows of one compute
    // unit per shader array and XCD.
    c->granularity = c->xcds * 4;
    if (c->total_cus % c->granularity != 0) c->granularity = c->xcds;
    e = hipSetDevice(device);
    if (e != hipSuccess) { delete c; return hip_fail(e); }
  }
  int words = (c->total_cus + 31) / 32;
  std::vector<uint32_t> full(words, 0);
  for (int i = 0; i < c->total_cus; ++i) full[i / 32] |= 1u << (i % 32);
  for (int ph = 0; ph < 2; ++ph) {
    spd_phase_state& s = c->phase[ph];
    s.active_cus = s.pending_cus = c->total_cus;
    s.active_mask = s.pending_mask = full;
    if (device >= 0) {
      int rc = get_masked_stream(c, ph, full, &s.stream);
      hipError_t e = hipSuccess;
      if (rc == SPD_OK) e = hipEventCreate(&s.ev_start);
      if (rc == SPD_OK && e == hipSuccess) e = hipEventCreate(&s.ev_end);
      if (rc == SPD_OK && e == hipSuccess) e = hipEventCreateWithFlags(&s.ev_switch, hipEventDisableTiming);
      if (rc == SPD_OK && e == hipSuccess) e = hipEventCreateWithFlags(&s.ev_cross, hipEventDisableTiming);
      for (spd_seal& seal : s.seals)
        if (rc == SPD_OK && e == hipSuccess) e = hipEventCreateWithFlags(&seal.ev, hipEventDisableTiming);
      if (rc == SPD_OK && e == hipSuccess) e = hipHostMalloc((void**)&s.flag, sizeof(uint64_t), hipHostMallocDefault);
      if (rc == SPD_OK && e == hipSuccess) {
        *s.flag = 0;
        e = hipHostGetDevicePointer((void**)&s.flag_dev, s.flag, 0);
      }
      if (rc == SPD_OK && e == hipSuccess) e = hipMalloc((void**)&s.rope_dev, sizeof(double) * ROPE_TABLE_DIM / 2);
      if (rc == SPD_OK && e == hipSuccess && ph == SPD_PHASE_DECODE) {
        e = hipMalloc((void**)&s.merge_counters, sizeof(uint32_t) * MERGE_COUNTERS);
        if (e == hipSuccess) e = hipMemset(s.merge_counters, 0, sizeof(uint32_t) * MERGE_COUNTERS);
        if (e == hipSuccess) e = hipDeviceSynchronize();
      }
      // The decode phase's staging ring exists from the start, with room for everything the entry point that
      // allocates nothing takes.
      if (rc == SPD_OK && e == hipSuccess && ph == SPD_PHASE_DECODE) {
        rc = scratch_resolve(device, &c->scratch);
        for (spd_stage& st : s.ring)
          if (rc == SPD_OK) rc = stage_alloc(&st, NOALLOC_RING_BYTES);
      }
      if (rc != SPD_OK || e != hipSuccess) {
        if (e != hipSuccess) hip_fail(e);
        spd_ctx_destroy(c);
        return rc != SPD_OK && rc != SPD_EHIP ? rc : SPD_EHIP;
      }
    }
  }
  *out = c;
  return SPD_OK;
}

extern "C" int spd_ctx_destroy(spd_ctx* ctx) {
  if (!ctx) return SPD_EINVAL;
  if (ctx->device >= 0) {
    (void)hipSetDevice(ctx->device);
    for (auto& kv : ctx->stream_cache) (void)hipStreamSynchronize(kv.second);
    for (int ph = 0; ph < 2; ++ph) {
      spd_phase_state& s = ctx->phase[ph];
      for (spd_stage& st : s.ring)
        if (st.host) (void)hipHostFree(st.host);
      for (char* h : s.kept) (void)hipHostFree(h);
      for (spd_seal& seal : s.seals)
        if (seal.ev) (void)hipEventDestroy(seal.ev);
      if (s.flag) (void)hipHostFree(s.flag);
      if (s.rope_dev) (void)hipFree(s.rope_dev);
      if (s.merge_counters) (void)hipFree(s.merge_counters);
      if (s.workspace) (void)hipFree(s.workspace);
      if (s.parts) (void)hipFree(s.parts);
      if (s.rows) (void)hipFree(s.rows);
      for (auto& r : s.ws_retired) (void)hipFree(r.first);
      for (hipEvent_t e : {s.ev_start, s.ev_end, s.ev_switch, s.ev_cross})
        if (e) (void)hipEventDestroy(e);
      for (auto& pair : s.kev)
        for (hipEvent_t e : pair)
          if (e) (void)hipEventDestroy(e);
    }
    for (auto& kv : ctx->stream_cache) (void)hipStreamDestroy(kv.second);
  }
  delete ctx;
  return SPD_OK;
}

extern "C" int spd_device_info(spd_ctx* ctx, int* total_cus, int* xcds, int* cu_granularity) {
  if (!ctx) return SPD_EINVAL;
  if (total_cus) *total_cus = ctx->total_cus;
  if (xcds) *xcds = ctx->xcds;
  if (cu_granularity) *cu_granularity = ctx->granularity;
  return SPD_OK;
}

extern "C" int spd_set_partition(spd_ctx* ctx, int prefill_cus, int decode_cus) {
  if (!ctx) return SPD_EINVAL;
  int words = (ctx->total_cus + 31) / 32;
  std::vector<uint32_t> pm(words), dm(words);
  int p = 0, d = 0;
  int rc = spd_partition_masks(ctx->total_cus, ctx->granularity, prefill_cus, decode_cus, pm.data(), dm.data(), &p, &d);
  if (rc != SPD_OK) return rc;
  std::lock_guard<std::mutex> lk(ctx->part_mu);
  hipStream_t ps = nullptr, ds = nullptr;
  if (ctx->device >= 0) {
    (void)hipSetDevice(ctx->device);
    // preparation: both streams exist before anything is staged, so a failure changes nothing
    if ((rc = get_masked_stream(ctx, SPD_PHASE_PREFILL, pm, &ps)) != SPD_OK) return rc;
    if ((rc = get_masked_stream(ctx, SPD_PHASE_DECODE, dm, &ds)) != SPD_OK) return rc;
  }
  spd_phase_state& P = ctx->phase[SPD_PHASE_PREFILL];
  spd_phase_state& D = ctx->phase[SPD_PHASE_DECODE];
  P.pending_stream = ps; P.pending_cus = p; P.pending_mask = pm; P.has_pending = true;
  D.pending_stream = ds; D.pending_cus = d; D.pending_mask = dm; D.has_pending = true;
  return SPD_OK;
}

extern "C" int spd_get_partition(spd_ctx* ctx, int* prefill_active, int* decode_active, int* prefill_pending,
                                 int* decode_pending) {
  if (!ctx) return SPD_EINVAL;
  std::lock_guard<std::mutex> lk(ctx->part_mu);
  if (prefill_active) *prefill_active = ctx->phase[0].active_cus;
  if (decode_active) *decode_active = ctx->phase[1].active_cus;
  if (prefill_pending) *prefill_pending = ctx->phase[0].has_pending ? ctx->phase[0].pending_cus : ctx->phase[0].active_cus;
  if (decode_pending) *decode_pending = ctx->phase[1].has_pending ? ctx->phase[1].pending_cus : ctx->phase[1].active_cus;
  return SPD_OK;
}

extern "C" int spd_phase_cu_mask(spd_ctx* ctx, int phase, uint32_t* words, int32_t cap, int32_t* n_words) {
  if (!ctx || phase < 0 || phase > 1 || !n_words || cap < 0 || (cap > 0 && !words)) return SPD_EINVAL;
  std::lock_guard<std::mutex> lk(ctx->part_mu);
  const std::vector<uint32_t>& m = ctx->phase[phase].active_mask;
  *n_words = (int32_t)m.size();
  if ((size_t)cap < m.size()) return SPD_EINVAL;
  memcpy(words, m.data(), m.size() * sizeof(uint32_t));
  return SPD_OK;
}

namespace spd {

// Step entry of one phase: adopt the staged partition, if any (asynchronous switching: the
// other phase is not consulted).  The new stream first waits, on the GPU, for the old
// stream's last work, so that the phase's own steps stay ordered across the switch.
int phase_enter(spd_ctx* ctx, int phase, hipStream_t* stream_out) {
  if (ctx->device < 0) return SPD_ESTATE;
  SPD_HIP(hipSetDevice(ctx->device));
  std::lock_guard<std::mutex> lk(ctx->part_mu);
  spd_phase_state& s = ctx->phase[phase];
  if (s.has_pending) {
    if (s.pending_stream != s.stream) {
      int rc = phase_seal(ctx, phase, s.stream);
      if (rc != SPD_OK) return rc;
      SPD_HIP(hipEventRecord(s.ev_switch, s.stream));
      SPD_HIP(hipStreamWaitEvent(s.pending_stream, s.ev_switch, 0));
      s.stream = s.pending_stream;
    }
    s.active_cus = s.pending_cus;
    s.active_mask = s.pending_mask;
    s.has_pending = false;
  }
  *stream_out = s.stream;
  return SPD_OK;
}

// One workgroup per compute unit gets one compute unit each only where every XCD contributes a multiple of 4 of them: an XCD deals
// its workgroups to its four shader arrays in turn (the partition granularity sees to that; with 10 per XCD some workgroups
// wait for others to finish, and a prefill step takes up to twice as long).  And not where the two phases' masks overlap: such a
// workgroup keeps its compute unit for the whole kernel, and the other phase's workgroups that are allowed nowhere else would
// wait that long.
bool phase_exclusive(spd_ctx* ctx, int phase, int* share) {
  std::lock_guard<std::mutex> lk(ctx->part_mu);
  const spd_phase_state &s = ctx->phase[phase], &o = ctx->phase[1 - phase];
  *share = std::max(1, s.has_pending ? s.pending_cus : s.active_cus);
  if (*share % ctx->xcds != 0 || (*share / ctx->xcds) % 4 != 0) return false;
  const std::vector<uint32_t>& m = s.has_pending ? s.pending_mask : s.active_mask;
  auto meets = [&](const std::vector<uint32_t>& other) {
    for (size_t i = 0; i < m.size() && i < other.size(); ++i)
      if (m[i] & other[i]) return true;
    return false;
  };
  return !meets(o.active_mask) && !(o.has_pending && meets(o.pending_mask));
}

static void raise_done_seq(spd_phase_state& s, uint64_t seq) {
  uint64_t cur = s.done_seq.load(std::memory_order_relaxed);
  while (cur < seq && !s.done_seq.compare_exchange_weak(cur, seq, std::memory_order_release)) {
  }
}

// Has step `seq` finished, as far as the phase's word in pinned memory says?  No runtime call.
static bool flag_says_done(spd_phase_state& s, uint64_t seq) {
  if (s.done_seq.load(std::memory_order_acquire) >= seq) return true;
  const uint64_t f = __atomic_load_n(s.flag, __ATOMIC_ACQUIRE);
  if (f < seq) return false;
  raise_done_seq(s, f);
  return true;
}

bool stream_capturing(spd_ctx* ctx, hipStream_t stream) {
  if (!ctx->phase[0].stream_lent.load(std::memory_order_relaxed) && !ctx->phase[1].stream_lent.load(std::memory_order_relaxed)) return false;
  hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
  return hipStreamIsCapturing(stream, &status) == hipSuccess && status == hipStreamCaptureStatusActive;
}

int stage_acquire(spd_ctx* ctx, int phase, size_t bytes, spd_stage** out, bool may_alloc) {
  spd_phase_state& s = ctx->phase[phase];
  for (int i = 0; i < STAGE_SLOTS && s.ring[s.ring_pos].captured; ++i) s.ring_pos = (s.ring_pos + 1) % STAGE_SLOTS;
  spd_stage& st = s.ring[s.ring_pos];
  if (st.captured) {                                     // all of them
    if (!may_alloc) return SPD_ESTATE;
    s.kept.push_back(st.host);
    st = spd_stage();
  }
  // The slot's last step has to be over, and the one STEPS_IN_FLIGHT steps back: what is queued still runs on the share it was
  // issued for, and a new partition is behind it.  The step after that one reports its end.  The word is polled, first in a
  // spin, then with pauses; the runtime is asked now and then only, because its calls keep the other phase's thread
  // from launching (and to notice a device error).
  const uint64_t over = std::max(st.seq, s.recent[s.recent_pos]);
  for (int spins = 0; over && !flag_says_done(s, over); ++spins) {
    if (spins < 4096) {
      __builtin_ia32_pause();
      continue;
    }
    std::this_thread::sleep_for(std::chrono::microseconds(20));
    if (spins % 64 == 0 && stream_capturing(ctx, s.stream)) {
      (void)phase_step_done(ctx, phase, over);           // (asks the step's event: this stream may not be asked now)
    } else if (spins % 64 == 0) {
      const hipError_t e = hipStreamQuery(s.stream);
      if (e == hipSuccess) raise_done_seq(s, s.issue_seq.load(std::memory_order_relaxed));
      else if (e != hipErrorNotReady) return hip_fail(e);
    }
  }
  st.seq = 0;
  if (st.cap < bytes) {
    if (!may_alloc) return SPD_ETOOBIG;
    size_t cap = std::max<size_t>(256 * 1024, st.cap);
    while (cap < bytes) cap *= 2;
    SPD_HIP(hipSetDevice(ctx->device));                  // (the calling thread's last call may have been for another GPU)
    int rc = stage_alloc(&st, cap);
    if (rc != SPD_OK) return rc;
  }
  *out = &st;
  return SPD_OK;
}

int stage_commit(spd_ctx* ctx, int phase, spd_stage* st, hipStream_t stream, bool capturing) {
  spd_phase_state& s = ctx->phase[phase];
  st->captured = capturing;
  st->seq = s.issue_seq.fetch_add(1, std::memory_order_release) + 1;
  if (!capturing) {
    s.recent[s.recent_pos] = st->seq;
    s.recent_pos = (s.recent_pos + 1) % STEPS_IN_FLIGHT;
  }
  s.ring_pos = (s.ring_pos + 1) % STAGE_SLOTS;
  return !capturing && s.stream_lent.load(std::memory_order_relaxed) ? phase_seal(ctx, phase, stream) : SPD_OK;
}

StepMark step_mark(spd_ctx* ctx, int phase, bool capturing) {
  spd_phase_state& s = ctx->phase[phase];
  return StepMark{capturing ? nullptr : s.flag_dev, s.issue_seq.load(std::memory_order_relaxed)};
}

int phase_seal(spd_ctx* ctx, int phase, hipStream_t stream) {
  spd_phase_state& s = ctx->phase[phase];
  std::lock_guard<std::mutex> lk(s.seal_mu);            // spd_phase_stream may be asked from any thread
  const uint64_t seq = s.issue_seq.load(std::memory_order_acquire);
  if (seq == 0 || s.sealed_seq >= seq || flag_says_done(s, seq) || stream_capturing(ctx, stream)) return SPD_OK;
  spd_seal& seal = s.seals[s.seal_pos];
  SPD_HIP(hipEventRecord(seal.ev, stream));
  seal.seq.store(seq, std::memory_order_release);       // after the record
  s.seal_pos = (s.seal_pos + 1) % STAGE_SLOTS;
  s.sealed_seq = seq;
  return SPD_OK;
}

bool phase_step_done(spd_ctx* ctx, int phase, uint64_t seq) {
  if (seq == 0 || ctx->device < 0) return true;
  spd_phase_state& s = ctx->phase[phase];
  if (flag_says_done(s, seq)) return true;
  (void)hipSetDevice(ctx->device);
  // A seal whose number is `seq` or later carries an event recorded behind that step's last kernel (the number is
  // stored after the record, so reading it first means the event is at least that recent).
  for (spd_seal& seal : s.seals) {
    const uint64_t q = seal.seq.load(std::memory_order_acquire);
    if (q >= seq && hipEventQuery(seal.ev) == hipSuccess) {
      raise_done_seq(s, q);
      return true;
    }
  }
  // The last step of the phase has no later one to report it: it has finished if the stream is idle.
  // (The count is read before the stream: whichever stream is current after that waits for the one before it.)
  const uint64_t issued = s.issue_seq.load(std::memory_order_acquire);
  hipStream_t stream;
  { std::lock_guard<std::mutex> lk(ctx->part_mu); stream = s.stream; }
  if (issued >= seq && !stream_capturing(ctx, stream) && hipStreamQuery(stream) == hipSuccess) {
    raise_done_seq(s, issued);
    return true;
  }
  (void)hipGetLastError();      // hipErrorNotReady is not an error to keep
  return false;
}

static void workspace_release_retired(spd_ctx* ctx, int phase) {
  spd_phase_state& s = ctx->phase[phase];
  std::lock_guard<std::mutex> lk(s.ws_mu);
  size_t keep = 0;
  for (auto& r : s.ws_retired) {
    if (phase_step_done(ctx, phase, r.second)) (void)hipFree(r.first);
    else s.ws_retired[keep++] = r;
  }
  s.ws_retired.resize(keep);
}

// At least `bytes` of device memory in `buf`.
static int buffer_reserve(spd_ctx* ctx, int phase, size_t bytes, char*& buf, size_t& buf_cap) {
  spd_phase_state& s = ctx->phase[phase];
  if (buf_cap < bytes) {
    size_t cap = std::max<size_t>(16u << 20, buf_cap);
    while (cap < bytes) cap *= 2;
    char* d = nullptr;
    SPD_HIP(hipSetDevice(ctx->device));                  // (the calling thread's last call may have been for another GPU)
    SPD_HIP(hipMalloc((void**)&d, cap));
    // Earlier steps of this phase may still read the old buffer: it is kept until the last of them (the step
    // issued most recently; the one being built takes the new buffer) is known to have finished.  No wait here.
    if (buf) {
      std::lock_guard<std::mutex> lk(s.ws_mu);
      s.ws_retired.emplace_back(buf, s.issue_seq.load(std::memory_order_acquire));
    }
    buf = d;
    buf_cap = cap;
    workspace_release_retired(ctx, phase);
  }
  return SPD_OK;
}

int workspace_reserve(spd_ctx* ctx, int phase, size_t bytes, char** out) {
  spd_phase_state& s = ctx->phase[phase];
  const int rc = buffer_reserve(ctx, phase, bytes, s.workspace, s.ws_cap);
  *out = s.workspace;
  return rc;
}

// Memory that a prefill step can do without, or null.
static char* spare_reserve(spd_ctx* ctx, size_t bytes, char*& buf, size_t& buf_cap) {
  spd_phase_state& s = ctx->phase[SPD_PHASE_PREFILL];
  // (a staged partition's stream waits for the current one when the step adopts it, and with that joins its capture)
  hipStream_t stream, staged;
  {
    std::lock_guard<std::mutex> lk(ctx->part_mu);
    stream = s.stream;
    staged = s.has_pending ? s.pending_stream : s.stream;
  }
  if (stream_capturing(ctx, stream) || (staged != stream && stream_capturing(ctx, staged))) return nullptr;
  const int error = g_last_hip_error;
  if (buffer_reserve(ctx, SPD_PHASE_PREFILL, bytes, buf, buf_cap) != SPD_OK) {
    (void)hipGetLastError();
    g_last_hip_error = error;
    return nullptr;
  }
  return buf;
}

float* parts_reserve(spd_ctx* ctx, size_t bytes) {
  spd_phase_state& s = ctx->phase[SPD_PHASE_PREFILL];
  return (float*)spare_reserve(ctx, bytes, s.parts, s.parts_cap);
}

char* rows_reserve(spd_ctx* ctx, size_t bytes) {
  spd_phase_state& s = ctx->phase[SPD_PHASE_PREFILL];
  return spare_reserve(ctx, bytes, s.rows, s.rows_cap);
}

int kernel_timing_mark(spd_ctx* ctx, int phase, int which, hipStream_t stream) {
  if (!ctx->kernel_timing) return SPD_OK;
  spd_phase_state& s = ctx->phase[phase];
  hipEvent_t& e = s.kev[s.kev_count % 256][which];
  if (!e) SPD_HIP(hipEventCreate(&e));
  SPD_HIP(hipEventRecord(e, stream));
  if (which == 1) ++s.kev_count;
  return SPD_OK;
}

}  // namespace spd

extern "C" int spd_set_kernel_timing(spd_ctx* ctx, int on) {
  if (!ctx) return SPD_EINVAL;
  if (ctx->device < 0) return SPD_ESTATE;
  ctx->kernel_timing = on != 0;
  return SPD_OK;
}

extern "C" int spd_phase_kernel_ms(spd_ctx* ctx, int phase, float* out, int32_t cap, int32_t* n_out) {
  if (!ctx || phase < 0 || phase > 1 || !n_out || cap < 0 || (cap > 0 && !out)) return SPD_EINVAL;
  if (ctx->device < 0) return SPD_ESTATE;
  int rc = spd_phase_sync(ctx, phase);
  if (rc != SPD_OK) return rc;
  spd_phase_state& s = ctx->phase[phase];
  uint64_t first = s.kev_count > 256 ? s.kev_count - 256 : 0;
  if (first < s.kev_read) first = s.kev_read;
  int32_t n = 0;
  for (uint64_t i = first; i < s.kev_count && n < cap; ++i, ++n)
    SPD_HIP(hipEventElapsedTime(&out[n], s.kev[i % 256][0], s.kev[i % 256][1]));
  s.kev_read = first + (uint64_t)n;
  *n_out = n;
  return SPD_OK;
}

extern "C" int spd_phase_sync(spd_ctx* ctx, int phase) {
  if (!ctx || phase < 0 || phase > 1) return SPD_EINVAL;
  if (ctx->device < 0) return SPD_ESTATE;
  hipStream_t s;
  { std::lock_guard<std::mutex> lk(ctx->part_mu); s = ctx->phase[phase].stream; }
  const uint64_t issued = ctx->phase[phase].issue_seq.load(std::memory_order_acquire);
  SPD_HIP(hipStreamSynchronize(s));
  raise_done_seq(ctx->phase[phase], issued);
  workspace_release_retired(ctx, phase);
  return SPD_OK;
}

extern "C" int spd_phase_query(spd_ctx* ctx, int phase, int* done) {
  if (!ctx || phase < 0 || phase > 1 || !done) return SPD_EINVAL;
  if (ctx->device < 0) return SPD_ESTATE;
  hipStream_t s;
  { std::lock_guard<std::mutex> lk(ctx->part_mu); s = ctx->phase[phase].stream; }
  const uint64_t issued = ctx->phase[phase].issue_seq.load(std::memory_order_acquire);
  hipError_t e = hipStreamQuery(s);
  if (e == hipSuccess) { raise_done_seq(ctx->phase[phase], issued); *done = 1; return SPD_OK; }
  if (e == hipErrorNotReady) { *done = 0; return SPD_OK; }
  return hip_fail(e);
}

extern "C" int spd_phase_wait_for(spd_ctx* ctx, int phase, int other) {
  if (!ctx || phase < 0 || phase > 1 || other < 0 || other > 1 || phase == other) return SPD_EINVAL;
  if (ctx->device < 0) return SPD_ESTATE;
  std::lock_guard<std::mutex> lk(ctx->part_mu);
  spd_phase_state& me = ctx->phase[phase];
  int rc = phase_seal(ctx, phase, me.stream);
  if (rc != SPD_OK) return rc;
  SPD_HIP(hipEventRecord(me.ev_cross, ctx->phase[other].stream));
  SPD_HIP(hipStreamWaitEvent(me.stream, me.ev_cross, 0));
  return SPD_OK;
}

extern "C" int spd_phase_stream(spd_ctx* ctx, int phase, void** hip_stream_out) {
  if (!ctx || phase < 0 || phase > 1 || !hip_stream_out) return SPD_EINVAL;
  if (ctx->device < 0) return SPD_ESTATE;
  std::lock_guard<std::mutex> lk(ctx->part_mu);
  *hip_stream_out = (void*)ctx->phase[phase].stream;
  ctx->phase[phase].stream_lent = true;                 // from here on every step gets its seal at once
  return phase_seal(ctx, phase, ctx->phase[phase].stream);
}

extern "C" int spd_phase_last_ms(spd_ctx* ctx, int phase, float* ms) {
  if (!ctx || phase < 0 || phase > 1 || !ms) return SPD_EINVAL;
  if (ctx->device < 0 || !ctx->phase[phase].timed) return SPD_ESTATE;
  SPD_HIP(hipEventSynchronize(ctx->phase[phase].ev_end));
  SPD_HIP(hipEventElapsedTime(ms, ctx->phase[phase].ev_start, ctx->phase[phase].ev_end));
  return SPD_OK;
}

extern "C" int spd_phase_copy(spd_ctx* ctx, int phase, void* dst, const void* src, uint64_t bytes) {
  if (!ctx || phase < 0 || phase > 1 || !dst || !src || bytes == 0 || bytes % 16 != 0) return SPD_EINVAL;
  if (((uintptr_t)dst | (uintptr_t)src) & 15) return SPD_EINVAL;
  hipStream_t stream;
  int rc = phase_enter(ctx, phase, &stream);
  if (rc != SPD_OK) return rc;
  if ((rc = phase_seal(ctx, phase, stream)) != SPD_OK) return rc;
  SPD_HIP(launch_copy(dst, src, bytes, ctx->phase[phase].active_cus, stream));
  return SPD_OK;
}

extern "C" int spd_phase_read(spd_ctx* ctx, int phase, const void* src, uint64_t bytes) {
  if (!ctx || phase < 0 || phase > 1 || !src || bytes == 0 || bytes % 16 != 0) return SPD_EINVAL;
  if ((uintptr_t)src & 15) return SPD_EINVAL;
  hipStream_t stream;
  int rc = phase_enter(ctx, phase, &stream);
  if (rc != SPD_OK) return rc;
  if ((rc = phase_seal(ctx, phase, stream)) != SPD_OK) return rc;
  SPD_HIP(launch_read(src, bytes, ctx->phase[phase].active_cus, nullptr, stream));
  return SPD_OK;
}

extern "C" int spd_phase_read_lds(spd_ctx* ctx, int phase, const void* src, uint64_t bytes) {
  if (!ctx || phase < 0 || phase > 1 || !src || bytes == 0 || bytes % 16 != 0) return SPD_EINVAL;
  if ((uintptr_t)src & 15) return SPD_EINVAL;
  hipStream_t stream;
  int rc = phase_enter(ctx, phase, &stream);
  if (rc != SPD_OK) return rc;
  if ((rc = phase_seal(ctx, phase, stream)) != SPD_OK) return rc;
  SPD_HIP(launch_read_lds(src, bytes, ctx->phase[phase].active_cus, nullptr, stream));
  return SPD_OK;
}

extern "C" int spd_clock_probe(spd_ctx* ctx, void* hip_stream, uint64_t iters, uint64_t* dev_out) {
  if (!ctx || !dev_out || iters == 0 || iters > (1ull << 32)) return SPD_EINVAL;
  if ((uintptr_t)dev_out & 7) return SPD_EINVAL;
  if (ctx->device < 0) return SPD_ESTATE;
  SPD_HIP(hipSetDevice(ctx->device));
  SPD_HIP(launch_clock_probe(iters, dev_out, (hipStream_t)hip_stream));
  return SPD_OK;
}

extern "C" int spd_issue_probe(spd_ctx* ctx, void* hip_stream, uint64_t* dev_out) {
  if (!ctx || !dev_out || ((uintptr_t)dev_out & 7)) return SPD_EINVAL;
  if (ctx->device < 0) return SPD_ESTATE;
  SPD_HIP(hipSetDevice(ctx->device));
  SPD_HIP(launch_issue_probe(dev_out, (hipStream_t)hip_stream));
  return SPD_OK;
}

extern "C" int spd_phase_probe_cus(spd_ctx* ctx, int phase, int32_t n_blocks, int32_t* ids, int32_t cap,
                                   int32_t* n_ids) {
  if (!ctx || phase < 0 || phase > 1 || n_blocks <= 0 || n_blocks > (1 << 20) || !ids || cap <= 0 || !n_ids)
    return SPD_EINVAL;
  hipStream_t stream;
  int rc = phase_enter(ctx, phase, &stream);
  if (rc != SPD_OK) return rc;
  char* ws = nullptr;
  if ((rc = workspace_reserve(ctx, phase, sizeof(int32_t) * (size_t)n_blocks, &ws)) != SPD_OK) return rc;
  if ((rc = phase_seal(ctx, phase, stream)) != SPD_OK) return rc;
  SPD_HIP(launch_probe((int32_t*)ws, n_blocks, stream));
  std::vector<int32_t> host((size_t)n_blocks);
  SPD_HIP(hipMemcpyAsync(host.data(), ws, sizeof(int32_t) * (size_t)n_blocks, hipMemcpyDeviceToHost, stream));
  SPD_HIP(hipStreamSynchronize(stream));
  std::set<int32_t> uniq(host.begin(), host.end());
  *n_ids = (int32_t)uniq.size();
  if ((size_t)cap < uniq.size()) return SPD_EINVAL;
  std::copy(uniq.begin(), uniq.end(), ids);
  return SPD_OK;
}
