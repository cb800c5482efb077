// Decode step, GQA: paged attention of one query row per request over the unified pool.
//
// Paper, Background "LLM Processing Phases" (decode produces the next token from the last
// token and the KV cache) and "Unified Memory Manager" (the cache is read through the block
// table).  For request b, query head h (KV head g = h / G):
//     out[b,h,:] = sum_{t<n} softmax_t(scale * q[b,h,:] . K[t,g,:]) * V[t,g,:]
//
// The step is bandwidth-bound: every K, V byte of the batch is read exactly once.  One
// workgroup (4 waves) owns one (request, KV head, chunk of the context) and serves all G
// query heads of the group from the same bytes.  Each wave streams whole 16-token tiles from
// HBM straight into matrix-core operand registers (the page layout is arranged so that every
// 16-byte-per-lane load of a wave is 1 KiB contiguous, see internal.h), keeps an online
// softmax per query in registers, and double-buffers the next two tiles while it works.
// The matrix cores are used because G query rows share each key (G*2*d flops per 2*d bytes):
// for G = 8 the fp32 vector units of a partial CU share cannot keep up with HBM.
//   S^T[key, query] = K_tile[16 x d] . Q^T[d x 16]       v_mfma_f32_16x16x32_bf16, d/32 steps
//   O^T[dim, query] += V_tile^T[16 x 16] . P^T[16 x 16]  v_mfma_f32_16x16x16_bf16, d/16 blocks
// Long contexts are split into chunks (split-K); partial (max, sum, O) triples go to a
// workspace and are merged by the launch itself or by a small second kernel (split_merge.h).
#include "internal.h"
#include "rope_device.h"
#include "split_merge.h"

namespace spd {

typedef unsigned short bf16_t;
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// two floats -> two bf16 (round to nearest even), packed low / high
__device__ inline uint32_t pack_bf16_rne(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));
}

template <int D>
struct TileFrag {          // two 16-token tiles, K and V parts, in operand order
  uint4 k[2][D / 32];
  uint4 v[2][D / 32];
};

// A 16-byte load of data that is read exactly once (KV pages in a decode step): marked non-temporal,
// so that the stream does not push the prefill partition's K/V tiles, which ARE re-read, out of the L2
// the two partitions share.
__device__ inline uint4 load_once(const uint4* p) {
  typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
  const u32x4 r = __builtin_nontemporal_load((const u32x4*)p);
  return uint4{r.x, r.y, r.z, r.w};
}

// LDS written above by lanes of this wave is read below by other lanes of it (a wave's LDS accesses are served in order)
__device__ inline void lds_visible_in_wave() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Page ids of the tiles one wave streams, in its lanes: lane 2 i + u holds where tile u of the wave's i-th step lies.
struct TileWindow { uint32_t lo, hi; };

template <int D>
__device__ inline void load_step(TileFrag<D>& f, const char* __restrict__ base, const TileWindow& w, int i, int lane) {
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const uint64_t off = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)w.hi, 2 * i + u) << 32) |
                         (uint32_t)__builtin_amdgcn_readlane((int)w.lo, 2 * i + u);
    const char* p = base + off;
    const uint4* kp = (const uint4*)p + lane;
    const uint4* vp = (const uint4*)(p + TILE_T * D * 2) + lane;
#pragma unroll
    for (int s = 0; s < D / 32; ++s) f.k[u][s] = load_once(kp + s * 64);
#pragma unroll
    for (int s = 0; s < D / 32; ++s) f.v[u][s] = load_once(vp + s * 64);
  }
}

// The token that this step appends is on its way to its page while its tile is on its way here: its key and value are
// put into the operand registers instead (krow, vrow: D entries each in LDS).
template <int D>
__device__ inline void patch_tile(TileFrag<D>& f, int u, int slot, const bf16_t* krow, const bf16_t* vrow, int col, int c4) {
#pragma unroll
  for (int s = 0; s < D / 32; ++s) {
    const uint4 kk = *(const uint4*)(krow + 8 * (4 * s + c4));
    if (col == slot) f.k[u][s] = kk;
    if (c4 == (slot >> 2)) {
      // 16 bytes = [(d / 16) % 2][token % 4] for d = 32 s + col and 32 s + 16 + col
      uint32_t w[4] = {f.v[u][s].x, f.v[u][s].y, f.v[u][s].z, f.v[u][s].w};
      const int t = slot & 3, sh = 16 * (t & 1);
      const uint32_t keep = ~(0xffffu << sh);
      const uint32_t v0 = (uint32_t)vrow[32 * s + col] << sh, v1 = (uint32_t)vrow[32 * s + 16 + col] << sh;
      if (t < 2) { w[0] = (w[0] & keep) | v0; w[2] = (w[2] & keep) | v1; }
      else       { w[1] = (w[1] & keep) | v0; w[3] = (w[3] & keep) | v1; }
      f.v[u][s] = uint4{w[0], w[1], w[2], w[3]};
    }
  }
}

template <int D>
__device__ inline void compute_step(const TileFrag<D>& f, const bf16x8 (&qf)[D / 32], f32x4 (&O)[D / 16], float& m,
                                    float& l, int tile, int n_tiles, int n, float c, int c4) {
  f32x4 S[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    S[u] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < D / 32; ++s)
      S[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, f.k[u][s]), qf[s], S[u], 0, 0, 0);
  }
  // lane holds, for query (lane % 16), the keys tile*16 + 4*c4 + i of each tile
  const bool tail = (tile + 2) * TILE_T > n;
  if (tail) {
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if ((tile + u) * TILE_T + 4 * c4 + i >= n) S[u][i] = -INFINITY;
  }
  float mx = fmaxf(fmaxf(fmaxf(S[0][0], S[0][1]), fmaxf(S[0][2], S[0][3])),
                   fmaxf(fmaxf(S[1][0], S[1][1]), fmaxf(S[1][2], S[1][3])));
  mx = fmaxf(mx, __shfl_xor(mx, 16));
  mx = fmaxf(mx, __shfl_xor(mx, 32));
  const float m_new = fmaxf(m, mx);
  const float alpha = __builtin_amdgcn_exp2f((m - m_new) * c);
  const float mc = m_new * c;
  float psum = 0.f;
  uint2 pb[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    float p[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      p[i] = __builtin_amdgcn_exp2f(S[u][i] * c - mc);
      psum += p[i];
    }
    pb[u].x = pack_bf16_rne(p[0], p[1]);
    pb[u].y = pack_bf16_rne(p[2], p[3]);
  }
  l = l * alpha + psum;
  m = m_new;
#pragma unroll
  for (int blk = 0; blk < D / 16; ++blk) O[blk] *= alpha;
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    int t = tile + u;
    t = t < n_tiles ? t : n_tiles - 1;
    const bool vtail = (t + 1) * TILE_T > n;      // tile holds slots past the context: their bytes are arbitrary
#pragma unroll
    for (int b2 = 0; b2 < D / 32; ++b2) {
      uint4 v = f.v[u][b2];
      if (vtail) {
        const int t0 = t * TILE_T + 4 * c4;
        const uint32_t m01 = (t0 + 0 < n ? 0x0000ffffu : 0u) | (t0 + 1 < n ? 0xffff0000u : 0u);
        const uint32_t m23 = (t0 + 2 < n ? 0x0000ffffu : 0u) | (t0 + 3 < n ? 0xffff0000u : 0u);
        v.x &= m01; v.y &= m23; v.z &= m01; v.w &= m23;
      }
      const s16x4 a0 = __builtin_bit_cast(s16x4, uint2{v.x, v.y});
      const s16x4 a1 = __builtin_bit_cast(s16x4, uint2{v.z, v.w});
      const s16x4 pv = __builtin_bit_cast(s16x4, pb[u]);
      O[2 * b2] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a0, pv, O[2 * b2], 0, 0, 0);
      O[2 * b2 + 1] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a1, pv, O[2 * b2 + 1], 0, 0, 0);
    }
  }
}

// Where a share has few workgroups the attention launch is the whole step: it rotates its query heads (RoPE), rotates the new
// token's key and puts key and value into their page (the workgroup of the request's last chunk, per KV head), and attends
// to the context with that token included.  As launches of their own the append and the rotation cost 5.6 us per step,
// and more than the attention itself in a batch of a few short contexts.  Where a compute unit has many workgroups
// they pay for that in turn, and decode_prepare_kernel does it for all of them.
struct GqaArgs {
  char* pool;
  uint64_t page_bytes;
  uint32_t head_bytes, tile_bytes;
  int tiles_per_page;
  const bf16_t *q, *k_new, *v_new;
  bf16_t* out;
  const char* items;
  int item_stride, Hkv, H, G;
  float c;                      // scale * log2(e)
  int max_chunks;
  const double* w;
  int rot, off, interleaved;
  float *ws_o, *ws_ml;
  int32_t* put_chunks;
  uint32_t* counters;
  StepMark mark;
};

// grid (n_items * n_kv_heads), block 256; workgroup i serves KV head i % n_kv_heads of work item
// i / n_kv_heads.  Heads vary fastest so that the round-robin placement of
// workgroups on the 8 XCDs gives every XCD the same mix of long and short chunks.
// WHOLE: the launch rotates and appends too; otherwise decode_prepare_kernel has, and this kernel's workgroups, of which a compute
// unit then has many in turn, start without that code.
template <int D, bool WHOLE>
__global__ __launch_bounds__(256, 2) void decode_gqa_kernel(GqaArgs a) {
  if constexpr (!WHOLE) {
    a.rot = 0;
    a.k_new = nullptr;
    a.mark.flag = nullptr;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) store_mark(a.mark);
  const int g = blockIdx.x % a.Hkv;
  const char* rec = a.items + (size_t)(blockIdx.x / a.Hkv) * a.item_stride;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave-uniform
  const int col = lane & 15, c4 = lane >> 4;
  __shared__ __attribute__((aligned(16))) float sm_o[4][16][D + 4];
  __shared__ float sm_m[4][16], sm_l[4][16];
  __shared__ int32_t sm_rec[256];
  __shared__ uint32_t sm_last;
  // The record (header, page ids) is fetched once per workgroup: it may lie in pinned host memory.
  const int words = a.item_stride >> 2;
  if ((int)threadIdx.x < words) sm_rec[threadIdx.x] = ((const int32_t*)rec)[threadIdx.x];
  const double w_lane = a.rot ? a.w[min(lane, (a.rot >> 1) - 1)] : 0.0;
  __syncthreads();
  const int b = __builtin_amdgcn_readfirstlane(sm_rec[0]), chunk = __builtin_amdgcn_readfirstlane(sm_rec[1]);
  const int n_chunks = __builtin_amdgcn_readfirstlane(sm_rec[2]), n = __builtin_amdgcn_readfirstlane(sm_rec[3]);
  if (a.put_chunks && chunk == 0 && g == 0 && threadIdx.x == 0) a.put_chunks[b] = n_chunks;
  auto page_id = [&](int i) -> int {               // i-th page of the chunk
    const int wd = min(i + DECODE_ITEM_WORDS, words - 1);
    int id = sm_rec[min(wd, 255)];
    if (words > 256 && wd > 255) id = ((const int32_t*)rec)[wd];
    return id;
  };
  const int n_tiles = (n + TILE_T - 1) / TILE_T;
  const int tile0 = __builtin_amdgcn_readfirstlane(sm_rec[4]), tile1 = tile0 + __builtin_amdgcn_readfirstlane(sm_rec[5]);
  const int n_steps = (tile1 - tile0 + 1) >> 1;
  const int my_steps = (n_steps - wave + 3) >> 2;                      // this wave's steps: wave, wave + 4, ...
  const bool interleaved = a.interleaved != 0;

  // Each wave has a piece of LDS of its own, later used for its part of the merge: nothing in it needs a barrier.
  float* cs = &sm_o[wave][0][0];                   // [D / 2] cosines, sines, then the new token's key and value
  float* sn = cs + D / 2;
  bf16_t* krow = (bf16_t*)(sn + D / 2);
  bf16_t* vrow = krow + D;

  // where tile u of step i (of the 32 the window holds) lies: lane 2 i + u
  char* pool_g = a.pool + (uint64_t)g * a.head_bytes;
  const int page0 = tile0 / a.tiles_per_page;
  auto fill_window = [&](int s0) -> TileWindow {
    const int t = min(tile0 + 2 * (wave + 4 * (s0 + (lane >> 1))) + (lane & 1), n_tiles - 1);   // out of range: the last tile, masked later
    const int pg = t / a.tiles_per_page;
    const uint64_t off = (uint64_t)(uint32_t)page_id(pg - page0) * a.page_bytes + (uint64_t)(t - pg * a.tiles_per_page) * a.tile_bytes;
    return TileWindow{(uint32_t)off, (uint32_t)(off >> 32)};
  };

  // ---- the loads that everything waits for first: query pieces, and in one wave the new token's key and value
  uint4 own[D / 32], oth[D / 32];
  const bf16_t* qrow = a.q + ((size_t)b * a.H + g * a.G + min(col, a.G - 1)) * D;
#pragma unroll
  for (int s = 0; s < D / 32; ++s) {
    const int e0 = 8 * (4 * s + c4);
    own[s] = *(const uint4*)(qrow + e0);
    if (a.rot) oth[s] = *(const uint4*)(qrow + rope_partner(e0, a.off, a.rot, interleaved));
  }
  // the new token's tile is the last one of the request: the wave whose step holds it does the append
  const bool appends = a.k_new != nullptr && tile1 == n_tiles && ((n_steps - 1) & 3) == wave;
  const int patch = appends ? n_tiles - 1 : -1;
  constexpr int PCS = D / 8;                       // 16-byte pieces of a head
  uint4 kv_own = uint4{0, 0, 0, 0}, kv_oth = uint4{0, 0, 0, 0};
  if (appends) {                                   // lanes 0 .. PCS - 1: pieces of the key, the next PCS: of the value
    const int pc = lane % PCS, e0 = 8 * pc;
    const bf16_t* src = (lane / PCS & 1) ? a.v_new : a.k_new;
    src += ((size_t)b * a.Hkv + g) * D;
    kv_own = *(const uint4*)(src + e0);
    if (a.rot && lane < PCS) kv_oth = *(const uint4*)(src + rope_partner(e0, a.off, a.rot, interleaved));
  }

  TileFrag<D> fa, fb;
  TileWindow win = TileWindow{0, 0};
  if (my_steps > 0) {
    win = fill_window(0);
    load_step<D>(fa, pool_g, win, 0, lane);
  }
  if (a.rot) {
    if (lane < (a.rot >> 1)) {
      const double turns = (double)(n - 1) * w_lane * 0.15915494309189535;
      const float ang = (float)((turns - __builtin_rint(turns)) * 6.283185307179586);
      sincosf(ang, &sn[lane], &cs[lane]);
    }
    lds_visible_in_wave();
  }
  bf16x8 qf[D / 32];
#pragma unroll
  for (int s = 0; s < D / 32; ++s) {
    uint4 piece = own[s];
    if (a.rot) piece = rope_rotate(own[s], oth[s], 8 * (4 * s + c4), a.off, a.rot, interleaved, cs, sn);
    if (col >= a.G) piece = uint4{0, 0, 0, 0};
    qf[s] = __builtin_bit_cast(bf16x8, piece);
  }
  if (appends) {
    const int pc = lane % PCS, t = (n - 1) % TILE_T;
    const int pg = (n_tiles - 1) / a.tiles_per_page;
    char* tile = pool_g + (uint64_t)(uint32_t)page_id(pg - page0) * a.page_bytes + (uint64_t)(n_tiles - 1 - pg * a.tiles_per_page) * a.tile_bytes;
    if (lane < PCS) {
      const uint4 piece = a.rot ? rope_rotate(kv_own, kv_oth, 8 * pc, a.off, a.rot, interleaved, cs, sn) : kv_own;
      *(uint4*)(krow + 8 * pc) = piece;
      *(uint4*)(tile + ((size_t)(pc * TILE_T + t) << 4)) = piece;
    } else if (lane < 2 * PCS) {
      *(uint4*)(vrow + 8 * pc) = kv_own;
    }
    lds_visible_in_wave();
    for (int d = lane; d < D; d += 64) ((bf16_t*)(tile + TILE_T * D * 2))[v_elem_offset(t, d)] = vrow[d];
  }

  f32x4 O[D / 16];
#pragma unroll
  for (int i = 0; i < D / 16; ++i) O[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY, l = 0.f;

  // Software pipeline over this wave's steps j = wave, wave + 4, ...: the loads of the next step
  // are in flight while the current one is consumed.  The steady-state loop body has no branch,
  // so the compiler can wait for exactly the older buffer (vmcnt = loads of the newer one).
  // Only a request's last step can hold the appended token, so the patch sits behind the steady state.
#define SPD_TILE(I) (tile0 + 2 * (wave + 4 * (I)))
#define SPD_LOAD(F, I) load_step<D>(F, pool_g, win, (I) - s0, lane)
#define SPD_COMP(F, I) compute_step<D>(F, qf, O, m, l, SPD_TILE(I), n_tiles, n, a.c, c4)
#define SPD_LAST(F, I)                                                                                              \
  do {                                                                                                              \
    if (patch >= 0) {                                                                                               \
      if (min(SPD_TILE(I), n_tiles - 1) == patch) patch_tile<D>(F, 0, (n - 1) % TILE_T, krow, vrow, col, c4);       \
      if (min(SPD_TILE(I) + 1, n_tiles - 1) == patch) patch_tile<D>(F, 1, (n - 1) % TILE_T, krow, vrow, col, c4);   \
    }                                                                                                               \
    SPD_COMP(F, I);                                                                                                 \
  } while (0)
  for (int s0 = 0; s0 < my_steps; s0 += 32) {      // 32 steps (of 128 tokens over the four waves) per window
    const int s1 = min(my_steps, s0 + 32);
    if (s0) {
      win = fill_window(s0);
      SPD_LOAD(fa, s0);
    }
    int i = s0;
    while (i + 2 < s1) {
      SPD_LOAD(fb, i + 1);
      SPD_COMP(fa, i);
      SPD_LOAD(fa, i + 2);
      SPD_COMP(fb, i + 1);
      i += 2;
    }
    if (i + 1 < s1) {
      SPD_LOAD(fb, i + 1);
      SPD_COMP(fa, i);
      SPD_LAST(fb, i + 1);
    } else {
      SPD_LAST(fa, i);
    }
  }
#undef SPD_TILE
#undef SPD_LOAD
#undef SPD_COMP
#undef SPD_LAST
  l += __shfl_xor(l, 16);
  l += __shfl_xor(l, 32);

  // merge the four waves' (m, l, O) through LDS
#pragma unroll
  for (int blk = 0; blk < D / 16; ++blk)
    *(f32x4*)&sm_o[wave][col][16 * blk + 4 * c4] = O[blk];
  if (c4 == 0) { sm_m[wave][col] = m; sm_l[wave][col] = l; }
  __syncthreads();
  const size_t head0 = (size_t)b * a.H + g * a.G;
  // two output dims per thread
  for (int idx = threadIdx.x; idx < a.G * (D / 2); idx += 256) {
    const int qh = idx / (D / 2), d = 2 * (idx % (D / 2));
    const float m_tot = fmaxf(fmaxf(sm_m[0][qh], sm_m[1][qh]), fmaxf(sm_m[2][qh], sm_m[3][qh]));
    float l_tot = 0.f, o0 = 0.f, o1 = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const float wgt = __builtin_amdgcn_exp2f((sm_m[w][qh] - m_tot) * a.c);
      l_tot += sm_l[w][qh] * wgt;
      o0 += sm_o[w][qh][d] * wgt;
      o1 += sm_o[w][qh][d + 1] * wgt;
    }
    const size_t head = head0 + qh;
    if (n_chunks == 1) {
      *(uint32_t*)(a.out + head * D + d) = pack_bf16_rne(o0 / l_tot, o1 / l_tot);
    } else {
      const size_t slot = head * a.max_chunks + chunk;
      store_partial(a.ws_o + slot * D + d, o0, o1, a.counters != nullptr);
      if (d == 0) store_partial(a.ws_ml + slot * 2, m_tot * a.c, l_tot, a.counters != nullptr);
    }
  }
  if (n_chunks == 1 || a.counters == nullptr) return;
  // ---- few chunks: the workgroup that finds itself to be the last of its (request, KV head) merges them
  if (!last_of(a.counters + (size_t)b * a.Hkv + g, (uint32_t)n_chunks, &sm_last)) return;
  const size_t slot0 = head0 * a.max_chunks;
  merge_in_launch<D, 256>(a.ws_o + slot0 * D, a.ws_ml + slot0 * 2, a.G, a.max_chunks, n_chunks, &sm_o[0][0][0], a.out + head0 * D);
}

// What the attention launch would otherwise do in every workgroup, done once per request: the queries are rotated into q_rot, the
// new token's key (rotated) and value go into their page.  Same arithmetic as in the attention launch, so the step's results do
// not depend on which of the two does it.  The records are read in device memory: read in pinned memory by a workgroup
// each they take 9 to 16 us (the more compute units ask, the longer), copied by a few workgroups beforehand 3.4.
// grid (n_items), block 256: the workgroup of a request's last chunk does the request.  Bound by latency: record, then rows.
// 256 requests of 15 .. 45 tokens, 32 query and 8 KV heads with RoPE, whole step: with everything in the attention launch 140 us on
// 64 CUs and 72 on 128, now 67 and 40.
template <int D>
__global__ __launch_bounds__(256) void decode_prepare_kernel(GqaArgs a, bf16_t* __restrict__ q_rot) {
  const int tid = threadIdx.x;
  const int32_t* head = (const int32_t*)(a.items + (size_t)blockIdx.x * a.item_stride);
  __shared__ float cs[D / 2], sn[D / 2];
  const double w = tid < (a.rot >> 1) ? a.w[tid] : 0.0;
  const int last_page = head[(a.item_stride >> 2) - 1];          // (a record's end repeats the chunk's last page)
  const int b = head[0], n = head[3], n_tiles = (n + TILE_T - 1) / TILE_T;
  if (head[4] + head[5] != n_tiles) return;        // not the request's last chunk
  const bool interleaved = a.interleaved != 0;
  constexpr int PCS = D / 8, BATCH = 4;            // 16-byte pieces of a head; loads on their way per thread
  const int n_q = a.rot ? a.H * PCS : 0, n_k = a.k_new ? a.Hkv * PCS : 0, n_v = a.k_new ? a.Hkv * D : 0;
  const bf16_t *q = a.q + (size_t)b * a.H * D, *k_new = a.k_new + (size_t)b * a.Hkv * D, *v_new = a.v_new + (size_t)b * a.Hkv * D;
  auto load = [&](const bf16_t* rows, int i, uint4& own, uint4& oth) {
    own = *(const uint4*)(rows + 8 * i);
    if (a.rot) oth = *(const uint4*)(rows + i / PCS * D + rope_partner(8 * (i % PCS), a.off, a.rot, interleaved));
  };
  auto rotated = [&](int i, const uint4& own, const uint4& oth) -> uint4 {
    return a.rot ? rope_rotate(own, oth, 8 * (i % PCS), a.off, a.rot, interleaved, cs, sn) : own;
  };
  // the first rows are on their way while the angles are formed
  uint4 own[BATCH], oth[BATCH], k = uint4{0, 0, 0, 0}, k_oth = k;
  bf16_t v[BATCH] = {};
  if (n_q) {
#pragma unroll
    for (int j = 0; j < BATCH; ++j) load(q, min(tid + 256 * j, n_q - 1), own[j], oth[j]);
  }
  if (n_k) {
    load(k_new, min(tid, n_k - 1), k, k_oth);
#pragma unroll
    for (int j = 0; j < BATCH; ++j) v[j] = v_new[min(tid + 256 * j, n_v - 1)];
  }
  if (a.rot) {
    if (tid < (a.rot >> 1)) {
      const double turns = (double)(n - 1) * w * 0.15915494309189535;
      const float ang = (float)((turns - __builtin_rint(turns)) * 6.283185307179586);
      sincosf(ang, &sn[tid], &cs[tid]);
    }
    __syncthreads();
  }
  bf16_t* to = q_rot + (size_t)b * a.H * D;
  for (int i0 = tid; i0 < n_q; i0 += 256 * BATCH) {
#pragma unroll
    for (int j = 0; j < BATCH; ++j) {
      const int i = i0 + 256 * j;
      if (i < n_q) *(uint4*)(to + 8 * i) = rotated(i, own[j], oth[j]);
    }
#pragma unroll
    for (int j = 0; j < BATCH; ++j) load(q, min(i0 + 256 * (BATCH + j), n_q - 1), own[j], oth[j]);
  }
  const int t = (n - 1) % TILE_T;
  char* tile = a.pool + (uint64_t)(uint32_t)last_page * a.page_bytes + (uint64_t)((n_tiles - 1) % a.tiles_per_page) * a.tile_bytes;
  for (int i = tid; i < n_k; i += 256) {
    if (i != tid) load(k_new, i, k, k_oth);
    *(uint4*)(tile + (uint64_t)(i / PCS) * a.head_bytes + ((size_t)(i % PCS * TILE_T + t) << 4)) = rotated(i, k, k_oth);
  }
  for (int i0 = tid; i0 < n_v; i0 += 256 * BATCH) {
#pragma unroll
    for (int j = 0; j < BATCH; ++j) {
      const int i = i0 + 256 * j;
      if (i < n_v) ((bf16_t*)(tile + (uint64_t)(i / D) * a.head_bytes + TILE_T * D * 2))[v_elem_offset(t, i % D)] = i0 == tid ? v[j] : v_new[i];
    }
  }
}

static GqaArgs gqa_args(const PoolGeom& g, char* pool_base, const DecodeLaunch& d) {
  GqaArgs a;
  a.pool = pool_base;
  a.page_bytes = g.page_bytes; a.head_bytes = g.head_bytes; a.tile_bytes = g.tile_bytes; a.tiles_per_page = g.tiles_per_page;
  a.q = (const bf16_t*)d.q; a.k_new = (const bf16_t*)d.k_new; a.v_new = (const bf16_t*)d.v_new; a.out = (bf16_t*)d.out;
  a.items = d.items; a.item_stride = d.item_stride;
  a.Hkv = g.Hkv; a.H = d.H; a.G = d.H / g.Hkv;
  a.c = d.scale * 1.4426950408889634f;
  a.max_chunks = d.max_chunks;
  a.w = d.w; a.rot = d.rot; a.off = d.off; a.interleaved = d.interleaved;
  a.ws_o = d.ws_o; a.ws_ml = d.ws_ml; a.put_chunks = d.put_chunks; a.counters = d.counters; a.mark = d.mark;
  return a;
}

template <int D>
static hipError_t launch_decode_gqa_t(const PoolGeom& g, char* pool_base, const DecodeLaunch& d, hipStream_t stream) {
  const dim3 grid((unsigned)d.n_wgs * g.Hkv);
  if (d.prepared) hipLaunchKernelGGL((decode_gqa_kernel<D, false>), grid, dim3(256), 0, stream, gqa_args(g, pool_base, d));
  else hipLaunchKernelGGL((decode_gqa_kernel<D, true>), grid, dim3(256), 0, stream, gqa_args(g, pool_base, d));
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || d.max_chunks <= 1 || d.counters) return e;
  return launch_merge_chunks<D>(d, stream);
}

hipError_t launch_decode_gqa(const PoolGeom& g, char* pool_base, const DecodeLaunch& d, hipStream_t stream) {
  if (g.dk == 128) return launch_decode_gqa_t<128>(g, pool_base, d, stream);
  if (g.dk == 64) return launch_decode_gqa_t<64>(g, pool_base, d, stream);
  return hipErrorInvalidValue;
}

hipError_t launch_decode_prepare(const PoolGeom& g, char* pool_base, const DecodeLaunch& d, int n_items, void* q_rot, hipStream_t stream) {
  const GqaArgs a = gqa_args(g, pool_base, d);
  if (g.dk == 128) hipLaunchKernelGGL(decode_prepare_kernel<128>, dim3((unsigned)n_items), dim3(256), 0, stream, a, (bf16_t*)q_rot);
  else if (g.dk == 64) hipLaunchKernelGGL(decode_prepare_kernel<64>, dim3((unsigned)n_items), dim3(256), 0, stream, a, (bf16_t*)q_rot);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace spd
