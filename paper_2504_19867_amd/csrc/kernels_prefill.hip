// Prefill step: causal attention over each request's prompt (varlen-packed batch).
//
// Paper, Background "LLM Processing Phases": the prefill phase processes the whole input
// context.  For request r, query head h (KV head g = h / (H / Hkv)), row i:
//     out[i,h,:] = sum_{j<=i} softmax_j(scale * q[i,h,:] . k[j,g,:]) * v[j,g,:]
// (The page write of K, V that belongs to the same step is kv_write_kernel.)
// With a cached prefix of p tokens (chunked prefill) the request's K, V hold p + len rows, all of them in its
// pages or brought together as dense rows, and query row i sits at position p + i: the sum runs over j <= p + i.
//
// A dense contraction, so it runs on the matrix cores.  One workgroup = 8 waves = one CU's worth
// of work; every wave owns 32 query rows of one head.  The 8 waves are HB query heads of ONE
// KV head (grouped-query attention: they all need the same K, V) times 8 / HB row sub-tiles,
// so each K/V tile fetched into LDS feeds 256 (row, head) pairs.
//
// Everything is kept TRANSPOSED so that a query is a lane (column), not a row:
//     S^T[key, query] = K_tile[64 x d] . Q^T[d x 32]          v_mfma_f32_32x32x16_bf16
//     O^T[dim, query] += V_tile^T[dv x 64] . P^T[64 x 32]
// With queries along lanes the softmax statistics (running max, running sum, rescale factor)
// are per-lane scalars, the row maximum needs one cross-lane exchange per tile (lane ^ 32), and
// the S^T accumulators are already in the B-operand order of the second product: P never
// leaves registers.  Q^T fragments live in registers for the whole workgroup.
//
// The kernel is persistent: one workgroup per compute unit of the prefill share walks a chain of
// work items (one item = one tile of query rows of one request for one group of heads), and the
// K/V tile loads run ahead of the compute across item boundaries, so that an item's first tiles,
// which a fresh workgroup would have to wait for, arrive while the item before is still computing.
//
// K and V tiles of 64 keys stream from global memory straight into a ring of LDS stages with
// global_load_lds_dwordx4 (no register staging, no LDS stores), ahead of the compute; one
// s_barrier per pair of tiles where the ring has four stages (one per tile with three; two in prefill_192_kernel).  K rows
// are read back with 16-byte reads in A-operand order; V stays in its natural [key][dim] order
// and the transposition that the second product needs is done by the LDS transpose read
// ds_read_b64_tr_b16.  Both tiles are XOR-swizzled at 16-byte granularity against bank conflicts.
// A step with cached tokens has its tiles out of the pages, unless dense_rows_pay (prefill_work.h): four units of 16 tokens each, in the
// order in which the pages (laid out for the decode kernel) have them, which is an operand order here too.  With the rows brought together in dense tensors first
// (by the page write's launch, once through HBM and back) 4 pieces of 201 .. 1024 tokens behind up to 7680 cached ones of the
// Llama-3-8B layer took 139 us on 256 CUs, now 128: the page write's launch 32 -> 17 us, this kernel 101 -> 103.
//
// The softmax keeps a reference per query that is moved to the running maximum only when a row sum
// shows that it must be (an item's first tile, or scores that have outgrown it by 2^60).
#include "internal.h"
#include <type_traits>

namespace spd {

typedef unsigned short bf16_t;
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));

constexpr int BN = 64;        // keys per LDS tile
constexpr int WAVES = 8;      // waves per workgroup

__device__ inline uint32_t cvt_pk_bf16(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));
}

// 16 bytes per lane from global memory (a wave-uniform base and a 32-bit per-lane offset) to LDS: lane i's data lands at
// lds_byte_addr + 16 * i.  The compiler does not see this write; completion is tracked by hand with vmcnt (below).
__device__ inline void dma16s(const void* sbase, uint32_t voff, uint32_t lds_byte_addr) {
  asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_byte_addr), "v"(voff), "s"(sbase) : "memory");
}
// s_waitcnt vmcnt(N) only (expcnt and lgkmcnt fields left at their maxima)
#define SPD_WAIT_VMCNT(N) __builtin_amdgcn_s_waitcnt(((N) & 15) | (7 << 4) | (15 << 8) | (((N) >> 4) << 14))

// XOR swizzles (in units of 16-byte chunks) of a dense K row and a dense V row
template <int DQK> __device__ inline int k_swz(int row) { return DQK == 128 ? (row & 15) : ((row >> 1) & 7); }
template <int DV> __device__ inline int v_swz(int row) { return DV == 128 ? 4 * (row & 3) : 4 * ((row >> 1) & 1); }

// Rows i .. i + 3 of a block of 32 rows of O^T into a staged row of the output, as out_pairs has them in bf16.  Out of pages row i is
// dim i / 2 + 16 (i % 2).
template <bool PAGED> __device__ inline uint2 out_pairs(float a, float b, float c, float d) {
  return PAGED ? uint2{cvt_pk_bf16(a, c), cvt_pk_bf16(b, d)} : uint2{cvt_pk_bf16(a, b), cvt_pk_bf16(c, d)};
}
template <bool PAGED> __device__ inline void stage_out(char* row, int i, uint2 pairs) {
  if constexpr (PAGED) {
    *(uint32_t*)(row + i) = pairs.x;
    *(uint32_t*)(row + i + 32) = pairs.y;
  } else {
    *(uint2*)(row + i * 2) = pairs;
  }
}

// PARTS: items may be parts of items (an instance of its own: the code for it costs the other steps up to 1 %).
// PAGED: K, V out of the pages (pages, units, head_units; see PrefillLists) instead of the dense rows k, v.
template <int DQK, int DV, int HB, bool PARTS, bool PAGED>
__global__ __launch_bounds__(512, 2) void prefill_kernel(const bf16_t* __restrict__ q, const bf16_t* __restrict__ k,
                                                         const bf16_t* __restrict__ v, const char* __restrict__ pages,
                                                         const int32_t* __restrict__ units, int head_units, bf16_t* __restrict__ out,
                                                         const PrefillWork* __restrict__ work,
                                                         const int32_t* __restrict__ chain, int H, int Hkv,
                                                         float c /* scale * log2(e) */, const PrefillRange* __restrict__ range, float* __restrict__ parts) {
  constexpr int QS = WAVES / HB;                // 32-row sub-tiles per workgroup
  constexpr int CHK = DQK / 8, CHV = DV / 8;    // 16-byte chunks per K / V row
  constexpr int K_BYTES = BN * DQK * 2, V_BYTES = BN * DV * 2, STAGE_BYTES = K_BYTES + V_BYTES;
  constexpr int NSTAGE = DQK > 128 ? 3 : 4;     // LDS ring
  constexpr int PD = NSTAGE - 1;                // tiles in flight ahead of the compute
  constexpr int NI = CHK + CHV;                 // 1 KiB load instructions per tile
  static_assert(NI % WAVES == 0, "tile loads must divide evenly over the waves");
  constexpr int LPW = NI / WAVES;               // load instructions per wave per tile
  constexpr int KS = DQK / 16, VB = DV / 32;
  constexpr int NS = 2 * KS;                    // MFMAs of S^T
  constexpr int RING = DQK > 128 ? 4 : 8;       // K operands in flight (fewer where registers are short)
  static_assert(NS >= RING, "operand ring longer than the first product");
  // a unit of 16 tokens as it lies in a page: K part, then V part
  constexpr int UNIT_K = TILE_T * DQK * 2, UNIT_BYTES = UNIT_K + TILE_T * DV * 2, UNIT_LOADS = UNIT_BYTES / 1024;
  constexpr int OPITCH = 32 * 2 + 16;           // bytes per staged output row piece (32 dims, padded)
  constexpr int EPI_BYTES = WAVES * 32 * OPITCH;  // output staging, apart from the K/V stages
  __shared__ __attribute__((aligned(1024))) char smem[NSTAGE * STAGE_BYTES + EPI_BYTES];

  const int G = H / Hkv;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n32 = lane & 31, hh = lane >> 5;
  const uint32_t k_pitch = (uint32_t)Hkv * DQK * 2, v_pitch = (uint32_t)Hkv * DV * 2;   // (dense rows)
  const uint32_t smem_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem;
  // this workgroup's chain of work items
  int it = __builtin_amdgcn_readfirstlane(chain[blockIdx.x]);
  const int it_end = __builtin_amdgcn_readfirstlane(chain[blockIdx.x + 1]);
  if (it >= it_end) return;

  // ---- tile loads.  Load instruction ii = wave + 8 j (j < LPW) fills 1 KiB of the stage.
  // Paged: a stage is the tile's four units one after the other, each as it lies in its page, so an instruction reads 1 KiB of
  // consecutive bytes, from an address that is the wave's but for the lane's 16 bytes.
  // Dense rows: the 64 consecutive 16-byte slots [64 ii, 64 ii + 64), K slots first (row = slot / CHK), then V slots;
  // slot s of a row holds the row's chunk s ^ swz(row).  The per-lane part of the address does not depend on the tile
  // (except past the prompt's end).
  auto slot_of = [&](int j, int& row, int& coff, uint32_t& pitch) __attribute__((always_inline)) {
    const int ii = wave + WAVES * j;
    if (ii < CHK) {
      const int slot = ii * 64 + lane, sl = slot % CHK;
      row = slot / CHK;
      coff = (sl ^ k_swz<DQK>(row)) * 16;
      pitch = k_pitch;
    } else {
      const int slot = (ii - CHK) * 64 + lane, sl = slot % CHV;
      row = slot / CHV;
      coff = (sl ^ v_swz<DV>(row)) * 16;
      pitch = v_pitch;
    }
  };
  uint32_t ld_voff[PAGED ? 1 : LPW];
  if constexpr (PAGED) {
    ld_voff[0] = (uint32_t)(wave % UNIT_LOADS * 1024 + lane * 16);
  } else {
#pragma unroll
    for (int j = 0; j < LPW; ++j) {
      int row, coff;
      uint32_t pitch;
      slot_of(j, row, coff, pitch);
      ld_voff[j] = (uint32_t)row * pitch + (uint32_t)coff;
    }
  }
  // ---- the chain's work items, 64 at a time, one per lane: item i sits in lane i - dsc_base.  An item is then had
  // with six lane reads, where a load from memory at every item boundary (one by the producer, one by the
  // compute side, each waited for at once, and every such wait also drains the tile loads in flight) cost the
  // chain about as much as three tiles.  The producer is at most a few items ahead of the compute side, which
  // moves the window when it is half way through it.  (Not with 192 dims: the touch below needs the full wait that
  // only the paired tiles have.)
  constexpr bool ITEM_LANES = DQK <= 128;
  static_assert(ITEM_LANES || !PARTS, "parts come by lanes");
  int dsc_base = it;
  int d_row0 = 0, d_len = 0, d_qtile = 0, d_head0 = 0, d_kvrow0 = 0, d_qoff = 0, d_kt0 = 0, d_kt1 = 0, d_part = 0;
  auto load_items = [&](int base) __attribute__((always_inline)) {
    const PrefillWork pw = work[min(base + lane, it_end - 1)];
    d_row0 = pw.row0; d_len = pw.len; d_qtile = pw.q_tile; d_head0 = pw.head0; d_kvrow0 = pw.kv_row0; d_qoff = pw.q_off;
    if constexpr (PARTS) {
      PrefillRange pr = {0, (pw.q_off + min(pw.len, (pw.q_tile + 1) * (32 * QS)) + BN - 1) / BN, -1};
      if (range) pr = range[min(base + lane, it_end - 1)];
      d_kt0 = pr.kt0; d_kt1 = pr.kt1; d_part = pr.part;
    }
    dsc_base = base;
  };
  auto item_of = [&](int i) __attribute__((always_inline)) -> PrefillWork {
    if constexpr (!ITEM_LANES) return work[i];
    const int l = i - dsc_base;
    return PrefillWork{__builtin_amdgcn_readlane(d_row0, l), __builtin_amdgcn_readlane(d_len, l),
                       __builtin_amdgcn_readlane(d_qtile, l), __builtin_amdgcn_readlane(d_head0, l),
                       __builtin_amdgcn_readlane(d_kvrow0, l), __builtin_amdgcn_readlane(d_qoff, l)};
  };
  if constexpr (ITEM_LANES) load_items(it);
  // ---- producer: the tile loads run ahead of the compute (a pair of tiles, or PD tiles where the
  // ring has three stages), across the items of the chain.
  // pt counts the tiles issued so far (tile number pt goes to stage pt % NSTAGE).
  int p_it = it, p_kt = 0, p_n = 0, p_kv_len = 0, pt = 0;
  const char *p_kb = nullptr, *p_vb = nullptr;  // dense rows
  // Paged: the numbers of the units that the item's next tiles lie in, 64 of them, one per lane; tile p_kt's are in the lanes from p_win
  // on.  They are had with one load per 16 tiles, which is not waited for before the next tile's loads go out.
  const int32_t* p_units = nullptr;
  int p_head = 0, p_win = 0, win = 0;
  bool win_new = false;
  auto load_window = [&]() __attribute__((always_inline)) {
    win = p_units[min(4 * p_kt + lane, (p_kv_len - 1) / TILE_T)];   // (units past the last one: that one again)
    p_win = 0;
    win_new = true;
  };
  auto producer_item = [&]() __attribute__((always_inline)) {                  // producer state for item p_it
    const PrefillWork pw = item_of(p_it);
    const int pg = pw.head0 / G;
    p_kv_len = pw.q_off + pw.len;
    p_n = PARTS ? __builtin_amdgcn_readlane(d_kt1, p_it - dsc_base) : (min(p_kv_len, pw.q_off + pw.q_tile * (32 * QS) + 32 * QS) + BN - 1) / BN;
    p_kt = PARTS ? __builtin_amdgcn_readlane(d_kt0, p_it - dsc_base) : 0;
    if constexpr (PAGED) {
      p_units = units + pw.kv_row0;
      p_head = pg * head_units;
      load_window();
    } else {
      p_kb = (const char*)(k + ((size_t)pw.kv_row0 * Hkv + pg) * DQK);
      p_vb = (const char*)(v + ((size_t)pw.kv_row0 * Hkv + pg) * DV);
    }
  };
  producer_item();
  auto produce_one = [&]() __attribute__((always_inline)) {
    if (p_it >= it_end) return;
    const uint32_t stage = smem_base + (uint32_t)(pt % NSTAGE) * STAGE_BYTES;
    if constexpr (PAGED) {
      // A full wait: loads into LDS and loads into registers are not known to return in one order.  (Behind a pair's barrier there
      // is nothing to wait for, and between a pair's tiles little.)
      if (win_new) SPD_WAIT_VMCNT(0);
      win_new = false;
#pragma unroll
      for (int j = 0; j < LPW; ++j) {
        const int u = (wave + WAVES * j) / UNIT_LOADS;
        const size_t unit = (size_t)(uint32_t)(__builtin_amdgcn_readlane(win, p_win + u) + p_head);
        dma16s(pages + unit * UNIT_BYTES, ld_voff[0], stage + (uint32_t)(wave + WAVES * j) * 1024);
      }
    } else {
      const int kv0 = p_kt * BN;
      const char* kb = p_kb + (size_t)kv0 * k_pitch;
      const char* vb = p_vb + (size_t)kv0 * v_pitch;
      if (kv0 + BN <= p_kv_len) {
#pragma unroll
        for (int j = 0; j < LPW; ++j) {
          const int ii = wave + WAVES * j;
          dma16s(ii < CHK ? kb : vb, ld_voff[j], stage + (uint32_t)ii * 1024);
        }
      } else {                                    // rows past the prompt re-read its last row
        const int last = p_kv_len - 1 - kv0;
#pragma unroll
        for (int j = 0; j < LPW; ++j) {
          const int ii = wave + WAVES * j;
          int row, coff;
          uint32_t pitch;
          slot_of(j, row, coff, pitch);
          dma16s(ii < CHK ? kb : vb, (uint32_t)min(row, last) * pitch + (uint32_t)coff, stage + (uint32_t)ii * 1024);
        }
      }
    }
    ++pt;
    if (++p_kt == p_n) {
      ++p_it;
      if (p_it < it_end) producer_item();
    } else if (PAGED && (p_win += BN / TILE_T) == 64) {
      load_window();
    }
  };

  // ---- LDS operand addresses (byte offsets inside a stage)
  // The tile loop is unrolled over the ring's stages so that the stage offset is part of each LDS
  // read's 16-bit immediate; stages 2 and 3 lie beyond its reach and get a second set of lane addresses.
  constexpr bool UNROLL = NSTAGE == 4 && 2 * STAGE_BYTES <= 65536;
  constexpr bool PAIRS = UNROLL;                // a ring of four holds the pair in use and the pair in flight
  static_assert(UNROLL || !PAGED, "pages are read a pair of tiles at a time");
  // K operand (S^T block b, k-step ks): row 32 b + n32, chunk 2 ks + hh.
  // (192 dims: the swizzle touches the low three bits of the chunk number only, so k-steps four apart differ by
  // 128 bytes and share a lane address; that frees eight registers)
  // V operand (16-key step kk, value block blk): two halves, 4 keys each.  Two transpose reads: in each group of 16 lanes
  // lane r supplies row (key) 4 hh + r / 4 and dims 4 (r % 4) .. + 3 of the group's 16 dims; the
  // hardware hands lane i of the group dim i of those 4 keys.
  // Out of pages both lie as the operands want them, chunk by chunk and in quads of tokens, and operands differ by constants: a lane
  // address each.  K: the token's 16 bytes.  V: consecutive 8 bytes per lane, so that row i of a block of 32 is its dim i / 2 + 16 (i % 2)
  // (with row i its dim i the reads have 2-way bank conflicts, 8 x 4096 tokens 9 % longer).  8-byte reads take the LDS twice as long as
  // transpose reads do, and the whole kernel up to 4 % longer than over dense rows.  (16-byte reads of a quad's dims m and m + 16, for two blocks at
  // once: their halves have to be sorted into operands, and long pieces take another 4 to 11 %.)
  constexpr int KOFFS = PAGED ? 1 : DQK == 192 ? 4 : KS, VOFFS = PAGED ? 1 : VB;
  int k_off[KOFFS], v_off[VOFFS];
  if constexpr (PAGED) {
    k_off[0] = (n32 >> 4) * UNIT_BYTES + hh * (TILE_T * 16) + (n32 & 15) * 16;
    v_off[0] = UNIT_K + lane * 8;
  } else {
#pragma unroll
    for (int ks = 0; ks < KOFFS; ++ks) k_off[ks] = n32 * (CHK * 16) + (((2 * ks + hh) ^ k_swz<DQK>(n32)) * 16);
    const int r16 = lane & 15;
    const int v_row = 4 * hh + (r16 >> 2);                       // plus 16 kk + 8 half
#pragma unroll
    for (int blk = 0; blk < VB; ++blk) {
      const int dim = 32 * blk + 16 * ((lane >> 4) & 1) + 4 * (r16 & 3);
      v_off[blk] = K_BYTES + v_row * (CHV * 16) + (((dim >> 3) ^ v_swz<DV>(v_row)) * 16) + (dim & 7) * 2;
    }
  }
  int k_off2[KOFFS], v_off2[VOFFS];
#pragma unroll
  for (int ks = 0; ks < KOFFS; ++ks) {
    k_off2[ks] = k_off[ks] + 2 * STAGE_BYTES;
    asm volatile("" : "+v"(k_off2[ks]));        // a value of its own, not "k_off + constant" to be recomputed
  }
#pragma unroll
  for (int blk = 0; blk < VOFFS; ++blk) {
    v_off2[blk] = v_off[blk] + 2 * STAGE_BYTES;
    asm volatile("" : "+v"(v_off2[blk]));
  }
  const uint32_t ones2 = 0x3f803f80u;           // (1.0, 1.0) in bf16

  int ct = 0;                                   // tiles consumed so far (tile number ct sits in stage ct % NSTAGE)
#pragma unroll
  for (int t = 0; t < (PAIRS ? 2 : PD); ++t) produce_one();

  // ---- state of the item being computed
  PrefillWork w;
  int kt_first = 0, kt_end = 0, part = -1;
  int h = 0, wave_q0 = 0, qi = 0, pos0 = 0, pos = 0, kt = 0;
  bool wave_active = false;
  bf16x8 qf[KS];                                // Q^T fragments (B operand: column = query, 8 consecutive dims per lane and k-step)
  f32x16 O[VB];
  float m = 0.f, l = 0.f;
  // The next item's query rows are touched ahead of time, one 128-byte line per lane, so that its fragment loads,
  // which nothing can overlap (every wave of the workgroup stands at the same item boundary), find them in the L2
  // instead of in HBM.  The touch goes out behind the first full wait of the item (a pair's barrier), so that it
  // has two tiles' time before the next one; the loaded word is never used, its register passes every full wait.
  uint32_t q_touch = 0;
  bool touch_next = false;
  auto touch_next_q = [&]() __attribute__((always_inline)) {
    const PrefillWork w2 = item_of(it + 1);
    constexpr int LINES = DQK / 64;               // 128-byte lines per query row
    int r2 = w2.q_tile * (32 * QS) + 32 * (wave / HB) + lane / LINES;
    r2 = r2 < w2.len ? r2 : w2.len - 1;
    const char* p2 = (const char*)(q + ((size_t)(w2.row0 + r2) * H + w2.head0 + wave % HB) * DQK) + (lane % LINES) * 128;
    asm volatile("global_load_dword %0, %1, off" : "=v"(q_touch) : "v"(p2) : "memory");
    touch_next = false;
  };
  auto item_begin = [&]() __attribute__((always_inline)) {
    if (ITEM_LANES && it - dsc_base >= 32) load_items(it);      // (the producer is past `it` and less than 32 items ahead)
    w = item_of(it);
    h = w.head0 + wave % HB;
    const int q_start = w.q_tile * (32 * QS);
    wave_q0 = q_start + 32 * (wave / HB);
    wave_active = wave_q0 < w.len;              // waves past the prompt's end only help loading
    qi = wave_q0 + n32;                         // this lane's query (row inside the request)
    const int qi_c = qi < w.len ? qi : w.len - 1;
    pos0 = w.q_off + wave_q0;                   // position of this wave's first query in the request
    // ... of this lane's query.  Out of pages lanes past the last row do as that row does (the keys behind it may be anything, and
    // one lane out of range moves the whole wave's references)
    pos = w.q_off + (PAGED ? qi_c : qi);
    const bf16_t* qp = q + ((size_t)(w.row0 + qi_c) * H + h) * DQK + 8 * hh;
#pragma unroll
    for (int s = 0; s < KS; ++s) qf[s] = __builtin_bit_cast(bf16x8, *(const uint4*)(qp + 16 * s));
    if constexpr (PARTS) {
      kt = kt_first = __builtin_amdgcn_readlane(d_kt0, it - dsc_base);
      kt_end = __builtin_amdgcn_readlane(d_kt1, it - dsc_base);
      part = __builtin_amdgcn_readlane(d_part, it - dsc_base);
    } else {
      kt_end = (min(w.q_off + w.len, w.q_off + q_start + 32 * QS) + BN - 1) / BN;
      kt = 0;
    }
#pragma unroll
    for (int i = 0; i < VB; ++i)
#pragma unroll
      for (int e = 0; e < 16; ++e) O[i][e] = 0.f;
    m = -INFINITY;
    l = 0.f;
    // Draw the compiler's wait for the Q loads to this point.  Left to itself it waits at their first
    // use, inside the tile, with a count that knows nothing of the tile loads issued by hand.
#pragma unroll
    for (int s = 0; s < KS; ++s) asm volatile("" ::"v"(__builtin_bit_cast(uint4, qf[s]).x));
    touch_next = ITEM_LANES && it + 1 < it_end;
  };
  auto item_end = [&]() __attribute__((always_inline)) {
    l += __shfl_xor(l, 32);
    if (PARTS && part >= 0) {
      // A part of an item: the sums as they are, register by register (1 KiB of consecutive bytes a time), and the softmax's
      // reference and row sums behind them, for prefill_merge_kernel.
      if (wave_active) {
        float* base = parts + (size_t)part * prefill_part_floats(DV) + wave * (DV * 32 + 64);
#pragma unroll
        for (int blk = 0; blk < VB; ++blk)
#pragma unroll
          for (int i4 = 0; i4 < 4; ++i4)
            *(f32x4*)(base + ((blk * 4 + i4) * 64 + lane) * 4) = f32x4{O[blk][4 * i4], O[blk][4 * i4 + 1], O[blk][4 * i4 + 2], O[blk][4 * i4 + 3]};
        if (hh == 0) *(f32x2*)(base + DV * 32 + 2 * n32) = f32x2{m, l};
      }
    } else
    // Output: a lane holds one query row in 8-byte bits, 8 KiB apart from its neighbour's.  Each wave
    // turns its block round, 32 dims at a time, in its own piece of LDS and writes 64-byte row pieces.
    if (wave_active) {
      char* ost = smem + NSTAGE * STAGE_BYTES + wave * (32 * OPITCH);
      const float inv = 1.f / l;
      bf16_t* obase = out + ((size_t)(w.row0 + wave_q0) * H + h) * DV;
      const int rows = min(32, w.len - wave_q0);
#pragma unroll
      for (int blk = 0; blk < VB; ++blk) {
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4) {
          const uint2 pk = out_pairs<PAGED>(O[blk][4 * i4] * inv, O[blk][4 * i4 + 1] * inv, O[blk][4 * i4 + 2] * inv, O[blk][4 * i4 + 3] * inv);
          stage_out<PAGED>(ost + n32 * OPITCH, 8 * i4 + 4 * hh, pk);
        }
#pragma unroll
        for (int itr = 0; itr < 2; ++itr) {       // 32 rows x 4 pieces of 16 bytes
          const int i = lane + 64 * itr;
          const int r = i >> 2, cc = i & 3;
          if (r < rows) *(uint4*)(obase + (size_t)r * H * DV + 32 * blk + cc * 8) = *(const uint4*)(ost + r * OPITCH + cc * 16);
        }
      }
    }
  };

  auto tile = [&](auto stc) __attribute__((always_inline)) {
    const int ST = stc;                         // ring stage of tile kt: a constant when the loop is unrolled
    const int kv0 = kt * BN;
    if constexpr (PAIRS) {
      // Tiles go in pairs: one wait and one barrier for two tiles, after which the waves run free
      // for two tiles' worth of work (the two waves of a SIMD drift apart, and one's matrix work
      // falls beside the other's softmax).  At the barrier the pair has landed and everyone is done
      // with the pair before, whose two stages are refilled, one now and one a tile later.
      if ((ST & 1) == 0) {
        SPD_WAIT_VMCNT(0);
        asm volatile("" : "+v"(q_touch));
        asm volatile("s_barrier" ::: "memory");
        produce_one();
        if (touch_next) touch_next_q();
      } else {
        produce_one();                          // the pair's second tile a tile later: eight loads at once queue up
      }
    } else {
      // this wave's loads of the tile are done when at most (tiles issued after it) * LPW remain
      const int later = pt - ct - 1;
      if (later >= 2) SPD_WAIT_VMCNT(2 * LPW);
      else if (later == 1) SPD_WAIT_VMCNT(LPW);
      else SPD_WAIT_VMCNT(0);
      // all waves: the tile has landed, and everyone is done with the one before, whose stage is refilled next
      asm volatile("s_barrier" ::: "memory");
      produce_one();
    }
    ++ct;
    if (!wave_active || kv0 > pos0 + 31) return;               // every key of the tile is in this wave's future

    const char* sbase = UNROLL ? smem + (ST & 1) * STAGE_BYTES : smem + ST * STAGE_BYTES;
    auto read_k = [&](int i) -> uint4 {
      const int ks = i / 2, b = i % 2;
      const int off = UNROLL && ST >= 2 ? k_off2[ks % KOFFS] : k_off[ks % KOFFS];
      if constexpr (PAGED) return *(const uint4*)(sbase + off + 2 * b * UNIT_BYTES + ks * (2 * TILE_T * 16));
      else return *(const uint4*)(sbase + off + (ks / KOFFS) * 128 + b * (32 * CHK * 16));
    };
    auto read_v = [&](int i, int half) -> s16x4 {
      const int kk = i / VB, blk = i % VB;
      const int off = UNROLL && ST >= 2 ? v_off2[blk % VOFFS] : v_off[blk % VOFFS];
      if constexpr (PAGED) return *(const s16x4*)(sbase + off + kk * UNIT_BYTES + blk * 1024 + half * 512);
      else return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(sbase + off + (16 * kk + 8 * half) * (CHV * 16)));
    };
    if constexpr (PAGED) {
      // Behind the request's last token the pages hold anything; p is 0 there, and so must V be.  Every wave sees to it itself, all to
      // the same effect, a lane for the 4 tokens of a dim that it reads itself.
      const int n = w.q_off + w.len - kv0;
      if (n < BN) {
        for (int g = n / 8; g < BN / 8; ++g) {        // 8 tokens, the first 4 in the lower half of the lanes
          char* p = smem + ST * STAGE_BYTES + v_off[0] + g / 2 * UNIT_BYTES + g % 2 * 512;
          uint2 x[VB];
          if (n > 8 * g) {
            const int keep = n - 8 * g - 4 * hh;
            const uint2 mask = {keep >= 2 ? ~0u : keep == 1 ? 0xffffu : 0u, keep >= 4 ? ~0u : keep == 3 ? 0xffffu : 0u};
#pragma unroll
            for (int blk = 0; blk < VB; ++blk) x[blk] = *(const uint2*)(p + blk * 1024);
#pragma unroll
            for (int blk = 0; blk < VB; ++blk) x[blk] = uint2{x[blk].x & mask.x, x[blk].y & mask.y};
          } else {
#pragma unroll
            for (int blk = 0; blk < VB; ++blk) x[blk] = uint2{0u, 0u};
          }
#pragma unroll
          for (int blk = 0; blk < VB; ++blk) *(uint2*)(p + blk * 1024) = x[blk];
        }
        asm volatile("" ::: "memory");
      }
    }

    // ---- S^T = K . Q^T.  Operand i: block b = i % 2 (32 keys), k-step ks = i / 2; LDS reads run
    // RING operands ahead of the MFMAs that consume them.
    __builtin_amdgcn_s_setprio(0);
    f32x16 S[2];
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int e = 0; e < 16; ++e) S[b][e] = 0.f;
    uint4 ring[RING];
#pragma unroll
    for (int i = 0; i < RING; ++i) ring[i] = read_k(i);
    __builtin_amdgcn_sched_barrier(0);          // keep the issue order below: the scheduler would
#pragma unroll                                  // otherwise sink every read next to its use
    for (int i = 0; i < NS; ++i) {
      S[i % 2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, ring[i % RING]), qf[i / 2], S[i % 2], 0, 0, 0);
      if (i + RING < NS) ring[i % RING] = read_k(i + RING);
      __builtin_amdgcn_sched_barrier(0);
    }
    // first V operands: in flight while the vector units do the softmax.  Operand j = 16-key step j / VB, value
    // block j % VB; a queue of VQ operands, read VAH ahead of the MFMA that takes them (a whole step ahead, two
    // steps' worth of registers; with 192 dims two operands ahead in a queue of three: registers are short there)
    constexpr int VAH = DQK > 128 ? 2 : VB, VQ = DQK > 128 ? VAH + 1 : 2 * VB;
    s16x4 vq[VQ][2];
#pragma unroll
    for (int j = 0; j < VAH; ++j) {
      vq[j][0] = read_v(j, 0);
      vq[j][1] = read_v(j, 1);
    }

    // lane holds, for the query at position pos, keys kv0 + 32b + 8*(i/4) + 4*hh + i%4
    if (kv0 + BN - 1 > pos0) {               // tile crosses this wave's diagonal (or the prompt's end)
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (kv0 + 32 * b + 8 * (i >> 2) + 4 * hh + (i & 3) > pos) S[b][i] = -INFINITY;
    }
    // p = exp2(S c - m c) against a reference m per query that need not be the running maximum: any
    // reference gives the same softmax as long as nothing overflows, and bf16 and fp32 keep their
    // relative precision over the whole exponent range.  So the tile's maximum is not computed at
    // all unless the row sum says that the reference is out of range (an item's first tile, where
    // m = -inf makes every p infinite or NaN, or a tile whose scores exceed the reference by 2^60):
    // then the reference moves to the true maximum, the accumulators are rescaled, and p is redone.
    // A wave's priority rises as it gets on with its tile: first product 0, softmax 3, second product 1.  The wave
    // that is further along is served first, so the two waves of a SIMD fall out of step instead of contending
    // phase by phase, and the softmax's vector instructions go out between the other wave's MFMAs (each of which
    // takes only a few issue cycles of the SIMD) instead of queueing behind them.
    __builtin_amdgcn_s_setprio(3);
    uint32_t pb[2][8];
    auto softmax_p = [&](float mc) -> float {
      float ls[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int i = 0; i < 16; i += 2) {
          const float p0 = __builtin_amdgcn_exp2f(S[b][i] * c - mc);
          const float p1 = __builtin_amdgcn_exp2f(S[b][i + 1] * c - mc);
          pb[b][i >> 1] = cvt_pk_bf16(p0, p1);
          // the row sum runs over the rounded values, the ones the second product multiplies: two per
          // instruction (the compiler places the wait states that a dot product's result needs).  As 4x4x4 MFMAs in the second
          // product, as in prefill_192_kernel: 8 x 4096 tokens of 64 heads on 128 CUs 3079 -> 3348 us.
          ls[(i >> 1) & 3] = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pb[b][i >> 1]),
                                                             __builtin_bit_cast(bf16x2, ones2), ls[(i >> 1) & 3], false);
        }
      return (ls[0] + ls[1]) + (ls[2] + ls[3]);
    };
    // (an item's first tile has no reference yet: the pass against it would be thrown away, so it is not made)
    float psum = INFINITY;
    if (kt != kt_first) psum = softmax_p(m * c);
    if (__builtin_amdgcn_ballot_w64(!(psum < 0x1p60f)) != 0) {
      float mx = S[0][0];
#pragma unroll
      for (int i = 1; i < 16; ++i) mx = fmaxf(mx, S[0][i]);
#pragma unroll
      for (int i = 0; i < 16; ++i) mx = fmaxf(mx, S[1][i]);
      {
        // the other half of the wave holds the other 32 keys of the same query: exchange on the
        // vector ALU (swap of the upper half of one register with the lower half of another;
        // written as machine code: the compiler's builtin for it loses the second result)
        float mx2 = mx;
        asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\ts_nop 1" : "+v"(mx), "+v"(mx2));
        mx = fmaxf(mx, mx2);
      }
      const float m_new = fmaxf(m, mx);
      // (a part of an item may begin with tiles whose scores are all -inf: they leave the sums at 0 and the reference where it is)
      const bool none = PARTS && m_new == -INFINITY;
      const float alpha = none ? 1.f : __builtin_amdgcn_exp2f((m - m_new) * c);
      l *= alpha;
#pragma unroll
      for (int blk = 0; blk < VB; ++blk)
#pragma unroll
        for (int e = 0; e < 16; ++e) O[blk][e] *= alpha;
      m = m_new;
      psum = softmax_p(none ? 0.f : m * c);
    }
    l += psum;
    __builtin_amdgcn_s_setprio(1);

    // ---- O^T += V^T . P^T : 16-key step kk multiplies with S^T block kk/2, registers 8*(kk%2) .. +7;
    // operand j + VAH is read while operand j multiplies
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int kk = 0; kk < BN / 16; ++kk) {
      const uint4 praw = uint4{pb[kk >> 1][4 * (kk & 1)], pb[kk >> 1][4 * (kk & 1) + 1], pb[kk >> 1][4 * (kk & 1) + 2],
                               pb[kk >> 1][4 * (kk & 1) + 3]};
#pragma unroll
      for (int blk = 0; blk < VB; ++blk) {
        const int j = kk * VB + blk;
        const uint2 lo = __builtin_bit_cast(uint2, vq[j % VQ][0]), hi = __builtin_bit_cast(uint2, vq[j % VQ][1]);
        const uint4 a = uint4{lo.x, lo.y, hi.x, hi.y};
        O[blk] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, praw),
                                                         O[blk], 0, 0, 0);
        if (j + VAH < (BN / 16) * VB) {
          vq[(j + VAH) % VQ][0] = read_v(j + VAH, 0);
          vq[(j + VAH) % VQ][1] = read_v(j + VAH, 1);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };


  // one tile of the chain; false when the chain is finished
  auto step = [&](auto stc) __attribute__((always_inline)) -> bool {
    tile(stc);
    if (++kt == kt_end) {
      item_end();
      if (++it >= it_end) return false;
      item_begin();
    }
    return true;
  };
  item_begin();
  if constexpr (UNROLL) {
    // the ring's stages in turn, each with its LDS offsets as immediates; items follow one another
    // without a break in the ring
    for (;;) {
      if (!step(std::integral_constant<int, 0>{})) break;
      if (!step(std::integral_constant<int, 1>{})) break;
      if (!step(std::integral_constant<int, 2>{})) break;
      if (!step(std::integral_constant<int, 3>{})) break;
    }
  } else {
    while (step(ct % NSTAGE)) {
    }
  }
}

// Items whose keys were shared out over several workgroups: one wave per (item, wave of the item, 32 dims) adds the parts up,
// each weighted with exp2((its reference - the largest one) c), and writes the rows as prefill_kernel does.
template <int DV, int HB, bool PAGED>
__global__ __launch_bounds__(256) void prefill_merge_kernel(bf16_t* __restrict__ out, const PrefillMerge* __restrict__ items, const float* __restrict__ parts,
                                                            int H, float c) {
  constexpr int QS = WAVES / HB, VB = DV / 32, OPITCH = 32 * 2 + 16;
  __shared__ __attribute__((aligned(16))) char smem[4 * 32 * OPITCH];
  const int tid = threadIdx.x, lane = tid & 63, n32 = lane & 31, hh = lane >> 5;
  const int unit = __builtin_amdgcn_readfirstlane((int)blockIdx.x * 4 + (tid >> 6));   // grid: exactly a wave per unit
  const int blk = unit % VB, wave = unit / VB % WAVES;
  const PrefillMerge it = items[unit / (VB * WAVES)];
  const int wave_q0 = it.q_tile * (32 * QS) + 32 * (wave / HB), rows = min(32, it.len - wave_q0);
  if (rows <= 0) return;
  const float* base = parts + (size_t)it.part0 * prefill_part_floats(DV) + wave * (DV * 32 + 64);
  float m = -INFINITY, l = 0.f;
  for (int p = 0; p < it.n_parts; ++p) m = fmaxf(m, base[p * prefill_part_floats(DV) + DV * 32 + 2 * n32]);
  float o[16];
#pragma unroll
  for (int e = 0; e < 16; ++e) o[e] = 0.f;
  for (int p = 0; p < it.n_parts; ++p) {
    const float* part = base + p * prefill_part_floats(DV);
    const f32x2 ml = *(const f32x2*)(part + DV * 32 + 2 * n32);
    const float f = __builtin_amdgcn_exp2f((ml.x - m) * c);
    l += ml.y * f;
#pragma unroll
    for (int i4 = 0; i4 < 4; ++i4) {
      const f32x4 v = *(const f32x4*)(part + ((blk * 4 + i4) * 64 + lane) * 4);
#pragma unroll
      for (int e = 0; e < 4; ++e) o[4 * i4 + e] += v[e] * f;
    }
  }
  char* ost = smem + (tid >> 6) * (32 * OPITCH);   // a piece of its own per wave
  const float inv = 1.f / l;
#pragma unroll
  for (int i4 = 0; i4 < 4; ++i4)
    stage_out<PAGED>(ost + n32 * OPITCH, 8 * i4 + 4 * hh, out_pairs<PAGED>(o[4 * i4] * inv, o[4 * i4 + 1] * inv, o[4 * i4 + 2] * inv, o[4 * i4 + 3] * inv));
  bf16_t* obase = out + ((size_t)(it.row0 + wave_q0) * H + it.head0 + wave % HB) * DV + 32 * blk;
#pragma unroll
  for (int itr = 0; itr < 2; ++itr) {
    const int i = lane + 64 * itr, r = i >> 2, cc = i & 3;
    if (r < rows) *(uint4*)(obase + (size_t)r * H * DV + cc * 8) = *(const uint4*)(ost + r * OPITCH + cc * 16);
  }
}

// ---- 192 / 128 dims (the un-absorbed heads of an MLA layer), where two_groups_pay (prefill_work.h) says that it is the faster one.
//
// The same contraction, tiles, operand orders and chains; what differs is how the two waves of a SIMD share it.  Waves w and
// w + 4 sit on one SIMD, and the two groups of four waves run half a tile apart, with an s_barrier at every change:
//   group 0:  | P.V of tile t - 1, K.Q of tile t | softmax of tile t, loads | P.V of tile t, ..
//   group 1:  | softmax of tile t - 1, loads     | P.V of t - 1, K.Q of t   | softmax of tile t, ..
// so that one wave of a SIMD feeds the matrix cores while the other one has the vector units.  With both waves taking a tile from
// end to end behind one barrier (prefill_kernel: three stages, registers for four K operands on the way) 4 prompts of 4096 tokens of
// 16 heads take 557 us on 128 CUs, here 490 (whole step on inputs of larger scores 658 / 532).  A matrix half takes about 1450 cycles (1280 of them 32x32x16 MFMAs), a vector half 1100 to 1300, an item's
// end about 3 us of both.  For 128 dims, whose tiles have a fifth fewer MFMAs for the same softmax, the order above it is
// the better one (2560 cycles per tile of both waves in either, but 5 instead of 7 us per item: 4 x 4096 tokens of 64 heads 1400 / 1460 us).
//
// v_dot2_f32_bf16 takes its turn in the matrix pipe: beside another wave's MFMAs one takes 72 cycles instead of 8, and a softmax
// with its row sum in dot products stands still.  The row sums are 4x4x4 MFMAs here, issued in the wave's own matrix half: with a first operand
// of ones every lane gets the sum of its own four bf16 values of p.
//
// The reference of the softmax lies 8 (in powers of two) above the largest score seen, so that p stays below 2 until a score exceeds
// that one by 9; the top exponent bit of any p tells (no sum, no maximum is formed to find out).
__global__ __launch_bounds__(512, 2) void prefill_192_kernel(const bf16_t* __restrict__ q, const bf16_t* __restrict__ k,
                                                             const bf16_t* __restrict__ v, bf16_t* __restrict__ out,
                                                             const PrefillWork* __restrict__ work,
                                                             const int32_t* __restrict__ chain, int H, int Hkv,
                                                             float c /* scale * log2(e) */) {
  constexpr int DQK = 192, DV = 128;
  constexpr int QS = WAVES;                     // 32-row sub-tiles per workgroup: every query head has keys of its own, a workgroup takes one
  constexpr int CHK = DQK / 8, CHV = DV / 8;    // 16-byte chunks per K / V row
  constexpr int K_BYTES = BN * DQK * 2, V_BYTES = BN * DV * 2;
  constexpr int NST = 3;                        // stages of the K ring and of the V ring
  constexpr int LK = CHK / WAVES, LV = CHV / WAVES;   // 1 KiB load instructions per wave for a K / V tile
  constexpr int KS = DQK / 16, VB = DV / 32;
  constexpr int NS = 2 * KS, NV = (BN / 16) * VB;     // MFMAs of either product
  constexpr int RING = 4, VAH = 2, VQ = VAH + 1;      // K operands, V operands on the way
  constexpr int OPITCH = 32 * 2 + 16;           // bytes per staged output row piece (32 dims, padded)
  constexpr int V_LDS = NST * K_BYTES, EPI_LDS = V_LDS + NST * V_BYTES;
  constexpr float ABOVE = 8.f;
  __shared__ __attribute__((aligned(1024))) char smem[EPI_LDS + WAVES * 32 * OPITCH];

  const int G = H / Hkv;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n32 = lane & 31, hh = lane >> 5;
  const uint32_t k_pitch = (uint32_t)Hkv * DQK * 2, v_pitch = (uint32_t)Hkv * DV * 2;
  const uint32_t smem_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem;
  int it = __builtin_amdgcn_readfirstlane(chain[blockIdx.x]);   // this workgroup's chain of work items
  const int it_end = __builtin_amdgcn_readfirstlane(chain[blockIdx.x + 1]);
  if (it >= it_end) return;

  // ---- tile loads: instruction wave + 8 j of a K (V) tile fills the 64 consecutive 16-byte slots from 64 (wave + 8 j) on; slot s
  // of a row holds the row's chunk s ^ swz(row).  K runs one tile ahead of V, which is needed one matrix half later.
  auto k_slot = [&](int j, int& row, int& coff) {
    const int slot = (wave + WAVES * j) * 64 + lane;
    row = slot / CHK;
    coff = ((slot % CHK) ^ k_swz<DQK>(row)) * 16;
  };
  auto v_slot = [&](int j, int& row, int& coff) {
    const int slot = (wave + WAVES * j) * 64 + lane;
    row = slot / CHV;
    coff = ((slot % CHV) ^ v_swz<DV>(row)) * 16;
  };
  uint32_t k_voff[LK], v_voff[LV];
#pragma unroll
  for (int j = 0; j < LK; ++j) {
    int row, coff;
    k_slot(j, row, coff);
    k_voff[j] = (uint32_t)row * k_pitch + (uint32_t)coff;
  }
#pragma unroll
  for (int j = 0; j < LV; ++j) {
    int row, coff;
    v_slot(j, row, coff);
    v_voff[j] = (uint32_t)row * v_pitch + (uint32_t)coff;
  }
  auto tiles_of = [&](const PrefillWork& pw) __attribute__((always_inline)) -> int {
    return (min(pw.q_off + pw.len, pw.q_off + pw.q_tile * (32 * QS) + 32 * QS) + BN - 1) / BN;
  };
  struct Producer { int it, kt, n, kv_len; const char* base; };   // the tile to be loaded next: kt of the n of item `it`
  Producer pk{it, 0, 0, 0, nullptr}, pv{it, 0, 0, 0, nullptr};
  auto producer_item = [&](Producer& p, bool is_k) __attribute__((always_inline)) {
    const PrefillWork pw = work[p.it];
    const size_t row = (size_t)pw.kv_row0 * Hkv + pw.head0 / G;
    p.kv_len = pw.q_off + pw.len;
    p.n = tiles_of(pw);
    p.base = is_k ? (const char*)(k + row * DQK) : (const char*)(v + row * DV);
    p.kt = 0;
  };
  producer_item(pk, true);
  producer_item(pv, false);
  auto advance = [&](Producer& p, bool is_k, uint32_t pitch) __attribute__((always_inline)) {
    p.base += (size_t)BN * pitch;
    if (__builtin_expect(++p.kt == p.n, 0)) {
      ++p.it;
      if (p.it < it_end) producer_item(p, is_k);
    }
  };
  auto load_k = [&](int stage) __attribute__((always_inline)) {
    if (__builtin_expect(pk.it >= it_end, 0)) return;
    const uint32_t lds = smem_base + stage * K_BYTES + wave * 1024;
    const int last = pk.kv_len - 1 - pk.kt * BN;
#pragma unroll
    for (int j = 0; j < LK; ++j) {
      if (__builtin_expect(last >= BN - 1, 1)) {
        dma16s(pk.base, k_voff[j], lds + j * (WAVES * 1024));
      } else {                                  // rows past the prompt re-read its last row
        int row, coff;
        k_slot(j, row, coff);
        dma16s(pk.base, (uint32_t)min(row, last) * k_pitch + (uint32_t)coff, lds + j * (WAVES * 1024));
      }
    }
    advance(pk, true, k_pitch);
  };
  auto load_v = [&](int stage) __attribute__((always_inline)) {
    if (__builtin_expect(pv.it >= it_end, 0)) return;
    const uint32_t lds = smem_base + V_LDS + stage * V_BYTES + wave * 1024;
    const int last = pv.kv_len - 1 - pv.kt * BN;
#pragma unroll
    for (int j = 0; j < LV; ++j) {
      if (__builtin_expect(last >= BN - 1, 1)) {
        dma16s(pv.base, v_voff[j], lds + j * (WAVES * 1024));
      } else {
        int row, coff;
        v_slot(j, row, coff);
        dma16s(pv.base, (uint32_t)min(row, last) * v_pitch + (uint32_t)coff, lds + j * (WAVES * 1024));
      }
    }
    advance(pv, false, v_pitch);
  };

  // ---- LDS operand addresses inside a stage, as in prefill_kernel; the stage is part of a read's immediate.  The swizzle touches
  // the low three bits of the chunk number only, so K steps four apart differ by 128 bytes and share a lane address.
  int k_off[4], v_off[VB];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) k_off[ks] = n32 * (CHK * 16) + (((2 * ks + hh) ^ k_swz<DQK>(n32)) * 16);
  const int r16 = lane & 15, v_row = 4 * hh + (r16 >> 2);
#pragma unroll
  for (int blk = 0; blk < VB; ++blk) {
    const int dim = 32 * blk + 16 * ((lane >> 4) & 1) + 4 * (r16 & 3);
    v_off[blk] = V_LDS + v_row * (CHV * 16) + (((dim >> 3) ^ v_swz<DV>(v_row)) * 16) + (dim & 7) * 2;
  }

  // ---- state of the item whose first product comes next, and of the tile between the halves
  PrefillWork w;
  int h = 0, wave_q0 = 0, pos0 = 0, pos = 0, n_kv_tiles = 0, kt = 0;
  bool wave_active = false, act = false, act_prev = false;   // has the wave keys in this tile, in the one before?
  bf16x8 qf[KS];
  f32x16 O[VB], S[2];
  uint32_t pb[2][8];
  f32x4 L;                                      // row sums: four times the same value
  float m;
  s16x4 vq[VQ][2];
  auto item_begin = [&]() __attribute__((always_inline)) {
    w = work[it];
    h = w.head0;
    const int q_start = w.q_tile * (32 * QS);
    wave_q0 = q_start + 32 * wave;
    wave_active = wave_q0 < w.len;              // waves past the prompt's end only help loading
    const int qi = wave_q0 + n32, qi_c = qi < w.len ? qi : w.len - 1;
    pos0 = w.q_off + wave_q0;
    pos = w.q_off + qi;
    const bf16_t* qp = q + ((size_t)(w.row0 + qi_c) * H + h) * DQK + 8 * hh;
    // (loads and wait in one piece: loads that the compiler knows of it counts, and waits for, in the middle of every tile)
    asm volatile("global_load_dwordx4 %0, %12, off\n\tglobal_load_dwordx4 %1, %12, off offset:32\n\tglobal_load_dwordx4 %2, %12, off offset:64\n\t"
                 "global_load_dwordx4 %3, %12, off offset:96\n\tglobal_load_dwordx4 %4, %12, off offset:128\n\tglobal_load_dwordx4 %5, %12, off offset:160\n\t"
                 "global_load_dwordx4 %6, %12, off offset:192\n\tglobal_load_dwordx4 %7, %12, off offset:224\n\tglobal_load_dwordx4 %8, %12, off offset:256\n\t"
                 "global_load_dwordx4 %9, %12, off offset:288\n\tglobal_load_dwordx4 %10, %12, off offset:320\n\tglobal_load_dwordx4 %11, %12, off offset:352\n\t"
                 "s_waitcnt vmcnt(0)"
                 : "=&v"(qf[0]), "=&v"(qf[1]), "=&v"(qf[2]), "=&v"(qf[3]), "=&v"(qf[4]), "=&v"(qf[5]), "=&v"(qf[6]), "=&v"(qf[7]), "=&v"(qf[8]),
                   "=&v"(qf[9]), "=&v"(qf[10]), "=&v"(qf[11])
                 : "v"(qp)
                 : "memory");
    n_kv_tiles = tiles_of(w);
    kt = 0;
  };
  auto reset_sums = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < VB; ++i)
#pragma unroll
      for (int e = 0; e < 16; ++e) O[i][e] = 0.f;
    m = -INFINITY;
    L = f32x4{0.f, 0.f, 0.f, 0.f};
  };
  bf16_t* o_base = nullptr;                     // the item that O belongs to: its first row of this wave, and how many there are
  int o_rows = 0;
  auto finish_item = [&]() __attribute__((always_inline)) {
    float l = L[0];
    l += __shfl_xor(l, 32);
    if (o_rows > 0) {
      char* ost = smem + EPI_LDS + wave * (32 * OPITCH);
      const float inv = 1.f / l;
#pragma unroll
      for (int blk = 0; blk < VB; ++blk) {
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4) {
          uint2 y;
          y.x = cvt_pk_bf16(O[blk][4 * i4] * inv, O[blk][4 * i4 + 1] * inv);
          y.y = cvt_pk_bf16(O[blk][4 * i4 + 2] * inv, O[blk][4 * i4 + 3] * inv);
          *(uint2*)(ost + n32 * OPITCH + (8 * i4 + 4 * hh) * 2) = y;
        }
#pragma unroll
        for (int itr = 0; itr < 2; ++itr) {     // 32 rows x 4 pieces of 16 bytes
          const int i = lane + 64 * itr;
          const int r = i >> 2, cc = i & 3;
          if (r < o_rows) *(uint4*)(o_base + (size_t)r * H * DV + 32 * blk + cc * 8) = *(const uint4*)(ost + r * OPITCH + cc * 16);
        }
      }
    }
  };
  auto barrier = [&]() __attribute__((always_inline)) {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  // Oᵀ += Vᵀ.Pᵀ of the tile in V stage `stage`; operand j + VAH is read while operand j multiplies, `beside(j)` after each of them
  auto second_product = [&](int stage, auto beside) __attribute__((always_inline)) {
    auto read_v = [&](int j, int half) __attribute__((always_inline)) -> s16x4 {
      return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(
          smem + v_off[j % VB] + stage * V_BYTES + (16 * (j / VB) + 8 * half) * (CHV * 16)));
    };
    const s16x4 ones = {0x3f80, 0x3f80, 0x3f80, 0x3f80};
#pragma unroll
    for (int j = 0; j < VAH; ++j) {
      vq[j][0] = read_v(j, 0);
      vq[j][1] = read_v(j, 1);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      const int kk = j / VB, blk = j % VB;
      const uint4 p = uint4{pb[kk >> 1][4 * (kk & 1)], pb[kk >> 1][4 * (kk & 1) + 1], pb[kk >> 1][4 * (kk & 1) + 2], pb[kk >> 1][4 * (kk & 1) + 3]};
      if (blk < 2) L = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(ones, __builtin_bit_cast(s16x4, blk ? uint2{p.z, p.w} : uint2{p.x, p.y}), L, 0, 0, 0);
      const uint2 lo = __builtin_bit_cast(uint2, vq[j % VQ][0]), hi = __builtin_bit_cast(uint2, vq[j % VQ][1]);
      O[blk] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, uint4{lo.x, lo.y, hi.x, hi.y}), __builtin_bit_cast(bf16x8, p),
                                                       O[blk], 0, 0, 0);
      if (j + VAH < NV) {
        vq[(j + VAH) % VQ][0] = read_v(j + VAH, 0);
        vq[(j + VAH) % VQ][1] = read_v(j + VAH, 1);
      }
      beside(j);
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  // K of tiles 0, 1 and V of tile 0, as the vector halves before the first one would load them
  load_k(0);
  load_k(1);
  load_v(0);
  item_begin();                                 // (waits for all of it)
  reset_sums();
  const bool second_group = wave >= WAVES / 2;
  barrier();
  if (second_group) barrier();                  // half a tile behind

  // tile number g of the chain, stage g % 3; false behind the last one
  auto step = [&](auto stc) __attribute__((always_inline)) -> bool {
    constexpr int ST = stc, PREV = (ST + NST - 1) % NST;
    auto read_k = [&](int i) __attribute__((always_inline)) -> uint4 {   // operand i: block i % 2 (32 keys), k-step i / 2
      return *(const uint4*)(smem + k_off[(i / 2) % 4] + ST * K_BYTES + ((i / 2) / 4) * 128 + (i % 2) * (32 * CHK * 16));
    };
    const int kv0 = kt * BN;
    uint4 ring[RING];
    act = wave_active && kv0 <= pos0 + 31;      // else every key of the tile is in this wave's future

    // ---- matrix half: the second product of the tile before, the first product of this one
    __builtin_amdgcn_s_setprio(1);
    if (__builtin_expect(act_prev, 1)) {
      second_product(PREV, [&](int j) __attribute__((always_inline)) {
        if (j >= NV - RING) ring[j - (NV - RING)] = read_k(j - (NV - RING));
      });
    } else {
#pragma unroll
      for (int i = 0; i < RING; ++i) ring[i] = read_k(i);
    }
    if (__builtin_expect(act, 1)) {
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int e = 0; e < 16; ++e) S[b][e] = 0.f;
#pragma unroll
      for (int i = 0; i < NS; ++i) {
        S[i % 2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, ring[i % RING]), qf[i / 2], S[i % 2], 0, 0, 0);
        if (i + RING < NS) ring[i % RING] = read_k(i + RING);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    __builtin_amdgcn_s_setprio(0);
    // What the vector half before loaded, K of tile g + 1 and V of tile g, has landed (the other group's next matrix half but
    // one and this wave's next one read it).
    SPD_WAIT_VMCNT(0);
    barrier();

    // ---- vector half
    const bool first = kt == 0, last = kt + 1 == n_kv_tiles, more = it + 1 < it_end;
    if (__builtin_expect(first, 0)) {           // the second product of the item before is complete
      if (o_base) {
        finish_item();
        reset_sums();
      }
      o_base = out + ((size_t)(w.row0 + wave_q0) * H + h) * DV;
      o_rows = wave_active ? min(32, w.len - wave_q0) : 0;
    }
    const int tile_pos0 = pos0, tile_pos = pos;
    ++kt;
    if (__builtin_expect(last && more, 0)) {    // the next first product is the next item's
      ++it;
      item_begin();
    }
    // K of tile g + 2 into the stage of tile g - 1, V of tile g + 1 into the stage of tile g - 2: both groups are done with those.
    // Inside an item the loads go between the groups of the softmax, so that the four waves' do not queue up in the address unit.
    const bool spread = act && !first && pk.it < it_end && pv.it < it_end && pk.kt + 1 < pk.n && pv.kt + 1 < pv.n;
    constexpr int K_ST = (ST + 2) % NST, V_ST = (ST + 1) % NST;
    if (__builtin_expect(!spread, 0)) {
      load_k(K_ST);
      load_v(V_ST);
    }
    auto load_piece = [&](int n) __attribute__((always_inline)) {   // n of 4: whole tiles, not their items' last ones
      if (!spread) return;
      const uint32_t lk = smem_base + K_ST * K_BYTES + wave * 1024, lv = smem_base + V_LDS + V_ST * V_BYTES + wave * 1024;
#pragma unroll
      for (int j = 0; j < LK; ++j)
        if (j * 2 / LK == n) dma16s(pk.base, k_voff[j], lk + j * (WAVES * 1024));
#pragma unroll
      for (int j = 0; j < LV; ++j)
        if (2 + j * 2 / LV == n) dma16s(pv.base, v_voff[j], lv + j * (WAVES * 1024));
      if (n == 3) {
        pk.base += (size_t)BN * k_pitch;
        pv.base += (size_t)BN * v_pitch;
        ++pk.kt;
        ++pv.kt;
      }
    };
    if (__builtin_expect(act, 1)) {
      // lane holds, for the query at position tile_pos, keys kv0 + 32b + 8*(i/4) + 4*hh + i%4
      if (__builtin_expect(kv0 + BN - 1 > tile_pos0, 0)) {   // tile crosses this wave's diagonal (or the prompt's end)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
          for (int i = 0; i < 16; ++i)
            if (kv0 + 32 * b + 8 * (i >> 2) + 4 * hh + (i & 3) > tile_pos) S[b][i] = -INFINITY;
      }
      // p = exp2(S c - mc) in pb; is any of them 2 or more, infinite or NaN?
      auto softmax_p = [&](float mc, bool loads) __attribute__((always_inline)) -> bool {
        uint32_t any = 0;
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
          for (int i = 0; i < 16; i += 4) {
#pragma unroll
            for (int e = i; e < i + 4; e += 2)
              pb[b][e >> 1] = cvt_pk_bf16(__builtin_amdgcn_exp2f(S[b][e] * c - mc), __builtin_amdgcn_exp2f(S[b][e + 1] * c - mc));
            any = any | pb[b][i >> 1] | pb[b][(i >> 1) + 1];
            const int u = b * 4 + i / 4;
            if (loads && (u & 1)) {
              __builtin_amdgcn_sched_barrier(0);
              load_piece(u >> 1);
              __builtin_amdgcn_sched_barrier(0);
            }
          }
        return (any & 0x40004000u) != 0;        // the top exponent bits
      };
      // an item's first tile has no reference yet; else the reference moves where a p is too large
      bool move = true;
      if (__builtin_expect(!first, 1)) move = softmax_p(m * c + ABOVE, true);
      if (__builtin_expect(__builtin_amdgcn_ballot_w64(move) != 0, 0)) {
        float mx = S[0][0];
#pragma unroll
        for (int i = 1; i < 16; ++i) mx = fmaxf(mx, S[0][i]);
#pragma unroll
        for (int i = 0; i < 16; ++i) mx = fmaxf(mx, S[1][i]);
        {
          float mx2 = mx;                       // the other half's 32 keys of the same query (see prefill_kernel)
          asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\ts_nop 1" : "+v"(mx), "+v"(mx2));
          mx = fmaxf(mx, mx2);
        }
        const float m_new = fmaxf(m, mx);
        const float alpha = __builtin_amdgcn_exp2f((m - m_new) * c);
#pragma unroll
        for (int e = 0; e < 4; ++e) L[e] *= alpha;
#pragma unroll
        for (int blk = 0; blk < VB; ++blk)
#pragma unroll
          for (int e = 0; e < 16; ++e) O[blk][e] *= alpha;
        m = m_new;
        softmax_p(m * c + ABOVE, false);
      }
    }
    act_prev = act;
    barrier();
    if (__builtin_expect(last && !more, 0)) {
      if (act_prev) second_product(ST, [](int) {});
      return false;
    }
    return true;
  };
  for (;;) {
    if (!step(std::integral_constant<int, 0>{})) break;
    if (!step(std::integral_constant<int, 1>{})) break;
    if (!step(std::integral_constant<int, 2>{})) break;
  }
  if (!second_group) barrier();                 // as many as the second group
  finish_item();
}

bool prefill_shape_supported(int dqk, int dv) {
  return (dqk == 64 && dv == 64) || (dqk == 128 && dv == 128) || (dqk == 192 && dv == 128);
}

// Query heads of one KV head that share a workgroup: the largest of 8, 4, 2, 1 dividing the group size.
int prefill_heads_per_block(int group) {
  for (int hb = WAVES; hb > 1; hb >>= 1)
    if (group % hb == 0) return hb;
  return 1;
}
int prefill_block_m(int group) { return 32 * (WAVES / prefill_heads_per_block(group)); }

// (Pages: the instance that takes parts also where there are none.)
template <int DQK, int DV, int HB>
static void launch_items(dim3 grid, hipStream_t stream, const bf16_t* q, const bf16_t* k, const bf16_t* v, bf16_t* out, const PrefillLists& d, int H,
                         int Hkv, float c) {
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, dim3(64 * WAVES), 0, stream, q, k, v, d.pages, d.units, d.head_units, out, d.work, d.chain, H, Hkv, c, d.range, d.parts);
  };
  auto merge = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)(d.n_merge * WAVES * (DV / 32) / 4)), dim3(256), 0, stream, out, d.merge, d.parts, H, c);
  };
  if constexpr (DQK <= 128) {
    if (d.pages) {
      launch(prefill_kernel<DQK, DV, HB, true, true>);
      if (d.n_merge) merge(prefill_merge_kernel<DV, HB, true>);
      return;
    }
    if (d.n_merge) {
      launch(prefill_kernel<DQK, DV, HB, true, false>);
      merge(prefill_merge_kernel<DV, HB, false>);
      return;
    }
  }
  launch(prefill_kernel<DQK, DV, HB, false, false>);
}

template <int DQK, int DV>
static void launch_hb(int hb, dim3 grid, hipStream_t stream, const bf16_t* q, const bf16_t* k, const bf16_t* v, bf16_t* out, const PrefillLists& d, int H,
                      int Hkv, float c) {
  if (hb == 8) launch_items<DQK, DV, 8>(grid, stream, q, k, v, out, d, H, Hkv, c);
  else if (hb == 4) launch_items<DQK, DV, 4>(grid, stream, q, k, v, out, d, H, Hkv, c);
  else if (hb == 2) launch_items<DQK, DV, 2>(grid, stream, q, k, v, out, d, H, Hkv, c);
  else launch_items<DQK, DV, 1>(grid, stream, q, k, v, out, d, H, Hkv, c);
}

hipError_t launch_prefill(const void* q, const void* k, const void* v, void* out, const PrefillLists& d, bool two_groups, int H, int Hkv, int dqk, int dv,
                          float scale, hipStream_t stream) {
  const float c = scale * 1.4426950408889634f;
  const int hb = prefill_heads_per_block(H / Hkv);
  const dim3 grid((unsigned)d.n_blocks);
  const bf16_t *qq = (const bf16_t*)q, *kk = (const bf16_t*)k, *vv = (const bf16_t*)v;
  if (dqk == 64 && dv == 64) launch_hb<64, 64>(hb, grid, stream, qq, kk, vv, (bf16_t*)out, d, H, Hkv, c);
  else if (dqk == 128 && dv == 128) launch_hb<128, 128>(hb, grid, stream, qq, kk, vv, (bf16_t*)out, d, H, Hkv, c);
  else if (dqk != 192 || dv != 128 || hb != 1) return hipErrorInvalidValue;   // (192 / 128: a latent layer's heads, each with keys of its own)
  else if (two_groups)
    hipLaunchKernelGGL(prefill_192_kernel, grid, dim3(64 * WAVES), 0, stream, qq, kk, vv, (bf16_t*)out, d.work, d.chain, H, Hkv, c);
  else launch_items<192, 128, 1>(grid, stream, qq, kk, vv, (bf16_t*)out, d, H, Hkv, c);
  return hipGetLastError();
}

}  // namespace spd
