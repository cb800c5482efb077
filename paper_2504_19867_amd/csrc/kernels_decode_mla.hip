// Decode step, MLA latent cache (DeepSeek-V2-style multi-head latent attention, absorbed form).
//
// Paper, Evaluation "Model": DeepSeek-V2-Lite / V3 are served through the same two workers; the
// paper names the model only.  Per token the cache holds ONE latent row c_t = [ckv_t (512) ;
// krope_t (64)] shared by all heads.  For request b and head h with absorbed query q[b,h,:576]:
//     s[h,t]      = scale * q[b,h,:] . c_t
//     out[b,h,:]  = sum_{t<n} softmax_t(s[h,:]) * c_t[0:512]
// so the same bytes act as keys (contraction over the 576 dims) and as values (contraction over
// the tokens).  34.8 kflop per 1152-byte row: the fp32 vector units cannot keep up with HBM, the
// matrix cores must; the heads (<= 16) are the MFMA column dimension.
//
// Bound: HBM, every cached row is read once.  One workgroup (4 waves, two workgroups per compute unit) owns one
// (request, chunk of the context); every wave takes tiles of 16 tokens (every fourth tile of the chunk) and does
// all there is to do with a tile by itself: HBM -> an LDS stage with global_load_lds_dwordx4, scores, softmax,
// value product for all 512 dims.  There is no barrier in the loop, no
// score is computed twice, and the waves drift apart: while some wait for their tiles, others compute.  With bf16 pages they share
// nothing (one stage per wave, 18 KiB each, 147 KiB per compute unit), with FP8 pages the stages (below).  A read-only loop of this shape takes 5.5 TB/s out of 128 compute
// units (half as many waves with two stages each: 4.8).  128 requests of 1024 .. 8192 tokens on 128 compute units, whole step: 149
// us, 4.7 TB/s (FP8 93 us); with a barrier-coupled ring of four stages, in which every wave computed the scores of all tokens, 169
// (242).
// What a chunk costs beyond its tiles (record, queries, first tile: 9 us; merge of the waves: 6 us) is covered by the
// other workgroup of the compute unit: as one workgroup of eight waves the same loop took 174 us at a batch of 128 requests
// of 1024 .. 8192 tokens on 128 compute units.
// Out of LDS a tile is read twice, in the two operand orders:
//     S^T[token, head] = C[16 x 576] . Q^T[576 x 16]      ds_read_b128       + v_mfma_f32_16x16x32_bf16
//     O^T[dim, head]  += C^T[16 dims x 16 tokens] . P^T    ds_read_b64_tr_b16 + v_mfma_f32_16x16x16_bf16
// The waves' (m, l, O) meet in LDS at the end of the chunk, half of the dims at a time.
//
// FP8 pages (656-byte rows: 512 E4M3 codes, 4 fp32 scales, 64 bf16 rope entries; kernels_kv_fp8.hip) go to LDS as they
// are.  Codes become bf16 on their way out of LDS (exact; two per instruction), the scales stay out of the
// operands: one score accumulator per block of 128 dims, summed with the tokens' scales in fp32, and the softmax weights
// multiplied with them per block.  ds_read_b64_tr_b8 hands a lane 8 rows of one dim: four tokens of a dim and the
// same four of the dim 16 further on, the operands of two products.  An FP8 tile is 10.25 KiB and its conversions keep the vector
// ALU as long as HBM its loads (the batch above without the in-loop loads 79 us, without the arithmetic 84), so the two have to run side by
// side: a workgroup's LDS holds seven stages, which its tiles pass round in order, and a wave loads its next tile while it consumes
// one, into the stage of the tile three before (the next wave's, which says in LDS when it has done with it; a wave only
// ever waits for an earlier tile).  115 -> 96 us together with fewer rescalings of O (8 us of it).  Loads that bring a tile's codes apart from its
// scales and rope entries, so that two stages per wave would fit, are pieces of 512 bytes across cache lines: 115 us without any
// arithmetic.  Scores as FP8 products, the queries as sums of two codes: no conversions, but longer chains, 104 us.
//
// The launch is the whole step: it rotates the query heads (RoPE), and the wave that holds the request's last
// tile rotates or quantises the new token's row, puts it into its page and into the tile in LDS.
#include "internal.h"
#include "fp8_row.h"
#include "rope_device.h"
#include "split_merge.h"

namespace spd {

typedef unsigned short bf16_t;
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef int i32x2 __attribute__((ext_vector_type(2)));

namespace mla {
constexpr int DL = 576;               // latent dims per token
constexpr int DV = 512;               // leading dims that act as values
constexpr int ROW_BYTES = DL * 2;     // 1152
constexpr int CH = DL / 8;            // 72 16-byte chunks per row
constexpr int TILE = 16;              // tokens per tile
constexpr int WAVES = MLA_THREADS / 64;
constexpr int KS = DL / 32;           // 18 k-steps of the score product
constexpr int VB = DV / 16;           // 32 value blocks of 16 dims
constexpr int HALF_PITCH = DV / 2 + 4;   // floats per (wave, head) of a half of O in the merge, padded
constexpr int MERGE_BYTES = WAVES * 16 * HALF_PITCH * 4;
template <bool FP8> constexpr int tile_bytes() { return FP8 ? TILE * FP8_ROW_BYTES : TILE * ROW_BYTES; }
template <bool FP8> constexpr int loads() { return tile_bytes<FP8>() / 1024; }    // 1 KiB load instructions: 18, 10 (and one of 256 bytes)
}  // namespace mla

struct MlaArgs {
  char* pool;
  uint64_t page_bytes;
  int tiles_per_page;
  const bf16_t *q, *k_new;
  bf16_t* out;
  const char* items;
  int item_stride, H;
  float c;                      // scale * log2(e)
  int max_chunks;
  const double* w;
  int rot, off, interleaved;
  float *ws_o, *ws_ml;
  int32_t* put_chunks;
  StepMark mark;
};

__device__ inline uint32_t mla_pack_bf16(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));
}
// 16 bytes per lane from global memory to LDS (lane i's land at lds_byte_addr + 16 i), non-temporal: a decode step reads
// every latent row once, and the L2 is shared with the prefill partition.  The compiler does not see the write to LDS.
__device__ inline void mla_dma16s(const void* sbase, uint32_t voff, uint32_t lds_byte_addr) {
  asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2 nt" ::"s"(lds_byte_addr), "v"(voff), "s"(sbase) : "memory");
}
// the same with 4 bytes per lane
__device__ inline void mla_dma4s(const void* sbase, uint32_t voff, uint32_t lds_byte_addr) {
  asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dword %1, %2 nt" ::"s"(lds_byte_addr), "v"(voff), "s"(sbase) : "memory");
}
// max over the four 16-lane rows of a wave, on the vector ALU: the row swaps exchange odd rows of
// the first register with even rows of the second (rows of 16, then of 32 lanes)
__device__ inline float mla_max_over_rows(float x) {
  float y = x;
  asm volatile("s_nop 1\n\tv_permlane16_swap_b32 %0, %1\n\ts_nop 1" : "+v"(x), "+v"(y));
  x = fmaxf(x, y);
  y = x;
  asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\ts_nop 1" : "+v"(x), "+v"(y));
  return fmaxf(x, y);
}
__device__ inline void mla_lds_visible_in_wave() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}
// two E4M3 codes of a word (its low or high half) as two bf16: exact
template <bool HI> __device__ inline uint32_t mla_codes_to_bf16(uint32_t w) {
  return __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w, 1.0f, HI));
}

// grid (n_wgs), block 256: workgroup i computes the chunk of record i, then those its record's `next` leads to.
template <bool FP8>
__global__ __launch_bounds__(64 * mla::WAVES, 2) void decode_mla_kernel(MlaArgs a) {
  using namespace mla;
  constexpr int NL = loads<FP8>(), TB = tile_bytes<FP8>(), STAGE = TB;
  static_assert(TB == NL * 1024 + (FP8 ? 256 : 0), "whole load instructions");
  constexpr int STAGES = FP8 ? 7 : WAVES;          // (as many as two workgroups' LDS holds)
  constexpr int SMEM = STAGES * STAGE > MERGE_BYTES ? STAGES * STAGE : MERGE_BYTES;
  __shared__ __attribute__((aligned(1024))) char smem[SMEM];
  __shared__ float sm_m[WAVES + 1][16], sm_l[WAVES][16];
  __shared__ float sm_cs[128], sm_sn[128];         // rotary_dim <= 256
  __shared__ int32_t sm_rec[64 * WAVES];           // header and page ids, a word per thread
  __shared__ __attribute__((aligned(16))) char sm_new[FP8 ? FP8_ROW_BYTES : ROW_BYTES];
  __shared__ uint4 sm_q[FP8 ? 2 : 1][64];          // FP8: the rope entries' query fragments (registers are full)
  __shared__ int sm_done[WAVES];                   // FP8: tiles that a wave has finished with
  if (blockIdx.x == 0 && threadIdx.x == 0) store_mark(a.mark);
  static_assert(DECODE_ITEM_WORDS + MLA_CHUNK_PAGES <= 64 * WAVES, "one thread per word of a record");
  const int words = a.item_stride >> 2;
  // Two workgroups per compute unit share the batch's tiles evenly, so a workgroup may go from one request's last tiles to
  // the next one's first: its chain of chunks
  for (int idx = blockIdx.x, rec_word = 0, first = 1;;) {
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));                    // what follows from it is made anew for every item: registers are full
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 15, c4 = lane >> 4;       // col: head (B operand / accumulator column) or token (A operand row)
  // the record (header, page ids) once per workgroup: it may lie in pinned host memory
  const bool has_word = tid < words;
  if (first && has_word) rec_word = ((const int32_t*)(a.items + (size_t)idx * a.item_stride))[tid];
  if (has_word) sm_rec[tid] = rec_word;
  if (FP8 && tid < WAVES) sm_done[tid] = 0;
  __syncthreads();
  first = 0;
  const int b = __builtin_amdgcn_readfirstlane(sm_rec[0]), chunk = __builtin_amdgcn_readfirstlane(sm_rec[1]);
  const int n_chunks = __builtin_amdgcn_readfirstlane(sm_rec[2]), n = __builtin_amdgcn_readfirstlane(sm_rec[3]);
  if (a.put_chunks && chunk == 0 && tid == 0) a.put_chunks[b] = n_chunks;
  const int tile0 = __builtin_amdgcn_readfirstlane(sm_rec[4]), n_tiles = __builtin_amdgcn_readfirstlane(sm_rec[5]);
  const int n_tiles_all = (n + TILE - 1) / TILE;
  const int page0 = tile0 / a.tiles_per_page;
  auto tile_addr = [&](int t) -> char* {           // t: tile of the chunk
    const int gt = tile0 + t, pg = gt / a.tiles_per_page;
    const int page = __builtin_amdgcn_readfirstlane(sm_rec[pg - page0 + DECODE_ITEM_WORDS]);
    return a.pool + (uint64_t)(uint32_t)page * a.page_bytes + (uint32_t)(gt - pg * a.tiles_per_page) * (uint32_t)TB;
  };

  // ---- tile loads: instruction j fills LDS slots [64 j, 64 j + 64) of the stage, 16 bytes each.  bf16 rows are 72
  // slots, slot s of row r holds the row's chunk s ^ (r & 7) (bank conflicts); nine instructions are eight rows, so
  // instruction j + 9 has j's pattern eight rows on.  FP8 rows lie as in the page (their pitch spreads over the banks).
  constexpr int NV = FP8 ? 1 : 9;
  uint32_t ld_off[NV];
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    const int slot = 64 * j + lane, row = slot / CH, sl = slot % CH;
    ld_off[j] = FP8 ? (uint32_t)lane * 16 : (uint32_t)(row * ROW_BYTES + ((sl ^ (row & 7)) * 16));
  }
  const uint32_t smem_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem;
  int at = wave;                                   // the tile's stage
  auto load_tile = [&](const char* src, int to) __attribute__((always_inline)) {
    const uint32_t stage_base = smem_base + (uint32_t)to * STAGE;
#pragma unroll
    for (int j = 0; j < NL; ++j) {
      if constexpr (FP8) {
        mla_dma16s(src + j * 1024, ld_off[0], stage_base + (uint32_t)j * 1024);
      } else {
        mla_dma16s(src + (j / 9) * (8 * ROW_BYTES), ld_off[j % 9], stage_base + (uint32_t)j * 1024);
      }
    }
    if constexpr (FP8) mla_dma4s(src + NL * 1024, ld_off[0] >> 2, stage_base + NL * 1024);
  };

  const bool interleaved = a.interleaved != 0;
  // the new token's row goes into its page and into the request's last tile
  const bool appends = a.k_new != nullptr && tile0 + n_tiles == n_tiles_all;
  // (the first tile's loads go out behind the queries': loads return in order, and the queries are needed first)
  // absorbed-query fragments: B operand, column = head, dims 8 (4 s + c4) .. + 7 for k-step s
  constexpr int KR = FP8 ? KS - 2 : KS;            // fragments in registers
  bf16x8 qf[KR];
  {
    const bf16_t* qrow = a.q + ((size_t)b * a.H + min(col, a.H - 1)) * DL;
    uint4 raw[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) raw[s] = *(const uint4*)(qrow + 8 * (4 * s + c4));
    __builtin_amdgcn_sched_barrier(0);
    if (wave < n_tiles) load_tile(tile_addr(wave), wave);
    __builtin_amdgcn_sched_barrier(0);

    // ---- rotation angles of the step's position; same arithmetic as the RoPE step
    if constexpr (!FP8) {
      if (a.rot) {
        if (tid < (a.rot >> 1)) {
          const double turns = (double)(n - 1) * a.w[tid] * 0.15915494309189535;
          const float ang = (float)((turns - __builtin_rint(turns)) * 6.283185307179586);
          sincosf(ang, &sm_sn[tid], &sm_cs[tid]);
        }
        __syncthreads();
      }
    }
    // ---- the new token's row, where the request's last tile is: into the page, and into LDS, from where it goes into the
    // tile once that is there
    if (appends) {
      if (wave == WAVES - 1) {
      const bf16_t* row_new = a.k_new + (size_t)b * DL;
      char* dst = tile_addr(n_tiles - 1) + ((n - 1) % TILE) * (FP8 ? FP8_ROW_BYTES : ROW_BYTES);
      if constexpr (FP8) {
        if (lane < 16) {
          Fp8Piece p;
          fp8_quantise(row_new, lane, p);
          fp8_store_row(dst, row_new, lane, p);
          fp8_store_row(sm_new, row_new, lane, p);
        }
      } else {
        for (int pc = lane; pc < CH; pc += 64) {
          uint4 piece = *(const uint4*)(row_new + 8 * pc);
          if (a.rot) {
            const uint4 oth = *(const uint4*)(row_new + rope_partner(8 * pc, a.off, a.rot, interleaved));
            piece = rope_rotate(piece, oth, 8 * pc, a.off, a.rot, interleaved, sm_cs, sm_sn);
          }
          *(uint4*)(dst + 16 * pc) = piece;
          *(uint4*)(sm_new + 16 * pc) = piece;
        }
      }
      }
      __syncthreads();
    }

#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const int e0 = 8 * (4 * s + c4);
      uint4 piece = raw[s];
      if constexpr (!FP8) {
        if (a.rot && 32 * s < a.off + a.rot && 32 * s + 32 > a.off) {
          // (64 rotating entries in the half layout: the partner piece is the lane's own of the k-step beside; a load would
          // return behind the tile's)
          uint4 oth;
          if (a.rot == 64) {
            const uint4 up = raw[s + 1 < KS ? s + 1 : s], down = raw[s > 0 ? s - 1 : 0];
            const bool first_half = e0 < a.off + 32;
            oth = uint4{first_half ? up.x : down.x, first_half ? up.y : down.y, first_half ? up.z : down.z, first_half ? up.w : down.w};
          } else {
            oth = *(const uint4*)(qrow + rope_partner(e0, a.off, a.rot, interleaved));
          }
          piece = rope_rotate(piece, oth, e0, a.off, a.rot, interleaved, sm_cs, sm_sn);
        }
      }
      if (col >= a.H) piece = uint4{0, 0, 0, 0};
      if (s < KR) qf[s] = __builtin_bit_cast(bf16x8, piece);
      else sm_q[s - KR][lane] = piece;             // (every wave writes, and reads, the same)
    }
  }

  // ---- LDS operand addresses (byte offsets inside the stage)
  // score operand (k-step s): row = col.  bf16: chunk 4 s + c4 in slot (4 s + c4) ^ (col & 7); bit 2 of the swizzle flips
  // the parity of s, hence two bases (even / odd s) + 128 * (s / 2).  FP8: 8 codes at 32 s + 8 c4.
  const int f = (col >> 2) & 1;
  const int k_base = col * ROW_BYTES + ((c4 ^ (col & 3)) * 16);
  const int k_even = k_base + 64 * f, k_odd = k_base + 64 * (1 - f);
  // (FP8: with the stage's offset, moved on from tile to tile; a copy of each without it would not fit the registers)
  int k8 = wave * STAGE + col * FP8_ROW_BYTES + 8 * c4, k8_rope = wave * STAGE + col * FP8_ROW_BYTES + 528 + 16 * c4;
  // value operand (16 dims of block blk).  bf16: in each 16-lane group, lane r supplies row 4 c4 + r / 4 and dims
  // 4 (r % 4) .. + 3; the transpose read hands lane i dim i of those 4 tokens.  FP8: lane r supplies row (token)
  // 4 c4 + (r / 2) % 4 and 8 dims of block 2 p + r / 8; lane i gets dim i of the 4 tokens of both blocks.
  int sc8 = wave * STAGE + 4 * c4 * FP8_ROW_BYTES + 512;     // FP8: the scales of token 4 c4 (+ i rows)
  const int v_row = 4 * c4 + (col >> 2);
  int v_base[4];                                   // by blk & 3; add 128 * (blk / 4)
#pragma unroll
  for (int b3 = 0; b3 < 4; ++b3) v_base[b3] = v_row * ROW_BYTES + (((2 * b3 + ((col & 3) >> 1)) ^ (v_row & 7)) * 16) + (col & 1) * 8;
  int v8 = wave * STAGE + (4 * c4 + ((col >> 1) & 3)) * FP8_ROW_BYTES + 16 * (col >> 3) + 8 * (col & 1);

  f32x4 O[VB];
#pragma unroll
  for (int i = 0; i < VB; ++i) O[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY, l = 0.f;                    // running maximum of the scores (FP8: the softmax's reference, as an exponent of 2), row sum
  // FP8: the value product runs on the codes, with softmax weights times scale / (scale of the wave's first token), so that
  // the weights lose nothing to their rounding that they would not lose without scales; O is multiplied at the end.
  float ref[4] = {1.f, 1.f, 1.f, 1.f}, inv_ref[4] = {1.f, 1.f, 1.f, 1.f};
  bool have_ref = false;
  auto uniform = [](float x) -> float { return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, x))); };

  for (int t = wave; t < n_tiles; t += WAVES) {     // (a fixed share for each wave: the result does not depend on who is faster)
    char* const stage = smem + at * STAGE;
    char* next_src = t + WAVES < n_tiles ? tile_addr(t + WAVES) : nullptr;
    const int next_at = FP8 ? (at + WAVES < STAGES ? at + WAVES : at + WAVES - STAGES) : at;
    // FP8: the next tile's stage is free when the tile three before this one, the next wave's, is finished with
    auto stage_is_free = [&]() -> bool {
      if (t < STAGES - WAVES) return true;
      const int owner = (wave + WAVES - (STAGES - WAVES)) % WAVES;
      return __builtin_amdgcn_readfirstlane(__hip_atomic_load(&sm_done[owner], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) > (t - (STAGES - WAVES)) / WAVES;
    };
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");             // the tile has landed
    const int tok0 = (tile0 + t) * TILE;
    if (tok0 + TILE >= n) {                                      // the request's last tile
      const int slot = (n - 1) - tok0;                           // its last token
      int ln = lane;
      uint32_t zero = 0;
      asm volatile("" : "+v"(ln), "+v"(zero));                   // what the rare tile needs takes no registers from the loop
      if (appends) {
        constexpr int PCS = FP8 ? FP8_ROW_BYTES / 16 : CH;
        for (int pc = ln; pc < PCS; pc += 64)
          *(uint4*)(stage + slot * (FP8 ? FP8_ROW_BYTES : ROW_BYTES) + (FP8 ? pc : pc ^ (slot & 7)) * 16) = *(const uint4*)(sm_new + 16 * pc);
      }
      // slots past the context hold arbitrary bytes: cleared (their weights are zero, but 0 x NaN is not)
      constexpr int RB = FP8 ? FP8_ROW_BYTES : ROW_BYTES;
      for (int i = (slot + 1) * (RB / 16) + ln; i < TILE * (RB / 16); i += 64) *(uint4*)(stage + 16 * i) = uint4{zero, zero, zero, zero};
      mla_lds_visible_in_wave();
    }

    // ---- S^T = C . Q^T, operand reads a few ahead of the MFMAs, several accumulators so that consecutive MFMAs do not wait
    // for each other
    f32x4 S;
    uint2 pb[FP8 ? 4 : 1];                         // P^T operands: softmax weights, with FP8 times the block's scale
    f32x4 sc[FP8 ? 4 : 1];                         // FP8: the four blocks' scales of tokens 4 c4 + i
    if constexpr (FP8) {
      constexpr int AHEAD = 4;
      uint2 ring[AHEAD];
      auto read_s = [&](int s) -> uint2 { return *(const uint2*)(smem + k8 + 32 * s); };
#pragma unroll
      for (int s = 0; s < AHEAD; ++s) ring[s] = read_s(s);
      const uint4 rope0 = *(const uint4*)(smem + k8_rope), rope1 = *(const uint4*)(smem + k8_rope + 64);
      // a block's sum is multiplied by the tokens' scales while the next block's products run
      f32x4 acc[2], scale;
      S = f32x4{0.f, 0.f, 0.f, 0.f};
      S = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, rope0), __builtin_bit_cast(bf16x8, sm_q[0][lane]), S, 0, 0, 0);
      S = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, rope1), __builtin_bit_cast(bf16x8, sm_q[1][lane]), S, 0, 0, 0);
#pragma unroll
      for (int sb = 0; sb <= 4; ++sb) {
        if (sb < 4) {
          f32x4& ac = acc[sb & 1];
          ac = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const int s = 4 * sb + k;
            const uint2 w = ring[s % AHEAD];
            if (s + AHEAD < 16) ring[s % AHEAD] = read_s(s + AHEAD);
            const uint4 op = uint4{mla_codes_to_bf16<false>(w.x), mla_codes_to_bf16<true>(w.x), mla_codes_to_bf16<false>(w.y), mla_codes_to_bf16<true>(w.y)};
            ac = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, op), qf[s], ac, 0, 0, 0);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
        if (sb > 0) S += acc[(sb - 1) & 1] * scale;
        if (sb < 4) {
#pragma unroll
          for (int i = 0; i < 4; ++i) scale[i] = *(const float*)(smem + sc8 + i * FP8_ROW_BYTES + 4 * sb);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    } else {
      constexpr int AHEAD = 4;
      uint4 ring[AHEAD];
      auto read_s = [&](int s) -> uint4 { return *(const uint4*)(stage + ((s & 1) ? k_odd : k_even) + 128 * (s >> 1)); };
#pragma unroll
      for (int s = 0; s < AHEAD; ++s) ring[s] = read_s(s);
      f32x4 acc[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
      __builtin_amdgcn_sched_barrier(0);           // keep the issue order below (reads stay ahead of their use)
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        acc[s % 2] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, ring[s % AHEAD]), qf[s], acc[s % 2], 0, 0, 0);
        if (s + AHEAD < KS) ring[s % AHEAD] = read_s(s + AHEAD);
        __builtin_amdgcn_sched_barrier(0);
      }
      S = acc[0] + acc[1];
    }
    if constexpr (FP8) {
      asm volatile("" : "+v"(S));                  // (the compiler would put the products behind the branch)
      if (next_src && stage_is_free()) {
        load_tile(next_src, next_at);
        next_src = nullptr;
      }
    }
    // the first value operands: in flight while the vector ALU does the softmax
    constexpr int VAH = FP8 ? 3 : 5, NVR = FP8 ? VB / 2 : VB;
    uint2 vring[VAH];
    auto read_v = [&](int r) -> uint2 {
      if constexpr (FP8)
        return __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr8_b64_v2i32((__attribute__((address_space(3))) i32x2*)(smem + v8 + 32 * r)));
      else
        return __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (__attribute__((address_space(3))) s16x4*)(stage + v_base[r & 3] + 128 * (r >> 2))));
    };
#pragma unroll
    for (int r = 0; r < VAH; ++r) vring[r] = read_v(r);
    __builtin_amdgcn_sched_barrier(0);

    if constexpr (FP8) __builtin_amdgcn_s_setprio(2);
    // lane holds, for head col, tokens tok0 + 4 c4 + i
    if (tok0 + TILE > n) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (tok0 + 4 * c4 + i >= n) S[i] = -INFINITY;
    }
    float mx = fmaxf(fmaxf(S[0], S[1]), fmaxf(S[2], S[3]));
    mx = mla_max_over_rows(mx);
    // O is rescaled only where some running maximum moved; with FP8, whose weights are rounded with their tokens' scales and are
    // never exact, where it passed a reference that is put 2^8 above it (in six tiles of ten one of 16 heads has a new maximum, and
    // 128 multiplications).  (Above: the weights are 1 at most, so that the sums leave fp32's range no earlier than with the maximum itself.)
    const float top = mx * a.c;
    const float m_new = FP8 ? (top > m ? top + 8.f : m) : fmaxf(m, mx);
    const bool moves = __builtin_amdgcn_ballot_w64(m_new > m) != 0;
    const float mc = FP8 ? m_new : m_new * a.c;
    float p[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) p[i] = __builtin_amdgcn_exp2f(S[i] * a.c - mc);
    const float psum = (p[0] + p[1]) + (p[2] + p[3]);
    if constexpr (FP8) {
#pragma unroll
      for (int i = 0; i < 4; ++i) sc[i] = *(const f32x4*)(smem + sc8 + i * FP8_ROW_BYTES);     // for the value product
      // (the reference stays near 1: relative to a scale at one end of fp32's range the others' would leave it at the other end)
      if (!have_ref) {
#pragma unroll
        for (int sb = 0; sb < 4; ++sb) {
          ref[sb] = uniform(fminf(fmaxf(sc[0][sb], 0x1p-16f), 0x1p16f));
          inv_ref[sb] = uniform(1.f / ref[sb]);
        }
        have_ref = true;
      }
#pragma unroll
      for (int sb = 0; sb < 4; ++sb)
        pb[sb] = uint2{mla_pack_bf16(p[0] * (sc[0][sb] * inv_ref[sb]), p[1] * (sc[1][sb] * inv_ref[sb])),
                       mla_pack_bf16(p[2] * (sc[2][sb] * inv_ref[sb]), p[3] * (sc[3][sb] * inv_ref[sb]))};
    } else {
      pb[0] = uint2{mla_pack_bf16(p[0], p[1]), mla_pack_bf16(p[2], p[3])};
    }
    if (moves) {
      const float alpha = __builtin_amdgcn_exp2f(FP8 ? m - m_new : (m - m_new) * a.c);
      l *= alpha;
#pragma unroll
      for (int blk = 0; blk < VB; ++blk) O[blk] *= alpha;
      m = m_new;
    }
    l += psum;

    if constexpr (FP8) __builtin_amdgcn_s_setprio(1);
    // ---- O^T += C^T . P^T
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int r = 0; r < NVR; ++r) {
      const uint2 v = vring[r % VAH];
      if constexpr (FP8) {
        const s16x4 pv = __builtin_bit_cast(s16x4, pb[r / 4]);
        const uint2 v0 = uint2{mla_codes_to_bf16<false>(v.x), mla_codes_to_bf16<true>(v.x)};
        const uint2 v1 = uint2{mla_codes_to_bf16<false>(v.y), mla_codes_to_bf16<true>(v.y)};
        if (r + VAH < NVR) vring[r % VAH] = read_v(r + VAH);
        O[2 * r] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s16x4, v0), pv, O[2 * r], 0, 0, 0);
        O[2 * r + 1] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s16x4, v1), pv, O[2 * r + 1], 0, 0, 0);
      } else {
        O[r] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s16x4, v), __builtin_bit_cast(s16x4, pb[0]), O[r], 0, 0, 0);
        if (r + VAH < NVR) vring[r % VAH] = read_v(r + VAH);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (FP8) __builtin_amdgcn_s_setprio(0);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");           // every read of the stage has returned
    if constexpr (FP8) {
      if (lane == 0) __hip_atomic_store(&sm_done[wave], t / WAVES + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      if (next_src)
        while (!stage_is_free()) __builtin_amdgcn_s_sleep(1);
    }
    if (next_src) load_tile(next_src, next_at);
    if constexpr (FP8) {
      const int by = (next_at - at) * STAGE;
      k8 += by; k8_rope += by; sc8 += by; v8 += by;
      asm volatile("" : "+v"(k8), "+v"(k8_rope), "+v"(sc8), "+v"(v8));
    }
    at = next_at;
  }

  // ---- merge the waves' (m, l, O)
  l += __shfl_xor(l, 16);
  l += __shfl_xor(l, 32);
  if (c4 == 0) sm_m[wave][col] = m;
  __syncthreads();                                 // also: every wave is done with its stage
  idx = __builtin_amdgcn_readfirstlane(sm_rec[6]);
  if (idx >= 0 && has_word) rec_word = ((const int32_t*)(a.items + (size_t)idx * a.item_stride))[tid];
  // (a wave without a tile has m = -inf: its weight is 0)
  float m_tot = sm_m[0][col];
#pragma unroll
  for (int w = 1; w < WAVES; ++w) m_tot = fmaxf(m_tot, sm_m[w][col]);
  const float mine = __builtin_amdgcn_exp2f(FP8 ? m - m_tot : (m - m_tot) * a.c);
  if (c4 == 0) {
    sm_l[wave][col] = l * mine;
    if (wave == 0) sm_m[WAVES][col] = FP8 ? m_tot : m_tot * a.c;
  }
  float* so = (float*)smem;                        // [wave][head][half of the dims]
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    if (half) __syncthreads();
#pragma unroll
    for (int blk = 0; blk < VB / 2; ++blk) {
      f32x4 o = O[half * (VB / 2) + blk];
      o *= FP8 ? mine * ref[2 * half + blk / 8] : mine;
      *(f32x4*)(so + (wave * 16 + col) * HALF_PITCH + 16 * blk + 4 * c4) = o;
    }
    __syncthreads();
    // four dims per thread, a wave per head
    const int d = 4 * lane;
#pragma unroll 2
    for (int h = wave; h < a.H; h += WAVES) {
      f32x4 o = f32x4{0.f, 0.f, 0.f, 0.f};
      float lt = 0.f;
#pragma unroll
      for (int w = 0; w < WAVES; ++w) {
        o += *(const f32x4*)(so + (w * 16 + h) * HALF_PITCH + d);
        lt += sm_l[w][h];
      }
      const size_t head = (size_t)b * a.H + h;
      if (n_chunks == 1) {
        const float inv = 1.f / lt;
        *(uint2*)(a.out + head * DV + half * (DV / 2) + d) = uint2{mla_pack_bf16(o[0] * inv, o[1] * inv), mla_pack_bf16(o[2] * inv, o[3] * inv)};
      } else {
        const size_t slot = head * a.max_chunks + chunk;
        *(f32x4*)(a.ws_o + slot * DV + half * (DV / 2) + d) = o;
        if (half == 0 && lane == 0) store_partial(a.ws_ml + slot * 2, sm_m[WAVES][h], lt, false);
      }
    }
  }
  if (idx < 0) break;
  __syncthreads();                                 // LDS belongs to the next chunk
  }
}

hipError_t launch_decode_mla(const PoolGeom& g, char* pool_base, const DecodeLaunch& d, hipStream_t stream) {
  MlaArgs a;
  a.pool = pool_base; a.page_bytes = g.page_bytes; a.tiles_per_page = g.P / mla::TILE;
  a.q = (const bf16_t*)d.q; a.k_new = (const bf16_t*)d.k_new; a.out = (bf16_t*)d.out;
  a.items = d.items; a.item_stride = d.item_stride; a.H = d.H;
  if (d.item_stride > 4 * MLA_THREADS) return hipErrorInvalidValue;    // words that the workgroup would not fetch
  a.c = d.scale * 1.4426950408889634f;
  a.max_chunks = d.max_chunks;
  a.w = d.w; a.rot = d.rot; a.off = d.off; a.interleaved = d.interleaved;
  a.ws_o = d.ws_o; a.ws_ml = d.ws_ml; a.put_chunks = d.put_chunks; a.mark = d.mark;
  const dim3 grid((unsigned)d.n_wgs), block(64 * mla::WAVES);
  if (g.kind == SPD_KV_MLA_LATENT_FP8) hipLaunchKernelGGL(decode_mla_kernel<true>, grid, block, 0, stream, a);
  else hipLaunchKernelGGL(decode_mla_kernel<false>, grid, block, 0, stream, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || d.max_chunks <= 1) return e;
  return launch_merge_chunks<mla::DV>(d, stream);
}

}  // namespace spd
