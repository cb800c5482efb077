// First step of the gated FFN: the gate and the up projection as ONE matrix product, with the
// activation applied to the accumulators.
//
// Paper, Evaluation "Implementation based on DistServe": the first two GEMMs of the gated FFN are
// fused into one.  With x [T, hidden] and the joint weight matrix w_gu [2 inter, hidden] (rows
// 64 b .. 64 b + 31 = gate rows 32 b .., rows 64 b + 32 .. 64 b + 63 = the up rows of the same outputs;
// stored tile by tile, 256 joint rows x 32 hidden entries, in the order the kernel's LDS stage has):
//     y = x . w_gu^T            out[t, 32 b + j] = silu(y[t, 64 b + j]) * y[t, 64 b + 32 + j]
// silu(z) = z / (1 + exp(-z)).  bf16 in, fp32 accumulation, one rounding to bf16 at the end.
//
// A dense contraction: v_mfma_f32_32x32x16_bf16.
//
// Prompt batches (ffn_gate_up_large_kernel): one workgroup = 8 waves computes a tile of 256 tokens x 256
// joint columns (= 128 outputs); the waves form a 2 x 4 grid, each with 128 tokens x 64 joint
// columns: one block of 32 gate columns and the 32 up columns that belong to them, so the
// activation needs nothing but the wave's own accumulators.  Both operands are contiguous along
// hidden; 32-wide slices of them stream from global memory straight into LDS rings
// (global_load_lds_dwordx4) and are read back with 16-byte reads in operand order.  The 16-byte chunks of
// a row in LDS are XOR-swizzled with bits of the row number, which spreads 16 consecutive rows over all banks.
//
// Decode batches of up to 128 tokens are bound by reading the weights once and have a kernel of their own
// (ffn_gate_up_stream_kernel); between 128 and 256 tokens there are 128 x 128 tiles (ffn_gate_up_small_kernel: four waves, two
// workgroups per compute unit), where those are the faster ones (small_tiles_pay).
#include "ffn_stream.h"
#include "internal.h"

#include <type_traits>

namespace spd {

namespace {

typedef unsigned short bf16_t;
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

constexpr int BK = 32;                          // hidden entries per slice

__device__ inline uint32_t cvt_bf16(float a) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, a}, bf16x2)) & 0xffffu;
}
// 16 bytes per lane from global memory to LDS: lane i's data lands at lds_byte_addr + 16 * i.
// The compiler does not see this write; completion is tracked by hand with vmcnt.
__device__ inline void dma16s(const void* sbase, uint32_t voff, uint32_t lds_byte_addr) {
  asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_byte_addr), "v"(voff), "s"(sbase) : "memory");
}
#define SPD_WAIT_VMCNT(N) __builtin_amdgcn_s_waitcnt(((N) & 15) | (7 << 4) | (15 << 8) | (((N) >> 4) << 14))

// Which tile the workgroups of an XCD take, in the order in which they take them.  Workgroup b runs on XCD b % xcds, and the
// workgroups of an XCD start in the order of b.  Every XCD takes a contiguous range of weight tiles (columns) and all token tiles;
// inside it the tiles are ordered so that the 16 or so workgroups running together form a block of about 4 x 4 tiles:
// each slice of x and of the weights that misses the XCD's L2 then feeds four workgroups.
struct TileOrder {
  int tiles_m, start, cnt;                        // this XCD's weight tiles: cnt from `start` on
  __device__ TileOrder(int tiles_m_, int tiles_n, int xcds) : tiles_m(tiles_m_) {
    const int xcd = (int)blockIdx.x % xcds, base = tiles_n / xcds, rem = tiles_n % xcds;
    cnt = base + (xcd < rem ? 1 : 0);
    start = xcd * base + min(xcd, rem);
  }
  __device__ int slots() const { return cnt * tiles_m; }
  __device__ void tile(int slot, int& tm, int& tn) const {
    const int full = cnt / 4;                     // column blocks of four weight tiles; the last one narrower
    const bool in_full = slot < full * 4 * tiles_m;
    const int cb = in_full ? slot / (4 * tiles_m) : full, wb = in_full ? 4 : cnt - 4 * full;
    const int q = slot - cb * 4 * tiles_m;
    tm = q / wb;
    tn = start + 4 * cb + q % wb;
  }
};

// 128 tokens x 128 joint columns, 2 x 2 waves with 64 tokens x 64 joint columns each, two workgroups per compute unit; a ring of
// four stages with one s_barrier per slice, operands read a slice ahead of the MFMAs into a second set of registers.
__global__ __launch_bounds__(256, 2) void ffn_gate_up_small_kernel(const bf16_t* __restrict__ x, const bf16_t* __restrict__ w,
                                                                   bf16_t* __restrict__ out, int T, int K, int I, int tiles_m,
                                                                   int tiles_n, int xcds, StepMark mark) {
  constexpr int MB = 2, WNW = 2, NSTAGE = 4, WAVES = 2 * WNW, BM = 64 * MB, BNP = 64 * WNW, PD = NSTAGE - 1;
  constexpr int A_BYTES = BM * BK * 2, B_BYTES = BNP * BK * 2, STAGE_BYTES = A_BYTES + B_BYTES;
  constexpr int A_LOADS = A_BYTES / 1024, B_LOADS = B_BYTES / 1024, LPW = (A_LOADS + B_LOADS) / WAVES;   // 1 KiB load instructions (per wave)
  static_assert(B_LOADS % WAVES == 0 && A_LOADS % WAVES == 0, "loads divide evenly over the waves");
  __shared__ __attribute__((aligned(1024))) char smem[NSTAGE * STAGE_BYTES];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n32 = lane & 31, hh = lane >> 5;
  const int wm = wave / WNW, wn = wave % WNW;
  const TileOrder order(tiles_m, tiles_n, xcds);
  const int slot = (int)blockIdx.x / xcds;
  if (slot >= order.slots()) return;
  int tm, tn;
  order.tile(slot, tm, tn);
  const int m0 = tm * BM, n0p = tn * BNP;
  const uint32_t smem_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem;
  const uint32_t pitch = (uint32_t)K * 2;

  // ---- slice loads.  Load instruction ii = wave + WAVES j fills the 64 consecutive 16-byte slots
  // [64 ii, 64 ii + 64) of the stage: x rows first (row = slot / 4), then weight rows; slot s of a
  // row holds the row's chunk s ^ ((row >> 2) & 3).  Token rows past T re-read row T - 1.
  // piece number of this wave's load j: below A_LOADS a piece of x, from there on pieces of the weights
  auto piece_of = [&](int j) __attribute__((always_inline)) -> int { return wave + WAVES * j; };
  uint32_t ld_voff[LPW];
#pragma unroll
  for (int j = 0; j < LPW; ++j) {
    const int ii = piece_of(j);
    if (ii < A_LOADS) {
      const int s = ii * 64 + lane, row = s >> 2, chunk = (s & 3) ^ ((row >> 2) & 3);
      ld_voff[j] = (uint32_t)min(row, T - 1 - m0) * pitch + (uint32_t)chunk * 16;
    } else {
      ld_voff[j] = (uint32_t)((ii - A_LOADS) * 64 + lane) * 16;   // the weights are stored in this very order
    }
  }
  const char* a_base = (const char*)(x + (size_t)m0 * K);
  // weight tile (joint rows 256 t .., slice ks) is 16 KiB at ((t * K / 32) + ks) * 16 KiB; a 128-row tile is half of one
  const char* b_base = (const char*)w + ((size_t)(n0p / 256) * (K / BK)) * 16384 + (size_t)(n0p % 256) * 64;
  const int n_slices = K / BK;
  int pt = 0, ct = 0;
  // load instruction j of slice pt; after the last one the slice counts as issued
  auto produce_piece = [&](int j) __attribute__((always_inline)) {
    if (pt >= n_slices) return;
    const uint32_t stage = __builtin_amdgcn_readfirstlane(smem_base + (uint32_t)(pt % NSTAGE) * STAGE_BYTES);
    const int ii = piece_of(j);
    dma16s(ii < A_LOADS ? a_base + (size_t)pt * (BK * 2) : b_base + (size_t)pt * 16384, ld_voff[j], stage + (uint32_t)ii * 1024);
    if (j == LPW - 1) ++pt;
  };
  auto produce_one = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < LPW; ++j) produce_piece(j);
  };

  // ---- LDS operand addresses inside a stage: row r, k-step ks (16 hidden entries), lane half hh
  // reads chunk 2 ks + hh of the row
  const int sw = (n32 >> 2) & 3;
  int a_off[2], b_off[2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
    a_off[ks] = (wm * (32 * MB) + n32) * 64 + (((2 * ks + hh) ^ sw) * 16);
    b_off[ks] = A_BYTES + (wn * 64 + n32) * 64 + (((2 * ks + hh) ^ sw) * 16);
  }

  // acc[mb][0] = gate, acc[mb][1] = up: element i of lane (n32, hh) is token 32 mb + 8 (i / 4) + 4 hh + i % 4,
  // column n32 of the wave's block
  f32x16 acc[MB][2];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[mb][nb][e] = 0.f;

#pragma unroll
  for (int t = 0; t < PD; ++t) produce_one();

  // The operands of slice t + 1 are read from LDS into a second set of registers while the matrix
  // cores work on slice t, so the barrier of a step guards the slice AFTER the one being multiplied.
  // Reads, tile loads and MFMAs alternate in program order: issued in a bunch behind the barrier, the
  // reads of all the waves keep the LDS pipe busy for most of a slice's matrix time, and no wave gets
  // to its MFMAs before its own reads are accepted.
  constexpr int N_READS = 2 * (MB + 2), N_MEM = N_READS + LPW, N_MFMA = 4 * MB;
  struct Ops { uint4 a[2][MB], b[2][2]; };
  auto read_op = [&](int slice, Ops& o, int n) __attribute__((always_inline)) {   // operand n in order of use
    const char* sbase = smem + (slice % NSTAGE) * STAGE_BYTES;
    const int ks = n / (MB + 2), r = n % (MB + 2);
    if (r < 2) o.b[ks][r] = *(const uint4*)(sbase + b_off[ks] + r * (32 * 64));
    else o.a[ks][r - 2] = *(const uint4*)(sbase + a_off[ks] + (r - 2) * (32 * 64));
  };
  auto load_ops = [&](int slice, Ops& o) __attribute__((always_inline)) {
#pragma unroll
    for (int n = 0; n < N_READS; ++n) read_op(slice, o, n);
  };
  // this wave's loads of slice s are done when at most (slices issued after it) * LPW remain
  auto wait_slice = [&](int s) __attribute__((always_inline)) {
    const int later = pt - s - 1;
    if (later >= 2) SPD_WAIT_VMCNT(2 * LPW);
    else if (later == 1) SPD_WAIT_VMCNT(LPW);
    else SPD_WAIT_VMCNT(0);
  };
  // one step: slice t + 1 becomes readable for all waves (and everyone is done reading slice t - 1,
  // whose stage is refilled); slice t is multiplied, and the step's memory instructions (the operand
  // reads of slice t + 1, with the four loads of slice t + 3 evenly among them) go behind its MFMAs
  auto step = [&](int t, const Ops& cur, Ops& nxt) __attribute__((always_inline)) {
    const bool more = t + 1 < n_slices;
    if (more) wait_slice(t + 1);
    asm volatile("s_barrier" ::: "memory");
    int n_mem = 0, n_read = 0;
#pragma unroll
    for (int i = 0; i < N_MFMA; ++i) {
      const int ks = i / (2 * MB), mb = (i % (2 * MB)) / 2, nb = i % 2;
      acc[mb][nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, cur.a[ks][mb]),
                                                            __builtin_bit_cast(bf16x8, cur.b[ks][nb]), acc[mb][nb], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (; n_mem * N_MFMA < (i + 1) * N_MEM; ++n_mem) {
        if (n_mem % (N_MEM / LPW) == 1) {
          produce_piece(n_mem / (N_MEM / LPW));
        } else {
          if (more) read_op(t + 1, nxt, n_read);
          ++n_read;
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  Ops o0, o1;
  wait_slice(0);
  asm volatile("s_barrier" ::: "memory");
  load_ops(0, o0);
  for (; ct < n_slices; ct += 2) {
    step(ct, o0, o1);
    if (ct + 1 < n_slices) step(ct + 1, o1, o0);
  }

  if (blockIdx.x == 0 && threadIdx.x == 0) store_mark(mark);

  // ---- activation and store: lanes 0..31 of a store hold 32 consecutive outputs of one token
  const int col = tn * (BNP / 2) + wn * 32 + n32;
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int t = m0 + wm * (32 * MB) + mb * 32 + 8 * (i >> 2) + 4 * hh + (i & 3);
      const float g = acc[mb][0][i], u = acc[mb][1][i];
      const float s = g * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(-1.4426950408889634f * g));
      if (t < T) out[(size_t)t * I + col] = (bf16_t)cvt_bf16(s * u);
    }
}

typedef unsigned int u32x4_any __attribute__((ext_vector_type(4), aligned(2)));   // `out` is only promised to be aligned to its entries

// 256 tokens x 256 joint columns.  Waves w and w + 4 sit on one SIMD, and the two groups of four waves run half a slice apart: while
// one group's MFMAs of a slice are issued, the other group starts the loads of a later slice and reads its operands of its slice out of
// LDS, then they change places; an s_barrier at every change.  So the matrix cores of a SIMD always have one wave that does
// nothing but feed them, and operand reads, tile loads, waits and the barriers' own latency fall beside the other wave's MFMAs.
//   slice u, group 0:  [loads, reads u | MFMAs u         | loads, reads u + 1 ..
//            group 1:  [MFMAs u - 1    | loads, reads u  | MFMAs u ..
// With both waves of a SIMD reading, loading and multiplying in one stream and one barrier per slice, a slice of both took 1600 cycles,
// 1024 of them MFMAs; now 1170.  8192 tokens of hidden 4096, inter 14336 on 128 CUs: 2388 -> 1930 us (1 PFLOP/s); the clock falls from 2.4
// to 2.2 .. 2.3 GHz there (256 CUs: 1.45), so power bounds what is left.  512 tokens: 183 -> 151 us.
// Loads ahead of the reads: 5 % faster than behind them, 12 % than among the MFMAs.  16x16x32 MFMAs draw less power and
// take 15 % more cycles: 2100 us.  A fifth stage, or another order of the slices on every XCD: no change.
//
// x comes in pairs of slices: a load instruction takes 8 rows x 128 bytes, whole cache lines.  (A slice at a time, 16 rows x 64
// bytes, every line is asked for twice: 256 tokens of hidden 4096, inter 14336 102 instead of 86 us on 128 CUs, 8192 tokens 1870
// instead of 1770.)  The ring holds three pairs of x and four slices of the weights, all 160 KiB; a step loads the weights of the
// slice three later and half the rows of the x pair that begins three or four later.
//
// A workgroup walks the tiles slot, slot + gridDim / xcds, ..: with one workgroup per compute unit the loads run ahead across tiles, so
// that a tile's first slices arrive while the one before is finished (2 % over one workgroup per tile).  The product is taken
// transposed (weights are the A operand), so that a lane has four consecutive outputs of one token.
__global__ __launch_bounds__(512, 2) void ffn_gate_up_large_kernel(const bf16_t* __restrict__ x, const bf16_t* __restrict__ w,
                                                                   bf16_t* __restrict__ out, int T, int K, int I, int tiles_m,
                                                                   int tiles_n, int xcds, StepMark mark) {
  if (blockIdx.x == 0 && threadIdx.x == 0) store_mark(mark);
  constexpr int BM = 256, X_PAIR = BM * 128, W_SLICE = BM * BK * 2, XP = 3, WS = 4;   // bytes of a pair / slice, stages of either ring
  constexpr int W_LDS = XP * X_PAIR;              // where the weights' stages begin
  __shared__ __attribute__((aligned(1024))) char smem[XP * X_PAIR + WS * W_SLICE];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n32 = lane & 31, hh = lane >> 5;
  const int wm = wave >> 2, wn = wave & 3;        // wm: also the wave's group
  const TileOrder order(tiles_m, tiles_n, xcds);
  const int n_slots = order.slots(), slot_step = (int)gridDim.x / xcds;
  int slot = (int)blockIdx.x / xcds;
  if (slot >= n_slots) return;
  const uint32_t smem_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem;
  const uint32_t pitch = (uint32_t)K * 2;
  // steps per tile: whole pairs of slices; with an odd number of slices the last step multiplies nothing
  const int n_slices = K / BK, n_steps = (n_slices + 1) & ~1;
  const bool odd = n_slices & 1;
  int left = ((n_slots - 1 - slot) / slot_step + 1) * n_steps;   // steps of all tiles of this workgroup from the current one on

  // ---- loads.  x: instruction ii = wave + 8 j (j < 2) of half `hf` of a pair fills the 64 consecutive 16-byte slots of rows
  // 128 hf + 8 ii .. + 7 of the stage (rows of 128 bytes); slot s of a row holds the row's chunk s ^ ((row >> 1) & 7).  Token rows
  // past T re-read row T - 1; where the pair's second slice lies past the end of the row the first one's chunks are read again.
  // Weights: the slice's 16 KiB in the order in which they are stored: slot s of a row of 64 bytes holds chunk s ^ ((row >> 2) & 3).
  const int x_chunk = (lane & 7) ^ ((4 * wave + (lane >> 4)) & 7);
  uint32_t x_voff[2][2];                          // [half][j]
  const uint32_t w_voff = (uint32_t)lane * 16;
  const char *x_ptr, *w_ptr;                      // the pair, the slice to be loaded next
  int x_slot = slot, x_left = n_steps, w_slot = slot, w_left = n_steps;   // their tiles, and steps until those tiles' end
  auto x_tile = [&]() __attribute__((always_inline)) {
    int tm, tn;
    order.tile(x_slot, tm, tn);
#pragma unroll
    for (int hf = 0; hf < 2; ++hf)
#pragma unroll
      for (int j = 0; j < 2; ++j)
        x_voff[hf][j] = (uint32_t)min(128 * hf + 8 * (wave + 8 * j) + (lane >> 3), T - 1 - tm * BM) * pitch + (uint32_t)x_chunk * 16;
    x_ptr = (const char*)(x + (size_t)(tm * BM) * K);
  };
  auto w_tile = [&]() __attribute__((always_inline)) {
    int tm, tn;
    order.tile(w_slot, tm, tn);
    w_ptr = (const char*)w + (size_t)tn * n_slices * W_SLICE + wave * 1024;
  };
  x_tile();
  w_tile();
  auto load_x = [&](int stage, int hf) __attribute__((always_inline)) {
    const uint32_t lds = smem_base + stage * X_PAIR + hf * (X_PAIR / 2) + wave * 1024;
    if (odd && x_left <= 2) {
#pragma unroll
      for (int j = 0; j < 2; ++j) dma16s(x_ptr, x_voff[hf][j] - (uint32_t)(x_chunk & 4) * 16, lds + j * 8192);
    } else {
#pragma unroll
      for (int j = 0; j < 2; ++j) dma16s(x_ptr, x_voff[hf][j], lds + j * 8192);
    }
    if (hf) x_ptr += 128;
    if (--x_left == 0) {
      x_left = n_steps;
      x_slot += slot_step;
      if (x_slot < n_slots) x_tile();
    }
  };
  auto load_w = [&](int stage) __attribute__((always_inline)) {
    const uint32_t lds = smem_base + W_LDS + stage * W_SLICE + wave * 1024;
#pragma unroll
    for (int j = 0; j < 2; ++j) dma16s(w_ptr + j * 8192, w_voff, lds + j * 8192);
    if (--w_left == 0) {
      w_left = n_steps;
      w_slot += slot_step;
      if (w_slot < n_slots) w_tile();
    } else if (!(odd && w_left == 1)) {
      w_ptr += W_SLICE;
    }
  };

  // ---- LDS operand addresses: k-step ks (16 hidden entries), lane half hh reads chunk 2 ks + hh of the slice's four (x: of the
  // pair's eight).  The loop is unrolled over the rings, so that the stage is part of a read's 16-bit immediate; the third pair of x
  // lies beyond its reach and gets lane addresses of its own.  (Vector instructions in the loop would wait for the other wave's MFMAs.)
  int x_off[2][2][2], w_off[2];                   // x: [third stage][slice of the pair][ks]
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
    w_off[ks] = W_LDS + (wn * 64 + n32) * 64 + ((2 * ks + hh) ^ ((n32 >> 2) & 3)) * 16;
#pragma unroll
    for (int sl = 0; sl < 2; ++sl) {
      x_off[0][sl][ks] = (wm * 128 + n32) * 128 + ((4 * sl + 2 * ks + hh) ^ ((n32 >> 1) & 7)) * 16;
      x_off[1][sl][ks] = x_off[0][sl][ks] + 2 * X_PAIR;
      asm volatile("" : "+v"(x_off[1][sl][ks]));   // a value of its own, not "x_off + constant" to be recomputed
    }
  }
  uint4 ox[2][4], ow[2][2];
  // acc[mb][0] = gate, acc[mb][1] = up: element i of lane (n32, hh) is output 8 (i / 4) + 4 hh + i % 4 of token 32 mb + n32
  f32x16 acc[4][2];
  auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int mb = 0; mb < 4; ++mb)
#pragma unroll
      for (int nb = 0; nb < 2; ++nb)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[mb][nb][e] = 0.f;
  };
  clear();
  auto barrier = [&]() __attribute__((always_inline)) {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };

  // ahead of the first step: the x pairs of slices 0, 1 and 2, 3, the weights of slices 0, 1, 2, as the steps -4 .. -1 would load them
  load_x(0, 0);
  load_x(0, 1);
  load_w(0);
  if (left > 2) load_x(1, 0);
  load_w(1);
  if (left > 2) {
    load_x(1, 1);
    load_w(2);
    SPD_WAIT_VMCNT(8);
  } else {
    SPD_WAIT_VMCNT(0);
  }
  barrier();                                      // slice 0 is there
  if (wm) barrier();                              // the second group starts half a slice later

  int ct = 0;                                     // slice of the tile
  int ready = 0;                                  // steps that need not wait: the end of a tile has awaited all loads up to it
  auto step = [&](auto stc) __attribute__((always_inline)) {
    constexpr int ST = stc, SL = ST & 1;          // step modulo the rings' common period; slice of the pair
    // Loading and reading half of step u.  The stages being loaded held slice u - 1 and pair u / 2 - 1, whose reads both groups had
    // behind them at the last barrier.  At this half's end the wave's own reads are done (the other group's next half
    // may load their stage), and so is what it loaded up to step u - 2, its part of slice u + 1 (which the other group
    // reads half a slice earlier than this wave).
    if (left > 4) load_x((ST / 2 + 2) % XP, SL);
    if (left > 3) load_w((ST + 3) % WS);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
      for (int r = 0; r < 2; ++r) ow[ks][r] = *(const uint4*)(smem + w_off[ks] + (ST % WS) * W_SLICE + r * (32 * 64));
#pragma unroll
      for (int r = 0; r < 4; ++r)
        ox[ks][r] = *(const uint4*)(smem + x_off[ST / 2 % XP == 2][SL][ks] + (ST / 2 % XP == 1 ? X_PAIR : 0) + r * (32 * 128));
    }
    __builtin_amdgcn_sched_barrier(0);
    if (ready > 0) --ready;
    else if (left >= 5) SPD_WAIT_VMCNT(8);        // four loads of this step, four of the one before
    else if (left == 4) SPD_WAIT_VMCNT(6);
    else if (left == 3) SPD_WAIT_VMCNT(2);
    else SPD_WAIT_VMCNT(0);
    __builtin_amdgcn_s_waitcnt(0xc07f);           // lgkmcnt(0)
    barrier();
    if (SL == 0 || ct < n_slices) {
      __builtin_amdgcn_s_setprio(1);
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int mb = 0; mb < 4; ++mb)
#pragma unroll
          for (int nb = 0; nb < 2; ++nb)
            acc[mb][nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, ow[ks][nb]),
                                                                  __builtin_bit_cast(bf16x8, ox[ks][mb]), acc[mb][nb], 0, 0, 0);
      __builtin_amdgcn_s_setprio(0);
    }
    barrier();
    --left;
    ++ct;
  };
  // ---- the tile's end: activation and store.  The halves of the wave exchange four outputs each, so that a lane stores eight
  // consecutive ones.  All loads so far are awaited ahead of the first store: the next two steps then have nothing to wait
  // for, and do not wait for the stores either.
  auto finish_tile = [&]() __attribute__((always_inline)) {
    int tm, tn;
    order.tile(slot, tm, tn);
#pragma unroll
    for (int mb = 0; mb < 4; ++mb) {
      uint32_t y[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        float v[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const float g = acc[mb][0][2 * i + e], u = acc[mb][1][2 * i + e];
          v[e] = g * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(-1.4426950408889634f * g)) * u;
        }
        y[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{v[0], v[1]}, bf16x2));
      }
      if (mb == 0) SPD_WAIT_VMCNT(0);
      const int t = tm * BM + wm * 128 + mb * 32 + n32;
      bf16_t* o = out + (size_t)t * I + tn * 128 + wn * 32 + 8 * hh;
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        // (machine code: the compiler's builtin for the swap loses the second result)
        asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\tv_permlane32_swap_b32 %2, %3\n\ts_nop 1"
                     : "+v"(y[4 * p]), "+v"(y[4 * p + 2]), "+v"(y[4 * p + 1]), "+v"(y[4 * p + 3]));
        if (t < T) *(u32x4_any*)(o + 16 * p) = u32x4_any{y[4 * p], y[4 * p + 1], y[4 * p + 2], y[4 * p + 3]};
      }
    }
  };
  // a pair of slices and, behind a tile's last one, its end; false behind the last tile
  auto pair = [&](auto pc) __attribute__((always_inline)) -> bool {
    constexpr int P = pc;
    step(std::integral_constant<int, 2 * P>{});
    step(std::integral_constant<int, 2 * P + 1>{});
    if (ct == n_steps) {
      finish_tile();
      if (left == 0) return false;
      slot += slot_step;
      clear();
      ct = 0;
      ready = 2;
    }
    return true;
  };
  for (;;) {
    if (!pair(std::integral_constant<int, 0>{})) break;
    if (!pair(std::integral_constant<int, 1>{})) break;
    if (!pair(std::integral_constant<int, 2>{})) break;
    if (!pair(std::integral_constant<int, 3>{})) break;
    if (!pair(std::integral_constant<int, 4>{})) break;
    if (!pair(std::integral_constant<int, 5>{})) break;
  }
  if (!wm) barrier();                             // as many as the second group
}

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2_any __attribute__((ext_vector_type(2), aligned(2)));   // `out` is only promised to be aligned to its entries

// Up to 128 tokens: bound by reading the weights once, i.e. by how many of their bytes are on the way at a time.
// The weights go straight from global memory into operand registers (a load is 1 KiB of consecutive bytes, 16 joint rows x 32
// entries in 16x16x32 operand order) and every wave streams rows of its own through a ring of RING slices in
// registers, which no barrier touches.  A wave has 16 gate rows and the 16 up rows that belong to them, against all 16 NB
// tokens.  The x rows, which all waves share, go through LDS, 256 hidden entries at a time in two stages, loaded
// one stage ahead: one barrier per 8 slices.  (<8, 4, 16, 2>, two halves of 128 rows: 128 entries, 4 slices.)
// The product is taken transposed (weights are the A operand): a lane then has four consecutive outputs of one token.
// <NB, 8, 8>: 256 joint rows per workgroup, 128 KiB of weights on the way per CU; <NB, 4, 16>: 128 rows, the same bytes on the
// way from four waves; five to seven waves where those fill the share's compute units better (ffn_stream_units).  <NB, 6, 8, 2>, <NB, 4, 16, 2>:
// 96 or 64 rows, two waves with half of the slices each, which add up at the end, where the wider ones leave compute units idle.  With the weights staged
// through LDS (at most 96 KiB on the way, a third to a fifth of the stages taken by x, a barrier per slice) 64 tokens of hidden 4096, inter
// 14336 took 68 us on 128 CUs and 48 on 256; now 54.8 and 42.7 us (4.3 and 5.5 TB/s) with the weights from HBM, copies of them cycled, and
// 52.8 on 128 CUs from one copy, most of which the memory-side cache then holds.  With eight waves a ring of 16 slices was slower (56 us
// instead of 55; 75 against 62 at 128 tokens), and so were loads without the non-temporal mark (61 us).
template <int NB, int WAVES, int RING, int SPLIT = 1>
__global__ __launch_bounds__(64 * WAVES, 1) void ffn_gate_up_stream_kernel(const bf16_t* __restrict__ x, const bf16_t* __restrict__ w,
                                                                           bf16_t* __restrict__ out, int T, int K, int I, StepMark mark) {
  if (blockIdx.x == 0 && threadIdx.x == 0) store_mark(mark);
  constexpr int UNITS = WAVES / SPLIT;            // waves w, w + UNITS, .. share a unit's rows, each with its part of the slices
  static_assert(WAVES % SPLIT == 0 && SPLIT <= 2, "the tail is one round");
  constexpr int XS = SPLIT * NB > 8 ? 4 : 8;      // slices per x stage
  constexpr int ROWS = 16 * NB, CHUNKS = 4 * XS;  // 16-byte chunks of a row per stage
  constexpr int PITCH = (ROWS + 1) * 16;          // bytes per chunk column [chunk][row]: the odd row spreads the writes over the banks
  constexpr int PIECES = ROWS * CHUNKS * SPLIT, XL = (PIECES + 64 * WAVES - 1) / (64 * WAVES);   // 16-byte pieces of a stage, per thread
  constexpr int STAGE = SPLIT * CHUNKS * PITCH;
  static_assert(RING % XS == 0, "whole stages per ring");
  __shared__ __attribute__((aligned(1024))) char smem[2 * STAGE];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n16 = lane & 15, c4 = lane >> 4;
  const int n_slices = K / BK, last = n_slices - 1;
  const int part = SPLIT > 1 ? wave / UNITS : 0, per_part = (n_slices + SPLIT - 1) / SPLIT, first = part * per_part, mine = min(per_part, n_slices - first);
  // this wave's rows: half `hf` of joint block `jb` (64 rows)
  // (where the waves of the last workgroup are more than there are rows left, the rest of them repeat the last rows and store nothing)
  const int n_units = I / 16, unit = (int)blockIdx.x * UNITS + (SPLIT > 1 ? wave % UNITS : wave), u = min(unit, n_units - 1), jb = u >> 1, hf = u & 1;
  const char* wb = (const char*)w + (size_t)(jb >> 2) * n_slices * 16384 + (size_t)((jb & 3) * 64 + hf * 16) * 64;
  const uint32_t w_off = (uint32_t)(n16 * 64 + ((c4 ^ ((n16 >> 2) & 3)) * 16));
  auto load_w = [&](int s, int half) __attribute__((always_inline)) -> u32x4 {   // half 0: gate, 1: up rows of slice s
    return __builtin_nontemporal_load((const u32x4*)(wb + (size_t)min(first + s, last) * 16384 + half * 2048 + w_off));
  };
  // x pieces: piece i of a part's stage is chunk i % CHUNKS of row i / CHUNKS; rows past T re-read row T - 1, entries past K the row's last ones
  u32x4 xr[XL];
  auto load_x = [&](int st) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < XL; ++j) {
      const int i = tid + 64 * WAVES * j, of = SPLIT > 1 ? min(i / (ROWS * CHUNKS), SPLIT - 1) : 0;
      const int row = min(i / CHUNKS - of * ROWS, T - 1), ch = min(of * per_part * (BK / 8) + st * CHUNKS + i % CHUNKS, K / 8 - 1);
      xr[j] = *(const u32x4*)((const char*)x + (size_t)row * K * 2 + (size_t)ch * 16);
    }
  };
  auto store_x = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < XL; ++j) {
      const int i = tid + 64 * WAVES * j;
      const int of = SPLIT > 1 ? i / (ROWS * CHUNKS) : 0;
      if (PIECES % (64 * WAVES) == 0 || i < PIECES)
        *(u32x4*)(smem + buf * STAGE + (of * CHUNKS + i % CHUNKS) * PITCH + (i / CHUNKS - of * ROWS) * 16) = xr[j];
    }
  };
  f32x4 acc[2][NB];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
  u32x4 wr[RING][2];
  load_x(0);
  store_x(0);
  // the next x pieces before the weights, as inside the loop: the compiler then waits for them with the weights still on their way
  load_x(1);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int s = 0; s < RING; ++s) {
    wr[s][0] = load_w(s, 0);
    wr[s][1] = load_w(s, 1);
  }
  int buf = 0;
  const int x_off = (part * CHUNKS + c4) * PITCH + n16 * 16;
  bf16x8 xv[2][NB];
  auto read_x = [&](bf16x8* o, const char* xs) __attribute__((always_inline)) {
#pragma unroll
    for (int b = 0; b < NB; ++b) o[b] = *(const bf16x8*)(xs + b * 256);
  };
  // RING slices from s0 on; with `tail` only those that there are
  auto round = [&](int s0, auto tail) __attribute__((always_inline)) {
#pragma unroll
    for (int r = 0; r < RING; ++r) {
      if (r % XS == 0) {
        // everyone's pieces of this stage are there, and everyone is done with the one before, which the next pieces replace
        __syncthreads();
        store_x(buf ^ 1);
        __builtin_amdgcn_sched_barrier(0);
        load_x((s0 + r) / XS + 2);
        __builtin_amdgcn_sched_barrier(0);
      }
      // the stage's x operands are read a slice ahead of the MFMAs
      const char* xs = smem + buf * STAGE + x_off;
      if (r % XS == 0) read_x(xv[0], xs);
      if (r % XS + 1 < XS) read_x(xv[(r + 1) & 1], xs + (r % XS + 1) * (4 * PITCH));
      __builtin_amdgcn_sched_barrier(0);
      if (!tail || s0 + r < mine) {
#pragma unroll
        for (int b = 0; b < NB; ++b) {
          acc[0][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wr[r][0]), xv[r & 1][b], acc[0][b], 0, 0, 0);
          acc[1][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wr[r][1]), xv[r & 1][b], acc[1][b], 0, 0, 0);
        }
      }
      if (!tail) {
        wr[r][0] = load_w(s0 + r + RING, 0);
        wr[r][1] = load_w(s0 + r + RING, 1);
        __builtin_amdgcn_sched_barrier(0);
      }
      if (r % XS == XS - 1) buf ^= 1;
    }
  };
  int s0 = 0;
  const int whole = n_slices - (SPLIT - 1) * per_part;            // slices that every part has: at most one less than some
  for (; s0 + RING <= whole; s0 += RING) round(s0, std::false_type{});
  if (s0 < per_part) round(s0, std::true_type{});
  if constexpr (SPLIT > 1) {                      // the second part's sums, through LDS, to the first
    static_assert(UNITS * 2 * NB * 1024 <= 2 * STAGE, "room for the sums");
    __syncthreads();
    f32x4* const sums = (f32x4*)smem + wave % UNITS * (2 * NB * 64) + lane;
    if (part == 1) {
#pragma unroll
      for (int i = 0; i < 2 * NB; ++i) sums[64 * i] = acc[i / NB][i % NB];
    }
    __syncthreads();
    if (part == 1) return;
#pragma unroll
    for (int i = 0; i < 2 * NB; ++i) acc[i / NB][i % NB] += sums[64 * i];
  }
  // element i of lane (n16, c4) is output 4 c4 + i of token n16 of its block
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const int t = 16 * b + n16;
    float y[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float g = acc[0][b][i];
      y[i] = g * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(-1.4426950408889634f * g)) * acc[1][b][i];
    }
    if (t < T && unit < n_units)
      *(u32x2_any*)(out + (size_t)t * I + 32 * jb + 16 * hf + 4 * c4) = u32x2_any{cvt_bf16(y[0]) | cvt_bf16(y[1]) << 16, cvt_bf16(y[2]) | cvt_bf16(y[3]) << 16};
  }
}

// The packed weights from the two weight matrices, one 16-byte piece per thread and step: piece
// number i of the output lies in tile i / 1024 = (tn, ks), row r = (i % 1024) / 4, slot s = i % 4, and
// holds the hidden entries 32 ks + 8 (s ^ ((r >> 2) & 3)) .. + 7 of joint row 256 tn + r.
__global__ __launch_bounds__(256) void ffn_pack_kernel(const uint4* __restrict__ wg, const uint4* __restrict__ wu,
                                                       uint4* __restrict__ dst, int n_ks, long n_pieces) {
  const long stride = (long)gridDim.x * blockDim.x;
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n_pieces; i += stride) {
    const long tile = i >> 10;
    const int r = (int)(i & 1023) >> 2, sl = (int)(i & 3);
    const long tn = tile / n_ks;
    const int ks = (int)(tile % n_ks);
    const long R = tn * 256 + r;                // joint row: blocks of 32 gate rows + their 32 up rows
    const long n = (R >> 6) * 32 + (R & 31);
    const uint4* src = ((R & 63) < 32 ? wg : wu) + n * (long)(n_ks * 4) + ks * 4 + (sl ^ ((r >> 2) & 3));
    dst[i] = *src;
  }
}

}  // namespace

// `persistent`: at most so many workgroups, one per compute unit of a share that has them to itself; 0: one per tile
template <int BM, typename Kernel>
static hipError_t launch_tiles(Kernel kernel, const void* x, const void* w_gu, void* out, int T, int K, int I, int xcds, int persistent,
                               const StepMark& mark, hipStream_t stream) {
  const int tiles_m = (T + BM - 1) / BM, tiles_n = 2 * I / BM;   // square tiles
  if (tiles_n < xcds || persistent % xcds) xcds = 1;
  int n = xcds > 1 ? ((tiles_n + xcds - 1) / xcds) * tiles_m * xcds : tiles_m * tiles_n;
  if (persistent) n = std::min(n, persistent);
  hipLaunchKernelGGL(kernel, dim3((unsigned)n), dim3(2 * BM), 0, stream, (const bf16_t*)x, (const bf16_t*)w_gu, (bf16_t*)out, T, K, I,
                     tiles_m, tiles_n, xcds, mark);
  return hipGetLastError();
}

template <int NB>
static hipError_t launch_stream(const void* x, const void* w_gu, void* out, int T, int K, int I, int cus, const StepMark& mark, hipStream_t stream) {
  const int units = I / 16;                       // of 16 gate and 16 up rows, a wave's
  auto launch = [&](auto kernel, int waves, int per_wg) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)((units + per_wg - 1) / per_wg)), dim3((unsigned)(64 * waves)), 0, stream, (const bf16_t*)x, (const bf16_t*)w_gu,
                       (bf16_t*)out, T, K, I, mark);
  };
  const int per_wg = ffn_stream_units(NB, units, K, cus);
  if constexpr (NB <= 4) {
    if (per_wg == 7) launch(ffn_gate_up_stream_kernel<NB, 7, 8>, 7, 7);
    if (per_wg == 6) launch(ffn_gate_up_stream_kernel<NB, 6, 8>, 6, 6);
    if (per_wg == 5) launch(ffn_gate_up_stream_kernel<NB, 5, 8>, 5, 5);
    if (per_wg == 3) launch(ffn_gate_up_stream_kernel<NB, 6, 8, 2>, 6, 3);
  }
  if (per_wg == 8) launch(ffn_gate_up_stream_kernel<NB, 8, 8>, 8, 8);
  if (per_wg == 4) launch(ffn_gate_up_stream_kernel<NB, 4, 16>, 4, 4);
  if (per_wg == 2) launch(ffn_gate_up_stream_kernel<NB, 4, 16, 2>, 4, 2);
  return hipGetLastError();
}

// 129 to 256 tokens: are the small tiles faster?  With each on a compute unit of its own they are (hidden 8192, inter 7168 on 224 CUs, 256
// tokens: 114 / 147 us).  An XCD deals its workgroups to its four shader arrays in turn; what counts is how many compute units of an array
// get two.  A large tile costs about 6 us and 0.56 a slice, small ones 1 and, with one such unit per array, about as much a slice, with two
// 0.7 (up to 160 tokens, most of whose second tile is one row again and again, 0.55 too).  Small / large, hidden x inter, tokens, CUs (units with two):
// 2048 x 5632, 256, 160 (1) 38.9 / 44.3 us; 4096 x 4096, 256, 96 (1) 69.7 / 78.2; 4096 x 8192, 256, 224 (1) 71.7 / 80.0, 192 (2) 97.4 / 79.7, at 160 tokens
// 0.97, at 176 1.04 of the large tiles' time; 8192 x 7168, 192, 192 (1) 149 / 139, 160 (2) 153 / 138; 4096 x 14336, 256, 256 (6) 104 / 86.  With two on every
// unit: 1024 x 2048, 256, 32 (1) 20.6 / 24.6; 4096 x 1792 86.3 / 76.6.  (8192 x 3584 on 96 CUs is the exception measured: 128 / 146.)
static bool small_tiles_pay(int T, int K, int I, int xcds, int cus) {
  const int columns = 2 * I / 128, per_xcd = (columns + xcds - 1) / xcds * 2;
  const int with_two = (per_xcd + 3) / 4 - cus / (4 * xcds);   // per shader array
  if (with_two <= 0) return true;
  if (K > 4096) return false;
  if (T <= 160) return with_two <= 2;
  return with_two == 1 && (K <= 2048 || 2 * columns * 2 <= 3 * cus);
}

hipError_t launch_ffn_gate_up(const void* x, const void* w_gu, void* out, int T, int K, int I, int xcds, int cus, bool exclusive,
                              const StepMark& mark, hipStream_t stream) {
  // up to 128 tokens: the weights streamed through registers, all tokens in one workgroup (measured at 100 and 128 tokens of
  // hidden 4096, inter 14336 on 128 CUs: 61 and 63 us, 96 and 105 us for 128 x 128 tiles)
  if (T <= 16) return launch_stream<1>(x, w_gu, out, T, K, I, cus, mark, stream);
  if (T <= 32) return launch_stream<2>(x, w_gu, out, T, K, I, cus, mark, stream);
  if (T <= 64) return launch_stream<4>(x, w_gu, out, T, K, I, cus, mark, stream);
  if (T <= 128) return launch_stream<8>(x, w_gu, out, T, K, I, cus, mark, stream);
  if (T <= 256 && small_tiles_pay(T, K, I, xcds, cus)) return launch_tiles<128>(ffn_gate_up_small_kernel, x, w_gu, out, T, K, I, xcds, 0, mark, stream);
  return launch_tiles<256>(ffn_gate_up_large_kernel, x, w_gu, out, T, K, I, xcds, exclusive ? cus : 0, mark, stream);
}

hipError_t launch_ffn_pack(const void* w_gate, const void* w_up, void* w_gu, int K, int I, hipStream_t stream) {
  const long n_pieces = 2L * I * K / 8;
  hipLaunchKernelGGL(ffn_pack_kernel, dim3((unsigned)std::min<long>((n_pieces + 255) / 256, 8192)), dim3(256), 0, stream,
                     (const uint4*)w_gate, (const uint4*)w_up, (uint4*)w_gu, K / 32, n_pieces);
  return hipGetLastError();
}

}  // namespace spd
