// Rotation of a head's 16-byte pieces, for the kernels that rotate rows on their way (same arithmetic as the RoPE step).
#pragma once

#include "internal.h"

namespace spd {

__device__ inline uint32_t rope_pack(float a, float b) {
  typedef float f32x2_ __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2_ __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2_{a, b}, bf16x2_));
}
__device__ inline float rope_bf_lo(uint32_t w) { return __builtin_bit_cast(float, w << 16); }
__device__ inline float rope_bf_hi(uint32_t w) { return __builtin_bit_cast(float, w & 0xffff0000u); }

// The two entries of a pair (a, b) rotated; the rounding is spelled out so that it is the same in every kernel (left to the
// compiler, which product is rounded before the sum depends on the code around it).
__device__ inline float rope_a(float a, float b, float c, float s) { return __builtin_fmaf(a, c, -(b * s)); }
__device__ inline float rope_b(float a, float b, float c, float s) { return __builtin_fmaf(b, c, a * s); }

// The two 16-byte pieces that hold 8 pairs (half layout: A the first, B the second entries; interleaved: four pairs each),
// rotated in place; cs, sn: the pairs' 8 cosines and sines.
__device__ inline void rope_rotate_pieces(uint4& A, uint4& B, bool interleaved, const float* cs, const float* sn) {
  uint32_t aw[4] = {A.x, A.y, A.z, A.w}, bw[4] = {B.x, B.y, B.z, B.w};
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    if (interleaved) {
      // word j of A holds pair j (low half = a, high half = b); word j of B holds pair 4 + j
      const float xa = rope_bf_lo(aw[j]), xb = rope_bf_hi(aw[j]);
      aw[j] = rope_pack(rope_a(xa, xb, cs[j], sn[j]), rope_b(xa, xb, cs[j], sn[j]));
      const float ya = rope_bf_lo(bw[j]), yb = rope_bf_hi(bw[j]);
      bw[j] = rope_pack(rope_a(ya, yb, cs[4 + j], sn[4 + j]), rope_b(ya, yb, cs[4 + j], sn[4 + j]));
    } else {
      const float a0 = rope_bf_lo(aw[j]), a1 = rope_bf_hi(aw[j]), b0 = rope_bf_lo(bw[j]), b1 = rope_bf_hi(bw[j]);
      aw[j] = rope_pack(rope_a(a0, b0, cs[2 * j], sn[2 * j]), rope_a(a1, b1, cs[2 * j + 1], sn[2 * j + 1]));
      bw[j] = rope_pack(rope_b(a0, b0, cs[2 * j], sn[2 * j]), rope_b(a1, b1, cs[2 * j + 1], sn[2 * j + 1]));
    }
  }
  A = uint4{aw[0], aw[1], aw[2], aw[3]};
  B = uint4{bw[0], bw[1], bw[2], bw[3]};
}

// The 16-byte piece `own` (entries e0 .. e0 + 7 of a head) rotated; `oth` is the piece with the other halves of its
// pairs (half layout).  Same arithmetic as the RoPE step.
__device__ inline uint4 rope_rotate(uint4 own, uint4 oth, int e0, int off, int rot, bool interleaved, const float* cs, const float* sn) {
  if (e0 < off || e0 >= off + rot) return own;
  uint32_t ow[4] = {own.x, own.y, own.z, own.w};
  const uint32_t tw[4] = {oth.x, oth.y, oth.z, oth.w};
  if (interleaved) {
    const int p0 = (e0 - off) >> 1;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float xa = rope_bf_lo(ow[j]), xb = rope_bf_hi(ow[j]);
      ow[j] = rope_pack(rope_a(xa, xb, cs[p0 + j], sn[p0 + j]), rope_b(xa, xb, cs[p0 + j], sn[p0 + j]));
    }
  } else {
    const int half = rot >> 1;
    const bool first = e0 < off + half;           // this piece holds the a side of its 8 pairs
    const int p0 = first ? e0 - off : e0 - off - half;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float m0 = rope_bf_lo(ow[j]), m1 = rope_bf_hi(ow[j]), o0 = rope_bf_lo(tw[j]), o1 = rope_bf_hi(tw[j]);
      const float c0 = cs[p0 + 2 * j], s0 = sn[p0 + 2 * j], c1 = cs[p0 + 2 * j + 1], s1 = sn[p0 + 2 * j + 1];
      ow[j] = first ? rope_pack(rope_a(m0, o0, c0, s0), rope_a(m1, o1, c1, s1)) : rope_pack(rope_b(o0, m0, c0, s0), rope_b(o1, m1, c1, s1));
    }
  }
  return uint4{ow[0], ow[1], ow[2], ow[3]};
}
// first entry of the piece that holds the other halves of the pairs of the piece at e0 (e0 itself where there is none)
__device__ inline int rope_partner(int e0, int off, int rot, bool interleaved) {
  if (interleaved || e0 < off || e0 >= off + rot) return e0;
  return e0 < off + (rot >> 1) ? e0 + (rot >> 1) : e0 - (rot >> 1);
}

}  // namespace spd
