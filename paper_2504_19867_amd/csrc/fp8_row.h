// One latent row quantised to the FP8 page format (kernels_kv_fp8.hip has the format), by 16 lanes of a wave: lane l owns
// ckv entries 32 l .. 32 l + 31, a quarter of a scale block (the block's maximum is formed over 4 neighbouring lanes).
#pragma once

#include "internal.h"

namespace spd {

struct Fp8Piece {
  uint32_t codes[8];
  float scale;
};

__device__ inline void fp8_quantise(const unsigned short* src, int l, Fp8Piece& out) {
  constexpr float E4M3_MAX = 448.f;
  auto lo = [](uint32_t w) { return __builtin_bit_cast(float, w << 16); };
  auto hi = [](uint32_t w) { return __builtin_bit_cast(float, w & 0xffff0000u); };
  auto clamp = [](float y) { return fminf(fmaxf(y, -E4M3_MAX), E4M3_MAX); };
  uint32_t w[16];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint4 p = *(const uint4*)(src + 32 * l + 8 * j);
    w[4 * j] = p.x; w[4 * j + 1] = p.y; w[4 * j + 2] = p.z; w[4 * j + 3] = p.w;
  }
  float amax = 0.f;
#pragma unroll
  for (int j = 0; j < 16; ++j) amax = fmaxf(amax, fmaxf(fabsf(lo(w[j])), fabsf(hi(w[j]))));
  amax = fmaxf(amax, __shfl_xor(amax, 1));
  amax = fmaxf(amax, __shfl_xor(amax, 2));
  out.scale = amax > 0.f ? amax / E4M3_MAX : 1.f;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    // four entries per word: entries 4 j .. 4 j + 3 = the two halves of w[2 j] and w[2 j + 1]
    int pk = 0;
    pk = __builtin_amdgcn_cvt_pk_fp8_f32(clamp(lo(w[2 * j]) / out.scale), clamp(hi(w[2 * j]) / out.scale), pk, false);
    pk = __builtin_amdgcn_cvt_pk_fp8_f32(clamp(lo(w[2 * j + 1]) / out.scale), clamp(hi(w[2 * j + 1]) / out.scale), pk, true);
    out.codes[j] = (uint32_t)pk;
  }
}

// the lane's part of the row, at `row` (a page's or a copy of it)
__device__ inline void fp8_store_row(char* row, const unsigned short* src, int l, const Fp8Piece& p) {
  *(uint4*)(row + 32 * l) = uint4{p.codes[0], p.codes[1], p.codes[2], p.codes[3]};
  *(uint4*)(row + 32 * l + 16) = uint4{p.codes[4], p.codes[5], p.codes[6], p.codes[7]};
  if ((l & 3) == 0) *(float*)(row + 512 + 4 * (l >> 2)) = p.scale;
  if (l < 8) *(uint4*)(row + 528 + 16 * l) = *(const uint4*)(src + 512 + 8 * l);
}

}  // namespace spd
