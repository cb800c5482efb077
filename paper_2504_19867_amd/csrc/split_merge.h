// Split-K partials of the decode kernels, merged inside the attention launch.
//
// A launch of its own for the merge costs a small step more than the merge itself (2.6 us of host time, and a gap on
// the stream), so where the launch has few workgroups the one that a counter finds to be the last of its group merges
// the group's chunks.  The eight XCDs' L2s are not coherent with each other inside a launch: partials and counters are
// stored and loaded at agent scope, past the L2, and no fence (a write-back and invalidation of the whole L2) is needed.
#pragma once

#include "internal.h"

namespace spd {

// two consecutive floats of a partial; `shared`: another workgroup of this launch reads them
__device__ inline void store_partial(float* p, float x, float y, bool shared) {
  typedef float f32x2_ __attribute__((ext_vector_type(2)));
  const f32x2_ v = {x, y};
  if (shared) __hip_atomic_store((uint64_t*)p, __builtin_bit_cast(uint64_t, v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else *(f32x2_*)p = v;
}

// Every thread of the workgroup has stored its partials: true in the workgroup that is the n-th to get here.  That one
// puts the counter back to zero for the phase's next step.
__device__ inline bool last_of(uint32_t* counter, uint32_t n, uint32_t* lds) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // this thread's partials are where the others will look
  __syncthreads();
  if (threadIdx.x == 0) {
    const uint32_t before = __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (before == n - 1) __hip_atomic_store(counter, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    *lds = before;
  }
  __syncthreads();
  return *lds == n - 1;
}

// Output dims d, d + 1 of one head over its chunks: o points at them in chunk 0's partial, chunks `stride` floats
// apart; ml holds (reference in log2 units, row sum) per chunk.
__device__ inline float __attribute__((ext_vector_type(2))) merge_chunks(const float* o, int stride, const float* ml, int n_chunks) {
  typedef float f32x2_ __attribute__((ext_vector_type(2)));
  auto load2 = [](const float* p) -> f32x2_ {
    return __builtin_bit_cast(f32x2_, __hip_atomic_load((const uint64_t*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
  };
  // reference and sums move together, chunk by chunk, so that all loads are in one pass
  float m = -INFINITY, l = 0.f;
  f32x2_ acc = {0.f, 0.f};
#pragma unroll 4
  for (int ck = 0; ck < n_chunks; ++ck) {
    const f32x2_ mlv = load2(ml + 2 * ck);
    const f32x2_ ov = load2(o + (size_t)ck * stride);
    const float m_new = fmaxf(m, mlv[0]);
    const float wo = __builtin_amdgcn_exp2f(m - m_new), wn = __builtin_amdgcn_exp2f(mlv[0] - m_new);
    l = l * wo + mlv[1] * wn;
    acc = acc * wo + ov * wn;
    m = m_new;
  }
  const float inv = 1.f / l;
  return acc * inv;
}

}  // namespace spd
