// Split-K partials of the decode kernels: how they are stored, and the two ways of merging them.
//
// A launch of its own for the merge costs 2.6 us of host time and a gap on the stream beside its own 4 to 5 us.  So where a
// request has few chunks (the host says so by handing out counters; GQA pools only) the workgroup that a counter finds to be the last
// of its group merges the group's chunks.  The eight XCDs' L2s are not coherent with each other inside a launch: partials
// and counters are stored and loaded at agent scope, past the L2, and no fence (a write-back and invalidation of the whole
// L2) is needed.
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

// Merge n_chunks (<= MERGE_IN_LAUNCH_CHUNKS) partials of `rows` (<= 16) heads into bf16 rows of D entries at `out`.  o, ml: the
// first head's chunk 0, heads max_chunks chunks apart.  lds: 2 x 16 x MERGE_IN_LAUNCH_CHUNKS floats that nobody uses.
template <int D, int THREADS>
__device__ inline void merge_in_launch(const float* o, const float* ml, int rows, int max_chunks, int n_chunks, float* lds, unsigned short* out) {
  typedef float f32x2_ __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2_ __attribute__((ext_vector_type(2)));
  auto load2 = [](const float* p) -> f32x2_ {
    return __builtin_bit_cast(f32x2_, __hip_atomic_load((const uint64_t*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
  };
  constexpr int NC = MERGE_IN_LAUNCH_CHUNKS, PAIRS = D / 2, BATCH = 4, RB = 2;
  float *sm = lds, *sl = lds + 16 * NC;
  const int tid = threadIdx.x;
  __syncthreads();
  for (int i = tid; i < rows * n_chunks; i += THREADS) {
    const f32x2_ v = load2(ml + ((size_t)(i / n_chunks) * max_chunks + i % n_chunks) * 2);
    sm[(i / n_chunks) * NC + i % n_chunks] = v[0];
    sl[(i / n_chunks) * NC + i % n_chunks] = v[1];
  }
  __syncthreads();
  // a thread keeps its pair of dims and walks over the rows, RB rows by BATCH chunks of loads in flight
  constexpr int STEP = THREADS / PAIRS;            // rows side by side
  static_assert(THREADS % PAIRS == 0, "whole rows");
  const int pr = 2 * (tid % PAIRS);
  for (int r0 = tid / PAIRS; r0 < rows; r0 += RB * STEP) {
    f32x2_ acc[RB];
    float l[RB], m[RB];
#pragma unroll
    for (int j = 0; j < RB; ++j) {
      const int r = min(r0 + j * STEP, rows - 1);
      acc[j] = f32x2_{0.f, 0.f};
      l[j] = 0.f;
      m[j] = -INFINITY;
      for (int ck = 0; ck < n_chunks; ++ck) m[j] = fmaxf(m[j], sm[r * NC + ck]);
    }
    for (int c0 = 0; c0 < n_chunks; c0 += BATCH) {
      f32x2_ v[BATCH][RB];
#pragma unroll
      for (int k = 0; k < BATCH; ++k)
#pragma unroll
        for (int j = 0; j < RB; ++j)
          v[k][j] = load2(o + ((size_t)min(r0 + j * STEP, rows - 1) * max_chunks + min(c0 + k, n_chunks - 1)) * D + pr);
#pragma unroll
      for (int k = 0; k < BATCH; ++k) {
        if (c0 + k >= n_chunks) break;
#pragma unroll
        for (int j = 0; j < RB; ++j) {
          const int r = min(r0 + j * STEP, rows - 1);
          const float w = __builtin_amdgcn_exp2f(sm[r * NC + c0 + k] - m[j]);
          l[j] += sl[r * NC + c0 + k] * w;
          acc[j] += v[k][j] * w;
        }
      }
    }
#pragma unroll
    for (int j = 0; j < RB; ++j)
      if (r0 + j * STEP < rows)
        *(uint32_t*)(out + (size_t)(r0 + j * STEP) * D + pr) = __builtin_bit_cast(uint32_t, __builtin_convertvector(acc[j] * (1.f / l[j]), bf16x2_));
  }
}

// The merge as a launch of its own.  grid (H, B): one (request, head) pair per workgroup.  D / 4 threads take a chunk (four dims each), the
// workgroup several chunks side by side, with four rounds of loads in flight; the sums meet in LDS.  THREADS: 128 (all
// workgroups of a batch are resident at once), or 1024 where requests have many chunks (a single long one can have hundreds).
template <int D, int THREADS>
__global__ __launch_bounds__(THREADS) void merge_chunks_kernel(unsigned short* __restrict__ out, const int32_t* __restrict__ chunks, int H,
                                                               int max_chunks, const float* __restrict__ ws_o, const float* __restrict__ ws_ml) {
  typedef float f32x2_ __attribute__((ext_vector_type(2)));
  typedef float f32x4_ __attribute__((ext_vector_type(4)));
  typedef __bf16 bf16x2_ __attribute__((ext_vector_type(2)));
  constexpr int TPC = D / 4, SIDE = THREADS / TPC, BATCH = 4;        // threads per chunk, chunks side by side
  const int h = blockIdx.x, b = blockIdx.y, lane = threadIdx.x & 63, side = threadIdx.x / TPC, d = 4 * (threadIdx.x % TPC);
  const int n_chunks = chunks[b];
  if (n_chunks <= 1) return;                       // one chunk: written directly by the attention kernel
  const size_t slot0 = ((size_t)b * H + h) * max_chunks;
  const float* ml = ws_ml + slot0 * 2;
  const float* o = ws_o + slot0 * D + d;
  f32x4_ v[BATCH], acc = {0.f, 0.f, 0.f, 0.f};
  f32x2_ w[BATCH];
  auto load = [&](int c0) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < BATCH; ++i) {
      const int ck = min(c0 + SIDE * i, n_chunks - 1);
      w[i] = *(const f32x2_*)(ml + 2 * ck);
      v[i] = *(const f32x4_*)(o + (size_t)ck * D);
    }
  };
  load(side);
  float m = -INFINITY, l = 0.f;
  for (int ck = lane; ck < n_chunks; ck += 64) m = fmaxf(m, ml[2 * ck]);
#pragma unroll
  for (int s = 1; s < 64; s <<= 1) m = fmaxf(m, __shfl_xor(m, s));
  for (int c0 = side; c0 < n_chunks; c0 += SIDE * BATCH) {
    if (c0 != side) load(c0);
#pragma unroll
    for (int i = 0; i < BATCH; ++i) {
      if (c0 + SIDE * i >= n_chunks) break;
      const float wgt = __builtin_amdgcn_exp2f(w[i][0] - m);
      l += w[i][1] * wgt;
      acc += v[i] * wgt;
    }
  }
  __shared__ f32x4_ so[SIDE][TPC];
  __shared__ float sl[SIDE];
  so[side][threadIdx.x % TPC] = acc;
  if (d == 0) sl[side] = l;
  __syncthreads();
  if ((int)threadIdx.x >= TPC) return;
  const int sides = min(SIDE, n_chunks);
  for (int s = 1; s < sides; ++s) {
    acc += so[s][threadIdx.x];
    l += sl[s];
  }
  acc *= 1.f / l;
  uint2 pk;
  pk.x = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2_{acc[0], acc[1]}, bf16x2_));
  pk.y = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2_{acc[2], acc[3]}, bf16x2_));
  *(uint2*)(out + ((size_t)b * H + h) * D + d) = pk;
}

template <int D>
inline hipError_t launch_merge_chunks(const DecodeLaunch& d, hipStream_t stream) {
  const dim3 grid((unsigned)d.H, (unsigned)d.B);
  if (d.max_chunks > 16)
    hipLaunchKernelGGL((merge_chunks_kernel<D, 1024>), grid, dim3(1024), 0, stream, (unsigned short*)d.out, d.n_chunks, d.H, d.max_chunks, d.ws_o, d.ws_ml);
  else
    hipLaunchKernelGGL((merge_chunks_kernel<D, 128>), grid, dim3(128), 0, stream, (unsigned short*)d.out, d.n_chunks, d.H, d.max_chunks, d.ws_o, d.ws_ml);
  return hipGetLastError();
}

}  // namespace spd
