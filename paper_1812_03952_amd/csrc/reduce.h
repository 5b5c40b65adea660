// reduce.h -- one-launch deterministic reductions and posts to the host,
// shared by the Krylov solvers.  Include inside an anonymous namespace.
//
// A dot over many workgroups ends in the launch that forms its partials: each
// workgroup stores its partials, counts itself off, and the last one to do so
// adds all partials in a fixed order.  A second launch for that costs 3 us of
// host time and 4 us on the device, and a copy of the result to the host 15 us
// until the host has it; a word that the device itself stores into pinned
// memory takes 9 us including the launch.
// Workgroups run on eight L2 caches that are not coherent with each other:
// partials are stored and loaded at agent scope, past those caches, and the
// count follows once the stores are complete.  An agent-scope fence instead
// would write back all of the cache's dirty lines in every workgroup.
#pragma once
#include <hip/hip_runtime.h>

constexpr int RED_T = 512;      // threads of a reducing workgroup
constexpr int RED_NB = 512;     // most workgroups (partials per dot)

// workgroups of a pass over `pairs` pairs of entries: one pair per thread
// until the chip is full (2 x 8 waves per CU), then a fixed number.  A
// function of the length only, so that a solve is bitwise reproducible.
static inline unsigned red_grid(int64_t pairs) {
  const int64_t b = (pairs + RED_T - 1) / RED_T;
  return (unsigned)(b < 1 ? 1 : (b > RED_NB ? RED_NB : b));
}

template <int CTRL, int RM> __device__ __forceinline__ double red_dpp_add(double x) {
  const double o = __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, RM, 0xf, false),
                                    __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, RM, 0xf, false));
  return x + o;
}
// the sum over the wave, in lane 63 (all lanes active): rows of 16 by
// shifts, then row 0 into 1 and 2 into 3, then both halves
__device__ __forceinline__ double wave_sum(double x) {
  x = red_dpp_add<0x111, 0xf>(x);
  x = red_dpp_add<0x112, 0xf>(x);
  x = red_dpp_add<0x114, 0xf>(x);
  x = red_dpp_add<0x118, 0xf>(x);
  x = red_dpp_add<0x142, 0xa>(x);
  x = red_dpp_add<0x143, 0xc>(x);
  return x;
}
__device__ __forceinline__ double lane_value(double x, int lane) {   // lane uniform
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), lane),
                          __builtin_amdgcn_readlane(__double2loint(x), lane));
}

// all of this wave's stores so far have reached their scope
__device__ __forceinline__ void stores_done() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0x0f70);                   // vmcnt(0)
  asm volatile("" ::: "memory");
}

// Sums of acc[0 .. K) and acc[M - 1] (as dot K) over the grid.  Returns true
// in every thread of the last workgroup, whose wave w then holds the sums of
// the dots k = w + 8 e in sum[e]; *cnt is zero again.
template <int M>
__device__ __forceinline__ bool reduce_grid(const double (&acc)[M], int K, double *__restrict__ part,
                                            unsigned *__restrict__ cnt, double (&sum)[(M + 7) / 8]) {
  __shared__ double sh[RED_T / 64][M];
  __shared__ int last;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nb = gridDim.x;
#pragma unroll
  for (int k = 0; k < M; ++k)
    if (k < K || k == M - 1) {
      const double v = wave_sum(acc[k]);
      if (lane == 63) sh[wv][k] = v;
    }
  __syncthreads();
  if (wv == 0) {
    if (lane <= K) {
      const int k = lane == K ? M - 1 : lane;
      double v = sh[0][k];
#pragma unroll
      for (int w = 1; w < RED_T / 64; ++w) v += sh[w][k];
      __hip_atomic_store(part + lane * RED_NB + blockIdx.x, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    stores_done();
    if (lane == 0)
      last = __hip_atomic_fetch_add(cnt, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (unsigned)nb - 1u;
  }
  __syncthreads();
  if (!last) return false;
#pragma unroll
  for (int e = 0; e < (M + 7) / 8; ++e) {
    const int k = wv + 8 * e;                           // the same for the wave
    sum[e] = 0.0;
    if (k > K) continue;
    double p[RED_NB / 64];
#pragma unroll
    for (int q = 0; q < RED_NB / 64; ++q)
      p[q] = __hip_atomic_load(part + k * RED_NB + min(lane + 64 * q, nb - 1), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
    double v = 0.0;
#pragma unroll
    for (int q = 0; q < RED_NB / 64; ++q) v += lane + 64 * q < nb ? p[q] : 0.0;
    sum[e] = lane_value(wave_sum(v), 63);
  }
  if (threadIdx.x == 0) __hip_atomic_store(cnt, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return true;
}

// values to pinned host memory, then the sequence number the host waits for
// (rs_wait_post); one lane calls it
__device__ __forceinline__ void post_host(rs_post *p, uint64_t seq, const double *v, int n) {
  for (int i = 0; i < n; ++i) __hip_atomic_store(&p->v[i], v[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  stores_done();
  __hip_atomic_store(&p->seq, seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
