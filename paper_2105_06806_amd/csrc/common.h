// Device helpers shared by the kernels of libedx (wave64 reductions).
#pragma once

#include <hip/hip_runtime.h>

namespace edx {

// Sum over a 64-lane wavefront; lane 0 holds the result.  Fixed shuffle tree,
// so the result does not depend on timing.
__device__ __forceinline__ double wave_sum(double x) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) x += __shfl_down(x, off, 64);
  return x;
}

// Block-wide sum of one double per thread; valid in thread 0.  `red` must hold
// blockDim.x / 64 doubles of shared memory.  Deterministic for a fixed block size.
__device__ __forceinline__ double block_sum(double x, double* red) {
  const int lane = threadIdx.x & 63;
  const int wid = threadIdx.x >> 6;
  x = wave_sum(x);
  __syncthreads();
  if (lane == 0) red[wid] = x;
  __syncthreads();
  double s = 0.0;
  if (threadIdx.x == 0) {
    const int nw = (blockDim.x + 63) >> 6;
    for (int i = 0; i < nw; ++i) s += red[i];
  }
  return s;
}

// Reductions folded into the kernel that needs their results: every workgroup
// (256 threads) sums the partial sums of the previous kernels for itself, in
// the order of the one-workgroup reduction (threads strided over the partials,
// wave trees, then the four waves in turn), so the values are the same.
// fold_load issues the loads of n <= 256 U partials (before the kernel's own
// loads, so that the latencies overlap); fold_sum2 adds up two such sets at
// once, valid in every thread; red holds 8 doubles.
template <int U>
__device__ __forceinline__ void fold_load(double (&x)[U], const double* __restrict__ part, int n) {
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int i = (int)threadIdx.x + 256 * u;
    x[u] = i < n ? part[i] : 0.0;
  }
}

template <int U, int V>
__device__ __forceinline__ void fold_sum2(const double (&x)[U], const double (&y)[V], double* red,
                                          double& sx, double& sy) {
  double s = 0.0, t = 0.0;
#pragma unroll
  for (int u = 0; u < U; ++u) s += x[u];
#pragma unroll
  for (int u = 0; u < V; ++u) t += y[u];
  s = wave_sum(s);
  t = wave_sum(t);
  const int wid = threadIdx.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) {
    red[wid] = s;
    red[4 + wid] = t;
  }
  __syncthreads();
  sx = ((red[0] + red[1]) + red[2]) + red[3];
  sy = ((red[4] + red[5]) + red[6]) + red[7];
}

// Streaming (non-temporal) 16-byte buffer store at byte offset `off`.  The whole
// offset goes into the lane offset and the scalar offset stays 0: with a
// register there the compiler takes the data registers as free at once (no wait
// state between the store and the next instruction), and on this chip the
// store's third dword then came out as that instruction's result now and then.
__device__ __forceinline__ void buf_store16_nt(__amdgpu_buffer_rsrc_t r, uint32_t off,
                                               unsigned int __attribute__((ext_vector_type(4))) x) {
  __builtin_amdgcn_raw_buffer_store_b128(x, r, (int)off, 0, 2);
}

// Counter-based SplitMix64 (Steele, Lea and Flood's finaliser): draw k of
// stream `seed` (the start vectors' element k takes draw k).
__device__ __forceinline__ uint64_t splitmix64(uint64_t seed, uint64_t k) {
  uint64_t z = seed + (k + 1) * 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

template <typename T>
__device__ __forceinline__ T ldg(const T* p) {
  return __builtin_nontemporal_load(p);
}

}  // namespace edx
