// Wavefront and block reductions for gfx950 (wave64).
//
// Sums are deterministic: every block writes its partial sums and a
// one-block kernel adds them in a fixed order.  Maxima of non-negative doubles use atomicMax
// on the IEEE bit pattern, which orders like the values and is
// order-independent.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ecpic {

constexpr int kBlock = 256;
constexpr int kWave = 64;

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
  return v;
}

__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, kWave));
  return v;
}

// sum over the four lanes of a quad, to each of them
__device__ __forceinline__ double quad_sum(double v) {
  auto swap = [](double u, auto perm) {
    constexpr int kPerm = decltype(perm)::value;
    return __hiloint2double(
        __builtin_amdgcn_mov_dpp(__double2hiint(u), kPerm, 0xf, 0xf, true),
        __builtin_amdgcn_mov_dpp(__double2loint(u), kPerm, 0xf, 0xf, true));
  };
  v += swap(v, std::integral_constant<int, 0xB1>{});  // lanes 1 0 3 2
  v += swap(v, std::integral_constant<int, 0x4E>{});  // lanes 2 3 0 1
  return v;
}

// Sum of M values over the block; the totals are valid in every thread of
// wave 0 (thread 0 uses them).  Must be called by all threads of the block.
template <int M>
__device__ __forceinline__ void block_sum(double (&v)[M]) {
  __shared__ double red_lds[kBlock / kWave][M > 0 ? M : 1];
  const int lane = threadIdx.x % kWave, wid = threadIdx.x / kWave;
#pragma unroll
  for (int m = 0; m < M; ++m) v[m] = wave_sum(v[m]);
  if (lane == 0)
#pragma unroll
    for (int m = 0; m < M; ++m) red_lds[wid][m] = v[m];
  __syncthreads();
  if (wid == 0) {
#pragma unroll
    for (int m = 0; m < M; ++m) {
      double s = lane < kBlock / kWave ? red_lds[lane][m] : 0.0;
      v[m] = wave_sum(s);
    }
  }
  __syncthreads();
}

__device__ __forceinline__ double block_max(double v) {
  __shared__ double max_lds[kBlock / kWave];
  const int lane = threadIdx.x % kWave, wid = threadIdx.x / kWave;
  v = wave_max(v);
  if (lane == 0) max_lds[wid] = v;
  __syncthreads();
  double r = 0.0;
  if (wid == 0) r = wave_max(lane < kBlock / kWave ? max_lds[lane] : 0.0);
  __syncthreads();
  return r;
}

// Block reductions without a barrier after the producing loops, so that a
// wavefront that finishes early does not wait for its block's slowest one:
// every wavefront reduces its lanes (sum, or max where ismax[m]) and leaves
// its M values in LDS; the last wavefront of the block to arrive (an LDS
// counter) combines the block's wavefronts in a fixed order.  Returns true
// in exactly one thread of the block (lane 0 of that wavefront), with the
// block's values in out.  Thread 0 must run late_reduce_init<M>() before a
// barrier that precedes the call.
template <int M>
__device__ __forceinline__ unsigned int* late_counter() {
  __shared__ unsigned int c;
  return &c;
}
template <int M>
__device__ __forceinline__ double* late_values() {
  __shared__ double v[M * (kBlock / kWave)];
  return v;
}
template <int M>
__device__ __forceinline__ void late_reduce_init() {
  if (threadIdx.x == 0) *late_counter<M>() = 0u;
}
template <int M>
__device__ __forceinline__ bool late_reduce(const double (&v)[M], const bool (&ismax)[M],
                                            double (&out)[M]) {
  constexpr int NW = kBlock / kWave;
  const int wid = threadIdx.x / kWave;
  double r[M];
#pragma unroll
  for (int m = 0; m < M; ++m) r[m] = ismax[m] ? wave_max(v[m]) : wave_sum(v[m]);
  if (threadIdx.x % kWave != 0) return false;
  double* vals = late_values<M>();
#pragma unroll
  for (int m = 0; m < M; ++m) vals[m * NW + wid] = r[m];
  __threadfence_block();  // the values before the arrival count
  if (atomicAdd(late_counter<M>(), 1u) != NW - 1) return false;
  __threadfence_block();
#pragma unroll
  for (int m = 0; m < M; ++m) {
    double a = vals[m * NW];
    for (int w = 1; w < NW; ++w) a = ismax[m] ? fmax(a, vals[m * NW + w]) : a + vals[m * NW + w];
    out[m] = a;
  }
  return true;
}

// bit-pattern atomicMax of a non-negative double (order-independent)
__device__ __forceinline__ void atomic_max_nonneg(double* slot, double v) {
  if (v > 0.0)
    atomicMax(reinterpret_cast<unsigned long long*>(slot), (unsigned long long)__double_as_longlong(v));
}

// Grid-wide sums, deterministic: every block writes its M block sums to
// region[m * gridDim.x + blockIdx.x]; a one-block finishing kernel (launched
// by the host after the producing kernels) adds each row in a fixed order.
// The kernel boundary in between makes the partials visible; no device-scope
// fences are needed inside the producing kernels.
template <int M>
__device__ __forceinline__ void block_partials(double (&v)[M], double* region) {
  block_sum<M>(v);
  if (threadIdx.x == 0)
#pragma unroll
    for (int m = 0; m < M; ++m) region[(size_t)m * gridDim.x + blockIdx.x] = v[m];
}

// Periodic minimum image of a node-index difference: raw mod n in
// (-n/2, n/2]; n is a power of two.
__device__ __forceinline__ int min_image(int raw, int n) {
  const int r = raw & (n - 1);
  return 2 * r > n ? r - n : r;
}

// t / d for 0 <= t < 2^22 and d >= 1, with inv_d = 1.0f / d: (t + 1/2) / d
// lies at least 1/(2d) away from an integer, further than the float rounding
// error (t + 1/2) 2^-23 / d, so the truncation is exact (no integer division)
__device__ __forceinline__ int div_small(int t, float inv_d) {
  return (int)(((float)t + 0.5f) * inv_d);
}

// The block of a grid that block blk stands for, so that every XCD (blocks go round robin
// to the 8 of them) takes a contiguous eighth
constexpr int kXcds = 8;
__device__ __forceinline__ int xcd_block(int blk, int blocks) {
  const int x = blk % kXcds;
  return x * (blocks / kXcds) + min(x, blocks % kXcds) + blk / kXcds;
}

// first particle of scatter block blk, and particle k of this thread in it: the
// block's lanes sit span / 64 particles apart, chunk / 64 consecutive particles
// each; span / chunk blocks share a span
__device__ __forceinline__ int64_t chunk_base(int chunk, int span, int blk) {
  const int per_span = span / chunk;
  return (int64_t)(blk / per_span) * span + (blk % per_span) * (chunk / kWave);
}
__device__ __forceinline__ int64_t chunk_particle(int64_t base, int span, int k) {
  const int lane = threadIdx.x % kWave, seg = 4 * (lane % 16) + lane / 16;
  return base + seg * (span / kWave) + (int)(threadIdx.x / kWave) + (kBlock / kWave) * k;
}

// block-wide minimum of M ints at once (one barrier pair for all of them)
template <int M, int BLOCK = kBlock>
__device__ __forceinline__ void block_min_ints(int (&v)[M]) {
  __shared__ int lds_i[M][BLOCK / kWave];
  const int lane = threadIdx.x % kWave, wid = threadIdx.x / kWave;
#pragma unroll
  for (int m = 0; m < M; ++m) {
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) v[m] = min(v[m], __shfl_xor(v[m], o, kWave));
    if (lane == 0) lds_i[m][wid] = v[m];
  }
  __syncthreads();
#pragma unroll
  for (int m = 0; m < M; ++m) {
    int r = lds_i[m][0];
#pragma unroll
    for (int w = 1; w < BLOCK / kWave; ++w) r = min(r, lds_i[m][w]);
    v[m] = r;
  }
  __syncthreads();
}

}  // namespace ecpic
