// Device helpers shared by the mesh kernels.
#pragma once

#include "index_wrap.hpp"
#include "kernels.hpp"

namespace fep3m {

__device__ __forceinline__ double block_sum(double v, double *red) {
  // Fixed-shape tree over the block (deterministic).
  const int t = threadIdx.x;
  red[t] = v;
  __syncthreads();
  for (int s = blockDim.x >> 1; s > 0; s >>= 1) {
    if (t < s) red[t] += red[t + s];
    __syncthreads();
  }
  double r = red[0];
  __syncthreads();
  return r;
}

// Fixed-shape block sum for any block of whole waves: shuffle tree inside
// each wave, then the wave sums in order.  red holds a value per wave.  The
// result is valid in thread 0.
__device__ __forceinline__ double block_sum_waves(double v, double *red) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  double r = 0.0;
  if (threadIdx.x == 0)
    for (int w = 0; w < int(blockDim.x >> 6); ++w) r += red[w];
  return r;
}

// An entry of op.dk / op.dm at a run-time local index, as a select over the
// compile-time indices: an indexed read of the by-value operator argument
// would copy the whole operator to scratch memory.
template <int PO, class T>
__device__ __forceinline__ T pick(const T (&v)[kMaxP], int k) {
  T r = v[0];
#pragma unroll
  for (int j = 1; j < PO; ++j) r = (k == j) ? v[j] : r;
  return r;
}

// Banded 1-D element-assembled operator on a column held in registers:
// out[o] = sum_j a[k][j] v[o + PO - k + j] (+ a[PO][j] v[o + j] for k = 0),
// k = o mod PO, with v indexed from one element below the first output.
// Every coefficient index is a compile-time constant, so the (wave-uniform)
// coefficients come from scalar registers.
template <int PO, int NOUT, class T>
__device__ __forceinline__ void band_apply(const T *__restrict__ a, const T (&v)[NOUT + PO + 1], T (&out)[NOUT]) {
  constexpr int Q1 = PO + 1;
#pragma unroll
  for (int o = 0; o < NOUT; ++o) {
    const int k = o % PO;
    T s = T(0);
#pragma unroll
    for (int j = 0; j < Q1; ++j) s += a[k * Q1 + j] * v[o + PO - k + j];
    if (k == 0) {
#pragma unroll
      for (int j = 0; j < Q1; ++j) s += a[PO * Q1 + j] * v[o + j];
    }
    out[o] = s;
  }
}

template <int PO, int NOUT, class T>
__device__ __forceinline__ void band_apply_acc(const T *__restrict__ a, const T (&v)[NOUT + PO + 1], T (&out)[NOUT]) {
  T t[NOUT];
  band_apply<PO, NOUT>(a, v, t);
#pragma unroll
  for (int o = 0; o < NOUT; ++o) out[o] += t[o];
}

}  // namespace fep3m
