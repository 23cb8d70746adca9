// Workgroup-wide reductions.
//
// Maximum of non-negative doubles, published with one atomic per
// workgroup.  Many atomics on one address serialise in the L2, so the waves of a
// workgroup combine through LDS first.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace thcsox {

// Every thread of the workgroup must call this (it contains a barrier).
// NWAVES = workgroup size / 64.  *addr holds the bits of a non-negative double,
// so the unsigned integer maximum is the floating-point maximum.
template <int NWAVES>
__device__ __forceinline__ void block_atomic_max(double v, unsigned long long* addr) {
  __shared__ double wmax[NWAVES];
  for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) wmax[wave] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    double m = wmax[0];
    for (int w = 1; w < NWAVES; ++w) m = fmax(m, wmax[w]);
    atomicMax(addr, (unsigned long long)__double_as_longlong(m));
  }
}

// Part `part` of `parts` of sum_pq A[p n + q] B[q n + p] by a workgroup of NWAVES waves, in
// a fixed order; the result is valid in thread 0.  Every thread of the workgroup must call this.  A
// wave takes blocks of 64 q and 32 p: lane q reads A down a column (64 lanes on
// consecutive addresses) and its own row of B along p, so every cache line is used
// whole and 48 loads are in flight (one element of B per lane and row, the plain
// loop, took 180 us at n = 300 with four waves).
template <int NWAVES>
__device__ __forceinline__ double block_trace(const double* A, const double* B, int n, int part = 0,
                                              int parts = 1) {
  typedef double d2u __attribute__((ext_vector_type(2), aligned(8)));
  constexpr int PB = 32;
  __shared__ double sums[NWAVES];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int nq = (n + 63) / 64, np = (n + PB - 1) / PB;
  double acc = 0.0;
  for (int it = part * NWAVES + wave; it < nq * np; it += parts * NWAVES) {
    const int q = it % nq * 64 + lane, p0 = it / nq * PB;
    const int qc = min(q, n - 1);
    double s = 0.0;
    if (p0 + PB <= n) {
      double a[PB];
      d2u b[PB / 2];
#pragma unroll
      for (int e = 0; e < PB; ++e) a[e] = A[(int64_t)(p0 + e) * n + qc];
#pragma unroll
      for (int e = 0; e < PB / 2; ++e)
        b[e] = *reinterpret_cast<const d2u*>(B + (int64_t)qc * n + p0 + 2 * e);
#pragma unroll
      for (int e = 0; e < PB; ++e) s = fma(a[e], b[e / 2][e % 2], s);
    } else {
#pragma unroll 8
      for (int p = p0; p < n; ++p) s = fma(A[(int64_t)p * n + qc], B[(int64_t)qc * n + p], s);
    }
    if (q < n) acc += s;
  }
  for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
  if (lane == 0) sums[wave] = acc;
  __syncthreads();
  double t = 0.0;
  if (threadIdx.x == 0)
    for (int w = 0; w < NWAVES; ++w) t += sums[w];
  return t;
}

}  // namespace thcsox
