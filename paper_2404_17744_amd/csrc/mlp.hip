// Residual MLP of the learned warm start: training and inference on the GPU.
//
// The network maps the tau-profile of one THC pair's first-iteration
// self-energy (m values, divided by the pair's largest magnitude over tau) to
// the profile of the converged one (divided by the same number):
//     z1 = x W1^T + b1,  h1 = silu(z1)          W1: [H][m]
//     z2 = h1 W2^T + b2, h2 = silu(z2)          W2: [H][H]
//     y  = x + h2 W3^T + b3                     W3: [m][H]
// loss = mean over the batch and m of (y - target)^2, silu(z) = z / (1 + e^-z).
// Weights, activations and accumulation are FP32; the GEMMs run on FP32 matrix
// cores.  Parameters are one packed array: W1, b1, W2, b2, W3, b3.
#include <hip/hip_runtime.h>
#include <new>

#include <cmath>
#include <string>
#include <vector>

#include "../../include/thcsox.h"
#include "error.hpp"
#include "mfma.hpp"

using namespace thcsox;

namespace {

constexpr int NT = 256;

__device__ __forceinline__ float silu(float z) { return z / (1.f + __expf(-z)); }
__device__ __forceinline__ float dsilu(float z) {
  const float s = 1.f / (1.f + __expf(-z));
  return s * (1.f + z * (1.f - s));
}

// ---------------------------------------------------------------------------
// The layers' FP32 products, C(i,j) = sum_k A(i,k) B(k,j) on the FP32 matrix cores
// (16x16x4), with what follows each product done on its accumulators:
//   HIDDEN   z = C + bias, h = silu(z)
//   OUTPUT   y = C + bias + x; with a target also d = 2 (y - t) / N and the
//            workgroup's sum of (y - t)^2
//   BACK     dz = C * silu'(z)
//   GRADIENT a slice of k of a weight gradient, stored as a partial sum, and the
//            slice's column sums of A (the bias gradient)
// A is contiguous in k (AC) or i, B in k (BC) or j.  Tiles of T = 32 WT square, four
// waves of T / 2 square, k steps of 32 double-buffered in LDS with one barrier each.
// What bounds them: at batch 4096 and H = 512 a layer is 2.1 GFLOP, 14 us at the
// matrix cores' rate, so what counts is filling the chip (the tile edge and the
// number of slices are picked for about two workgroups per compute unit: a weight
// gradient sums over the whole batch into few tiles) and not passing over the
// activations again.  Training step at m = 64, H = 512, batch 4096: 4.4 ms with
// 64 x 64 tiles over the whole batch and bias, activation and column-sum passes of
// their own (0.75 ms for each column sum).
enum Epilogue { HIDDEN, OUTPUT, BACK, GRADIENT };

struct G32 {
  int M, N, K;
  const float* A; int64_t lda;   // AC: A[i lda + k], else A[k lda + i]
  const float* B; int64_t ldb;   // BC: B[j ldb + k], else B[k ldb + j]
  float* C;                      // h, y or dz [M][N]; GRADIENT: [slices][M N + M]
  float* Z;                      // HIDDEN: z (null: not kept); BACK: z (read)
  const float* bias;             // [N]
  const float* x;                // OUTPUT: [M][N]
  const float* t;                // OUTPUT: target [M][N] or null
  float* D;                      // OUTPUT with a target: [M][N]
  float scale;                   // OUTPUT with a target: 1 / count
  double* part;                  // OUTPUT with a target: [workgroups]
  int kslice;                    // GRADIENT: k per slice (a multiple of GBK)
};

constexpr int GBK = 32;
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));

// LDS panel of T rows x 32 k.  KC: rows of 128 bytes, 16-byte piece c of row r at
// c ^ (r / 2 mod 8); else [k][row] with 16 floats of padding.  A fragment takes k =
// 4 s + g for lane group g: both put its 64 lanes on 64 banks.
template <int T, bool KC> struct GPanel {
  static constexpr int LD = KC ? GBK : T + 16;
  static constexpr int SIZE = KC ? T * GBK : GBK * LD;
};

// ALIGNED: contiguous extents and strides are multiples of 4 and the bases 16-byte
// aligned; else four single loads.
template <int WT, bool AC, bool BC, int EPI, bool ALIGNED>
__global__ __launch_bounds__(NT) void gemm32_kernel(G32 g, int ntj) {
  constexpr int T = 32 * WT;
  using LA = GPanel<T, AC>;
  using LB = GPanel<T, BC>;
  __shared__ __attribute__((aligned(16))) float sA[2][LA::SIZE];
  __shared__ __attribute__((aligned(16))) float sB[2][LB::SIZE];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wr = wave >> 1, wc = wave & 1;
  const int i0 = (int)(blockIdx.x / ntj) * T, j0 = (int)(blockIdx.x % ntj) * T;
  const int k_lo = EPI == GRADIENT ? blockIdx.y * g.kslice : 0;
  const int k_hi = EPI == GRADIENT ? min(g.K, k_lo + g.kslice) : g.K;

  // four consecutive elements from x on, addresses clamped into [0, lim)
  auto quad = [&](const float* p, int x, int lim) -> f4 {
    if (ALIGNED) return *reinterpret_cast<const f4*>(p + min(x, lim - 4));
    return f4{p[min(x, lim - 1)], p[min(x + 1, lim - 1)], p[min(x + 2, lim - 1)],
              p[min(x + 3, lim - 1)]};
  };
  f4 ra[WT], rb[WT];
  auto fetch = [&](bool kc, const float* P, int64_t ld, int r0, int rows, int k0, int e) -> f4 {
    if (kc) return quad(P + (int64_t)min(r0 + (e >> 3), rows - 1) * ld, k0 + 4 * (e & 7), g.K);
    return quad(P + (int64_t)min(k0 + e / (T / 4), g.K - 1) * ld, r0 + 4 * (e % (T / 4)), rows);
  };
  auto load = [&](int k0) {
#pragma unroll
    for (int t = 0; t < WT; ++t) {
      ra[t] = fetch(AC, g.A, g.lda, i0, g.M, k0, tid + NT * t);
      rb[t] = fetch(BC, g.B, g.ldb, j0, g.N, k0, tid + NT * t);
    }
  };
  // store one quad, zero past k_hi (what lies past M or N only reaches outputs that
  // are not stored)
  auto put = [&](bool kc, float* s, int ld, int e, int k0, f4 v) {
    if (kc) {
      const int r = e >> 3, c = e & 7, k = k0 + 4 * c;
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] = k + q < k_hi ? v[q] : 0.f;
      *reinterpret_cast<f4*>(s + r * GBK + ((c ^ ((r >> 1) & 7)) << 2)) = v;
    } else {
      const int kk = e / (T / 4);
      if (k0 + kk >= k_hi) v = f4{0.f, 0.f, 0.f, 0.f};
      *reinterpret_cast<f4*>(s + kk * ld + 4 * (e % (T / 4))) = v;
    }
  };
  auto store = [&](int buf, int k0) {
#pragma unroll
    for (int t = 0; t < WT; ++t) {
      put(AC, sA[buf], LA::LD, tid + NT * t, k0, ra[t]);
      put(BC, sB[buf], LB::LD, tid + NT * t, k0, rb[t]);
    }
  };
  const int fr = lane & 15, fg = lane >> 4;
  auto frag = [&](bool kc, const float* s, int ld, int r, int st) -> float {
    return kc ? s[r * GBK + ((st ^ ((r >> 1) & 7)) << 2) + fg] : s[(4 * st + fg) * ld + r];
  };

  // acc[ti][tj]: the tile's transpose, so that a lane holds four consecutive j of row
  // i = 16 ti + lane % 16
  f4 acc[WT][WT];
#pragma unroll
  for (int ti = 0; ti < WT; ++ti)
#pragma unroll
    for (int tj = 0; tj < WT; ++tj) acc[ti][tj] = f4{0.f, 0.f, 0.f, 0.f};
  float csum = 0.f;   // GRADIENT, first column of tiles: thread i < T sums row i of A

  load(k_lo);
  store(0, k_lo);
  if (k_lo + GBK < k_hi) load(k_lo + GBK);
  __syncthreads();
  int cur = 0;
  for (int k0 = k_lo; k0 < k_hi; k0 += GBK, cur ^= 1) {
    if (k0 + GBK < k_hi) store(cur ^ 1, k0 + GBK);
    if (k0 + 2 * GBK < k_hi) load(k0 + 2 * GBK);
#pragma unroll
    for (int st = 0; st < GBK / 4; ++st) {
      float a[WT], b[WT];
#pragma unroll
      for (int t = 0; t < WT; ++t) {
        a[t] = frag(AC, sA[cur], LA::LD, 16 * (WT * wr + t) + fr, st);
        b[t] = frag(BC, sB[cur], LB::LD, 16 * (WT * wc + t) + fr, st);
      }
#pragma unroll
      for (int ti = 0; ti < WT; ++ti)
#pragma unroll
        for (int tj = 0; tj < WT; ++tj) acc[ti][tj] = mfma1(b[tj], a[ti], acc[ti][tj]);
    }
    if (EPI == GRADIENT && j0 == 0 && tid < T) {
#pragma unroll 8
      for (int k = 0; k < GBK; ++k) csum += sA[cur][k * LA::LD + tid];
    }
    __syncthreads();
  }

  double sse = 0.0;
  const int64_t slice = EPI == GRADIENT ? (int64_t)blockIdx.y * ((int64_t)g.M * g.N + g.M) : 0;
#pragma unroll
  for (int ti = 0; ti < WT; ++ti) {
    const int i = i0 + 16 * (WT * wr + ti) + fr;
    if (i >= g.M) continue;
#pragma unroll
    for (int tj = 0; tj < WT; ++tj) {
      const int j = j0 + 16 * (WT * wc + tj) + 4 * fg;
      if (j >= g.N) continue;
      const int64_t at = (int64_t)i * g.N + j;
      const bool whole = j + 3 < g.N;
      auto get = [&](const float* p) -> f4 {
        if (whole) return *reinterpret_cast<const f4u*>(p);
        return f4{p[0], j + 1 < g.N ? p[1] : 0.f, j + 2 < g.N ? p[2] : 0.f, 0.f};
      };
      auto set = [&](float* p, f4 v) {
        if (whole) {
          *reinterpret_cast<f4u*>(p) = v;
        } else {
          p[0] = v[0];
          if (j + 1 < g.N) p[1] = v[1];
          if (j + 2 < g.N) p[2] = v[2];
        }
      };
      f4 v = acc[ti][tj];
      if constexpr (EPI == HIDDEN) {
        v += get(g.bias + j);
        if (g.Z != nullptr) set(g.Z + at, v);
        set(g.C + at, f4{silu(v[0]), silu(v[1]), silu(v[2]), silu(v[3])});
      } else if constexpr (EPI == OUTPUT) {
        v += get(g.x + at) + get(g.bias + j);
        if (g.C != nullptr) set(g.C + at, v);
        if (g.t != nullptr) {
          const f4 r = v - get(g.t + at);
          set(g.D + at, 2.f * r * g.scale);
#pragma unroll
          for (int q = 0; q < 4; ++q)
            if (j + q < g.N) sse += (double)r[q] * r[q];
        }
      } else if constexpr (EPI == BACK) {
        const f4 z = get(g.Z + at);
        set(g.C + at, f4{v[0] * dsilu(z[0]), v[1] * dsilu(z[1]), v[2] * dsilu(z[2]),
                         v[3] * dsilu(z[3])});
      } else {
        set(g.C + slice + at, v);
      }
    }
  }
  if (EPI == GRADIENT && j0 == 0 && tid < T && i0 + tid < g.M)
    g.C[slice + (int64_t)g.M * g.N + i0 + tid] = csum;
  if (EPI == OUTPUT && g.t != nullptr) {
    __shared__ double red[NT];
    red[tid] = sse;
    __syncthreads();
    for (int o = NT / 2; o > 0; o >>= 1) {
      if (tid < o) red[tid] += red[tid + o];
      __syncthreads();
    }
    if (tid == 0) g.part[blockIdx.x] = red[0];
  }
}

int64_t tiles_of(int M, int N, int T) {
  return (((int64_t)M + T - 1) / T) * (((int64_t)N + T - 1) / T);
}

// Tile edge of a product that is not sliced: the least of rounds of tiles over 256
// compute units x tile area x the cost per element of that tile relative to the
// largest (smaller tiles load more per product).
int tile_edge(int M, int N) {
  auto cost = [&](int T, double rel) {
    return std::ceil(tiles_of(M, N, T) / 256.0) * (double)T * T * rel;
  };
  const double c4 = cost(128, 1.0), c2 = cost(64, 1.2), c1 = cost(32, 1.8);
  return c4 <= c2 && c4 <= c1 ? 128 : c2 <= c1 ? 64 : 32;
}

// Slices of k for a weight gradient of M x N tiles of 64: about 512 workgroups, at
// most 64 slices, each of at least two k steps
constexpr int MAX_SLICES = 64;
int slices_of(int M, int N, int K) {
  const int want = (int)std::min<int64_t>(MAX_SLICES, std::max<int64_t>(1, 512 / tiles_of(M, N, 64)));
  return std::max(1, std::min(want, K / (2 * GBK)));
}

template <bool AC, bool BC, int EPI>
hipError_t gemm32(const G32& g, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0 || g.K <= 0) return hipErrorInvalidValue;
  auto four = [](int64_t v) { return (v & 3) == 0; };
  const bool al = four(AC ? g.K : g.M) && four(BC ? g.K : g.N) && four(g.lda) && four(g.ldb) &&
                  (reinterpret_cast<uintptr_t>(g.A) & 15) == 0 &&
                  (reinterpret_cast<uintptr_t>(g.B) & 15) == 0;
  const int T = EPI == GRADIENT ? 64 : tile_edge(g.M, g.N);
  const int64_t tiles = tiles_of(g.M, g.N, T);
  // (a launch of more than 2^32 - 1 threads would be cut short without an error)
  if (tiles > 0xffffffffLL / NT) return hipErrorInvalidValue;
  const dim3 grid((unsigned)tiles, EPI == GRADIENT ? (g.K + g.kslice - 1) / g.kslice : 1);
  const int ntj = (g.N + T - 1) / T;
  if (T == 64) {
    if (al) gemm32_kernel<2, AC, BC, EPI, true><<<grid, NT, 0, s>>>(g, ntj);
    else gemm32_kernel<2, AC, BC, EPI, false><<<grid, NT, 0, s>>>(g, ntj);
  } else if constexpr (EPI != GRADIENT) {
    if (T == 128) {
      if (al) gemm32_kernel<4, AC, BC, EPI, true><<<grid, NT, 0, s>>>(g, ntj);
      else gemm32_kernel<4, AC, BC, EPI, false><<<grid, NT, 0, s>>>(g, ntj);
    } else {
      if (al) gemm32_kernel<1, AC, BC, EPI, true><<<grid, NT, 0, s>>>(g, ntj);
      else gemm32_kernel<1, AC, BC, EPI, false><<<grid, NT, 0, s>>>(g, ntj);
    }
  }
  return hipGetLastError();
}

// The three layers' weight and bias gradients summed over their slices, in order,
// into the packed array (W, b of each layer follow each other in both), and the
// loss over its workgroups' sums (by the last workgroup).
struct SliceSums {
  const float* src[3];
  int64_t len[3];      // M N + M
  int slices[3];
  float* out;          // packed gradients
  const double* part; int nparts; double* loss;
};
__global__ __launch_bounds__(NT) void sum_slices(SliceSums a, int64_t total) {
  if (blockIdx.x == gridDim.x - 1) {
    __shared__ double red[NT];
    double s = 0.0;
    for (int i = threadIdx.x; i < a.nparts; i += NT) s += a.part[i];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int o = NT / 2; o > 0; o >>= 1) {
      if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
      __syncthreads();
    }
    if (threadIdx.x == 0) *a.loss = red[0];
    return;
  }
  for (int64_t e = (int64_t)blockIdx.x * NT + threadIdx.x; e < total;
       e += (int64_t)(gridDim.x - 1) * NT) {
    int64_t at = e;
    int l = 0;
    while (at >= a.len[l]) at -= a.len[l++];
    float s = 0.f;
#pragma unroll 8
    for (int q = 0; q < a.slices[l]; ++q) s += a.src[l][(int64_t)q * a.len[l] + at];
    a.out[e] = s;
  }
}

__global__ void adam(float* p, const float* g, float* m1, float* m2, int64_t count, float lr,
                     float b1, float b2, float eps, float c1, float c2) {
  for (int64_t e = (int64_t)blockIdx.x * NT + threadIdx.x; e < count; e += (int64_t)gridDim.x * NT) {
    const float gi = g[e];
    const float a = b1 * m1[e] + (1.f - b1) * gi;
    const float v = b2 * m2[e] + (1.f - b2) * gi * gi;
    m1[e] = a;
    m2[e] = v;
    p[e] -= lr * (a / c1) / (sqrtf(v / c2) + eps);
  }
}

// scale[e] = max_k |S[k][e]| over the m tau points of pair e (1 if all zero);
// consecutive threads take consecutive pairs, so every read of a tau slice is coalesced
__global__ void pair_scale_kernel(const double* S, int m, int64_t aa, double* scale) {
  for (int64_t e = (int64_t)blockIdx.x * NT + threadIdx.x; e < aa; e += (int64_t)gridDim.x * NT) {
    double mx = 0.0;
#pragma unroll 8
    for (int k = 0; k < m; ++k) mx = fmax(mx, fabs(S[(int64_t)k * aa + e]));
    scale[e] = mx > 0.0 ? mx : 1.0;
  }
}

// The network's rows x[b][k] and the THC self-energy's slices S[k][pair] are each other's
// transposes: blocks of 64 pairs x 64 tau points go through LDS, so that both sides
// are touched in whole lines (S in runs of 64 pairs, x in runs of up to 64 tau points).
// naux = 505, 64 tau points: 37 us each, 5.3 TB/s (106 and 309 us with one side strided).
// Few tau points leave most of a block's threads idle, few pairs most of the chip, and
// listed pairs are scattered anyhow: there one thread per element is faster (the rules
// are with gather_by_blocks and scatter_by_blocks).
constexpr int PT = 64;             // pairs and tau points per block
constexpr int PTS = NT / PT;       // rows of a block per pass

// x[b][k] = S[k][pair_b] / scale[pair_b]; pair_b = pairs[b] (or b if pairs is null): one
// thread per element, consecutive threads along tau
__global__ void pair_gather_kernel(const double* S, int m, int64_t aa, const double* scale,
                                   const int64_t* pairs, int64_t npairs, float* x) {
  for (int64_t e = (int64_t)blockIdx.x * NT + threadIdx.x; e < npairs * m;
       e += (int64_t)gridDim.x * NT) {
    const int64_t b = e / m;
    const int k = (int)(e % m);
    const int64_t pr = pairs ? pairs[b] : b;
    x[e] = (pr >= 0 && pr < aa) ? (float)(S[(int64_t)k * aa + pr] / scale[pr]) : 0.f;
  }
}

// the same by blocks
__global__ __launch_bounds__(NT) void pair_gather_blocks(const double* __restrict__ S, int m,
                                                         int64_t aa,
                                                         const double* __restrict__ scale,
                                                         const int64_t* __restrict__ pairs,
                                                         int64_t npairs, int64_t first,
                                                         float* __restrict__ x) {
  __shared__ float t[PT][PT + 1];   // [tau][pair]
  const int tx = threadIdx.x % PT, ty = threadIdx.x / PT;
  const int64_t b0 = first + (int64_t)blockIdx.x * PT;
  const int64_t b = b0 + tx;
  const int64_t pr = b < npairs ? (pairs ? pairs[b] : b) : -1;
  const bool in = pr >= 0 && pr < aa;   // a pair outside the array reads as zero
  const double sc = in ? scale[pr] : 1.0;
  for (int k0 = 0; k0 < m; k0 += PT) {
    const int nk = min(PT, m - k0);
    double v[PT / PTS];
#pragma unroll
    for (int e = 0; e < PT / PTS; ++e)
      v[e] = S[(int64_t)(k0 + min(ty + e * PTS, nk - 1)) * aa + (in ? pr : 0)];
#pragma unroll
    for (int e = 0; e < PT / PTS; ++e)
      if (ty + e * PTS < nk) t[ty + e * PTS][tx] = in ? (float)(v[e] / sc) : 0.f;
    __syncthreads();
    // consecutive threads along tau, then along pairs
    const int rows = (int)(npairs - b0 < PT ? npairs - b0 : PT);
    for (int e = threadIdx.x; e < rows * nk; e += NT) {
      const int r = e / nk, k = e - r * nk;
      x[(b0 + r) * m + k0 + k] = t[k][r];
    }
    __syncthreads();
  }
}

// S[k][pair] = y[pair][k] * scale[pair] for every pair: one thread per element, consecutive
// threads along pairs
__global__ void pair_scatter_kernel(const float* y, int m, int64_t aa, const double* scale,
                                    double* S) {
  for (int64_t e = (int64_t)blockIdx.x * NT + threadIdx.x; e < aa * m; e += (int64_t)gridDim.x * NT) {
    const int k = (int)(e / aa);
    const int64_t pr = e % aa;
    S[e] = (double)y[pr * m + k] * scale[pr];
  }
}

// the same by blocks
__global__ __launch_bounds__(NT) void pair_scatter_blocks(const float* __restrict__ y, int m,
                                                          int64_t aa,
                                                          const double* __restrict__ scale,
                                                          int64_t first, double* __restrict__ S) {
  __shared__ float t[PT][PT + 1];   // [tau][pair]
  const int tx = threadIdx.x % PT, ty = threadIdx.x / PT;
  const int64_t p0 = first + (int64_t)blockIdx.x * PT;
  const int rows = (int)(aa - p0 < PT ? aa - p0 : PT);
  const double sc = tx < rows ? scale[p0 + tx] : 0.0;
  for (int k0 = 0; k0 < m; k0 += PT) {
    const int nk = min(PT, m - k0);
    float v[PT * PT / NT];   // all in flight together (addresses clamped into the block)
#pragma unroll
    for (int i = 0; i < PT * PT / NT; ++i) {
      const int e = min((int)threadIdx.x + i * NT, rows * nk - 1), r = e / nk;
      v[i] = y[(p0 + r) * m + k0 + e - r * nk];
    }
#pragma unroll
    for (int i = 0; i < PT * PT / NT; ++i) {
      const int e = (int)threadIdx.x + i * NT, r = e / nk;
      if (e < rows * nk) t[e - r * nk][r] = v[i];
    }
    __syncthreads();
    if (tx < rows)
      for (int k = ty; k < nk; k += PTS)
        S[(int64_t)(k0 + k) * aa + p0 + tx] = (double)t[k][tx] * sc;
    __syncthreads();
  }
}

// Runs go(first pair, workgroups) for the two kernels by blocks, a workgroup per block of
// pairs, in as many launches as it takes: one of more than 2^32 threads drops the excess
// without an error (a loop over blocks in the kernels cost 6 to 9 % at 16 to 32 tau points).
template <typename Go>
void by_blocks(int64_t npairs, Go go) {
  constexpr int64_t MOST = int64_t(1) << 23;
  for (int64_t first = 0; first < npairs; first += MOST * PT)
    go(first, (unsigned)std::min(MOST, (npairs - first + PT - 1) / PT));
}

// Where blocks pay (us, per element against by blocks; aa pairs in S):
//   all pairs, aa = 255025: m = 16 13.5 / 15.1, 24 23.2 / 18.1; 40000: 32 5.8 / 6.7, 48 10.4 /
//   8.0; 10201: 64 4.4 / 5.9, 95 9.4 / 8.1; with S beyond the 256 MB cache (aa = 3.24e6):
//   m = 12 138 / 164, 16 199 / 179
//   listed pairs (aa = 255025): 4096: m = 64 4.5 / 10.1, 95 9.4 / 16.1; 32768: 64 42 / 41,
//   95 62 / 57; 262144: 16 75 / 73, 64 318 / 297 (aa = 10201: 16 21 / 30, 64 101 / 97)
bool gather_by_blocks(bool listed, int64_t npairs, int64_t aa, int m) {
  if (listed) return (npairs >= 32768 && m > 64) || (npairs >= 131072 && m >= 48);
  return (m >= 24 && (m > 64 || npairs * m >= 1500000)) || (m >= 16 && aa * m > 32000000);
}
//   scatter, aa = 255025: m = 8 12.0 / 19.7, 12 24.9 / 20.7; 40000: 16 4.6 / 6.2, 24 7.4 /
//   7.0; 10201: 100 7.3 / 8.1
bool scatter_by_blocks(int64_t aa, int m) { return m >= 12 && aa >= 20000 && aa * m >= 900000; }

unsigned blocks_for(int64_t n) {
  int64_t b = (n + NT - 1) / NT;
  return (unsigned)(b > 4096 ? 4096 : (b < 1 ? 1 : b));
}

// ---------------------------------------------------------------------------
// Inference with bf16 weights: one fused kernel per 64 or 128 rows on the bf16 matrix
// cores (16x16x32, FP32 accumulation); the hidden activations never leave LDS.
// Each layer's input (x, h1, h2) is rounded to bf16 (nearest, ties to even);
// bias, silu and the residual add on the exact FP32 x stay in FP32.
//
// Eight waves: in layers 1 and 2 wave w owns the hidden units [16 HT w,
// 16 HT (w + 1)) of all rows, taking the weight rows as the MFMA's first
// operand and the activation rows (from LDS) as its second, so a lane's four
// results are four consecutive hidden units of one row: one 8-byte LDS write of
// the next layer's bf16 input.  Layer 3's output tiles are dealt to the waves; a
// lane's results are four consecutive outputs of one row, one 16-byte store.
// What bounds it: the weights come from L2 for every block of rows, one flop per row
// and byte, so 128 rows (all of the LDS at H = 512) halve the 17 TB/s that 64 rows
// need at the 1127 TFLOP/s of a large library product; the next k step's weights are
// loaded while one is multiplied.  m = 64, H = 512, 255025 rows: 373 us (563 with 64 rows
// and no prefetch), about half of it the silu of two hidden layers, which no wave's
// products overlap.
constexpr int INW = 8, INTH = 64 * INW;
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ bf16x4 to_bf16x4(float a, float b, float c, float d) {
  return bf16x4{(__bf16)a, (__bf16)b, (__bf16)c, (__bf16)d};
}

template <int HT, int MT, int RB>   // hidden width H = 128 HT, m = 16 MT, RB rows per workgroup
__global__ __launch_bounds__(INTH) void mlp_infer_bf16_kernel(
    const float* __restrict__ x, float* __restrict__ y, int64_t batch,
    const __bf16* __restrict__ W1, const float* __restrict__ b1,
    const __bf16* __restrict__ W2, const float* __restrict__ b2,
    const __bf16* __restrict__ W3, const float* __restrict__ b3) {
  constexpr int H = 128 * HT, m = 16 * MT, RT = RB / 16;   // row tiles
  constexpr int XLD = m + 8, HLD = H + 8;   // padded rows (in bf16): 16-lane reads hit distinct banks
  __shared__ __attribute__((aligned(16))) __bf16 xs[RB * XLD];
  __shared__ __attribute__((aligned(16))) __bf16 hs[RB * HLD];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t r0 = (int64_t)blockIdx.x * RB;
  const int rows = (int)(batch - r0 < RB ? batch - r0 : RB);
  for (int e = tid; e < RB * m / 4; e += INTH) {
    const int r = e / (m / 4), c = 4 * (e % (m / 4));
    const f4 v = r < rows ? *reinterpret_cast<const f4*>(x + (r0 + r) * m + c) : f4{0.f, 0.f, 0.f, 0.f};
    *reinterpret_cast<bf16x4*>(&xs[r * XLD + c]) = to_bf16x4(v[0], v[1], v[2], v[3]);
  }
  __syncthreads();
  const int fr = lane & 15, fk = 8 * (lane >> 4);   // fragment row, k offset
  const int hid0 = 16 * HT * wave;
  f4 acc[HT][RT];
  // one hidden layer: acc = W rows [hid0, hid0 + 16 HT) . act^T over K, act in LDS
  auto layer = [&](const __bf16* __restrict__ W, const __bf16* act, int ld, int K) {
#pragma unroll
    for (int t = 0; t < HT; ++t)
#pragma unroll
      for (int p = 0; p < RT; ++p) acc[t][p] = f4{0.f, 0.f, 0.f, 0.f};
    bf16x8 next[HT];
#pragma unroll
    for (int t = 0; t < HT; ++t)
      next[t] = *reinterpret_cast<const bf16x8*>(W + (int64_t)(hid0 + 16 * t + fr) * K + fk);
    for (int k0 = 0; k0 < K; k0 += 32) {
      bf16x8 a[HT], b[RT];
#pragma unroll
      for (int t = 0; t < HT; ++t) a[t] = next[t];
      const int kn = min(k0 + 32, K - 32);   // (the last step loads its own again)
#pragma unroll
      for (int t = 0; t < HT; ++t)
        next[t] = *reinterpret_cast<const bf16x8*>(W + (int64_t)(hid0 + 16 * t + fr) * K + kn + fk);
#pragma unroll
      for (int p = 0; p < RT; ++p)
        b[p] = *reinterpret_cast<const bf16x8*>(&act[(16 * p + fr) * ld + k0 + fk]);
#pragma unroll
      for (int t = 0; t < HT; ++t)
#pragma unroll
        for (int p = 0; p < RT; ++p) acc[t][p] = mfma1(a[t], b[p], acc[t][p]);
    }
  };
  // h = bf16(silu(acc + bias)) into hs[row][hid]
  auto to_hidden = [&](const float* __restrict__ bias) {
#pragma unroll
    for (int t = 0; t < HT; ++t) {
      const int h = hid0 + 16 * t + 4 * (lane >> 4);
      const f4 bv = *reinterpret_cast<const f4*>(bias + h);
#pragma unroll
      for (int p = 0; p < RT; ++p)
        *reinterpret_cast<bf16x4*>(&hs[(16 * p + fr) * HLD + h]) =
            to_bf16x4(silu(acc[t][p][0] + bv[0]), silu(acc[t][p][1] + bv[1]),
                      silu(acc[t][p][2] + bv[2]), silu(acc[t][p][3] + bv[3]));
    }
  };
  layer(W1, xs, XLD, m);
  to_hidden(b1);
  __syncthreads();
  layer(W2, hs, HLD, H);
  __syncthreads();   // every wave has read all of h1
  to_hidden(b2);
  __syncthreads();
  // layer 3: of the MT x RT output tiles a wave takes one block of 16 outputs and
  // RT MT / 8 of its row tiles, so its weights serve them all
  constexpr int PT3 = RT * MT / INW;   // row tiles per wave
  static_assert(PT3 >= 1 && RT % PT3 == 0, "the output tiles are dealt out evenly");
  const int o = wave / (RT / PT3), p3 = wave % (RT / PT3) * PT3;
  f4 c[PT3];
#pragma unroll
  for (int p = 0; p < PT3; ++p) c[p] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
  for (int k0 = 0; k0 < H; k0 += 32) {
    const bf16x8 a = *reinterpret_cast<const bf16x8*>(W3 + (int64_t)(16 * o + fr) * H + k0 + fk);
#pragma unroll
    for (int p = 0; p < PT3; ++p)
      c[p] = mfma1(a, *reinterpret_cast<const bf16x8*>(&hs[(16 * (p3 + p) + fr) * HLD + k0 + fk]), c[p]);
  }
#pragma unroll
  for (int p = 0; p < PT3; ++p) {
    const int row = 16 * (p3 + p) + fr, out0 = 16 * o + 4 * (lane >> 4);
    if (row < rows) {
      const f4 xv = *reinterpret_cast<const f4*>(x + (r0 + row) * m + out0);
      const f4 bv = *reinterpret_cast<const f4*>(b3 + out0);
      *reinterpret_cast<f4*>(y + (r0 + row) * m + out0) = xv + (c[p] + bv);
    }
  }
}

// FP32 -> bf16 (nearest, ties to even)
__global__ void round_bf16_kernel(const float* src, __bf16* dst, int64_t n) {
  for (int64_t e = (int64_t)blockIdx.x * NT + threadIdx.x; e < n; e += (int64_t)gridDim.x * NT)
    dst[e] = (__bf16)src[e];
}

}  // namespace

struct thcsox_mlp_s {
  int m = 0, H = 0, maxb = 0;
  int64_t np = 0;
  int64_t oW1, ob1, oW2, ob2, oW3, ob3;
  hipStream_t stream = nullptr;
  float *P = nullptr, *Gr = nullptr, *M1 = nullptr, *M2 = nullptr;
  float *Z1 = nullptr, *H1 = nullptr, *Z2 = nullptr, *H2 = nullptr, *D = nullptr;
  float *DZ1 = nullptr, *DZ2 = nullptr;
  float* slices[3] = {};     // partial weight and bias gradients of each layer
  double *part = nullptr, *loss = nullptr;
  __bf16* Pb = nullptr;      // bf16 copy of the parameters (inference), made on first use
  int pb_step = -1;          // the training step it was rounded at
  int step = 0;
  std::vector<void*> allocs;
  ~thcsox_mlp_s() {
    for (void* p : allocs) (void)hipFree(p);
  }
};

namespace {

template <typename T>
int malloc_into(thcsox_mlp_s* q, T** p, size_t count) {
  void* v = nullptr;
  hipError_t e = hipMalloc(&v, std::max<size_t>(16, count * sizeof(T)));
  if (e != hipSuccess) {
    (void)hipGetLastError();
    return set_error(THCSOX_ENOMEM, std::string("hipMalloc failed: ") + hipGetErrorString(e));
  }
  q->allocs.push_back(v);
  *p = static_cast<T*>(v);
  return 0;
}

#define MTRY(expr)                                                                        \
  do {                                                                                    \
    hipError_t e_ = (expr);                                                               \
    if (e_ != hipSuccess)                                                                 \
      return set_error(THCSOX_EDEVICE, std::string(#expr) + ": " + hipGetErrorString(e_)); \
  } while (0)

// The hidden layers for rows [0, B) of x (keep: z1, z2 for a backward pass), then
// y = the output, or (t given) d and the loss sums of the batch.
int forward(thcsox_mlp_s* q, const float* x, float* y, const float* t, int B, bool keep) {
  const hipStream_t s = q->stream;
  const int m = q->m, H = q->H;
  G32 g{};
  g.M = B; g.N = H; g.K = m; g.A = x; g.lda = m; g.B = q->P + q->oW1; g.ldb = m;
  g.bias = q->P + q->ob1; g.C = q->H1; g.Z = keep ? q->Z1 : nullptr;
  MTRY((gemm32<true, true, HIDDEN>(g, s)));
  g.K = H; g.A = q->H1; g.lda = H; g.B = q->P + q->oW2; g.ldb = H;
  g.bias = q->P + q->ob2; g.C = q->H2; g.Z = keep ? q->Z2 : nullptr;
  MTRY((gemm32<true, true, HIDDEN>(g, s)));
  g.N = m; g.A = q->H2; g.B = q->P + q->oW3; g.bias = q->P + q->ob3; g.x = x; g.C = y; g.Z = nullptr;
  g.t = t; g.D = q->D; g.scale = 1.f / (float)((int64_t)B * m); g.part = q->part;
  MTRY((gemm32<true, true, OUTPUT>(g, s)));
  return 0;
}

// the shape of layer l's weight gradient
void layer_shape(const thcsox_mlp_s* q, int l, int* M, int* N) {
  *M = l == 2 ? q->m : q->H;
  *N = l == 0 ? q->m : q->H;
}

// gradients of the mean-squared loss into q->Gr, sum of squares into q->loss
int backward(thcsox_mlp_s* q, const float* x, int B) {
  const hipStream_t s = q->stream;
  const int m = q->m, H = q->H;
  SliceSums ss{};
  // g[i][j] = sum_b dz[b][i] in[b][j] in slices of the batch
  auto weights = [&](int l, const float* dz, const float* in) -> hipError_t {
    G32 g{};
    layer_shape(q, l, &g.M, &g.N);
    g.K = B; g.A = dz; g.lda = g.M; g.B = in; g.ldb = g.N; g.C = q->slices[l];
    const int n = slices_of(g.M, g.N, B);
    g.kslice = ((B + n - 1) / n + GBK - 1) / GBK * GBK;
    ss.src[l] = g.C;
    ss.len[l] = (int64_t)g.M * g.N + g.M;
    ss.slices[l] = (B + g.kslice - 1) / g.kslice;
    return gemm32<false, false, GRADIENT>(g, s);
  };
  // dz_out[b][j] = silu'(z[b][j]) sum_i dz[b][i] W[i][j]
  auto back = [&](int l, const float* dz, const float* W, float* z, float* out) -> hipError_t {
    G32 g{};
    g.M = B;
    layer_shape(q, l, &g.K, &g.N);
    g.A = dz; g.lda = g.K; g.B = W; g.ldb = g.N; g.Z = z; g.C = out;
    return gemm32<true, false, BACK>(g, s);
  };
  MTRY(weights(2, q->D, q->H2));
  MTRY(back(2, q->D, q->P + q->oW3, q->Z2, q->DZ2));
  MTRY(weights(1, q->DZ2, q->H1));
  MTRY(back(1, q->DZ2, q->P + q->oW2, q->Z1, q->DZ1));
  MTRY(weights(0, q->DZ1, x));
  ss.out = q->Gr;
  ss.part = q->part;
  ss.nparts = (int)tiles_of(B, m, tile_edge(B, m));
  ss.loss = q->loss;
  sum_slices<<<blocks_for(q->np) + 1, NT, 0, s>>>(ss, q->np);
  MTRY(hipGetLastError());
  return 0;
}

}  // namespace

extern "C" {

static int thcsox_mlp_create_impl(thcsox_mlp_t* out, int m, int hidden, int max_batch,
                      const float* params_host, void* hip_stream) {
  clear_error();
  if (out == nullptr || params_host == nullptr) return set_error(THCSOX_EINVAL, "NULL argument");
  *out = nullptr;
  if (m <= 0 || hidden <= 0 || max_batch <= 0) return set_error(THCSOX_EINVAL, "bad sizes");
  auto* q = new thcsox_mlp_s();
  q->m = m; q->H = hidden; q->maxb = max_batch;
  q->stream = static_cast<hipStream_t>(hip_stream);
  const int64_t H = hidden;
  q->oW1 = 0; q->ob1 = q->oW1 + H * m; q->oW2 = q->ob1 + H; q->ob2 = q->oW2 + H * H;
  q->oW3 = q->ob2 + H; q->ob3 = q->oW3 + (int64_t)m * H; q->np = q->ob3 + m;
  const int64_t B = max_batch;
  int rc;
  if ((rc = malloc_into(q, &q->P, q->np)) || (rc = malloc_into(q, &q->Gr, q->np)) ||
      (rc = malloc_into(q, &q->M1, q->np)) || (rc = malloc_into(q, &q->M2, q->np)) ||
      (rc = malloc_into(q, &q->Z1, B * H)) || (rc = malloc_into(q, &q->H1, B * H)) ||
      (rc = malloc_into(q, &q->Z2, B * H)) || (rc = malloc_into(q, &q->H2, B * H)) ||
      (rc = malloc_into(q, &q->D, B * m)) ||
      (rc = malloc_into(q, &q->DZ1, B * H)) || (rc = malloc_into(q, &q->DZ2, B * H)) ||
      (rc = malloc_into(q, &q->part, tiles_of(max_batch, m, 32))) ||
      (rc = malloc_into(q, &q->loss, 1))) {
    delete q;
    return rc;
  }
  for (int l = 0; l < 3; ++l) {
    int M, N;
    layer_shape(q, l, &M, &N);
    const int n = slices_of(M, N, max_batch);   // no smaller batch takes more
    if ((rc = malloc_into(q, &q->slices[l], (size_t)n * ((size_t)M * N + M)))) {
      delete q;
      return rc;
    }
  }
  hipError_t e;
  if ((e = hipMemcpyAsync(q->P, params_host, sizeof(float) * q->np, hipMemcpyHostToDevice,
                          q->stream)) ||
      (e = hipMemsetAsync(q->M1, 0, sizeof(float) * q->np, q->stream)) ||
      (e = hipMemsetAsync(q->M2, 0, sizeof(float) * q->np, q->stream)) ||
      (e = hipStreamSynchronize(q->stream))) {
    delete q;
    return set_error(THCSOX_EDEVICE, std::string("mlp create: ") + hipGetErrorString(e));
  }
  *out = q;
  return 0;
}

int thcsox_mlp_create(thcsox_mlp_t* out, int m, int hidden, int max_batch,
                      const float* params_host, void* hip_stream) {
  try {   // host containers: no exception may cross the C interface
    return thcsox_mlp_create_impl(out, m, hidden, max_batch, params_host, hip_stream);
  } catch (const std::bad_alloc&) {
    return set_error(THCSOX_ENOMEM, "host allocation failed");
  }
}

int thcsox_mlp_forward(thcsox_mlp_t q, const float* x_dev, float* y_dev, int batch) {
  clear_error();
  if (q == nullptr || x_dev == nullptr || y_dev == nullptr || batch < 0)
    return set_error(THCSOX_EINVAL, "bad argument");
  for (int b0 = 0; b0 < batch; b0 += q->maxb) {
    const int B = std::min(q->maxb, batch - b0);
    const int rc = forward(q, x_dev + (int64_t)b0 * q->m, y_dev + (int64_t)b0 * q->m, nullptr, B,
                           false);
    if (rc) return rc;
  }
  return 0;
}

int thcsox_mlp_gradients(thcsox_mlp_t q, const float* x_dev, const float* target_dev, int batch,
                         float* grads_host, double* loss_host) {
  clear_error();
  if (q == nullptr || x_dev == nullptr || target_dev == nullptr || batch <= 0 ||
      batch > q->maxb)
    return set_error(THCSOX_EINVAL, "bad argument (batch must be in 1..max_batch)");
  int rc = forward(q, x_dev, nullptr, target_dev, batch, true);
  if (rc) return rc;
  if ((rc = backward(q, x_dev, batch))) return rc;
  double sse = 0.0;
  MTRY(hipMemcpyAsync(&sse, q->loss, sizeof(double), hipMemcpyDeviceToHost, q->stream));
  if (grads_host)
    MTRY(hipMemcpyAsync(grads_host, q->Gr, sizeof(float) * q->np, hipMemcpyDeviceToHost,
                        q->stream));
  MTRY(hipStreamSynchronize(q->stream));
  if (loss_host) *loss_host = sse / ((double)batch * q->m);
  return 0;
}

int thcsox_mlp_train_step(thcsox_mlp_t q, const float* x_dev, const float* target_dev, int batch,
                          float lr, double* loss_host) {
  clear_error();
  if (q == nullptr || x_dev == nullptr || target_dev == nullptr || batch <= 0 ||
      batch > q->maxb)
    return set_error(THCSOX_EINVAL, "bad argument (batch must be in 1..max_batch)");
  int rc = forward(q, x_dev, nullptr, target_dev, batch, true);
  if (rc) return rc;
  if ((rc = backward(q, x_dev, batch))) return rc;
  q->step += 1;
  const float b1 = 0.9f, b2 = 0.999f;
  const float c1 = 1.f - std::pow(b1, (float)q->step), c2 = 1.f - std::pow(b2, (float)q->step);
  adam<<<blocks_for(q->np), NT, 0, q->stream>>>(q->P, q->Gr, q->M1, q->M2, q->np, lr, b1, b2,
                                                1e-8f, c1, c2);
  MTRY(hipGetLastError());
  if (loss_host) {
    double sse = 0.0;
    MTRY(hipMemcpyAsync(&sse, q->loss, sizeof(double), hipMemcpyDeviceToHost, q->stream));
    MTRY(hipStreamSynchronize(q->stream));
    *loss_host = sse / ((double)batch * q->m);
  }
  return 0;
}

int thcsox_mlp_forward_bf16(thcsox_mlp_t q, const float* x_dev, float* y_dev, int64_t batch) {
  clear_error();
  if (q == nullptr || batch < 0) return set_error(THCSOX_EINVAL, "bad argument");
  const int HT = q->H / 128, MT = q->m / 16;
  if (q->H % 128 != 0 || (HT != 1 && HT != 2 && HT != 4) || q->m % 16 != 0 ||
      (MT != 2 && MT != 4))
    return set_error(THCSOX_EINVAL, "bf16 inference needs m in {32, 64} and H in {128, 256, 512}");
  if (batch == 0) return 0;
  if (x_dev == nullptr || y_dev == nullptr) return set_error(THCSOX_EINVAL, "NULL argument");
  if (q->Pb == nullptr) {
    void* v = nullptr;
    hipError_t e = hipMalloc(&v, sizeof(__bf16) * (size_t)q->np);
    if (e != hipSuccess) {
      (void)hipGetLastError();
      return set_error(THCSOX_ENOMEM, std::string("hipMalloc failed: ") + hipGetErrorString(e));
    }
    q->allocs.push_back(v);
    q->Pb = static_cast<__bf16*>(v);
  }
  if (q->pb_step != q->step) {
    round_bf16_kernel<<<blocks_for(q->np), NT, 0, q->stream>>>(q->P, q->Pb, q->np);
    MTRY(hipGetLastError());
    q->pb_step = q->step;
  }
  // 128 rows per workgroup where that still fills the chip twice (it then reads the
  // weights half as often), else 64
  const bool big = HT >= 2 && batch >= 2 * 256 * 128;
  const int64_t nblk = (batch + (big ? 127 : 63)) / (big ? 128 : 64);
  if (nblk > 0x7fffffffLL) return set_error(THCSOX_EINVAL, "batch too large");
  const __bf16 *W1 = q->Pb + q->oW1, *W2 = q->Pb + q->oW2, *W3 = q->Pb + q->oW3;
  const float *b1 = q->P + q->ob1, *b2 = q->P + q->ob2, *b3 = q->P + q->ob3;
  auto go = [&](auto kernel) {
    kernel<<<(unsigned)nblk, INTH, 0, q->stream>>>(x_dev, y_dev, batch, W1, b1, W2, b2, W3, b3);
  };
  if (MT == 4) {
    if (HT == 4) big ? go(mlp_infer_bf16_kernel<4, 4, 128>) : go(mlp_infer_bf16_kernel<4, 4, 64>);
    else if (HT == 2) big ? go(mlp_infer_bf16_kernel<2, 4, 128>) : go(mlp_infer_bf16_kernel<2, 4, 64>);
    else go(mlp_infer_bf16_kernel<1, 4, 64>);
  } else {
    if (HT == 4) big ? go(mlp_infer_bf16_kernel<4, 2, 128>) : go(mlp_infer_bf16_kernel<4, 2, 64>);
    else if (HT == 2) big ? go(mlp_infer_bf16_kernel<2, 2, 128>) : go(mlp_infer_bf16_kernel<2, 2, 64>);
    else go(mlp_infer_bf16_kernel<1, 2, 64>);
  }
  MTRY(hipGetLastError());
  return 0;
}

int thcsox_mlp_params(thcsox_mlp_t q, float* params_host) {
  clear_error();
  if (q == nullptr || params_host == nullptr) return set_error(THCSOX_EINVAL, "NULL argument");
  MTRY(hipMemcpyAsync(params_host, q->P, sizeof(float) * q->np, hipMemcpyDeviceToHost, q->stream));
  MTRY(hipStreamSynchronize(q->stream));
  return 0;
}

int thcsox_pair_scale(int m, int naux, const double* S_dev, double* scale_dev, void* hip_stream) {
  clear_error();
  if (m <= 0 || naux <= 0 || S_dev == nullptr || scale_dev == nullptr)
    return set_error(THCSOX_EINVAL, "bad argument");
  const int64_t aa = (int64_t)naux * naux;
  pair_scale_kernel<<<blocks_for(aa), NT, 0, static_cast<hipStream_t>(hip_stream)>>>(
      S_dev, m, aa, scale_dev);
  MTRY(hipGetLastError());
  return 0;
}

int thcsox_pair_gather(int m, int naux, const double* S_dev, const double* scale_dev,
                       const long long* pairs_dev, long long npairs, float* x_dev, void* hip_stream) {
  clear_error();
  const int64_t aa = (int64_t)naux * naux;
  if (m <= 0 || naux <= 0 || S_dev == nullptr || scale_dev == nullptr || x_dev == nullptr ||
      npairs < 0 || (pairs_dev == nullptr && npairs > aa))
    return set_error(THCSOX_EINVAL, "bad argument");
  if (npairs == 0) return 0;
  const int64_t* pairs = reinterpret_cast<const int64_t*>(pairs_dev);
  const hipStream_t s = static_cast<hipStream_t>(hip_stream);
  if (gather_by_blocks(pairs != nullptr, npairs, aa, m))
    by_blocks(npairs, [&](int64_t first, unsigned blocks) {
      pair_gather_blocks<<<blocks, NT, 0, s>>>(S_dev, m, aa, scale_dev, pairs, npairs, first, x_dev);
    });
  else
    pair_gather_kernel<<<blocks_for(npairs * m), NT, 0, s>>>(S_dev, m, aa, scale_dev, pairs, npairs,
                                                             x_dev);
  MTRY(hipGetLastError());
  return 0;
}

int thcsox_pair_scatter(int m, int naux, const float* y_dev, const double* scale_dev,
                        double* S_dev, void* hip_stream) {
  clear_error();
  if (m <= 0 || naux <= 0 || S_dev == nullptr || scale_dev == nullptr || y_dev == nullptr)
    return set_error(THCSOX_EINVAL, "bad argument");
  const int64_t aa = (int64_t)naux * naux;
  const hipStream_t s = static_cast<hipStream_t>(hip_stream);
  if (scatter_by_blocks(aa, m))
    by_blocks(aa, [&](int64_t first, unsigned blocks) {
      pair_scatter_blocks<<<blocks, NT, 0, s>>>(y_dev, m, aa, scale_dev, first, S_dev);
    });
  else
    pair_scatter_kernel<<<blocks_for(aa * m), NT, 0, s>>>(y_dev, m, aa, scale_dev, S_dev);
  MTRY(hipGetLastError());
  return 0;
}

int thcsox_mlp_destroy(thcsox_mlp_t q) {
  if (q == nullptr) return 0;
  (void)hipStreamSynchronize(q->stream);
  delete q;
  return 0;
}

}  // extern "C"
