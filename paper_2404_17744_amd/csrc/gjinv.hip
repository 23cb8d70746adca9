// Batched in-place Gauss-Jordan inversion in FP64, complex (the Dyson equation's
// matrices, one per frequency) or real (1 + V Pi0 of the static screening).
//
// Columns are eliminated in order with partial pivoting, but no row moves: the
// pivot of column c is the largest |a_ic| over the rows not used yet, p_c its row,
// and the finished array S holds the inverse as  A^-1[i][j] = S[p_i][c : p_c = j].
// Panels of bw columns:
//   gj_panel: one workgroup per matrix.  Every thread holds its rows' bw panel
//     elements in registers; a column costs one pivot search (a 64-bit key of the
//     magnitude with its low bits replaced by the row, reduced over the lanes by
//     DPP and over the waves through LDS), the pivot row read from LDS by all, and a
//     rank-1 update in registers.  The panel ends as W, its columns of the product of the panel's
//     elimination matrices.
//   gj_trail: every other column j gets the same eliminations at once,
//     A[:, j] += (W - E) A[p rows, j] with E the unit columns of the panel's pivot
//     rows, as a product on the f64 matrix cores (a complex product is four real
//     ones).  A workgroup owns 32 columns; their pivot rows go to LDS first.
// What bounds it: the trailing update reads and writes each matrix once per panel,
// so wide panels pay (32 columns while a thread's row fits its registers), and it
// keeps the next 16 rows' loads in flight while one group is multiplied (256
// matrices of n = 300: 199 us a panel, 3.7 TB/s; 245 without).  The panel is a serial
// chain of n pivot steps (69 us per 32 columns at n = 300, 49 at n = 77).  Together
// 2.7 ms per 256 matrices of n = 300; 7.6 ms with panels of 8 columns in LDS, row
// swaps in memory and the update on the vector units.
#include <algorithm>

#include "kernels.hpp"
#include "mfma.hpp"

namespace thcsox {
namespace {

constexpr int TCOLS = 32;        // columns per gj_trail workgroup
constexpr int TNT = 256;         // its threads (4 wavefronts)
constexpr int ROW_BITS = 14;     // low bits of a pivot key that hold the row (n <= 9216)
constexpr unsigned long long ROW_MASK = (1ull << ROW_BITS) - 1;

__device__ __forceinline__ double mag2(double a) { return a * a; }
__device__ __forceinline__ double mag2(double2 a) { return fma(a.x, a.x, a.y * a.y); }
__device__ __forceinline__ double mul(double a, double b) { return a * b; }
__device__ __forceinline__ double2 mul(double2 a, double2 b) {
  return make_double2(fma(a.x, b.x, -a.y * b.y), fma(a.x, b.y, a.y * b.x));
}
__device__ __forceinline__ double submul(double c, double a, double b) { return fma(-a, b, c); }
__device__ __forceinline__ double2 submul(double2 c, double2 a, double2 b) {
  return make_double2(fma(-a.x, b.x, fma(a.y, b.y, c.x)), fma(-a.x, b.y, fma(-a.y, b.x, c.y)));
}
__device__ __forceinline__ double neg(double a) { return -a; }
__device__ __forceinline__ double2 neg(double2 a) { return make_double2(-a.x, -a.y); }
// 1 / d: the hardware estimate and two Newton steps (full precision); the plain
// division where the estimate or its square would leave the range
__device__ __forceinline__ double fast_recip(double d) {
  if (!(fabs(d) > 1e-290 && fabs(d) < 1e290)) return d != 0.0 ? 1.0 / d : 0.0;
  double r = __builtin_amdgcn_rcp(d);
  r = fma(r, fma(-d, r, 1.0), r);
  return fma(r, fma(-d, r, 1.0), r);
}
__device__ __forceinline__ double recip(double p) { return fast_recip(p); }
__device__ __forceinline__ double2 recip(double2 p) {
  const double d = mag2(p);
  if (!(d > 1e-290 && d < 1e290))
    return d > 0.0 ? make_double2(p.x / d, -p.y / d) : make_double2(0.0, 0.0);
  const double r = fast_recip(d);
  return make_double2(p.x * r, -p.y * r);
}
// Largest of the wavefront's keys, in every lane: row shifts and row broadcasts
// bring it to lane 63 without going through LDS.
template <int CTRL, int ROWS>
__device__ __forceinline__ unsigned long long dpp_max(unsigned long long v) {
  const int lo = __builtin_amdgcn_update_dpp((int)v, (int)v, CTRL, ROWS, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp((int)(v >> 32), (int)(v >> 32), CTRL, ROWS, 0xf, false);
  const unsigned long long o = ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo;
  return o > v ? o : v;
}
__device__ __forceinline__ unsigned long long wave_max(unsigned long long v) {
  v = dpp_max<0x111, 0xf>(v);   // row_shr 1, 2, 4, 8: lane 15 of each row of 16
  v = dpp_max<0x112, 0xf>(v);
  v = dpp_max<0x114, 0xf>(v);
  v = dpp_max<0x118, 0xf>(v);
  v = dpp_max<0x142, 0xa>(v);   // row_bcast 15 into rows 1 and 3
  v = dpp_max<0x143, 0xc>(v);   // row_bcast 31 into rows 2 and 3
  const unsigned lo = __builtin_amdgcn_readlane((int)v, 63);
  const unsigned hi = __builtin_amdgcn_readlane((int)(v >> 32), 63);
  return ((unsigned long long)hi << 32) | lo;
}
template <typename E> __device__ __forceinline__ E zero_of();
template <> __device__ __forceinline__ double zero_of<double>() { return 0.0; }
template <> __device__ __forceinline__ double2 zero_of<double2>() { return make_double2(0.0, 0.0); }

// Panel [k, k + bw), bw <= BW, of matrix blockIdx.x; thread t owns the rows
// t + blockDim.x rr, rr < RPT.  piv[c] = p_c; col[r] = the column whose pivot is row
// r, or -1.  X (may be null) receives the pivot rows as they are before the
// trailing update, [bw][n].  flag[0] is set to 1 for a zero or non-finite pivot.
template <typename E, int BW, int RPT, int MAXT>
__global__ __launch_bounds__(MAXT) void gj_panel(E* __restrict__ Am, int n, int k, int bw,
                                                 int* __restrict__ piv, int* __restrict__ col,
                                                 int* __restrict__ flag, E* __restrict__ X) {
  constexpr int NWAVE = MAXT / 64;
  __shared__ __attribute__((aligned(16))) unsigned long long key[2][NWAVE];
  __shared__ __attribute__((aligned(16))) E prow[2][BW];
  __shared__ int prows[BW];
  static_assert(BW > 1, "a panel has at least two columns");
  const int tid = threadIdx.x, w = blockIdx.x;
  E* A = Am + (int64_t)w * n * n;
  int* cl = col + (int64_t)w * n;
  E v[RPT][BW];
  bool used[RPT];
#pragma unroll
  for (int rr = 0; rr < RPT; ++rr) {
    const int i = tid + rr * blockDim.x;
    used[rr] = i >= n || (k > 0 && cl[min(i, n - 1)] >= 0);
    // clamped addresses, so that no load waits in a branch for the one before it
    const E* row = A + (int64_t)min(i, n - 1) * n + k;
#pragma unroll
    for (int t = 0; t < BW; ++t) v[rr][t] = row[min(t, bw - 1)];
#pragma unroll
    for (int t = 0; t < BW; ++t)
      if (t >= bw) v[rr][t] = zero_of<E>();
  }
  // the wave's best candidate for the column in v[.][0]: magnitude first, then the
  // smallest row
  auto post = [&](int buf) {
    unsigned long long best = 0;
#pragma unroll
    for (int rr = 0; rr < RPT; ++rr)
      if (!used[rr]) {
        const unsigned long long b = (unsigned long long)__double_as_longlong(mag2(v[rr][0]));
        const unsigned long long kk =
            ((b & ~(1ull << 63)) & ~ROW_MASK) | (ROW_MASK - (unsigned)(tid + rr * blockDim.x));
        best = kk > best ? kk : best;
      }
    best = wave_max(best);
    if ((tid & 63) == 0) key[buf][tid >> 6] = best;
  };
  if (tid < 2 * NWAVE) key[tid / NWAVE][tid % NWAVE] = 0;   // waves that are not there
  __syncthreads();
  post(0);
  // The registers rotate: column t is always v[.][0], and eliminating it writes every
  // other one place further down and its own result last.
  for (int t = 0; t < bw; ++t) {
    __syncthreads();
    unsigned long long best = key[t & 1][0];
#pragma unroll
    for (int x = 1; x < NWAVE; ++x) best = key[t & 1][x] > best ? key[t & 1][x] : best;
    const int r = (int)(ROW_MASK - (best & ROW_MASK));
    // the pivot row, unscaled, for everybody (a second buffer: the row of column t
    // may still be read while that of t + 1 is written)
#pragma unroll
    for (int rr = 0; rr < RPT; ++rr)
      if (tid + rr * (int)blockDim.x == r) {
#pragma unroll
        for (int tt = 0; tt < BW; ++tt) prow[t & 1][tt] = v[rr][tt];
        used[rr] = true;
        prows[t] = r;   // (piv is written after the loop: a barrier waits for stores to memory)
        const double m = mag2(v[rr][0]);
        if (!(m > 0.0) || !isfinite(m)) atomicExch(flag, 1);
      }
    __syncthreads();
    // The pivot row is read in groups of eight, the next group in flight while one is
    // used (left to itself the compiler reads each element just before its use and
    // waits for it).
    constexpr int G = BW < 8 ? BW : 8;
    const E* pr = prow[t & 1];
    E p[2][G];
#pragma unroll
    for (int e = 0; e < G; ++e) p[0][e] = pr[e];
    const E pinv = recip(p[0][0]);
    E f[RPT];
#pragma unroll
    for (int rr = 0; rr < RPT; ++rr) {
      f[rr] = mul(v[rr][0], pinv);
      if (tid + rr * (int)blockDim.x == r) {   // the pivot row itself: 0 + pinv times it
        f[rr] = neg(pinv);
#pragma unroll
        for (int tt = 1; tt < BW; ++tt) v[rr][tt] = zero_of<E>();
      }
      v[rr][0] = submul(v[rr][1], f[rr], p[0][1]);
    }
    // the next column's candidates go out before the rest of the row is updated
    if (t + 1 < bw) post((t + 1) & 1);
#pragma unroll
    for (int g = 0; g < BW / G; ++g) {
      if (g + 1 < BW / G) {
#pragma unroll
        for (int e = 0; e < G; ++e) p[(g + 1) & 1][e] = pr[(g + 1) * G + e];
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int e = 0; e < G; ++e) {
        const int tt = g * G + e;
        if (tt < 2) continue;
#pragma unroll
        for (int rr = 0; rr < RPT; ++rr) v[rr][tt - 1] = submul(v[rr][tt], f[rr], p[g & 1][e]);
      }
    }
#pragma unroll
    for (int rr = 0; rr < RPT; ++rr) v[rr][BW - 1] = neg(f[rr]);
  }
  // after bw turns column t sits in register BW - bw + t
#pragma unroll
  for (int rr = 0; rr < RPT; ++rr) {
    const int i = tid + rr * blockDim.x;
    if (i >= n) continue;
#pragma unroll
    for (int e = 0; e < BW; ++e)
      if (e >= BW - bw) A[(int64_t)i * n + k + e - (BW - bw)] = v[rr][e];
    int c = k > 0 ? cl[i] : -1;
    for (int t = 0; t < bw; ++t)
      if (prows[t] == i) c = k + t;
    cl[i] = c;
  }
  if (tid < bw) piv[(int64_t)w * n + k + tid] = prows[tid];
  if (X != nullptr)
    for (int j = tid; j < n; j += blockDim.x) {
#pragma unroll
      for (int t = 0; t < BW; ++t)
        if (t < bw) X[(int64_t)t * n + j] = A[(int64_t)prows[t] * n + j];
    }
}

// Trailing update of the columns blockIdx.x * 32 .. + 31 outside the panel.  X null:
// the workgroup takes all rows and reads the pivot rows from the matrix itself
// before it writes any; else it takes the 16-row groups blockIdx.y * 4 + wave,
// strided, and reads the pivot rows from X.  KS k-steps of 4 cover the panel.
template <typename E, int KS>
__global__ __launch_bounds__(TNT, 2) void gj_trail(E* __restrict__ Am, int n, int k, int bw,
                                                const int* __restrict__ piv,
                                                const E* __restrict__ Xc) {
  constexpr bool CPLX = sizeof(E) == 16;
  constexpr int NT = TCOLS / 16;   // column tiles
  __shared__ __attribute__((aligned(16))) E Xs[4 * KS][TCOLS];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int w = blockIdx.z, j0 = blockIdx.x * TCOLS;
  if (j0 >= k && j0 + TCOLS <= k + bw) return;   // all panel columns
  E* A = Am + (int64_t)w * n * n;
  const int* pv = piv + (int64_t)w * n + k;
  const E* X = Xc;
  for (int e = tid; e < 4 * KS * TCOLS; e += TNT) {
    const int t = e / TCOLS, c = e % TCOLS, j = min(j0 + c, n - 1);
    E x = zero_of<E>();
    if (t < bw) x = X != nullptr ? X[(int64_t)t * n + j] : A[(int64_t)pv[t] * n + j];
    Xs[t][c] = x;
  }
  const int fr = lane & 15, fg = lane >> 4;
  int pt[KS];   // the pivot rows of this lane's k
#pragma unroll
  for (int s = 0; s < KS; ++s) pt[s] = 4 * s + fg < bw ? pv[4 * s + fg] : -1;
  __syncthreads();   // X is in LDS (the rows it was read from may be written now)
  // one 16-row group in registers: its rows of W - E (rows past the end repeat the
  // last and are not stored) and its part of the matrix
  struct Group {
    E wf[KS];
    d4 re[NT], im[NT];
  };
  auto load = [&](Group& g, int i0) {
    const int iw = min(i0 + fr, n - 1);
#pragma unroll
    for (int s = 0; s < KS; ++s) g.wf[s] = A[(int64_t)iw * n + k + min(4 * s + fg, bw - 1)];
#pragma unroll
    for (int c = 0; c < NT; ++c)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = min(i0 + out_row<MODE_F64>(lane, r), n - 1), j = min(j0 + 16 * c + fr, n - 1);
        if constexpr (CPLX) {
          const double2 a = A[(int64_t)i * n + j];
          g.re[c][r] = a.x;
          g.im[c][r] = a.y;
        } else {
          g.re[c][r] = A[(int64_t)i * n + j];
        }
      }
  };
  auto update = [&](Group& g, int i0) {
    const int iw = min(i0 + fr, n - 1);
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const bool unit = iw == pt[s], in = 4 * s + fg < bw;
      if constexpr (CPLX) {
        g.wf[s].x = in ? g.wf[s].x - (unit ? 1.0 : 0.0) : 0.0;
        g.wf[s].y = in ? g.wf[s].y : 0.0;
      } else {
        g.wf[s] = in ? g.wf[s] - (unit ? 1.0 : 0.0) : 0.0;
      }
    }
#pragma unroll
    for (int s = 0; s < KS; ++s)
#pragma unroll
      for (int c = 0; c < NT; ++c) {
        const E x = Xs[4 * s + fg][16 * c + fr];
        if constexpr (CPLX) {
          g.re[c] = mfma1(g.wf[s].x, x.x, g.re[c]);
          g.im[c] = mfma1(g.wf[s].x, x.y, g.im[c]);
          g.re[c] = mfma1(-g.wf[s].y, x.y, g.re[c]);
          g.im[c] = mfma1(g.wf[s].y, x.x, g.im[c]);
        } else {
          g.re[c] = mfma1(g.wf[s], x, g.re[c]);
        }
      }
#pragma unroll
    for (int c = 0; c < NT; ++c)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = i0 + out_row<MODE_F64>(lane, r), j = j0 + 16 * c + fr;
        if (i < n && j < n && (j < k || j >= k + bw)) {
          if constexpr (CPLX) A[(int64_t)i * n + j] = make_double2(g.re[c][r], g.im[c][r]);
          else A[(int64_t)i * n + j] = g.re[c][r];
        }
      }
  };
  // the next group's loads are in flight while one is multiplied
  const int stride = 16 * 4 * gridDim.y;
  int i0 = 16 * (4 * blockIdx.y + wave);
  if (i0 >= n) return;
  Group g0, g1;
  load(g0, i0);
  for (;;) {
    if (i0 + stride < n) load(g1, i0 + stride);
    update(g0, i0);
    if ((i0 += stride) >= n) break;
    if (i0 + stride < n) load(g0, i0 + stride);
    update(g1, i0);
    if ((i0 += stride) >= n) break;
  }
}

// All panels with the register blocking (BW columns, RPT rows per thread, at most
// MAXT threads).
template <typename E, int BW, int RPT, int MAXT>
hipError_t eliminate(E* Am, int n, int nw, int* piv, int* col, int* flag, E* X, hipStream_t s) {
  constexpr int KS = BW >= 4 ? BW / 4 : 1;
  const int threads = ((n + RPT - 1) / RPT + 63) / 64 * 64;
  // one matrix: its rows are dealt to as many workgroups as have 16-row groups
  const unsigned splits = X != nullptr ? (unsigned)((n + 63) / 64) : 1u;
  for (int k = 0; k < n; k += BW) {
    const int bw = std::min(BW, n - k);
    gj_panel<E, BW, RPT, MAXT><<<nw, threads, 0, s>>>(Am, n, k, bw, piv, col, flag, X);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    gj_trail<E, KS><<<dim3((unsigned)((n + TCOLS - 1) / TCOLS), splits, (unsigned)nw), TNT, 0, s>>>(
        Am, n, k, bw, piv, X);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace

// The panel width is what a thread's registers hold: 512 threads have 256 each, 1024
// have 128 (a complex element takes 4, a real one 2).
hipError_t gj_inverse(double2* Am, int n, int nw, int* piv, int* col, int* flag, hipStream_t s) {
  if (n <= 0 || nw <= 0 || nw > 65535 || n > GJ_MAX_N) return hipErrorInvalidValue;
  if (n <= 512) return eliminate<double2, 32, 1, 512>(Am, n, nw, piv, col, flag, nullptr, s);
  if (n <= 1024) return eliminate<double2, 16, 1, 1024>(Am, n, nw, piv, col, flag, nullptr, s);
  if (n <= 2048) return eliminate<double2, 8, 2, 1024>(Am, n, nw, piv, col, flag, nullptr, s);
  if (n <= 4096) return eliminate<double2, 4, 4, 1024>(Am, n, nw, piv, col, flag, nullptr, s);
  return eliminate<double2, 2, 9, 1024>(Am, n, nw, piv, col, flag, nullptr, s);
}

hipError_t gj_inverse(double* Am, int n, int* piv, int* col, int* flag, double* X, hipStream_t s) {
  if (n <= 0 || n > GJ_MAX_N || X == nullptr) return hipErrorInvalidValue;
  if (n <= 512) return eliminate<double, 32, 1, 512>(Am, n, 1, piv, col, flag, X, s);
  if (n <= 1024) return eliminate<double, 32, 1, 1024>(Am, n, 1, piv, col, flag, X, s);
  if (n <= 2048) return eliminate<double, 16, 2, 1024>(Am, n, 1, piv, col, flag, X, s);
  if (n <= 4096) return eliminate<double, 8, 4, 1024>(Am, n, 1, piv, col, flag, X, s);
  return eliminate<double, 4, 9, 1024>(Am, n, 1, piv, col, flag, X, s);
}

}  // namespace thcsox
