// Device kernels of libthcsox for gfx950.  Host launchers are declared in
// kernels.hpp; the C interface that sequences them is in thcsox.hip.
#include "kernels.hpp"
#include "mfma.hpp"
#include "reduce.hpp"

namespace thcsox {

namespace {

constexpr int NT = 256;   // threads per workgroup (4 wavefronts of 64)

__device__ __forceinline__ double pow2_scale(const unsigned long long* amax) {
  if (amax == nullptr) return 1.0;
  unsigned long long b = *amax;
  if (b == 0ull) return 1.0;
  double x = __longlong_as_double((long long)b);
  if (!(x < 1e300)) return 1.0;   // inf / nan: leave unscaled, the result shows it
  return ldexp(1.0, -ilogb(x));
}

// ---------------------------------------------------------------------------
// Small kernels
// ---------------------------------------------------------------------------
// Several arrays split in one launch (a launch of a few microseconds is mostly its own
// latency): blocks first[q] .. first[q + 1] - 1 take job q.  A block takes NT / wide rows of
// wide = 2^lw >= ldk threads each (one row of NT threads from ldk > NT / 2 on).
struct SplitJobs {
  SplitArgs job[SPLIT_JOBS];
  int first[SPLIT_JOBS];   // blocks before job q
  int lw[SPLIT_JOBS];
};
template <int M>
__global__ __launch_bounds__(NT) void split_kernel(SplitJobs jobs, int njobs) {
  using T = typename ModeT<M>::T;
  constexpr int NP = ModeT<M>::NP;
  int q = 0;
  while (q + 1 < njobs && (int)blockIdx.x >= jobs.first[q + 1]) ++q;
  const SplitArgs a = jobs.job[q];
  const int lw = jobs.lw[q], wide = 1 << lw;
  const unsigned row = (blockIdx.x - jobs.first[q]) * (NT >> lw) + (threadIdx.x >> lw);
  if (row >= (unsigned)a.rows1 * (unsigned)a.rows2) return;   // (rows < 2^31)
  const int64_t r1 = row / (unsigned)a.rows2, r2 = row % (unsigned)a.rows2;
  const double sc = pow2_scale(a.amax ? a.amax + r2 * a.amax_s2 : nullptr);
  T* dst = static_cast<T*>(a.dst);
  const int64_t so = r1 * a.s1 + r2 * a.s2;
  const int64_t dof = r1 * a.d1 + r2 * a.d2;
  for (int c = threadIdx.x & (wide - 1); c < a.ldk; c += wide) {
    double x = 0.0;
    if (c < a.cols) {
      x = a.src_f32 ? (double)static_cast<const float*>(a.src)[so + (int64_t)c * a.sc]
                    : static_cast<const double*>(a.src)[so + (int64_t)c * a.sc];
      x *= sc;
    }
    T o[NP];
    Split<M>::run(x, o);
    if (a.c32) {   // planes interleaved per 32-wide chunk
#pragma unroll
      for (int p = 0; p < NP; ++p) dst[dof + (c >> 5) * 64 + 32 * p + (c & 31)] = o[p];
    } else {
#pragma unroll
      for (int p = 0; p < NP; ++p) dst[p * a.d_plane + dof + c] = o[p];
    }
  }
}

// out = max over rows r < rows of sum_{c < len} x[r ld + c]^2 (max-reduced, bits)
__global__ __launch_bounds__(NT) void rownorm2_kernel(const double* x, int64_t rows, int len,
                                                      int64_t ld, unsigned long long* out) {
  double m = 0.0;
  for (int64_t r = (int64_t)blockIdx.x * NT + threadIdx.x; r < rows; r += (int64_t)gridDim.x * NT) {
    const double* xr = x + r * ld;
    double s = 0.0;
    for (int c = 0; c < len; ++c) s = fma(xr[c], xr[c], s);
    m = fmax(m, s);
  }
  block_atomic_max<NT / 64>(m, out);
}

// amax_a[b] = bound_b * 2^-14, bound_b = (1 + 2^-10) |U row|max su |Gb column|max(b) sg(b):
// by Cauchy-Schwarz |A| <= bound_b for A formed from the scaled planes.  One workgroup per
// b: 64 columns at a time, their rows dealt to the 16 waves.  (n = 97, 16
// tau points: 5.9 us; one wave a column block, a clearing launch and one for the scale took
// 17.)
constexpr int CW = 16;
__global__ __launch_bounds__(64 * CW) void ascale_kernel(const unsigned long long* unorm2,
                                                         const unsigned long long* amax_u,
                                                         const double* G, int n, int64_t stride,
                                                         const unsigned long long* amax_gb,
                                                         int64_t gb_stride, unsigned long long* amax_a) {
  __shared__ double part[CW][64];
  const int b = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const double* g = G + (int64_t)b * stride;
  double m = 0.0;
  for (int v0 = 0; v0 < n; v0 += 64) {
    const int v = min(v0 + lane, n - 1);   // (the last column again past the end)
    double s = 0.0;
#pragma unroll 4
    for (int r = wave; r < n; r += CW) s = fma(g[(int64_t)r * n + v], g[(int64_t)r * n + v], s);
    __syncthreads();
    part[wave][lane] = s;
    __syncthreads();
    if (wave == 0) {
      double t = 0.0;
      for (int w = 0; w < CW; ++w) t += part[w][lane];
      m = fmax(m, t);
    }
  }
  if (wave > 0) return;
  for (int o = 32; o > 0; o >>= 1) m = fmax(m, __shfl_xor(m, o, 64));
  if (lane > 0) return;
  const double un = sqrt(__longlong_as_double((long long)*unorm2));
  const double bound = (1.0 + 0x1p-10) * un * pow2_scale(amax_u) * sqrt(m) *
                       pow2_scale(amax_gb + (int64_t)b * gb_stride);
  amax_a[b] = (unsigned long long)__double_as_longlong(bound * 0x1p-14);
}

__global__ __launch_bounds__(NT) void absmax_kernel(const double* x, const double* x2, int64_t len,
                                                    int64_t stride, unsigned long long* amax,
                                                    unsigned long long* amax2) {
  const int64_t b = blockIdx.y;
  const double* xb = (blockIdx.z ? x2 : x) + b * stride;
  if (blockIdx.z) amax = amax2;
  double m = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x; i < len; i += (int64_t)gridDim.x * NT)
    m = fmax(m, fabs(xb[i]));
  block_atomic_max<NT / 64>(m, amax + b);
}

__global__ void fill_u64_kernel(unsigned long long* p, int64_t n, unsigned long long v) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

// One workgroup per 32 x 32 tile of Sthc: sum the partial D tiles over z and
// scale.  With the symmetric path only the tiles on and above the diagonal are
// read: each writes itself and (through LDS) its transpose below the diagonal,
// and inside a diagonal tile the entries with R > P come from the mirrored
// position.
constexpr int DT = 32;          // reduction tile edge
static_assert(SYM_BLOCK % DT == 0, "a tile on or above the diagonal lies in blocks that are written");
constexpr int DRP = NT / DT;    // rows per pass
constexpr int DEL = DT / DRP;   // elements per thread
// (vector types of element alignment: rows of any length are read in 16- or 32-byte pieces)
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
typedef double d4u __attribute__((ext_vector_type(4), aligned(8)));
__device__ __forceinline__ void add4(const float* p, double* acc) {
  const f4u v = *reinterpret_cast<const f4u*>(p);
#pragma unroll
  for (int e = 0; e < 4; ++e) acc[e] += (double)v[e];
}
__device__ __forceinline__ void add4(const double* p, double* acc) {
  const d4u v = *reinterpret_cast<const d4u*>(p);
#pragma unroll
  for (int e = 0; e < 4; ++e) acc[e] += v[e];
}

template <typename T>
__global__ __launch_bounds__(NT) void dreduce_kernel(DReduceArgs a) {
  __shared__ double t[DT][DT + 1];
  const int set = blockIdx.y;
  const double f = pow2_scale(a.amax_gt + set) * pow2_scale(a.amax_gx + set) *
                   pow2_scale(a.amax_gb - set) *
                   pow2_scale(a.amax_a != nullptr ? a.amax_a + set : nullptr) * pow2_scale(a.amax_u) *
                   pow2_scale(a.amax_u2 != nullptr ? a.amax_u2 : a.amax_u);
  const double inv = 1.0 / f;   // exact: a power of two
  const int64_t nn = (int64_t)a.naux * a.naux;
  const bool sym = a.sym != nullptr && a.sym[set] != 0;
  double* const Sthc = a.Sthc + set * a.s_set;
  const int nt = (a.naux + DT - 1) / DT;
  const int rb = blockIdx.x / nt, pb = blockIdx.x % nt;
  // symmetric D: the tiles below the diagonal are written by their transposes
  if (sym && rb > pb) return;
  // sum over z: thread = (row ar, four consecutive columns ac..ac+3), one load for the
  // four except at the end of a row (single loads for every odd row length took 18
  // instead of 8 us at naux = 485, 16 partial tiles)
  const int ar = threadIdx.x / (DT / 4), ac = 4 * (threadIdx.x % (DT / 4));
  const int gr = rb * DT + ar, gc = pb * DT + ac;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  if (gr < a.naux) {
    const T* D0 = reinterpret_cast<const T*>(a.Dpart) + set * a.d_set + (int64_t)gr * a.naux + gc;
    if (gc + 3 < a.naux) {
#pragma unroll 4
      for (int z = 0; z < a.vsplit; ++z) add4(D0 + z * nn, acc);
    } else {
      for (int z = 0; z < a.vsplit; ++z)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (gc + e < a.naux) acc[e] += (double)D0[z * nn + e];
    }
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) t[ar][ac + e] = acc[e];
  __syncthreads();
  const int col = threadIdx.x % DT, row0 = threadIdx.x / DT;
#pragma unroll
  for (int i = 0; i < DEL; ++i) {
    const int lr = row0 + DRP * i, lc = col;
    // element (R, P) of tile (rb, pb); on a symmetric diagonal tile the lower
    // half comes from the upper
    const int R = rb * DT + lr, P = pb * DT + lc;
    if (R < a.naux && P < a.naux) {
      const double v = (sym && rb == pb && R > P) ? t[lc][lr] : t[lr][lc];
      Sthc[(int64_t)R * a.s_ld + P] = -inv * v;
    }
    // symmetric, off the diagonal: element (R2, P2) of the transposed tile (pb, rb)
    if (sym && rb < pb) {
      const int R2 = pb * DT + lr, P2 = rb * DT + lc;
      if (R2 < a.naux && P2 < a.naux) Sthc[(int64_t)R2 * a.s_ld + P2] = -inv * t[lc][lr];
    }
  }
}

// max |G[k][i][j] - G[k][j][i]| over j > i and max |G[k][i][j]|; a row of workgroups per k
// strides over G[k].
__global__ __launch_bounds__(NT) void asym_kernel(const double* G, int n, unsigned long long* asym,
                                                  unsigned long long* amax) {
  const int k = blockIdx.y;
  const double* g = G + (int64_t)k * n * n;
  double m = 0.0, x = 0.0;
  for (int64_t e = (int64_t)blockIdx.x * NT + threadIdx.x; e < (int64_t)n * n;
       e += (int64_t)gridDim.x * NT) {
    const int i = (int)(e / n), j = (int)(e % n);
    const double v = g[e];
    x = fmax(x, fabs(v));
    if (j > i) m = fmax(m, fabs(v - g[(int64_t)j * n + i]));
  }
  block_atomic_max<NT / 64>(m, asym + k);
  __syncthreads();   // (both use the same LDS)
  block_atomic_max<NT / 64>(x, amax + k);
}

__global__ void sym_flags_kernel(const unsigned long long* asym, const unsigned long long* amax,
                                 int m, double rtol, int* flag) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= m) return;
  // the reference magnitude is the largest |G| on the whole grid: Sigma's error
  // is measured against its largest element, which comes from the largest G
  double gmax = 0.0;
  for (int j = 0; j < m; ++j) gmax = fmax(gmax, __longlong_as_double((long long)amax[j]));
  auto ok = [&](int j) { return __longlong_as_double((long long)asym[j]) <= rtol * gmax; };
  flag[k] = (ok(k) && ok(m - 1 - k)) ? 1 : 0;
}

__global__ __launch_bounds__(NT) void khatri_rao_kernel(const double* X, int n, int naux, int q0,
                                                        double* KR) {
  const int64_t row = blockIdx.x;          // (q - q0) * n + s
  const int q = q0 + (int)(row / n), s = (int)(row % n);
  for (int Q = threadIdx.x; Q < naux; Q += NT)
    KR[row * naux + Q] = X[(int64_t)q * naux + Q] * X[(int64_t)s * naux + Q];
}

constexpr int EW = 8;   // waves per workgroup (one per tau point)
__global__ __launch_bounds__(64 * EW) void energy_partials_kernel(const double* G, const double* S,
                                                                  int n, int m, double* tr) {
  const int k = blockIdx.x;
  const int64_t nn = (int64_t)n * n;
  const double t = block_trace<EW>(G + (int64_t)(m - 1 - k) * nn, S + (int64_t)k * nn, n);
  if (threadIdx.x == 0) tr[k] = t;
}

__global__ void energy_final_kernel(const double* tr, const double* w, int m, double* E) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    double s = 0.0;
    for (int k = 0; k < m; ++k) s = fma(w[k], tr[k], s);
    *E = -0.5 * s;
  }
}

// Pi0 (+)= sum_l w[l] Pi_l + w[m-1-l] Pi_l^T over nb matrices: one 32 x 32 tile per
// workgroup, the transposed sum taken from the mirrored tile (read along its rows)
// through LDS.  Bound by reading each Pi twice.
constexpr int WT = 32;
__global__ __launch_bounds__(NT) void weighted_pair_sum_kernel(const double* __restrict__ Pi,
                                                               const double* __restrict__ w, int m,
                                                               int l0, int nb, int naux,
                                                               double* __restrict__ Pi0,
                                                               int accumulate) {
  __shared__ double t[WT][WT + 1];
  const int i0 = blockIdx.y * WT, j0 = blockIdx.x * WT;
  const int tx = threadIdx.x % WT, ty = threadIdx.x / WT;   // 32 x 8
  const int64_t aa = (int64_t)naux * naux;
  constexpr int PER = WT * WT / NT;
  double here[PER] = {}, there[PER] = {};
#pragma unroll 4
  for (int b = 0; b < nb; ++b) {
    const int l = l0 + b;
    const double wl = w[l], wu = m - 1 - l == l ? 0.0 : w[m - 1 - l];
    const double* P = Pi + b * aa;
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      const int r = ty + e * (NT / WT);
      if (i0 + r < naux && j0 + tx < naux)
        here[e] = fma(wl, P[(int64_t)(i0 + r) * naux + j0 + tx], here[e]);
      if (j0 + r < naux && i0 + tx < naux)
        there[e] = fma(wu, P[(int64_t)(j0 + r) * naux + i0 + tx], there[e]);
    }
  }
#pragma unroll
  for (int e = 0; e < PER; ++e) t[ty + e * (NT / WT)][tx] = there[e];
  __syncthreads();
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    const int r = ty + e * (NT / WT);
    if (i0 + r < naux && j0 + tx < naux) {
      double* d = Pi0 + (int64_t)(i0 + r) * naux + j0 + tx;
      const double v = here[e] + t[tx][r];
      *d = accumulate ? *d + v : v;
    }
  }
}

__global__ __launch_bounds__(NT) void add_identity_kernel(double* A, int n, int* clear) {
  const int i = blockIdx.x * NT + threadIdx.x;
  if (i == 0) *clear = 0;
  if (i < n) A[(int64_t)i * n + i] += 1.0;
}

inline unsigned cdiv(int64_t a, int64_t b) { return (unsigned)((a + b - 1) / b); }

}  // namespace

hipError_t weighted_pair_sum(const double* Pi, const double* w, int m, int l0, int nb, int naux,
                             double* Pi0, int accumulate, hipStream_t s) {
  if (naux <= 0 || nb <= 0) return hipSuccess;
  const unsigned nt = cdiv(naux, WT);
  weighted_pair_sum_kernel<<<dim3(nt, nt), NT, 0, s>>>(Pi, w, m, l0, nb, naux, Pi0, accumulate);
  return hipGetLastError();
}

hipError_t add_identity(double* A, int n, int* clear, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  add_identity_kernel<<<cdiv(n, NT), NT, 0, s>>>(A, n, clear);
  return hipGetLastError();
}

hipError_t split_planes(int mode, const SplitArgs* a, int njobs, hipStream_t s) {
  if (njobs < 1 || njobs > SPLIT_JOBS) return hipErrorInvalidValue;
  SplitJobs jobs{};
  int64_t blocks = 0;
  for (int q = 0; q < njobs; ++q) {
    int lw = 5;
    while ((1 << lw) < NT && (1 << lw) < a[q].ldk) ++lw;
    jobs.job[q] = a[q];
    jobs.first[q] = (int)blocks;
    jobs.lw[q] = lw;
    const int64_t rows = (int64_t)a[q].rows1 * a[q].rows2, per = NT >> lw;
    blocks += (rows + per - 1) / per;
    // (a launch of more than 2^32 - 1 threads would be cut short without an error)
    if (rows < 0 || rows > 0x7fffffff || blocks > 0xffffffffLL / NT) return hipErrorInvalidValue;
  }
  if (blocks == 0) return hipSuccess;
  const dim3 grid((unsigned)blocks);
  switch (mode) {
    case MODE_F64: split_kernel<MODE_F64><<<grid, NT, 0, s>>>(jobs, njobs); break;
    case MODE_F32: split_kernel<MODE_F32><<<grid, NT, 0, s>>>(jobs, njobs); break;
    case MODE_BF16X3: split_kernel<MODE_BF16X3><<<grid, NT, 0, s>>>(jobs, njobs); break;
    case MODE_F16X2: split_kernel<MODE_F16X2><<<grid, NT, 0, s>>>(jobs, njobs); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t absmax64(const double* x, int64_t len, int64_t stride, int batch,
                    unsigned long long* amax, hipStream_t s, const double* x2,
                    unsigned long long* amax2) {
  if (len <= 0 || batch <= 0) return hipSuccess;
  // a few workgroups per row: one atomic each
  unsigned bx = cdiv(len, NT);
  if (bx > 64) bx = 64;
  absmax_kernel<<<dim3(bx, batch, x2 != nullptr ? 2 : 1), NT, 0, s>>>(x, x2, len, stride, amax, amax2);
  return hipGetLastError();
}

hipError_t rownorm2_max(const double* x, int64_t rows, int len, int64_t ld,
                        unsigned long long* out, hipStream_t s) {
  if (rows <= 0 || len <= 0) return hipSuccess;
  unsigned b = cdiv(rows, NT);
  if (b > 1024) b = 1024;
  rownorm2_kernel<<<b, NT, 0, s>>>(x, rows, len, ld, out);
  return hipGetLastError();
}

hipError_t ascale_bound(const unsigned long long* unorm2, const unsigned long long* amax_u,
                        const double* G, int n, int64_t stride, const unsigned long long* amax_gb,
                        int64_t gb_stride, int nb, unsigned long long* amax_a, hipStream_t s) {
  if (nb <= 0 || n <= 0) return hipSuccess;
  ascale_kernel<<<nb, 64 * CW, 0, s>>>(unorm2, amax_u, G, n, stride, amax_gb, gb_stride, amax_a);
  return hipGetLastError();
}

hipError_t fill_u64(unsigned long long* p, int64_t n, unsigned long long v, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  unsigned b = cdiv(n, NT);
  if (b > 4096) b = 4096;
  fill_u64_kernel<<<b, NT, 0, s>>>(p, n, v);
  return hipGetLastError();
}

hipError_t dreduce(const DReduceArgs& a, hipStream_t s) {
  if (a.naux <= 0) return hipSuccess;
  const unsigned nt = cdiv(a.naux, DT);
  if (a.dpart_f32) dreduce_kernel<float><<<dim3(nt * nt, a.nsets), NT, 0, s>>>(a);
  else dreduce_kernel<double><<<dim3(nt * nt, a.nsets), NT, 0, s>>>(a);
  return hipGetLastError();
}

hipError_t asym64(const double* G, int n, int m, unsigned long long* asym, unsigned long long* amax,
                  hipStream_t s) {
  if (n <= 0 || m <= 0) return hipSuccess;
  unsigned bx = cdiv((int64_t)n * n, NT);
  if (bx > 256) bx = 256;
  asym_kernel<<<dim3(bx, m), NT, 0, s>>>(G, n, asym, amax);
  return hipGetLastError();
}

hipError_t sym_flags(const unsigned long long* asym, const unsigned long long* amax, int m,
                     double rtol, int* flag, hipStream_t s) {
  if (m <= 0) return hipSuccess;
  sym_flags_kernel<<<cdiv(m, 64), 64, 0, s>>>(asym, amax, m, rtol, flag);
  return hipGetLastError();
}

hipError_t khatri_rao(const double* X, int n, int naux, int q0, int q1, double* KR,
                      hipStream_t s) {
  const int64_t rows = (int64_t)(q1 - q0) * n;
  if (rows <= 0) return hipSuccess;
  khatri_rao_kernel<<<(unsigned)rows, NT, 0, s>>>(X, n, naux, q0, KR);
  return hipGetLastError();
}

hipError_t energy_partials(const double* G, const double* S, int n, int m, double* tr,
                           hipStream_t s) {
  energy_partials_kernel<<<m, 64 * EW, 0, s>>>(G, S, n, m, tr);
  return hipGetLastError();
}

hipError_t energy_final(const double* tr, const double* w, int m, double* E, hipStream_t s) {
  energy_final_kernel<<<1, 64, 0, s>>>(tr, w, m, E);
  return hipGetLastError();
}

}  // namespace thcsox
