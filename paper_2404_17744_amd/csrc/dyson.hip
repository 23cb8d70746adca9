// One self-consistency step in FP64 on the GPU: Sigma(tau) -> Sigma(i w_n) ->
// Dyson equation (Sec. "Definitions", Eq. Dyson, orthonormal basis) ->
// G(i w_n) -> G(tau) and the density matrix.
//
// tau grid: the m roots of the Chebyshev polynomial T_m mapped to [0, beta].
//   forward : Sigma(i w_n) = sum_l T_nl c_l, c = Chebyshev interpolation
//             coefficients of Sigma(tau) through the roots, and
//             T_nl = int_0^beta exp(i w_n tau) T_l(2 tau / beta - 1) dtau,
//             w_n = (2n+1) pi / beta, n = 0 .. nw-1.
//   Dyson   : G(i w_n) = [(i w_n + mu) 1 - F - Sigma(i w_n)]^-1
//   backward: real coefficients minimising sum_n |sum_l T_nl c_l - G(i w_n)|^2,
//             G(tau_k) = sum_l c_l T_l(x_k),  gamma = -G(beta^-) = -sum_l c_l.
// The three linear maps are folded into two real matrices built on the host
// at plan time (Wf: [2 nw][m], Wb: [m + 1][2 nw]); each step is then two FP64
// matrix-core GEMMs around a batched complex Gauss-Jordan inversion.
#include <hip/hip_runtime.h>

#include <cmath>
#include <complex>
#include <map>
#include <mutex>
#include <new>
#include <string>
#include <tuple>
#include <vector>

#include "../../include/thcsox.h"
#include "error.hpp"
#include "kernels.hpp"
#include "reduce.hpp"

using namespace thcsox;

namespace {

constexpr int NT = 256;

// ----------------------------------------------------------------------------
// Host tables (FP64)
// ----------------------------------------------------------------------------

// Gauss-Legendre nodes and weights on [-1, 1] (Newton iteration on P_q).
void gauss_legendre(int q, std::vector<double>& x, std::vector<double>& w) {
  x.resize(q);
  w.resize(q);
  for (int i = 0; i < q; ++i) {
    double z = std::cos(M_PI * (i + 0.75) / (q + 0.5));
    for (int it = 0; it < 100; ++it) {
      double p0 = 1.0, p1 = z;
      for (int k = 2; k <= q; ++k) {
        const double p2 = ((2.0 * k - 1.0) * z * p1 - (k - 1.0) * p0) / k;
        p0 = p1;
        p1 = p2;
      }
      const double dp = q * (z * p1 - p0) / (z * z - 1.0);
      const double dz = p1 / dp;
      z -= dz;
      if (std::fabs(dz) < 1e-16) break;
    }
    double p0 = 1.0, p1 = z;
    for (int k = 2; k <= q; ++k) {
      const double p2 = ((2.0 * k - 1.0) * z * p1 - (k - 1.0) * p0) / k;
      p0 = p1;
      p1 = p2;
    }
    const double dp = q * (z * p1 - p0) / (z * z - 1.0);
    x[i] = z;
    w[i] = 2.0 / ((1.0 - z * z) * dp * dp);
  }
}

struct Tables {
  std::vector<double> Wf;   // [2 nw][m]: rows 0..nw-1 real part, nw..2nw-1 imaginary part
  std::vector<double> Wb;   // [m + 1][2 nw]: G(tau_k) rows, then the gamma row
};

// T[n][l] = int_0^beta exp(i w_n tau) T_l(2 tau/beta - 1) dtau by composite
// Gauss-Legendre over equal panels in x = 2 tau / beta - 1.
std::vector<std::complex<double>> cheb_matsubara(int m, int nw, double beta) {
  const int q = 16;
  const double amax = (2.0 * nw - 1.0) * M_PI / 2.0;          // largest w_n beta / 2
  const int panels = std::max(64, (int)std::ceil(amax / M_PI * 4.0) + 2 * m);
  std::vector<double> gx, gw;
  gauss_legendre(q, gx, gw);
  const int npt = panels * q;
  std::vector<double> xs(npt), ws(npt);
  for (int p = 0; p < panels; ++p) {
    const double a = -1.0 + 2.0 * p / panels, h = 1.0 / panels;   // half width
    for (int i = 0; i < q; ++i) {
      xs[p * q + i] = a + h + h * gx[i];
      ws[p * q + i] = h * gw[i];
    }
  }
  std::vector<double> Tl((size_t)npt * m);   // T_l(x) by recurrence
  for (int i = 0; i < npt; ++i) {
    double t0 = 1.0, t1 = xs[i];
    Tl[(size_t)i * m] = 1.0;
    if (m > 1) Tl[(size_t)i * m + 1] = t1;
    for (int l = 2; l < m; ++l) {
      const double t2 = 2.0 * xs[i] * t1 - t0;
      Tl[(size_t)i * m + l] = t2;
      t0 = t1;
      t1 = t2;
    }
  }
  std::vector<std::complex<double>> T((size_t)nw * m);
  std::vector<std::complex<double>> acc(m);
  for (int n = 0; n < nw; ++n) {
    const double wn = (2.0 * n + 1.0) * M_PI / beta;
    std::fill(acc.begin(), acc.end(), std::complex<double>(0.0, 0.0));
    for (int i = 0; i < npt; ++i) {
      const double tau = 0.5 * beta * (1.0 + xs[i]);
      const std::complex<double> e = std::polar(ws[i] * 0.5 * beta, wn * tau);
      const double* t = &Tl[(size_t)i * m];
      for (int l = 0; l < m; ++l) acc[l] += e * t[l];
    }
    for (int l = 0; l < m; ++l) T[(size_t)n * m + l] = acc[l];
  }
  return T;
}

// Least-squares pseudo-inverse P = (A^T A)^-1 A^T of a tall A [r][c] by
// Householder QR: A = Q R, P = R^-1 Q^T.
std::vector<double> pinv_qr(std::vector<double> A, int r, int c) {
  std::vector<double> Qt((size_t)r * r, 0.0);   // accumulate Q^T applied to identity rows
  for (int i = 0; i < r; ++i) Qt[(size_t)i * r + i] = 1.0;
  std::vector<double> v(r);
  for (int k = 0; k < c; ++k) {
    double norm = 0.0;
    for (int i = k; i < r; ++i) norm += A[(size_t)i * c + k] * A[(size_t)i * c + k];
    norm = std::sqrt(norm);
    const double akk = A[(size_t)k * c + k];
    const double alpha = akk > 0 ? -norm : norm;
    for (int i = 0; i < r; ++i) v[i] = 0.0;
    v[k] = akk - alpha;
    for (int i = k + 1; i < r; ++i) v[i] = A[(size_t)i * c + k];
    double vn = 0.0;
    for (int i = k; i < r; ++i) vn += v[i] * v[i];
    if (vn == 0.0) continue;
    // H = I - 2 v v^T / (v^T v) applied to A (columns k..c-1) and to Qt
    for (int j = k; j < c; ++j) {
      double s = 0.0;
      for (int i = k; i < r; ++i) s += v[i] * A[(size_t)i * c + j];
      s = 2.0 * s / vn;
      for (int i = k; i < r; ++i) A[(size_t)i * c + j] -= s * v[i];
    }
    for (int j = 0; j < r; ++j) {
      double s = 0.0;
      for (int i = k; i < r; ++i) s += v[i] * Qt[(size_t)i * r + j];
      s = 2.0 * s / vn;
      for (int i = k; i < r; ++i) Qt[(size_t)i * r + j] -= s * v[i];
    }
  }
  // P = R^-1 (first c rows of Qt), R upper triangular in A[0..c-1][0..c-1]
  std::vector<double> P((size_t)c * r);
  for (int j = 0; j < r; ++j) {
    for (int i = c - 1; i >= 0; --i) {
      double s = Qt[(size_t)i * r + j];
      for (int k2 = i + 1; k2 < c; ++k2) s -= A[(size_t)i * c + k2] * P[(size_t)k2 * r + j];
      P[(size_t)i * r + j] = s / A[(size_t)i * c + i];
    }
  }
  return P;
}

Tables build_tables(int m, int nw, double beta) {
  std::vector<double> x(m);
  for (int k = 0; k < m; ++k) x[k] = -std::cos((2.0 * k + 1.0) * M_PI / (2.0 * m));
  std::vector<double> Tev((size_t)m * m);   // Tev[k][l] = T_l(x_k)
  for (int k = 0; k < m; ++k) {
    double t0 = 1.0, t1 = x[k];
    Tev[(size_t)k * m] = 1.0;
    if (m > 1) Tev[(size_t)k * m + 1] = t1;
    for (int l = 2; l < m; ++l) {
      const double t2 = 2.0 * x[k] * t1 - t0;
      Tev[(size_t)k * m + l] = t2;
      t0 = t1;
      t1 = t2;
    }
  }
  const auto T = cheb_matsubara(m, nw, beta);
  Tables tb;
  // forward: c_l = (2 - delta_l0)/m sum_k T_l(x_k) F_k ; F(i w_n) = sum_l T_nl c_l
  tb.Wf.assign((size_t)2 * nw * m, 0.0);
  for (int n = 0; n < nw; ++n)
    for (int k = 0; k < m; ++k) {
      std::complex<double> s(0.0, 0.0);
      for (int l = 0; l < m; ++l)
        s += T[(size_t)n * m + l] * ((l == 0 ? 1.0 : 2.0) / m) * Tev[(size_t)k * m + l];
      tb.Wf[(size_t)n * m + k] = s.real();
      tb.Wf[(size_t)(nw + n) * m + k] = s.imag();
    }
  // backward: c = pinv([Re T; Im T]) [Re G; Im G]
  std::vector<double> A((size_t)2 * nw * m);
  for (int n = 0; n < nw; ++n)
    for (int l = 0; l < m; ++l) {
      A[(size_t)n * m + l] = T[(size_t)n * m + l].real();
      A[(size_t)(nw + n) * m + l] = T[(size_t)n * m + l].imag();
    }
  const auto P = pinv_qr(A, 2 * nw, m);   // [m][2nw]
  tb.Wb.assign((size_t)(m + 1) * 2 * nw, 0.0);
  for (int k = 0; k < m; ++k)
    for (int j = 0; j < 2 * nw; ++j) {
      double s = 0.0;
      for (int l = 0; l < m; ++l) s += Tev[(size_t)k * m + l] * P[(size_t)l * 2 * nw + j];
      tb.Wb[(size_t)k * 2 * nw + j] = s;
    }
  for (int j = 0; j < 2 * nw; ++j) {
    double s = 0.0;
    for (int l = 0; l < m; ++l) s += P[(size_t)l * 2 * nw + j];
    tb.Wb[(size_t)m * 2 * nw + j] = -s;   // gamma = -sum_l c_l
  }
  return tb;
}

// tables depend only on (m, nw, beta): cache them for repeated plans
const Tables& tables_for(int m, int nw, double beta) {
  static std::mutex mu;
  static std::map<std::tuple<int, int, double>, Tables> cache;
  std::lock_guard<std::mutex> lk(mu);
  auto key = std::make_tuple(m, nw, beta);
  auto it = cache.find(key);
  if (it == cache.end()) it = cache.emplace(key, build_tables(m, nw, beta)).first;
  return it->second;
}

// ----------------------------------------------------------------------------
// Kernels
// ----------------------------------------------------------------------------

// Am[w] = (i w_w + mu) 1 - F - Sigma(i w_w) as complex [n][n]; wfreq[w] = w_w.
__global__ __launch_bounds__(NT) void build_a(const double* __restrict__ S, const double* __restrict__ F,
                                              double mu, const double* __restrict__ wfreq, int n,
                                              int nw, double2* __restrict__ Am,
                                              int* __restrict__ flag) {
  const int w = blockIdx.y;
  if (w == 0 && blockIdx.x == 0 && threadIdx.x == 0) *flag = 0;   // before the elimination
  const double wn = wfreq[w];
  const int64_t nn = (int64_t)n * n;
  const double* Sre = S + (int64_t)w * nn;
  const double* Sim = S + (int64_t)(nw + w) * nn;
  double2* A = Am + (int64_t)w * nn;
  for (int64_t e = (int64_t)blockIdx.x * NT + threadIdx.x; e < nn; e += (int64_t)gridDim.x * NT) {
    const int64_t i = e / n, j = e % n;
    double re = -F[e] - Sre[e], im = -Sim[e];
    if (i == j) {
      re += mu;
      im += wn;
    }
    A[e] = make_double2(re, im);
  }
}

// Gstack[w][ij] = Re G(i w)_ij, Gstack[nw + w][ij] = Im G(i w)_ij.
__global__ __launch_bounds__(NT) void extract_inv(const double2* __restrict__ Am,
                                                  const int* __restrict__ piv,
                                                  const int* __restrict__ col, int n, int nw,
                                                  double* __restrict__ Gs) {
  const int w = blockIdx.y;
  const int64_t nn = (int64_t)n * n;
  const double2* A = Am + (int64_t)w * nn;
  const int* pv = piv + (int64_t)w * n;
  const int* cl = col + (int64_t)w * n;
  for (int64_t e = (int64_t)blockIdx.x * NT + threadIdx.x; e < nn; e += (int64_t)gridDim.x * NT) {
    const int i = (int)(e / n), j = (int)(e % n);
    const double2 v = A[(int64_t)pv[i] * n + cl[j]];
    Gs[(int64_t)w * nn + e] = v.x;
    Gs[(int64_t)(nw + w) * nn + e] = v.y;
  }
}

// tr[w] = Re Tr G(i w_w), tr[nw + w] = Im Tr G(i w_w): the diagonal of each
// inverse, read through the pivot permutations (one workgroup per frequency).
__global__ __launch_bounds__(NT) void inv_traces(const double2* __restrict__ Am,
                                                 const int* __restrict__ piv,
                                                 const int* __restrict__ col, int n, int nw,
                                                 double* __restrict__ tr) {
  __shared__ double r_re[NT], r_im[NT];
  const int w = blockIdx.x;
  const double2* A = Am + (int64_t)w * n * n;
  const int* pv = piv + (int64_t)w * n;
  const int* cl = col + (int64_t)w * n;
  double re = 0.0, im = 0.0;
  for (int i = threadIdx.x; i < n; i += NT) {
    const double2 v = A[(int64_t)pv[i] * n + cl[i]];
    re += v.x;
    im += v.y;
  }
  r_re[threadIdx.x] = re;
  r_im[threadIdx.x] = im;
  __syncthreads();
  for (int o = NT / 2; o > 0; o >>= 1) {
    if (threadIdx.x < o) {
      r_re[threadIdx.x] += r_re[threadIdx.x + o];
      r_im[threadIdx.x] += r_im[threadIdx.x + o];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    tr[w] = r_re[0];
    tr[nw + w] = r_im[0];
  }
}

// out[b] = workgroup b's part of sum_pq A[p][q] B[q][p] (fixed order); the host adds them.
constexpr int TW = 4;              // its waves
constexpr int TRACE_PARTS = 64;    // workgroups at most
__global__ __launch_bounds__(64 * TW) void trace_ab(const double* A, const double* B, int n,
                                                    double* out) {
  const double t = block_trace<TW>(A, B, n, blockIdx.x, gridDim.x);
  if (threadIdx.x == 0) out[blockIdx.x] = t;
}

int dfail(int code, const std::string& m) { return set_error(code, m); }

// Minv[i][j] = S[piv[i]][col[j]]
__global__ __launch_bounds__(NT) void unpack_real(const double* __restrict__ S,
                                                  const int* __restrict__ piv,
                                                  const int* __restrict__ col, int n,
                                                  double* __restrict__ Minv) {
  const int64_t nn = (int64_t)n * n;
  for (int64_t e = (int64_t)blockIdx.x * NT + threadIdx.x; e < nn; e += (int64_t)gridDim.x * NT) {
    const int i = (int)(e / n), j = (int)(e % n);
    Minv[e] = S[(int64_t)piv[i] * n + col[j]];
  }
}

}  // namespace

namespace thcsox {
hipError_t gj_unpack(const double* S, const int* piv, const int* col, int n, double* Minv,
                     hipStream_t s) {
  if (n <= 0) return hipErrorInvalidValue;
  const unsigned bx = (unsigned)std::min<int64_t>(1024, ((int64_t)n * n + NT - 1) / NT);
  unpack_real<<<bx, NT, 0, s>>>(S, piv, col, n, Minv);
  return hipGetLastError();
}
}  // namespace thcsox

struct thcsox_dyson_s {
  int n = 0, m = 0, nw = 0;
  double beta = 0, mu = 0;
  hipStream_t stream = nullptr;
  double* F = nullptr;     // [n][n]
  double* Wf = nullptr;    // [2nw][m]
  double* Wb = nullptr;    // [m+1][2nw]
  double* wfreq = nullptr; // [nw] the frequencies w_j
  double* Siw = nullptr;   // [2nw][n n]
  double2* Am = nullptr;   // [nw][n][n]
  int* piv = nullptr;      // [nw][n]
  int* col = nullptr;      // [nw][n]
  double* Gs = nullptr;    // [2nw][n n]
  double* Gout = nullptr;  // [m+1][n n]
  int* flag = nullptr;
  double* scal = nullptr;  // [TRACE_PARTS]
  double* traces = nullptr;   // [2 nw]
  double* Dw = nullptr;       // [2nw][n n], commutator DIIS: Sigma_out - Sigma_in in frequency
  bool have_g = false;        // Gs holds the G(i w) of a completed step
  std::vector<double> gamma_row;   // the gamma row of Wb (host)
  std::vector<void*> allocs;
  ~thcsox_dyson_s() {
    for (void* p : allocs) (void)hipFree(p);
  }
};

namespace {
template <typename T>
int dalloc(thcsox_dyson_s* d, T** p, size_t count) {
  void* q = nullptr;
  hipError_t e = hipMalloc(&q, std::max<size_t>(16, count * sizeof(T)));
  if (e != hipSuccess) {
    (void)hipGetLastError();
    return dfail(THCSOX_ENOMEM, std::string("hipMalloc failed: ") + hipGetErrorString(e));
  }
  d->allocs.push_back(q);
  *p = static_cast<T*>(q);
  return 0;
}

#define DTRY(expr)                                                                      \
  do {                                                                                  \
    hipError_t e_ = (expr);                                                             \
    if (e_ != hipSuccess)                                                               \
      return dfail(THCSOX_EDEVICE, std::string(#expr) + ": " + hipGetErrorString(e_));  \
  } while (0)
}  // namespace

namespace {

// Sigma(i w) (real and imaginary rows) = Wf . Sigma(tau)
int dy_forward(thcsox_dyson_s* d, const double* Sigma_dev) {
  const int64_t nn = (int64_t)d->n * d->n;
  Gemm64Args g{};
  g.M = 2 * d->nw; g.N = (int)nn; g.K = d->m; g.batch = 1; g.alpha = 1.0; g.beta = 0.0;
  g.A = d->Wf; g.a_i = d->m; g.a_k = 1;
  g.B = Sigma_dev; g.b_k = nn; g.b_j = 1;
  g.C = d->Siw; g.c_i = nn; g.c_j = 1; g.cj_in = nn; g.cj_out = 0;
  DTRY(gemm64(g, d->stream));
  return 0;
}

// G(i w) = [(i w + mu) 1 - F - Sigma(i w)]^-1 for every frequency, left in Am
// (permuted by piv and col); flag set for a singular matrix.
int dy_invert(thcsox_dyson_s* d, double mu) {
  const int n = d->n, nw = d->nw;
  const int64_t nn = (int64_t)n * n;
  const hipStream_t s = d->stream;
  const unsigned bx = (unsigned)std::min<int64_t>(64, (nn + NT - 1) / NT);
  build_a<<<dim3(bx, nw), NT, 0, s>>>(d->Siw, d->F, mu, d->wfreq, n, nw, d->Am, d->flag);
  DTRY(hipGetLastError());
  DTRY(gj_inverse(d->Am, n, nw, d->piv, d->col, d->flag, s));
  return 0;
}

// Tr gamma of the inverses in Am: gamma = sum_j Wb[m][j] [Re G; Im G]_j, so only
// the traces of the G(i w) are needed.  Synchronises the stream.
int dy_electrons(thcsox_dyson_s* d, double* N) {
  inv_traces<<<d->nw, NT, 0, d->stream>>>(d->Am, d->piv, d->col, d->n, d->nw, d->traces);
  DTRY(hipGetLastError());
  std::vector<double> tr((size_t)2 * d->nw);
  int flag = 0;
  DTRY(hipMemcpyAsync(tr.data(), d->traces, sizeof(double) * tr.size(), hipMemcpyDeviceToHost,
                      d->stream));
  DTRY(hipMemcpyAsync(&flag, d->flag, sizeof(int), hipMemcpyDeviceToHost, d->stream));
  DTRY(hipStreamSynchronize(d->stream));
  if (flag) return dfail(THCSOX_ENONFINITE, "singular matrix in the Dyson solve");
  double acc = 0.0;
  for (size_t j = 0; j < tr.size(); ++j) acc += d->gamma_row[j] * tr[j];
  *N = acc;
  return 0;
}

// unpack the inverses, fit back to tau: G_dev[m][n][n] and gamma_dev[n][n]
int dy_backward(thcsox_dyson_s* d, double* G_dev, double* gamma_dev) {
  const int n = d->n, m = d->m, nw = d->nw;
  const int64_t nn = (int64_t)n * n;
  const hipStream_t s = d->stream;
  const unsigned bx = (unsigned)std::min<int64_t>(64, (nn + NT - 1) / NT);
  extract_inv<<<dim3(bx, nw), NT, 0, s>>>(d->Am, d->piv, d->col, n, nw, d->Gs);
  DTRY(hipGetLastError());
  d->have_g = true;
  // [G(tau_0) .. G(tau_{m-1}); gamma] = Wb . [Re G(i w); Im G(i w)]
  Gemm64Args g{};
  g.M = m + 1; g.N = (int)nn; g.K = 2 * nw; g.batch = 1; g.alpha = 1.0; g.beta = 0.0;
  g.A = d->Wb; g.a_i = 2 * nw; g.a_k = 1;
  g.B = d->Gs; g.b_k = nn; g.b_j = 1;
  g.C = d->Gout; g.c_i = nn; g.c_j = 1; g.cj_in = nn; g.cj_out = 0;
  DTRY(gemm64(g, s));
  DTRY(hipMemcpyAsync(G_dev, d->Gout, sizeof(double) * m * nn, hipMemcpyDeviceToDevice, s));
  if (gamma_dev)
    DTRY(hipMemcpyAsync(gamma_dev, d->Gout + (int64_t)m * nn, sizeof(double) * nn,
                        hipMemcpyDeviceToDevice, s));
  int flag = 0;
  DTRY(hipMemcpyAsync(&flag, d->flag, sizeof(int), hipMemcpyDeviceToHost, s));
  DTRY(hipStreamSynchronize(s));
  if (flag) return dfail(THCSOX_ENONFINITE, "singular matrix in the Dyson solve");
  return 0;
}

}  // namespace

namespace {
// The plan on given transform tables (Wf [2 nw][m], Wb [m + 1][2 nw]) and
// frequencies wf[nw]; F_dev is checked to be device memory.
int dyson_create(thcsox_dyson_t* out, int n, int m, int nw, double beta, double mu,
                 const std::vector<double>& wf, const std::vector<double>& Wf,
                 const std::vector<double>& Wb, const double* F_dev, void* hip_stream) {
  hipPointerAttribute_t a;
  if (hipPointerGetAttributes(&a, F_dev) != hipSuccess ||
      (a.type != hipMemoryTypeDevice && a.type != hipMemoryTypeManaged)) {
    (void)hipGetLastError();
    return dfail(THCSOX_ENOTDEV, "F_dev is not device memory");
  }
  auto* d = new (std::nothrow) thcsox_dyson_s();
  if (d == nullptr) return dfail(THCSOX_ENOMEM, "host allocation failed");
  d->n = n; d->m = m; d->nw = nw; d->beta = beta; d->mu = mu;
  d->stream = static_cast<hipStream_t>(hip_stream);
  const int64_t nn = (int64_t)n * n;
  int rc;
  if ((rc = dalloc(d, &d->F, nn)) || (rc = dalloc(d, &d->Wf, (size_t)2 * d->nw * d->m)) ||
      (rc = dalloc(d, &d->Wb, (size_t)(d->m + 1) * 2 * d->nw)) ||
      (rc = dalloc(d, &d->wfreq, (size_t)d->nw)) ||
      (rc = dalloc(d, &d->Siw, (size_t)2 * d->nw * nn)) ||
      (rc = dalloc(d, &d->Am, (size_t)d->nw * nn)) ||
      (rc = dalloc(d, &d->piv, (size_t)d->nw * n)) ||
      (rc = dalloc(d, &d->col, (size_t)d->nw * n)) ||
      (rc = dalloc(d, &d->Gs, (size_t)2 * d->nw * nn)) ||
      (rc = dalloc(d, &d->Gout, (size_t)(d->m + 1) * nn)) || (rc = dalloc(d, &d->flag, 1)) ||
      (rc = dalloc(d, &d->scal, TRACE_PARTS)) || (rc = dalloc(d, &d->traces, (size_t)2 * d->nw))) {
    delete d;
    return rc;
  }
  d->gamma_row.assign(Wb.begin() + (size_t)d->m * 2 * d->nw, Wb.begin() + (size_t)(d->m + 1) * 2 * d->nw);
  hipError_t e;
  if ((e = hipMemcpyAsync(d->F, F_dev, sizeof(double) * nn, hipMemcpyDeviceToDevice, d->stream)) ||
      (e = hipMemcpyAsync(d->Wf, Wf.data(), sizeof(double) * Wf.size(),
                          hipMemcpyHostToDevice, d->stream)) ||
      (e = hipMemcpyAsync(d->Wb, Wb.data(), sizeof(double) * Wb.size(),
                          hipMemcpyHostToDevice, d->stream)) ||
      (e = hipMemcpyAsync(d->wfreq, wf.data(), sizeof(double) * wf.size(),
                          hipMemcpyHostToDevice, d->stream)) ||
      (e = hipStreamSynchronize(d->stream))) {
    delete d;
    return dfail(THCSOX_EDEVICE, std::string("dyson plan: ") + hipGetErrorString(e));
  }
  *out = d;
  return 0;
}
}  // namespace

extern "C" {

int thcsox_dyson_plan(thcsox_dyson_t* out, int n, int ntau, int n_matsubara, double beta,
                      double mu, const double* tau_host, const double* F_dev, void* hip_stream) {
  clear_error();
  if (out == nullptr) return dfail(THCSOX_EINVAL, "out is NULL");
  *out = nullptr;
  if (n <= 0 || ntau <= 1 || n_matsubara <= 0 || !(beta > 0.0))
    return dfail(THCSOX_EINVAL, "need n > 0, ntau > 1, n_matsubara > 0, beta > 0");
  if (n > GJ_MAX_N)
    return dfail(THCSOX_EINVAL, "n too large for the Dyson inversion (n <= 9216)");
  if (2 * n_matsubara < ntau)
    return dfail(THCSOX_EINVAL, "need 2 n_matsubara >= ntau for the least-squares fit");
  if (tau_host == nullptr || F_dev == nullptr) return dfail(THCSOX_EINVAL, "NULL argument");
  for (int k = 0; k < ntau; ++k) {
    const double x = -std::cos((2.0 * k + 1.0) * M_PI / (2.0 * ntau));
    if (std::fabs(tau_host[k] - 0.5 * beta * (1.0 + x)) > 1e-12 * beta)
      return dfail(THCSOX_EINVAL, "tau grid is not the Chebyshev-root grid");
  }
  try {   // host tables: no exception may cross the C interface
    const Tables& tb = tables_for(ntau, n_matsubara, beta);
    std::vector<double> wf(n_matsubara);
    for (int j = 0; j < n_matsubara; ++j) wf[j] = (2.0 * j + 1.0) * M_PI / beta;
    return dyson_create(out, n, ntau, n_matsubara, beta, mu, wf, tb.Wf, tb.Wb, F_dev, hip_stream);
  } catch (const std::bad_alloc&) {
    return dfail(THCSOX_ENOMEM, "host allocation failed");
  }
}

int thcsox_dyson_plan_sampled(thcsox_dyson_t* out, int n, int ntau, int nfreq, double beta,
                              double mu, const int* freq_n_host, const double* Wf_host,
                              const double* Wb_host, const double* F_dev, void* hip_stream) {
  clear_error();
  if (out == nullptr) return dfail(THCSOX_EINVAL, "out is NULL");
  *out = nullptr;
  if (n <= 0 || ntau <= 1 || nfreq <= 0 || !(beta > 0.0))
    return dfail(THCSOX_EINVAL, "need n > 0, ntau > 1, nfreq > 0, beta > 0");
  if (n > GJ_MAX_N)
    return dfail(THCSOX_EINVAL, "n too large for the Dyson inversion (n <= 9216)");
  if (2 * nfreq < ntau) return dfail(THCSOX_EINVAL, "need 2 nfreq >= ntau for the fit");
  if (freq_n_host == nullptr || Wf_host == nullptr || Wb_host == nullptr || F_dev == nullptr)
    return dfail(THCSOX_EINVAL, "NULL argument");
  for (int j = 0; j < nfreq; ++j)
    if (freq_n_host[j] < 0 || (j > 0 && freq_n_host[j] <= freq_n_host[j - 1]))
      return dfail(THCSOX_EINVAL, "freq_n must be ascending and >= 0");
  try {   // host copies of the tables: no exception may cross the C interface
    std::vector<double> Wf(Wf_host, Wf_host + (size_t)2 * nfreq * ntau);
    std::vector<double> Wb(Wb_host, Wb_host + (size_t)(ntau + 1) * 2 * nfreq);
    for (double v : Wf)
      if (!std::isfinite(v)) return dfail(THCSOX_EINVAL, "Wf has a non-finite entry");
    for (double v : Wb)
      if (!std::isfinite(v)) return dfail(THCSOX_EINVAL, "Wb has a non-finite entry");
    // the plan's last table row gives gamma = -G(beta^-) directly
    for (size_t j = (size_t)ntau * 2 * nfreq; j < Wb.size(); ++j) Wb[j] = -Wb[j];
    std::vector<double> wf(nfreq);
    for (int j = 0; j < nfreq; ++j) wf[j] = (2.0 * freq_n_host[j] + 1.0) * M_PI / beta;
    return dyson_create(out, n, ntau, nfreq, beta, mu, wf, Wf, Wb, F_dev, hip_stream);
  } catch (const std::bad_alloc&) {
    return dfail(THCSOX_ENOMEM, "host allocation failed");
  }
}

int thcsox_dyson_step(thcsox_dyson_t d, const double* Sigma_dev, double* G_dev, double* gamma_dev) {
  clear_error();
  if (d == nullptr || Sigma_dev == nullptr || G_dev == nullptr)
    return dfail(THCSOX_EINVAL, "NULL argument");
  int rc;
  if ((rc = dy_forward(d, Sigma_dev)) || (rc = dy_invert(d, d->mu))) return rc;
  return dy_backward(d, G_dev, gamma_dev);
}

int thcsox_dyson_step_mu(thcsox_dyson_t d, const double* Sigma_dev, double nelec, double tol,
                         double* mu_io, double* G_dev, double* gamma_dev, int* evals_out) {
  clear_error();
  if (d == nullptr || Sigma_dev == nullptr || G_dev == nullptr || mu_io == nullptr)
    return dfail(THCSOX_EINVAL, "NULL argument");
  if (!(nelec >= 0.0) || !(nelec <= d->n) || !(tol > 0.0) || !std::isfinite(*mu_io))
    return dfail(THCSOX_EINVAL, "need 0 <= nelec <= n, tol > 0 and a finite starting mu");
  int rc;
  if ((rc = dy_forward(d, Sigma_dev))) return rc;
  // f(mu) = Tr gamma(mu) - nelec, one Dyson solve per evaluation; the last
  // evaluated mu is the answer, so its inverses are the ones left in Am
  int evals = 0;
  auto f = [&](double mu, double* val) -> int {
    int r;
    if ((r = dy_invert(d, mu)) || (r = dy_electrons(d, val))) return r;
    *val -= nelec;
    ++evals;
    return 0;
  };
  constexpr int MAX_EVAL = 80;
  constexpr double STEP = 0.1;   // first bracketing step (Ha), doubled while the sign holds
  double a = *mu_io, fa, b, fb, mu = a;
  bool done = false;
  if ((rc = f(a, &fa))) return rc;
  if (std::fabs(fa) <= tol) done = true;
  if (!done) {
    double step = fa > 0 ? -STEP : STEP;
    b = a + step;
    if ((rc = f(b, &fb))) return rc;
    while (fa * fb > 0 && evals < MAX_EVAL) {
      a = b;
      fa = fb;
      step *= 2.0;
      b = a + step;
      if ((rc = f(b, &fb))) return rc;
    }
    mu = b;
    if (std::fabs(fb) <= tol) done = true;
    else if (fa * fb > 0) return dfail(THCSOX_ENONFINITE, "no bracket for the chemical potential");
  }
  // Illinois variant of regula falsi on the bracket (a, b)
  while (!done) {
    if (evals >= MAX_EVAL) return dfail(THCSOX_ENONFINITE, "chemical potential search did not converge");
    const double c = (a * fb - b * fa) / (fb - fa);
    double fc;
    if ((rc = f(c, &fc))) return rc;
    mu = c;
    if (std::fabs(fc) <= tol || std::fabs(b - a) <= 1e-14 * (1.0 + std::fabs(c))) break;
    if (fc * fb < 0) {
      a = b;
      fa = fb;
    } else {
      fa *= 0.5;
    }
    b = c;
    fb = fc;
  }
  d->mu = mu;
  *mu_io = mu;
  if (evals_out) *evals_out = evals;
  return dy_backward(d, G_dev, gamma_dev);
}

int thcsox_dyson_commutator(thcsox_dyson_t d, const double* Sigma_in_dev,
                            const double* Sigma_out_dev, double* e_dev) {
  clear_error();
  if (d == nullptr || Sigma_in_dev == nullptr || Sigma_out_dev == nullptr || e_dev == nullptr)
    return dfail(THCSOX_EINVAL, "NULL argument");
  for (const void* q : {(const void*)Sigma_in_dev, (const void*)Sigma_out_dev, (const void*)e_dev}) {
    hipPointerAttribute_t a;
    if (hipPointerGetAttributes(&a, q) != hipSuccess ||
        (a.type != hipMemoryTypeDevice && a.type != hipMemoryTypeManaged)) {
      (void)hipGetLastError();
      return dfail(THCSOX_ENOTDEV, "arrays must be device memory");
    }
  }
  if (!d->have_g) return dfail(THCSOX_EINVAL, "no Dyson step has been taken on this plan");
  const int n = d->n, nw = d->nw, m = d->m;
  const int64_t nn = (int64_t)n * n;
  const hipStream_t s = d->stream;
  if (d->Dw == nullptr) {
    int rc = dalloc(d, &d->Dw, (size_t)2 * nw * nn);
    if (rc) return rc;
  }
  // D(i w) = Wf (Sigma_out - Sigma_in), as [Re; Im] rows
  Gemm64Args g{};
  g.M = 2 * nw; g.N = (int)nn; g.K = m; g.batch = 1; g.alpha = 1.0; g.beta = 0.0;
  g.A = d->Wf; g.a_i = m; g.a_k = 1;
  g.B = Sigma_out_dev; g.b_k = nn; g.b_j = 1;
  g.C = d->Dw; g.c_i = nn; g.c_j = 1; g.cj_in = nn; g.cj_out = 0;
  g.more = 1; g.A_t[0] = d->Wf; g.B_t[0] = Sigma_in_dev; g.sign[0] = -1.0;
  DTRY(gemm64(g, s));
  // e = G D - D G per frequency, G = Gr + i Gi from the last step (d->Gs), D = Dr + i Di:
  //   Re e = Gr Dr - Gi Di - Dr Gr + Di Gi,  Im e = Gr Di + Gi Dr - Dr Gi - Di Gr
  const double* Gr = d->Gs;
  const double* Gi = d->Gs + (int64_t)nw * nn;
  const double* Dr = d->Dw;
  const double* Di = d->Dw + (int64_t)nw * nn;
  double* er = e_dev;
  double* ei = e_dev + (int64_t)nw * nn;
  // four products each, summed in one pass (eight products into e one after the other
  // read and wrote e eight times: 2.6 ms against 1.8 at n = 300, 256 frequencies)
  Gemm64Args p{};
  p.M = n; p.N = n; p.K = n; p.batch = nw; p.alpha = 1.0; p.beta = 0.0;
  p.a_i = n; p.a_k = 1; p.a_b = nn;
  p.b_k = n; p.b_j = 1; p.b_b = nn;
  p.c_i = n; p.c_j = 1; p.cj_in = n; p.cj_out = 0; p.c_b = nn;
  p.more = 3;
  auto sum4 = [&](double* C, const double* A0, const double* B0, const double* A1, const double* B1,
                  double s1, const double* A2, const double* B2, const double* A3,
                  const double* B3, double s3) -> hipError_t {
    p.C = C;
    p.A = A0; p.B = B0;
    p.A_t[0] = A1; p.B_t[0] = B1; p.sign[0] = s1;
    p.A_t[1] = A2; p.B_t[1] = B2; p.sign[1] = -1.0;
    p.A_t[2] = A3; p.B_t[2] = B3; p.sign[2] = s3;
    return gemm64(p, s);
  };
  DTRY(sum4(er, Gr, Dr, Gi, Di, -1.0, Dr, Gr, Di, Gi, 1.0));
  DTRY(sum4(ei, Gr, Di, Gi, Dr, 1.0, Dr, Gi, Di, Gr, -1.0));
  return 0;
}

int thcsox_dyson_onebody(thcsox_dyson_t d, const double* gamma_dev, double* E1_host) {
  clear_error();
  if (d == nullptr || gamma_dev == nullptr || E1_host == nullptr)
    return dfail(THCSOX_EINVAL, "NULL argument");
  // a wave for each block of 64 x 32 elements, up to TRACE_PARTS workgroups
  const int64_t items = (int64_t)((d->n + 63) / 64) * ((d->n + 31) / 32);
  const int parts = (int)std::min<int64_t>(TRACE_PARTS, (items + TW - 1) / TW);
  trace_ab<<<parts, 64 * TW, 0, d->stream>>>(d->F, gamma_dev, d->n, d->scal);
  DTRY(hipGetLastError());
  double sums[TRACE_PARTS];
  DTRY(hipMemcpyAsync(sums, d->scal, sizeof(double) * parts, hipMemcpyDeviceToHost, d->stream));
  DTRY(hipStreamSynchronize(d->stream));
  double e1 = 0.0;
  for (int b = 0; b < parts; ++b) e1 += sums[b];
  *E1_host = e1;
  return 0;
}

int thcsox_dyson_destroy(thcsox_dyson_t d) {
  if (d == nullptr) return 0;
  (void)hipStreamSynchronize(d->stream);
  delete d;
  return 0;
}

}  // extern "C"
