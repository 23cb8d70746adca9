// Strided FP64 GEMM on the f64 matrix cores (projections, back-projection, U
// precontraction, the direct term, screening, the Dyson transforms).
//
// What bounds it.  A 16x16x4 f64 MFMA holds a SIMD's matrix core for 64 cycles,
// so issue slots and LDS reads are plentiful; the operand bytes are what a tile
// size decides.  A T x T tile needs 16 T bytes per k for 2 T^2 flops: at T = 64
// the full rate takes 9 TB/s out of the L2s, at 128 half of that.  So:
//   - square tiles of 128, 64 or 32 (four waves of 64, 32 or 16 square; the
//     dispatch below picks one), two LDS buffers and one barrier a k step: step t + 1
//     goes from registers to LDS and step t + 2's loads are issued before the
//     products of step t, which give them thousands of cycles.  k steps of 16, and
//     of 32 or 64 where small tiles alone on a compute unit would otherwise wait
//     for the latency of each short step's loads;
//   - at 128 two workgroups share a compute unit (64-68 KiB of LDS, 256
//     registers), so one's barrier is covered by the other's products;
//   - tiles are dealt to the XCDs in contiguous runs and walked in bands of eight
//     rows, so that the tiles on one XCD at a time share operand panels in its L2;
//   - loads carry no branch (addresses are clamped into the array): with the bounds
//     as branches each load waited for the one before it (44 TFLOP/s).
// Measured on V Pi of 12 matrices of 1800 (1800 x 1800 x 1800): 52 TFLOP/s, 67 counting
// the padding to 1920 and the last of six rounds of tiles (64 x 64 tiles with one
// LDS buffer and branches, the kernel before this one: 35); the f64 matrix peak
// is 78.6 and a library product of 8192 reaches 72.
#include <cmath>
#include <type_traits>

#include "kernels.hpp"
#include "mfma.hpp"

namespace thcsox {
namespace {

constexpr int NT = 256;      // threads per workgroup (4 wavefronts)
constexpr int NXCD = 8;
constexpr int BAND = 8;      // row tiles per band of the tile walk
// a launch of more than 2^32 - 1 threads would be cut short without an error
constexpr int64_t MAX_GRID = 0xffffffffLL / NT;
typedef double d2 __attribute__((ext_vector_type(2)));

// An operand's panel in LDS.  Within 16 k lane group g takes k = 2 g, 2 g + 1, 8 + 2 g
// and 9 + 2 g in the four MFMA steps.
// KC (k contiguous in memory): rows of BK k, 16-byte pair c of row r at the piece
//   swz(r, c): a lane reads its four k in the pieces g and 4 + g of each 16, and 16
//   rows at one pair touch 16 distinct 16-byte columns of the banks.
// otherwise (row index contiguous): [k][row], 64 bytes of padding per k, so that
//   lane groups two k apart fall on different halves of the banks.
template <int T, int BK, bool KC>
struct PanelLayout {
  static constexpr int LD = KC ? BK : T + 8;
  static constexpr int SIZE = KC ? T * BK : BK * LD;
};
template <int BK>
__device__ __forceinline__ int swz(int r, int c) {
  return BK == 16 ? c ^ ((r >> 1) & 7) : c ^ (r & 15);   // two rows of 128 bytes, or one of 256 or 512
}

// How pairs along an operand's contiguous dimension are read: 16-byte aligned, at
// any 8-byte address, or as two 8-byte loads (contiguous extent of 1).
enum Access { ALIGNED, UNALIGNED, SINGLE };
typedef double d2u __attribute__((ext_vector_type(2), aligned(8)));

// Elements x, x + 1 of the lim from p on, without a branch: addresses are clamped
// into the array, so what lies past lim is some element of it.  The callers zero
// it along k; along i and j it only reaches outputs that are not stored.
template <Access ACC>
__device__ __forceinline__ d2 pair_at(const double* p, int x, int lim) {
  if constexpr (ACC == SINGLE) return d2{p[min(x, lim - 1)], p[min(x + 1, lim - 1)]};
  const int xc = min(x, lim - 2);
  d2 v = ACC == ALIGNED ? *reinterpret_cast<const d2*>(p + xc) : *reinterpret_cast<const d2u*>(p + xc);
  if (ACC == UNALIGNED) v[0] = x > xc ? v[1] : v[0];
  return v;
}

// AC / BC: A / B contiguous in k (otherwise in i / j).
template <int WT, int BK, bool AC, bool BC, Access ACC>
__global__ __launch_bounds__(NT, WT == 2 && BK == 16 ? 4 : 2) void gemm64_kernel(Gemm64Args g, int nti, int ntj) {
  constexpr int T = 32 * WT;           // tile edge
  constexpr int RP = BK / 2;           // pairs per row of a panel contiguous in k
  constexpr int NP = T * RP / NT;      // pairs per thread and operand panel
  using LA = PanelLayout<T, BK, AC>;
  using LB = PanelLayout<T, BK, BC>;
  __shared__ __attribute__((aligned(16))) double sA[2][LA::SIZE];
  __shared__ __attribute__((aligned(16))) double sB[2][LB::SIZE];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wr = wave >> 1, wc = wave & 1;

  // tile of this workgroup: a contiguous run of tiles per XCD, bands of BAND rows
  const unsigned total = gridDim.x, per = total / NXCD, rem = total % NXCD;
  const unsigned xcd = blockIdx.x % NXCD;
  const unsigned tile = xcd * per + min(xcd, rem) + blockIdx.x / NXCD;
  const unsigned tpb = (unsigned)nti * ntj;
  const int64_t b = tile / tpb;
  const int w = (int)(tile % tpb);
  const int i_lo = w / (BAND * ntj) * BAND, bh = min(BAND, nti - i_lo);
  const int in = w - i_lo * ntj;
  const int i0 = (i_lo + in % bh) * T, j0 = in / bh * T;
  int lt = 0, lk = 0;   // the step to load next: term lt, from k = lk
  const double* A = g.A + b * g.a_b;
  const double* B = g.B + b * g.b_b;

  struct Held {   // a step in registers
    d2 a[NP], b[NP];
    int k0;
    double sign;
  };
  auto load = [&](Held& h) {
    const int k0 = h.k0 = lk;
    h.sign = lt == 0 ? 1.0 : g.sign[lt - 1];
#pragma unroll
    for (int t = 0; t < NP; ++t) {
      const int e = tid + NT * t;
      if (AC) {   // row i, k pair
        const int i = min(i0 + e / RP, g.M - 1);
        h.a[t] = pair_at<ACC>(A + (int64_t)i * g.a_i, k0 + 2 * (e % RP), g.K);
      } else {    // one k, i pair
        const int k = min(k0 + e / (T / 2), g.K - 1);
        h.a[t] = pair_at<ACC>(A + (int64_t)k * g.a_k, i0 + 2 * (e % (T / 2)), g.M);
      }
      if (BC) {
        const int j = min(j0 + e / RP, g.N - 1);
        h.b[t] = pair_at<ACC>(B + (int64_t)j * g.b_j, k0 + 2 * (e % RP), g.K);
      } else {
        const int k = min(k0 + e / (T / 2), g.K - 1);
        h.b[t] = pair_at<ACC>(B + (int64_t)k * g.b_k, j0 + 2 * (e % (T / 2)), g.N);
      }
    }
    lk += BK;
    if (lk >= g.K && lt < g.more) {
      lk = 0;
      A = g.A_t[lt] + b * g.a_b;
      B = g.B_t[lt] + b * g.b_b;
      ++lt;
    }
  };
  // what lies past K in the pair e of a panel whose step starts at k0
  auto cut = [&](bool kc, int e, int k0, d2 v) {
    const int k = k0 + (kc ? 2 * (e % RP) : e / (T / 2));
    return d2{k < g.K ? v[0] : 0.0, k + (kc ? 1 : 0) < g.K ? v[1] : 0.0};
  };
  auto put = [&](bool kc, double* s, int ld, int e, d2 v) {
    const int at = kc ? e / RP * BK + (swz<BK>(e / RP, e % RP) << 1)
                      : e / (T / 2) * ld + 2 * (e % (T / 2));
    *reinterpret_cast<d2*>(s + at) = v;
  };
  auto store = [&](int buf, Held& h) {
    if (h.k0 + BK > g.K) {
#pragma unroll
      for (int t = 0; t < NP; ++t) {
        h.a[t] = cut(AC, tid + NT * t, h.k0, h.a[t]);
        h.b[t] = cut(BC, tid + NT * t, h.k0, h.b[t]);
      }
    }
    if (g.more > 0) {
#pragma unroll
      for (int t = 0; t < NP; ++t) h.a[t] *= h.sign;
    }
#pragma unroll
    for (int t = 0; t < NP; ++t) {
      put(AC, sA[buf], LA::LD, tid + NT * t, h.a[t]);
      put(BC, sB[buf], LB::LD, tid + NT * t, h.b[t]);
    }
  };
  const int fr = lane & 15, fg = lane >> 4;
  // elements k = 16 kb + 8 h + 2 fg and the next of row 16 t + fr of the wave's part
  auto frag = [&](bool kc, const double* s, int ld, int r0, int t, int kb, int h) -> d2 {
    const int r = r0 + 16 * t + fr;
    if (kc) return *reinterpret_cast<const d2*>(s + r * BK + (swz<BK>(r, 8 * kb + 4 * h + fg) << 1));
    const int k = 16 * kb + 8 * h + 2 * fg;
    return d2{s[k * ld + r], s[(k + 1) * ld + r]};
  };

  d4 acc[WT][WT];
#pragma unroll
  for (int ti = 0; ti < WT; ++ti)
#pragma unroll
    for (int tj = 0; tj < WT; ++tj) acc[ti][tj] = d4{0.0, 0.0, 0.0, 0.0};

  auto multiply = [&](int buf) {
#pragma unroll
    for (int kh = 0; kh < BK / 8; ++kh) {
      d2 a[WT], bb[WT];
#pragma unroll
      for (int t = 0; t < WT; ++t) {
        a[t] = frag(AC, sA[buf], LA::LD, 16 * WT * wr, t, kh >> 1, kh & 1);
        bb[t] = frag(BC, sB[buf], LB::LD, 16 * WT * wc, t, kh >> 1, kh & 1);
      }
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int ti = 0; ti < WT; ++ti)
#pragma unroll
          for (int tj = 0; tj < WT; ++tj) acc[ti][tj] = mfma1(a[ti][s], bb[tj][s], acc[ti][tj]);
    }
  };
  // In step st the buffer st mod 2 is multiplied while step st + 1 goes from registers to
  // the other one and later steps load: st + 2, and st + 3 where registers allow.
  constexpr bool DEEP = WT < 4;
  const int steps = (g.K + BK - 1) / BK * (g.more + 1);
  Held h0, h1;
  Held& later = DEEP ? h1 : h0;
  load(h0);
  if (DEEP && steps > 1) load(h1);
  store(0, h0);
  if (steps > (DEEP ? 2 : 1)) load(h0);
  __syncthreads();
  auto step = [&](int st, int cur, Held& h) {
    if (st + 1 < steps) store(cur ^ 1, h);
    if (st + (DEEP ? 3 : 2) < steps) load(h);
    multiply(cur);
    __syncthreads();
  };
  for (int st = 0; st < steps; st += 2) {
    step(st, 0, later);
    if (st + 1 < steps) step(st + 1, 1, h0);
  }
#pragma unroll
  for (int tj = 0; tj < WT; ++tj) {
    const int j = j0 + 16 * (WT * wc + tj) + fr;
    if (j >= g.N) continue;
    double* C = g.C + b * g.c_b + ((int64_t)j / g.cj_in) * g.cj_out + ((int64_t)j % g.cj_in) * g.c_j;
    auto row = [&](int ti, int r) { return i0 + 16 * (WT * wr + ti) + out_row<MODE_F64>(lane, r); };
    if (g.beta != 0.0) {   // the column's old values first, all in flight together
      double old[WT][4];
#pragma unroll
      for (int ti = 0; ti < WT; ++ti)
#pragma unroll
        for (int r = 0; r < 4; ++r) old[ti][r] = C[(int64_t)min(row(ti, r), g.M - 1) * g.c_i];
#pragma unroll
      for (int ti = 0; ti < WT; ++ti)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (row(ti, r) < g.M)
            C[(int64_t)row(ti, r) * g.c_i] = g.alpha * acc[ti][tj][r] + g.beta * old[ti][r];
    } else {
#pragma unroll
      for (int ti = 0; ti < WT; ++ti)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (row(ti, r) < g.M) C[(int64_t)row(ti, r) * g.c_i] = g.alpha * acc[ti][tj][r];
    }
  }
}

template <int WT, int BK, Access ACC>
hipError_t launch(const Gemm64Args& g, bool ac, bool bc, hipStream_t s) {
  const int64_t nti = (g.M + 32 * WT - 1) / (32 * WT), ntj = ((int64_t)g.N + 32 * WT - 1) / (32 * WT);
  const int64_t total = nti * ntj * g.batch;
  if (total > MAX_GRID) return hipErrorInvalidValue;
  const dim3 grid((unsigned)total);
  const int ni = (int)nti, nj = (int)ntj;
  if (ac && bc) gemm64_kernel<WT, BK, true, true, ACC><<<grid, NT, 0, s>>>(g, ni, nj);
  else if (ac) gemm64_kernel<WT, BK, true, false, ACC><<<grid, NT, 0, s>>>(g, ni, nj);
  else if (bc) gemm64_kernel<WT, BK, false, true, ACC><<<grid, NT, 0, s>>>(g, ni, nj);
  else gemm64_kernel<WT, BK, false, false, ACC><<<grid, NT, 0, s>>>(g, ni, nj);
  return hipGetLastError();
}

}  // namespace

hipError_t gemm64(const Gemm64Args& g, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0 || g.batch <= 0) return hipSuccess;
  if (g.K <= 0 || g.more < 0 || g.more > 3) return hipErrorInvalidValue;
  // the contiguous dimension of each operand
  if ((g.a_k != 1 && g.a_i != 1) || (g.b_j != 1 && g.b_k != 1)) return hipErrorInvalidValue;
  const bool ac = g.a_k == 1, bc = g.b_j != 1;
  const int ext_a = ac ? g.K : g.M, ext_b = bc ? g.K : g.N;   // contiguous extents
  if (ext_a < 2 || ext_b < 2) return launch<1, 64, SINGLE>(g, ac, bc, s);
  // 16-byte loads need even strides, even extents and 16-byte aligned bases (tile
  // starts are even)
  auto even = [](int64_t x) { return (x & 1) == 0; };
  uintptr_t low = reinterpret_cast<uintptr_t>(g.A) | reinterpret_cast<uintptr_t>(g.B);
  for (int t = 0; t < g.more; ++t)
    low |= reinterpret_cast<uintptr_t>(g.A_t[t]) | reinterpret_cast<uintptr_t>(g.B_t[t]);
  const bool aligned = even(ext_a) && even(ext_b) && even(ac ? g.a_i : g.a_k) && even(g.a_b) &&
                       even(bc ? g.b_j : g.b_k) && even(g.b_b) &&
                       (low & 15) == 0;
  // tile edge: the least of rounds of tiles over 256 compute units x tile area x
  // the cost per element of that tile on a full unit relative to the largest
  auto cost = [&](int t, double rel) {
    const double tiles = std::ceil((double)g.M / t) * std::ceil((double)g.N / t) * g.batch;
    return std::ceil(tiles / 256.0) * (double)t * t * rel;
  };
  const double c4 = cost(128, 1.0), c2 = cost(64, 1.3), c1 = cost(32, 2.0);
  auto go = [&](auto wt, auto bk) {
    constexpr int W = decltype(wt)::value, K = decltype(bk)::value;
    return aligned ? launch<W, K, ALIGNED>(g, ac, bc, s) : launch<W, K, UNALIGNED>(g, ac, bc, s);
  };
  using std::integral_constant;
  if (c4 <= c2 && c4 <= c1) return go(integral_constant<int, 4>(), integral_constant<int, 16>());
  if (c2 <= c1) {
    // 64: short steps where three or more workgroups share a compute unit, else long
    // ones (1740 tiles, K = 1800: 390 us at 16, 423 at 32; 256 tiles, K = 485: 58, 48)
    const double tiles = std::ceil(g.M / 64.0) * std::ceil(g.N / 64.0) * g.batch;
    if (tiles >= 768) return go(integral_constant<int, 2>(), integral_constant<int, 16>());
    return go(integral_constant<int, 2>(), integral_constant<int, 32>());
  }
  return go(integral_constant<int, 1>(), integral_constant<int, 64>());
}

}  // namespace thcsox
