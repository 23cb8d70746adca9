// The fused B/C/D stage of the THC-SOX sequence in the FP64 mode, and the dispatch of
// the other modes' kernels:
//
//   D_PR = sum_v C_RvP B_PRv,   B_PRv = sum_q G_Rq A_Pqv,   C_RvP = sum_w U_Rvw G_wP
//
// A workgroup owns a 64 (R) x 64 (P) tile of D of one tau point and a range of v.
// For every v it forms both length-n contractions on the f64 matrix cores,
//   accB[R][P] = sum_q Gt[R][q] A[v][P][q]      accC[R][P] = sum_w U[R][v][w] GXt[P][w]
// which land in the same MFMA output layout, so D += B o C is a register-to-register
// product.  Neither B (naux^2 n) nor C ever reaches memory.
//
// What bounds it: the f64 matrix cores (a 16x16x4 product holds one for 64 cycles), as
// long as something keeps them fed.  Operands go from memory straight to LDS, 16 k
// of four panels (G, A_v, U_v, GX: 64 rows of 128 bytes each, 32 KiB) per stage, one
// stage ahead in the other of two buffers, so that two workgroups share a compute
// unit: each SIMD has a wave of the other one to run while this one waits at its
// barrier (one a stage).  A wave owns 32 x 32 of the tile (16 x 16 tiles alternating
// between the waves): 32 products a stage against
// 16 fragment reads.  Matrix cores busy 81 % of the cycles
// (counters); n = 200, naux = 1100, symmetric: 1.70 ms a tau point (57 TFLOP/s
// algorithmic, 72 is what a large library product reaches), 3.34 with panels staged
// through registers and one workgroup of 136 KiB per unit.
#include <algorithm>

#include "kernels.hpp"
#include "mfma.hpp"
#include "panel.hpp"

namespace thcsox {
namespace {

constexpr int NXCD = 8;      // accelerator complex dies of an MI355X
constexpr int TD = 64;       // tile edge of D
constexpr int DK = 16;       // k per stage
// two waves' 16 x 16 tiles side by side make a strip (see SYM_BLOCK)
static_assert(SYM_BLOCK == 32 && TD % SYM_BLOCK == 0, "the strips are the blocks of a symmetric D");
constexpr int BAND = 1;      // R blocks per band of the tile walk (measured at n = 300: 5 % faster than 4)

// One panel of a stage: 64 rows of 16 k, the eight 16-byte pieces of row r permuted by
// XOR with r / 2 mod 8, so that 16 rows read at one piece touch all of the banks.
struct Stage64 {
  double g[TD * DK], a[TD * DK], u[TD * DK], x[TD * DK];
};
__device__ __forceinline__ int sw64(int r, int c) { return c ^ ((r >> 1) & 7); }

// One tile's range of v.  Each wave forms TI x TJ tiles of 16 x 16 out of its 2 x 2: rows
// beyond 32 TI and columns beyond 32 TJ lie past naux.  TRI: a diagonal tile of a symmetric
// D, of which only the 16 x 16 tiles ti <= tj of each wave are formed: they hold every
// element on and above the diagonal.
template <int TI, int TJ, bool TRI>
__device__ __forceinline__ void fused_f64_tile(const FusedArgs& f, Stage64& b0, Stage64& b1, int set,
                                               int z, int R0, int P0) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wr = wave >> 1, wc = wave & 1;
  // v range: XCD x owns the consecutive ranges x q .. x q + q - 1 (q = vsplit / NXCD),
  // and the ranges split n as evenly as floor division allows, so every XCD gets
  // the same number of v to within one; range r is [r n / vsplit, (r + 1) n / vsplit)
  const int vr = (z % NXCD) * (f.vsplit / NXCD) + z / NXCD;
  const int v_lo = __builtin_amdgcn_readfirstlane((int)((int64_t)vr * f.n / f.vsplit));
  const int v_hi = __builtin_amdgcn_readfirstlane((int)((int64_t)(vr + 1) * f.n / f.vsplit));
  const int kst = (f.n + DK - 1) / DK;   // rows are zero from n to ldk
  const int nstage = (v_hi - v_lo) * kst;
  const int64_t ldk = f.ldk;
  const int rows_r = min(TD, f.naux - R0), rows_p = min(TD, f.naux - P0);

  // operands (rows past the valid range lie beyond the buffer resources and read as zero)
  const double* Gt = static_cast<const double*>(f.Gt) + set * f.g_set + R0 * ldk;
  const double* GX = static_cast<const double*>(f.GXt) + set * f.g_set + P0 * ldk;
  const double* U = static_cast<const double*>(f.U) + (int64_t)R0 * f.n * ldk;
  const double* A = static_cast<const double*>(f.A) + set * f.a_set + P0 * ldk;
  // (byte counts below 2^31: checked by the launcher)
  const i4 rG = raw_rsrc(Gt, rows_r * f.ldk * 8);
  const i4 rX = raw_rsrc(GX, rows_p * f.ldk * 8);
  i4 rA, rU;
  auto set_v = [&](int v) {
    rA = raw_rsrc(A + (int64_t)v * f.naux * ldk, rows_p * f.ldk * 8);
    rU = raw_rsrc(U + v * ldk, ((rows_r - 1) * f.n * f.ldk + f.ldk) * 8);
  };
  // memory to LDS: one instruction moves 8 rows x 128 bytes; wave w moves the 8-row
  // slabs w and w + 4 of each panel.  Lane l lands at slab row l / 8, piece l % 8, and
  // loads the piece sw64 maps there.
  uint32_t dR[2], dU[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int row = (wave + 4 * j) * 8 + (lane >> 3);
    const int c = sw64(row, lane & 7);
    dR[j] = (uint32_t)(row * f.ldk + 2 * c) * 8;
    dU[j] = (uint32_t)(row * (f.n * f.ldk) + 2 * c) * 8;
  }
  int lv = v_lo, lk = 0;   // the next stage to load
  auto fetch = [&](Stage64& s) {
    const int so = lk * DK * 8;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int slab = (wave + 4 * j) * 8 * DK;
      if (j < TI) dma16_untracked(rG, lds_addr(&s.g[slab]), dR[j], so);
      if (j < TJ) dma16_untracked(rA, lds_addr(&s.a[slab]), dR[j], so);
      if (j < TI) dma16_untracked(rU, lds_addr(&s.u[slab]), dU[j], so);
      if (j < TJ) dma16_untracked(rX, lds_addr(&s.x[slab]), dR[j], so);
    }
    if (++lk == kst) {
      lk = 0;
      if (++lv < v_hi) set_v(lv);
    }
  };
  // fragments: lane group g takes k = 2 g, 2 g + 1, 8 + 2 g and 9 + 2 g in the stage's four
  // products, the 16-byte pieces g and 4 + g of its row (2 g and 2 g + 1 cost bank
  // conflicts on a tenth of the cycles; sw64 depends on the row mod 16 only)
  const int lr = lane & 15, fg = lane >> 4;
  const int o0 = lr * DK + 2 * sw64(lr, fg), o1 = lr * DK + 2 * sw64(lr, 4 + fg);
  typedef double d2 __attribute__((ext_vector_type(2)));
  auto frag = [&](const double* p, int row0, double (&o)[4]) {
    const d2 lo = *reinterpret_cast<const d2*>(p + row0 * DK + o0);
    const d2 hi = *reinterpret_cast<const d2*>(p + row0 * DK + o1);
    o[0] = lo[0]; o[1] = lo[1]; o[2] = hi[0]; o[3] = hi[1];
  };
  d4 accB[TI][TJ], accC[TI][TJ], accD[TI][TJ];
  const d4 zero = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int ti = 0; ti < TI; ++ti)
#pragma unroll
    for (int tj = TRI ? ti : 0; tj < TJ; ++tj) accB[ti][tj] = accC[ti][tj] = accD[ti][tj] = zero;
  auto product = [&](d4 (&acc)[TI][TJ], const double* rows, const double* cols) {
    double r[TI][4], c[TJ][4];
#pragma unroll
    for (int t = 0; t < TI; ++t) frag(rows, 16 * wr + 32 * t, r[t]);
#pragma unroll
    for (int t = 0; t < TJ; ++t) frag(cols, 16 * wc + 32 * t, c[t]);
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int ti = 0; ti < TI; ++ti)
#pragma unroll
        for (int tj = TRI ? ti : 0; tj < TJ; ++tj) acc[ti][tj] = mfma1(r[ti][s], c[tj][s], acc[ti][tj]);
  };
  // (the loads are issued in inline assembly: left to the compiler, a read of one
  // buffer waits for the loads just issued into the other)
  if (nstage > 0) {
    set_v(v_lo);
    fetch(b0);
  }
  int ks = 0, st = 0;
  auto stage = [&](Stage64& cur, Stage64& nxt) {
    // this wave's loads of the stage have landed; after the barrier every wave's have,
    // and every wave is done with the other buffer
    __asm__ volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if (st + 1 < nstage) fetch(nxt);
    product(accB, cur.g, cur.a);
    product(accC, cur.u, cur.x);
    if (++ks == kst) {   // all k of this v done: D += B o C
      ks = 0;
#pragma unroll
      for (int ti = 0; ti < TI; ++ti)
#pragma unroll
        for (int tj = TRI ? ti : 0; tj < TJ; ++tj) {
#pragma unroll
          for (int r = 0; r < 4; ++r)
            accD[ti][tj][r] = fma(accB[ti][tj][r], accC[ti][tj][r], accD[ti][tj][r]);
          accB[ti][tj] = accC[ti][tj] = zero;
        }
    }
    ++st;
  };
  while (st < nstage) {
    stage(b0, b1);
    if (st < nstage) stage(b1, b0);
  }
  // the partial tile (zeros for an empty v range)
  double* D = f.Dpart + set * f.d_set + (int64_t)z * f.naux * f.naux;
#pragma unroll
  for (int ti = 0; ti < TI; ++ti)
#pragma unroll
    for (int tj = TRI ? ti : 0; tj < TJ; ++tj)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int R = R0 + 16 * wr + 32 * ti + out_row<MODE_F64>(lane, r);
        const int P = P0 + 16 * wc + 32 * tj + lr;
        if (R < f.naux && P < f.naux) D[(int64_t)R * f.naux + P] = accD[ti][tj][r];
      }
}

__global__ __launch_bounds__(NT, 2) void fused_f64_kernel(FusedArgs f) {
  __shared__ __attribute__((aligned(16))) Stage64 b0;
  __shared__ __attribute__((aligned(16))) Stage64 b1;
  // XCD-aware placement.  Workgroups are dealt round-robin to the XCDs, so
  // workgroup b runs on XCD b % NXCD.  Each XCD takes vsplit / NXCD partial
  // slots z = xcd, xcd + NXCD, ... (a block of consecutive v ranges, below)
  // for every tile, and walks the tiles in bands of BAND R blocks, P block by P
  // block: the workgroups resident on one XCD at a time share the U_v and A_v
  // panels through that XCD's L2.
  const int nb = (f.naux + TD - 1) / TD, tiles = nb * nb;
  const int b = blockIdx.x;
  const int xcd = b % NXCD, local = b / NXCD;
  const int z = xcd + NXCD * (local / tiles);
  const int to = local % tiles;
  const int rb0 = to / (BAND * nb) * BAND, bh = min(BAND, nb - rb0);
  const int within = to - rb0 * nb;
  const int P0 = __builtin_amdgcn_readfirstlane((within / bh) * TD);
  const int R0 = __builtin_amdgcn_readfirstlane((rb0 + within % bh) * TD);
  // symmetric D: a tile wholly below the diagonal is the mirror of one above it
  const int set = blockIdx.y;
  if (f.sym != nullptr && f.sym[set] != 0 && R0 >= P0 + TD) return;
  // The last block of columns or rows forms only the 32-wide strips that hold a THC point,
  // and a diagonal tile of a symmetric D only its upper triangle: 1.88 -> 1.70 ms at n = 200,
  // naux = 1100 (12 of the last 64)
  const bool one_p = f.naux - P0 <= 32, one_r = f.naux - R0 <= 32;
  const bool diag = f.sym != nullptr && f.sym[set] != 0 && R0 == P0;
  if (one_r && one_p) fused_f64_tile<1, 1, false>(f, b0, b1, set, z, R0, P0);
  else if (one_p) fused_f64_tile<2, 1, false>(f, b0, b1, set, z, R0, P0);
  else if (one_r) fused_f64_tile<1, 2, false>(f, b0, b1, set, z, R0, P0);
  else if (diag) fused_f64_tile<2, 2, true>(f, b0, b1, set, z, R0, P0);
  else fused_f64_tile<2, 2, false>(f, b0, b1, set, z, R0, P0);
}

inline unsigned cdiv(int64_t a, int64_t b) { return (unsigned)((a + b - 1) / b); }

}  // namespace

void fused_tile(int mode, int* rows, int* cols) {
  switch (mode) {
    case MODE_F64: *rows = *cols = TD; break;
    default: fused_f16_tile(rows, cols); break;   // FP32, fp16x2 and bf16x3: 128 x 128
  }
}

int fused_xcds() { return NXCD; }

hipError_t sox_fused(int mode, const FusedArgs& f, hipStream_t s) {
  if (mode == MODE_F16X2 || mode == MODE_F32) return sox_fused_pairs(mode, f, s);   // own checks
  if (mode == MODE_BF16X3) return sox_fused_bf3(f, s);
  if (mode != MODE_F64 || f.vsplit % NXCD != 0 || (int64_t)f.vsplit * f.vchunk < f.n ||
      f.dpart_f32 || f.ldk % DK != 0 || f.ldk < f.n)
    return hipErrorInvalidValue;
  // buffer offsets inside one tile's rows of U are 32-bit
  if ((int64_t)TD * f.n * f.ldk * 8 > 0x7fffffffLL) return hipErrorInvalidValue;
  const dim3 grid(cdiv(f.naux, TD) * cdiv(f.naux, TD) * f.vsplit, f.nsets);
  fused_f64_kernel<<<grid, NT, 0, s>>>(f);
  return hipGetLastError();
}

}  // namespace thcsox
