// The fused B/C/D stage in the bf16x3 mode, 128 x 128 tiles of D per workgroup:
//
//   D_PR = sum_v C_RvP B_PRv,   B_PRv = sum_q G_Rq A_Pqv,   C_RvP = sum_w U_Rvw G_wP
//
// Every operand is split into three bf16 planes x = x0 + x1 + x2 (about the 24
// bits of an FP32 significand; bf16 keeps FP32's exponent range, so A needs no
// scale); a product is formed from the six plane products x0 y2 + x1 y1 + x2 y0
// + x0 y1 + x1 y0 + x0 y0 on the bf16 matrix cores (16x16x32, FP32
// accumulation).  The operands are K-major rows, one array per plane.
//
// Work split.  A workgroup owns a 128 x 128 tile of D and a range of v, one v at
// a time.  Four waves (one per SIMD) in a 2 x 2 arrangement each own 64 x 64 of
// the tile (16 x 16 tiles alternating between the waves of a row and of a column): the
// accumulators of B and C (128 registers) live in the matrix-core
// registers (AGPRs), the partial sum of D (FP32, at most 8 v) and the fragments of the
// three planes in the ordinary ones.  D is updated once per v: D += B o C.  (The fp16x2
// kernel takes two v per pass: two planes of two v there, three planes of one v here.)
//
// Pipeline: that of the fp16x2 kernel.  A k chunk is two phases, B (G, A_v) and C (GX,
// U_v), each of which reads a half stage of two panels of 128 rows x 32 k x 3 planes (48
// KiB; a plane of a panel is 128 rows of 64 bytes, each row's four 16-byte chunks placed
// by lds_chunk).  LDS holds three half stages and 16 KiB through which D goes to memory.
// A phase forms its 4 x 4 tiles in four steps, a column (B) or a row (C) of them each; the
// fragments of G or GX are read for the whole phase, those of A or U one step ahead.
// Before the last step of a phase every wave waits for the next half stage and at the
// workgroup barrier, then reads that step's fragments of the next phase and begins to
// load the half stage after the next two into the buffer that the barrier set free: a
// load has two phases to land.  n = 120, naux = 600: 181 -> 146 us a tau point against
// two buffers with D in LDS and loads one phase ahead.  The first chunk of a v starts the
// accumulators from zero inside the MFMA.  Past the last chunk the loads repeat it
// (never used).  The compiler keeps 635 scalar values of the 14 tile forms in lanes of
// vector registers (67 with one form).
#include <type_traits>

#include "dtile.hpp"
#include "kernels.hpp"
#include "mfma.hpp"
#include "panel.hpp"

namespace thcsox {
namespace {

constexpr int NW = 4, NTH = 64 * NW;
constexpr int KC = 32;           // k per chunk (one bf16 MFMA)
constexpr int NPL = 3;           // bf16 planes
constexpr int PP = TT * KC;      // elements of one plane of a panel
constexpr int FLUSH_V = 8;       // v per FP32 partial sum of D
constexpr int NXCD = 8;

// One half stage: panel 0 is the v-independent operand (G or GX), panel 1 the
// per-v one (A_v or U_v); [panel][plane][row * 32 + k].
constexpr int HALF3 = 2 * NPL * PP;   // elements
struct Smem3 {
  __bf16 st[3 * HALF3];   // the half stages of three phases
  float d[32 * TT];       // 32 rows of D on their way to memory
};

// One tile's range of v.  Each wave forms TI x TJ tiles of 16 x 16 out of its 4 x 4: the rows R of the workgroup's tile
// beyond 32 TI and the columns P beyond 32 TJ lie past naux and are neither loaded nor
// multiplied.  TRI: a diagonal tile of a symmetric D, of which only the 16 x 16 tiles ti
// <= tj of each wave are formed: they hold every element on and above the diagonal.  (A
// D element's products and their order do not depend on TI, TJ and TRI.)
template <int TI, int TJ, bool TRI>
__device__ __forceinline__ void fused_bf3_tile(const FusedArgs& f, Smem3& sm, int set, int z, int R0,
                                               int P0) {
  int tid = threadIdx.x;
  // (the compiler must not merge the forms' address arithmetic above their branch)
  __asm__ volatile("" : "+v"(tid));
  __asm__ volatile("" : "+s"(set));
  __asm__ volatile("" : "+s"(z));
  __asm__ volatile("" : "+s"(R0));
  __asm__ volatile("" : "+s"(P0));
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wr = wave >> 1, wc = wave & 1;
  const int naux = f.naux, n = f.n, ldk = f.ldk;

  // v range: XCD x owns the consecutive ranges x q .. x q + q - 1 (q = vsplit /
  // 8); range r is v in [r n / vsplit, (r + 1) n / vsplit)
  const int vr = (z % NXCD) * (f.vsplit / NXCD) + z / NXCD;
  const int v_lo = __builtin_amdgcn_readfirstlane((int)((int64_t)vr * n / f.vsplit));
  const int v_hi = __builtin_amdgcn_readfirstlane((int)((int64_t)(vr + 1) * n / f.vsplit));
  const int nv = v_hi - v_lo;
  const int kst = ldk / KC;
  const int rows_r = min(TT, naux - R0), rows_p = min(TT, naux - P0);

  // operands, plane 0 (rows past the valid range lie beyond the buffer resources and read
  // as zero; byte counts below 2^31: checked by the launcher)
  const __bf16* Gt = static_cast<const __bf16*>(f.Gt) + set * f.g_set + (int64_t)R0 * ldk;
  const __bf16* GX = static_cast<const __bf16*>(f.GXt) + set * f.g_set + (int64_t)P0 * ldk;
  const __bf16* Ub = static_cast<const __bf16*>(f.U) + (int64_t)R0 * n * ldk;
  const __bf16* Ab = static_cast<const __bf16*>(f.A) + set * f.a_set + (int64_t)P0 * ldk;
  const int r_bytes = rows_r * ldk * 2, p_bytes = rows_p * ldk * 2;
  const int u_bytes = ((rows_r - 1) * n * ldk + ldk) * 2;

  // memory -> LDS: one instruction moves 16 rows x 64 bytes of one plane; wave w
  // moves the 16-row slabs w and w + 4 of each plane of each panel.  Lane l
  // lands at slab row l / 4, physical chunk l % 4, and loads the logical chunk
  // lds_chunk maps there (the map is its own inverse for a given row).
  const int drow = wave * 16 + (lane >> 2), dch = 8 * lds_chunk(drow, lane & 3);
  uint32_t dR = (uint32_t)((drow * ldk + dch) * 2), dU = (uint32_t)((drow * (n * ldk) + dch) * 2);
  const uint32_t sR = 64 * ldk * 2, sU = sR * n;   // 64 rows further (the same chunks)
  // fetch cursors (v, k chunk) of the two kinds of half stages, clamped to the last chunk
  // (no branch: one would keep a phase's loads and MFMAs apart)
  int vB = 0, kB = 0, vC = 0, kC = 0;
  auto next = [&](int& v, int& k) {
    const bool wrap = k == kst - 1, last = wrap && v == nv - 1;
    k = last ? k : (wrap ? 0 : k + 1);
    v += wrap && !last ? 1 : 0;
  };
  // loads q of a half stage into the buffer at sm.st + buf: the slabs of the panel of rows
  // and of the panel of columns, three planes each
  constexpr int LR = NPL * (TI > 2 ? 2 : 1), LP = NPL * (TJ > 2 ? 2 : 1), NL = LR + LP;
  auto dst = [&](int buf, int panel, int p, int j) {
    return lds_addr(sm.st) + (uint32_t)(buf + (panel * NPL + p) * PP + (wave + NW * j) * 16 * 32) * 2;
  };
  auto dmaB = [&](int q, int buf) {
    const int so = kB * KC * 2, p = q % NPL;   // bytes to the k chunk; plane
    if (q < LR) {
      const int j = q / NPL;
      dma16_untracked(raw_rsrc(Gt + p * f.g_plane, r_bytes), dst(buf, 0, p, j), dR + j * sR, so);
    } else {
      const int j = (q - LR) / NPL;
      dma16_untracked(raw_rsrc(Ab + p * f.a_plane + (int64_t)(v_lo + vB) * naux * ldk, p_bytes),
                      dst(buf, 1, p, j), dR + j * sR, so);
    }
  };
  auto dmaC = [&](int q, int buf) {
    const int so = kC * KC * 2, p = q % NPL;
    if (q < LP) {
      const int j = q / NPL;
      dma16_untracked(raw_rsrc(GX + p * f.g_plane, p_bytes), dst(buf, 0, p, j), dR + j * sR, so);
    } else {
      const int j = (q - LP) / NPL;
      dma16_untracked(raw_rsrc(Ub + p * f.u_plane + (int64_t)(v_lo + vC) * ldk, u_bytes),
                      dst(buf, 1, p, j), dU + j * sU, so);
    }
  };

  // fragment (row r, k chunk lane / 16) of a plane at r * 32 + lds_chunk(r, lane / 16) * 8.
  // The 16 x 16 tiles alternate between the two waves of a row or column, so both work in
  // a short tile; the map repeats every 32 rows, so tile t is 32 t rows further.
  const int lr = lane & 15, kc = lane >> 4;
  const int oR = (wr * 16 + lr) * 32 + lds_chunk(wr * 16 + lr, kc) * 8;   // R side rows
  const int oP = (wc * 16 + lr) * 32 + lds_chunk(wc * 16 + lr, kc) * 8;   // P side rows
  // fragments: G and GX of a whole phase [plane][tile]; A and U of one tile column or row at
  // a time, [step parity][plane]
  bf16x8 gs[NPL][TI], xs[NPL][TJ], ma[2][NPL], mu[2][NPL];
  auto rd = [&](int buf, int panel, int p, int off, int t) {
    return *reinterpret_cast<const bf16x8*>(sm.st + buf + (panel * NPL + p) * PP + off + t * 32 * 32);
  };
  // reads q of what a step takes and, from q = 3 on, of what a phase takes
  auto readB = [&](int q, int buf, int par, int t) {
    if (q < NPL) ma[par][q] = rd(buf, 1, q, oP, t);
    else gs[q % NPL][q / NPL - 1] = rd(buf, 0, q % NPL, oR, q / NPL - 1);
  };
  auto readC = [&](int q, int buf, int par, int t) {
    if (q < NPL) mu[par][q] = rd(buf, 1, q, oR, t);
    else xs[q % NPL][q / NPL - 1] = rd(buf, 0, q % NPL, oP, q / NPL - 1);
  };

  // accumulators [ti][tj]: rows R of tile ti, columns P of tile tj (each v starts them
  // from zero inside its first MFMAs), and the partial sum of D
  f4 B[TI][TJ], C[TI][TJ], D[TI][TJ];
  const f4 zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int ti = 0; ti < TI; ++ti)
#pragma unroll
    for (int tj = TRI ? ti : 0; tj < TJ; ++tj) B[ti][tj] = C[ti][tj] = D[ti][tj] = zero;
  using PR = Products<NPL>;   // plane pairs, smallest terms first
  // B products: B[ti][tj] += G[ti] . A_v[tj]
  auto mfmaB = [&](int ti, int tj, int par, bool first) {
    f4 a = first ? zero : B[ti][tj];
#pragma unroll
    for (int q = 0; q < PR::N; ++q)
      a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(gs[PR::a(q)][ti], ma[par][PR::b(q)], a, 0, 0, 0);
    B[ti][tj] = a;
  };
  // C products: C[ti][tj] += U_v[ti] . GX[tj]
  auto mfmaC = [&](int ti, int tj, int par, bool first) {
    f4 a = first ? zero : C[ti][tj];
#pragma unroll
    for (int q = 0; q < PR::N; ++q)
      a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(mu[par][PR::a(q)], xs[PR::b(q)][tj], a, 0, 0, 0);
    C[ti][tj] = a;
  };
  auto dupdate = [&](int ti, int tj) {
#pragma unroll
    for (int r = 0; r < 4; ++r) D[ti][tj][r] = fmaf(B[ti][tj][r], C[ti][tj][r], D[ti][tj][r]);
  };

  // A phase's steps: B takes the columns tj one by one, C the rows ti (a triangle from its
  // short end, so that the last step, which has the most reads, is the longest).  share:
  // what slots 0 .. s - 1 of S do of n items.
  auto row_of = [](int i) { return TRI ? TI - 1 - i : i; };
  auto share = [](int n_items, int s, int S) { return s * n_items / S; };
  int b0 = 0, b1 = HALF3, b2 = 2 * HALF3;   // buffers of B(t), C(t), B(t+1)
  auto chunk = [&](auto first_c, auto last_c) {
    constexpr bool first = decltype(first_c)::value, last = decltype(last_c)::value;
    // (the offsets of the other rows are formed here, not kept in registers over the loops)
    __asm__ volatile("" : "+v"(dR));
    __asm__ volatile("" : "+v"(dU));
#pragma unroll
    for (int i = 0; i < TJ; ++i) {
      const bool end = i == TJ - 1;
      if (end) {   // C(t) has landed, every wave has read B(t)
        vm_lds_barrier<NL>();
        next(vC, kC);
      }
      const int tiles = TRI ? i + 1 : TI;
      const int reads = end ? NPL + NPL * TJ : NPL, pace = (reads + max(tiles - 1, 1) - 1) / max(tiles - 1, 1);
      const int q0 = end ? 0 : share(NL, i + 1, TJ), q1 = end ? share(NL, 1, TI) : share(NL, i + 2, TJ);
#pragma unroll
      for (int u = 0; u < tiles; ++u) {
#pragma unroll
        for (int q = u * pace; q < min((u + 1) * pace, reads); ++q) {
          if (end) readC(q, b1, 0, row_of(0));
          else readB(q, b0, (i + 1) % 2, i + 1);
        }
#pragma unroll
        for (int q = q0 + share(q1 - q0, u, tiles); q < q0 + share(q1 - q0, u + 1, tiles); ++q) {
          if (end) dmaC(q, b0);
          else dmaB(q, b2);
        }
        mfmaB(u, i, i % 2, first);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
#pragma unroll
    for (int i = 0; i < TI; ++i) {
      const bool end = i == TI - 1;
      if (end) {   // B(t+1) has landed, every wave has read C(t)
        vm_lds_barrier<NL>();
        next(vB, kB);
      }
      const int ti = row_of(i), tj0 = TRI ? ti : 0, tiles = TJ - tj0;
      const int reads = end ? NPL + NPL * TI : NPL, pace = (reads + max(tiles - 1, 1) - 1) / max(tiles - 1, 1);
      const int q0 = end ? 0 : share(NL, i + 1, TI), q1 = end ? share(NL, 1, TJ) : share(NL, i + 2, TI);
#pragma unroll
      for (int u = 0; u < tiles; ++u) {
#pragma unroll
        for (int q = u * pace; q < min((u + 1) * pace, reads); ++q) {
          if (end) readB(q, b2, 0, 0);
          else readC(q, b1, (i + 1) % 2, row_of(i + 1));
        }
#pragma unroll
        for (int q = q0 + share(q1 - q0, u, tiles); q < q0 + share(q1 - q0, u + 1, tiles); ++q) {
          if (end) dmaB(q, b1);
          else dmaC(q, b0);
        }
        mfmaC(ti, tj0 + u, i % 2, first);
        if (last && i > 0) {   // D of the row before
          const int tb = row_of(i - 1), t0 = TRI ? tb : 0;
#pragma unroll
          for (int tj = 0; tj < TJ; ++tj)
            if (tj >= t0 && (tj - t0) * tiles / (TJ - t0) == u) dupdate(tb, tj);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if (last) {
      const int tb = row_of(TI - 1);
#pragma unroll
      for (int tj = TRI ? tb : 0; tj < TJ; ++tj) dupdate(tb, tj);
    }
    const int b = b2;
    b2 = b1;
    b1 = b0;
    b0 = b;
  };

  if (nv > 0) {
#pragma unroll
    for (int q = 0; q < NL; ++q) dmaB(q, b0);
#pragma unroll
    for (int q = 0; q < NL; ++q) dmaC(q, b1);
    next(vB, kB);
    constexpr int SLOT = NL / TJ;   // share(NL, 1, TJ)
#pragma unroll
    for (int q = 0; q < SLOT; ++q) dmaB(q, b2);
    vm_lds_barrier<NL + SLOT>();
#pragma unroll
    for (int q = 0; q < NPL + NPL * TI; ++q) readB(q, b0, 0, 0);
  }
  const std::true_type yes;
  const std::false_type no;
  int iv = 0;
  do {
    if (nv > 0) {
      if (kst == 1) {
        chunk(yes, yes);
      } else {
        chunk(yes, no);
        for (int k = 2; k < kst; ++k) chunk(no, no);
        chunk(no, yes);
      }
      ++iv;
    }
    // (an empty range writes zeros)
    if (iv == nv || iv % FLUSH_V == 0)
      store_d<TI, TJ, TRI>(D, sm.d, f, set, z, R0, P0, wave, iv <= FLUSH_V);
  } while (iv < nv);
  // the last (repeated) memory-to-LDS loads land before the workgroup may end
  __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

__global__ __launch_bounds__(NTH) __attribute__((amdgpu_waves_per_eu(1, 1)))
void fused_bf3_kernel(FusedArgs f) {
  __shared__ __attribute__((aligned(16))) Smem3 sm;
  const int naux = f.naux;

  // tile and v range: XCD-aware order (workgroup b runs on XCD b mod 8; each XCD
  // owns the partial slots z = xcd, xcd + 8, ..., a block of consecutive v
  // ranges, and walks the tiles of one slot in bands of two R blocks, P by P
  // with R fastest, so its resident workgroups share panels in its L2).  With
  // symmetric D only the tiles on or above the diagonal are walked.  The integer
  // divisions run on the vector unit; readfirstlane marks their results uniform.
  const int nb = (naux + TT - 1) / TT;
  const int set = blockIdx.y;
  const bool symm = f.sym != nullptr && f.sym[set] != 0;
  const int ntl = symm ? nb * (nb + 1) / 2 : nb * nb;
  const int b = blockIdx.x;
  const int xcd = b % NXCD, local = b / NXCD;
  if (local >= ntl * (f.vsplit / NXCD)) return;
  const int z = __builtin_amdgcn_readfirstlane(xcd + NXCD * (local / ntl));
  int t = local % ntl, r0 = 0;
  for (;;) {   // the band of rows r0, r0 + 1 (one row at the end when nb is odd)
    const int rows = min(2, nb - r0);
    const int cnt = symm ? (rows == 2 ? 2 * (nb - r0) - 1 : nb - r0) : rows * nb;
    if (t < cnt) break;
    t -= cnt;
    r0 += 2;
  }
  int rb, pb;
  if (symm) {   // (r0, r0), then (r0, p), (r0 + 1, p) for p > r0
    rb = t == 0 ? r0 : r0 + (t - 1) % 2;
    pb = t == 0 ? r0 : r0 + 1 + (t - 1) / 2;
  } else {
    const int rows = min(2, nb - r0);
    rb = r0 + t % rows;
    pb = t / rows;
  }
  const int P0 = __builtin_amdgcn_readfirstlane(pb * TT);
  const int R0 = __builtin_amdgcn_readfirstlane(rb * TT);

  // The last block of naux % 128 columns or rows forms only the 32-wide strips that hold a
  // THC point, and a diagonal tile of a symmetric D only its upper triangle: 190 -> 181 us a
  // tau point at n = 120, naux = 600 (88 of the last 128), general
  const int tj = min((naux - P0 + 31) / 32, 4), ti = min((naux - R0 + 31) / 32, 4);
  const bool diag = symm && R0 == P0;
#define THCSOX_TILE(TI, TJ, TRI) fused_bf3_tile<TI, TJ, TRI>(f, sm, set, z, R0, P0)
  if (diag) {
    if (tj == 4) THCSOX_TILE(4, 4, true);
    else if (tj == 3) THCSOX_TILE(3, 3, true);
    else if (tj == 2) THCSOX_TILE(2, 2, true);
    else THCSOX_TILE(1, 1, true);
  } else if (ti == 4) {
    if (tj == 4) THCSOX_TILE(4, 4, false);
    else if (tj == 3) THCSOX_TILE(4, 3, false);
    else if (tj == 2) THCSOX_TILE(4, 2, false);
    else THCSOX_TILE(4, 1, false);
  } else if (tj == 4) {
    if (ti == 3) THCSOX_TILE(3, 4, false);
    else if (ti == 2) THCSOX_TILE(2, 4, false);
    else THCSOX_TILE(1, 4, false);
  } else {   // the corner of a general D
    if (ti == 3) THCSOX_TILE(3, 3, false);
    else if (ti == 2) THCSOX_TILE(2, 2, false);
    else THCSOX_TILE(1, 1, false);
  }
#undef THCSOX_TILE
}

inline unsigned cdiv_bf3(int64_t a, int64_t b) { return (unsigned)((a + b - 1) / b); }

}  // namespace

hipError_t sox_fused_bf3(const FusedArgs& f, hipStream_t s) {
  const int vmax = (f.n + f.vsplit - 1) / f.vsplit;   // longest v range
  if (f.vsplit % NXCD != 0 || f.ldk % KC != 0 || f.ldk < f.n ||
      (f.dpart_f32 && vmax > FLUSH_V))
    return hipErrorInvalidValue;
  // buffer offsets inside one tile's rows of U (rows of 2 ldk bytes) are 32-bit
  if ((int64_t)TT * f.n * f.ldk * 2 > 0x7fffffffLL) return hipErrorInvalidValue;
  const unsigned nb = cdiv_bf3(f.naux, TT);
  fused_bf3_kernel<<<dim3(nb * nb * f.vsplit, f.nsets), NTH, 0, s>>>(f);
  return hipGetLastError();
}

}  // namespace thcsox
