// The fused B/C/D stage in the fp16x2 and FP32 modes, 128 x 128 tiles of D per
// workgroup:
//
//   D_PR = sum_v C_RvP B_PRv,   B_PRv = sum_q G_Rq A_Pqv,   C_RvP = sum_w U_Rvw G_wP
//
// fp16x2: every operand is a power-of-two scaled value split into two fp16
// planes x = x0 + x1; a product is formed from the plane products x1 y0 + x0 y1
// + x0 y0 on the f16 matrix cores (16x16x32, FP32 accumulation).  The operands
// are K-major rows with the two planes interleaved per 32-wide k chunk (layout
// c32: row r, plane p, k at r * 2 ldk + (k / 32) * 64 + 32 p + k % 32), so one
// 128-byte request fetches both planes of a row's chunk.  FP32: plain K-major
// FP32 rows, whose 32-wide k chunks are 128 bytes too, so both modes share the
// loads, the LDS layout and the schedule below; a chunk is eight 16x16x4 FP32
// MFMAs per tile instead of three 16x16x32 f16 ones.
//
// Work split.  A workgroup owns a 128 x 128 tile of D and a range of v, taken
// two v at a time: the k loop of a pair forms B and C for both v at once, so
// the v-independent panels (G rows R, GX rows P) are loaded once per pair and
// feed four products.  Four waves (one per SIMD) in a 2 x 2 arrangement each
// own 64 x 64 of the tile (16 x 16 tiles alternating between the waves of a row and
// of a column): the four accumulator sets B1, B2, C1, C2 (256
// registers) live in the matrix-core registers (AGPRs); the partial sum of D (FP32, at
// most 8 v) and the fragments in the ordinary ones.  D is updated once per pair, row
// by row among the last products: D += B1 o C1 + B2 o C2.
//
// Pipeline.  A k chunk is two phases, B and C, each of which reads a half stage of three
// panels of 128 rows x 32 k x 2 planes (FP32: one plane of 4-byte elements; 48 KiB either
// way): G, A_v1, A_v2, then GX, U_v1, U_v2.  LDS holds three of them (144 KiB; the other 16
// take D to memory).  A phase forms its 4 x 4 tiles in four steps, a column (B) or a row
// (C) of them each: the fragments of G or GX are read for the whole phase, those of A or U
// one step ahead.  Before the last step of a phase every wave waits for the next half
// stage and at the workgroup barrier, then reads that step's fragments of the next phase
// and begins to load the half stage after the next two into the buffer that the barrier
// set free.  So a load has two phases to land.
//
// What bounds it: the matrix cores run 0.65 of the time; the rest is the LDS writes of the
// loads and the fragment reads that one wave per SIMD hides only in part (n = 300, naux =
// 1800, a pair of v of a full tile: 21.3 us; 19.9 with loads that always hit the L2, 16.8
// without the loads, 13.8 without the reads either).  The L2 misses come at a plain copy's
// rate (7.7 GB a tau point in 1.65 ms).  Two buffers with D in LDS, loads one phase ahead and
// fragments read a phase ahead (which spilled) took 25.8, and its 64 single-word stores a
// thread 8.6 instead of 3.4 us a tile.  Whole launches: n = 300, symmetric, fp16x2 1.83 ->
// 1.62 ms a tau point; n = 97, naux = 485 30.2 -> 24.0 us; n = 149, naux = 797, general,
// FP32 590 -> 555 us.  The loads are issued in inline assembly: tracked ones would make the
// compiler wait before it reads another part of LDS.  The first chunk of a pair starts the
// accumulators from zero inside the MFMA (no register clearing).  Past the last chunk the
// loads repeat it (never used).  The compiler keeps 257 scalar values of the 14 tile forms
// in lanes of vector registers (FP32: 217, and 9 vector registers in scratch).
#include <type_traits>

#include "dtile.hpp"
#include "kernels.hpp"
#include "mfma.hpp"
#include "panel.hpp"

namespace thcsox {
namespace {

constexpr int NW = 4, NTH = 64 * NW;
constexpr int KC = 32;           // k per chunk (one f16 MFMA)
constexpr int PANEL = TT * KC * 2;   // halves per panel (both planes)
constexpr int FLUSH_PAIRS = 4;   // pairs per FP32 partial sum of D (8 v)
constexpr int NXCD16 = 8;

// One half stage: three panels, each [row][plane][32] (128-byte rows) with the
// eight 16-byte chunks of a row permuted by sw8.
constexpr int HALF = 3 * PANEL;   // halves
struct Smem {
  _Float16 st[3 * HALF];   // the half stages of three phases
  float d[32 * TT];        // 32 rows of D on their way to memory
};

// Physical 16-byte chunk of logical chunk c (= 4 plane + k / 8) in LDS row r.
// Fragment reads take 16 consecutive rows at one logical chunk; XOR-ing the
// chunk with (r / 2) mod 8 places the 16 rows' chunks at all eight positions of
// two consecutive 128-byte rows (rocprofv3 counts no LDS bank conflicts).
__device__ __forceinline__ int sw8(int r, int c) { return c ^ ((r >> 1) & 7); }

// One tile's range of pairs.  M = MODE_F16X2 or MODE_F32.  Each wave forms TI x TJ tiles of 16 x 16 out of its 4 x 4: the
// rows R of the workgroup's tile beyond 32 TI and the columns P beyond 32 TJ lie past
// naux and are neither loaded nor multiplied.  TRI: a diagonal tile of a symmetric D, of
// which only the 16 x 16 tiles ti <= tj of each wave are formed: they hold every element
// on and above the diagonal.  (A D element's products and their order do not depend on
// TI, TJ and TRI.)
template <int M, int TI, int TJ, bool TRI>
__device__ __forceinline__ void fused_tile(const FusedArgs& f, Smem& sm, int set, int z, int R0,
                                           int P0) {
  constexpr bool F32 = M == MODE_F32;
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

  // pair range: XCD x owns the consecutive ranges x q .. x q + q - 1
  // (q = vsplit / 8); range r is pairs [r np / vsplit, (r + 1) np / vsplit)
  const int npair = (n + 1) / 2;
  const int vr = (z % NXCD16) * (f.vsplit / NXCD16) + z / NXCD16;
  const int p_lo = __builtin_amdgcn_readfirstlane((int)((int64_t)vr * npair / f.vsplit));
  const int p_hi = __builtin_amdgcn_readfirstlane((int)((int64_t)(vr + 1) * npair / f.vsplit));
  const int npr = p_hi - p_lo;
  const int kst = (n + KC - 1) / KC;   // chunks with any k < n (rows are zero from n to ldk)
  const int ld2 = 2 * ldk;   // halves per c32 row
  const int rows_r = min(TT, naux - R0), rows_p = min(TT, naux - P0);

  const _Float16* Gt = static_cast<const _Float16*>(f.Gt) + set * f.g_set;
  const _Float16* GX = static_cast<const _Float16*>(f.GXt) + set * f.g_set;
  // (byte counts below 2^31: checked by the launcher)
  const i4 rG = raw_rsrc(Gt + (int64_t)R0 * ld2, rows_r * ld2 * 2);
  const i4 rX = raw_rsrc(GX + (int64_t)P0 * ld2, rows_p * ld2 * 2);
  const _Float16* Ubase = static_cast<const _Float16*>(f.U) + (int64_t)R0 * n * ld2;
  const _Float16* Abase = static_cast<const _Float16*>(f.A) + set * f.a_set + (int64_t)P0 * ld2;
  const int64_t a_v = (int64_t)naux * ld2;   // halves between v slabs of A

  // memory -> LDS: one instruction moves 8 rows x 128 bytes; wave w moves the
  // 8-row slabs w, w + 4, w + 8, w + 12 of each panel.  Lane l lands at slab row
  // l / 8, physical chunk l % 8, and loads the logical chunk sw8 maps there.
  // Rows past the valid range lie beyond the buffer resource and read as zero.
  const int drow = wave * 8 + (lane >> 3), dch = 8 * sw8(drow, lane & 7);
  uint32_t dR = (uint32_t)((drow * ld2 + dch) * 2), dU = (uint32_t)((drow * (n * ld2) + dch) * 2);
  const uint32_t sR = 32 * ld2 * 2, sU = sR * n;   // 32 rows further (the same chunks)
  // fetch cursors (pair, k chunk) of the two kinds of half stages, clamped to the last
  // chunk, and the resources of their pairs: A slabs v1, v2 (rows P) and U rows (R, v1),
  // (R, v2); a missing second v (odd n) gets empty resources, so its panels read as zero
  // and B2 = 0
  i4 rA1, rA2, rU1, rU2;
  const int a_bytes = rows_p * ld2 * 2;
  const int u_bytes = ((rows_r - 1) * n * ld2 + ld2) * 2;
  int pB = 0, kB = 0, pC = 0, kC = 0;
  auto set_b = [&]() {
    const int v1 = 2 * (p_lo + pB);
    rA1 = raw_rsrc(Abase + (int64_t)v1 * a_v, a_bytes);
    rA2 = raw_rsrc(Abase + (int64_t)(v1 + 1) * a_v, v1 + 1 < n ? a_bytes : 0);
  };
  auto set_c = [&]() {
    const int v1 = 2 * (p_lo + pC);
    rU1 = raw_rsrc(Ubase + (int64_t)v1 * ld2, u_bytes);
    rU2 = raw_rsrc(Ubase + (int64_t)(v1 + 1) * ld2, v1 + 1 < n ? u_bytes : 0);
  };
  // (no branch: one would keep a phase's loads and MFMAs apart)
  auto next = [&](int& pr, int& k) {
    const bool wrap = k == kst - 1, last = wrap && pr == npr - 1;
    k = last ? k : (wrap ? 0 : k + 1);
    pr += wrap && !last ? 1 : 0;
  };
  // loads q of a half stage into the buffer at sm.st + buf
  constexpr int NB = TI + 2 * TJ, NC = TJ + 2 * TI;   // loads of a B and a C half per wave
  auto dst = [&](int buf, int panel, int j) {
    return lds_addr(sm.st) + (uint32_t)(buf + panel * PANEL + (wave + NW * j) * 8 * 64) * 2;
  };
  auto dmaB = [&](int q, int buf) {
    const int so = kB * KC * 4;   // bytes to the k chunk (both planes)
    if (q < TI) dma16_untracked(rG, dst(buf, 0, q), dR + q * sR, so);
    else if ((q - TI) % 2 == 0) dma16_untracked(rA1, dst(buf, 1, (q - TI) / 2), dR + (q - TI) / 2 * sR, so);
    else dma16_untracked(rA2, dst(buf, 2, (q - TI) / 2), dR + (q - TI) / 2 * sR, so);
  };
  auto dmaC = [&](int q, int buf) {
    const int so = kC * KC * 4;
    if (q < TJ) dma16_untracked(rX, dst(buf, 0, q), dR + q * sR, so);
    else if ((q - TJ) % 2 == 0) dma16_untracked(rU1, dst(buf, 1, (q - TJ) / 2), dU + (q - TJ) / 2 * sU, so);
    else dma16_untracked(rU2, dst(buf, 2, (q - TJ) / 2), dU + (q - TJ) / 2 * sU, so);
  };

  // fp16x2: fragment (row r, plane p, k chunk lane / 16) at halves r * 64 + sw8(r, 4 p +
  // lane / 16) * 8.  FP32: the 16x16x4 MFMA takes one k per lane group, and any
  // assignment of the chunk's 32 k to its eight MFMAs j and four lane groups serves
  // when both operands use it: lane group g takes k = 8 g + j, two 16-byte reads
  // at logical chunks 2 g and 2 g + 1 (in "planes" 0 and 1 below).  sw8 depends on
  // r mod 16 only, so the rows of tile t are 32 t * 64 halves further (the tiles of
  // the two waves of a row or column alternate, so both waves work in a short tile).
  const int lr = lane & 15, kc = lane >> 4;
  const int rr = wr * 16 + lr, rc = wc * 16 + lr;
  const int c0 = F32 ? 2 * kc : kc, c1 = F32 ? 2 * kc + 1 : 4 + kc;
  const int oR[2] = {rr * 64 + sw8(rr, c0) * 8, rr * 64 + sw8(rr, c1) * 8};
  const int oP[2] = {rc * 64 + sw8(rc, c0) * 8, rc * 64 + sw8(rc, c1) * 8};
  // fragments: G and GX of a whole phase [plane][tile]; of A and U the two v of one tile
  // column or row at a time, [step parity][2 v + plane]
  f16x8 gs[2][TI], xs[2][TJ], ma[2][4], mu[2][4];
  auto rd = [&](int buf, int panel, int off, int t) {
    return *reinterpret_cast<const f16x8*>(sm.st + buf + panel * PANEL + off + t * 32 * 64);
  };
  // reads q of what a step takes (m) and, from q = 4 on, of what a phase takes (s)
  auto readB = [&](int q, int buf, int par, int t) {
    if (q < 4) ma[par][q] = rd(buf, 1 + q / 2, oP[q % 2], t);
    else gs[q % 2][(q - 4) / 2] = rd(buf, 0, oR[q % 2], (q - 4) / 2);
  };
  auto readC = [&](int q, int buf, int par, int t) {
    if (q < 4) mu[par][q] = rd(buf, 1 + q / 2, oR[q % 2], t);
    else xs[q % 2][(q - 4) / 2] = rd(buf, 0, oP[q % 2], (q - 4) / 2);
  };

  // accumulators [ti][tj]: rows R of tile ti, columns P of tile tj (each pair starts them
  // from zero inside its first MFMAs), and the partial sum of D
  f4 B1[TI][TJ], B2[TI][TJ], C1[TI][TJ], C2[TI][TJ], D[TI][TJ];
  const f4 zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int ti = 0; ti < TI; ++ti)
#pragma unroll
    for (int tj = TRI ? ti : 0; tj < TJ; ++tj)
      B1[ti][tj] = B2[ti][tj] = C1[ti][tj] = C2[ti][tj] = D[ti][tj] = zero;
  // FP32: operand j (k = 8 g + j) of a fragment pair
  auto el = [](const f16x8& lo, const f16x8& hi, int j) {
    return j < 4 ? __builtin_bit_cast(f4, lo)[j] : __builtin_bit_cast(f4, hi)[j - 4];
  };
  // B products: acc[ti][tj] += G[ti] . A_m[tj] (fp16x2: planes x1 y0 + x0 y1 + x0 y0;
  // FP32: eight 16x16x4 products, the two v interleaved)
  auto mfmaB = [&](int ti, int tj, int par, bool first) {
    f4 a1 = first ? zero : B1[ti][tj], a2 = first ? zero : B2[ti][tj];
    if constexpr (F32) {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const float g = el(gs[0][ti], gs[1][ti], j);
        a1 = __builtin_amdgcn_mfma_f32_16x16x4f32(g, el(ma[par][0], ma[par][1], j), a1, 0, 0, 0);
        a2 = __builtin_amdgcn_mfma_f32_16x16x4f32(g, el(ma[par][2], ma[par][3], j), a2, 0, 0, 0);
      }
    } else {
      a1 = __builtin_amdgcn_mfma_f32_16x16x32_f16(gs[1][ti], ma[par][0], a1, 0, 0, 0);
      a1 = __builtin_amdgcn_mfma_f32_16x16x32_f16(gs[0][ti], ma[par][1], a1, 0, 0, 0);
      a1 = __builtin_amdgcn_mfma_f32_16x16x32_f16(gs[0][ti], ma[par][0], a1, 0, 0, 0);
      a2 = __builtin_amdgcn_mfma_f32_16x16x32_f16(gs[1][ti], ma[par][2], a2, 0, 0, 0);
      a2 = __builtin_amdgcn_mfma_f32_16x16x32_f16(gs[0][ti], ma[par][3], a2, 0, 0, 0);
      a2 = __builtin_amdgcn_mfma_f32_16x16x32_f16(gs[0][ti], ma[par][2], a2, 0, 0, 0);
    }
    B1[ti][tj] = a1;
    B2[ti][tj] = a2;
  };
  // C products: acc[ti][tj] += U_m[ti] . GX[tj]
  auto mfmaC = [&](int ti, int tj, int par, bool first) {
    f4 a1 = first ? zero : C1[ti][tj], a2 = first ? zero : C2[ti][tj];
    if constexpr (F32) {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const float x = el(xs[0][tj], xs[1][tj], j);
        a1 = __builtin_amdgcn_mfma_f32_16x16x4f32(el(mu[par][0], mu[par][1], j), x, a1, 0, 0, 0);
        a2 = __builtin_amdgcn_mfma_f32_16x16x4f32(el(mu[par][2], mu[par][3], j), x, a2, 0, 0, 0);
      }
    } else {
      a1 = __builtin_amdgcn_mfma_f32_16x16x32_f16(mu[par][1], xs[0][tj], a1, 0, 0, 0);
      a1 = __builtin_amdgcn_mfma_f32_16x16x32_f16(mu[par][0], xs[1][tj], a1, 0, 0, 0);
      a1 = __builtin_amdgcn_mfma_f32_16x16x32_f16(mu[par][0], xs[0][tj], a1, 0, 0, 0);
      a2 = __builtin_amdgcn_mfma_f32_16x16x32_f16(mu[par][3], xs[0][tj], a2, 0, 0, 0);
      a2 = __builtin_amdgcn_mfma_f32_16x16x32_f16(mu[par][2], xs[1][tj], a2, 0, 0, 0);
      a2 = __builtin_amdgcn_mfma_f32_16x16x32_f16(mu[par][2], xs[0][tj], a2, 0, 0, 0);
    }
    C1[ti][tj] = a1;
    C2[ti][tj] = a2;
  };
  auto dupdate = [&](int ti, int tj) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      D[ti][tj][r] = fmaf(B1[ti][tj][r], C1[ti][tj][r], D[ti][tj][r]);
      D[ti][tj][r] = fmaf(B2[ti][tj][r], C2[ti][tj][r], D[ti][tj][r]);
    }
  };

  // A phase's steps: B takes the columns tj one by one, C the rows ti (a triangle from its
  // short end, so that the last step, which has the most reads, is the longest).  share:
  // what slots 0 .. s - 1 of S do of n items.
  auto row_of = [](int i) { return TRI ? TI - 1 - i : i; };
  auto share = [](int n_items, int s, int S) { return s * n_items / S; };
  int b0 = 0, b1 = HALF, b2 = 2 * HALF;   // buffers of B(t), C(t), B(t+1)
  auto chunk = [&](auto first_c, auto last_c) {
    constexpr bool first = decltype(first_c)::value, last = decltype(last_c)::value;
    // (the offsets of the other rows are formed here, not kept in registers over the loops)
    __asm__ volatile("" : "+v"(dR));
    __asm__ volatile("" : "+v"(dU));
#pragma unroll
    for (int i = 0; i < TJ; ++i) {
      const bool end = i == TJ - 1;
      if (end) {   // C(t) has landed, every wave has read B(t)
        vm_lds_barrier<NB>();
        next(pC, kC);
        set_c();
      }
      const int tiles = TRI ? i + 1 : TI;
      const int reads = end ? 4 + 2 * TJ : 4, pace = (reads + max(tiles - 1, 1) - 1) / max(tiles - 1, 1);
      const int q0 = end ? 0 : share(NB, i + 1, TJ), q1 = end ? share(NC, 1, TI) : share(NB, i + 2, TJ);
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
        vm_lds_barrier<NC>();
        next(pB, kB);
        set_b();
      }
      const int ti = row_of(i), tj0 = TRI ? ti : 0, tiles = TJ - tj0;
      const int reads = end ? 4 + 2 * TI : 4, pace = (reads + max(tiles - 1, 1) - 1) / max(tiles - 1, 1);
      const int q0 = end ? 0 : share(NC, i + 1, TI), q1 = end ? share(NB, 1, TJ) : share(NC, i + 2, TI);
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
          const int tb = row_of(i - 1);
#pragma unroll
          for (int tj = 0; tj < TJ; ++tj)
            if (tj >= (TRI ? tb : 0) && (tj - (TRI ? tb : 0)) * tiles / (TJ - (TRI ? tb : 0)) == u) dupdate(tb, tj);
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

  if (npr > 0) {
    set_b();
    set_c();
#pragma unroll
    for (int q = 0; q < NB; ++q) dmaB(q, b0);
#pragma unroll
    for (int q = 0; q < NC; ++q) dmaC(q, b1);
    next(pB, kB);
    set_b();
    constexpr int SLOT = NB / TJ;   // share(NB, 1, TJ)
#pragma unroll
    for (int q = 0; q < SLOT; ++q) dmaB(q, b2);
    vm_lds_barrier<NC + SLOT>();
#pragma unroll
    for (int q = 0; q < 4 + 2 * TI; ++q) readB(q, b0, 0, 0);
  }
  const std::true_type yes;
  const std::false_type no;
  int pr = 0;
  do {
    if (npr > 0) {
      if (kst == 1) {
        chunk(yes, yes);
      } else {
        chunk(yes, no);
        for (int k = 2; k < kst; ++k) chunk(no, no);
        chunk(no, yes);
      }
      ++pr;
    }
    // (an empty range writes zeros)
    if (pr == npr || pr % FLUSH_PAIRS == 0)
      store_d<TI, TJ, TRI>(D, sm.d, f, set, z, R0, P0, wave, pr <= FLUSH_PAIRS);
  } while (pr < npr);
  // the last (repeated) memory-to-LDS loads land before the workgroup may end
  __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

template <int M>
__device__ __forceinline__ void fused_pair_body(const FusedArgs& f, Smem& sm) {
  const int naux = f.naux;

  // tile and pair range: XCD-aware order (workgroup b runs on XCD b mod 8; each
  // XCD owns the partial slots z = xcd, xcd + 8, ..., a block of consecutive
  // pair ranges, and walks the tiles of one slot in bands of two R blocks, P by
  // P with R fastest, so its resident workgroups share panels in its L2).  With
  // symmetric D only the tiles on or above the diagonal are walked (nb (nb + 1)
  // / 2 of them; the grid has nb^2 per slot, the rest exit at once).  The
  // integer divisions run on the vector unit; readfirstlane marks their results
  // uniform so that buffer resources and offsets stay scalar.
  const int nb = (naux + TT - 1) / TT;
  const int set = blockIdx.y;
  const bool symm = f.sym != nullptr && f.sym[set] != 0;
  const int ntl = symm ? nb * (nb + 1) / 2 : nb * nb;
  const int b = blockIdx.x;
  const int xcd = b % NXCD16, local = b / NXCD16;
  if (local >= ntl * (f.vsplit / NXCD16)) return;
  const int z = __builtin_amdgcn_readfirstlane(xcd + NXCD16 * (local / ntl));
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

  // The last block of naux % 128 columns or rows forms only the 32-wide strips that hold
  // a THC point, and a diagonal tile of a symmetric D only its upper triangle.  Against
  // full 128 x 128 products everywhere: n = 149, naux = 797 (29 of the last 128), general,
  // FP32: 696 -> 590 us a tau point; n = 300, naux = 1800 (8 of 128), symmetric, fp16x2:
  // 1927 -> 1833 us
  const int tj = min((naux - P0 + 31) / 32, 4), ti = min((naux - R0 + 31) / 32, 4);
  const bool diag = symm && R0 == P0;
#define THCSOX_TILE(TI, TJ, TRI) fused_tile<M, TI, TJ, TRI>(f, sm, set, z, R0, P0)
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

__global__ __launch_bounds__(NTH) __attribute__((amdgpu_waves_per_eu(1, 1)))
void fused_f16_kernel(FusedArgs f) {
  __shared__ __attribute__((aligned(16))) Smem sm;
  fused_pair_body<MODE_F16X2>(f, sm);
}

__global__ __launch_bounds__(NTH) __attribute__((amdgpu_waves_per_eu(1, 1)))
void fused_f32_kernel(FusedArgs f) {
  __shared__ __attribute__((aligned(16))) Smem sm;
  fused_pair_body<MODE_F32>(f, sm);
}

inline unsigned cdiv16(int64_t a, int64_t b) { return (unsigned)((a + b - 1) / b); }

}  // namespace

void fused_f16_tile(int* rows, int* cols) {
  *rows = TT;
  *cols = TT;
}

hipError_t sox_fused_pairs(int mode, const FusedArgs& f, hipStream_t s) {
  if (mode != MODE_F16X2 && mode != MODE_F32) return hipErrorInvalidValue;
  const int npair = (f.n + 1) / 2;
  const int pairs_max = (npair + f.vsplit - 1) / f.vsplit;   // longest pair range
  if (f.vsplit % NXCD16 != 0 || f.ldk % KC != 0 || f.ldk < f.n ||
      (f.dpart_f32 && pairs_max > FLUSH_PAIRS))
    return hipErrorInvalidValue;
  // buffer offsets inside one tile's rows of U (rows of 4 ldk bytes) are 32-bit
  if ((int64_t)TT * f.n * f.ldk * 4 > 0x7fffffffLL) return hipErrorInvalidValue;
  const unsigned nb = cdiv16(f.naux, TT);
  if (mode == MODE_F16X2) fused_f16_kernel<<<dim3(nb * nb * f.vsplit, f.nsets), NTH, 0, s>>>(f);
  else fused_f32_kernel<<<dim3(nb * nb * f.vsplit, f.nsets), NTH, 0, s>>>(f);
  return hipGetLastError();
}

}  // namespace thcsox
