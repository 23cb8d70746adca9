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
// the tile: the accumulators of B and C (128 registers) live in the matrix-core
// registers (AGPRs), the fragments of the three planes in the ordinary ones.  The
// partial sum of D (FP32, at most 8 v) lives in LDS, one private 16-byte slot per
// lane and MFMA tile, updated once per v: D += B o C.  (The fp16x2 kernel takes
// two v per pass in the same registers and LDS: two planes of two v there, three
// planes of one v here.)
//
// Pipeline.  A k chunk is two half stages, each two panels of 128 rows x 32 k x
// 3 planes (48 KiB): the B half (G, A_v) in LDS buffer sB and the C half (GX,
// U_v) in sC; with 64 KiB for D the workgroup uses the full 160 KiB of LDS.  A
// plane of a panel is 128 rows of 64 bytes, each row's four 16-byte chunks
// placed by lds_chunk.  Chunk t runs as
//   phase B(t): barrier (C(t) is in sC, every wave has read B(t) from sB);
//               loads of B(t+1) -> sB; fragments of C(t) <- sC;
//               matrix cores: B += products of B(t) (fragments read before)
//   phase C(t): barrier (B(t+1) is in sB, every wave has read C(t) from sC);
//               loads of C(t+1) -> sC; fragments of B(t+1) <- sB;
//               matrix cores: C += products of C(t)
// so each half stage is loaded one phase ahead of its fragment reads, and each
// fragment is read one phase ahead of its products.  The first chunk of a v
// starts the accumulators from zero inside the MFMA.  Past the last chunk the
// loads repeat it (never used).
#include "kernels.hpp"
#include "mfma.hpp"
#include "panel.hpp"

namespace thcsox {
namespace {

constexpr int TT = 128;          // tile edge of D (R and P)
constexpr int NW = 4, NTH = 64 * NW;
constexpr int KC = 32;           // k per chunk (one bf16 MFMA)
constexpr int NPL = 3;           // bf16 planes
constexpr int PP = TT * KC;      // elements of one plane of a panel
constexpr int FLUSH_V = 8;       // v per FP32 partial sum of D
constexpr int NXCD = 8;

// One half stage: panel 0 is the v-independent operand (G or GX), panel 1 the
// per-v one (A_v or U_v); [panel][plane][row * 32 + k].
struct Half3 {
  __bf16 s[2][NPL][PP];
};

__device__ __forceinline__ void bf3_vm_lds_barrier() {
  // this wave's memory loads (including those that write LDS) and LDS accesses
  // complete, then the workgroup barrier
  __asm__ volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// One tile's range of v.  sB: G, A_v; sC: GX, U_v; sD: the partial sum of D.  Each wave
// forms TI x TJ tiles of 16 x 16 out of its 4 x 4: the rows R of the workgroup's tile
// beyond 32 TI and the columns P beyond 32 TJ lie past naux and are neither loaded nor
// multiplied.  TRI: a diagonal tile of a symmetric D, of which only the 16 x 16 tiles ti
// <= tj of each wave are formed: they hold every element on and above the diagonal.  (A
// D element's products and their order do not depend on TI, TJ and TRI.)
template <int TI, int TJ, bool TRI>
__device__ __forceinline__ void fused_bf3_tile(const FusedArgs& f, Half3& sB, Half3& sC, f4* sD, int set,
                                               int z, int R0, int P0) {
  int tid = threadIdx.x;
  // (the compiler must not merge the forms' address arithmetic above their branch)
  __asm__ volatile("" : "+v"(tid), "+s"(set), "+s"(z), "+s"(R0), "+s"(P0));
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

  // operand planes (rows past the valid range lie beyond the buffer resources
  // and read as zero)
  const __bf16* Gt = static_cast<const __bf16*>(f.Gt) + set * f.g_set;
  const __bf16* GX = static_cast<const __bf16*>(f.GXt) + set * f.g_set;
  const __bf16* Ub = static_cast<const __bf16*>(f.U);
  const __bf16* Ab = static_cast<const __bf16*>(f.A) + set * f.a_set;
  __amdgpu_buffer_rsrc_t rG[NPL], rX[NPL];
#pragma unroll
  for (int p = 0; p < NPL; ++p) {
    rG[p] = make_rsrc(Gt + p * f.g_plane + (int64_t)R0 * ldk, (int64_t)rows_r * ldk * 2);
    rX[p] = make_rsrc(GX + p * f.g_plane + (int64_t)P0 * ldk, (int64_t)rows_p * ldk * 2);
  }
  const int64_t a_bytes = (int64_t)rows_p * ldk * 2;
  const int64_t u_bytes = ((int64_t)(rows_r - 1) * n * ldk + ldk) * 2;
  // per v: A rows (v, P) and U rows (R, v)
  __amdgpu_buffer_rsrc_t rA[NPL], rU[NPL];
  auto set_v = [&](int iv) {
    const int v = v_lo + iv;
#pragma unroll
    for (int p = 0; p < NPL; ++p) {
      rA[p] = make_rsrc(Ab + p * f.a_plane + ((int64_t)v * naux + P0) * ldk, a_bytes);
      rU[p] = make_rsrc(Ub + p * f.u_plane + ((int64_t)R0 * n + v) * ldk, u_bytes);
    }
  };

  // memory -> LDS: one instruction moves 16 rows x 64 bytes of one plane; wave w
  // moves the 16-row slabs w and w + 4 of each plane of each panel.  Lane l
  // lands at slab row l / 4, physical chunk l % 4, and loads the logical chunk
  // lds_chunk maps there (the map is its own inverse for a given row).
  uint32_t dR[2], dU[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int row = (wave + NW * j) * 16 + (lane >> 2);
    const int c = lds_chunk(row, lane & 3);
    dR[j] = (uint32_t)((row * ldk + 8 * c) * 2);
    dU[j] = (uint32_t)((row * (n * ldk) + 8 * c) * 2);
  }
  auto dmaB = [&](int k0) {
    const int so = k0 * 2;   // bytes to the k chunk
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int slab = (wave + NW * j) * 16 * 32;
#pragma unroll
      for (int p = 0; p < NPL; ++p) {
        if (2 * j < TI) __builtin_amdgcn_raw_ptr_buffer_load_lds(rG[p], &sB.s[0][p][slab], 16, dR[j], so, 0, 0);
        if (2 * j < TJ) __builtin_amdgcn_raw_ptr_buffer_load_lds(rA[p], &sB.s[1][p][slab], 16, dR[j], so, 0, 0);
      }
    }
  };
  auto dmaC = [&](int k0) {
    const int so = k0 * 2;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int slab = (wave + NW * j) * 16 * 32;
#pragma unroll
      for (int p = 0; p < NPL; ++p) {
        if (2 * j < TJ) __builtin_amdgcn_raw_ptr_buffer_load_lds(rX[p], &sC.s[0][p][slab], 16, dR[j], so, 0, 0);
        if (2 * j < TI) __builtin_amdgcn_raw_ptr_buffer_load_lds(rU[p], &sC.s[1][p][slab], 16, dU[j], so, 0, 0);
      }
    }
  };

  // fragment (row r, k chunk lane / 16) of a plane at r * 32 + lds_chunk(r, lane / 16) * 8.
  // The 16 x 16 tiles alternate between the two waves of a row or column, so both work in
  // a short tile; the map repeats every 32 rows, so tile t is 32 t rows further.
  const int lr = lane & 15, kc = lane >> 4;
  const int fR = (wr * 16 + lr) * 32 + lds_chunk(wr * 16 + lr, kc) * 8;   // R side rows
  const int fP = (wc * 16 + lr) * 32 + lds_chunk(wc * 16 + lr, kc) * 8;   // P side rows
  // fragments of one half stage: the shared operand s (G or GX) and the per-v
  // operand m (A_v or U_v), [plane][tile]
  struct FragsB { bf16x8 s[NPL][TI], m[NPL][TJ]; } fb;
  struct FragsC { bf16x8 s[NPL][TJ], m[NPL][TI]; } fc;
  auto rd = [&](const __bf16* base, int off, int t) {
    return *reinterpret_cast<const bf16x8*>(base + off + t * 32 * 32);
  };
  auto readB = [&](FragsB& fr) {   // G (R side), A_v (P side)
#pragma unroll
    for (int p = 0; p < NPL; ++p)
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        if (t < TI) fr.s[p][t] = rd(sB.s[0][p], fR, t);
        if (t < TJ) fr.m[p][t] = rd(sB.s[1][p], fP, t);
      }
  };
  auto readC = [&](FragsC& fr) {   // GX (P side), U_v (R side)
#pragma unroll
    for (int p = 0; p < NPL; ++p)
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        if (t < TJ) fr.s[p][t] = rd(sC.s[0][p], fP, t);
        if (t < TI) fr.m[p][t] = rd(sC.s[1][p], fR, t);
      }
  };

  // accumulators [ti][tj]: rows R of tile ti, columns P of tile tj (cleared once
  // here; each v then starts them from zero inside its first MFMAs)
  f4 B[TI][TJ], C[TI][TJ];
  const f4 zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int ti = 0; ti < TI; ++ti)
#pragma unroll
    for (int tj = TRI ? ti : 0; tj < TJ; ++tj) B[ti][tj] = C[ti][tj] = zero;
  using PR = Products<NPL>;   // plane pairs, smallest terms first
  // B products: B[ti][tj] += G[ti] . A_v[tj]
  auto mfmaB = [&](const FragsB& fr, bool first) {
#pragma unroll
    for (int ti = 0; ti < TI; ++ti)
#pragma unroll
      for (int tj = TRI ? ti : 0; tj < TJ; ++tj) {
        f4 a = first ? zero : B[ti][tj];
#pragma unroll
        for (int q = 0; q < PR::N; ++q)
          a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fr.s[PR::a(q)][ti], fr.m[PR::b(q)][tj], a,
                                                      0, 0, 0);
        B[ti][tj] = a;
      }
  };
  // C products: C[ti][tj] += U_v[ti] . GX[tj]
  auto mfmaC = [&](const FragsC& fr, bool first) {
#pragma unroll
    for (int ti = 0; ti < TI; ++ti)
#pragma unroll
      for (int tj = TRI ? ti : 0; tj < TJ; ++tj) {
        f4 a = first ? zero : C[ti][tj];
#pragma unroll
        for (int q = 0; q < PR::N; ++q)
          a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fr.m[PR::a(q)][ti], fr.s[PR::b(q)][tj], a,
                                                      0, 0, 0);
        C[ti][tj] = a;
      }
  };

  // the partial sum of D: slot (wave, tile) of each lane, 64 lanes x 16 bytes
  f4* const Dw = sD + wave * 16 * 64 + lane;
  auto dzero = [&]() {
#pragma unroll
    for (int tt = 0; tt < TI * TJ; ++tt) Dw[tt * 64] = zero;
  };
  auto dupdate = [&]() {
#pragma unroll
    for (int ti = 0; ti < TI; ++ti)
#pragma unroll
      for (int tj = TRI ? ti : 0; tj < TJ; ++tj) {
        f4 d = Dw[(ti * TJ + tj) * 64];
#pragma unroll
        for (int r = 0; r < 4; ++r) d[r] = fmaf(B[ti][tj][r], C[ti][tj][r], d[r]);
        Dw[(ti * TJ + tj) * 64] = d;
      }
  };
  // D tile -> partial tile z (FP32 store, or FP64 add unless first): thread t
  // takes column P0 + t % 128 and rows R0 + t / 128 + 2 i, reading each element
  // from the LDS slot of the lane that formed it (lane 16 (R % 16 / 4) + P % 16
  // of wave 2 (R / 16 % 2) + P / 16 % 2, tile (R / 32, P / 32), element R % 4),
  // so the global writes are coalesced rows.  Barriers before (other waves'
  // slots) and after (the slots may be cleared next).
  auto flush = [&](bool first) {
    __syncthreads();
    const float* sDf = reinterpret_cast<const float*>(sD);
    const int Pt = tid & (TT - 1), P = P0 + Pt;
    const int pslot = ((Pt >> 4) & 1) * 16 * 64 + (Pt >> 5) * 64 + (Pt & 15);
    const int64_t zo = set * f.d_set + (int64_t)z * naux * naux + P;
    for (int Rt = tid >> 7; Rt < TT; Rt += NTH / TT) {
      const int R = R0 + Rt;
      if (R < naux && P < naux && (!TRI || (Rt >> 5) <= (Pt >> 5))) {
        const int slot = pslot + ((Rt >> 4) & 1) * 2 * 16 * 64 + (Rt >> 5) * TJ * 64 + ((Rt >> 2) & 3) * 16;
        const float v = sDf[slot * 4 + (Rt & 3)];
        const int64_t o = zo + (int64_t)R * naux;
        if (f.dpart_f32) {   // one range = one FP32 partial sum (first is true)
          reinterpret_cast<float*>(f.Dpart)[o] = v;
        } else {
          f.Dpart[o] = (first ? 0.0 : f.Dpart[o]) + (double)v;
        }
      }
    }
    __syncthreads();
  };

  dzero();
  // fetch cursor over (v, chunk), clamped to the last chunk
  int cv = 0, ck = 0;
  auto advance = [&]() {
    const bool last = (cv == nv - 1) && (ck == kst - 1);
    const bool wrap = (ck == kst - 1);
    ck = last ? ck : (wrap ? 0 : ck + 1);
    if (wrap && !last) set_v(++cv);
  };
  if (nv > 0) {
    set_v(0);
    dmaB(0);
    dmaC(0);
    advance();
    bf3_vm_lds_barrier();
    readB(fb);
  }
  // spread a phase's memory-to-LDS loads over its MFMAs: 12 over 96 in a full tile
  constexpr int NR = TI > 2 ? 6 : 3, NP = TJ > 2 ? 6 : 3;   // loads of a panel of rows, of columns
  auto spread = [&]() {
    constexpr int NM = PR::N * (TRI ? TI * (TI + 1) / 2 : TI * TJ);
    constexpr int MPL = NM / (NR + NP) < 8 ? NM / (NR + NP) : 8;
#pragma unroll
    for (int i = 0; i < NR + NP; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x010, 1, 0);     // one memory instruction
      __builtin_amdgcn_sched_group_barrier(0x008, MPL, 0);   // MPL MFMAs
    }
  };
  auto chunk = [&](bool first) {
    bf3_vm_lds_barrier();
    dmaB(ck * KC);
    readC(fc);
    mfmaB(fb, first);
    spread();
    bf3_vm_lds_barrier();
    dmaC(ck * KC);
    advance();
    readB(fb);
    mfmaC(fc, first);
    spread();
  };
  int done = 0;
  for (int iv = 0; iv < nv; ++iv) {
    chunk(true);
    for (int k = 1; k < kst; ++k) chunk(false);
    dupdate();
    ++done;
    if (done % FLUSH_V == 0 && iv + 1 < nv) {
      flush(done == FLUSH_V);
      dzero();
    }
  }
  // the last (repeated) memory-to-LDS loads land before the workgroup may end
  __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");
  flush(done <= FLUSH_V);   // also writes zeros for an empty range
}

__global__ __launch_bounds__(NTH) __attribute__((amdgpu_waves_per_eu(1, 1)))
void fused_bf3_kernel(FusedArgs f) {
  __shared__ __attribute__((aligned(16))) Half3 sB;
  __shared__ __attribute__((aligned(16))) Half3 sC;
  __shared__ __attribute__((aligned(16))) f4 sD[NW * 16 * 64];
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
#define THCSOX_TILE(TI, TJ, TRI) fused_bf3_tile<TI, TJ, TRI>(f, sB, sC, sD, set, z, R0, P0)
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
