// What the 128 x 128 fused kernels (fused_f16.hip, fused_bf3.hip) share: the waits of
// their pipeline and the way a tile of D goes to memory.
#pragma once
#include "kernels.hpp"
#include "mfma.hpp"

namespace thcsox {
namespace {

constexpr int TT = 128;          // tile edge of D (R and P)
// two waves' 16 x 16 tiles side by side make a strip: a diagonal tile forms the strips' blocks
// on and above its diagonal
static_assert(SYM_BLOCK == 32 && TT % SYM_BLOCK == 0, "the strips are the blocks of a symmetric D");

// All but the newest LEFT of this wave's memory loads (including those that write LDS)
// and all of its LDS accesses complete, then the workgroup barrier.
template <int LEFT>
__device__ __forceinline__ void vm_lds_barrier() {
  __asm__ volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(LEFT) : "memory");
}
// The same for the LDS accesses alone.
__device__ __forceinline__ void lds_barrier() {
  __asm__ volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// D tile -> partial tile z (FP32 store, or FP64 add unless first; D is cleared), 32 rows at
// a time through lds (32 x TT floats) so that rows are written in 16-byte pieces (of
// element alignment); the 16 columns of a tile are permuted by the row, else its four row
// groups share banks.  Lane l of wave w holds rows 32 ti + 16 (w / 2) + 4 (l / 16) + r and column
// 32 tj + 16 (w % 2) + l % 16 of the tile in D[ti][tj][r].
template <int TI, int TJ, bool TRI>
__device__ __forceinline__ void store_d(f4 (&D)[TI][TJ], float* lds, const FusedArgs& f, int set, int z,
                                        int R0, int P0, int wave, bool first) {
  typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
  typedef double d4u __attribute__((ext_vector_type(4), aligned(8)));
  // (its addresses are computed here, not kept in registers over the k loops)
  uint32_t all = ~0u;
  __asm__ volatile("" : "+s"(all));
  const int ft = 64 * wave + (int)__builtin_amdgcn_mbcnt_hi(all, __builtin_amdgcn_mbcnt_lo(all, 0));
  const int fr = (ft & 15), fk = (ft >> 4) & 3, frow = ft >> 5, col = (ft & 31) * 4;
#pragma unroll
  for (int ti = 0; ti < TI; ++ti) {
#pragma unroll
    for (int tj = TRI ? ti : 0; tj < TJ; ++tj)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        lds[(wave / 2 * 16 + 4 * fk + r) * TT + ((((2 * tj + wave % 2) ^ fk) << 4) | fr)] = D[ti][tj][r];
        D[ti][tj][r] = 0.f;
      }
    lds_barrier();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = frow + 8 * i;
      const int R = R0 + 32 * ti + row, P = P0 + col;
      if (R < f.naux && P < f.naux && (!TRI || ti <= (col >> 5))) {
        const f4 v = *reinterpret_cast<const f4*>(&lds[row * TT + (col ^ (((row >> 2) & 3) << 4))]);
        const int64_t o = set * f.d_set + ((int64_t)z * f.naux + R) * f.naux + P;
        const int left = f.naux - P;
        if (f.dpart_f32) {   // one range = one FP32 partial sum (first is true)
          float* dst = reinterpret_cast<float*>(f.Dpart) + o;
          if (left >= 4) {
            *reinterpret_cast<f4u*>(dst) = v;
          } else {
#pragma unroll
            for (int e = 0; e < 3; ++e)
              if (e < left) dst[e] = v[e];
          }
        } else {
          double* dst = f.Dpart + o;
          if (left >= 4) {
            d4u w = {v[0], v[1], v[2], v[3]};
            if (!first) w += *reinterpret_cast<const d4u*>(dst);
            *reinterpret_cast<d4u*>(dst) = w;
          } else {
#pragma unroll
            for (int e = 0; e < 3; ++e)
              if (e < left) dst[e] = (first ? 0.0 : dst[e]) + (double)v[e];
          }
        }
      }
    }
    lds_barrier();
  }
}

}  // namespace
}  // namespace thcsox
