// One row task of the row pass (see ntt_device.hpp), shared by the batch
// kernels (row_kernel.inc) and the job-table kernels (pm_jobs.hip).
//
//   ROW_FWD  the last c stages of Alg. 5 on one row, in place
//   ROW_INV  the first c stages of Alg. 6 (scaled by 1/N), in place
//   ROW_MUL  the row of a forward, the row of b forward, pointwise product
//            mod q, inverse; with R = 1 this is all of Eq. 2 for one pair
//   ROW_SQR  as ROW_MUL with b = a (one forward transform)
//   ROW_FMUL the fused product of Sec. III-B (Alg. 8): truncated rows of a and
//            b, Alg. 7 on adjacent pairs, truncated inverse rows
#pragma once
#include "ntt_device.hpp"
#include "pm_internal.hpp"

namespace pm {

// Words of a split's row pass (R > 1) come from and go to a column pass in lazy
// form: below H from the forward columns, below GIN to the inverse columns. With
// R = 1 the input is canonical (which is below H too) and the output is made so
// (single). lg = log2 N: the inverse scales by 1/N.
template <int GEO, int KIND, int MODE, typename W, typename MT>
__device__ __forceinline__ void row_task(const W* A, const W* B, W* Cout, const W* tf, const W* ti, uint32_t Rr,
                                         bool active, bool single, uint32_t lg, const MT& M, W* lds, uint32_t t) {
  using G = RowGeom<GEO>;
  using L = LazyRule<W, KIND>;
  constexpr int NX = (MODE == ROW_MUL || MODE == ROW_FMUL) ? 2 : 1;
  W x[NX][G::E];
#pragma unroll
  for (int i = 0; i < NX; ++i)
#pragma unroll
    for (int j = 0; j < G::E; ++j) x[i][j] = 0;
  if constexpr (MODE == ROW_INV) {
    if (active) gmem_get<GEO, G::NR - 1>(A, x[0], t);
    inv_rounds<GEO, KIND, false, Q1>(lds, x[0], t, ti, Rr, lg, M);
  } else {
    if (active) gmem_get<GEO, 0>(A, x[0], t);
    if constexpr (NX == 2) {
      if (active) gmem_get<GEO, 0>(B, x[1], t);
    }
    fwd_rounds<GEO, KIND, MODE == ROW_FMUL, L::H>(lds, x, t, tf, Rr, M);
    if constexpr (MODE == ROW_FWD) {
      canon_all<KIND>(x[0], M);
      if (active) gmem_put<GEO, G::NR - 1>(Cout, x[0], t);
      return;
    }
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (MODE == ROW_FMUL) {
      // fused product (Alg. 8): Alg. 7 on adjacent pairs of the truncated rows
      const FusedTw<GEO, W> ftw = fused_twiddles<GEO>(t, tf, Rr);
      fused_hadamard<GEO, KIND>(x[0], x[1], ftw, M);
      inv_rounds<GEO, KIND, true, 2 * Q1>(lds, x[0], t, ti, Rr, lg - 1, M);
    } else {
#pragma unroll
      for (int j = 0; j < G::E; ++j) x[0][j] = mul_lazy<KIND>(x[0][j], x[NX - 1][j], M);   // NX = 1: a = b
      inv_rounds<GEO, KIND, false, L::PW>(lds, x[0], t, ti, Rr, lg, M);
    }
  }
  if (single) canon_all<KIND>(x[0], M);
  if (active) gmem_put<GEO, 0>(Cout, x[0], t);
}

// Register budget: 4 waves per SIMD (<= 128 VGPRs).
template <int MODE>
struct RowWaves {
  static constexpr int value = 4;
};

}  // namespace pm
