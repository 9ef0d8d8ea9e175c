// One row task of the row pass (see ntt_device.hpp), shared by the batch
// kernels (row_kernel.inc) and the job-table kernels (jobs_kernels.inc).
//
//   ROW_FWD  the last c stages of Alg. 5 on one row, in place
//   ROW_INV  the first c stages of Alg. 6 (scaled by 1/N), in place
//   ROW_MUL  the row of a forward, the row of b forward, pointwise product
//            mod q, inverse; with R = 1 this is all of Eq. 2 for one pair
//   ROW_SQR  as ROW_MUL with b = a (one forward transform)
#pragma once
#include "ntt_device.hpp"
#include "pm_internal.hpp"

namespace pm {

template <int GEO, int KIND, typename W>
constexpr bool product_in_blocks() {
  return RowGeom<GEO>::LC >= 3 && (sizeof(W) == 4 || KIND == KIND_WIDE);
}

// A transform's row ends (the inverse: starts) with 16 consecutive words per
// thread, so that the lanes of a wave store 16 bytes each at a stride of 128: one
// more LDS exchange to round 0's layout makes them whole lines. Forward
// transforms of N = 2^16 x 384: 217 -> 198 us for both passes, 182 with the
// twiddles loaded ahead (RowTwRound).
// Coefficient-major rows move whole lines in any layout.
template <int GEO>
constexpr bool exchange_io() { return RowGeom<GEO>::EB == 4 && RowGeom<GEO>::NR > 1 && !(GEO & ROW_GEO_SAME); }

// Words of a split's row pass (R > 1) come from and go to a column pass in lazy
// form: below H from the forward columns, below GIN to the inverse columns. With
// R = 1 the input is canonical (which is below H too) and the output is made so
// (single). lg = log2 N: the inverse scales by 1/N. st: the step between words.
// BIN: the forward rows' bound where it is known to be lower (col_bound), which saves
// the reductions of one stage in ten.
template <int GEO, int KIND, int MODE, int BIN = 0, typename W, typename MT, typename S = Unit>
__device__ __forceinline__ void row_task(const W* A, const W* Bp, W* Cout, const W* tf, const W* ti, uint32_t Rr,
                                         bool active, bool single, uint32_t lg, const MT& M, W* lds, uint32_t t,
                                         S st = S{}) {
  using G = RowGeom<GEO>;
  using L = LazyRule<W, KIND>;
  constexpr int NX = MODE == ROW_MUL ? 2 : 1;
  constexpr int B = BIN ? BIN : L::H;
  // the product leaves out the two smallest strides of its three transforms
  // where it can (blk4_mul): not for moduli beyond 60 bits on 64-bit words
  constexpr int TR = (MODE == ROW_MUL || MODE == ROW_SQR) && product_in_blocks<GEO, KIND, W>() ? 2 : 0;
  Tw<W>* const table = (Tw<W>*)(lds + (G::TW_LDS ? G::LDS_ROW : 0));
  W x[NX][G::E];
#pragma unroll
  for (int i = 0; i < NX; ++i)
#pragma unroll
    for (int j = 0; j < G::E; ++j) x[i][j] = 0;
  if constexpr (MODE == ROW_INV) {
    W tl = 0;
    if constexpr (G::TW_LDS) tl = tw_lds_word(ti, t, Rr);
    const RowTw<GEO, 0, 1, W> tws(t, ti, Rr, table);
    if constexpr (exchange_io<GEO>()) {
      if (active) gmem_get<GEO, 0>(A, x[0], t, st);
      exchange<GEO, 0, G::NR - 1>(lds, x[0], t);
    } else {
      if (active) gmem_get<GEO, G::NR - 1>(A, x[0], t, st);
    }
    if constexpr (G::TW_LDS) tw_lds_put<KIND>(table, tl, t, M);
    inv_rounds<GEO, KIND, 0, Q1>(lds, x[0], t, tws, lg, M);
  } else {
    W tl = 0;
    if constexpr (G::TW_LDS) tl = tw_lds_word(tf, t, Rr);
    if (active) gmem_get<GEO, 0>(A, x[0], t, st);
    if constexpr (NX == 2) {
      if (active) gmem_get<GEO, 0>(Bp, x[1], t, st);
    }
    const RowTw<GEO, TR, NX, W> tws(t, tf, Rr, table);
    if constexpr (G::TW_LDS) tw_lds_put<KIND>(table, tl, t, M);      // read after round 0's exchange
    if constexpr (MODE == ROW_FWD) {
      fwd_rounds<GEO, KIND, TR, B>(lds, x, t, tws, M);
      canon_all<KIND>(x[0], M);
      if constexpr (exchange_io<GEO>()) {
        exchange<GEO, G::NR - 1, 0>(lds, x[0], t);
        if (active) gmem_put<GEO, 0>(Cout, x[0], t, st);
      } else {
        if (active) gmem_put<GEO, G::NR - 1>(Cout, x[0], t, st);
      }
      return;
    } else {
      const RowTw<GEO, TR, 1, W> iws(t, ti, Rr, table);
      if constexpr (TR == 2) {
        const Blk4Tw<GEO, W> gs(t, tf, Rr);
        fwd_rounds<GEO, KIND, TR, B>(lds, x, t, tws, M);
        __builtin_amdgcn_sched_barrier(0);
        W il = 0;
        if constexpr (G::TW_LDS) il = tw_lds_word(ti, t, Rr);
        blk4_mul<GEO, KIND>(x[0], x[NX - 1], gs, t, M);         // NX = 1: a = b
        // the forward table's last reads are behind round 2's exchange
        if constexpr (G::TW_LDS) tw_lds_put<KIND>(table, il, t, M);
        inv_rounds<GEO, KIND, TR, L::B4>(lds, x[0], t, iws, lg - TR, M);
      } else {
        fwd_rounds<GEO, KIND, TR, B>(lds, x, t, tws, M);
        __builtin_amdgcn_sched_barrier(0);
        W il = 0;
        if constexpr (G::TW_LDS) il = tw_lds_word(ti, t, Rr);
#pragma unroll
        for (int j = 0; j < G::E; ++j) x[0][j] = mul_lazy<KIND>(x[0][j], x[NX - 1][j], M);
        if constexpr (G::TW_LDS) tw_lds_put<KIND>(table, il, t, M);
        inv_rounds<GEO, KIND, TR, L::PW>(lds, x[0], t, iws, lg, M);
      }
    }
  }
  if (single) canon_all<KIND>(x[0], M);
  if (active) gmem_put<GEO, 0>(Cout, x[0], t, st);
}

// Register budget: 4 waves per SIMD (<= 128 VGPRs).
constexpr int ROW_WAVES = 4;

}  // namespace pm
