// Device building blocks of the merged NTTs (Alg. 5 and Alg. 6) on gfx950.
//
// Decomposition. A polynomial of N = R*C coefficients is viewed as an R x C
// row-major matrix (R = 2^s rows, C = 2^c columns). Unrolling the loops of
// Alg. 5 shows that a butterfly at stride k pairs j and j+k inside group
// i = j / (2k) of stage m = N / (2k), with twiddle psi_br[m + i]:
//   * strides k >= C (the first s stages) pair rows of one column; every
//     column runs the same R-point merged NTT with twiddles psi_br[1..R);
//   * strides k < C (the last c stages) stay inside one row r; with
//     mm = C / (2k) groups per row the twiddle index is (R + r)*mm + i_row,
//     i_row = (column index) / (2k).
// Alg. 6 has the same (m, k, i) structure, run in the opposite stage order,
// so the inverse uses the same indices on psi_inv_br. No transposition and no
// extra twiddle table is needed. R = 1 is the single-pass case.
//
// Row pass. A row of C = 2^c words is held by T = C/16 threads, 16 words per
// thread in registers. The c stages are taken in rounds of four from the top
// (largest stride first): a round whose butterfly bits are [p, p+4) gives
// each thread the 16 words whose index bits [p, p+4) vary, so the round's
// four stages are radix-16 in registers. Rounds exchange data through LDS.
// The last round always holds bits [0, 4) (16 consecutive words per thread);
// when c is not a multiple of 4 it runs only the remaining c mod 4 stages.
// The small-batch geometry does the same with rounds of two stages and 4
// words per thread: four times the threads per row, for batches too small
// to fill the GPU with 16-word threads.
//
// Words inside a transform are lazy (lazymod.hpp): each routine states the
// bounds it takes and leaves, in sixteenths of q. The product's two forward rows
// run together, round by round, so that they share every twiddle load and
// companion; the inverse rows scale by 1/N in their last stage.
//
// Column pass. One thread per column holds the R = 2^s words of that column
// in registers and runs the s column stages; twiddles are uniform per launch.
// In the software-pipelined kernels a 32-word column (s = 5) is held by two
// lanes of one wave instead, 16 words each (col32_fwd_pair below), so that the
// column code needs no more registers than the row code beside it.
#pragma once
#include <type_traits>

#include "lazymod.hpp"

namespace pm {

// Row geometry code GEO: bits [0, 5) = c (row of 2^c words); bit 5 set =
// rounds of two stages with 4 words per thread (the small-batch geometry,
// more threads per row), clear = rounds of four stages with 16 words per
// thread. For the 16-word geometry GEO = c.
constexpr int row_geo(int logc, int ebx) { return logc | (ebx == 2 ? 32 : 0); }
// bit 6: workgroups of at least 256 threads, several rows each (the job
// tables' row kernel, one workgroup size for every row length)
constexpr int ROW_GEO_SHARED = 64;
// bit 7: the rows of a workgroup are the same row of several polynomials, so they
// share its twiddles
constexpr int ROW_GEO_SAME = 128;

template <int GEO>
struct RowGeom {
  static constexpr int LC = GEO & 31;                  // log2(row length)
  static constexpr int EBX = (GEO & 32) ? 2 : 4;       // index bits per round
  static constexpr int EB = LC < EBX ? LC : EBX;       // log2(words per thread)
  static constexpr int E = 1 << EB;
  static constexpr int LOGT = LC - EB;
  static constexpr int T = 1 << LOGT;                  // threads per row
  static constexpr int NR = LC <= EBX ? 1 : (LC + EBX - 1) / EBX;   // rounds
  // rows shorter than a workgroup share one only below a wave: a row with its own
  // workgroup waits for no other row and has scalar twiddles in round 0
  static constexpr int WGMIN = (GEO & ROW_GEO_SHARED) ? 256 : 64;
  static constexpr int WG = T < WGMIN ? WGMIN : T;     // threads per workgroup
  static constexpr int ROWS = WG / T;                  // rows per workgroup
  static constexpr int LDS_ROW = (1 << LC) + ((1 << LC) >> 4);  // padded words
  // rows of 2^12 words keep round 1's 240 twiddles and companions beside the row
  // (TwLds): 38.9 KB, still four workgroups to a CU's 160 KB
  static constexpr bool TW_LDS = LC == 12 && EBX == 4;
  static constexpr int LDS_TW = TW_LDS ? 2 * T : 0;
  static constexpr int LDS_WORDS = NR > 1 ? ROWS * LDS_ROW + LDS_TW : 1;
  // register-bit base p and butterfly bits [lo, hi) of round rho (forward order)
  static constexpr int hi(int rho) { return LC - EBX * rho; }
  static constexpr int lo(int rho) { return hi(rho) - EBX > 0 ? hi(rho) - EBX : 0; }
  static constexpr int p(int rho) { return rho == NR - 1 ? 0 : hi(rho) - EBX; }
};

// Index inside the row of register j of thread t when the register bits are [p, p+EB).
template <int P, int EB>
__device__ __forceinline__ uint32_t reg_index(uint32_t t, uint32_t j) {
  return ((t >> P) << (P + EB)) | (j << P) | (t & ((1u << P) - 1u));
}

// Scheduling fence between stages: stops the compiler from hoisting the
// twiddle loads and butterflies of later stages, which bounds register use.
#ifndef PM_STAGE_FENCE
#define PM_STAGE_FENCE 1
#endif
__device__ __forceinline__ void stage_fence() {
#if PM_STAGE_FENCE
  __builtin_amdgcn_sched_barrier(0);
#endif
}

// LDS slot of row word idx is idx + idx/16: one pad word per 16 keeps strided
// 64-bit accesses spread over the banks. With idx = th*2^(P+EB) + j*2^P + tl
// (tl < 2^P, j < 2^EB) the slot splits into a per-thread base plus a
// per-register constant, so every LDS access is one instruction with an
// immediate offset:
//   slot = [a + a/16 + tl + tl/16] + [j*2^P + (j*2^P)/16],  a = th*2^(P+EB)
// (exact for every round of both geometries: the low part j*2^P + tl never
// carries into the next multiple of 16 above a). For EB = 4, a + a/16 =
// th*(2^(P+4) + 2^P).
template <int P, int EB>
__device__ __forceinline__ uint32_t lds_base(uint32_t t) {
  const uint32_t th = t >> P, tl = t & ((1u << P) - 1u);
  if constexpr (EB == 4) {
    return th * ((16u << P) + (1u << P)) + tl + (tl >> 4);
  } else {
    const uint32_t a = th << (P + EB);
    return a + (a >> 4) + tl + (tl >> 4);
  }
}
template <int P>
__device__ __forceinline__ constexpr uint32_t lds_off(uint32_t j) {
  return (j << P) + ((j << P) >> 4);
}
// Row offset of register j: per-thread base plus a per-register constant.
template <int P, int EB>
__device__ __forceinline__ uint32_t row_base(uint32_t t) {
  return ((t >> P) << (P + EB)) | (t & ((1u << P) - 1u));
}

// Round 0 of a workgroup with one row (or one row of several polynomials): its
// twiddles are the same for every thread (companions on the scalar unit).
template <int GEO, int RHO>
constexpr bool uniform_round() { return RHO == 0 && (RowGeom<GEO>::ROWS == 1 || (GEO & ROW_GEO_SAME)); }

// Stages of round RHO when the TR smallest strides are left out.
template <int GEO, int RHO, int TR>
constexpr int round_stages() {
  constexpr int HI = RowGeom<GEO>::hi(RHO), LO = RowGeom<GEO>::lo(RHO) > TR ? RowGeom<GEO>::lo(RHO) : TR;
  return HI > LO ? HI - LO : 0;
}

// A round as a register block. The stage that pairs register bit jb of a round
// at register base p has mm = 2^(LC-1-p-jb) groups per row, and the thread's
// group g of it uses the twiddle at Rr*mm + (t >> p)*2^(EB-1-jb) + g: with
//   rb = Rr*2^(LC-EB-p) + (t >> p)
// that is rb*2^(EB-1-jb) + g for every stage of the round.
template <int GEO>
__device__ __forceinline__ uint32_t round_block(uint32_t t, uint32_t Rr, int p) {
  using G = RowGeom<GEO>;
  return (Rr << (G::LC - G::EB - p)) + (t >> p);
}

// Where a round's twiddles and companions come from: TwMem reads each when its stage comes up;
// TwRegs holds all of the round's, loaded ahead (before the exchange that
// precedes the round, whose barriers then hide the latency). The transforms' rows
// use TwRegs (15 words beside the 16 of the row), the product's, which hold two
// rows, TwMem: with TwRegs they spill. TwLds: round 1 of a 2^12-word row, where 16
// threads share each twiddle: every thread makes one companion (load_tw_lds)
// and reads fifteen from LDS instead of making fifteen (product rows 174 -> 168
// in VALU cost, -3 %).
template <int EB, typename W>
struct TwMem {
  const W* __restrict__ tw;
  uint32_t rb;
  __device__ __forceinline__ TwMem(const W* __restrict__ t, uint32_t r, int, int) : tw(t), rb(r) {}
  __device__ __forceinline__ W raw(int jb, int g) const { return tw[(rb << (EB - 1 - jb)) + g]; }
  template <int KIND, bool UNI, typename MT>
  __device__ __forceinline__ Tw<W> get(int jb, int g, const MT& M) const {
    return tw_make<KIND, UNI>(raw(jb, g), M);
  }
};
template <int EB, typename W>
struct TwRegs {
  W v[1 << EB];
  __device__ __forceinline__ TwRegs() {}
  __device__ __forceinline__ TwRegs(const W* __restrict__ tw, uint32_t rb, int jlo, int jhi) {
#pragma unroll
    for (int jb = 0; jb < EB; ++jb)
      if (jb >= jlo && jb < jhi) {
#pragma unroll
        for (int g = 0; g < (1 << (EB - 1 - jb)); ++g) v[(1 << (EB - 1 - jb)) + g] = tw[(rb << (EB - 1 - jb)) + g];
      }
  }
  __device__ __forceinline__ W raw(int jb, int g) const { return v[(1 << (EB - 1 - jb)) + g]; }
  template <int KIND, bool UNI, typename MT>
  __device__ __forceinline__ Tw<W> get(int jb, int g, const MT& M) const {
    return tw_make<KIND, UNI>(raw(jb, g), M);
  }
};
// Round 1 of a 2^12-word row (register base 4): stage s of the round has the
// twiddles (Rr << (4+s)) + [0, 16 << s), kept at slot (16 << s) + i - 16; a thread's
// group g of it is slot ((16 + t/16) << s) + g - 16.
template <typename W>
struct TwLds {
  const Tw<W>* p;      // slots of the thread's row of the table
  uint32_t r16;        // 16 + t/16
  __device__ __forceinline__ W raw(int, int) const { return 0; }      // (never the row's last stage)
  template <int KIND, bool UNI, typename MT>
  __device__ __forceinline__ Tw<W> get(int jb, int g, const MT&) const { return p[(r16 << (3 - jb)) + g - 16]; }
};
// The word of slot t (slots from 240 on are not read), and its entry with the
// companion; every thread writes one, so that no branch is needed. One companion
// a thread costs nothing as the closer one of tw_uni, and its bound saves a reduction
// of half the words in every fourth stage.
template <typename W>
__device__ __forceinline__ W tw_lds_word(const W* __restrict__ tw, uint32_t t, uint32_t Rr) {
  const uint32_t j = t < 240 ? t + 16 : 16, s = 27 - __builtin_clz(j);      // floor(log2 j) - 4
  return tw[(Rr << (4 + s)) + j - (16u << s)];
}
template <int KIND, typename W, typename MT>
__device__ __forceinline__ void tw_lds_put(Tw<W>* table, W w, uint32_t t, const MT& M) {
  table[t] = tw_uni<KIND>(w, M);
}

// Forward (CT) stages pairing register bits [JLO, JHI), largest first, on the
// registers of NX operands x[0..NX) that share every twiddle (and its
// companion). tw = psi_br of this limb; words below B on entry, below
// ct_bound(B, JHI - JLO) on return.
template <int EB, int JLO, int JHI, int KIND, bool UNI, int B, int NX, typename W, typename TW, typename MT>
__device__ __forceinline__ void fwd_block(W (&x)[NX][1 << EB], const TW& tw, const MT& M) {
  int bound = B;
#pragma unroll
  for (int jb = JHI - 1; jb >= JLO; --jb) {
    const CtStage st = ct_stage<W, KIND>(bound, UNI);
#pragma unroll
    for (int g = 0; g < (1 << (EB - 1 - jb)); ++g) {
      const Tw<W> xi = tw.template get<KIND, UNI>(jb, g, M);
#pragma unroll
      for (int i = 0; i < NX; ++i) {
#pragma unroll
        for (int s = 0; s < (1 << jb); ++s) {
          const int j = (g << (jb + 1)) | s;
          ct_lazy<KIND>(x[i][j], x[i][j | (1 << jb)], xi, st.red, st.k, M);
        }
      }
    }
    bound = st.out;
    if (EB == 4) stage_fence();
  }
}

// Inverse (GS) stages pairing register bits [JLO, JHI), smallest first, on
// words below BIN (<= LazyRule::GIN); words below GIN on return. LAST: the block
// ends with the row's top stride, whose stage also scales by 2^-lg, the inverse
// of the transform's length (1/N of Eq. 2 as one factor, no halving in the
// butterflies).
template <int EB, int JLO, int JHI, int KIND, bool UNI, int BIN, bool LAST, typename W, typename TW, typename MT>
__device__ __forceinline__ void inv_block(W (&x)[1 << EB], const TW& tw, uint32_t lg, const MT& M) {
  GsBounds<W, KIND, 1 << EB> B(BIN);
#pragma unroll
  for (int jb = JLO; jb < JHI; ++jb) {
#pragma unroll
    for (int g = 0; g < (1 << (EB - 1 - jb)); ++g) {
      if (LAST && jb == JHI - 1) {
        const W xi = tw.raw(jb, g);
        const W c = inv_pow2<W>(lg, M);
        const Tw<W> tc = tw_uni<KIND>(c, M), tcw = tw_make<KIND, UNI>(mulmod<KIND>(xi, c, M), M);
#pragma unroll
        for (int s = 0; s < (1 << jb); ++s)
          gs_lazy_scaled<KIND>(x[s], x[s | (1 << jb)], tc, tcw, ceil_q(B.b[s | (1 << jb)]), M);
      } else {
        const Tw<W> tx = tw.template get<KIND, UNI>(jb, g, M);
#pragma unroll
        for (int s = 0; s < (1 << jb); ++s) {
          const int j = (g << (jb + 1)) | s;
          gs_track<KIND>(x, B, j, j | (1 << jb), tx, UNI, M);
        }
      }
    }
    if (EB == 4) stage_fence();
  }
}

// Register bits [JLO, JHI) of round RHO's stages when the TR smallest strides
// are left out.
template <int GEO, int RHO, int TR>
struct Round {
  using G = RowGeom<GEO>;
  static constexpr int P = G::p(RHO), JHI = G::hi(RHO) - P, JLO = JHI - round_stages<GEO, RHO, TR>();
  // companions short by less than two (tw_uni): the scalar unit's and the table's
  static constexpr bool UNI = uniform_round<GEO, RHO>() || (G::TW_LDS && RHO == 1);
  template <typename TW, typename W>
  static __device__ __forceinline__ TW twiddles(uint32_t t, const W* __restrict__ tw, uint32_t Rr) {
    return TW(tw, round_block<GEO>(t, Rr, P), JLO, JHI);
  }
};

// Twiddle sources of a row transform's rounds, get<RHO>() called before the exchange that
// precedes round RHO.
// RowTwAll (4 words per thread, calls bound by latency): every round's twiddles
// (three per thread and round) loaded when the kernel starts, beside its data.
template <int GEO, int TR, typename W>
struct RowTwAll {
  using G = RowGeom<GEO>;
  using TW = TwRegs<G::EB, W>;
  TW r[G::NR];
  template <int RHO>
  __device__ __forceinline__ void load(uint32_t t, const W* __restrict__ tw, uint32_t Rr) {
    r[RHO] = Round<GEO, RHO, TR>::template twiddles<TW>(t, tw, Rr);
    if constexpr (RHO + 1 < G::NR) load<RHO + 1>(t, tw, Rr);
  }
  __device__ __forceinline__ RowTwAll(uint32_t t, const W* __restrict__ tw, uint32_t Rr, const Tw<W>*) {
    load<0>(t, tw, Rr);
  }
  template <int RHO>
  __device__ __forceinline__ const TW& get() const { return r[RHO]; }
};
// RowTwRound (16 words per thread): a round's at a time; NX = 1: ahead of the
// round (TwRegs), NX = 2: each as its stage comes up (TwMem).
template <int GEO, int TR, int NX, typename W>
struct RowTwRound {
  using G = RowGeom<GEO>;
  uint32_t t, Rr;
  const W* __restrict__ tw;
  const Tw<W>* table;         // round 1's twiddles in LDS (RowGeom::TW_LDS)
  __device__ __forceinline__ RowTwRound(uint32_t t_, const W* __restrict__ tw_, uint32_t Rr_, const Tw<W>* table_)
      : t(t_), Rr(Rr_), tw(tw_), table(table_) {}
  template <int RHO>
  __device__ __forceinline__ auto get() const {
    if constexpr (G::TW_LDS && RHO == 1) return TwLds<W>{table, 16 + (t >> 4)};
    else return get_mem<RHO>();
  }
  template <int RHO>
  __device__ __forceinline__ auto get_mem() const {
    using TW = typename std::conditional<NX == 1 && !uniform_round<GEO, RHO>(), TwRegs<G::EB, W>, TwMem<G::EB, W>>::type;
    return Round<GEO, RHO, TR>::template twiddles<TW>(t, tw, Rr);
  }
};
template <int GEO, int TR, int NX, typename W>
using RowTw = typename std::conditional<RowGeom<GEO>::EBX == 2 && (RowGeom<GEO>::NR > 1), RowTwAll<GEO, TR, W>,
                                        RowTwRound<GEO, TR, NX, W>>::type;

// LDS exchanges only run for rows of at least two rounds, where every round's
// register bits are EB = EBX wide; a single-round row (c <= EBX) has P = 0
// and one thread per row, so its global accesses use t << EB directly.
template <int GEO, int RHO, typename W>
__device__ __forceinline__ void lds_put(W* lds, const W (&x)[RowGeom<GEO>::E], uint32_t t) {
  using G = RowGeom<GEO>;
  constexpr int P = G::p(RHO);
  W* b = lds + lds_base<P, G::EB>(t);
#pragma unroll
  for (int j = 0; j < G::E; ++j) b[lds_off<P>(j)] = x[j];
}

template <int GEO, int RHO, typename W>
__device__ __forceinline__ void lds_get(const W* lds, W (&x)[RowGeom<GEO>::E], uint32_t t) {
  using G = RowGeom<GEO>;
  constexpr int P = G::p(RHO);
  const W* b = lds + lds_base<P, G::EB>(t);
#pragma unroll
  for (int j = 0; j < G::E; ++j) x[j] = b[lds_off<P>(j)];
}

// Where the words of a row are: next to each other, or (coefficient-major
// batches) `step` words apart, `lane` words from a start that is the same for the
// whole workgroup.
struct Unit {
  static constexpr uint32_t step = 1, lane = 0;
  template <typename W>
  __device__ __forceinline__ W* at(W* row, uint32_t i) const { return row + i; }
};
struct Strided {
  uint32_t step, lane;
  // word i of the row as a scalar address (opaque: the compiler would walk
  // from word to word in vector registers and keep the addresses of the loads
  // for the stores, 32 registers)
  template <typename W>
  __device__ __forceinline__ W* at(W* row, uint32_t i) const { return row + opaque_s(i * step); }
};

template <int GEO, int RHO, typename W, typename S>
__device__ __forceinline__ void gmem_get(const W* __restrict__ row, W (&x)[RowGeom<GEO>::E], uint32_t t, S s) {
  using G = RowGeom<GEO>;
  constexpr int P = G::p(RHO);
  const uint32_t tb = ((G::NR > 1) ? row_base<P, G::EB>(t) : (t << G::EB)) * s.step + s.lane;
#pragma unroll
  for (int j = 0; j < G::E; ++j) x[j] = s.at(row, j << P)[tb];
}

template <int GEO, int RHO, typename W, typename S>
__device__ __forceinline__ void gmem_put(W* __restrict__ row, const W (&x)[RowGeom<GEO>::E], uint32_t t, S s) {
  using G = RowGeom<GEO>;
  constexpr int P = G::p(RHO);
  const uint32_t tb = ((G::NR > 1) ? row_base<P, G::EB>(t) : (t << G::EB)) * s.step + s.lane;
#pragma unroll
  for (int j = 0; j < G::E; ++j) s.at(row, j << P)[tb] = x[j];
}

// Move registers from round FROM's layout to round TO's layout through LDS.
// All threads of the workgroup must call it (it holds two barriers).
template <int GEO, int FROM, int TO, typename W>
__device__ __forceinline__ void exchange(W* lds, W (&x)[RowGeom<GEO>::E], uint32_t t) {
  __syncthreads();
#if PM_POISON_LDS
  // Debug build: fill the row's LDS with words above every modulus before
  // each exchange, so a slot read without being written in this exchange (a
  // missing barrier or an indexing error) corrupts the result.
  for (uint32_t i = t; i < (uint32_t)RowGeom<GEO>::LDS_ROW; i += RowGeom<GEO>::T) lds[i] = ~(W)0;
  __syncthreads();
#endif
  lds_put<GEO, FROM>(lds, x, t);
  __syncthreads();
  lds_get<GEO, TO>(lds, x, t);
}

// All row stages of the forward transform of NX rows that share a twiddle row,
// without the stages of the TR smallest strides (the last of Alg. 5): rounds
// RHO..NR-1. Words below B on entry (at most LazyRule::H); on return x holds the
// rows in the last round's layout (E consecutive words per thread), below H.
template <int GEO, int KIND, int TR, int B, int RHO = 0, int NX, typename W, typename TW, typename MT>
__device__ __forceinline__ void fwd_rounds(W* lds, W (&x)[NX][RowGeom<GEO>::E], uint32_t t, const TW& tws,
                                           const MT& M) {
  using G = RowGeom<GEO>;
  using R = Round<GEO, RHO, TR>;
  const auto tr = tws.template get<RHO>();
  if constexpr (RHO > 0) {
#pragma unroll
    for (int i = 0; i < NX; ++i) exchange<GEO, RHO - 1, RHO>(lds, x[i], t);
  }
  fwd_block<G::EB, R::JLO, R::JHI, KIND, R::UNI, B>(x, tr, M);
  if constexpr (RHO + 1 < G::NR)
    fwd_rounds<GEO, KIND, TR, ct_bound<W, KIND>(B, R::JHI - R::JLO, R::UNI), RHO + 1>(lds, x, t, tws, M);
}

// All row stages of the inverse transform without those of the TR smallest
// strides (the first of Alg. 6), from the last round's layout back to round
// 0's layout, scaled by 2^-lg: rounds RHO..0. Words below BIN on entry, below GIN
// on return.
template <int GEO, int KIND, int TR, int BIN, int RHO = RowGeom<GEO>::NR - 1, typename W, typename TW, typename MT>
__device__ __forceinline__ void inv_rounds(W* lds, W (&x)[RowGeom<GEO>::E], uint32_t t, const TW& tws, uint32_t lg,
                                           const MT& M) {
  static_assert(BIN <= LazyRule<W, KIND>::GIN, "inverse input bound");
  using G = RowGeom<GEO>;
  using R = Round<GEO, RHO, TR>;
  const auto tr = tws.template get<RHO>();
  if constexpr (RHO + 1 < G::NR) exchange<GEO, RHO + 1, RHO>(lds, x, t);
  inv_block<G::EB, R::JLO, R::JHI, KIND, R::UNI, BIN, RHO == 0>(x, tr, lg, M);
  if constexpr (RHO > 0) inv_rounds<GEO, KIND, TR, LazyRule<W, KIND>::GIN, RHO - 1>(lds, x, t, tws, lg, M);
}

// Product of the truncated rows (TR = 2): with the strides 2 and 1 left out, four
// neighbouring words are a residue modulo x^4 - g, and residues are multiplied
// as polynomials of degree 3 (the paper's fused product, Sec. III-B, does the same with
// one stage left out, residues modulo x^2 - alpha^2). g is the square of the
// stride-2 twiddle, which is the stride-4 twiddle of the same words up to a
// sign: block i of the polynomial has g = (-1)^i psi_br[N/8 + i/2], a word the
// thread has used two stages before. 16 plain products and four reductions
// replace two stages of three transforms, four reduced products and the twelve
// twiddles a thread of 16 words reads for the last two stages: for the
// rows of 2^12 words 6,310 -> 6,010 VALU instructions a thread (260 a block).
// x = x y for the E consecutive words of a thread (last round's layout), rows of
// at least 8 words; products below LazyRule::B4.
template <int GEO, typename W>
struct Blk4Tw {
  using G = RowGeom<GEO>;
  static_assert(G::LC >= 3 && G::E >= 4, "blocks of four words in rows of at least eight");
  W v[(G::E + 7) / 8];
  __device__ __forceinline__ Blk4Tw(uint32_t t, const W* __restrict__ tw, uint32_t Rr) {
    const uint32_t base = Rr * (1u << (G::LC - 3)) + ((t << G::EB) >> 3);
#pragma unroll
    for (int i = 0; i < (G::E + 7) / 8; ++i) v[i] = tw[base + i];
  }
};
template <int GEO, int KIND, typename W, typename MT>
__device__ __forceinline__ void blk4_mul(W (&x)[RowGeom<GEO>::E], const W (&y)[RowGeom<GEO>::E],
                                         const Blk4Tw<GEO, W>& gs, uint32_t t, const MT& M) {
  using G = RowGeom<GEO>;
#pragma unroll
  for (int j = 0; j < G::E; j += 4) {
    const Tw<W> g = tw_vec<KIND>(gs.v[j >> 3], M);
    const bool neg = G::E >= 8 ? (j & 4) != 0 : (t & 1) != 0;
    W a[4] = {x[j], x[j + 1], x[j + 2], x[j + 3]}, b[4] = {y[j], y[j + 1], y[j + 2], y[j + 3]};
    mul_mod_x4<KIND>(a, b, g, neg, M);
#pragma unroll
    for (int i = 0; i < 4; ++i) x[j + i] = a[i];
    if (G::EB == 4) stage_fence();         // registers: one block at a time
  }
}

// A radix-2^LOGR block of stages at any depth of Alg. 5 / Alg. 6, its 2^LOGR
// words in registers. A block of stages s0..s0+LOGR-1 touches 2^LOGR words at
// stride N >> (s0+LOGR) that share the index bits above bit log2(N) - s0; with
// h those high bits and rb = 2^s0 + h, stage s0+j's group g (within the block)
// uses the twiddle at (rb << j) + g. UNI: rb is the same for the whole
// workgroup. Words below B on entry, below ct_bound(B, LOGR) on return. TR: without
// the block's TR smallest strides.
template <int LOGR, int KIND, bool UNI, int B, int TR = 0, int LM = 0, typename W, typename MT>
__device__ __forceinline__ void blk_fwd(W (&x)[1 << LOGR], const W* __restrict__ tw, uint32_t rb, const MT& M) {
  constexpr int m = 1 << LM, k = (1 << LOGR) >> (LM + 1);
  constexpr CtStage st = ct_stage<W, KIND>(B, UNI);
  const W* t = tw + (rb << LM);
#pragma unroll
  for (int g = 0; g < m; ++g) {
    const Tw<W> xi = tw_make<KIND, UNI>(t[g], M);
#pragma unroll
    for (int s = 0; s < k; ++s) ct_lazy<KIND>(x[2 * g * k + s], x[2 * g * k + s + k], xi, st.red, st.k, M);
    if (LOGR >= 5) stage_fence();      // registers: no butterflies of the next group ahead
  }
  if constexpr (LM + 1 < LOGR - TR) blk_fwd<LOGR, KIND, UNI, st.out, TR, LM + 1>(x, tw, rb, M);
}

// Inverse block on words with the bounds B (at most GIN on entry and on return).
// SCALE: its last stage is the transform's last and scales by 2^-lg.
template <int LOGR, int KIND, bool UNI, bool SCALE, int LM, typename W, typename MT>
__device__ __forceinline__ void blk_inv_stage(W (&x)[1 << LOGR], GsBounds<W, KIND, 1 << LOGR>& B,
                                              const W* __restrict__ tw, uint32_t rb, uint32_t lg, const MT& M) {
  constexpr int m = 1 << LM, k = (1 << LOGR) >> (LM + 1);
  const W* t = tw + (rb << LM);
  if constexpr (LM == 0 && SCALE) {
    const W c = inv_pow2<W>(lg, M);
    const Tw<W> tc = tw_uni<KIND>(c, M), tcw = tw_make<KIND, UNI>(mulmod<KIND>(t[0], c, M), M);
#pragma unroll
    for (int s = 0; s < k; ++s) gs_lazy_scaled<KIND>(x[s], x[s + k], tc, tcw, ceil_q(B.b[s + k]), M);
  } else {
#pragma unroll
    for (int g = 0; g < m; ++g) {
      const Tw<W> tx = tw_make<KIND, UNI>(t[g], M);
#pragma unroll
      for (int s = 0; s < k; ++s) gs_track<KIND>(x, B, 2 * g * k + s, 2 * g * k + s + k, tx, UNI, M);
      if (LOGR >= 5) stage_fence();
    }
  }
  if constexpr (LM > 0) blk_inv_stage<LOGR, KIND, UNI, SCALE, LM - 1>(x, B, tw, rb, lg, M);
}
template <int LOGR, int KIND, bool UNI, int BIN, bool SCALE, int TR = 0, typename W, typename MT>
__device__ __forceinline__ void blk_inv(W (&x)[1 << LOGR], const W* __restrict__ tw, uint32_t rb, uint32_t lg,
                                        const MT& M) {
  GsBounds<W, KIND, 1 << LOGR> B(BIN);
  blk_inv_stage<LOGR, KIND, UNI, SCALE, LOGR - 1 - TR>(x, B, tw, rb, lg, M);
}

// x = x y for a block that ends with stride 1 (forward stages but TR done), words
// J and up: modulo x^4 - g as blk4_mul (TR = 2), or pointwise. Recursive: the
// largest block's loop is beyond what the compiler unrolls.
template <int LOGR, int KIND, bool UNI, int TR, int J = 0, typename W, typename MT>
__device__ __forceinline__ void blk_mul(W (&x)[1 << LOGR], const W (&y)[1 << LOGR], const W* __restrict__ tw,
                                        uint32_t rb, const MT& M) {
  if constexpr (TR == 2) {
    static_assert(LOGR >= 3, "a stage of stride 4 in the block");
    const Tw<W> g = tw_make<KIND, UNI>(tw[(rb << (LOGR - 3)) + (J >> 3)], M);
    W a[4] = {x[J], x[J + 1], x[J + 2], x[J + 3]}, b[4] = {y[J], y[J + 1], y[J + 2], y[J + 3]};
    mul_mod_x4<KIND>(a, b, g, (J & 4) != 0, M);
#pragma unroll
    for (int i = 0; i < 4; ++i) x[J + i] = a[i];
    stage_fence();
    if constexpr (J + 4 < (1 << LOGR)) blk_mul<LOGR, KIND, UNI, TR, J + 4>(x, y, tw, rb, M);
  } else {
    x[J] = mul_lazy<KIND>(x[J], y[J], M);
    if constexpr (J + 1 < (1 << LOGR)) blk_mul<LOGR, KIND, UNI, TR, J + 1>(x, y, tw, rb, M);
  }
}

// Column pass: the R = 2^LOGR words of one column (stride C) in registers, the
// block at depth 0. Forward: canonical words in, below H out (the row pass
// reduces them). Inverse: the row pass's words (below GIN, already scaled by
// 1/N) in, canonical words out.
template <int LOGR, int KIND, typename W, typename MT>
__device__ __forceinline__ void col_fwd(W (&x)[1 << LOGR], const W* __restrict__ tw, const MT& M) {
  blk_fwd<LOGR, KIND, true, Q1>(x, tw, 1, M);
}

template <int LOGR, int KIND, typename W, typename MT>
__device__ __forceinline__ void col_inv(W (&x)[1 << LOGR], const W* __restrict__ tw, const MT& M) {
  blk_inv<LOGR, KIND, true, LazyRule<W, KIND>::GIN, false>(x, tw, 1, 0, M);
  canon_all<KIND>(x, M);
}

// Bound on the words that a forward column pass of 2^LOGR rows leaves (LOGR = 0:
// none, canonical words): col_bound for the forms here (col_fwd, col32_fwd_pair),
// colq_bound for k_colq, whose companions are all tw_vec's. For 64-bit KIND_WIDE
// and LOGR = 2, 3, 4 the second is the larger: 160, 256, 144 against 144, 224, 112.
template <int LOGR, int KIND, typename W>
constexpr int colq_bound() { return ct_bound<W, KIND>(Q1, LOGR, false); }
template <int LOGR, int KIND, typename W>
constexpr int col_bound() {
  constexpr int one = ct_bound<W, KIND>(Q1, LOGR, true);
  if (LOGR != 5) return one;
  constexpr int pair = ct_bound<W, KIND>(ct_stage<W, KIND>(Q1, true).out, 4, false);
  return one > pair ? one : pair;
}

// Exchange between the two halves of a wave (v_permlane32_swap, gfx950).
// Afterwards lanes 32..63 hold in p what lanes 0..31 held in q, and lanes
// 0..31 hold in q what lanes 32..63 held in p; lanes 0..31 keep p and lanes
// 32..63 keep q. Every lane of the wave must be active.
__device__ __forceinline__ void half_swap(uint32_t& p, uint32_t& q) {
  const auto r = __builtin_amdgcn_permlane32_swap(p, q, false, false);
  p = r[0];
  q = r[1];
}

__device__ __forceinline__ void half_swap(uint64_t& p, uint64_t& q) {
  uint32_t p0 = lo32(p), p1 = hi32(p), q0 = lo32(q), q1 = hi32(q);
  half_swap(p0, q0);
  half_swap(p1, q1);
  p = pack64(p0, p1);
  q = pack64(q0, q1);
}

// Column pass of R = 32 words held by the lanes l and l + 32 of one wave
// (h = 0 and 1), 16 words each. The first stage of Alg. 5 (stride 16 rows)
// pairs row i with row i + 16, so half h starts with rows
// col32_split_row(j, h) = (j & 7) + 8h + 16 (j >> 3) in y[j]: y[k] and y[8+k]
// are the pairs of that stage. One exchange of eight words (y[8+k] of h = 0
// with y[k] of h = 1) then leaves half h with rows 16h + j in y[j], the block
// of rows whose last four column stages use the twiddles of blk_fwd with
// rb = 2 + h. The inverse (Alg. 6) runs the same steps in reverse
// order: the block's four stages, the same exchange, then the stride-16 stage.
__device__ __forceinline__ uint32_t col32_split_row(int j, uint32_t h) { return (j & 7) + 8 * h + 16 * (j >> 3); }
__device__ __forceinline__ uint32_t col32_block_row(int j, uint32_t h) { return 16 * h + j; }

template <int KIND, typename W, typename MT>
__device__ __forceinline__ void col32_fwd_pair(W (&y)[16], const W* __restrict__ tw, uint32_t h, const MT& M) {
  constexpr CtStage st = ct_stage<W, KIND>(Q1, true);
  const Tw<W> xi = tw_uni<KIND>(tw[1], M);
#pragma unroll
  for (int k = 0; k < 8; ++k) ct_lazy<KIND>(y[k], y[8 + k], xi, st.red, st.k, M);
#pragma unroll
  for (int k = 0; k < 8; ++k) half_swap(y[k], y[8 + k]);
  blk_fwd<4, KIND, false, st.out>(y, tw, 2 + h, M);
}

template <int KIND, typename W, typename MT>
__device__ __forceinline__ void col32_inv_pair(W (&y)[16], const W* __restrict__ tw, uint32_t h, const MT& M) {
  constexpr int GIN = LazyRule<W, KIND>::GIN;
  blk_inv<4, KIND, false, GIN, false>(y, tw, 2 + h, 0, M);
#pragma unroll
  for (int k = 0; k < 8; ++k) half_swap(y[k], y[8 + k]);
  const Tw<W> xi = tw_uni<KIND>(tw[1], M);
#pragma unroll
  for (int k = 0; k < 8; ++k) gs_lazy<KIND>(y[k], y[8 + k], xi, ceil_q(GIN), M);
  canon_all<KIND>(y, M);
}

}  // namespace pm
