// Interleaved (coefficient-major) batch layout, the storage of the paper's
// throughput-optimised multi-block design (Sec. V-C): within a limb the batch
// is an N x P matrix with coefficient j of polynomial p at [j * P + p], so the
// lanes of a wave, which hold consecutive polynomials, read and write
// consecutive words at every stage.
//
// Each thread runs one radix-2^LOGR block of stages (blk_fwd / blk_inv) of one
// polynomial with its 2^LOGR words in registers; a transform is a short
// sequence of such passes over HBM. A block of stages s0..s0+LOGR-1 is one
// grid row (blockIdx.y), so its twiddles are uniform across the workgroup.
//
// Words between the passes of one transform are lazy (below LazyRule's H on the
// way forward, below GIN on the way back); the last pass of a transform or a product
// makes them canonical (LAST). The 1/N scaling is in the last stage of an
// inverse transform (SCALE) or of the product's middle.
//
//   IL_FWD  stages of Alg. 5 on one or two operands (A -> C, B -> D)
//   IL_INV  stages of Alg. 6 (A -> C)
//   IL_MUL  products of N <= 2^IL_MUL_MAXR, one block (A, B -> C); longer ones have
//           their middle in il_rows.hip
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ntt_device.hpp"
#include "pm_internal.hpp"

namespace pm {

// Waves per SIMD: a block of 2^6 words needs 128 VGPRs for its data (3 waves), the
// fused block of 2^5 words per operand as many (2 waves).
template <int LOGR, int MODE>
struct IlWaves {
  static constexpr int value = MODE == IL_MUL ? (LOGR == 5 ? 2 : 4) : (LOGR >= 5 ? 3 : 5);
};

template <int LOGR, int KIND, int MODE, bool LAST, bool SCALE>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu((IlWaves<LOGR, MODE>::value), 8)))
k_il(const uint64_t* A, const uint64_t* B, uint64_t* C, uint64_t* D, const uint64_t* __restrict__ twf,
     const uint64_t* __restrict__ twi, uint32_t log2n, uint32_t s0, uint32_t polys, uint32_t nops, LimbSet ls) {
  constexpr int R = 1 << LOGR;
  using L = LazyRule<uint64_t, KIND>;
  constexpr int H = L::H;
  const uint32_t p0 = blockIdx.x * blockDim.x;    // first polynomial of the workgroup
  const uint32_t lane = threadIdx.x;
  if (p0 + lane >= polys) return;
  const uint32_t limb = (MODE == IL_FWD) ? blockIdx.z / nops : blockIdx.z;
  const uint32_t op = (MODE == IL_FWD) ? blockIdx.z - limb * nops : 0;
  const uint32_t lk = log2n - s0 - LOGR;          // log2 of the block's stride
  const uint32_t h = blockIdx.y >> lk, lo = blockIdx.y & ((1u << lk) - 1);
  const size_t N = (size_t)1 << log2n;
  // everything but the lane index is uniform: word i of the block sits at
  // base + i * step + lane
  const size_t base = (size_t)limb * N * polys + ((((size_t)h << (log2n - s0)) | lo) * polys) + p0;
  const size_t step = ((size_t)polys) << lk;
  const uint32_t rb = (1u << s0) + h;
  const Mod M = ls.mod[limb];
  uint64_t x[R];
  if constexpr (MODE == IL_FWD) {
    const uint64_t* src = (op ? B : A) + base;
    uint64_t* dst = (op ? D : C) + base;
#pragma unroll
    for (int i = 0; i < R; ++i) x[i] = (src + i * step)[lane];
    blk_fwd<LOGR, KIND, true, H>(x, twf + (size_t)limb * N, rb, M);
    if (LAST) canon_all<KIND>(x, M);
#pragma unroll
    for (int i = 0; i < R; ++i) (dst + i * step)[lane] = x[i];
  } else if constexpr (MODE == IL_INV) {
    const uint64_t* src = A + base;
    uint64_t* dst = C + base;
#pragma unroll
    for (int i = 0; i < R; ++i) x[i] = (src + i * step)[lane];
    blk_inv<LOGR, KIND, true, L::GIN, SCALE>(x, twi + (size_t)limb * N, rb, log2n, M);
    if (LAST) canon_all<KIND>(x, M);
#pragma unroll
    for (int i = 0; i < R; ++i) (dst + i * step)[lane] = x[i];
  } else {
    constexpr int TR = LOGR >= 3 && KIND == KIND_WIDE ? 2 : 0;      // as product_in_blocks
    const uint64_t* tf = twf + (size_t)limb * N;
    const uint64_t* sa = A + base;
    const uint64_t* sb = B + base;
    uint64_t* dst = C + base;
#pragma unroll
    for (int i = 0; i < R; ++i) x[i] = (sa + i * step)[lane];
    blk_fwd<LOGR, KIND, true, H, TR>(x, tf, rb, M);
    uint64_t y[R];
#pragma unroll
    for (int i = 0; i < R; ++i) y[i] = (sb + i * step)[lane];
    blk_fwd<LOGR, KIND, true, H, TR>(y, tf, rb, M);
    blk_mul<LOGR, KIND, true, TR>(x, y, tf, rb, M);
    blk_inv<LOGR, KIND, true, TR == 2 ? L::B4 : L::PW, SCALE, TR>(x, twi + (size_t)limb * N, rb, log2n - TR, M);
    if (LAST) canon_all<KIND>(x, M);
#pragma unroll
    for (int i = 0; i < R; ++i) (dst + i * step)[lane] = x[i];
  }
}

template <int LOGR, int KIND, int MODE, bool LAST, bool SCALE>
static void il_launch(const IlArgs& a, hipStream_t s) {
  const uint32_t bs = a.polys >= 256 ? 256u : ((a.polys + 63) / 64) * 64;
  const uint32_t nz = (MODE == IL_FWD) ? a.limbs * a.nops : a.limbs;
  dim3 grid((a.polys + bs - 1) / bs, 1u << (a.log2n - LOGR), nz);
  hipLaunchKernelGGL((k_il<LOGR, KIND, MODE, LAST, SCALE>), grid, dim3(bs), 0, s, a.A, a.B, a.C, a.D, a.twf, a.twi,
                     a.log2n, a.s0, a.polys, a.nops, *a.ls);
}

template <int LOGR, int KIND>
static void il_launch_mode(const IlArgs& a, int mode, hipStream_t s) {
  const bool first = a.s0 == 0, last = a.s0 + LOGR == a.log2n;   // block of the first / last stages of Alg. 5
  if (mode == IL_FWD) {
    if (last) il_launch<LOGR, KIND, IL_FWD, true, false>(a, s);
    else il_launch<LOGR, KIND, IL_FWD, false, false>(a, s);
  } else if (mode == IL_INV) {
    if (!first) il_launch<LOGR, KIND, IL_INV, false, false>(a, s);
    else if (a.scale) il_launch<LOGR, KIND, IL_INV, true, true>(a, s);
    else il_launch<LOGR, KIND, IL_INV, true, false>(a, s);
  } else if constexpr (LOGR <= IL_MUL_MAXR) {
    il_launch<LOGR, KIND, IL_MUL, true, true>(a, s);
  }
}

template <int LOGR>
static void il_launch_kind(const IlArgs& a, int kind, int mode, hipStream_t s) {
  if (kind == KIND_WIDE) il_launch_mode<LOGR, KIND_WIDE>(a, mode, s);
  else il_launch_mode<LOGR, KIND_ANY>(a, mode, s);
}

hipError_t launch_il(int logr, int kind, int mode, const IlArgs& a, hipStream_t s) {
  if (logr < 1 || logr > IL_MAXR || a.s0 + (uint32_t)logr > a.log2n) return hipErrorInvalidValue;
  if (mode == IL_MUL && (logr > IL_MUL_MAXR || (uint32_t)logr != a.log2n)) return hipErrorInvalidValue;
  switch (logr) {
    case 1: il_launch_kind<1>(a, kind, mode, s); break;
    case 2: il_launch_kind<2>(a, kind, mode, s); break;
    case 3: il_launch_kind<3>(a, kind, mode, s); break;
    case 4: il_launch_kind<4>(a, kind, mode, s); break;
    case 5: il_launch_kind<5>(a, kind, mode, s); break;
    default: il_launch_kind<6>(a, kind, mode, s); break;
  }
  return hipGetLastError();
}

}  // namespace pm
