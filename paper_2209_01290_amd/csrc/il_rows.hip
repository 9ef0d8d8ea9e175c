// Coefficient-major batches (see il_kernels.hip), LC stages in one pass: the last
// ones of Alg. 5, the first ones of Alg. 6, or both around the pointwise product
// (the product's middle), as the row pass of the [poly][N] layout does them (row_task),
// for 16 polynomials per workgroup. Lane groups of 16 hold the same word of 16
// neighbouring polynomials (whole 128-byte lines); the polynomials' LDS rows are one
// word apart from a multiple of the banks, so that those 16 lanes hit 16 different
// pairs of banks. All 16 use one row's twiddles: round 0's are uniform.
//
// It takes 6 to 10 stages where a register block takes up to 6 (2 x 5 for the
// product): products of N = 2^12 pass over memory as 4 + 8 + 4 stages, 9 operand batches
// instead of 15, transforms of 2^13..2^15 in two passes instead of three. N = 2^12 x 999,
// products: 102 -> 88 us, of which the row pass 46 (98 MB: 15 at the memory's
// rate; it is bound by its instructions as the rows of the other layout are);
// N = 2^14 x 600, products: 306 -> 237; transforms of N = 2^13 x 4096: 255 -> 203.
//
// grid: x = 16 polynomials, y = row of 2^LC coefficients, z = limb.
#include "ntt_row.hpp"
#include "pm_internal.hpp"

namespace pm {
namespace {

constexpr int ILP = 16;         // polynomials per workgroup

template <int LC, int KIND, int MODE>
__global__ void __launch_bounds__(ILP * RowGeom<LC>::T) __attribute__((amdgpu_waves_per_eu(4, 8)))
k_il_row(const uint64_t* A, const uint64_t* B, uint64_t* C, const uint64_t* twf, const uint64_t* twi, uint32_t log2n,
         uint32_t polys, LimbSet ls) {
  constexpr int GEO = LC | ROW_GEO_SAME;
  using G = RowGeom<GEO>;
  static_assert(!G::TW_LDS, "the row's LDS holds the row alone");
  __shared__ alignas(16) uint64_t lds[ILP * (G::LDS_ROW + 1)];
  const uint32_t sub = threadIdx.x % ILP, t = threadIdx.x / ILP;
  const uint32_t limb = blockIdx.z, r = blockIdx.y;
  const bool active = blockIdx.x * ILP + sub < polys;
  const size_t N = (size_t)1 << log2n;
  const size_t off = ((size_t)limb * N + ((size_t)r << LC)) * polys + blockIdx.x * ILP;
  const uint32_t R = 1u << (log2n - LC);
  const Mod M = ls.mod[limb];
  row_task<GEO, KIND, MODE>(A + off, B + off, C + off, twf + (size_t)limb * N, twi + (size_t)limb * N, R + r, active,
                              R == 1, log2n, M, lds + sub * (G::LDS_ROW + 1), t, Strided{polys, sub});
}

template <int LC, int KIND, int MODE>
void il_row_launch(const IlArgs& a, hipStream_t s) {
  dim3 grid((a.polys + ILP - 1) / ILP, 1u << (a.log2n - LC), a.limbs), block(ILP * RowGeom<LC>::T);
  hipLaunchKernelGGL((k_il_row<LC, KIND, MODE>), grid, block, 0, s, a.A, a.B, a.C, a.twf, a.twi, a.log2n, a.polys, *a.ls);
}

template <int LC, int KIND>
void il_row_mode(int mode, const IlArgs& a, hipStream_t s) {
  if (mode == IL_FWD) il_row_launch<LC, KIND, ROW_FWD>(a, s);
  else if (mode == IL_INV) il_row_launch<LC, KIND, ROW_INV>(a, s);
  else il_row_launch<LC, KIND, ROW_MUL>(a, s);
}

template <int LC>
void il_row_kind(int kind, int mode, const IlArgs& a, hipStream_t s) {
  if (kind == KIND_WIDE) il_row_mode<LC, KIND_WIDE>(mode, a, s);
  else il_row_mode<LC, KIND_ANY>(mode, a, s);
}

}  // namespace

hipError_t launch_il_row(int logc, int kind, int mode, const IlArgs& a, hipStream_t s) {
  if (logc < IL_ROW_MIN || logc > IL_ROW_MAX || (uint32_t)logc > a.log2n) return hipErrorInvalidValue;
  switch (logc) {
    case 6: il_row_kind<6>(kind, mode, a, s); break;
    case 7: il_row_kind<7>(kind, mode, a, s); break;
    case 8: il_row_kind<8>(kind, mode, a, s); break;
    case 9: il_row_kind<9>(kind, mode, a, s); break;
    default: il_row_kind<10>(kind, mode, a, s); break;
  }
  return hipGetLastError();
}

}  // namespace pm
