// Lazily reduced modular arithmetic of the transforms' butterflies, on both
// word types. The butterflies work on representatives that may exceed q: a
// word stands for its residue and is only known to be below B q for a bound B
// that the code tracks at compile time. Canonical words come back at the end
// of a transform (canon), so results are the same words as with a full
// reduction in every butterfly.
//
// Twiddle products use a precomputed quotient (Shoup's method): for a twiddle
// w with companion p ~ w 2^64 / q, k = hi64(v p) is v w / q up to a small
// deficit, and v w - k q needs the low 64 bits of both products only. Alg. 4
// costs 22 VALU instructions a product, this 11, and the product accumulates
// onto u, so u + v w costs no addition. The caller's tables hold w alone; p is
// computed in the kernel from the modulus' Barrett constant: on the scalar
// unit where the twiddle is uniform over the workgroup (tw_uni), else in
// the lanes (tw_vec, 6 instructions, once for all butterflies that share the
// twiddle).
//
// The quotient drops what does not fit the cheap instruction sequence, so it
// may fall short of v w / q. With d the companion's deficit, for v < V q
//   v w - k q < (3 + d V / H) q,   H q <= 2^64 the headroom,
// three for the dropped fractions of the 64 x 64 high product (two cross
// products rounded down one by one, the low product left out).
//
// What bounds it: the transforms' rows are bound by VALU issue (97 % of the
// rate their instruction mix allows), so time follows the instruction count
// weighted by issue rate: 14 instructions for a CT butterfly and 15 for a GS one
// plus about 1.3 to 2 for reductions, against 32 and 40.8 with Alg. 4 and full
// reductions in every butterfly. The product rows of N = 2^16 x 384 (6144 rows
// of 2^12 words) went from 0.447 to 0.27 ms, 11,116 to 5,700 VALU instructions
// a thread (the products modulo x^4 - g below among them). Under them the clock
// falls to 2.15 of 2.4 GHz (the power limit).
//
// Two rules per word type (LazyRule<W, KIND>); bounds are in sixteenths of q:
//   64-bit, KIND_WIDE (34 <= len(q) <= 60): H = 16; words may grow over several
//     stages before one operand is reduced (red2).
//   64-bit KIND_ANY (any len(q) <= 62) and 32-bit words (len(q) <= 30): H = 4,
//     quotients exact up to one, products < 2 q (Harvey's butterflies), one
//     conditional subtraction a stage.
#pragma once
#include "modarith.hpp"
#include "modarith32.hpp"

namespace pm {

constexpr int Q1 = 16;                       // one q in bound units

template <typename W, int KIND>
struct LazyRule {                            // H = 4
  static constexpr int H = 4 * Q1;
  static constexpr int GIN = 2 * Q1;         // bound on the words between two inverse rounds
  static constexpr int PW = 2 * Q1;          // bound on pointwise products
  static constexpr int B4 = 2 * Q1;          // bound on the products modulo x^4 - g
  static constexpr int rmax(int, bool) { return 2 * Q1; }
};
template <>
struct LazyRule<uint64_t, KIND_WIDE> {
  static constexpr int H = 16 * Q1;
  static constexpr int GIN = 8 * Q1;
  static constexpr int PW = 72;
  static constexpr int B4 = 6 * Q1;
  // bound on a twiddle product of a word below v: companion deficit < 2
  // (tw_uni) or < 4 (tw_vec)
  static constexpr int rmax(int v, bool uni) { return 3 * Q1 + ((uni ? 2 : 4) * v + 15) / 16; }
};
constexpr int ceil_q(int b) { return (b + Q1 - 1) / Q1; }
// What the stages rely on: after a reduction a CT butterfly's sum and difference fit H;
// a GS butterfly on words below GIN fits H, and its product and every word that enters
// the inverse rounds is below GIN again.
template <typename W, int KIND>
constexpr bool rule_holds() {
  using L = LazyRule<W, KIND>;
  return 2 * Q1 + ceil_q(L::rmax(L::H, false)) * Q1 <= L::H && 2 * L::GIN <= L::H && L::rmax(L::H, false) <= L::GIN &&
         L::PW <= L::GIN && L::B4 <= L::GIN;
}
static_assert(rule_holds<uint64_t, 0>() && rule_holds<uint64_t, 1>() && rule_holds<uint32_t, 0>() &&
              rule_holds<uint32_t, 1>(), "KIND_WIDE, KIND_ANY");

// A twiddle and its companion.
template <typename W>
struct Tw { W w, p; };

// Scalar values the compiler must take as they are: a 64-bit subtraction or a
// zero-extension it would rebuild from their definition costs more than the
// multiply-add written here.
__device__ __forceinline__ uint32_t opaque_s(uint32_t x) { asm("" : "+s"(x)); return x; }
__device__ __forceinline__ uint64_t opaque_s(uint64_t x) { asm("" : "+s"(x)); return x; }
__device__ __forceinline__ uint64_t neg_q(const Mod& M) { return opaque_s(0 - M.q); }
// k q for a small constant k
template <typename W, typename MT>
__device__ __forceinline__ W mult_q(int k, const MT& M) { return opaque_s((W)((W)k * M.q)); }

// x + (h << 32), as one addition to the high word
__device__ __forceinline__ uint64_t add_high(uint64_t x, uint32_t h) {
  asm("" : "+v"(h));
  h += hi32(x);
  asm("" : "+v"(h));
  return pack64(lo32(x), h);
}

__device__ __forceinline__ int len_q(const Mod& M) { return 64 - __builtin_clzll(M.q); }

// ------------------------------------------------------------ 64-bit words --
// hi64(a b) up to a deficit < 3. The last term is added as a multiply by one,
// which needs no zero-extended register pair.
__device__ __forceinline__ uint64_t mulhi_low3(uint64_t a, uint64_t b) {
  const uint64_t x = (uint64_t)hi32(a) * hi32(b) + __umulhi(lo32(a), hi32(b));
  return (uint64_t)__umulhi(hi32(a), lo32(b)) * opaque_s(1u) + x;
}

// hi64(a b), exact.
__device__ __forceinline__ uint64_t mulhi_exact(uint64_t a, uint64_t b) {
  const uint64_t e = (uint64_t)lo32(a) * hi32(b) + __umulhi(lo32(a), lo32(b));
  const uint64_t f = (uint64_t)hi32(a) * lo32(b) + lo32(e);
  return (uint64_t)hi32(a) * hi32(b) + hi32(e) + hi32(f);
}

// a.b + c.d + e.f + g.h modulo 2^32 as four multiply-adds (the compiler would
// narrow them to three multiplies and two additions more).
__device__ __forceinline__ uint32_t cross4(uint64_t v, uint64_t w, uint64_t k, uint64_t nq) {
  uint64_t x, cc;
  asm("v_mad_u64_u32 %0, %1, %2, %3, 0\n\tv_mad_u64_u32 %0, %1, %4, %5, %0\n\t"
      "v_mad_u64_u32 %0, %1, %6, %7, %0\n\tv_mad_u64_u32 %0, %1, %8, %9, %0"
      : "=&v"(x), "=&s"(cc)
      : "v"(lo32(v)), "v"(hi32(w)), "v"(hi32(v)), "v"(lo32(w)), "v"(lo32(k)), "s"(hi32(nq)), "v"(hi32(k)),
        "s"(lo32(nq)));
  return lo32(x);
}

// acc + v w - k q modulo 2^64
__device__ __forceinline__ uint64_t fma_q(uint64_t v, uint64_t w, uint64_t k, uint64_t acc, const Mod& M) {
  const uint64_t nq = neg_q(M);
  uint64_t s = (uint64_t)lo32(v) * lo32(w) + acc;
  s = (uint64_t)lo32(k) * lo32(nq) + s;
  return add_high(s, cross4(v, w, k, nq));
}

// Companions. With ws = w 2^(64-m) and 2^(m+64)/q = 2^64 + M.ml (+ fraction):
// w 2^64/q = ws + ws M.ml / 2^64. tw_uni: deficit < 2; tw_vec: < 4 for
// KIND_WIDE. KIND_ANY: the exact floor in both (one correction).
template <int KIND>
__device__ __forceinline__ uint64_t companion(uint64_t w, bool uni, const Mod& M) {
  const uint64_t ws = w << (64 - len_q(M));
  if (KIND == KIND_WIDE) return ws + (uni ? mulhi_exact(ws, M.ml) : mulhi_low3(ws, M.ml));
  const uint64_t p = ws + mulhi_exact(ws, M.ml);
  return p + ((0 - p * M.q) >= M.q ? 1 : 0);      // remainder w 2^64 - p q < 2q
}

// u + v t.w mod q (mul_add_tw) and v t.w mod q: the product is below rmax(V) for v < V q.
template <int KIND>
__device__ __forceinline__ uint64_t mul_add_tw(uint64_t& u, uint64_t v, const Tw<uint64_t>& t, const Mod& M) {
  const uint64_t k = KIND == KIND_WIDE ? mulhi_low3(v, t.p) : mulhi_exact(v, t.p);
  return fma_q(v, t.w, k, u, M);
}
template <int KIND>
__device__ __forceinline__ uint64_t mul_tw(uint64_t v, const Tw<uint64_t>& t, const Mod& M) {
  uint64_t zero = 0;
  return mul_add_tw<KIND>(zero, v, t, M);
}

// x < H q -> below 2q. KIND_WIDE: k = hi32(x1 c) with x1 = x >> 32 and
// c = floor(2^64/q) = 2^64/q - f: x/q - k < x0/q + f x1/2^32 + 1 < 2, since
// f x1/2^32 < f 16q/2^64 <= 16/17 for len(q) = 60 and x0/q < 1/2 for len(q) = 34
// (each is below 2^-20 where the other is not small).
template <int KIND>
__device__ __forceinline__ uint64_t red2(uint64_t x, const Mod& M) {
  if (KIND != KIND_WIDE) return csub(x, 2 * M.q);
  const int m = len_q(M);
  const uint32_t c = (uint32_t)(((uint64_t)1 << (64 - m)) | (M.ml >> m));
  const uint64_t nq = neg_q(M);
  const uint32_t k = __umulhi(hi32(x), opaque_s(c));
  return add_high((uint64_t)k * lo32(nq) + x, k * hi32(nq));
}

// x < 2q -> canonical; x < H q -> canonical.
__device__ __forceinline__ uint64_t csub1(uint64_t x, const Mod& M) { return csub(x, M.q); }
template <int KIND>
__device__ __forceinline__ uint64_t canon(uint64_t x, const Mod& M) { return csub1(red2<KIND>(x, M), M); }

// Pointwise product of lazy words: Alg. 4's quotient without its correction.
// Operands are brought below 2q first; the product is below PW.
//   x < 4 q^2 < 2^(2m+2), c = x >> (m-2) < 2^(m+4) <= 2^64, mu = floor(2^(m+62)/q):
//   c mu / 2^64 falls short of x/q by less than 1/2 (bits below c) + 1 (mu),
//   mulhi_low3 by less than 3: r < 4.5 q.
template <int KIND>
__device__ __forceinline__ uint64_t mul_lazy2(uint64_t a, uint64_t b, const Mod& M) {   // operands < 2q
  const uint32_t a0 = lo32(a), a1 = hi32(a), b0 = lo32(b), b1 = hi32(b);
  const uint64_t P00 = (uint64_t)a0 * b0;
  const uint64_t mid = (uint64_t)a1 * b0 + (uint64_t)a0 * b1;
  const uint64_t P11 = (uint64_t)a1 * b1;
  unsigned cy1, cy2;
  const uint32_t x0 = lo32(P00);
  const uint32_t x1 = __builtin_addc(hi32(P00), lo32(mid), 0u, &cy1);
  const uint32_t x2 = __builtin_addc(lo32(P11), hi32(mid), cy1, &cy2);
  const uint32_t x3 = hi32(P11) + cy2;
  const uint64_t c = pack64(__builtin_amdgcn_alignbit(x2, x1, M.s1), __builtin_amdgcn_alignbit(x3, x2, M.s1));
  const uint64_t k = mulhi_low3(c, ((uint64_t)1 << 62) | (M.ml >> 2));
  const uint64_t nq = neg_q(M);
  return add_high((uint64_t)lo32(k) * lo32(nq) + pack64(x0, x1), lo32(k) * hi32(nq) + hi32(k) * lo32(nq));
}

template <int KIND>
__device__ __forceinline__ uint64_t mul_lazy(uint64_t a, uint64_t b, const Mod& M) {
  if (KIND == KIND_WIDE) return mul_lazy2<KIND>(red2<KIND>(a, M), red2<KIND>(b, M), M);
  return mulmod<KIND>(canon<KIND>(a, M), canon<KIND>(b, M), M);
}

// ------------------------------------------------------------ 32-bit words --
// Companion of ws = w 2^(32-m), 2^(m+32)/q = 2^32 + M.ml: deficit < 2. The
// product of v < 4q is below 2q: its quotient's deficit is 1 + d v/2^32 <= 2,
// for len(q) <= 29 (v < 2^31) as it is, for len(q) = 30 with the exact floor.
template <int KIND>
__device__ __forceinline__ uint32_t companion(uint32_t w, bool, const Mod32& M) {
  const uint32_t ws = w << (30 - M.s);           // s = m - 2
  const uint32_t p = ws + __umulhi(ws, M.ml);
  if (KIND == KIND_WIDE) return p;
  return p + ((0u - p * M.q) >= M.q ? 1u : 0u);
}

// v w - k q modulo 2^32 as two multiply-adds, which take 64-bit addends: only the
// low words matter, so the high ones are left as they come (opaque, or the compiler
// makes four 32-bit instructions of the two). The product rows of 2^12 words:
// 727 -> 679 in instructions weighted by issue rate, with mul_mod_x4's; products of
// N = 2^16 x 768: 438 -> 409 us.
__device__ __forceinline__ uint32_t sub_kq(uint64_t s, uint32_t v, const Tw<uint32_t>& t, const Mod32& M) {
  s = (uint64_t)__umulhi(v, t.p) * opaque_s(0u - M.q) + s;
  asm("" : "+v"(s));
  return lo32(s);
}
template <int KIND>
__device__ __forceinline__ uint32_t mul_tw(uint32_t v, const Tw<uint32_t>& t, const Mod32& M) {
  return sub_kq((uint64_t)v * t.w, v, t, M);
}
template <int KIND>
__device__ __forceinline__ uint32_t mul_add_tw(uint32_t& u, uint32_t v, const Tw<uint32_t>& t, const Mod32& M) {
  uint32_t h;
  asm volatile("" : "=v"(h));       // any word
  uint64_t p = pack64(u, h);
  asm("" : "+v"(p));
  u = lo32(p);
  uint64_t s = (uint64_t)v * t.w + p;
  asm("" : "+v"(s));
  return sub_kq(s, v, t, M);
}

template <int KIND>
__device__ __forceinline__ uint32_t red2(uint32_t x, const Mod32& M) { return min(x, x - 2 * M.q); }

__device__ __forceinline__ uint32_t csub1(uint32_t x, const Mod32& M) { return min(x, x - M.q); }
template <int KIND>
__device__ __forceinline__ uint32_t canon(uint32_t x, const Mod32& M) { return csub1(red2<KIND>(x, M), M); }

template <int KIND>
__device__ __forceinline__ uint32_t mul_lazy(uint32_t a, uint32_t b, const Mod32& M) {
  return mulmod<KIND>(canon<KIND>(a, M), canon<KIND>(b, M), M);
}

// -------------------------------------------------------------- butterflies --
template <int KIND, typename W, typename MT>
__device__ __forceinline__ Tw<W> tw_vec(W w, const MT& M) { return {w, companion<KIND>(w, false, M)}; }
template <int KIND, typename W, typename MT>
__device__ __forceinline__ Tw<W> tw_uni(W w, const MT& M) { return {w, companion<KIND>(w, true, M)}; }
template <int KIND, bool UNI, typename W, typename MT>
__device__ __forceinline__ Tw<W> tw_make(W w, const MT& M) { return UNI ? tw_uni<KIND>(w, M) : tw_vec<KIND>(w, M); }

// One CT stage on words below b: the product is below r; u is reduced first
// when b + K q would exceed the headroom (K q >= r keeps the difference >= 0).
struct CtStage { bool red; int k, out; };
template <typename W, int KIND>
constexpr CtStage ct_stage(int b, bool uni) {
  using L = LazyRule<W, KIND>;
  const int k = ceil_q(L::rmax(b, uni));
  const bool red = b + k * Q1 > L::H;
  return {red, k, (red ? 2 * Q1 : b) + k * Q1};
}
template <typename W, int KIND>
constexpr int ct_bound(int b, int stages, bool uni) {
  for (int i = 0; i < stages; ++i) b = ct_stage<W, KIND>(b, uni).out;
  return b;
}

// (u, v) -> (u + w v, u - w v + K q)
template <int KIND, typename W, typename MT>
__device__ __forceinline__ void ct_lazy(W& u, W& v, const Tw<W>& t, bool red, int k, const MT& M) {
  if (red) u = red2<KIND>(u, M);
  const W s = mul_add_tw<KIND>(u, v, t, M);
  v = ((u << 1) + mult_q<W>(k, M)) - s;
  u = s;
}

// (u, v) -> (u + v, w (u - v + K q)), v below K q
template <int KIND, typename W, typename MT>
__device__ __forceinline__ void gs_lazy(W& u, W& v, const Tw<W>& t, int k, const MT& M) {
  const W d = u + mult_q<W>(k, M) - v;
  u = u + v;
  v = mul_tw<KIND>(d, t, M);
}

// The last GS stage of a transform with the scaling by N^-1 folded in:
// (u, v) -> (c (u + v), c w (u - v)); c = 1/N, cw = w/N.
template <int KIND, typename W, typename MT>
__device__ __forceinline__ void gs_lazy_scaled(W& u, W& v, const Tw<W>& c, const Tw<W>& cw, int k, const MT& M) {
  const W d = u + mult_q<W>(k, M) - v;
  u = mul_tw<KIND>((W)(u + v), c, M);
  v = mul_tw<KIND>(d, cw, M);
}

// 2^-lg mod q for 2^lg | q - 1
template <typename W, typename MT>
__device__ __forceinline__ W inv_pow2(uint32_t lg, const MT& M) { return (W)(M.q - ((M.q - 1) >> lg)); }

// Bounds of E words through inverse stages, kept in a local array whose values
// fold to constants in the unrolled code.
template <typename W, int KIND, int E>
struct GsBounds {
  int b[E];
  __device__ __forceinline__ explicit GsBounds(int in) {
#pragma unroll
    for (int j = 0; j < E; ++j) b[j] = in;
  }
};

// Butterfly of registers i and j (stage twiddle t) with the bounds' upkeep:
// a sum above half the headroom is reduced (unless keep), so that the next
// stage's sum and difference fit.
template <int KIND, int E, typename W, typename MT>
__device__ __forceinline__ void gs_track(W (&x)[E], GsBounds<W, KIND, E>& B, int i, int j, const Tw<W>& t, bool uni,
                                         const MT& M) {
  using L = LazyRule<W, KIND>;
  const int k = ceil_q(B.b[j]), s = B.b[i] + B.b[j], d = B.b[i] + k * Q1;
  gs_lazy<KIND>(x[i], x[j], t, k, M);
  B.b[j] = L::rmax(d, uni);
  if (s > L::H / 2) {
    x[i] = red2<KIND>(x[i], M);
    B.b[i] = 2 * Q1;
  } else {
    B.b[i] = s;
  }
}

// ------------------------------------------------- products modulo x^4 - g --
// a = a b mod (x^4 - g) on polynomials of four coefficients, g = g.w or -g.w
// (neg). With z = g b (three twiddle products) every coefficient is a sum of four
// plain products, reduced once.

// 64-bit words, 34 <= len(q) <= 60. The operands are brought below 2q < 2^61 and split
// into 31 low and 30 high bits, so that the sums of partial products
// (4 x 2^62, 8 x 2^61, 4 x 2^60) fit 64 bits and need no carries.
struct Limbs { uint32_t lo, hi; };
__device__ __forceinline__ Limbs limbs31(uint64_t x) {
  return {lo32(x) & 0x7fffffffu, __builtin_amdgcn_alignbit(hi32(x), lo32(x), 31)};
}

// S = c0 + c1 2^31 + c2 2^62 < 16 q^2 to a word below 6q: c = S >> m < 16 q, and
// with 2^m/q = 1 + ml/2^64 the quotient c + hi64(c ml) falls short of S/q by
// less than 2 (bits below c) + 1 (ml) + 3 (mulhi_low3).
__device__ __forceinline__ uint64_t reduce_sum(uint64_t c0, uint64_t c1, uint64_t c2, const Mod& M) {
  const uint64_t u = c1 + (c0 >> 31);               // < 2^64: c1 < 2^64 - 3 2^33 + 8
  const uint64_t h = c2 + (u >> 31);                // S >> 62
  uint64_t s = (uint64_t)lo32(c1) * opaque_s(0x80000000u) + c0;      // S modulo 2^64
  s = add_high(s, (hi32(c1) << 31) + (lo32(c2) << 30));
  const uint64_t h2 = h >> 2;                       // S >> 64
  const uint32_t sh = (uint32_t)len_q(M) - 32;
  const uint64_t c = pack64(__builtin_amdgcn_alignbit(lo32(h2), hi32(s), sh),
                            __builtin_amdgcn_alignbit(hi32(h2), lo32(h2), sh));
  const uint64_t k = c + mulhi_low3(c, M.ml);
  const uint64_t nq = neg_q(M);
  return add_high((uint64_t)lo32(k) * lo32(nq) + s, lo32(k) * hi32(nq) + hi32(k) * lo32(nq));
}

template <int KIND>
__device__ __forceinline__ void mul_mod_x4(uint64_t (&a)[4], const uint64_t (&b)[4], const Tw<uint64_t>& g, bool neg,
                                           const Mod& M) {
  static_assert(KIND == KIND_WIDE, "len(q) <= 60");
  Limbs A[4], B[4], Z[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint64_t bi = red2<KIND>(b[i], M);
    A[i] = limbs31(red2<KIND>(a[i], M));
    B[i] = limbs31(bi);
    if (i) {
      const uint64_t z = mul_tw<KIND>(bi, g, M);        // < 3.5 q
      Z[i] = limbs31(red2<KIND>(neg ? mult_q<uint64_t>(4, M) - z : z, M));
    }
  }
#pragma unroll
  for (int n = 0; n < 4; ++n) {
    uint64_t c0 = 0, c1 = 0, c2 = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const Limbs& v = i <= n ? B[n - i] : Z[4 + n - i];
      c0 = (uint64_t)A[i].lo * v.lo + c0;
      c1 = (uint64_t)A[i].lo * v.hi + c1;
      c1 = (uint64_t)A[i].hi * v.lo + c1;
      c2 = (uint64_t)A[i].hi * v.hi + c2;
    }
    a[n] = reduce_sum(c0, c1, c2, M);
  }
}

// 32-bit words: operands below 2q, S < 16 q^2 < 2^64. With R = 2^32 mod q the sum
// hi32(S) R + lo32(S) < 2^32 q is S modulo q; c = it >> m < 2^32, and the quotient
// c + hi32(c ml) falls short by less than 2 + 1 + 1, so r < 4q < 2^32. (Canonical
// operands would need no second sum: four multiply-adds against eleven conditional
// subtractions, 94 -> 80 instructions a block.)
template <int KIND>
__device__ __forceinline__ void mul_mod_x4(uint32_t (&a)[4], const uint32_t (&b)[4], const Tw<uint32_t>& g, bool neg,
                                           const Mod32& M) {
  const uint32_t R = opaque_s(0u - (uint32_t)((((uint64_t)1 << 32) | M.ml) >> (M.s + 2)) * M.q);
  uint32_t A[4], B[4], Z[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    A[i] = red2<KIND>(a[i], M);
    B[i] = red2<KIND>(b[i], M);
    if (i) {
      const uint32_t z = mul_tw<KIND>(B[i], g, M);               // < 2q
      Z[i] = neg ? 2 * M.q - z : z;                                   // <= 2q
    }
  }
#pragma unroll
  for (int n = 0; n < 4; ++n) {
    uint64_t s = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) s = (uint64_t)A[i] * (i <= n ? B[n - i] : Z[4 + n - i]) + s;
    s = (uint64_t)(uint32_t)(s >> 32) * R + (uint32_t)s;
    const uint32_t c = __builtin_amdgcn_alignbit((uint32_t)(s >> 32), (uint32_t)s, M.s + 2);
    const uint32_t k = c + __umulhi(c, M.ml);
    a[n] = red2<KIND>((uint32_t)s - k * M.q, M);
  }
}

// Canonical words from words below H q.
template <int KIND, int E, typename W, typename MT>
__device__ __forceinline__ void canon_all(W (&x)[E], const MT& M) {
#pragma unroll
  for (int j = 0; j < E; ++j) x[j] = canon<KIND>(x[j], M);
}

}  // namespace pm
