// Device building blocks of the gfx950 FFT: complex arithmetic in FP32 and
// packed FP16, constant-twiddle radix-2/4/8/16 DFTs, storage conversions
// (FP32, FP16, OCP FP8 E4M3/E5M2) and the precision-mode policies.
//
// Everything here is device code compiled for gfx950 only.  No twiddle or
// filter table is evaluated on the device: twiddles come from host-built FP64
// tables rounded once (the paper, Sec. III-A, ties the poor "42 dB" FP16
// folklore to recurrence-built tables), and the few radix constants below are
// exact decimal expansions rounded by the compiler.  The only device
// trigonometry is per row or per pulse, outside the transforms: the autofocus
// phasor exp(i phi_m) (FP64 sincos, sar.hip) and the three migration phasors
// per row of the RCMC compression (FP32 sincospif, rows.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace bfp {

typedef _Float16 f16;
typedef f16 h2 __attribute__((ext_vector_type(2)));  // (re, im) in one VGPR

struct __attribute__((aligned(8))) c32 {
  float x, y;
};

// ------------------------------------------------------------ FP32 ops ---
// Contraction is off in these helpers and the complex products use explicit
// FMAs: with the compiler free to fuse a product into whichever neighbouring
// add it finds, two kernels doing the same arithmetic on the same data
// (one row or two rows per thread, a fused or a separate pass) could round
// differently.  Written out, every kernel gets the same bits.
#define BFP_NO_CONTRACT _Pragma("clang fp contract(off)")
__device__ __forceinline__ c32 cadd(c32 a, c32 b) { return c32{a.x + b.x, a.y + b.y}; }
__device__ __forceinline__ c32 csub(c32 a, c32 b) { return c32{a.x - b.x, a.y - b.y}; }
// a - i b and a + i b
__device__ __forceinline__ c32 csub_i(c32 a, c32 b) { return c32{a.x + b.y, a.y - b.x}; }
__device__ __forceinline__ c32 cadd_i(c32 a, c32 b) { return c32{a.x - b.y, a.y + b.x}; }
__device__ __forceinline__ c32 cmul(c32 a, c32 b) {
  BFP_NO_CONTRACT
  return c32{__builtin_fmaf(a.x, b.x, -(a.y * b.y)), __builtin_fmaf(a.x, b.y, a.y * b.x)};
}
__device__ __forceinline__ c32 cconj(c32 a) { return c32{a.x, -a.y}; }

// ----------------------------------------------------- packed FP16 ops ---
__device__ __forceinline__ h2 cadd(h2 a, h2 b) { return a + b; }
__device__ __forceinline__ h2 csub(h2 a, h2 b) { return a - b; }
__device__ __forceinline__ h2 csub_i(h2 a, h2 b) { return a + h2{b.y, -b.x}; }
__device__ __forceinline__ h2 cadd_i(h2 a, h2 b) { return a + h2{-b.y, b.x}; }
__device__ __forceinline__ h2 cmul(h2 a, h2 b) {
  // a b = b.y (-ay, ax) + b.x (ax, ay): both products take b's halves as
  // broadcasts and a's as a swizzle, all source modifiers of the packed
  // instructions.  The swizzled product comes first: with register-held
  // twiddles the compiler then needs no wait state between the two
  // instructions (the other order costs one per product)
  const h2 t = h2{-a.y, a.x} * h2{b.y, b.y};
  return __builtin_elementwise_fma(a, h2{b.x, b.x}, t);
}
__device__ __forceinline__ h2 cconj(h2 a) { return h2{a.x, -a.y}; }

// Exact power-of-two scaling a . 2^-K (the block-floating-point shift) as an
// ldexp instruction: exact for normal results, round-to-nearest-even into
// subnormals, and never contracted into a neighbouring FMA, so the shifted
// value is the same in every kernel.
__device__ __forceinline__ f16 ldexp16(f16 v, int k) {
  return (f16)__builtin_amdgcn_ldexph((__fp16)v, k);
}
template <int K>
__device__ __forceinline__ c32 pow2(c32 a) {
  if constexpr (K == 0) return a;
  else return c32{__builtin_ldexpf(a.x, -K), __builtin_ldexpf(a.y, -K)};
}
// Packed FP16 variant: one v_pk_mul_f16 by (2^-K, +/-2^-K), the same
// correctly rounded product as ldexp.  Contraction is off for this product,
// so the compiler cannot fuse it into a neighbouring FMA.
__device__ __forceinline__ h2 pk_scale(h2 a, h2 s) {
#pragma clang fp contract(off)
  return a * s;
}
template <int K>
__device__ __forceinline__ h2 pow2(h2 a) {
  static_assert(K >= 0 && K <= 14, "2^-K must be a normal FP16 number");
  if constexpr (K == 0) return a;
  else return pk_scale(a, h2{(f16)(1.0f / (1 << K)), (f16)(1.0f / (1 << K))});
}
// conj(a) as a sign flip (one instruction on a packed FP16 pair)
__device__ __forceinline__ c32 conj_store(c32 a) { return c32{a.x, -a.y}; }
__device__ __forceinline__ h2 conj_store(h2 a) {
  return __builtin_bit_cast(h2, __builtin_bit_cast(uint32_t, a) ^ 0x80000000u);
}
// conj(a) . 2^-K
template <int K>
__device__ __forceinline__ c32 conj_pow2(c32 a) {
  if constexpr (K == 0) return c32{a.x, -a.y};
  else return c32{__builtin_ldexpf(a.x, -K), -__builtin_ldexpf(a.y, -K)};
}
template <int K>
__device__ __forceinline__ h2 conj_pow2(h2 a) {
  static_assert(K >= 0 && K <= 14, "2^-K must be a normal FP16 number");
  if constexpr (K == 0) return h2{a.x, -a.y};
  else return pk_scale(a, h2{(f16)(1.0f / (1 << K)), (f16)(-1.0f / (1 << K))});
}

// ----------------------------------------------------- butterflies ------
// (a, b) -> (a + w b, a - w b), every operation an explicit FMA (contraction
// off), so every kernel gets the same bits.  NEGI takes -i w for w (a swap of
// components and a sign, free as operand selects), CJ returns the conjugated
// results (signs only).  The forms differ in how w is given (the FMA butterfly
// of Linzer and Feig, 1993):
//   bf_one   w = 1 (or -i): additions;
//   bf_tan   w = g (1 + i t), |t| <= 1 (COS), or w = g (t + i) (!COS):
//            u = b + t (i b) (or t b + i b), then a +- g u: 6 FMAs, against
//            8 operations for a product and two sums, with one rounding less;
//   bf_twice w = (re, im): s = a + w b, then 2 a - s: 6 FMAs, one rounding
//            more on the difference.
template <bool NEGI, bool CJ, class C>
__device__ __forceinline__ void bf_one(C &a, C &b) {
  const C p = CJ ? cconj(a) : a, q = CJ ? cconj(b) : b;
  if constexpr (!NEGI) {
    a = cadd(p, q);
    b = csub(p, q);
  } else if constexpr (CJ) {  // conj(a -+ i b) = conj a +- i conj b
    a = cadd_i(p, q);
    b = csub_i(p, q);
  } else {
    a = csub_i(p, q);
    b = cadd_i(p, q);
  }
}

// acc + g u and acc - g u, conjugated if CJ; NEGI: -i u for u
template <bool NEGI, bool CJ>
__device__ __forceinline__ void bf_scaled(c32 &a, c32 &b, c32 u, float g) {
  BFP_NO_CONTRACT
  const float ux = NEGI ? u.y : u.x, uy = NEGI ? -u.x : u.y;
  const c32 p = c32{__builtin_fmaf(ux, g, a.x), CJ ? __builtin_fmaf(-uy, g, -a.y) : __builtin_fmaf(uy, g, a.y)};
  const c32 q = c32{__builtin_fmaf(-ux, g, a.x), CJ ? __builtin_fmaf(uy, g, -a.y) : __builtin_fmaf(-uy, g, a.y)};
  a = p;
  b = q;
}
template <bool COS>
__device__ __forceinline__ c32 bf_turn(c32 b, float t) {
  BFP_NO_CONTRACT
  if constexpr (COS) return c32{__builtin_fmaf(-b.y, t, b.x), __builtin_fmaf(b.x, t, b.y)};
  else return c32{__builtin_fmaf(b.x, t, -b.y), __builtin_fmaf(b.y, t, b.x)};
}
template <bool COS, bool NEGI, bool CJ>
__device__ __forceinline__ void bf_tan(c32 &a, c32 &b, c32 w) {  // w = (g, t)
  bf_scaled<NEGI, CJ>(a, b, bf_turn<COS>(b, w.y), w.x);
}

template <bool NEGI, bool CJ>
__device__ __forceinline__ void bf_twice(c32 &a, c32 &b, c32 w) {
  BFP_NO_CONTRACT
  const c32 c = CJ ? cconj(a) : a;
  const float wx = NEGI ? w.y : w.x, wy = NEGI ? -w.x : w.y;
  const float sg = CJ ? -1.0f : 1.0f;  // folds into the operands' signs
  a = c32{__builtin_fmaf(wx, b.x, __builtin_fmaf(-wy, b.y, a.x)),
          __builtin_fmaf(sg * wx, b.y, __builtin_fmaf(sg * wy, b.x, sg * a.y))};
  b = c32{__builtin_fmaf(2.0f, c.x, -a.x), __builtin_fmaf(2.0f, c.y, -a.y)};
}

// ------------------------------------------------------------ DFTs ------
// Length-R DFT of x_r omega^r, omega = W_{NS R}^m the twiddle base of a
// Stockham pass, by decimation in time: with E and O the DFT_{R/2} of the
// even and odd elements on base omega^2,
//   X_k = E_k + (omega W_R^k) O_k,  X_{k + R/2} = E_k - (omega W_R^k) O_k,
// so the twiddles are merged into the butterflies, and since
// omega W_R^{k + R/4} = -i omega W_R^k a level takes R/4 values: R/2 for all
// levels (level R first, then R/2 ...; level 2 one), where separate products
// take R - 1.  The angle of omega W_R^k lies in (-2 pi (k + 1) / R,
// -2 pi k / R]: from R = 8 on each k < R/4 is on one side of -pi/4 for every
// m, and the tangent form is chosen at compile time.  At R = 4 the angle of
// omega spans (-pi/2, 0] and at R = 2 (-pi, 0]: those take (re, im), as
// bf_twice.  A radix-16 pass takes 192 operations on 16 values (220 with 15
// products and a 4 x 4 DFT16) and half the table reads.  It rounds each
// level's twiddles anew: 2 to 5% more FP32 error than products, so it serves
// the mode whose error is the FP16 rounding of its exchanges, 2000 times
// larger.
template <int R>
constexpr int tw_level() { return R >= 4 ? R / 4 : 1; }  // those of level R

template <int R, bool CJ>
__device__ __forceinline__ void dft_tw(c32 (&x)[R], const c32 *w) {
  if constexpr (R == 2) {
    bf_twice<false, CJ>(x[0], x[1], w[0]);
  } else {
    c32 e[R / 2], o[R / 2];
#pragma unroll
    for (int k = 0; k < R / 2; ++k) {
      e[k] = x[2 * k];
      o[k] = x[2 * k + 1];
    }
    dft_tw<R / 2, false>(e, w + tw_level<R>());
    dft_tw<R / 2, false>(o, w + tw_level<R>());
#pragma unroll
    for (int k = 0; k < R / 4; ++k) {
      const int k2 = k + R / 4;
      if constexpr (R == 4) {
        bf_twice<false, CJ>(e[k], o[k], w[k]);
        bf_twice<true, CJ>(e[k2], o[k2], w[k]);
      } else if (k < R / 8) {
        bf_tan<true, false, CJ>(e[k], o[k], w[k]);
        bf_tan<true, true, CJ>(e[k2], o[k2], w[k]);
      } else {
        bf_tan<false, false, CJ>(e[k], o[k], w[k]);
        bf_tan<false, true, CJ>(e[k2], o[k2], w[k]);
      }
    }
#pragma unroll
    for (int k = 0; k < R / 2; ++k) {
      x[k] = e[k];
      x[k + R / 2] = o[k];
    }
  }
}

// tan and cos of pi e / 8 (e = 1, 2), to 20 significant digits
constexpr float kTan8[3] = {0.0f, 0.41421356237309504880f, 1.0f};
constexpr float kCos8[3] = {1.0f, 0.92387953251128675613f, 0.70710678118654752440f};

// How the first level of a first pass takes its pairs (x_r, x_{r + R/2}):
//   LeafPlain   a + b, a - b;
//   LeafScaled  a + s b, a - s b as FMAs, a scaled already: the block shift
//               s = 2^-K of an inverse then costs FP32 pairs half its
//               multiplications, with the same bits (s b is exact).  With an
//               s that the compiler cannot see to be 1, FP16 operands reach
//               the FMA without a conversion (v_fma_mix_f32).
struct LeafPlain {};
struct LeafScaled {
  float s;
};
__device__ __forceinline__ LeafScaled leaf_one() {
  float s = 1.0f;
  asm("" : "+s"(s));
  return LeafScaled{s};
}
template <class C, int K>
using FoldLeaf = std::conditional_t<std::is_same<C, c32>::value && (K > 0), LeafScaled, LeafPlain>;
template <class C, int K>
__device__ __forceinline__ FoldLeaf<C, K> fold_leaf() {
  if constexpr (std::is_same<C, c32>::value && K > 0) return LeafScaled{1.0f / (1 << K)};
  else return LeafPlain{};
}
// element e of E on its way into such a first pass: conj(z) 2^-K, or z 2^-K
// (CONJ = false), with the factor left to the leaf in the second half
template <int K, int E, bool CONJ = true, class C>
__device__ __forceinline__ C fold_in(C z, int e) {
  if (std::is_same<C, c32>::value && K > 0 && e >= E / 2) return CONJ ? conj_store(z) : z;
  return CONJ ? conj_pow2<K>(z) : pow2<K>(z);
}

template <class C>
__device__ __forceinline__ void bf_leaf(C &a, C &b, LeafPlain) {
  bf_one<false, false>(a, b);
}
__device__ __forceinline__ void bf_leaf(c32 &a, c32 &b, LeafScaled l) {
  BFP_NO_CONTRACT
  const c32 p = c32{__builtin_fmaf(b.x, l.s, a.x), __builtin_fmaf(b.y, l.s, a.y)};
  b = c32{__builtin_fmaf(-b.x, l.s, a.x), __builtin_fmaf(-b.y, l.s, a.y)};
  a = p;
}

// The same with omega = 1 (the first pass, and transforms in one pass):
// W_R^k = cos a - i sin a, a = 2 pi k / R, are constants.
template <int R, bool CJ = false, class Leaf = LeafPlain>
__device__ __forceinline__ void dft(c32 (&x)[R], Leaf leaf = Leaf{}) {
  static_assert(R == 2 || R == 4 || R == 8 || R == 16, "radix");
  if constexpr (R == 2) {
    if constexpr (CJ) bf_one<false, true>(x[0], x[1]);  // a last pass of radix 2
    else bf_leaf(x[0], x[1], leaf);
  } else {
    c32 e[R / 2], o[R / 2];
#pragma unroll
    for (int k = 0; k < R / 2; ++k) {
      e[k] = x[2 * k];
      o[k] = x[2 * k + 1];
    }
    dft<R / 2>(e, leaf);
    dft<R / 2>(o, leaf);
    bf_one<false, CJ>(e[0], o[0]);
    bf_one<true, CJ>(e[R / 4], o[R / 4]);
#pragma unroll
    for (int k = 1; k < R / 4; ++k) {
      const int k2 = k + R / 4, s = 16 / R * k;  // a = pi s / 8
      if (s <= 2) {  // cos a (1 - i tan a)
        const c32 w = c32{kCos8[s], -kTan8[s]};
        bf_tan<true, false, CJ>(e[k], o[k], w);
        bf_tan<true, true, CJ>(e[k2], o[k2], w);
      } else {       // -sin a (-cot a + i), with sin a = cos(pi/2 - a)
        const c32 w = c32{-kCos8[4 - s], -kTan8[4 - s]};
        bf_tan<false, false, CJ>(e[k], o[k], w);
        bf_tan<false, true, CJ>(e[k2], o[k2], w);
      }
    }
#pragma unroll
    for (int k = 0; k < R / 2; ++k) {
      x[k] = e[k];
      x[k + R / 2] = o[k];
    }
  }
}

// ---------------------------------------------- DFTs after products ------
// DFTs by radix-4 steps, for the passes whose twiddles are products ahead of
// the DFT (kSteps).  CJ returns the conjugated outputs: the last combining
// step takes conjugated operands (conj(x + y) = conj x + conj y, conj(-i y) =
// i conj y), source negations of the adds.
#define BFP_C8 0.70710678118654752440f
#define BFP_C16 0.92387953251128675613f
#define BFP_S16 0.38268343236508977173f

template <class C>
__device__ __forceinline__ C rot_mi(C a) { return C{a.y, -a.x}; }  // x (-i)
// x k, and the constant c + i s in the type of a product's operand
__device__ __forceinline__ c32 times_k(c32 a, float k) {
  BFP_NO_CONTRACT
  return c32{a.x * k, a.y * k};
}
__device__ __forceinline__ h2 times_k(h2 a, float k) { return a * h2{(f16)k, (f16)k}; }
__device__ __forceinline__ c32 pair_of(c32, float c, float s) { return c32{c, s}; }
__device__ __forceinline__ h2 pair_of(h2, float c, float s) { return h2{(f16)c, (f16)s}; }

// a * W_R^e, W_R = exp(-2 pi i / R), e a compile-time constant below R / 2 + 2
template <int R, int e, class C>
__device__ __forceinline__ C mulw(C a) {
  if constexpr (e == 0) return a;
  else if constexpr (4 * e == R) return rot_mi(a);
  else if constexpr (8 * e == R) return times_k(cadd(a, rot_mi(a)), BFP_C8);      // e^{-i pi/4}
  else if constexpr (8 * e == 3 * R) return times_k(csub(rot_mi(a), a), BFP_C8);  // e^{-3i pi/4}
  else {
    static_assert(R == 16 && (e == 1 || e == 3 || e == 9), "odd powers of W_16 of a 4 x 4 DFT16");
    return cmul(a, pair_of(C{}, e == 1 ? BFP_C16 : e == 3 ? BFP_S16 : -BFP_C16,
                           e == 1 ? -BFP_S16 : e == 3 ? -BFP_C16 : BFP_S16));
  }
}

// (leaf: how a first pass takes its pairs, LeafPlain after products)
template <bool CJ = false, class C, class Leaf = LeafPlain>
__device__ __forceinline__ void dft4(C &a, C &b, C &c, C &d, Leaf leaf = Leaf{}) {
  C s0 = a, s1 = c, s2 = b, s3 = d;
  bf_leaf(s0, s1, leaf);
  bf_leaf(s2, s3, leaf);
  if constexpr (CJ) {
    s0 = cconj(s0);
    s1 = cconj(s1);
    s2 = cconj(s2);
    s3 = cconj(s3);
    a = cadd(s0, s2);
    c = csub(s0, s2);
    b = cadd_i(s1, s3);  // conj((a-c) - i(b-d))
    d = csub_i(s1, s3);  // conj((a-c) + i(b-d))
  } else {
    a = cadd(s0, s2);
    c = csub(s0, s2);
    b = csub_i(s1, s3);  // (a-c) - i(b-d)
    d = cadd_i(s1, s3);  // (a-c) + i(b-d)
  }
}

// In place, natural order in and out.
template <int R, bool CJ, class C, class Leaf = LeafPlain>
__device__ __forceinline__ void dft_steps(C (&v)[R], Leaf leaf = Leaf{}) {
  if constexpr (R == 2) {
    static_assert(!CJ, "conjugates fold into a radix-4 step only");
    const C t = v[0], u = v[1];
    v[0] = cadd(t, u);
    v[1] = csub(t, u);
  } else if constexpr (R == 4) {
    dft4<CJ>(v[0], v[1], v[2], v[3], leaf);
  } else if constexpr (R == 8) {
    // n = n2 + 2 n1 (n2 < 2, n1 < 4), k = k1 + 4 k2
    static_assert(!CJ, "conjugates fold into a radix-4 step only");
    dft4(v[0], v[2], v[4], v[6], leaf);  // n2 = 0 -> slots 0,2,4,6 hold k1 = 0..3
    dft4(v[1], v[3], v[5], v[7], leaf);  // n2 = 1
    v[3] = mulw<8, 1>(v[3]);
    v[5] = mulw<8, 2>(v[5]);
    v[7] = mulw<8, 3>(v[7]);
    C y[8];
#pragma unroll
    for (int k1 = 0; k1 < 4; ++k1) {
      y[k1] = cadd(v[2 * k1], v[2 * k1 + 1]);
      y[k1 + 4] = csub(v[2 * k1], v[2 * k1 + 1]);
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = y[i];
  } else {
    static_assert(R == 16, "radix");
    // n = n2 + 4 n1, k = k1 + 4 k2: DFT4 over n1, twiddle W16^{n2 k1},
    // DFT4 over n2.
#pragma unroll
    for (int n2 = 0; n2 < 4; ++n2) dft4(v[n2], v[n2 + 4], v[n2 + 8], v[n2 + 12], leaf);
    // slot n2 + 4 k1 now holds Y[n2][k1]
    v[5] = mulw<16, 1>(v[5]);
    v[6] = mulw<16, 2>(v[6]);
    v[7] = mulw<16, 3>(v[7]);
    v[9] = mulw<16, 2>(v[9]);
    v[10] = mulw<16, 4>(v[10]);
    v[11] = mulw<16, 6>(v[11]);
    v[13] = mulw<16, 3>(v[13]);
    v[14] = mulw<16, 6>(v[14]);
    v[15] = mulw<16, 9>(v[15]);
#pragma unroll
    for (int k1 = 0; k1 < 4; ++k1) dft4<CJ>(v[4 * k1], v[4 * k1 + 1], v[4 * k1 + 2], v[4 * k1 + 3]);
    // slot k2 + 4 k1 holds X[k1 + 4 k2]: transpose the 4x4 slot grid
    C y[16];
#pragma unroll
    for (int k1 = 0; k1 < 4; ++k1)
#pragma unroll
      for (int k2 = 0; k2 < 4; ++k2) y[k1 + 4 * k2] = v[k2 + 4 * k1];
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = y[i];
  }
}

// ----------------------------------------------------- storage types ----
struct __attribute__((aligned(2))) fp8x2 {
  uint8_t x, y;
};

// OCP FP8 codec on gfx950's conversion instructions: v_cvt_pk_f32_fp8 /
// v_cvt_pk_f32_bf8 decode two bytes exactly (E4M3: bias 7, 3 mantissa bits,
// 0x7F/0xFF NaN; E5M2: bias 15, 2 mantissa bits, exponent 31 = inf/NaN), and
// v_cvt_pk_fp8_f32 / v_cvt_pk_bf8_f32 round two FP32 values to nearest-even.
// Saturation (|x| above the largest finite value maps to it, sign kept, NaN
// stays NaN) is the IEEE 754-2019 maximum and minimum ahead of the rounding
// (v_maximum3_f32, v_minimum3_f32), which propagate NaN: two instructions per
// value where a compare and select takes three.
// The codec is checked bit for bit against the host encoder over the whole
// range, subnormals, saturation and NaN included.
typedef float f32x2 __attribute__((ext_vector_type(2)));
template <int MANT>
struct Fp8Codec {
  static_assert(MANT == 3 || MANT == 2, "E4M3 or E5M2");
  static constexpr float kMax = MANT == 3 ? 448.0f : 57344.0f;
  static __device__ __forceinline__ float sat(float x) {
    return __builtin_elementwise_minimum(__builtin_elementwise_maximum(x, -kMax), kMax);
  }
  // bytes 0 and 1 of `bits` -> (x, y)
  static __device__ __forceinline__ c32 decode2(uint32_t bits) {
    f32x2 v;
    if constexpr (MANT == 3) v = __builtin_amdgcn_cvt_pk_f32_fp8((int)bits, false);
    else v = __builtin_amdgcn_cvt_pk_f32_bf8((int)bits, false);
    return c32{v.x, v.y};
  }
  // (x, y) -> bytes 0 and 1
  static __device__ __forceinline__ uint32_t encode2(float x, float y) {
    if constexpr (MANT == 3) return (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(sat(x), sat(y), 0, false) & 0xFFFFu;
    else return (uint32_t)__builtin_amdgcn_cvt_pk_bf8_f32(sat(x), sat(y), 0, false) & 0xFFFFu;
  }
};

// ------------------------------------------------------ streaming I/O ---
// Row data is read once and written once: nontemporal loads and stores keep
// it from displacing the twiddle and filter tables in the caches.
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
template <class T>
__device__ __forceinline__ T ld_stream(const T *p) {
  static_assert(sizeof(T) == 2 || sizeof(T) == 4 || sizeof(T) == 8, "unsupported element size");
  if constexpr (sizeof(T) == 2)
    return __builtin_bit_cast(T, __builtin_nontemporal_load(reinterpret_cast<const uint16_t *>(p)));
  else if constexpr (sizeof(T) == 4)
    return __builtin_bit_cast(T, __builtin_nontemporal_load(reinterpret_cast<const uint32_t *>(p)));
  else
    return __builtin_bit_cast(T, __builtin_nontemporal_load(reinterpret_cast<const u32x2 *>(p)));
}
template <class T>
__device__ __forceinline__ void st_stream(T *p, T v) {
  static_assert(sizeof(T) == 2 || sizeof(T) == 4 || sizeof(T) == 8, "unsupported element size");
  if constexpr (sizeof(T) == 2)
    __builtin_nontemporal_store(__builtin_bit_cast(uint16_t, v), reinterpret_cast<uint16_t *>(p));
  else if constexpr (sizeof(T) == 4)
    __builtin_nontemporal_store(__builtin_bit_cast(uint32_t, v), reinterpret_cast<uint32_t *>(p));
  else
    __builtin_nontemporal_store(__builtin_bit_cast(u32x2, v), reinterpret_cast<u32x2 *>(p));
}

// The same through a pointer known to address global memory: a uniform base
// can then stay in scalar registers (global loads and stores take a scalar
// base, a 32-bit lane offset and an immediate).
template <class T>
using global_ptr = __attribute__((address_space(1))) T *;
template <class T>
__device__ __forceinline__ T ld_stream_g(global_ptr<const T> p) {
  static_assert(sizeof(T) == 2 || sizeof(T) == 4 || sizeof(T) == 8, "unsupported element size");
  if constexpr (sizeof(T) == 2)
    return __builtin_bit_cast(T, __builtin_nontemporal_load(reinterpret_cast<global_ptr<const uint16_t>>(p)));
  else if constexpr (sizeof(T) == 4)
    return __builtin_bit_cast(T, __builtin_nontemporal_load(reinterpret_cast<global_ptr<const uint32_t>>(p)));
  else
    return __builtin_bit_cast(T, __builtin_nontemporal_load(reinterpret_cast<global_ptr<const u32x2>>(p)));
}
template <class T>
__device__ __forceinline__ T ld_cached_g(global_ptr<const T> p) {
  static_assert(sizeof(T) == 2 || sizeof(T) == 4 || sizeof(T) == 8, "unsupported element size");
  if constexpr (sizeof(T) == 2)
    return __builtin_bit_cast(T, *reinterpret_cast<global_ptr<const uint16_t>>(p));
  else if constexpr (sizeof(T) == 4)
    return __builtin_bit_cast(T, *reinterpret_cast<global_ptr<const uint32_t>>(p));
  else
    return __builtin_bit_cast(T, *reinterpret_cast<global_ptr<const u32x2>>(p));
}
template <class T>
__device__ __forceinline__ void st_stream_g(global_ptr<T> p, T v) {
  static_assert(sizeof(T) == 2 || sizeof(T) == 4 || sizeof(T) == 8, "unsupported element size");
  if constexpr (sizeof(T) == 2)
    __builtin_nontemporal_store(__builtin_bit_cast(uint16_t, v), reinterpret_cast<global_ptr<uint16_t>>(p));
  else if constexpr (sizeof(T) == 4)
    __builtin_nontemporal_store(__builtin_bit_cast(uint32_t, v), reinterpret_cast<global_ptr<uint32_t>>(p));
  else
    __builtin_nontemporal_store(__builtin_bit_cast(u32x2, v), reinterpret_cast<global_ptr<u32x2>>(p));
}

// Row outputs that the next call reads (a spectrum, compressed rows, an
// image): written through the XCD's L2 as it fills (agent scope), they are
// still in the 256 MB last-level cache when that call starts, which
// nontemporal stores pass by, and no dirty lines are left to write back at the
// kernel's end, as plain stores leave them.  A forward and an inverse of
// 16384 x 4096 FP16: 161 against 182 us with nontemporal and 163 with plain
// spectrum stores (the forward transform by itself, streaming, 91, 90, 94).
// The inverse's own output, the end of a chain, is better not kept (178 us),
// nor is the uneven batch's (6% more time).
template <class T>
__device__ __forceinline__ void st_kept_g(global_ptr<T> p, T v) {
  static_assert(sizeof(T) == 2 || sizeof(T) == 4 || sizeof(T) == 8, "unsupported element size");
  if constexpr (sizeof(T) == 2)
    __scoped_atomic_store_n(reinterpret_cast<global_ptr<uint16_t>>(p), __builtin_bit_cast(uint16_t, v),
                            __ATOMIC_RELAXED, __MEMORY_SCOPE_DEVICE);
  else if constexpr (sizeof(T) == 4)
    __scoped_atomic_store_n(reinterpret_cast<global_ptr<uint32_t>>(p), __builtin_bit_cast(uint32_t, v),
                            __ATOMIC_RELAXED, __MEMORY_SCOPE_DEVICE);
  else
    __scoped_atomic_store_n(reinterpret_cast<global_ptr<unsigned long long>>(p),
                            __builtin_bit_cast(unsigned long long, v), __ATOMIC_RELAXED, __MEMORY_SCOPE_DEVICE);
}
// How a row output is stored: nontemporal, through to the last-level cache
// (st_kept_g), or plainly
enum RowStore { ROW_STREAMED, ROW_KEPT, ROW_CACHED };
template <RowStore HOW, class T>
__device__ __forceinline__ void st_row(T *p, T v) {
  if constexpr (HOW == ROW_KEPT) st_kept_g((global_ptr<T>)p, v);
  else if constexpr (HOW == ROW_CACHED) *p = v;
  else st_stream(p, v);
}

// --------------------------------------------------- precision policies --
// Each mode defines:
//   Store: HBM element; Lds: on-chip element between passes;
//   Comp: register arithmetic type; Tw: twiddle table element;
//   Filt: filter element;
//   kMerged: twiddles merged into the butterflies (dft_tw), or a product per
//   value (twiddle) ahead of the DFT, by dft_steps (kSteps) or dft;
//   first_leaf(): how a first pass takes values as decoded
// and the conversions/multiplies the engine needs.

// FP32 throughout, twiddles as products ahead of radix-4 steps: merged into
// the butterflies they take 5% less arithmetic and half the table reads, but
// each level rounds its twiddles anew, and results lie up to 6% further from
// FP64 (64 points 1.04, 512 1.04, 2048 1.02, 4096 1.00 of the error of a
// forward transform, 1.06, 1.05, 1.02, 0.99 of a compression's).
struct ModeFP32 {
  typedef c32 Store; typedef c32 Lds; typedef c32 Comp; typedef c32 Tw; typedef c32 Filt;
  static constexpr bool kMerged = false, kSteps = true;
  static __device__ __forceinline__ LeafPlain first_leaf() { return LeafPlain{}; }
  static __device__ __forceinline__ Comp decode(Store s) { return s; }
  static __device__ __forceinline__ Store encode(Comp v) { return v; }
  static __device__ __forceinline__ Comp load(const Store *p, unsigned i) { return ld_stream(p + i); }
  static __device__ __forceinline__ void store(Store *p, unsigned i, Comp v) { st_stream(p + i, v); }
  static __device__ __forceinline__ Lds to_lds(Comp v) { return v; }
  static __device__ __forceinline__ Comp from_lds(Lds v) { return v; }
  static __device__ __forceinline__ Comp twiddle(Lds v, Tw w) { return cmul(v, w); }
  static __device__ __forceinline__ Comp fmul(Comp v, Filt h) { return cmul(v, h); }
  static __device__ __forceinline__ Comp round_store(Comp v) { return v; }
};

// Pure packed FP16, twiddles as products ahead of radix-4 steps: a twiddle is
// then one rounded pair of FP16 numbers.  Merged into the butterflies as the
// two rounded factors of bf_tan it puts 2.5% (a transform of 8192 points), 3.1%
// (16384) and 3.5% (a round trip of 16384) more error on the result.
struct ModeFP16 {
  typedef h2 Store; typedef h2 Lds; typedef h2 Comp; typedef h2 Tw; typedef h2 Filt;
  static constexpr bool kMerged = false, kSteps = true;
  static __device__ __forceinline__ LeafPlain first_leaf() { return LeafPlain{}; }
  static __device__ __forceinline__ Comp decode(Store s) { return s; }
  static __device__ __forceinline__ Store encode(Comp v) { return v; }
  static __device__ __forceinline__ Comp load(const Store *p, unsigned i) { return ld_stream(p + i); }
  static __device__ __forceinline__ void store(Store *p, unsigned i, Comp v) { st_stream(p + i, v); }
  static __device__ __forceinline__ Lds to_lds(Comp v) { return v; }
  static __device__ __forceinline__ Comp from_lds(Lds v) { return v; }
  static __device__ __forceinline__ Comp twiddle(Lds v, Tw w) { return cmul(v, w); }
  static __device__ __forceinline__ Comp fmul(Comp v, Filt h) { return cmul(v, h); }
  static __device__ __forceinline__ Comp round_store(Comp v) { return v; }
};

__device__ __forceinline__ c32 h2_to_c32(h2 v) { return c32{(float)v.x, (float)v.y}; }

// Natural logarithm of a positive FP32 value from the hardware base-2
// logarithm (v_log_f32, about 1 ulp) and one multiply, instead of the
// library's correctly-scaled sequence (about 11 instructions more).  The
// hardware instruction does not take denormal inputs, so arguments below the
// smallest normal number are raised to it: for an image power p that small
// the terms p ln p and p (ln p + c) are below 1e-36.
__device__ __forceinline__ float ln_pos(float a) {
  return __builtin_amdgcn_logf(fmaxf(a, 1.17549435e-38f)) * 0.693147180559945309f;
}
// Rounded as a pair (v_cvt_pk_f16_f32).  Two scalar conversions may be folded
// into the FMAs that made v.x and v.y (v_fma_mixlo/mixhi_f16), in one kernel
// and not in another, and would then round once where the pair rounds twice.
__device__ __forceinline__ h2 c32_to_h2(c32 v) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  return __builtin_convertvector((f32x2{v.x, v.y}), h2);
}

struct ModeF16StoreF32 {
  typedef h2 Store; typedef h2 Lds; typedef c32 Comp; typedef c32 Tw; typedef h2 Filt;
  static constexpr bool kMerged = true, kSteps = false;
  static __device__ __forceinline__ LeafScaled first_leaf() { return leaf_one(); }
  static __device__ __forceinline__ Comp decode(Store s) { return h2_to_c32(s); }
  static __device__ __forceinline__ Store encode(Comp v) { return c32_to_h2(v); }
  static __device__ __forceinline__ Comp load(const Store *p, unsigned i) { return h2_to_c32(ld_stream(p + i)); }
  static __device__ __forceinline__ void store(Store *p, unsigned i, Comp v) { st_stream(p + i, c32_to_h2(v)); }
  static __device__ __forceinline__ Lds to_lds(Comp v) { return c32_to_h2(v); }
  static __device__ __forceinline__ Comp from_lds(Lds v) { return h2_to_c32(v); }
  // cmul(v, h) with its plain products as FMAs on 0, which take h as stored
  // (v_fma_mix_f32): a product needs a conversion
  static __device__ __forceinline__ Comp fmul(Comp v, Filt h) {
    BFP_NO_CONTRACT
    const c32 f = h2_to_c32(h);
    return c32{__builtin_fmaf(v.x, f.x, __builtin_fmaf(-v.y, f.y, 0.0f)),
               __builtin_fmaf(v.x, f.y, __builtin_fmaf(v.y, f.x, 0.0f))};
  }
  static __device__ __forceinline__ Comp round_store(Comp v) { return h2_to_c32(c32_to_h2(v)); }
};

// FP16 operands, FP32 accumulation: a b as (a.x, a.y) . (b.x, -b.y) and
// (a.x, a.y) . (b.y, b.x) with v_dot2_f32_f16.  The instruction has no operand
// selects, and its sign modifiers are folded by the compiler only for both
// halves at once: the second operands are one flip of the high sign and one
// rotation (a table of both operands doubles its reads, which cost more than
// the two instructions: 37 against 27 us for the 2048 x 4096 compression).
__device__ __forceinline__ c32 cmul_dot2(h2 a, h2 b) {
  const uint32_t u = __builtin_bit_cast(uint32_t, b);
  const h2 re = __builtin_bit_cast(h2, u ^ 0x80000000u);
  const h2 im = __builtin_bit_cast(h2, __builtin_amdgcn_alignbit(u, u, 16));
  return c32{__builtin_amdgcn_fdot2(a, re, 0.0f, false), __builtin_amdgcn_fdot2(a, im, 0.0f, false)};
}

struct ModeF16MulF32Acc {
  typedef h2 Store; typedef h2 Lds; typedef c32 Comp; typedef h2 Tw; typedef h2 Filt;
  static constexpr bool kMerged = false, kSteps = false;
  static __device__ __forceinline__ LeafScaled first_leaf() { return leaf_one(); }
  static __device__ __forceinline__ Comp decode(Store s) { return h2_to_c32(s); }
  static __device__ __forceinline__ Store encode(Comp v) { return c32_to_h2(v); }
  static __device__ __forceinline__ Comp load(const Store *p, unsigned i) { return h2_to_c32(ld_stream(p + i)); }
  static __device__ __forceinline__ void store(Store *p, unsigned i, Comp v) { st_stream(p + i, c32_to_h2(v)); }
  static __device__ __forceinline__ Lds to_lds(Comp v) { return c32_to_h2(v); }
  static __device__ __forceinline__ Comp from_lds(Lds v) { return h2_to_c32(v); }
  static __device__ __forceinline__ Comp twiddle(Lds v, Tw w) { return cmul_dot2(v, w); }
  static __device__ __forceinline__ Comp fmul(Comp v, Filt h) { return cmul_dot2(c32_to_h2(v), h); }
  static __device__ __forceinline__ Comp round_store(Comp v) { return h2_to_c32(c32_to_h2(v)); }
};

// The same with radix-4 steps instead of the recursive dft (4% more arithmetic,
// 61 instead of 72 registers at 16384 points, 60 instead of 79 at 8192), for
// the forward transforms of those sizes: two 1024-thread or four 512-thread
// workgroups then fit a CU.  16M points in 8192-point rows 29.6 against 31.6
// us, 33.3 against 35.2 in 16384-point ones (dft held to 64 registers by
// spills), 35.2 against 42.5 on radix plan 1.
struct ModeF16MulSteps : ModeF16MulF32Acc {
  static constexpr bool kSteps = true;
};

// FP8 storage around the arithmetic of ModeFP32: rows are its results, rounded.
template <int MANT, int BIAS>
struct ModeFP8 {
  typedef fp8x2 Store; typedef c32 Lds; typedef c32 Comp; typedef c32 Tw; typedef c32 Filt;
  static constexpr bool kMerged = false, kSteps = true;
  static __device__ __forceinline__ LeafPlain first_leaf() { return LeafPlain{}; }
  typedef Fp8Codec<MANT> Codec;
  static __device__ __forceinline__ Comp decode(Store b) {
    return Codec::decode2(__builtin_bit_cast(uint16_t, b));
  }
  static __device__ __forceinline__ Comp load(const Store *p, unsigned i) { return decode(ld_stream(p + i)); }
  static __device__ __forceinline__ Store encode(Comp v) {
    return __builtin_bit_cast(fp8x2, (uint16_t)Codec::encode2(v.x, v.y));
  }
  static __device__ __forceinline__ void store(Store *p, unsigned i, Comp v) { st_stream(p + i, encode(v)); }
  static __device__ __forceinline__ Lds to_lds(Comp v) { return v; }
  static __device__ __forceinline__ Comp from_lds(Lds v) { return v; }
  static __device__ __forceinline__ Comp twiddle(Lds v, Tw w) { return cmul(v, w); }
  static __device__ __forceinline__ Comp fmul(Comp v, Filt h) { return cmul(v, h); }
  static __device__ __forceinline__ Comp round_store(Comp v) { return decode(encode(v)); }
};
typedef ModeFP8<3, 7> ModeE4M3;
typedef ModeFP8<2, 15> ModeE5M2;

// the arithmetic of a mode's row kernel by size and operation (FWD: the
// forward transform)
template <class M, int LOG2N, bool FWD>
using KernelMode = std::conditional_t<std::is_same<M, ModeF16MulF32Acc>::value && LOG2N >= 13 && FWD, ModeF16MulSteps, M>;

__device__ __forceinline__ c32 to_c32(c32 v) { return v; }
__device__ __forceinline__ c32 to_c32(h2 v) { return h2_to_c32(v); }

__device__ __forceinline__ bool finite_c(c32 v) {
  return __builtin_isfinite(v.x) && __builtin_isfinite(v.y);
}
__device__ __forceinline__ bool finite_c(h2 v) {
  return __builtin_isfinite((float)v.x) && __builtin_isfinite((float)v.y);
}

}  // namespace bfp
