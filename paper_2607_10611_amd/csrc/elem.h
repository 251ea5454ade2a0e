// Per-element device code of the step: random draws, storage-format codecs and
// the update's arithmetic.  madd.hip's kernels are built from it, and the
// measurement probes check the same functions.
#pragma once

#include <hip/hip_runtime.h>

#include <math.h>
#include <stdint.h>

#include "exact.h"

namespace madd_detail {

struct Scalars {
  float B1, B2, OMB1, OMB2;  // b1, b2, 1-b1, 1-b2
  float SA;                  // eta_a / (1 - b1^t)   (eta_a without bias correction)
  float IBC2;                // 1 / (1 - b2^t)       (1 without bias correction)
  float LRM, EPS, TAU, GMAX; // eta_m, eps, tau, g_max
  float ULO, UHI;            // u_m clip bounds
  float WMAX;                // final weight clamp
  uint32_t key0, key1;       // Philox key = seed
  uint32_t t;                // step (Philox counter word 2)
};

typedef float f4 __attribute__((ext_vector_type(4)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));
typedef uint32_t u2 __attribute__((ext_vector_type(2)));
// The same at any address their elements may have: one instruction each at
// every alignment on gfx950.
typedef f4 f4_any __attribute__((aligned(4)));
typedef u4 u4_any __attribute__((aligned(4)));
typedef u2 u2_any __attribute__((aligned(2)));
typedef uint32_t u1_any __attribute__((aligned(1)));

// ---------------------------------------------------------------------------
// Philox4x32-10 (Salmon, Moraes, Dror, Shaw; SC'11)
// ---------------------------------------------------------------------------

__device__ __forceinline__ u4 philox10(u4 c, uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const uint64_t p0 = (uint64_t)0xD2511F53u * c.x;  // one v_mad_u64_u32 each
    const uint64_t p1 = (uint64_t)0xCD9E8D57u * c.z;
    c = u4{(uint32_t)(p1 >> 32) ^ c.y ^ k0, (uint32_t)p1, (uint32_t)(p0 >> 32) ^ c.w ^ k1,
           (uint32_t)p0};
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  return c;
}

// 128 random bits for the group of eight elements j = idx >> 3 on a stream:
// 0 rounds the weights, 1, 2, 3 the stochastically rounded bf16 moments
// m, v, v_e.
__device__ __forceinline__ u4 draw_group(uint64_t j, const Scalars& s, uint32_t stream = 0u) {
  return philox10(u4{(uint32_t)j, (uint32_t)(j >> 32), s.t, stream}, s.key0, s.key1);
}

__device__ __forceinline__ uint32_t lane16(u4 r, uint32_t lane) {
  const uint32_t word = (lane < 2) ? r.x : (lane < 4) ? r.y : (lane < 6) ? r.z : r.w;
  return (lane & 1u) ? (word >> 16) : (word & 0xFFFFu);
}

// 16-bit draw of a single element.
__device__ __forceinline__ uint32_t draw_one(uint64_t idx, const Scalars& s, uint32_t stream = 0u) {
  return lane16(draw_group(idx >> 3, s, stream), (uint32_t)(idx & 7u));
}

// ---------------------------------------------------------------------------
// Storage-format codecs (bit level)
// ---------------------------------------------------------------------------

enum : int { WF_BF16 = 0, WF_E4M3 = 1, WF_E5M2 = 2, WF_FP32 = 3, WF_MXFP4 = 4, WF_NVFP4 = 5 };
enum : int { GF_FP32 = 0, GF_BF16 = 1 };
// storage of the moments: fp32, bf16 rounded to nearest-even, bf16 rounded
// stochastically (streams 1, 2, 3)
enum : int { SF_FP32 = 0, SF_BF16 = 1, SF_BF16_SR = 2 };

__device__ __forceinline__ float dec_bf16(uint32_t c) { return __uint_as_float(c << 16); }

// BF16 encoding with gfx950's conversion instructions.  v_cvt_pk_bf16_f32
// rounds to nearest-even; v_cvt_sr_bf16_f32 adds the high 16 bits of its
// random operand to the 16 discarded bits and truncates, which with the draw
// placed there is the stochastic rule above (carry into the kept half with
// probability low16 / 2^16).  Both match the integer definitions bit for bit
// on every non-NaN fp32 (checked exhaustively on the device) and turn a NaN
// into a quieted truncation of it, so a NaN is first replaced by the
// canonical 0x7FC00000, whose conversion is the canonical code 0x7FC0.
typedef float f2v __attribute__((ext_vector_type(2)));
typedef __bf16 bf2v __attribute__((ext_vector_type(2)));
typedef short s2v __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float canon_nan(float x) {
  return (x == x) ? x : __uint_as_float(0x7FC00000u);
}

// Two values, `a` in the low half, neither a NaN other than the canonical one
// (whose sum with a draw keeps its high half).  The stochastic rule is its
// integer definition, (bits + draw) >> 16: two additions at 2 cycles and a
// byte permutation at 4 against two conversions at 8 each.
__device__ __forceinline__ uint32_t enc_bf16x2(float a, float b, bool sr, uint32_t ra,
                                               uint32_t rb) {
  if (sr)
    return __builtin_amdgcn_perm(__float_as_uint(b) + rb, __float_as_uint(a) + ra, 0x07060302u);
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f2v{a, b}, bf2v));
}

__device__ __forceinline__ uint32_t enc_bf16(float x, bool sr, uint32_t r16) {
  if (sr) {
    const s2v r = __builtin_amdgcn_cvt_sr_bf16_f32(s2v{0, 0}, canon_nan(x), r16 << 16, false);
    return __builtin_bit_cast(uint32_t, r) & 0xFFFFu;
  }
  return (uint32_t)__builtin_bit_cast(uint16_t, (__bf16)canon_nan(x));
}

// Minifloat description: M mantissa bits, exponent bias, minimum normal
// exponent, largest finite magnitude and its code, NaN code.
template <int WF>
struct Mini;
template <>
struct Mini<WF_E4M3> {
  static constexpr int M = 3, BIAS = 7, EMIN = -6;
  static constexpr float MAXV = 448.0f;
  static constexpr uint32_t MAXCODE = 0x7Eu, NANCODE = 0x7Fu;
  static constexpr uint32_t RESCALE_BITS = (127u + 127u - 7u) << 23;  // 2^(127 - BIAS)
};
template <>
struct Mini<WF_E5M2> {
  static constexpr int M = 2, BIAS = 15, EMIN = -14;
  static constexpr float MAXV = 57344.0f;
  static constexpr uint32_t MAXCODE = 0x7Bu, NANCODE = 0x7Fu;
  static constexpr uint32_t RESCALE_BITS = (127u + 127u - 15u) << 23;
};

// Branch-free decode: the code's exponent and mantissa fields, placed at the
// top of an fp32's exponent and mantissa fields, read as 2^(E-127) (1.M) for
// E > 0 and as the fp32 subnormal M 2^(-149+23-M) for E = 0; one multiply by
// 2^(127 - BIAS) rescales both exactly (fp32 denormals are kept).
template <int WF>
__device__ __forceinline__ float dec_fp8(uint32_t c) {
  using F = Mini<WF>;
  const uint32_t mag = c & 0x7Fu;
  float v = __uint_as_float(mag << (23 - F::M)) * __uint_as_float(F::RESCALE_BITS);
  if constexpr (WF == WF_E4M3) {
    v = (mag == 0x7Fu) ? __uint_as_float(0x7FC00000u) : v;
  } else {  // E5M2: all-ones exponent is Inf (mantissa 0) or NaN
    v = (mag >= 0x7Cu) ? __uint_as_float((mag & 3u) ? 0x7FC00000u : 0x7F800000u) : v;
  }
  return __uint_as_float(__float_as_uint(v) | ((c & 0x80u) << 24));
}

// FP8 codes with gfx950's conversion instructions.  On every fp32 clamped to
// the largest finite value they are the grid definitions bit for bit, also in
// the subnormal binades (madd_check_encoders of bench_probes/madd_probes.h: every
// input but NaN in every position of a group, the draws on both sides of each
// input's threshold): RNE by v_cvt_pk_{fp8,bf8}_f32, and
// v_cvt_sr_{fp8,bf8}_f32 with the draw in the high half of its random operand
// compares it with the top 16 bits of the discarded fraction.  The codes of
// NaN are left to the caller.  One conversion (8 cycles per wave, two codes per
// instruction to nearest) replaces about nine integer and ldexp operations at 4.
template <int WF>
__device__ __forceinline__ float clamp_fp8(float x) {
  return __builtin_amdgcn_fmed3f(x, -Mini<WF>::MAXV, Mini<WF>::MAXV);
}
template <int WF, int BYTE>
__device__ __forceinline__ uint32_t cvt_sr_fp8(float a, uint32_t r16, uint32_t old) {
  if constexpr (WF == WF_E4M3)
    return (uint32_t)__builtin_amdgcn_cvt_sr_fp8_f32(a, (int)(r16 << 16), (int)old, BYTE);
  else
    return (uint32_t)__builtin_amdgcn_cvt_sr_bf8_f32(a, (int)(r16 << 16), (int)old, BYTE);
}
template <int WF, bool HIGH>
__device__ __forceinline__ uint32_t cvt_pk_fp8(float a, float b, uint32_t old) {
  if constexpr (WF == WF_E4M3)
    return (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(a, b, (int)old, HIGH);
  else
    return (uint32_t)__builtin_amdgcn_cvt_pk_bf8_f32(a, b, (int)old, HIGH);
}
template <int WF>
__device__ __forceinline__ uint32_t enc_fp8(float x, bool sr, uint32_t r16) {
  const float a = clamp_fp8<WF>(x);
  const uint32_t c = (sr ? cvt_sr_fp8<WF, 0>(a, r16, 0u) : cvt_pk_fp8<WF, false>(a, 0.0f, 0u)) & 0xFFu;
  return (x == x) ? c : Mini<WF>::NANCODE;
}
// Four codes of non-NaN values, the first in the low byte.
template <int WF, bool SR>
__device__ __forceinline__ uint32_t enc_fp8x4(const float (&x)[4], const uint32_t (&r)[4]) {
  const float a = clamp_fp8<WF>(x[0]), b = clamp_fp8<WF>(x[1]), c = clamp_fp8<WF>(x[2]),
              d = clamp_fp8<WF>(x[3]);
  if constexpr (SR) {
    uint32_t q = cvt_sr_fp8<WF, 0>(a, r[0], 0u);
    q = cvt_sr_fp8<WF, 1>(b, r[1], q);
    q = cvt_sr_fp8<WF, 2>(c, r[2], q);
    return cvt_sr_fp8<WF, 3>(d, r[3], q);
  } else {
    return cvt_pk_fp8<WF, true>(c, d, cvt_pk_fp8<WF, false>(a, b, 0u));
  }
}
// The values of four codes.  The instruction gives NaN codes without a sign
// the other NaN; a quad that holds one is decoded code by code.
template <int WF>
__device__ __forceinline__ void dec_fp8x4(uint32_t raw, float (&x)[4]) {
  f2v a, b;
  if constexpr (WF == WF_E4M3) {
    a = __builtin_amdgcn_cvt_pk_f32_fp8((int)raw, false);
    b = __builtin_amdgcn_cvt_pk_f32_fp8((int)raw, true);
  } else {
    a = __builtin_amdgcn_cvt_pk_f32_bf8((int)raw, false);
    b = __builtin_amdgcn_cvt_pk_f32_bf8((int)raw, true);
  }
  x[0] = a.x;
  x[1] = a.y;
  x[2] = b.x;
  x[3] = b.y;
  constexpr uint32_t kToNan = (0x80u - (WF == WF_E4M3 ? 0x7Fu : 0x7Du)) * 0x01010101u;
  if (__builtin_expect((((raw & 0x7F7F7F7Fu) + kToNan) & 0x80808080u) != 0u, 0)) {
#pragma unroll
    for (int k = 0; k < 4; ++k) x[k] = dec_fp8<WF>((raw >> (8 * k)) & 0xFFu);
  }
}

// FP16 codes of the block scales (IEEE: RNE, overflow to Inf).
__device__ __forceinline__ float dec_fp16(uint32_t c) {
  return (float)__builtin_bit_cast(_Float16, (uint16_t)c);
}

__device__ __forceinline__ uint32_t enc_fp16_rne(float x) {
  return (x == x) ? (uint32_t)__builtin_bit_cast(uint16_t, (_Float16)x) : 0x7E00u;
}

// MXFP4 (OCP Microscaling): E2M1 elements sharing an E8M0 power-of-two scale.
// E2M1 magnitudes of codes 0..7, doubled (0 1 2 3 4 6 8 12), one per nibble.
__device__ __forceinline__ float dec_e2m1(uint32_t c) {
  const float mag = (float)((0xC8643210u >> (4u * (c & 7u))) & 0xFu) * 0.5f;
  return (c & 8u) ? -mag : mag;
}

// E2M1 codes of values already divided by the block scale, not NaN, saturating
// at +-6, with gfx950's conversions (checked with the FP8 ones).  The
// stochastic one draws its second element from other bits of the random
// operand, so each element takes one, with a zero beside it.
__device__ __forceinline__ uint32_t cvt_sr_e2m1(float x, uint32_t r16) {  // code in bits 0-3
  const float a = __builtin_amdgcn_fmed3f(x, -6.0f, 6.0f);
  return __builtin_amdgcn_cvt_scalef32_sr_pk_fp4_f32(0u, f2v{a, 0.0f}, r16 << 16, 1.0f, 0);
}
// Four codes, one per nibble, the first lowest.
template <bool SR>
__device__ __forceinline__ uint32_t enc_e2m1x4(const float (&x)[4], const uint32_t (&r)[4]) {
  if constexpr (SR) {
    uint32_t c[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) c[k] = cvt_sr_e2m1(x[k], r[k]);
    const uint32_t lo = (c[0] & 0xFu) | ((c[1] << 4) & ~0xFu);  // byte 0 counts
    const uint32_t hi = (c[2] & 0xFu) | ((c[3] << 4) & ~0xFu);
    return __builtin_amdgcn_perm(hi, lo, 0x0C0C0400u);
  } else {
    const uint32_t q = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(0u, x[0], x[1], 1.0f, 0);
    return __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(q, x[2], x[3], 1.0f, 1) & 0xFFFFu;
  }
}
__device__ __forceinline__ void dec_e2m1x4(uint32_t raw, float (&x)[4]) {
  const f2v a = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(raw, 1.0f, 0);
  const f2v b = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(raw, 1.0f, 1);
  x[0] = a.x;
  x[1] = a.y;
  x[2] = b.x;
  x[3] = b.y;
}

// E8M0: 2^(c - 127); code 0 is the fp32 subnormal 2^-127; code 255 is NaN.
__device__ __forceinline__ float dec_e8m0(uint32_t c) {
  if (c == 0xFFu) return __uint_as_float(0x7FC00000u);
  return __uint_as_float(c == 0u ? 0x00400000u : (c << 23));
}

// Scale code of a block whose largest |w'| has the raw bits amax_bits:
// s = floor(log2 amax) - 2 clamped to [-127, 127] (code s + 127); 1.0 for an
// all-zero block; NaN when the block holds a non-finite value.  For a normal
// amax floor(log2 amax) is its unbiased exponent field, so the code is the
// biased field minus 2; a subnormal amax clamps to code 0.
__device__ __forceinline__ uint32_t mx_scale(uint32_t amax_bits) {
  if (amax_bits >= 0x7F800000u) return 0xFFu;
  if (amax_bits == 0u) return 127u;
  const uint32_t ef = amax_bits >> 23;
  return ef > 2u ? ef - 2u : 0u;
}

// 2^-s for a finite scale code (a normal float for every code the rule
// produces, 0..252), so that w' * 2^-s is the exact quotient w' / 2^s.
__device__ __forceinline__ float mx_inv_scale(uint32_t code) {
  return __uint_as_float((code < 0xFFu ? 254u - code : 127u) << 23);
}

template <int WF>
__device__ __forceinline__ uint32_t encode(float x, bool sr, uint32_t r16) {
  if constexpr (WF == WF_BF16) return enc_bf16(x, sr, r16);
  else if constexpr (WF == WF_FP32) return (x == x) ? __float_as_uint(x) : 0x7FC00000u;
  else return enc_fp8<WF>(x, sr, r16);
}

template <int WF>
__device__ __forceinline__ float decode(uint32_t c) {
  if constexpr (WF == WF_BF16) return dec_bf16(c);
  else if constexpr (WF == WF_FP32) return __uint_as_float(c);
  else if constexpr (WF == WF_MXFP4 || WF == WF_NVFP4) return dec_e2m1(c);  // before the scale
  else return dec_fp8<WF>(c);
}

// Block-scale rule: scale = RNE_fp16(amax / FMAX), with 1.0 for an all-zero
// block, the smallest subnormal on underflow, the largest finite value on
// overflow and NaN for a block holding a non-finite value.  `amax_bits` is the
// largest |w'| as raw bits (unsigned order = magnitude order, NaN above Inf).
template <int WF>
__device__ __forceinline__ uint32_t block_scale(uint32_t amax_bits) {
  if (amax_bits >= 0x7F800000u) return 0x7E00u;
  if (amax_bits == 0u) return 0x3C00u;
  uint32_t s = enc_fp16_rne(__uint_as_float(amax_bits) / Mini<WF>::MAXV);
  if (s == 0u) s = 1u;
  if (s == 0x7C00u) s = 0x7BFFu;
  return s;
}

// ---------------------------------------------------------------------------
// The per-element step (fixed FP32 operation order)
// ---------------------------------------------------------------------------

__device__ __forceinline__ float clampf(float x, float lo, float hi) {
  return x < lo ? lo : (x > hi ? hi : x);  // NaN passes through
}

// The exponential moving averages of one element; `ge` receives the exponent
// gradient.
__device__ __forceinline__ void moments_elem(float w, float g, float& m, float& v, float& ve,
                                             float& ge, const Scalars& s) {
  const float LN2 = 0.693147182464599609375f;  // fp32(ln 2)
  m = fmaf(s.B1, m, s.OMB1 * g);
  v = fmaf(s.B2, v, s.OMB2 * (g * g));
  ge = (LN2 * w) * g;
  ve = fmaf(s.B2, ve, s.OMB2 * (ge * ge));
}

// The new weight from the updated moments, with the general square root and
// division: every operand and hyper-parameter.  u_a, then the weight it enters.
//
// CLAMP = false drops the g_max and w_max clamps; the host selects it only
// when both bounds are +infinity, where the clamps are the identity (also for
// NaN and infinite arguments), so the results are the same bits.
__device__ __forceinline__ float add_update(float m, float v, const Scalars& s) {
  return -((s.SA * m) / (sqrtf(v * s.IBC2) + s.EPS));
}
template <bool CLAMP>
__device__ __forceinline__ float weight_elem(float w, float ge, float ua, float ve,
                                             const Scalars& s) {
  // multiplicative branch
  float r = ge / (sqrtf(ve * s.IBC2) + s.EPS);
  if (CLAMP) r = clampf(r, -s.GMAX, s.GMAX);
  const float ut = -(s.LRM * r);
  // relative conversion and clip
  const float aw = fabsf(w);
  const float rho = aw > s.TAU ? aw : s.TAU;
  const float um = clampf(ut / rho, s.ULO, s.UHI);
  // combine, optional final clamp
  const float wn = fmaf(w, um, w) + ua;
  return CLAMP ? clampf(wn, -s.WMAX, s.WMAX) : wn;
}

// The same new weight from the range-limited square root and division of
// exact.h (142 instead of 254 VALU cycles per element and wave, counted from
// the measured rates of the instructions).  Powers of two move the
// intermediates into their ranges: v IBC2 and v_e IBC2 are formed 2^80 times
// larger (v's smallest denormal becomes 2^-69, and v IBC2 below 2^48 stays
// finite), the two numerators SA m and g_e are raised by 2^64, and the factors
// leave again in operations that are there anyway (the addition of eps, the
// product with eta_m, the final addition), so that each stays one rounding of
// the same real number.  Where that is not so:
//  * v IBC2 below 2^-126, which fp32 would round to a denormal: its root is
//    below 2^-62 either way, less than half an ulp of eps >= 2^-38;
//  * a quotient below 2^-126: g_e's then changes u_m below 2^-25, which leaves
//    w + w u_m = w; m's changes |w'| >= 2^-100 by less than half an ulp;
//  * |ut| below 2^-70: u_m stays below 2^-25 since tau >= 2^-40;
//  * anything beyond a range: NaN, an infinity or a value above 2^60 in u_m's
//    quotient or in w'.
// So w' is the general path's, bit for bit, if `lo` (least |w'|) is at least
// 2^-100 and `hi` (largest |w'| or |ut / rho|; NaN if any is) below 2^60,
// and the hyper-parameters are in the ranges of `usable`.  A zero weight's w'
// is u_a alone, which needs no bound but to be normal, w + w u_m being a zero of
// ut's sign; with a zero SA m all of g_e, r, ut and u_a are zeros of the general
// path's signs, and w' with them.
struct FastScalars {
  float ibc2;  // 2^80 IBC2
  float lrm;   // 2^-64 eta_m
  bool usable;
};

// Hyper-parameters outside `usable` (eps = 0 among them) take the general form
// in every group; 41M elements with eps = 1e-15 are 0.71-1.01 of the time that the
// kernels with the general form alone and the compiler's wave counts took, over
// 54 combinations of formats, moments and copies.
//
// Uniform, on the scalar unit: positive floats order like their bits, and a
// normal float times 2^k is k added to its exponent field.
__device__ __forceinline__ FastScalars fast_scalars(const Scalars& s) {
  auto within = [](float x, int lo, int hi) {  // 2^lo <= x < 2^hi
    const uint32_t b = __float_as_uint(x), l = (uint32_t)(127 + lo) << 23,
                   h = (uint32_t)(127 + hi) << 23;
    return b - l < h - l;
  };
  const uint32_t lrm = __float_as_uint(s.LRM), alrm = lrm & 0x7FFFFFFFu;
  FastScalars f;
  f.ibc2 = __uint_as_float(__float_as_uint(s.IBC2) + (80u << 23));
  f.lrm = alrm == 0u ? s.LRM : __uint_as_float(lrm - (64u << 23));
  f.usable = within(s.EPS, -38, 20) && within(s.TAU, -40, 60) && within(s.IBC2, 0, 40) &&
             (alrm == 0u || within(__uint_as_float(alrm), -60, 20)) &&
             __float_as_uint(s.ULO) <= 0xBF7FFFF0u;  // r_max <= 1 - 2^-20
  return f;
}

template <bool CLAMP>
__device__ __forceinline__ float weight_elem_fast(float w, float ge, float m, float v, float ve,
                                                  const Scalars& s, const FastScalars& f,
                                                  float& lo, float& hi) {
  using namespace madd_exact;
  const float da = fmaf(sqrt_in_range(v * f.ibc2), kTwoM40, s.EPS);
  const float qa = div_in_range((s.SA * m) * kTwo64, da);  // 2^64 u_a, negated
  const float de = fmaf(sqrt_in_range(ve * f.ibc2), kTwoM40, s.EPS);
  float r = div_in_range(ge * kTwo64, de);
  if (CLAMP) r = clampf(r, -(s.GMAX * kTwo64), s.GMAX * kTwo64);
  const float ut = -(f.lrm * r);
  const float q = div_in_range(ut, max_abs(w, s.TAU));
  const float um = __builtin_amdgcn_fmed3f(q, s.ULO, s.UHI);
  const float wn = fmaf(qa, -kTwoM64, fmaf(w, um, w));
  lo = fminf(fabsf(wn), lo);
  hi = __builtin_elementwise_maximum(
      __builtin_elementwise_maximum(__builtin_fabsf(q), __builtin_fabsf(wn)), hi);
  return CLAMP ? clampf(wn, -s.WMAX, s.WMAX) : wn;
}

// The step of four elements: m, v, v_e updated in place, the new weights.
// Where the range-limited arithmetic does not vouch for all four, the general
// one takes them again; true if it did.  CANON: NaNs of the moments and the new
// weights leave as the canonical one (the range-limited path has none), for
// encoders that do not look at NaNs.
template <bool CLAMP, bool CANON_M, bool CANON_W>
__device__ __forceinline__ bool step_four(const float (&w)[4], f4 g, f4& m, f4& v, f4& ve,
                                          float (&wn)[4], const Scalars& s) {
  const FastScalars f = fast_scalars(s);
  bool ok = false;
  float ge[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    float a = m[k], b = v[k], c = ve[k];
    moments_elem(w[k], g[k], a, b, c, ge[k], s);
    m[k] = a;
    v[k] = b;
    ve[k] = c;
  }
  float hi = __builtin_inff();
  if (f.usable) {  // uniform
    float lo = madd_exact::kTwo60;
    hi = 0.0f;
#pragma unroll
    for (int k = 0; k < 4; ++k)
      wn[k] = weight_elem_fast<CLAMP>(w[k], ge[k], m[k], v[k], ve[k], s, f, lo, hi);
    ok = lo >= madd_exact::kTwoM100 && hi < madd_exact::kTwo60;
    if (__builtin_expect(!ok, 0)) {
      ok = hi < madd_exact::kTwo60;
#pragma unroll
      for (int k = 0; k < 4; ++k)
        ok = ok && (fabsf(wn[k]) >= madd_exact::kTwoM100 ||
                    (w[k] == 0.0f &&
                     (fabsf(wn[k]) > madd_exact::kTwoM126 || s.SA * m[k] == 0.0f)));
    }
  }
  // A wave with one group here pays for both forms; groups that only hold zero
  // weights with a denormal u_a take the general u_a alone.  41M elements, bf16
  // moments, us (general form for all / for every group that fails the group
  // guard / this): 1% zero weights, E4M3 135 / 166 / 119; half of the elements in
  // rows without a gradient whose moments have decayed to denormals, E4M3
  // 137 / 159 / 127, NVFP4 179 / 189 / 158.
  if (__builtin_expect(!ok, 0)) {
    bool zeros = hi < madd_exact::kTwo60;
#pragma unroll
    for (int k = 0; k < 4; ++k)
      zeros = zeros && (fabsf(wn[k]) >= madd_exact::kTwoM100 || w[k] == 0.0f);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const float ua = add_update(m[k], v[k], s);
      if (!zeros) {
        wn[k] = weight_elem<CLAMP>(w[k], ge[k], ua, ve[k], s);
        if (CANON_W) wn[k] = canon_nan(wn[k]);
        if (CANON_M) {
          m[k] = canon_nan(m[k]);
          v[k] = canon_nan(v[k]);
          ve[k] = canon_nan(ve[k]);
        }
      } else if (w[k] == 0.0f) {
        wn[k] = fmaf(w[k], -(s.LRM * ge[k]), w[k]) + ua;
        if (CLAMP) wn[k] = clampf(wn[k], -s.WMAX, s.WMAX);
      }
    }
  }
  return !ok;
}

}  // namespace madd_detail
