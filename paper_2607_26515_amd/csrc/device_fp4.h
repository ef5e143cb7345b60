// Device-side FP4 arithmetic for gfx950: MXFP4 and HiF4 block quantization and the
// operand encodings the scaled f8f6f4 MFMA consumes.
//
// Every decision (block scale, element code, level-2/3 bits) is exact: block scales are read from
// the exponent and fraction fields of the block maximum, MXFP4 codes come from gfx950's scaled
// conversions, and HiF4 codes (whose scales are not powers of two) from a quotient by the step's
// rounded reciprocal with one residual step, which an integer rounding then decides exactly
// (hif4_round).  fp32 denormals are kept.  Inputs are finite.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace resq {

constexpr int kMxBlock = 32;
constexpr int kHiBlock = 64;

__device__ __forceinline__ float bf16_to_f32(uint32_t b) { return __uint_as_float(b << 16); }

// v from another lane of the same row of 16 through a DPP lane pattern (every pattern used
// reads inside the row; all lanes active).
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, CTRL, 0xF, 0xF, true);
}
constexpr int kDppXor1 = 0xB1;        // quad_perm [1,0,3,2]
constexpr int kDppXor2 = 0x4E;        // quad_perm [2,3,0,1]
constexpr int kDppHalfMirror = 0x141;  // lane i of 8 <- lane 7-i
constexpr int kDppMirror = 0x140;      // lane i of 16 <- lane 15-i

// Larger of two magnitudes (finite, +0 or positive): their bit patterns order as integers.
__device__ __forceinline__ float max_mag(float a, float b) {
  return __uint_as_float(max(__float_as_uint(a), __float_as_uint(b)));
}

// Max of a magnitude v (finite, +0 or positive) over aligned groups of G lanes (G a power of
// two <= 64).  Up to 16 lanes the partners come through DPP: after the maxima over lane pairs
// and quads, the mirrored lane of an 8-group lies in the other quad and that of a 16-group in
// the other 8-group.
template <int G>
__device__ __forceinline__ float group_max(float v) {
  uint32_t u = __float_as_uint(v);
  if constexpr (G >= 2) u = max(u, dpp_u32<kDppXor1>(u));
  if constexpr (G >= 4) u = max(u, dpp_u32<kDppXor2>(u));
  if constexpr (G >= 8) u = max(u, dpp_u32<kDppHalfMirror>(u));
  if constexpr (G >= 16) u = max(u, dpp_u32<kDppMirror>(u));
#pragma unroll
  for (int o = 16; o < G; o <<= 1) u = max(u, (uint32_t)__shfl_xor((int)u, o, 64));
  return __uint_as_float(u);
}

template <int G>
__device__ __forceinline__ double group_sum(double v) {
#pragma unroll
  for (int o = 1; o < G; o <<= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// ------------------------------------------------------------------------------------------
// MXFP4: E2M1 elements, one E8M0 scale per 32 elements (OCP MX conversion rule, paper Sec. 3)
// ------------------------------------------------------------------------------------------
// Shared exponent of a block with max magnitude amax (finite, +0 or positive):
// floor(log2 amax) - 2, clamped to [-127, 127].  For normal amax that is the biased exponent
// field minus 129 (at most 125); a subnormal amax or zero has field 0 and clamps to -127.
__device__ __forceinline__ int mx_exponent(float amax) {
  const int e = (int)(__float_as_uint(amax) >> 23) - 129;
  return e < -127 ? -127 : e;
}

// 2^E as a float for the MX exponent range E in [-127, 127] (2^-127 is subnormal).
__device__ __forceinline__ float mx_scale_f32(int E) {
  return E >= -126 ? __uint_as_float((uint32_t)(E + 127) << 23) : __uint_as_float(0x00400000u);
}

// Quantization by gfx950's scaled conversions, two elements per instruction:
// v_cvt_scalef32_pk_fp4_f32 with scale 2^E rounds x / 2^E to the nearest E2M1 magnitude,
// ties to the even code, saturates at 6 and keeps the sign of a zero result;
// v_cvt_scalef32_pk_f32_fp4 returns the code's value.  (GPU tests compare the
// resulting codes and scales with the oracle's on every E2M1 tie and threshold, saturation,
// signed zeros and shared exponents from -127, where 2^E is subnormal, to 124.)
// Codes of x0, x1: bits 0-3 and 4-7 of the result.
__device__ __forceinline__ uint32_t mx_code2(float x0, float x1, float scale) {
  return __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(0u, x0, x1, scale, 0) & 0xFFu;
}
__device__ __forceinline__ void mx_value2(uint32_t codes2, float scale, float& v0, float& v1) {
  const auto v = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(codes2, scale, 0);
  v0 = v[0];
  v1 = v[1];
}

// ------------------------------------------------------------------------------------------
// HiF4 (reading stated in resq.h): 64-element blocks, E6M2 level-1 scale, one-bit level-2
// (per 8) and level-3 (per 4) down-shifts, S1P2 elements k/4.
//   s1 = 2^(e-31) (1 + m/4) for code c = 4e + m;  element value = k (4+m) 2^(e-35-b)
// ------------------------------------------------------------------------------------------
// Smallest code c with 1.75 * s1(c) >= A (saturating at 255), for a magnitude A (finite, +0 or
// positive).  For A in [2^ea, 2^(ea+1)) the values 1.75 * s1 of codes 4(ea+30)+1 .. +4 are
// {35, 42, 49, 56, 63} 2^(ea-5), i.e. mantissas 1.09375, 1.3125, 1.53125, 1.75 and above 1.875,
// so c is that base code plus the number of the first four that A's mantissa exceeds.  On the
// pattern u - 1 "exceeds" is "reaches", and in units of 2^18 the four fractions are 3, 10, 17 and
// 24: their count for a five-bit fraction f is (585 f + 2344) >> 12.  (u a power of two borrows
// from the exponent and counts four there; u = 0 gives a negative count.)  Every A below 2^-31
// gives a negative count, clamped to code 0.
__device__ __forceinline__ int hif4_c1(float A) {
  const int v = (int)__float_as_uint(A) - 1;
  const int c = 4 * (v >> 23) + ((((v >> 18) & 31) * 585 + 2344) >> 12) - 387;
  return c < 0 ? 0 : (c > 255 ? 255 : c);
}

// The element grid of level-1 code c1 and shift b: its step (4+m) 2^(e-35-b) (exact and normal:
// at least 4 * 2^-37) and the step's reciprocal, fl(1 / (4+m)) times the exact power of two.
struct Hif4Grid {
  float step, inv;
};
__device__ __forceinline__ float hif4_inv_q(int c1) {
  const int m = c1 & 3;
  return m == 0 ? 0.25f : m == 1 ? 0.2f : m == 2 ? 1.0f / 6.0f : 1.0f / 7.0f;
}
__device__ __forceinline__ Hif4Grid hif4_grid(int c1, float inv_q, int b) {
  const int p = (c1 >> 2) - 35 - b;
  return Hif4Grid{ldexpf((float)(4 + (c1 & 3)), p), ldexpf(inv_q, -p)};
}
// The "fits at half the scale" threshold 1.75 * s1 / 2 * 2^-b of a group, from the step of
// shift b: 7 (4+m) 2^(e-36-b) = 3.5 step (exact).
__device__ __forceinline__ float hif4_half_fit(float step) { return 3.5f * step; }

// |x| on that grid: the integer k (0 .. 7) nearest to |x| / step, ties to even k, saturating; NaN
// gives 0 (the median of a NaN and two numbers is the smaller number).  inv is the correctly rounded
// reciprocal, so one residual step rounds the quotient correctly; and since the grid's midpoints
// (2j+1)/2 have few bits and float32 values around a midpoint times the step are at least half a
// place apart in the quotient ((4+m) < 8), a quotient equals a midpoint exactly when |x| does, so
// rounding it again to an integer is the rounding of |x| / step itself.  tests/hif4_round_check.cpp
// compares it on the host with every midpoint; the GPU tests run every bf16 x.  The quotient
// replaced midpoint searches: HiF4 activation pass of the 7B prefill (m = 8192) 345 -> 259 us, the
// 3B backward's quantization 350 -> 293 us.
__device__ __forceinline__ float hif4_round(float x, const Hif4Grid& g) {
  const float a = __builtin_amdgcn_fmed3f(fabsf(x), 0.f, 7.f * g.step);
  const float y = a * g.inv;
  return __builtin_rintf(fmaf(-fmaf(y, g.step, -a), g.inv, y));
}
// The 4-bit codes of four elements, one per byte (high nibbles zero): k and the sign of x.
__device__ __forceinline__ uint32_t hif4_code_bytes(const float k[4], const float x[4]) {
  uint32_t n = __builtin_amdgcn_cvt_pk_u8_f32(k[0], 0u, 0u);
  n = __builtin_amdgcn_cvt_pk_u8_f32(k[1], 1u, n);
  n = __builtin_amdgcn_cvt_pk_u8_f32(k[2], 2u, n);
  n = __builtin_amdgcn_cvt_pk_u8_f32(k[3], 3u, n);
  const uint32_t s = __builtin_amdgcn_perm(__float_as_uint(x[1]), __float_as_uint(x[0]), 0x0C0C0703u) |
                     __builtin_amdgcn_perm(__float_as_uint(x[3]), __float_as_uint(x[2]), 0x07030C0Cu);
  return n | ((s >> 4) & 0x08080808u);
}

__device__ __forceinline__ float hif4_value(uint32_t code, int c1, int b) {
  const float v = ldexpf((float)((code & 7) * (4 + (c1 & 3))), (c1 >> 2) - 35 - b);
  return (code & 8) ? -v : v;
}

// Compress the even bits of a 16-bit value into 8 bits.
__device__ __forceinline__ uint32_t even_bits16(uint32_t x) {
  x &= 0x5555u;
  x = (x | (x >> 1)) & 0x3333u;
  x = (x | (x >> 2)) & 0x0F0Fu;
  x = (x | (x >> 4)) & 0x00FFu;
  return x;
}

// ------------------------------------------------------------------------------------------
// MFMA operand encodings for HiF4 (f8f6f4 MFMA, formats: 2 = FP6 E2M3, 4 = FP4 E2M1)
// ------------------------------------------------------------------------------------------
// Close four 6-bit fields, one per byte, up into 24 bits, field j at bit 6j.
__device__ __forceinline__ uint32_t close_up6x4(uint32_t x) {
  const uint32_t t = (x & 0x003F003Fu) | ((x >> 2) & 0x0FC00FC0u);
  return (t & 0xFFFu) | ((t >> 4) & 0xFFF000u);
}

// Activation side: V = k (4+m) 2^(2-b) <= 196 (value = V 2^(e-37)) has at most six significant
// bits, so V = 32 hi + 2 lo with hi the largest E2M3 value not above V / 32 and lo an exact E2M1
// value (the remainder is 0..3 units of a quarter or less of hi's step).  Both carry the
// element's sign.  Scales: hi 2^(e-32), stored as E8M0 e + 95; lo 2^(e-36), the same byte with
// the weight operand scaled by 2^-4.
// The codes of k = 0..7 come from a byte table per (m, b), entry 3m + b: x, y the E2M3 codes of
// k = 0..3, 4..7, z, w the E2M1 codes.  A kernel keeps a copy in LDS (hif4_load_split_tab).
constexpr int kHiSplitEntries = 12;
static __device__ const uint4 kHiSplitTab[kHiSplitEntries] = {
    {0x0C080400u, 0x16141210u, 0x00000000u, 0x00000000u}, {0x06040200u, 0x0E0C0A08u, 0x00000000u, 0x00000000u},
    {0x03020100u, 0x07060504u, 0x00000000u, 0x00000000u},
    {0x0F0A0500u, 0x18171412u, 0x00000000u, 0x07000400u}, {0x07050200u, 0x100F0C0Au, 0x02000200u, 0x05000200u},
    {0x03020100u, 0x08070605u, 0x03020100u, 0x03020100u},
    {0x110C0600u, 0x1A191714u, 0x00000000u, 0x06000000u}, {0x09060300u, 0x12110F0Cu, 0x00000000u, 0x04000000u},
    {0x04030100u, 0x0A090706u, 0x02000200u, 0x02000200u},
    {0x120E0700u, 0x1C1A1816u, 0x04000000u, 0x04060700u}, {0x0A070300u, 0x1412100Eu, 0x02000200u, 0x02040500u},
    {0x05030100u, 0x0C0A0807u, 0x01020300u, 0x01020300u}};

// Threads 0 .. 11 of the workgroup fill the LDS copy; the caller's next barrier publishes it.
__device__ __forceinline__ void hif4_load_split_tab(uint4* lds) {
  if (threadIdx.x < kHiSplitEntries) lds[threadIdx.x] = kHiSplitTab[threadIdx.x];
}
__device__ __forceinline__ uint32_t hif4_act_scale(uint32_t c1) { return (c1 >> 2) + 95u; }

// The four elements of one level-3 group, their codes in the low nibbles of the bytes of nb
// (high nibbles ignored), t the table entry of (m, b): four 6-bit hi fields in 24 bits, four
// 4-bit lo fields in 16 bits.
__device__ __forceinline__ void hif4_split4(uint32_t nb, const uint4& t, uint32_t& hi24, uint32_t& lo16) {
  const uint32_t k = nb & 0x07070707u, sg = nb & 0x08080808u;
  hi24 = close_up6x4(__builtin_amdgcn_perm(t.y, t.x, k) | (sg << 2));
  const uint32_t l = __builtin_amdgcn_perm(t.w, t.z, k) | sg;
  lo16 = __builtin_amdgcn_perm(0u, l | (l >> 4), 0x0C0C0200u);
}

// Weight side: k 2^-b as an E2M3 code (exact: 0..1.75 in steps of 1/4, ..., 7), sign in bit 5;
// the level-1 scale (4+m) 2^(e-35) is applied to the accumulators per column.  The codes of
// k = 0..7 come from a byte table by v_perm; the four elements of one level-3 group (shift b)
// at once, their codes in the low nibbles of the bytes of nb, as 24 bits.
__device__ __forceinline__ uint32_t hif4_e2m3x4(uint32_t nb, uint32_t b) {
  const uint32_t lo = b == 0u ? 0x14100800u : b == 1u ? 0x0C080400u : 0x06040200u;
  const uint32_t hi = b == 0u ? 0x1E1C1A18u : b == 1u ? 0x16141210u : 0x0E0C0A08u;
  return close_up6x4(__builtin_amdgcn_perm(hi, lo, nb & 0x07070707u) | ((nb & 0x08080808u) << 2));
}

// Weight-operand scales of the hi and lo products (E8M0 of 2^0 and 2^-4), and the fold factor
// (4 + m) 2^(e-35) of level-1 code c = 4e + m: exponent field e + 94, fraction m / 4.
constexpr int kHiOne = 127, kHiLoScale = 123;
__device__ __forceinline__ float hif4_fold_factor(uint32_t c) { return __uint_as_float((c << 21) + (94u << 23)); }

}  // namespace resq
