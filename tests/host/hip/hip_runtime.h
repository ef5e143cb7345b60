// The little of HIP's device environment that device_fp4.h needs, for a host compiler: the checks
// in tests/ compile the device's own arithmetic with it.  Lane exchanges are not modelled (they
// return their argument; the checks do not call them).
#pragma once

#include <algorithm>
#include <array>
#include <cmath>
#include <cstdint>
#include <cstring>

#define __device__
#define __host__
#define __forceinline__ inline

struct uint4 {
  uint32_t x, y, z, w;
};
struct HostDim {
  unsigned x = 0, y = 0, z = 0;
};
static HostDim threadIdx;

inline uint32_t __float_as_uint(float f) {
  uint32_t u;
  std::memcpy(&u, &f, 4);
  return u;
}
inline float __uint_as_float(uint32_t u) {
  float f;
  std::memcpy(&f, &u, 4);
  return f;
}
template <typename T>
T __shfl_xor(T v, int, int) { return v; }
using std::max;
using std::min;

// v_med3_f32: the median; with a NaN operand, the smallest of the others.
inline float host_fmed3(float a, float b, float c) {
  if (std::isnan(a) || std::isnan(b) || std::isnan(c)) return std::fmin(std::fmin(a, b), c);
  return std::fmax(std::fmin(a, b), std::fmin(std::fmax(a, b), c));
}
// v_cvt_pk_u8_f32: byte `i` of `old` replaced by f rounded to nearest even and clamped to 0 .. 255 (NaN: 0).
inline uint32_t host_cvt_pk_u8(float f, uint32_t i, uint32_t old) {
  const float r = std::isnan(f) ? 0.f : std::fmin(std::fmax(std::nearbyint(f), 0.f), 255.f);
  return (old & ~(0xFFu << (8 * i))) | ((uint32_t)r << (8 * i));
}
// v_perm_b32: selector bytes 0 .. 3 take a byte of b, 4 .. 7 one of a, 0x0C is zero.
inline uint32_t host_perm(uint32_t a, uint32_t b, uint32_t sel) {
  const uint64_t src = ((uint64_t)a << 32) | b;
  uint32_t r = 0;
  for (int i = 0; i < 4; ++i) {
    const uint32_t s = (sel >> (8 * i)) & 0xFFu;
    if (s < 8) r |= (uint32_t)((src >> (8 * s)) & 0xFFu) << (8 * i);
  }
  return r;
}
#define __builtin_amdgcn_fmed3f host_fmed3
#define __builtin_amdgcn_cvt_pk_u8_f32 host_cvt_pk_u8
#define __builtin_amdgcn_perm host_perm
#define __builtin_amdgcn_mov_dpp(v, ctrl, row, bank, bound) (v)
#define __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(old, a, b, scale, sel) (old)
#define __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(codes, scale, sel) (std::array<float, 2>{0.f, 0.f})
