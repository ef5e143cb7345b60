// One lane record of a fragment-major MFMA operand (layout in pack.hip): the 32 K-major codes
// (one uint4, element 2i in the low nibble of byte i) of row 32t + l%32, K elements
// 64kb + 32(l/32) .. +31, and their scale word (MX: the E8M0 byte; HiF4: the metadata word
// of the 64-block), written as record `gid` (fragment gid / 64, lane gid % 64) of `frag` plus
// its scale byte in `fscale`.
#pragma once

#include "device_fp4.h"
#include "gemm_hif4_geo.h"
#include "kernels.h"

namespace resq {

// Four consecutive 4-bit codes (nibbles 4g .. 4g+3 of w) spread to the bytes of a word: their
// codes in the low nibbles, the high nibbles undefined.
template <int G>
__device__ __forceinline__ uint32_t spread_codes4(uint32_t w) {
  const uint32_t t = __builtin_amdgcn_perm(w, w, G ? 0x0C030C02u : 0x0C010C00u);
  return t | (t << 4);
}

// Nibble mask keeping the elements whose bit is set in `keep` (bit e = element e of a word).
__device__ __forceinline__ uint32_t nibble_mask8(uint32_t keep) {
  uint32_t m = 0;
#pragma unroll
  for (int e = 0; e < 8; ++e) m |= ((keep >> e) & 1u) * (0xFu << (4 * e));
  return m;
}

// half = l / 32 (which 32-element half of the 64-element HiF4 block the record holds); tab: the
// split table in LDS (activation records only).
template <int MODE>
__device__ __forceinline__ void store_frag_record(uint8_t* __restrict__ frag, uint8_t* __restrict__ fscale,
                                                  int64_t gid, uint4 cw, uint32_t scale, int half,
                                                  const uint4* tab) {
  if constexpr (MODE == kPackMx) {
    *reinterpret_cast<uint4*>(frag + gid * 16) = cw;
    fscale[gid] = (uint8_t)scale;
  } else {
    const uint32_t words[4] = {cw.x, cw.y, cw.z, cw.w};
    const uint32_t c1 = scale & 0xFFu, l2 = scale >> (8 + 4 * half), l3 = scale >> (16 + 8 * half);
    uint32_t h[8], l[8];  // per level-3 group: 24 bits of hi (or of the weight), 16 bits of lo
#pragma unroll
    for (int g = 0; g < 8; ++g) {
      const uint32_t w = words[g >> 1], nb = (g & 1) ? spread_codes4<1>(w) : spread_codes4<0>(w);
      const uint32_t b = ((l2 >> (g >> 1)) & 1u) + ((l3 >> g) & 1u);
      if constexpr (MODE == kPackHiA) hif4_split4(nb, tab[3u * (c1 & 3u) + b], h[g], l[g]);
      else h[g] = hif4_e2m3x4(nb, b);
    }
    uint8_t* f = frag + (gid >> 6) * (MODE == kPackHiA ? kHiAFrag : kHiBFrag);
    const int lane = (int)(gid & 63);
    uint32_t a[6];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      a[3 * q] = h[4 * q] | (h[4 * q + 1] << 24);
      a[3 * q + 1] = (h[4 * q + 1] >> 8) | (h[4 * q + 2] << 16);
      a[3 * q + 2] = (h[4 * q + 2] >> 16) | (h[4 * q + 3] << 8);
    }
    *reinterpret_cast<uint4*>(f + lane * 16) = make_uint4(a[0], a[1], a[2], a[3]);
    *reinterpret_cast<uint2*>(f + kHiTail + lane * 8) = make_uint2(a[4], a[5]);
    if constexpr (MODE == kPackHiA) {
      *reinterpret_cast<uint4*>(f + kHiLo + lane * 16) = make_uint4(l[0] | (l[1] << 16), l[2] | (l[3] << 16),
                                                                    l[4] | (l[5] << 16), l[6] | (l[7] << 16));
      fscale[gid] = (uint8_t)hif4_act_scale(c1);
    } else {
      fscale[gid] = (uint8_t)c1;
    }
  }
}

}  // namespace resq
