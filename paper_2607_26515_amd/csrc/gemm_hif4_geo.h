// Compile-time geometry of the HiF4 GEMM (gemm_hif4.hip): the fragment-major operand layouts,
// the LDS image of one K step, the assignment of copy instructions to waves, and each copy's
// source offset and LDS target.
//
// Plain C++17 constexpr functions (no HIP types), so that a host-side check compiles the same
// code: it rebuilds every wave's copies, verifies that the copies of one K step fill exactly
// the LDS bytes the waves then read with the source bytes the reader expects, and replays the
// kernel's issue / wait / barrier / read sequence.
#pragma once

#include "gemm_geo.h"

namespace resq {

// A fragment (32 rows x 64 K elements, 64 lane records) in memory, planes of all 64 lanes:
//   A (activations, one term): E2M3 "hi" bytes 0-15 of every lane, hi bytes 16-23, then the
//     16 bytes of E2M1 "lo" (device_fp4.h, kHiSplitTab): 40 bytes per lane;
//   B (weights): E2M3 bytes 0-15 of every lane, then bytes 16-23: 24 bytes per lane.
// A lane reads its MFMA operands as one 16-byte and one 8-byte piece into consecutive
// registers (six for E2M3, four for E2M1), so no register copies assemble them.
constexpr int kHiAFrag = 64 * 40, kHiBFrag = 64 * 24;
constexpr int kHiTail = 1024, kHiLo = 1536;  // offsets of the 8-byte plane and of lo

template <int WM_, int WN_, int TM_, int TN_, int NT_, int NS_, int KG_>
struct HiGeo {
  static constexpr int WM = WM_, WN = WN_, TM = TM_, TN = TN_, NT = NT_, NS = NS_, KG = KG_;
  static constexpr int WT = WM * WN;                  // waves per K group
  static constexpr int W = WT * KG;                   // waves
  static constexpr int MTW = WM * TM, NTW = WN * TN;  // row / column tiles per workgroup
  static constexpr int SAJ = (MTW + 3) / 4;           // scale copies per A term (4 fragments each)
  static constexpr int SBJ = (NTW + 3) / 4;
  // LDS image of one K step: A [term][row tile] fragments, B [col tile] fragments, A scales
  // [term][copy][4 x 64 B], B scales [copy][4 x 64 B].  A stage holds KG such images (BLK
  // bytes apart), then the dump area of padding copies.
  static constexpr int B_OFF = NT * MTW * kHiAFrag;
  static constexpr int SA_OFF = B_OFF + NTW * kHiBFrag;
  static constexpr int SB_OFF = SA_OFF + NT * SAJ * 256;
  static constexpr int BLK = (SB_OFF + SBJ * 256 + 255) / 256 * 256;
  static constexpr int DUMP_OFF = KG * BLK;
  static constexpr int STAGE = DUMP_OFF + kDumpBytes;
  // Copies of one stage.  The A then B fragments of a K step are one run of bytes in LDS; JF
  // copies of 1024 bytes (16 per lane) cover the stage's KG runs.  Every wave issues the same
  // number: XF each and, where a few are left over (4 REM <= 2 W), those as pieces of 256
  // bytes (4 per lane) beside the scale copies; otherwise XF is rounded up and the missing
  // copies write zeros to the dump area (each costs 1 KB of LDS writes).
  static_assert(NT * MTW * kHiAFrag % 1024 == 0 && NTW * kHiBFrag % 1024 == 0, "whole copies");
  static constexpr int JA1 = NT * MTW * kHiAFrag / 1024, JF1 = JA1 + NTW * kHiBFrag / 1024, JS1 = NT * SAJ + SBJ;
  static constexpr int JF = KG * JF1, JS = KG * JS1;
  static constexpr bool PIECES = 4 * (JF % W) <= 2 * W;
  static constexpr int XF = PIECES ? JF / W : (JF + W - 1) / W;
  static constexpr int REM4 = PIECES ? 4 * (JF % W) : 0;
  static constexpr int XS = (REM4 + JS + W - 1) / W;
  static constexpr int JW = XF + XS;
  // the K groups' accumulators are summed through the (then idle) LDS of the stages
  static constexpr int RED = (KG - 1) * WT * TM * TN * 16 * 64 * 4;
  static constexpr size_t LDS = (size_t)(NS * STAGE > RED ? NS * STAGE : RED);
  // Register sets and the loop's unroll: A operands alternate per row tile, B per K step.
  static constexpr int U = NS % 2 == 0 ? NS : 2 * NS;
  static_assert(NS >= 2, "at least two stages");
};

// Every configuration of the HiF4 GEMM, as X(tile configuration, WM, WN, TM, TN, NS, KG), with
// the tile configurations of gemm_geo.h.  Each runs with one or two activation terms.
#define RESQ_HIF4_CONFIGS(X)                                                        \
  X(0, 2, 2, 1, 1, 4, 2) X(0, 2, 2, 1, 1, 2, 2) X(0, 2, 2, 1, 1, 2, 1)              \
  X(3, 4, 2, 1, 3, 2, 1) X(2, 2, 2, 2, 3, 2, 1) X(4, 2, 2, 1, 2, 2, 2)

// A copy of a wave: source offset in operand A's or B's buffer (is_a, wave-uniform), LDS target
// and K step within the stage.
struct HiSlot {
  uint32_t voff, lds, kk;
  bool is_a;
};

// The piece of `bytes` bytes per lane starting at byte `at` of the stage's runs of fragments.
template <class G>
constexpr HiSlot hi_slot_run(int at, int bytes, int lane, const SlotArgs& a) {
  const int kk = at / (G::JF1 * 1024), run = at % (G::JF1 * 1024);
  HiSlot c{kBad, (uint32_t)(kk * G::BLK + run), (uint32_t)kk, run < G::B_OFF};
  if (c.is_a) {
    const int p = run + lane * bytes, f = p / kHiAFrag, t = f / G::MTW, i = f % G::MTW;
    if (a.T0 + i < a.mt) c.voff = a.frag_a(t) + ((a.T0 + i) * a.nkb + kk) * kHiAFrag + p % kHiAFrag;
  } else {
    const int p = run - G::B_OFF + lane * bytes, j = p / kHiBFrag;
    if (a.N0 + j < a.nt) c.voff = a.b_frag_off + ((a.N0 + j) * a.nkb + kk) * kHiBFrag + p % kHiBFrag;
  }
  return c;
}

// Copy x of wave `wave`, 16 bytes per lane: copy wave + W x of the fragments.
template <class G>
constexpr HiSlot hi_slot_f(int wave, int x, int lane, const SlotArgs& a) {
  const int jc = wave + G::W * x;
  if (jc < G::JF) return hi_slot_run<G>(jc * 1024, 16, lane, a);
  return HiSlot{kBad, (uint32_t)G::DUMP_OFF, 0u, false};
}

// Copy x of wave `wave`, 4 bytes per lane: the pieces of the fragments' last copies, then the A
// scales of term t for row tiles 4 (jl % SAJ) .. +3, then the B scales (16 lanes per fragment).
template <class G>
constexpr HiSlot hi_slot_s(int wave, int x, int lane, const SlotArgs& a) {
  const int jp = wave + G::W * x, jc = jp - G::REM4;
  if (jc < 0) return hi_slot_run<G>(G::XF * G::W * 1024 + jp * 256, 4, lane, a);
  const int kk = jc / G::JS1, jl = jc % G::JS1;
  HiSlot c{kBad, (uint32_t)G::DUMP_OFF, (uint32_t)kk, jl < G::NT * G::SAJ};
  if (jc < G::JS) {
    if (c.is_a) {
      const int t = jl / G::SAJ, i = 4 * (jl % G::SAJ) + lane / 16;
      if (i < G::MTW && a.T0 + i < a.mt)
        c.voff = a.scale_a(t) + ((a.T0 + i) * a.nkb + kk) * 64 + (lane % 16) * 4;
      c.lds = (uint32_t)(kk * G::BLK + G::SA_OFF + jl * 256);
    } else {
      const int q = jl - G::NT * G::SAJ, j = 4 * q + lane / 16;
      if (j < G::NTW && a.N0 + j < a.nt)
        c.voff = a.b_sc_off + ((a.N0 + j) * a.nkb + kk) * 64 + (lane % 16) * 4;
      c.lds = (uint32_t)(kk * G::BLK + G::SB_OFF + q * 256);
    }
  }
  return c;
}

}  // namespace resq
