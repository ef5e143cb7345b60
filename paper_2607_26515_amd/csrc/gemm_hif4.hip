// HiF4 GEMM on gfx950 scaled MFMA (v_mfma_scale_f32_32x32x64_f8f6f4); MXFP4 is gemm.hip.
//
// HiF4's level-1 scale s1 = 2^e (1 + m/4) is not a power of two, so no FP4/FP6 operand can carry
// it.  An activation value is V 2^(e-37) with V = k (4+m) 2^(2-b) <= 196 of at most six
// significant bits: V = 32 hi + 2 lo exactly, hi an E2M3 operand (V truncated to E2M3's
// grid) and lo the remainder, an E2M1 operand.  The weight element k 2^-b is one exact E2M3
// operand; its block's whole level-1 scale (4 + m_w) 2^(e_w-35) is constant per output column,
// i.e. per lane, and is applied once per 64-K step: acc += s_w P, with P the step's sums.
// The hi and lo products share the activation's scale byte; the factor 16 between them is the
// weight operand's constant scale (2^0 and 2^-4).
//
// Data movement and K groups are those of gemm.hip.  The loop runs in half steps, one per
// row tile of the wave: while the MFMAs of one row tile run, the operands of the next one
// are read from LDS into the other register set (A alternates per row tile, B per K step), and
// the finished tiles' folds are issued between the MFMAs.  The barrier that publishes the
// next stage stands before the last row tile's MFMAs, whose operands are in registers, so no
// wave waits for LDS with an empty matrix pipe.
//
// Bound by MFMA issue together with the fold's VALU work (16 FMAs per tile and step) and, at
// two workgroups per CU, by the stages' copies from L2.  Two E2M3 terms of 48 bytes per lane with
// E3M2 weights, a step's reads ahead of its MFMAs: 7B prefill GEMMs (m = 8192) 3.69 ms, 3B backward
// GEMMs (m = 8192) 1.13 ms; as above 3.12 and 0.99 ms.  Without the fold (wrong results) the
// prefill loop takes 2.84 ms, without copies 2.50 ms.
#include "gemm_core.h"
#include "gemm_hif4.h"
#include "gemm_hif4_geo.h"

namespace resq {
namespace {

typedef int v2i __attribute__((ext_vector_type(2)));

template <class G>
__global__ __launch_bounds__(64 * G::W)
__attribute__((amdgpu_waves_per_eu(G::TM * G::TN > 1 ? 2 : G::KG)))
void gemm_hif4_kernel(GemmParams p) {
  constexpr int WM = G::WM, WN = G::WN, TM = G::TM, TN = G::TN, NT = G::NT, NS = G::NS, KG = G::KG;
  static_assert(G::LDS <= 160 * 1024, "a workgroup's LDS is at most 160 KB on gfx950");
  static_assert((NS - 1) * G::JW < 64, "the vmcnt waits must fit the 6-bit counter");
  extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];

  const uint32_t b = blockIdx.x;
  const uint32_t wgid = (b % kXcds) * p.per_xcd + b / kXcds;
  if (wgid >= p.n_wg) return;
  const uint32_t ntiles = p.grid_m * p.grid_n;
  const uint32_t split = p.ksplit == 1 ? 0u : wgid / ntiles;  // split-major
  const uint32_t tile = wgid - split * ntiles;
  uint32_t wg_m, wg_n;
  tile_coords(tile, p.grid_m, p.grid_n, wg_m, wg_n);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform
  const int kg = wave / G::WT, wt = wave % G::WT;             // K group, wave within it
  const int wm = wt % WM, wn = wt / WM;
  const uint32_t T0 = wg_m * G::MTW, N0 = wg_n * G::NTW;
  const uint32_t kbeg = (uint32_t)(split * p.kper);                    // this split's K steps:
  const uint32_t klen = (uint32_t)min((int64_t)p.kper, p.nkb - kbeg);  // kbeg .. kbeg+klen-1

  // ---- this wave's copy slots (gemm_hif4_geo.h) ----
  SlotArgs sargs{};
  sargs.a_frag0 = p.a_frag_off[0];
  sargs.a_frag1 = p.a_frag_off[1];
  sargs.a_sc0 = p.a_sc_off[0];
  sargs.a_sc1 = p.a_sc_off[1];
  sargs.b_frag_off = p.b_frag_off;
  sargs.b_sc_off = p.b_sc_off;
  sargs.T0 = T0;
  sargs.N0 = N0;
  sargs.mt = (uint32_t)p.mt_tiles;
  sargs.nt = (uint32_t)p.nt_tiles;
  sargs.nkb = (uint32_t)p.nkb;
  HiSlot sf[G::XF], ss[G::XS];
#pragma unroll
  for (int x = 0; x < G::XF; ++x) sf[x] = hi_slot_f<G>(wave, x, lane, sargs);
#pragma unroll
  for (int x = 0; x < G::XS; ++x) ss[x] = hi_slot_s<G>(wave, x, lane, sargs);
  // bytes a copy advances per K step: a fragment of its operand, or a fragment's scales
  auto frag_bytes = [](const HiSlot& c) { return (uint32_t)(c.is_a ? kHiAFrag : kHiBFrag); };
  uint32_t kstep_f[G::XF], kstep_s[G::XS];
#pragma unroll
  for (int x = 0; x < G::XF; ++x) kstep_f[x] = frag_bytes(sf[x]);
#pragma unroll
  for (int x = 0; x < G::XS; ++x) kstep_s[x] = wave + G::W * x < G::REM4 ? frag_bytes(ss[x]) : 64u;

  // Copy stage s of this split (its K steps kbeg + s*KG + kk, kk < KG) into stage buffer
  // `buf`; K steps past the split's end copy zeros (through a zero-size buffer).
  const uint32_t nsteps = (klen + KG - 1) / KG;
  auto issue = [&](int buf, uint32_t s) {
    const uint32_t k0 = s * KG;
    const uint32_t kb = kbeg + k0;
    const uint32_t left = __builtin_amdgcn_readfirstlane(k0 < klen ? klen - k0 : 0u);
    const __amdgpu_buffer_rsrc_t ra = make_rsrc(p.a, p.a_bytes), rb = make_rsrc(p.b, p.b_bytes);
    const __amdgpu_buffer_rsrc_t za = make_rsrc(p.a, 0u);
    auto inside = [&](const HiSlot& c) { return KG == 1 ? left > 0u : c.kk < left; };
    uint8_t* st = smem + buf * G::STAGE;
#pragma unroll
    for (int x = 0; x < G::XF; ++x)
      copy_to_lds<16>(inside(sf[x]) ? (sf[x].is_a ? ra : rb) : za, st + sf[x].lds, sf[x].voff, kb * kstep_f[x]);
#pragma unroll
    for (int x = 0; x < G::XS; ++x)
      copy_to_lds<4>(inside(ss[x]) ? (ss[x].is_a ? ra : rb) : za, st + ss[x].lds, ss[x].voff, kb * kstep_s[x]);
  };

  v16f acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  struct AOp {  // one row tile's operands, per term
    v8i hi[NT], lo[NT];
    int s[NT];
  };
  struct BOp {  // one K step's weight operands
    v8i x[TN];
    uint32_t c[TN];  // level-1 codes
  };
  AOp A[2];
  BOp B[2];
  // LDS byte offsets of this lane's 16-byte, 8-byte and scale pieces of its wave's first A and B
  // fragments; opaque, so that every read is one of these plus a constant instruction offset.
  // The 8-byte pieces have a register per term and column tile: reads off one register would be
  // merged in pairs, and the pairs copied apart into the operands.
  uint32_t a16 = kg * G::BLK + wm * TM * kHiAFrag + lane * 16;
  uint32_t as = kg * G::BLK + G::SA_OFF + wm * TM * 64 + lane;
  uint32_t b16 = kg * G::BLK + G::B_OFF + wn * TN * kHiBFrag + lane * 16;
  uint32_t bs = kg * G::BLK + G::SB_OFF + wn * TN * 64 + lane;
  uint32_t a8[NT], b8[TN];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    a8[t] = a16 - lane * 8 + t * G::MTW * kHiAFrag + kHiTail;
    asm("" : "+v"(a8[t]));
  }
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    b8[j] = b16 - lane * 8 + j * kHiBFrag + kHiTail;
    asm("" : "+v"(b8[j]));
  }
  asm("" : "+v"(a16), "+v"(as), "+v"(b16), "+v"(bs));
  auto read_a = [&](AOp& o, int buf, int i) {
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int f = buf * G::STAGE + (t * G::MTW + i) * kHiAFrag;
      const v4i x = *reinterpret_cast<const v4i*>(smem + a16 + f);
      const v2i y = *reinterpret_cast<const v2i*>(smem + a8[t] + buf * G::STAGE + i * kHiAFrag);
      const v4i z = *reinterpret_cast<const v4i*>(smem + a16 + f + kHiLo);
      o.hi[t] = v8i{x[0], x[1], x[2], x[3], y[0], y[1], 0, 0};
      o.lo[t] = v8i{z[0], z[1], z[2], z[3], 0, 0, 0, 0};
      o.s[t] = smem[as + buf * G::STAGE + (t * G::SAJ * 4 + i) * 64];
    }
  };
  auto read_b = [&](BOp& o, int buf) {
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int f = buf * G::STAGE + j * kHiBFrag;
      const v4i x = *reinterpret_cast<const v4i*>(smem + b16 + f);
      const v2i y = *reinterpret_cast<const v2i*>(smem + b8[j] + buf * G::STAGE);
      o.x[j] = v8i{x[0], x[1], x[2], x[3], y[0], y[1], 0, 0};
      o.c[j] = smem[bs + buf * G::STAGE + j * 64];
    }
  };

  // One row tile's TN tiles.  Tile by tile, the step's sums P of a tile are folded into its
  // accumulators under the next tile's MFMAs; the last one's fold is pending across half steps.
  v16f Pp = {};
  float fp = 0.f;
  auto tiles = [&](const AOp& a, const BOp& o, int i) {
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int x = i * TN + j, xp = x == 0 ? TM * TN - 1 : x - 1, ip = xp / TN, jp = xp % TN;
      v16f P = v16f{};
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        P = mfma<2, 2>(a.hi[t], o.x[j], P, a.s[t], kHiOne);
        P = mfma<4, 2>(a.lo[t], o.x[j], P, a.s[t], kHiLoScale);
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[ip][jp][r] = fmaf(Pp[r], fp, acc[ip][jp][r]);
      Pp = P;
      fp = hif4_fold_factor(o.c[j]);
    }
  };

  // Half step (k, i) multiplies row tile i of step k, whose operands are in registers, and reads
  // those of the next half step.  Before the last half step of step k: wait for this wave's
  // copies of stage k+1 (the NS-2 later stages stay outstanding) and for its LDS reads, barrier
  // (stage k+1 is visible to every wave, and every wave has read all of stage k's buffer), then
  // refill that buffer with stage k+NS.  Steps past the end multiply zeros.  The loop is
  // unrolled so that every buffer and register-set index is a constant.
#pragma unroll
  for (int s = 0; s < NS; ++s) issue(s, (uint32_t)s);
  wait_vmcnt<(NS - 1) * G::JW>();
  lds_barrier();
  read_b(B[0], 0);
  read_a(A[0], 0, 0);
  for (uint32_t k0 = 0; k0 < nsteps; k0 += G::U) {
#pragma unroll
    for (int u = 0; u < G::U; ++u) {
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const int h = u * TM + i;  // half step: its A set is h % 2
        if (i == TM - 1) {
          wait_vmcnt<(NS - 2) * G::JW>();
          lds_barrier();
          __builtin_amdgcn_sched_barrier(0);
          issue(u % NS, k0 + u + NS);
          read_b(B[(u + 1) & 1], (u + 1) % NS);
          read_a(A[(h + 1) & 1], (u + 1) % NS, 0);
        } else {
          read_a(A[(h + 1) & 1], u % NS, i + 1);
        }
        tiles(A[h & 1], B[u & 1], i);
        // per MFMA: a copy, two LDS reads, a quarter of a tile's fold
#pragma unroll
        for (int q = 0; q < TN * NT * 2; ++q) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                      // MFMA
          if (i == TM - 1) __builtin_amdgcn_sched_group_barrier(0x010, 1, 0);  // copy
          __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);                     // LDS read
          __builtin_amdgcn_sched_group_barrier(0x002, 8 / NT, 0);               // fold
        }
        __builtin_amdgcn_sched_barrier(0);  // keep the half step's MFMAs ahead of the next one's reads
      }
    }
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[TM - 1][TN - 1][r] = fmaf(Pp[r], fp, acc[TM - 1][TN - 1][r]);
  wait_vmcnt<0>();
  finish_tile<WM, WN, TM, TN, KG, G::LDS>(p, acc, smem, kg, wt, wm, wn, lane, T0, N0, tile, split);
}

template <int WM, int WN, int TM, int TN, int NS, int KG>
void launch_cfg(GemmParams p, int n_terms, hipStream_t s) {
  if (n_terms > 1) launch_tiles<WM, WN, TM, TN>(gemm_hif4_kernel<HiGeo<WM, WN, TM, TN, 2, NS, KG>>, KG,
                                                HiGeo<WM, WN, TM, TN, 2, NS, KG>::LDS, p, s);
  else launch_tiles<WM, WN, TM, TN>(gemm_hif4_kernel<HiGeo<WM, WN, TM, TN, 1, NS, KG>>, KG,
                                    HiGeo<WM, WN, TM, TN, 1, NS, KG>::LDS, p, s);
}

}  // namespace

bool launch_gemm_hif4(const GemmParams& p, int cfg, int ns, int kg, int n_terms, hipStream_t s) {
#define RESQ_HIF4_LAUNCH(C, WM, WN, TM, TN, NS, KG)      \
  if (cfg == C && ns == NS && kg == KG) {                \
    launch_cfg<WM, WN, TM, TN, NS, KG>(p, n_terms, s);   \
    return true;                                         \
  }
  RESQ_HIF4_CONFIGS(RESQ_HIF4_LAUNCH)
#undef RESQ_HIF4_LAUNCH
  return false;
}

}  // namespace resq
