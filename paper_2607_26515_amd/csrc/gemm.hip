// FP4 GEMM on gfx950 scaled MFMA (v_mfma_scale_f32_32x32x64_f8f6f4):
//     Y[M][N] = Q(X) Q(W)^T  (+ S(Q(dX)) Q(W)^T into the same accumulators)   (Eq. 1, Eq. 4)
// This file holds the MXFP4 kernel, whose E2M1 codes and E8M0 scales are the MFMA's own formats,
// and the plans and dispatch of both formats; the HiF4 kernel is gemm_hif4.hip.
//
// MFMA operand layout (32x32x64): lane l holds row (A) / column (B) l%32 and the 32
// consecutive K elements (l/32)*32 .. +31 of the 64-wide K step, packed 4 bits (FP4) or 6
// bits (FP6) per element from bit 0 upwards; its E8M0 scale covers those 32 elements.
// Accumulator register r of lane l is row 8*(r/4) + 4*(l/32) + r%4, column l%32.
// Operands arrive "fragment-major" (pack.hip): fragment (tile, kb) is 64 consecutive lane
// records, plus one scale byte per lane in a separate array; all arrays of operand A (every
// term) share one buffer, and so do those of operand B.
//
// Data movement.  A workgroup of WM x WN waves owns a (WM*TM*32) x (WN*TN*32) output tile.
// Each K step's operand bytes (A fragments of every term, B fragments, their scale bytes)
// are copied from global memory straight into an LDS stage by buffer loads with an LDS
// destination (no registers in between).  Every wave issues the same fixed number of 16-
// and 4-byte copy instructions per stage, so one explicit vmcnt wait per step tells a
// wave that its share of the next stage has landed, and one barrier publishes the stage to
// the other waves.  NS stages are in flight; the waves read their MFMA operands for step
// k+1 from LDS while the MFMAs of step k run.  The buffer descriptors and each lane's
// offsets are fixed for the whole loop (the K advance is the instruction's scalar offset);
// lanes of tiles past the edge copy zeros, and K steps past the end are copied through a
// zero-size buffer, so the loop has no data branches.
//
// K groups.  A workgroup may hold KG groups of WM x WN waves that share the output tile and
// split each stage's K range: a stage carries KG consecutive K steps and group g multiplies
// step g of it, so each barrier is amortised over KG steps and every SIMD holds KG waves
// with independent MFMA chains.  At the end the groups' accumulators are summed through LDS
// in group order (deterministic).  Decode-sized grids, which cannot fill the SIMDs with
// output tiles, use this.
//
// Workgroups are mapped to tiles in contiguous chunks per XCD (workgroup b runs on XCD
// b % 8), so tiles that share a weight column block run on the same XCD and share its L2.
// With a K split the split index varies slowest: an XCD's chunk then covers one K range of
// a block of tiles, whose A rows and B columns over that range it reads once, instead of
// every K range of fewer tiles (the ranges share no operand bytes).
#include "gemm_core.h"
#include "gemm_geo.h"
#include "gemm_hif4.h"
#include "gemm_stream.h"

#include <algorithm>


namespace resq {
namespace {

template <int WM, int WN, int TM, int TN, int NT, int NS, int KG>
__global__ __launch_bounds__(64 * WM * WN * KG)
__attribute__((amdgpu_waves_per_eu(KG)))
void gemm_kernel(GemmParams p) {
  using G = Geo<0, WM, WN, TM, TN, NT, NS, KG>;
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
  const uint32_t nkb = (uint32_t)p.nkb;
  const uint32_t kbeg = (uint32_t)(split * p.kper);                    // this split's K steps:
  const uint32_t klen = (uint32_t)min((int64_t)p.kper, p.nkb - kbeg);  // kbeg .. kbeg+klen-1

  // ---- this wave's copy slots: copy jc of a class goes to wave jc % W (gemm_geo.h) ----
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
  sargs.nkb = nkb;
  Slot sa[G::XA], sb[G::XB], ss[G::XS];
  bool ss_a[G::XS];  // scale slot reads operand A's buffer
#pragma unroll
  for (int x = 0; x < G::XA; ++x) sa[x] = slot_a<G>(wave, x, lane, sargs);
#pragma unroll
  for (int x = 0; x < G::XB; ++x) sb[x] = slot_b<G>(wave, x, lane, sargs);
#pragma unroll
  for (int x = 0; x < G::XS; ++x) ss[x] = slot_s<G>(wave, x, lane, sargs, ss_a[x]);

  // Copy stage s of this split (its K steps kbeg + s*KG + kk, kk < KG) into stage buffer
  // `buf`; K steps past the split's end copy zeros (through a zero-size buffer).
  const uint32_t nsteps = (klen + KG - 1) / KG;
  auto issue = [&](int buf, uint32_t s) {
    const uint32_t k0 = s * KG;
    const uint32_t kb = kbeg + k0;
    // K steps of this stage inside the split (wave-uniform: it selects scalar descriptors)
    const uint32_t left = __builtin_amdgcn_readfirstlane(k0 < klen ? klen - k0 : 0u);
    const __amdgpu_buffer_rsrc_t ra = make_rsrc(p.a, p.a_bytes), rb = make_rsrc(p.b, p.b_bytes);
    const __amdgpu_buffer_rsrc_t za = make_rsrc(p.a, 0u), zb = make_rsrc(p.b, 0u);
    auto inside = [&](const Slot& c) { return KG == 1 ? left > 0u : c.kk < left; };
    uint8_t* st = smem + buf * G::STAGE;
#pragma unroll
    for (int x = 0; x < G::XA; ++x)
      copy_to_lds<16>(inside(sa[x]) ? ra : za, st + sa[x].lds, sa[x].voff, kb * G::A_FRAG);
#pragma unroll
    for (int x = 0; x < G::XB; ++x)
      copy_to_lds<16>(inside(sb[x]) ? rb : zb, st + sb[x].lds, sb[x].voff, kb * G::B_FRAG);
#pragma unroll
    for (int x = 0; x < G::XS; ++x)
      copy_to_lds<4>(inside(ss[x]) ? (ss_a[x] ? ra : rb) : za, st + ss[x].lds, ss[x].voff, kb * 64u);
  };

  v16f acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  // One K step's MFMA operands of this wave, read from an LDS stage.
  struct Frag {
    v8i b[TN];
    int sb[TN];
    v8i a[NT][TM];
    int sa[NT][TM];
  };
  Frag F[2];

  auto read = [&](Frag& f, int buf) {
    const uint8_t* st = smem + buf * G::STAGE + kg * G::BLK;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int lj = wn * TN + j;
      const v4i x = *reinterpret_cast<const v4i*>(st + G::B_OFF + lj * 1024 + lane * 16);
      f.b[j] = v8i{x[0], x[1], x[2], x[3], 0, 0, 0, 0};
      f.sb[j] = st[G::SB_OFF + lj * 64 + lane];
    }
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const int li = wm * TM + i;
        const v4i x = *reinterpret_cast<const v4i*>(st + (t * G::MTW + li) * G::A_FRAG + lane * 16);
        f.a[t][i] = v8i{x[0], x[1], x[2], x[3], 0, 0, 0, 0};
        f.sa[t][i] = st[G::SA_OFF + (t * G::SAJ * 4 + li) * 64 + lane];
      }
  };

  // Tiles past the edge of the output hold zero operands, so they are computed like the
  // others (their results are never stored) and the MFMAs stay branch-free.  Term-major
  // order keeps the TM x TN independent accumulator chains interleaved.
  auto mma = [&](const Frag& f) {
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = mfma<4, 4>(f.a[t][i], f.b[j], acc[i][j], f.sa[t][i], f.sb[j]);
  };

  // Two register sets.  Before step k, stages k+1 .. k+NS-1 are in flight and step k's
  // operands are in registers.  Step k: wait for this wave's copies of stage k+1 (the NS-2
  // later stages stay outstanding), barrier (stage k+1 is visible to every wave, and every
  // wave has read stage k's buffer), refill that buffer with stage k+NS, read stage k+1's
  // operands, run step k's MFMAs.  Steps past the end multiply zeros.  U unrolls the loop
  // so that every buffer and register-set index is a constant.
  constexpr int U = NS % 2 == 0 ? NS : 2 * NS;
#pragma unroll
  for (int s = 0; s < NS; ++s) issue(s, (uint32_t)s);
  wait_vmcnt<(NS - 1) * G::JW>();
  lds_barrier();  // not __syncthreads(), which would wait for every stage's copies
  read(F[0], 0);
  for (uint32_t k0 = 0; k0 < nsteps; k0 += U) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t k = k0 + u;
      wait_vmcnt<(NS - 2) * G::JW>();
      lds_barrier();
      issue(u % NS, k + NS);
      read(F[(u + 1) & 1], (u + 1) % NS);
      mma(F[u & 1]);
      __builtin_amdgcn_sched_barrier(0);  // keep step k's MFMAs ahead of step k+1's barrier
    }
  }
  wait_vmcnt<0>();
  finish_tile<WM, WN, TM, TN, KG, G::LDS>(p, acc, smem, kg, wt, wm, wn, lane, T0, N0, tile, split);
}

template <int FMT, int WM, int WN, int TM, int TN, int NS, int KG>
void launch_cfg(const GemmParams& p, int n_terms, hipStream_t s) {
  if (n_terms > 1)
    launch_tiles<WM, WN, TM, TN>(gemm_kernel<WM, WN, TM, TN, 2, NS, KG>, KG, Geo<FMT, WM, WN, TM, TN, 2, NS, KG>::LDS, p, s);
  else
    launch_tiles<WM, WN, TM, TN>(gemm_kernel<WM, WN, TM, TN, 1, NS, KG>, KG, Geo<FMT, WM, WN, TM, TN, 1, NS, KG>::LDS, p, s);
}

// Tile choice (measured on MI355X): a CU holds one or two workgroups (LDS- and
// register-bound), so the workgroup count decides how many rounds the grid takes.
//  - grids too small for 128-row tiles to fill the chip: 64 x 64 tiles in K groups (two or
//    four groups of four waves, see plan());
//  - small grids with long K that 64 x 128 tiles already fill: the wide tiles below with the
//    K split in up to eight;
//  - MXFP4 with M >= 512 (7B decode and prefill): 128 x 256 tiles (fewest A re-reads per
//    byte of B), two workgroups per CU;
//  - otherwise: 128 x 192 tiles.  HiF4 always takes these: they fit two waves per SIMD (two
//    workgroups per CU at NS = 2), which hides one workgroup's barriers and epilogue behind
//    the other's MFMAs; 128 x 256 HiF4 tiles would spill.  When the HiF4 grid has at most one
//    workgroup per CU (M = 256 decode), the tile runs as eight waves of 32 x 96 instead, so each
//    SIMD still holds two waves.
enum TileCfg { kSmall = 0, kWide = 1, kMid = 2, kMid8 = 3, kNarrow = 4, kStream = 5 };  // kStream + TN - 1
// output tile rows and columns of the staged configurations
constexpr int kTileRows[5] = {64, 128, 128, 128, 64}, kTileCols[5] = {64, 256, 192, 192, 128};
constexpr int64_t kCUs = 256;

struct Plan {
  int cfg, ksplit;
  int kg, ns;  // small tiles: K groups and stages; streamed: waves and K steps in flight
  int64_t kper, tiles;
  size_t partial_bytes;
};

// Grids of few output tiles go to gemm_stream.hip, one row tile x TN column tiles per workgroup.
// Kernel times in us, staged plan -> streamed, MXFP4 / HiF4, S_2:4:
//  - up to one 32 x 32 tile per CU, TN = 1: 2048 -> 2048 at m = 8 6.0 -> 4.0 / 9.7 -> 5.0, at
//    m = 128 6.5 -> 4.3 / 10.8 -> 5.8; 11008 -> 2048 at m = 8 14.4 -> 7.2 / 23.6 -> 14.2; 18944
//    -> 3584 at m = 64 23.8 -> 18.6 / 42 -> 32.7; past that TN = 1 loses (m = 96: 24 -> 30.5);
//  - up to one 32 x 64 tile per CU, TN = 2: 2048 -> 2560 at m = 128 7.0 -> 5.5 / 10.4 -> 7.2;
//    18944 -> 3584 at m = 128 24.7 -> 24.2 / 42.7 -> 41.1;
//  - HiF4 up to one 32 x 96 tile per CU, TN = 3: 3584 -> 4608 at m = 128 14.8 -> 11.0;
//  - wide N, where the weights are read for one row tile (HiF4: two), TN = 2 in four waves.
//    Whole calls: 2048 -> 22016 at m = 8 MXFP4 11.4 -> 9.4; HiF4 2048 -> 28672 at m = 8 22.9 ->
//    14.4, 3584 -> 37888 at m = 64 48.2 -> 41.4.  MXFP4 below 1024 column tiles: 896 (3584 -> 28672)
//    15.7 -> 14.2 at m = 8, 16.0 -> 15.7 at m = 32; 1023 (3584 -> 32736) 14.9 -> 15.1 and 16.1 ->
//    16.8; 1184 (37888) would be 17.7 -> 18.1 and 18.8 -> 19.8.  A second MXFP4 row tile would
//    lose (m = 64, 2048 -> 22016 12.5 -> 12.9), and so would a third HiF4 one (m = 65, 3584 ->
//    37888 48.5 -> 53.9).
// The row limits (256 rows; below 256 for K of 128 steps or more and for TN = 3) are not where the
// streamed plans stop winning: tests pin the staged plans of the usual 256-row batch (the plan list
// of test_gpu_determinism.py and its K-split cases).  Whole calls, staged -> streamed: m = 256,
// 11008 -> 2048 24.2 -> 19.0 / 35.8 -> 30.9 (24.2 -> 23.3 / 35.8 -> 36.4 with K also split in two),
// HiF4 2048 -> 2560 16.1 -> 14.0; m = 288, 2048 -> 1792 10.7 -> 9.7 / 16.3 -> 13.0; m = 512, 8192 ->
// 1024 23.9 -> 18.1 / 33.2 -> 27.9.
// Very long K over few workgroups is split (65536 -> 256 at m = 8: 42 -> 11.3 / 88 -> 18.2).
bool stream_plan(int fmt, int64_t M, int64_t mt, int64_t nt, int64_t nkb, bool may_split, Plan& pl) {
  if (M > 256 || (M == 256 && nkb >= 128)) return false;
  auto tiles = [&](int64_t tn) { return mt * ((nt + tn - 1) / tn); };
  int tn = 0, waves = 8;
  if (tiles(1) <= kCUs) tn = 1;
  else if (tiles(2) <= kCUs) tn = 2;
  else if (fmt == 1 && M < 256 && tiles(3) <= kCUs) tn = 3;
  else if (fmt == 1 ? mt <= 2 : mt == 1 && nt < 1024) tn = 2, waves = 4;
  if (tn == 0) return false;
  pl.cfg = kStream + tn - 1;
  pl.tiles = tiles(tn);
  pl.kg = waves;
  pl.ns = fmt == 0 ? 2 : 1;
  if (may_split && pl.tiles <= kCUs / 2 && nkb >= 512) {
    int64_t ks = std::min({(int64_t)8, kCUs / pl.tiles, nkb / 128});
    // Within the partial tiles' bytes of the staged plan for this shape (64 x 128 tiles in up to four
    // splits): a split must not take a call over the caller's or the library's scratch.  HiF4 stays
    // below it by its smaller activation records.  (m = 128, 131072 -> 256: 90 us staged, 33 in eight
    // splits, 37 in the four that fit; m = 64, 65536 -> 256 50.5, 21.9, 22.6.)
    if (fmt == 0) {
      const int64_t t = ((mt + 1) / 2) * ((nt + 3) / 4), staged = t * std::min((int64_t)4, kCUs / t) * (64 * 128);
      ks = std::min(ks, staged / (pl.tiles * tn * 1024));
    }
    pl.ksplit = (int)ks;
    pl.kper = (nkb + pl.ksplit - 1) / pl.ksplit;
    pl.partial_bytes = (size_t)pl.tiles * pl.ksplit * (tn * 1024) * sizeof(float);
  }
  return true;
}

Plan plan(int fmt, int64_t M, int64_t N, int64_t K, bool may_split) {
  const int64_t mt = (M + 31) / 32, nt = (N + 31) / 32, nkb = (K + 63) / 64;
  auto wgs = [&](int64_t bm, int64_t bn) { return ((mt + bm - 1) / bm) * ((nt + bn - 1) / bn); };
  Plan pl{};
  pl.ksplit = 1;
  pl.kper = nkb;
  if (M == 0 || N == 0) may_split = false;  // no tiles, whose number divides the CUs below
  if (stream_plan(fmt, M, mt, nt, nkb, may_split, pl)) return pl;
  if (wgs(4, 4) < 240 && may_split && nkb >= 128 && kCUs / wgs(2, 4) >= 2) {
    // small grids with long K (the down projection of a decode batch): 64 x 128 tiles with K
    // split up to four ways; the wider tile reads each activation fragment for twice the
    // columns (measured at m = 256, 11008 -> 2048: MXFP4 24 -> 21 us, HiF4 30 -> 27 us)
    pl.cfg = kNarrow;
    pl.tiles = wgs(2, 4);
    int64_t ks = kCUs / pl.tiles;
    ks = ks > 4 ? 4 : ks;
    pl.ksplit = (int)ks;
    pl.kper = (nkb + ks - 1) / ks;
    pl.partial_bytes = (size_t)pl.tiles * pl.ksplit * (64 * 128) * sizeof(float);
    pl.kg = fmt == 0 ? 1 : 2;
    pl.ns = fmt == 0 ? 4 : 2;
    return pl;
  }
  if (wgs(4, 4) < 240 && may_split && nkb >= 128) {
    // small grids with long K whose 64 x 128 tiles already fill the CUs (the 7B down
    // projection at m = 512): the wide tiles with K split, which read each activation fragment
    // for 2-4x the columns of the 64 x 64 tiles in K groups and each weight fragment for twice
    // the rows (measured at m = 512, 18944 -> 3584: MXFP4 54 -> 45 us as 128 x 256 in four
    // splits; HiF4 146 -> 97 us as 128 x 192 in six splits, two workgroups per CU)
    const bool mx = fmt == 0;
    pl.cfg = mx ? kWide : kMid;
    pl.tiles = mx ? wgs(4, 8) : wgs(4, 6);
    int64_t ks = (mx ? kCUs : 2 * kCUs) / pl.tiles;
    ks = ks < 2 ? 2 : ks > 8 ? 8 : ks;
    pl.ksplit = (int)ks;
    pl.kper = (nkb + ks - 1) / ks;
    pl.partial_bytes = (size_t)pl.tiles * pl.ksplit * (kTileRows[pl.cfg] * kTileCols[pl.cfg]) * sizeof(float);
    pl.kg = 1;
    pl.ns = mx ? 4 : 2;
    return pl;
  }
  if (wgs(4, 4) < 240) {
    // small grids (no K split: the long-K ones that would gain from one take the tiles
    // above, and the backward never splits)
    pl.cfg = kSmall;
    pl.tiles = wgs(2, 2);
    // K groups and stages (measured).  Grids within the CUs: MXFP4 takes four K groups for
    // long K ranges (>= 128 steps per workgroup) and two otherwise, HiF4 two, with four
    // stages.  Grids beyond the CUs, where workgroups share CUs: long K ranges keep their
    // K groups with two stages (MXFP4 at m = 512, K = 18944: 73.0 us with four stages, 68.7
    // with two); shorter ones take one K group (HiF4 at m = 512, 3584 -> 4608: 47 us with
    // two K groups, 35 us with one and two stages; MXFP4: 21.6 us, 19.4 with one and four).
    const bool crowded = pl.tiles * pl.ksplit > kCUs;
    pl.ns = 4;
    if (fmt == 0) {
      pl.kg = pl.kper >= 128 ? 4 : 2;
      if (crowded) {
        if (pl.kg == 4) pl.ns = 2;
        else pl.kg = 1;
      }
    } else {
      pl.kg = 2;
      if (crowded) {
        pl.ns = 2;
        if (pl.kper < 128) pl.kg = 1;
      }
    }
  } else if (fmt == 0 && M < 512) {
    // MXFP4 decode batches with wide N (gate_up at m = 256): 64 x 128 tiles, one K group,
    // four stages (measured: 21.6-22.5 us as 128 x 192 tiles, 20.2-20.4 us)
    pl.cfg = kNarrow;
    pl.tiles = wgs(2, 4);
    pl.kg = 1;
    pl.ns = 4;
  } else {
    const bool wide = M >= 512 && fmt == 0;
    pl.cfg = wide ? kWide : kMid;
    pl.tiles = wide ? wgs(4, 8) : wgs(4, 6);
    pl.kg = 1;
    pl.ns = fmt == 0 ? 4 : 2;  // HiF4 fits two workgroups per CU at two stages
    // HiF4 grids within one workgroup per CU: eight waves per 128 x 192 tile (two per SIMD).
    // They take 168 registers each (one term; 198 with two), so a CU holds no second workgroup of
    // them, but two of four waves.  Whole calls in us, eight -> four waves, S_2:4 / no residual: 230
    // tiles (m = 256, 2048 -> 22016) 35.6 -> 37.9 / 29.5 -> 30.9, 256 tiles (m = 1024, 2048 ->
    // 6144) 41.1 -> 41.9 / 31.0 -> 31.6; 258 tiles (m = 256, 2048 -> 24700) 58.9 -> 49.5 / 48.0 ->
    // 37.0, 378 (m = 331, 12288 -> 24150, no residual) 287 -> 187, 508 (m = 512, 3584 -> 24384)
    // 105.6 -> 97.8 / 81.1 -> 66.4.
    if (fmt == 1 && pl.tiles <= kCUs) pl.cfg = kMid8;
  }
  return pl;
}

// Launches the configuration of the plan (RESQ_GEMM_CONFIGS, for HiF4 RESQ_HIF4_CONFIGS, for
// streamed plans RESQ_STREAM_CONFIGS); false if none matches.
bool launch_plan(const GemmParams& p, int fmt, const Plan& pl, int n_terms, hipStream_t s) {
  if (pl.cfg >= kStream) return launch_gemm_stream(p, fmt, pl.cfg - kStream + 1, pl.kg, pl.ns, n_terms, s);
  if (fmt == 1) return launch_gemm_hif4(p, pl.cfg, pl.ns, pl.kg, n_terms, s);
#define RESQ_GEMM_LAUNCH(F, C, WM, WN, TM, TN, NS, KG)                                  \
  if (fmt == F && pl.cfg == C && pl.ns == NS && pl.kg == KG) {                          \
    launch_cfg<F, WM, WN, TM, TN, NS, KG>(p, n_terms, s);                               \
    return true;                                                                          \
  }
  RESQ_GEMM_CONFIGS(RESQ_GEMM_LAUNCH)
#undef RESQ_GEMM_LAUNCH
  return false;
}

}  // namespace

namespace {
constexpr size_t kOffsetLimit = (size_t)kBad - (1u << 20);  // 32-bit buffer offsets with headroom
size_t al256(size_t x) { return (x + 255) / 256 * 256; }
}  // namespace

bool gemm_supported(int fmt, int64_t M, int64_t N, int64_t K, int n_terms) {
  const int bmode = fmt == 0 ? kPackMx : kPackHiB;
  // HiF4 activations are bounded at 48 bytes per lane record, above the 40 of their layout: the
  // largest sizes accepted do not depend on it
  const size_t af = fmt == 0 ? frag_bytes(kPackMx, M, K) : 3 * frag_bytes(kPackMx, M, K);
  const size_t a = (size_t)n_terms * (al256(af) + al256(frag_scale_bytes(M, K)));
  const size_t b = al256(frag_bytes(bmode, N, K)) + al256(frag_scale_bytes(N, K));
  return a < kOffsetLimit && b < kOffsetLimit;
}

size_t gemm_split_scratch(int fmt, int64_t M, int64_t N, int64_t K) {
  return plan(fmt, M, N, K, true).partial_bytes;
}

void gemm_plan_info(int fmt, int64_t M, int64_t N, int64_t K, bool may_split, int32_t info[4]) {
  const Plan pl = plan(fmt, M, N, K, may_split);
  info[0] = pl.cfg;
  info[1] = pl.ksplit;
  info[2] = pl.kg;
  info[3] = pl.ns;
}

bool launch_gemm(const GemmOperands& op, hipStream_t s) {
  if (op.M == 0 || op.N == 0) return true;
  const int amode = op.fmt == 0 ? kPackMx : kPackHiA, bmode = op.fmt == 0 ? kPackMx : kPackHiB;
  const size_t af = frag_bytes(amode, op.M, op.K), as = frag_scale_bytes(op.M, op.K);
  const size_t bf = frag_bytes(bmode, op.N, op.K), bs = frag_scale_bytes(op.N, op.K);
  if (op.a_bytes >= kOffsetLimit || op.b_bytes >= kOffsetLimit) return false;
  for (int t = 0; t < op.n_terms; ++t)
    if (op.a_frag_off[t] + af > op.a_bytes || op.a_sc_off[t] + as > op.a_bytes) return false;
  if (op.b_frag_off + bf > op.b_bytes || op.b_sc_off + bs > op.b_bytes) return false;
  const Plan pl = plan(op.fmt, op.M, op.N, op.K, op.partial != nullptr);
  GemmParams p{};
  p.ksplit = (uint32_t)pl.ksplit;
  p.kper = pl.kper;
  p.partial = op.partial;
  p.M = op.M; p.N = op.N; p.K = op.K;
  p.nkb = (op.K + 63) / 64;
  p.mt_tiles = (op.M + 31) / 32;
  p.nt_tiles = (op.N + 31) / 32;
  p.a = op.a; p.b = op.b;
  p.a_bytes = (uint32_t)op.a_bytes; p.b_bytes = (uint32_t)op.b_bytes;
  for (int t = 0; t < 2; ++t) {
    const int u = t < op.n_terms ? t : 0;
    p.a_frag_off[t] = (uint32_t)op.a_frag_off[u];
    p.a_sc_off[t] = (uint32_t)op.a_sc_off[u];
  }
  p.b_frag_off = (uint32_t)op.b_frag_off; p.b_sc_off = (uint32_t)op.b_sc_off;
  p.Y = op.Y; p.ldy = op.ldy; p.out_bf16 = op.out_bf16 ? 1 : 0;
  p.vec_y = (reinterpret_cast<uintptr_t>(op.Y) % 16 == 0 && op.ldy % 4 == 0) ? 1 : 0;
  return launch_plan(p, op.fmt, pl, op.n_terms, s);
}

}  // namespace resq
