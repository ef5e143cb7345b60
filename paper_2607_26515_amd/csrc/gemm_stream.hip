// The GEMM for grids of few output tiles (decoding a few sequences up to a few hundred), both
// formats: gemm.hip's stream_plan() says which.
//
// Such a call streams the weights with little reuse to stage through LDS, and the staged loop
// spends its time on the latency of its stages: a barrier and a copy wait per step.  Here each
// wave loads its operands straight from memory into registers, U K steps ahead, without
// barriers.  A workgroup of W waves owns one row tile x TN column tiles, and its waves take the K
// steps in turn (wave w steps w, w + W, ..), so that the workgroup streams consecutive
// fragments; at the end the W partial tiles are added through LDS in wave order, in float64
// (deterministic).
// Lanes of rows past M load nothing.  U: one or two steps ahead are enough with 8 waves
// (HiF4 2048 -> 2048 at m = 16: 6.2 us with one, 6.6 with two, 8 with three: the loads past a
// short K's end cost more than the depth gains).  A row tile per workgroup, not two: 2048 ->
// 2048 at m = 128 takes 5.5 us (HiF4) with one, 8.3 with two.
#include "gemm_core.h"
#include "gemm_geo.h"
#include "gemm_hif4_geo.h"
#include "gemm_stream.h"

namespace resq {
namespace {

typedef int v2i __attribute__((ext_vector_type(2)));

__device__ __forceinline__ v4i load16(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
  return __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0));
}
__device__ __forceinline__ v2i load8(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
  return __builtin_bit_cast(v2i, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
}
__device__ __forceinline__ int load1(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
  return (int)(uint8_t)__builtin_amdgcn_raw_buffer_load_b8(r, voff, soff, 0);
}

template <int FMT, int NT, int TN, int W, int U>
__global__ __launch_bounds__(64 * W) void gemm_stream_kernel(GemmParams p) {
  extern __shared__ __attribute__((aligned(16))) float red[];  // W partial tiles of TN * 1024 floats
  constexpr uint32_t A_FRAG = FMT == 0 ? 1024 : kHiAFrag, B_FRAG = FMT == 0 ? 1024 : kHiBFrag;

  const uint32_t b = blockIdx.x;
  const uint32_t wgid = (b % kXcds) * p.per_xcd + b / kXcds;
  if (wgid >= p.n_wg) return;
  const uint32_t ntiles = p.grid_m * p.grid_n;
  const uint32_t split = p.ksplit == 1 ? 0u : wgid / ntiles;
  const uint32_t tile = wgid - split * ntiles;
  uint32_t T0, wg_n;
  tile_coords(tile, p.grid_m, p.grid_n, T0, wg_n);
  const uint32_t N0 = wg_n * TN, nkb = (uint32_t)p.nkb;
  const int tid = threadIdx.x, lane = tid & 63;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t kbeg = (uint32_t)(split * p.kper);
  const uint32_t klen = (uint32_t)min((int64_t)p.kper, p.nkb - kbeg);

  const __amdgpu_buffer_rsrc_t ra = make_rsrc(p.a, p.a_bytes), rb = make_rsrc(p.b, p.b_bytes);
  const __amdgpu_buffer_rsrc_t zero = make_rsrc(p.a, 0u);
  // this lane's operand offsets at K step 0 (kBad: past the edge, the loads return zeros)
  const bool row_in = (int64_t)T0 * 32 + (lane & 31) < p.M;
  uint32_t va[NT], vas[NT], vb[TN], vbs[TN];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    va[t] = row_in ? p.a_frag_off[t] + T0 * nkb * A_FRAG + lane * 16 : kBad;
    vas[t] = row_in ? p.a_sc_off[t] + T0 * nkb * 64 + lane : kBad;
  }
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const bool in = N0 + j < (uint32_t)p.nt_tiles;
    vb[j] = in ? p.b_frag_off + (N0 + j) * nkb * B_FRAG + lane * 16 : kBad;
    vbs[j] = in ? p.b_sc_off + (N0 + j) * nkb * 64 + lane : kBad;
  }
  // offsets of the 8-byte pieces (HiF4); kBad stays past the buffer
  const uint32_t tail = kHiTail - lane * 8;

  struct Step {
    v8i a[NT][FMT == 0 ? 1 : 2], b[TN];
    int sa[NT], sb[TN];
  };
  Step S[U];
  auto load = [&](Step& s, uint32_t i) {  // this wave's i-th K step (zeros past the end)
    const uint32_t k = wave + W * i;
    const bool in = k < klen;  // wave-uniform
    const __amdgpu_buffer_rsrc_t qa = in ? ra : zero, qb = in ? rb : zero;
    const uint32_t kb = kbeg + k;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const v4i x = load16(qb, vb[j], kb * B_FRAG);
      if constexpr (FMT == 0) {
        s.b[j] = v8i{x[0], x[1], x[2], x[3], 0, 0, 0, 0};
      } else {
        const v2i y = load8(qb, vb[j] == kBad ? kBad : vb[j] + tail, kb * B_FRAG);
        s.b[j] = v8i{x[0], x[1], x[2], x[3], y[0], y[1], 0, 0};
      }
      s.sb[j] = load1(qb, vbs[j], kb * 64u);
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const v4i x = load16(qa, va[t], kb * A_FRAG);
      if constexpr (FMT == 0) {
        s.a[t][0] = v8i{x[0], x[1], x[2], x[3], 0, 0, 0, 0};
      } else {
        const v2i y = load8(qa, row_in ? va[t] + tail : kBad, kb * A_FRAG);
        const v4i z = load16(qa, row_in ? va[t] + kHiLo : kBad, kb * A_FRAG);
        s.a[t][0] = v8i{x[0], x[1], x[2], x[3], y[0], y[1], 0, 0};
        s.a[t][1] = v8i{z[0], z[1], z[2], z[3], 0, 0, 0, 0};
      }
      s.sa[t] = load1(qa, vas[t], kb * 64u);
    }
  };

  v16f acc[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[j][r] = 0.f;
  auto multiply = [&](const Step& s) {
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      if constexpr (FMT == 0) {
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[j] = mfma<4, 4>(s.a[t][0], s.b[j], acc[j], s.sa[t], s.sb[j]);
      } else {
        v16f P = v16f{};
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          P = mfma<2, 2>(s.a[t][0], s.b[j], P, s.sa[t], kHiOne);
          P = mfma<4, 2>(s.a[t][1], s.b[j], P, s.sa[t], kHiLoScale);
        }
        const float f = hif4_fold_factor((uint32_t)s.sb[j]);
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[j][r] = fmaf(P[r], f, acc[j][r]);
      }
    }
  };

  const uint32_t n = wave < klen ? (klen - wave + W - 1) / W : 0u;  // this wave's K steps
#pragma unroll
  for (int u = 0; u < U; ++u) {
    load(S[u], u);
    __builtin_amdgcn_sched_barrier(0);  // steps stay in order: each waits for its own loads only
  }
  for (uint32_t i = 0; i < n; i += U)
#pragma unroll
    for (int u = 0; u < U; ++u) {
      multiply(S[u]);
      load(S[u], i + u + U);
      __builtin_amdgcn_sched_barrier(0);
    }

  // Add the waves' tiles in wave order, in float64 with one rounding: eight float32 additions at
  // nearly the result's magnitude would round more than the longer chains of fewer waves did
  // (HiF4, error against 64 bits: staged 4.5e-8, streamed 5.2e-8 in float32, 3.0e-8 so).
  // Accumulator registers 4q .. 4q+3 hold rows 8q .. 8q+7.
  const uint32_t rows = (uint32_t)min((int64_t)32, p.M - (int64_t)T0 * 32);
  constexpr int TE = TN * 1024;
#pragma unroll
  for (int q = 0; q < 4; ++q)
    if (8u * q < rows)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) red[wave * TE + (j * 16 + 4 * q + e) * 64 + lane] = acc[j][4 * q + e];
  __syncthreads();
  for (int e = tid; e < TE; e += 64 * W) {
    const int l = e & 63, r = (e >> 6) & 15, j = e >> 10;
    if (8u * (r >> 2) >= rows) continue;
    double sum = red[e];
#pragma unroll
    for (int w = 1; w < W; ++w) sum += (double)red[w * TE + e];
    const float v = (float)sum;
    if (p.ksplit > 1) {
      p.partial[((size_t)tile * p.ksplit + split) * TE + e] = v;
      continue;
    }
    const int64_t row = (int64_t)T0 * 32 + 8 * (r >> 2) + 4 * (l >> 5) + (r & 3);
    const int64_t col = ((int64_t)N0 + j) * 32 + (l & 31);
    if (row < p.M && col < p.N) store_y(p.Y, row * p.ldy + col, v, p.out_bf16);
  }
}

template <int FMT, int TN, int W, int U>
void launch(const GemmParams& p, int n_terms, hipStream_t s) {
  constexpr size_t lds = (size_t)W * TN * 1024 * 4;
  if (n_terms > 1) launch_tiles<1, 1, 1, TN>(gemm_stream_kernel<FMT, 2, TN, W, U>, W, lds, p, s);
  else launch_tiles<1, 1, 1, TN>(gemm_stream_kernel<FMT, 1, TN, W, U>, W, lds, p, s);
}

}  // namespace

bool launch_gemm_stream(const GemmParams& p, int fmt, int tn, int waves, int steps, int n_terms, hipStream_t s) {
#define RESQ_STREAM_LAUNCH(F, TN, W, U)                     \
  if (fmt == F && tn == TN && waves == W && steps == U) {   \
    launch<F, TN, W, U>(p, n_terms, s);                     \
    return true;                                            \
  }
  RESQ_STREAM_CONFIGS(RESQ_STREAM_LAUNCH)
#undef RESQ_STREAM_LAUNCH
  return false;
}

}  // namespace resq
