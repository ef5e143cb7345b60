// Device code shared by the FP4 GEMM kernels (gemm.hip: MXFP4, gemm_hif4.hip: HiF4): launch
// parameters, the tile order, global -> LDS copies, waits and barriers, and the epilogue (K
// group reduction, split-K partials, the output tile through LDS).
#pragma once

#include "kernels.h"
#include "device_fp4.h"
#include "profiler.h"

namespace resq {

struct GemmParams {
  int64_t M, N, K, nkb, mt_tiles, nt_tiles;
  // Operand A: one buffer with the fragments and scale bytes of every term at these byte
  // offsets; operand B: one buffer with its fragments and scale bytes.
  const uint8_t* a;
  const uint8_t* b;
  uint32_t a_bytes, b_bytes;
  uint32_t a_frag_off[2], a_sc_off[2], b_frag_off, b_sc_off;
  void* Y;        // float32, or bf16 bits when out_bf16
  int64_t ldy;
  int out_bf16;   // store Y as bf16 (round to nearest, ties to even) instead of float32
  int vec_y;      // Y and ldy allow 16-byte stores of four consecutive outputs
  // grid bookkeeping (32-bit: the workgroup count is far below 2^31)
  uint32_t grid_m, grid_n, per_xcd, n_wg;
  // split-K: ksplit workgroups per tile, each over kper K steps, each writing its partial
  // tile (summed by splitk_reduce_kernel)
  uint32_t ksplit;
  int64_t kper;
  float* partial;
};

namespace {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void* lds_ptr_t;

constexpr int kXcds = 8;

// Output tile of linear tile index `tile`: tiles run in groups of kGroupRows row tiles;
// within a group, row tiles vary fastest, then column tiles.  A run of consecutive tiles (the
// workgroups resident on one XCD at a time) then covers a compact block of rows and columns
// that share their A row strips and B column strips in that XCD's L2.
constexpr uint32_t kGroupRows = 8;
__device__ __forceinline__ void tile_coords(uint32_t tile, uint32_t grid_m, uint32_t grid_n, uint32_t& wg_m,
                                            uint32_t& wg_n) {
  const uint32_t group = tile / (kGroupRows * grid_n);
  const uint32_t first = group * kGroupRows;
  const uint32_t rows = min(kGroupRows, grid_m - first);
  const uint32_t in = tile - first * grid_n;
  wg_m = first + in % rows;
  wg_n = in / rows;
}

// float32 -> bf16 bits, round to nearest, ties to even (finite inputs).
__device__ __forceinline__ uint16_t f32_to_bf16_rne(float x) {
  const uint32_t u = __float_as_uint(x);
  return (uint16_t)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}

__device__ __forceinline__ void store_y(void* Y, int64_t idx, float v, int out_bf16) {
  if (out_bf16) reinterpret_cast<uint16_t*>(Y)[idx] = f32_to_bf16_rne(v);
  else reinterpret_cast<float*>(Y)[idx] = v;
}

// Four consecutive outputs; Y + idx is 16-byte aligned (float32) or 8-byte aligned (bf16).
__device__ __forceinline__ void store_y4(void* Y, int64_t idx, const v4f& v, int out_bf16) {
  if (out_bf16) {
    const uint32_t lo = f32_to_bf16_rne(v[0]) | ((uint32_t)f32_to_bf16_rne(v[1]) << 16);
    const uint32_t hi = f32_to_bf16_rne(v[2]) | ((uint32_t)f32_to_bf16_rne(v[3]) << 16);
    *reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(Y) + idx) = make_uint2(lo, hi);
  } else {
    *reinterpret_cast<v4f*>(reinterpret_cast<float*>(Y) + idx) = v;
  }
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* p, uint32_t bytes) {
  // raw buffer (32-bit dwords, no swizzle); num_records = bytes bounds every access
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes, 0x00020000);
}

template <int FA, int FB>
__device__ __forceinline__ v16f mfma(const v8i& a, const v8i& b, const v16f& c, int sa, int sb) {
  return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, FA, FB, 0, sa, 0, sb);
}

// Buffer load of SZ bytes per lane into LDS: lane l's bytes land at lds + SZ * l.  The lane's
// offset is voff + soff (soff: the wave-uniform K advance); lanes whose voff lies past the
// buffer's num_records read zeros, and a zero-size buffer makes the whole copy read zeros.
template <int SZ>
__device__ __forceinline__ void copy_to_lds(__amdgpu_buffer_rsrc_t r, void* lds, uint32_t voff, uint32_t soff) {
  if constexpr (SZ == 16) __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_ptr_t)lds, 16, voff, soff, 0, 0);
  else __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_ptr_t)lds, 4, voff, soff, 0, 0);
}

// s_waitcnt on vmcnt only (expcnt and lgkmcnt left at their maxima).
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt field is 6 bits");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

// Workgroup barrier that also waits for this wave's LDS reads (lgkmcnt) but not for its
// outstanding LDS-destination copies (vmcnt is waited for explicitly).  __syncthreads()
// would wait for every outstanding copy; the memory clobber keeps the compiler from moving
// memory accesses across the barrier.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// The end of a GEMM workgroup, after its last copy has landed: sum the KG groups' accumulators,
// then store the tile (or this split's partial tile).  T0, N0: the workgroup's first row and
// column tile; kg, wt, wm, wn: this wave's K group, index within it, and row and column.
// LDS: the workgroup's LDS bytes.
template <int WM, int WN, int TM, int TN, int KG, size_t LDS>
__device__ __forceinline__ void finish_tile(const GemmParams& p, v16f (&acc)[TM][TN], uint8_t* smem, int kg, int wt,
                                            int wm, int wn, int lane, uint32_t T0, uint32_t N0, uint32_t tile,
                                            uint32_t split) {
  constexpr int WT = WM * WN, W = WT * KG;
  if constexpr (KG > 1) {
    // sum the K groups' accumulators in group order: groups 1.. park theirs in LDS, group 0
    // adds them and stores the tile
    __syncthreads();  // every wave is done with the stage buffers
    float* red = reinterpret_cast<float*>(smem);
    constexpr int PER = TM * TN * 16 * 64;  // floats per wave
    if (kg > 0) {
      float* dst = red + ((size_t)(kg - 1) * WT + wt) * PER;
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r) dst[((i * TN + j) * 16 + r) * 64 + lane] = acc[i][j][r];
    }
    __syncthreads();
    if (kg > 0) return;
#pragma unroll
    for (int g = 1; g < KG; ++g) {
      const float* src = red + ((size_t)(g - 1) * WT + wt) * PER;
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[i][j][r] += src[((i * TN + j) * 16 + r) * 64 + lane];
    }
  }

  if (p.ksplit > 1) {
    // split K: write this split's partial tile in register order (coalesced per wave)
    constexpr int TE = 64 * WT * TM * TN * 16;  // floats per tile
    float* part = p.partial + ((size_t)tile * p.ksplit + split) * TE + (size_t)wt * TM * TN * 16 * 64;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) part[((i * TN + j) * 16 + r) * 64 + lane] = acc[i][j][r];
    return;
  }

  // Y through LDS, eight rows at a time: accumulator registers 4q .. 4q+3 of a tile hold its
  // rows 8q .. 8q+7 (lanes 0-31 rows 8q .. 8q+3, lanes 32-63 rows 8q+4 .. 8q+7), so the wave
  // writes those registers of its TN tiles into its own LDS slot as an 8 x (TN x 32) row-major
  // block and reads it back 16 bytes per lane: each store then covers whole row segments of
  // TN x 32 columns, not 32 columns of two rows.  The slot is this wave's alone (K groups: its
  // reduction slot, already consumed; one group: after a barrier that ends every wave's reads
  // of the stage buffers), and one wave's LDS accesses complete in order, so only the
  // compiler needs to be kept from reordering them.
  constexpr int RW = TN * 32;  // floats per staged row
  static_assert(KG > 1 || (size_t)W * 8 * RW * 4 <= LDS, "staging slots fit the stage buffers");
  if constexpr (KG == 1) __syncthreads();
  float* slot = reinterpret_cast<float*>(smem) + (size_t)wt * (KG > 1 ? TM * TN * 16 * 64 : 8 * RW);
  const int half = lane >> 5, l32 = lane & 31;
  const int64_t col0 = ((int64_t)N0 + wn * TN) * 32;
  // read once: past each memory clobber below the parameters, and what is computed from them, would
  // be formed again (MXFP4, 41 alternating runs: backward m = 4096, 11008 x 2048 188.4 -> 184.9 us,
  // the 3B layer's four linears 636.4 -> 627.9; m = 256, 2048 -> 22016 21.1 -> 20.7; HiF4 within 0.5%)
  const int64_t M = p.M, N = p.N, ldy = p.ldy;
  const int out_bf16 = p.out_bf16;
  void* const Y = p.Y;
  bool wide[TN];  // a lane's columns of store s: one 16-byte store
#pragma unroll
  for (int s = 0; s < TN; ++s) wide[s] = p.vec_y && col0 + (4 * lane + 256 * s) % RW + 3 < N;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) slot[(4 * half + e) * RW + j * 32 + l32] = acc[i][j][4 * q + e];
      asm volatile("" ::: "memory");
      const int64_t row0 = ((int64_t)T0 + wm * TM + i) * 32 + 8 * q;
#pragma unroll
      for (int s = 0; s < TN; ++s) {
        const int f = 4 * lane + 256 * s;  // flat float index in the 8 x RW block
        const v4f v = *reinterpret_cast<const v4f*>(slot + f);
        const int64_t row = row0 + f / RW, col = col0 + f % RW;
        if (row < M) {
          if (wide[s]) {
            store_y4(Y, row * ldy + col, v, out_bf16);
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if (col + e < N) store_y(Y, row * ldy + col + e, v[e], out_bf16);
          }
        }
      }
      asm volatile("" ::: "memory");
    }
}

// Sum the ksplit partial tiles of each output tile in split order (deterministic) and store
// Y.  Partial element e = wave, tile (i, j), accumulator register r, lane -- the gemm_kernel
// register order; workgroup b handles the 1024 elements of one (wave, i, j) of one tile.
template <int WM, int WN, int TM, int TN>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const float* __restrict__ partial,
                                                            int ksplit, uint32_t grid_m, uint32_t grid_n,
                                                            int64_t M, int64_t N, void* __restrict__ Y,
                                                            int64_t ldy, int out_bf16) {
  constexpr int PARTS = WM * WN * TM * TN, TE = 1024 * PARTS;
  const uint32_t tile = blockIdx.x / PARTS;
  const int part = (int)(blockIdx.x % PARTS);
  uint32_t wg_m, wg_n;
  tile_coords(tile, grid_m, grid_n, wg_m, wg_n);
  const float* src = partial + (size_t)tile * ksplit * TE + part * 1024;
  const int ij = part % (TM * TN), wave = part / (TM * TN);
  const int i = ij / TN, j = ij % TN, wm = wave % WM, wn = wave / WM;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int e = threadIdx.x + 256 * q;  // register r = e / 64, lane = e % 64
    const int lane = e & 63, r = e >> 6;
    float v = src[e];
    for (int k = 1; k < ksplit; ++k) v += src[(size_t)k * TE + e];
    const int64_t row = ((int64_t)wg_m * WM * TM + wm * TM + i) * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
    const int64_t col = ((int64_t)wg_n * WN * TN + wn * TN + j) * 32 + (lane & 31);
    if (row < M && col < N) store_y(Y, row * ldy + col, v, out_bf16);
  }
}

// Grid bookkeeping, the GEMM launch and, with a K split, the reduction launch.
template <int WM, int WN, int TM, int TN, typename Kernel>
void launch_tiles(Kernel kernel, int kg, size_t lds, GemmParams p, hipStream_t s) {
  p.grid_m = (uint32_t)((p.mt_tiles + WM * TM - 1) / (WM * TM));
  p.grid_n = (uint32_t)((p.nt_tiles + WN * TN - 1) / (WN * TN));
  p.n_wg = p.grid_m * p.grid_n * p.ksplit;
  p.per_xcd = (p.n_wg + kXcds - 1) / kXcds;
  launch_timed(kernel, dim3(p.per_xcd * kXcds), dim3(64 * WM * WN * kg), (uint32_t)lds, s, p);
  if (p.ksplit > 1)
    launch_timed(splitk_reduce_kernel<WM, WN, TM, TN>, dim3(p.grid_m * p.grid_n * WM * WN * TM * TN), dim3(256),
                 0u, s, (const float*)p.partial, (int)p.ksplit, p.grid_m, p.grid_n, p.M, p.N, p.Y, p.ldy,
                 p.out_bf16);
}

}  // namespace
}  // namespace resq
