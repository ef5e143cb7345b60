// Global selections of the residual sparsity functions (paper Sec. 4.3): S_alpha% over
// channels, S^{32x64}_alpha% over 32-row x 64-column blocks, and an element-wise variant.
//
// Each one ranks items by a key computed from the dense Q(dX) (dequantized values), keeps the
// `keep` largest (floor(count * alpha / 100), the caller's count; alpha = 50 in the paper's
// experiments), and breaks ties by the lowest index:
//   channel j      : sum over rows i = 0, 1, ..., m-1 of value(i, j)^2, float64, in that order
//   block (I, J)   : over the block's rows in order, each row adding its per-scale-block sums
//                    (exact; written by the residual pass) in column order, float64
//   element (i, j) : |value(i, j)| (exact in float32), index i * d + j
// Non-negative IEEE keys order like their bit patterns, so the k-th largest key is found by a
// most-significant-digit-first radix select on the bits (channel and block keys: 10-bit digits from
// the first bit in which the float64 keys differ, 8-bit ones where the keys are streamed; element
// keys: exponent then mantissa digits), after which the keys equal to it are ranked by index.  Pruned codes become the +0 code in place.
#include "kernels.h"
#include "frag.h"
#include "hist.h"

namespace resq {
namespace {

constexpr int kThreads = 256;
constexpr int kSelThreads = 1024;   // single-workgroup select (channel and block keys)
constexpr int kWordsPerThread = 4;  // element-wise passes: 4 code words = 32 elements

// MXFP4: |value| of the 8 elements of one 32-bit code word, as float32 bit patterns (exact,
// denormals included), two per hardware conversion.
__device__ __forceinline__ void mx_word_keys(uint32_t cw, uint32_t scale, uint32_t key[8]) {
  const uint32_t mag = cw & 0x77777777u;  // magnitudes only
  const float sc = mx_scale_f32((int)scale - 127);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    float v0, v1;
    mx_value2((mag >> (8 * q)) & 0xFFu, sc, v0, v1);
    key[2 * q] = __float_as_uint(v0);
    key[2 * q + 1] = __float_as_uint(v1);
  }
}

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

// HiF4 keys of word Q of a scale word's codes (elements 8Q .. 8Q + 7, one level-2 group and two
// level-3 groups): value k (4 + m) 2^(e - 35 - b).  The eight magnitudes k spread to the bytes
// of two dwords, one 16-bit-lane multiply by 4 + m forms four products k (4 + m) <= 49 at once
// (no carry crosses a byte), each byte converts to float32 exactly, and ldexp applies the
// group's 2^(e - 35 - b) (exact: the smallest nonzero value, 4 * 2^-37, is normal).  f2 holds
// 4 + m in both 16-bit lanes, e35 = e - 35; l2 and l3 are the level-2 and level-3 shift bits from
// word 0's group on.
__device__ __forceinline__ void hif4_word_keys(uint32_t cw, uint32_t f2, int e35, uint32_t l2, uint32_t l3,
                                               int Q, uint32_t key[8]) {
  const uint32_t ta = __builtin_amdgcn_perm(cw, cw, 0x0C010C00u), tb = __builtin_amdgcn_perm(cw, cw, 0x0C030C02u);
  const uint32_t ka = (ta | (ta << 4)) & 0x07070707u, kb = (tb | (tb << 4)) & 0x07070707u;
  const uint32_t pa = __builtin_bit_cast(uint32_t, __builtin_bit_cast(u16x2, ka) * __builtin_bit_cast(u16x2, f2));
  const uint32_t pb = __builtin_bit_cast(uint32_t, __builtin_bit_cast(u16x2, kb) * __builtin_bit_cast(u16x2, f2));
  const int b2 = (int)((l2 >> Q) & 1u);
  const int ea = e35 - b2 - (int)((l3 >> (2 * Q)) & 1u), eb = e35 - b2 - (int)((l3 >> (2 * Q + 1)) & 1u);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    key[i] = __float_as_uint(ldexpf((float)((pa >> (8 * i)) & 0xFFu), ea));
    key[4 + i] = __float_as_uint(ldexpf((float)((pb >> (8 * i)) & 0xFFu), eb));
  }
}

// Scale word of element (row, j): MX E8M0 byte or the HiF4 meta word.
template <int FMT>
__device__ __forceinline__ uint32_t scale_at(const void* scales, int64_t row, int64_t d, int64_t j) {
  if constexpr (FMT == 0) return reinterpret_cast<const uint8_t*>(scales)[row * (d / 32) + j / 32];
  else return reinterpret_cast<const uint32_t*>(scales)[row * (d / 64) + j / 64];
}

// Wave scans and reductions through DPP (row shifts, then row 15 -> row broadcasts): a step is one
// vector instruction, where a shuffle is an LDS round trip.
// Lanes that a step gives no source take `none`.
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_take(uint32_t none, uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)none, (int)x, CTRL, ROWS, 0xF, false);
}
// Inclusive combination over the lanes up to this one: of its row of 16, or of the wave.
template <typename Op>
__device__ __forceinline__ uint32_t row_scan(uint32_t x, uint32_t none, Op op) {
  x = op(x, dpp_take<0x111, 0xF>(none, x));
  x = op(x, dpp_take<0x112, 0xF>(none, x));
  x = op(x, dpp_take<0x114, 0xF>(none, x));
  return op(x, dpp_take<0x118, 0xF>(none, x));
}
template <typename Op>
__device__ __forceinline__ uint32_t wave_scan(uint32_t x, uint32_t none, Op op) {
  x = row_scan(x, none, op);
  x = op(x, dpp_take<0x142, 0xA>(none, x));
  return op(x, dpp_take<0x143, 0xC>(none, x));
}
__device__ __forceinline__ uint32_t lane_value(uint32_t x, int lane) {
  return (uint32_t)__builtin_amdgcn_readlane((int)x, lane);
}

// a + b of the lanes N apart, in halves: lanes with (lane & N) == 0 get a's sum, the others b's.
template <int N>
__device__ __forceinline__ double swap_add(double a, double b) {
  const uint64_t x = (uint64_t)__double_as_longlong(a), y = (uint64_t)__double_as_longlong(b);
  uint32_t p[2][2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const uint32_t u = (uint32_t)(x >> (32 * h)), v = (uint32_t)(y >> (32 * h));
    if constexpr (N == 32) {
      const auto r = __builtin_amdgcn_permlane32_swap(u, v, false, false);
      p[0][h] = r[0]; p[1][h] = r[1];
    } else {
      const auto r = __builtin_amdgcn_permlane16_swap(u, v, false, false);
      p[0][h] = r[0]; p[1][h] = r[1];
    }
  }
  return __longlong_as_double((long long)((uint64_t)p[0][1] << 32 | p[0][0])) +
         __longlong_as_double((long long)((uint64_t)p[1][1] << 32 | p[1][0]));
}

// ---------------------------------------------------------------------------------------
// Channel keys.  Workgroup = 64 channels x all rows: a lane takes the 8 channels of one code word
// (4 bytes) in every 128th row, so that a wave's load is 8 rows of 32 consecutive bytes; 8 lanes'
// sums are combined in the wave, 16 waves' through LDS.  The result equals the defined row-by-row
// sum exactly whenever no float64 addition of either order rounds: every square v^2 is a multiple
// of 2^L, L = twice the exponent of the smallest step that a scale word of the channel's nonzero
// code words allows (MXFP4: half the scale; HiF4: a level-1 step of e - 37), so if the total is
// below 2^(L+53) every partial sum, in any order, is a multiple of 2^L below 2^(L+53) and thus
// exact.  The check uses 2^(L+52) to absorb any rounding of the computed total; a channel that
// fails it is summed again row by row in the defined order.
// One channel per lane (8-byte row pieces, a decode and a lowest-bit search per element) took
// 22.7 us at m = 512, d = 18944 and 6.0 us at d = 3584, MXFP4; this way 7.4 us and 4.8 us.
// ---------------------------------------------------------------------------------------
constexpr int kChanThreads = 1024;  // 16 waves
constexpr int kChanPerWg = 64;      // channels per workgroup
constexpr int kNoBit = 1 << 20;      // "no nonzero term yet" for the lowest-bit exponent

template <int FMT>
__device__ __forceinline__ float decode_at(uint32_t cbyte, uint32_t sc, int64_t j) {
  const uint32_t c = (cbyte >> (4 * (j & 1))) & 15u;
  if constexpr (FMT == 0) {
    float v0, v1;
    mx_value2(c, mx_scale_f32((int)sc - 127), v0, v1);
    return v0;
  } else {
    const int p = (int)(j & 63);
    const int b = (int)((sc >> (8 + p / 8)) & 1u) + (int)((sc >> (16 + p / 4)) & 1u);
    return hif4_value(c, (int)(sc & 0xFFu), b);
  }
}

template <int FMT>
__global__ __launch_bounds__(kChanThreads) void channel_keys_kernel(const uint8_t* __restrict__ codes,
                                                                    const void* __restrict__ scales,
                                                                    int64_t m, int64_t d,
                                                                    double* __restrict__ keys) {
  constexpr int NW = kChanThreads / 64, WPR = kChanPerWg / 8, RW = 64 / WPR, RS = NW * RW, U = 4;
  __shared__ double part[NW][kChanPerWg];
  __shared__ int low[NW][WPR];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int cq = lane % WPR;  // code word within the workgroup's 64 channels
  const int64_t j0 = (int64_t)blockIdx.x * kChanPerWg + 8 * cq;
  double acc[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] = 0.0;
  int lo = kNoBit;
  if (j0 < d) {  // d % 8 == 0
    for (int64_t r = wave * RW + lane / WPR; r < m; r += RS * U) {
      uint32_t cw[U], sc[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {  // loads issued together
        const int64_t row = r + u * RS;
        cw[u] = row < m ? *reinterpret_cast<const uint32_t*>(codes + row * (d / 2) + j0 / 2) : 0u;
        sc[u] = row < m ? scale_at<FMT>(scales, row, d, j0) : 0u;
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        uint32_t key[8];
        int step;
        if constexpr (FMT == 0) {
          mx_word_keys(cw[u], sc[u], key);
          step = (int)sc[u] - 128;
        } else {
          const int e = (int)((sc[u] >> 2) & 63u);
          hif4_word_keys(cw[u], (4u + (sc[u] & 3u)) * 0x00010001u, e - 35, sc[u] >> 8, sc[u] >> 16, cq, key);
          step = e - 37;
        }
        if (cw[u] & 0x77777777u) lo = min(lo, 2 * step);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const double v = (double)__uint_as_float(key[e]);
          acc[e] = fma(v, v, acc[e]);  // exact square: at most 6 significant bits in v
        }
      }
    }
  }
  // the wave's RW = 8 row lanes of each code word: halving exchanges leave one channel in each
  // lane (lane halves, then odd and even rows of 16 lanes swap in registers; then 8 lanes on)
  static_assert(RW == 8, "three halving exchanges");
#pragma unroll
  for (int e = 0; e < 4; ++e) acc[e] = swap_add<32>(acc[e], acc[e + 4]);
#pragma unroll
  for (int e = 0; e < 2; ++e) acc[e] = swap_add<16>(acc[e], acc[e + 2]);
  const bool up = (lane & 8) != 0;
  const uint64_t send = (uint64_t)__double_as_longlong(up ? acc[0] : acc[1]);
  const uint64_t got = (uint64_t)dpp_take<0x128, 0xF>(0u, (uint32_t)(send >> 32)) << 32 |
                       dpp_take<0x128, 0xF>(0u, (uint32_t)send);  // rotated by 8 within 16 lanes
  acc[0] = (up ? acc[1] : acc[0]) + __longlong_as_double((long long)got);
  const int ch = 8 * cq + ((lane & 32) ? 4 : 0) + ((lane & 16) ? 2 : 0) + (up ? 1 : 0);
  lo = min(lo, (int)dpp_take<0x128, 0xF>(0u, (uint32_t)lo));
  lo = min(lo, __shfl_xor(lo, 16, 64));
  lo = min(lo, __shfl_xor(lo, 32, 64));
  part[wave][ch] = acc[0];
  if (lane < WPR) low[wave][lane] = lo;
  __syncthreads();
  const int64_t j = (int64_t)blockIdx.x * kChanPerWg + threadIdx.x;
  if (threadIdx.x >= kChanPerWg || j >= d) return;  // thread c finishes channel c
  double sum = 0.0;
  lo = kNoBit;
#pragma unroll 4
  for (int w = 0; w < NW; ++w) {
    sum += part[w][threadIdx.x];
    lo = min(lo, low[w][threadIdx.x / 8]);
  }
  if (sum != 0.0 && !(sum < ldexp(1.0, lo + 52))) {
    // some addition may round: the defined order, rows 0 .. m-1
    sum = 0.0;
    for (int64_t r = 0; r < m; ++r) {
      const float v = decode_at<FMT>(codes[r * (d / 2) + j / 2], scale_at<FMT>(scales, r, d, j), j);
      sum += (double)v * (double)v;
    }
  }
  keys[j] = sum;
}

// ---------------------------------------------------------------------------------------
// Block keys: one thread per 32 x 64 block, rows in order, scale blocks in column order.
// ---------------------------------------------------------------------------------------
// Key of block t = (I, J): the per-scale-block sums of squares of its rows, rows in order,
// scale blocks (P per 64 columns) in column order.
template <int P>
__device__ __forceinline__ double block_key(const double* __restrict__ partials, int64_t m, int64_t d, int64_t t) {
  const int64_t nJ = d / 64;
  const int64_t I = (int64_t)((uint64_t)t / (uint64_t)nJ), J = t - I * nJ;
  const int64_t r1 = (32 * I + 32 < m) ? 32 * I + 32 : m;
  const int64_t ld = d / 64 * P;  // scale blocks per row
  double acc = 0.0;
#pragma unroll 1
  for (int h = 0; h < 32; h += 16) {  // 16 rows at a time: their loads issued together
    double v[16][P];
#pragma unroll
    for (int i = 0; i < 16; ++i)
#pragma unroll
      for (int q = 0; q < P; ++q)
        v[i][q] = 32 * I + h + i < r1 ? partials[(32 * I + h + i) * ld + J * P + q] : 0.0;
#pragma unroll
    for (int i = 0; i < 16; ++i)  // rows in order, scale blocks in column order
#pragma unroll
      for (int q = 0; q < P; ++q)
        if (32 * I + h + i < r1) acc += v[i][q];
  }
  return acc;
}

template <int FMT>
__global__ __launch_bounds__(kThreads) void block_keys_kernel(const double* __restrict__ partials,
                                                              int64_t m, int64_t d,
                                                              double* __restrict__ keys) {
  const int64_t t = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (t < ((m + 31) / 32) * (d / 64)) keys[t] = block_key<FMT == 0 ? 2 : 1>(partials, m, d, t);
}

// ---------------------------------------------------------------------------------------
// Workgroup-wide exclusive scan of one uint32 per thread (any multiple of 64 threads).
// ---------------------------------------------------------------------------------------
template <int NT, typename T = uint32_t>
__device__ __forceinline__ T block_exclusive_scan(T v, T* wsum, T& total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  T x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const T y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) wsum[wave] = x;
  __syncthreads();
  T before = 0, all = 0;
#pragma unroll
  for (int w = 0; w < NT / 64; ++w) {
    const T s = wsum[w];
    if (w < wave) before += s;
    all += s;
  }
  __syncthreads();
  total = all;
  return before + x - v;
}

// Radix digit choice over an LDS histogram of nb <= NT bins: the digit holding the k-th
// largest key (k >= 1; k = 0 picks the top digit) and k's rank among the keys with that digit.
// A suffix scan over the bins runs on all threads; every thread of the block must call this,
// and all read the result from out[0] (digit) and out[1] (rank) after it returns.
template <int NT>
__device__ __forceinline__ void choose_digit(const uint32_t* hist, int nb, uint32_t k,
                                             uint32_t* wsum, uint32_t* out) {
  const int tid = threadIdx.x;
  const uint32_t v = tid < nb ? hist[nb - 1 - tid] : 0u;  // bins from the top down
  uint32_t total;
  const uint32_t above = block_exclusive_scan<NT>(v, wsum, total);  // keys in higher bins
  if (tid < nb && ((above < k && k <= above + v) || (k == 0 && tid == 0))) {
    out[0] = (uint32_t)(nb - 1 - tid);
    out[1] = k - above;
  }
  __syncthreads();
}

// ---------------------------------------------------------------------------------------
// Single-workgroup top-k over n float64 keys -> bit mask (bit b of byte i = item 8i + b).
// Thread t owns keys t, t + 1024, ...  Their upper 32 bits below the sign, t = key >> 31, lie in
// LDS as t' = t less the smallest nonzero t (plus one; 0 stays 0): the same order, and the
// first digit starts at the highest bit in which they differ.  Digit passes of 10 bits narrow
// the threshold; once the keys sharing its digits fit one per thread, their whole bit patterns are
// fetched, one per thread, and once they fit one wave they are ranked directly.  Only where
// more than 1024 keys agree in all of t' do passes over the whole keys (from global memory) follow.  The
// threshold's ties are ranked in index order from a table of per-slot, per-wave tie counts
// that one wave scans, unless all of them are kept.
//
// What bounds it is one workgroup's latency: barriers, LDS round trips and, on a kernel that runs
// each instruction only a few times, fetching its code.  So the loops over a thread's keys stay
// rolled, which is why the keys lie in LDS; with up to 20 keys per thread in registers (every loop
// unrolled, 21 KB of code) and 8-bit digits at byte positions, 18944 keys took 22.0 us and
// 3584 keys 9.7 us, now 15.1 to 17.0 us and 7.4 to 8.5 us.
// ---------------------------------------------------------------------------------------
constexpr int kMaxTopKeys = 20480;  // t' in LDS: 80 KB

// BLOCKS: the keys (at most 1024) are the block keys, summed here from `partials` and left in `keys`.
template <bool BLOCKS>
__global__ __launch_bounds__(kSelThreads) void select_top_kernel(uint64_t* __restrict__ keys,
                                                                 const double* __restrict__ partials,
                                                                 int64_t m, int64_t d, int n, uint32_t k,
                                                                 uint8_t* __restrict__ bits,
                                                                 uint8_t* __restrict__ bits_copy) {
  constexpr int NW = kSelThreads / 64;
  constexpr int BITS = 10, NB = 1 << BITS;   // one bin per thread
  constexpr int HW = kLdsCopies * (NB + 1);  // hist.h copies
  constexpr int LOW = 31;                    // key bits below t
  static_assert(NW == 16, "one row of lanes holds the waves' values");
  static_assert(NB == kSelThreads, "thread t chooses among the digits at bin NB - 1 - t");
  __shared__ uint32_t tk[kMaxTopKeys];
  __shared__ uint32_t hist[HW];
  __shared__ uint32_t wsum[NW], red_min[NW], red_max[NW], red_low[NW];
  __shared__ uint32_t list[kSelThreads];
  __shared__ uint64_t few[64];
  __shared__ uint64_t found;
  __shared__ uint32_t ch[3], fch[2], nlist, nfew;
  __shared__ uint32_t tcnt[kMaxTopKeys / 64];  // [slot][wave]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint64_t below = (1ull << lane) - 1ull;  // lanes before this one
  constexpr uint64_t kLowMask = (1ull << LOW) - 1ull;

  for (int i = tid; i < HW; i += kSelThreads) hist[i] = 0;
  if (tid == 0) { nlist = 0; nfew = 0; }
  // tbase: one less than the smallest nonzero t; low: the OR of the bits below t
  uint32_t tbase = ~0u, tmax = 0, low = 0;
  if constexpr (BLOCKS) {
    if (tid < n) {
      const uint64_t key = (uint64_t)__double_as_longlong(block_key<1>(partials, m, d, tid));
      keys[tid] = key;
      tk[tid] = tmax = (uint32_t)(key >> LOW);
      tbase = tmax - 1u;  // 0 wraps to the top
      low = (uint32_t)(key & kLowMask);
    } else {
      tk[tid] = 0;
    }
  } else {
    constexpr int U = 10;  // loads in flight per thread
    for (int i0 = tid; i0 - tid < n; i0 += U * kSelThreads) {
      uint64_t v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] = i0 + u * kSelThreads < n ? keys[i0 + u * kSelThreads] : 0;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const uint32_t t = (uint32_t)(v[u] >> LOW);
        if (u * kSelThreads + i0 - tid < n) tk[i0 + u * kSelThreads] = t;  // past n: 0
        tbase = min(tbase, t - 1u);
        tmax = max(tmax, t);
        low |= (uint32_t)(v[u] & kLowMask);
      }
    }
  }
  const auto umin = [](uint32_t x, uint32_t y) { return min(x, y); };
  const auto umax = [](uint32_t x, uint32_t y) { return max(x, y); };
  const auto uor = [](uint32_t x, uint32_t y) { return x | y; };
  const auto uadd = [](uint32_t x, uint32_t y) { return x + y; };
  tbase = wave_scan(tbase, ~0u, umin);
  tmax = wave_scan(tmax, 0u, umax);
  low = wave_scan(low, 0u, uor);
  if (lane == 63) { red_min[wave] = tbase; red_max[wave] = tmax; red_low[wave] = low; }
  __syncthreads();  // also ends the clearing
  tbase = lane_value(row_scan(red_min[lane % NW], ~0u, umin), NW - 1);
  tmax = lane_value(row_scan(red_max[lane % NW], 0u, umax), NW - 1);
  low = lane_value(row_scan(red_low[lane % NW], 0u, uor), NW - 1);
  // no key has a bit below t (sums of few-bit squares often have none): the passes end there
  const int end = low ? 0 : LOW;
  const uint32_t top = tmax ? tmax - tbase : 0u;
  // f(slot, item, t) for the slots in batches of B, whose LDS reads are issued together.  The items
  // past n in the last slot count as further zero keys: they rank after every real one.
  constexpr int B = 5;
  auto each = [&](auto f) {
#pragma unroll 1
    for (int q0 = 0; q0 * kSelThreads < n; q0 += B) {
      uint32_t t[B];
#pragma unroll
      for (int u = 0; u < B; ++u) t[u] = (q0 + u) * kSelThreads < n ? tk[(q0 + u) * kSelThreads + tid] : 0u;
#pragma unroll
      for (int u = 0; u < B; ++u)
        if ((q0 + u) * kSelThreads < n) f(q0 + u, (q0 + u) * kSelThreads + tid, t[u]);
    }
  };

  // threshold T (in the terms (t' << LOW) + low bits): the keys above it are kept, and krem of the
  // `ties` equal to it, in index order
  uint64_t T = 0;
  const int slots = (n + kSelThreads - 1) / kSelThreads;
  uint32_t krem = k, ties = (uint32_t)(slots * kSelThreads);
  int shift = LOW + (top ? 32 - __builtin_clz(top) : 0);  // bits not yet fixed
  uint64_t prefix = 0;                                     // T's fixed bits, shifted down by `shift`
  uint64_t mine = 0;                                       // this thread's gathered key
  bool first = true, gathered = false, have = false;
  if (k == 0) shift = end;
#pragma unroll 1
  while (shift > end) {
    const int s2 = max(shift - BITS, shift > LOW ? LOW : 0);
    const uint32_t dm = (1u << (shift - s2)) - 1u;
    if (first && shift > LOW) {  // every key counts; t becomes t'
      each([&](int, int i, uint32_t t) {
        t = max(t, tbase) - tbase;
        tk[i] = t;
        hist_add_copies(hist, NB, t >> (s2 - LOW), true);
      });
      first = false;
    } else if (gathered) {
      hist_add_copies(hist, NB, (uint32_t)(mine >> s2) & dm, have);
    } else if (shift > LOW) {
      each([&](int, int, uint32_t t) {
        hist_add_copies(hist, NB, (t >> (s2 - LOW)) & dm, t >> (shift - LOW) == (uint32_t)prefix);
      });
    } else {  // more than 1024 keys agree in t'
      const uint32_t tt = (uint32_t)(prefix >> (LOW - shift));
#pragma unroll 1
      for (int i = tid; i < n; i += kSelThreads) {
        if (tk[i] != tt) continue;
        const uint64_t v = ((uint64_t)tt << LOW) | (keys[i] & kLowMask);
        hist_add_copies(hist, NB, (uint32_t)(v >> s2) & dm, v >> shift == prefix);
      }
    }
    __syncthreads();
    // digit choice: thread t holds bin NB - 1 - t, and clears it for the next pass
    const uint32_t sum = hist_sum_copies(hist, NB, NB - 1 - tid);
#pragma unroll
    for (int c = 0; c < kLdsCopies; ++c) hist[c * (NB + 1) + NB - 1 - tid] = 0;
    const uint32_t incl = wave_scan(sum, 0u, uadd);
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    const uint32_t before = row_scan(lane < wave ? wsum[lane % NW] : 0u, 0u, uadd);  // lower waves' sums
    const uint32_t over = lane_value(before, NW - 1) + incl - sum;  // keys in higher bins
    if (over < krem && krem <= over + sum) {
      ch[0] = (uint32_t)(NB - 1 - tid);
      ch[1] = krem - over;
      ch[2] = sum;
    }
    __syncthreads();
    prefix = (prefix << (shift - s2)) | ch[0];
    krem = ch[1];
    ties = ch[2];
    shift = s2;
    have = have && mine >> shift == prefix;
    if (shift == end) break;
    if (!gathered && shift >= LOW && ties <= (uint32_t)kSelThreads) {
      // the candidates' indices, in any order (what follows only counts them), then their keys
      const int ts = shift - LOW;
      const uint32_t p = (uint32_t)prefix;
      uint32_t cnt = 0;
      each([&](int, int, uint32_t t) { cnt += t >> ts == p; });
      const uint32_t upto = wave_scan(cnt, 0u, uadd);
      uint32_t base = 0;
      if (lane == 63 && upto) base = atomicAdd(&nlist, upto);
      base = lane_value(base, 63) + upto - cnt;
      each([&](int, int i, uint32_t t) {
        if (t >> ts == p) list[base++] = (uint32_t)i;
      });
      __syncthreads();
      have = tid < (int)ties;
      if (have) {
        const uint32_t i = list[tid];
        mine = ((uint64_t)tk[i] << LOW) | ((int)i < n ? keys[i] & kLowMask : 0);
      }
      gathered = true;
    }
    if (gathered && ties <= 64u) {
      if (have) few[atomicAdd(&nfew, 1u)] = mine;
      __syncthreads();
      if (wave == 0) {
        const bool in = lane < (int)ties;
        const uint64_t x = in ? few[lane] : 0;
        uint32_t more = 0, same = 0;
#pragma unroll 8
        for (uint32_t i = 0; i < ties; ++i) {
          const uint64_t o = few[i];
          more += o > x;
          same += o == x;
        }
        if (in && more < krem && krem <= more + same) {  // equal keys write equal values
          found = x;
          fch[0] = krem - more;
          fch[1] = same;
        }
      }
      __syncthreads();
      prefix = found >> end;
      krem = fch[0];
      ties = fch[1];
      shift = end;
    }
  }
  T = prefix << end;
  const uint32_t Tt = (uint32_t)(T >> LOW);
  const bool rank_ties = krem != 0 && krem != ties;  // else all or none of them are kept
  // Where bits below t' count, the keys with T's t' get their order against T into t: one up, one
  // down or as it is.  (No key but 0 is below 2^-1000 and t = ~0 would be a NaN of all ones: neither
  // step wraps.)
  if (end == 0 && k != 0) {
    auto settle = [&](int i, uint64_t v) { tk[i] += v > T ? 1u : v < T ? ~0u : 0u; };
    if (gathered) {
      __syncthreads();
      if (tid < (int)nlist && (uint32_t)(mine >> LOW) == Tt) settle((int)list[tid], mine);
    } else {
#pragma unroll 1
      for (int i = tid; i < n; i += kSelThreads)
        if (tk[i] == Tt) settle(i, ((uint64_t)Tt << LOW) | (keys[i] & kLowMask));
    }
    __syncthreads();
  }
  if (rank_ties) {
    uint32_t c = 0;  // lane q: slot q's ties in this wave
    each([&](int q, int, uint32_t t) {
      const uint32_t b = (uint32_t)__popcll(__ballot(t == Tt));
      c = lane == q ? b : c;
    });
    if (lane < slots) tcnt[lane * NW + wave] = c;
    __syncthreads();
    // exclusive prefix of the tie counts in index order (slot-major, then wave), by wave 0
    if (wave == 0) {
      uint32_t run = 0;
#pragma unroll 1
      for (int e0 = 0; e0 < slots * NW; e0 += 64) {
        const uint32_t v = e0 + lane < slots * NW ? tcnt[e0 + lane] : 0u;
        const uint32_t incl = wave_scan(v, 0u, uadd);
        if (e0 + lane < slots * NW) tcnt[e0 + lane] = run + incl - v;
        run += lane_value(incl, 63);
      }
    }
    __syncthreads();
  }
  // keep bits: lane q takes slot q's 8 bytes of this wave's keys
  const uint64_t ties_kept = krem != 0 && !rank_ties ? ~0ull : 0ull;
  const uint32_t r0 = rank_ties && lane < slots ? tcnt[lane * NW + wave] : 0u;
  uint64_t mask = 0;
  each([&](int q, int, uint32_t t) {
    const uint64_t eq = __ballot(t == Tt);
    uint64_t bal = __ballot(t > Tt) | (eq & ties_kept);
    if (rank_ties && eq != 0)
      bal |= __ballot(t == Tt && lane_value(r0, q) + (uint32_t)__popcll(eq & below) < krem);
    mask = lane == q ? bal : mask;
  });
  if (k == 0) mask = 0;
  const int i0 = lane * kSelThreads + wave * 64;
  if (lane < slots && i0 < n) {
    const bool wide = ((uintptr_t)bits % 8 == 0) && (bits_copy == nullptr || (uintptr_t)bits_copy % 8 == 0);
    if (wide && i0 + 64 <= n) {
      *reinterpret_cast<uint64_t*>(bits + (i0 >> 3)) = mask;
      if (bits_copy) *reinterpret_cast<uint64_t*>(bits_copy + (i0 >> 3)) = mask;
    } else {
      for (int e = 0; e < 64 && i0 + e < n; e += 8) {
        bits[(i0 + e) >> 3] = (uint8_t)(mask >> e);
        if (bits_copy) bits_copy[(i0 + e) >> 3] = (uint8_t)(mask >> e);
      }
    }
  }
}

// ---------------------------------------------------------------------------------------
// The same top-k for more keys than select_top_kernel's LDS holds (n > kMaxTopKeys):
// each radix pass streams the keys from global memory (they stay in L2), and the threshold's
// ties are ranked in index order chunk by chunk (1024 consecutive keys per chunk, one per
// thread, a workgroup scan per chunk).  One workgroup, so no cross-workgroup protocol.
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(kSelThreads) void select_top_stream_kernel(const uint64_t* __restrict__ keys,
                                                                        int64_t n, int64_t k,
                                                                        uint8_t* __restrict__ bits,
                                                                        uint8_t* __restrict__ bits_copy) {
  constexpr int NW = kSelThreads / 64;
  __shared__ uint32_t hc[kLdsCopies * 257];  // hist.h copies of the pass's 256 bins
  __shared__ uint32_t hist[256];             // their sums
  __shared__ uint32_t ch[2];
  __shared__ uint32_t wsum[NW];
  __shared__ uint64_t found;
  const int tid = threadIdx.x, lane = tid & 63;
  uint64_t prefix = 0, mask = 0;
  uint32_t krem = (uint32_t)k;
  for (int shift = 56; shift >= 0; shift -= 8) {
    for (int i = tid; i < kLdsCopies * 257; i += kSelThreads) hc[i] = 0;
    __syncthreads();
    for (int64_t base = 0; base < n; base += kSelThreads) {
      const int64_t i = base + tid;
      const uint64_t key = i < n ? keys[i] : 0;
      hist_add_copies(hc, 256, (uint32_t)((key >> shift) & 255u), i < n && (key & mask) == prefix);
    }
    __syncthreads();
    if (tid < 256) hist[tid] = hist_sum_copies(hc, 256, tid);
    __syncthreads();
    choose_digit<kSelThreads>(hist, 256, krem, wsum, ch);
    prefix |= (uint64_t)ch[0] << shift;
    krem = ch[1];
    mask |= (uint64_t)255 << shift;
    const uint32_t in_bin = hist[ch[0]];
    __syncthreads();
    if (in_bin == 1 && shift > 0) {
      // a single key has this prefix: it is the threshold
      for (int64_t base = 0; base < n; base += kSelThreads) {
        const int64_t i = base + tid;
        if (i < n && (keys[i] & mask) == prefix) found = keys[i];
      }
      __syncthreads();
      prefix = found;
      break;
    }
  }
  const uint64_t T = prefix;
  uint32_t seen = 0;  // ties in earlier chunks
  for (int64_t base = 0; base < n; base += kSelThreads) {
    const int64_t i = base + tid;
    const bool in = i < n;
    const uint64_t key = in ? keys[i] : 0;
    const bool tie = in && key == T;
    uint32_t total;
    const uint32_t rank = seen + block_exclusive_scan<kSelThreads>(tie ? 1u : 0u, wsum, total);
    const bool keep = in && (key > T || (tie && rank < krem));
    const uint64_t bal = __ballot(keep);
    if ((lane & 7) == 0 && in) {
      const uint8_t byte = (uint8_t)(bal >> lane);
      bits[i >> 3] = byte;
      if (bits_copy) bits_copy[i >> 3] = byte;
    }
    seen += total;
  }
}

void launch_top(double* keys, int64_t n, int64_t k, uint8_t* bits, uint8_t* bits_copy, hipStream_t s) {
  uint64_t* kk = (uint64_t*)keys;
  if (n <= kMaxTopKeys)
    hipLaunchKernelGGL((select_top_kernel<false>), dim3(1), dim3(kSelThreads), 0, s, kk, (const double*)nullptr,
                       (int64_t)0, (int64_t)0, (int)n, (uint32_t)k, bits, bits_copy);
  else
    hipLaunchKernelGGL(select_top_stream_kernel, dim3(1), dim3(kSelThreads), 0, s, (const uint64_t*)kk, n, k, bits, bits_copy);
}

// Block keys, then the top-k over them.  HiF4 blocks up to one per thread: the top-k sums the
// keys itself (one launch fewer; measured at m = 512, d = 3584: 10.0 us against 4.1 + 6.6 us).
// MXFP4 has two scale blocks per 64 columns, and one workgroup reading twice the partial sums
// takes longer than the separate key launch (12.0 us against 4.2 + 6.2 us).
void launch_block_top(int fmt, const double* partials, int64_t m, int64_t d, int64_t keep, const SelectWs& ws,
                      uint8_t* bits_copy, hipStream_t s) {
  const int64_t nb = ((m + 31) / 32) * (d / 64);
  if (fmt == 1 && nb <= kSelThreads) {
    hipLaunchKernelGGL((select_top_kernel<true>), dim3(1), dim3(kSelThreads), 0, s, (uint64_t*)ws.keys, partials,
                       m, d, (int)nb, (uint32_t)keep, ws.group_bits, bits_copy);
    return;
  }
  const dim3 g((unsigned)((nb + kThreads - 1) / kThreads));
  if (fmt == 0) hipLaunchKernelGGL((block_keys_kernel<0>), g, dim3(kThreads), 0, s, partials, m, d, ws.keys);
  else hipLaunchKernelGGL((block_keys_kernel<1>), g, dim3(kThreads), 0, s, partials, m, d, ws.keys);
  launch_top(ws.keys, nb, keep, ws.group_bits, bits_copy, s);
}

// Channel keys of the dense Q(dX), then the top-k over them.
void launch_channel_top(int fmt, const uint8_t* codes, const void* scales, int64_t m, int64_t d, int64_t keep,
                        const SelectWs& ws, uint8_t* bits_copy, hipStream_t s) {
  const dim3 g((unsigned)((d + kChanPerWg - 1) / kChanPerWg));
  if (fmt == 0) hipLaunchKernelGGL((channel_keys_kernel<0>), g, dim3(kChanThreads), 0, s, codes, scales, m, d, ws.keys);
  else hipLaunchKernelGGL((channel_keys_kernel<1>), g, dim3(kChanThreads), 0, s, codes, scales, m, d, ws.keys);
  launch_top(ws.keys, d, keep, ws.group_bits, bits_copy, s);
}

// Apply kept channels (KIND 0) or kept blocks (KIND 1): one thread per code word; grid x
// covers the d/8 words of a row, y the rows (grid-stride).
template <int KIND>
__global__ __launch_bounds__(kThreads) void apply_groups_kernel(uint32_t* __restrict__ codes,
                                                                int64_t m, int64_t d,
                                                                const uint8_t* __restrict__ gbits,
                                                                uint8_t* __restrict__ keep_mask) {
  const int64_t c8 = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (c8 >= d / 8) return;
  for (int64_t row = blockIdx.y; row < m; row += gridDim.y) {
    uint32_t kb;
    if constexpr (KIND == 0) {
      kb = gbits[c8];
    } else {
      const int64_t bit = (row / 32) * (d / 64) + c8 / 8;
      kb = ((gbits[bit >> 3] >> (bit & 7)) & 1u) ? 0xFFu : 0u;
    }
    const int64_t w = row * (d / 8) + c8;
    codes[w] &= nibble_mask8(kb);
    if (keep_mask) keep_mask[w] = (uint8_t)kb;
  }
}

// ---------------------------------------------------------------------------------------
// Element-wise 50%: radix select over the float32 |value| patterns of the decoded Q(dX).
// FP4 values of both formats have no set bits below mantissa bit 17 (MXFP4: at most two
// significant bits, subnormal only in bits 21-22; HiF4: k (4+m) < 64 at a normal exponent),
// so two digit passes fix the threshold exactly: the exponent field (bits 23-30, 256 bins),
// then mantissa bits 17-22 (64 bins) among the keys with the chosen exponent.
// hist: [0, 256) exponent counts, [256, 320) mantissa counts.  Each kernel after the first
// recomputes the choice from the histograms, so no workgroup waits for another.
// ---------------------------------------------------------------------------------------
constexpr int kUHist = kElemHistBins;       // hist.h: 256 exponent bins, then 64 mantissa bins
constexpr int kHistCopies = kElemHistCopies;  // hist.h: copies that readers sum

// Threshold ties.  The second pass counts, per workgroup, the keys of the chosen exponent by
// their six mantissa bits; the threshold is one of those 64 patterns and FP4 keys have no
// lower bits, so that table holds every workgroup's tie count for whichever threshold the
// pass's global histogram then fixes.  The counts are also summed per group of kSuper
// workgroups, so that a workgroup finds the ties of all earlier workgroups in
// O(nwg / kSuper + kSuper) reads.  A group's sums are kSuperCopies copies (workgroup w adds
// into copy w % kSuperCopies), so that the atomics of a group's workgroups do not all hit one
// address; with a single group no workgroup reads them, and none are formed.
constexpr int kSuper = 256;
constexpr int kSuperCopies = 8;
constexpr int kMantBins = 64;

__global__ void uzero_kernel(uint32_t* hist, int words) {
  for (int i = threadIdx.x; i < words; i += blockDim.x) hist[i] = 0;
}

// A thread's 32 elements (4 words of codes from word w0, one scale block): the raw codes and
// scale, loaded before the threshold is known so that their latency overlaps its reads, then
// the keys.
struct ThreadWords {
  uint4 cw;
  uint32_t sc;
  int jpos;
};

template <int FMT>
__device__ __forceinline__ ThreadWords thread_words(const uint8_t* codes, const void* scales, int64_t d, int64_t w0) {
  ThreadWords t;
  t.cw = *reinterpret_cast<const uint4*>(codes + 4 * w0);
  const uint32_t e0 = (uint32_t)(8 * w0), row = e0 / (uint32_t)d, j = e0 - row * (uint32_t)d;
  t.sc = scale_at<FMT>(scales, row, d, j);
  t.jpos = FMT == 0 ? 0 : (int)(j & 63);
  return t;
}

template <int FMT>
__device__ __forceinline__ void thread_keys(const ThreadWords& t, uint32_t key[32]) {
  if constexpr (FMT == 1) {
    const uint32_t f2 = (4u + (t.sc & 3u)) * 0x00010001u;
    const int e35 = (int)((t.sc >> 2) & 63u) - 35;
    const uint32_t l2 = t.sc >> (8 + t.jpos / 8), l3 = t.sc >> (16 + t.jpos / 4);
    hif4_word_keys(t.cw.x, f2, e35, l2, l3, 0, key);
    hif4_word_keys(t.cw.y, f2, e35, l2, l3, 1, key + 8);
    hif4_word_keys(t.cw.z, f2, e35, l2, l3, 2, key + 16);
    hif4_word_keys(t.cw.w, f2, e35, l2, l3, 3, key + 24);
  } else {
    mx_word_keys(t.cw.x, t.sc, key);
    mx_word_keys(t.cw.y, t.sc, key + 8);
    mx_word_keys(t.cw.z, t.sc, key + 16);
    mx_word_keys(t.cw.w, t.sc, key + 24);
  }
}

// Resolve the threshold from the global histogram (all threads call this; wave 0 reads the
// histogram, summing its copies, and scans it, one barrier for the rest): out[0] = exponent
// digit, out[1] = rank within it; with full, out[2] = threshold key T and out[3] = the number
// of keys equal to T that are kept.  Lane l holds exponent bins 255 - 4l .. 252 - 4l and
// mantissa bin 63 - l, each digit chosen as by a scan from the top bin down.
__device__ __forceinline__ void load_choice(const uint32_t* hist, uint32_t k, bool full, uint32_t* out) {
  if (threadIdx.x < 64) {
    const int lane = threadIdx.x;
    uint32_t v[4] = {0u, 0u, 0u, 0u}, mv = 0u;
#pragma unroll
    for (int c = 0; c < kHistCopies; ++c) {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] += hist[c * kUHist + 255 - 4 * lane - e];
      if (full) mv += hist[c * kUHist + 256 + 63 - lane];
    }
    // exponent digit: the bin holding the k-th largest key (k = 0: the top bin)
    const uint32_t sum = v[0] + v[1] + v[2] + v[3];
    uint32_t incl = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t y = __shfl_up(incl, o, 64);
      if (lane >= o) incl += y;
    }
    uint32_t above = incl - sum, de = 0, ke = 0;
    bool found = false;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if ((above < k && k <= above + v[e]) || (k == 0 && lane == 0 && e == 0)) {
        de = (uint32_t)(255 - 4 * lane - e);
        ke = k - above;
        found = true;
      }
      above += v[e];
    }
    uint64_t who = __ballot(found);
    int src = who ? __ffsll((unsigned long long)who) - 1 : 0;
    de = __shfl(de, src, 64);
    ke = __shfl(ke, src, 64);
    if (full) {
      // mantissa digit among the keys of exponent de, for rank ke
      uint32_t mincl = mv;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(mincl, o, 64);
        if (lane >= o) mincl += y;
      }
      const uint32_t mabove = mincl - mv;
      const bool hit = (mabove < ke && ke <= mabove + mv) || (ke == 0 && lane == 0);
      who = __ballot(hit);
      src = who ? __ffsll((unsigned long long)who) - 1 : 0;
      const uint32_t dm = (uint32_t)(63 - src), krem = __shfl(ke - mabove, src, 64);
      if (lane == 0) {
        out[2] = (de << 23) | (dm << 17);
        out[3] = krem;
      }
    }
    if (lane == 0) {
      out[0] = de;
      out[1] = ke;
    }
  }
  __syncthreads();
}

template <int FMT, int PASS>
__global__ __launch_bounds__(kThreads) void uhist_kernel(const uint8_t* __restrict__ codes,
                                                         const void* __restrict__ scales, int64_t m,
                                                         int64_t d, uint32_t keep,
                                                         uint32_t* __restrict__ hist,
                                                         uint32_t* __restrict__ super_counts,
                                                         uint32_t* __restrict__ tie_counts) {
  constexpr int NB = PASS == 0 ? 256 : 64, OFF = PASS == 0 ? 0 : 256;
  __shared__ uint32_t lc[kLdsCopies * (NB + 1)];  // this workgroup's counts (hist.h copies)
  __shared__ uint32_t ch[4];
  const int tid = threadIdx.x;
  const int64_t w0 = ((int64_t)blockIdx.x * kThreads + tid) * kWordsPerThread;
  const bool in = w0 < m * (d / 8);
  ThreadWords tw{};
  if (in) tw = thread_words<FMT>(codes, scales, d, w0);
  for (int i = tid; i < kLdsCopies * (NB + 1); i += kThreads) lc[i] = 0;
  uint32_t want = 0;
  if constexpr (PASS == 1) {
    load_choice(hist, keep, false, ch);  // its barrier also ends the clearing
    want = ch[0];
  } else {
    __syncthreads();
  }
  uint32_t key[32];
  if (in) thread_keys<FMT>(tw, key);
  else
#pragma unroll
    for (int e = 0; e < 32; ++e) key[e] = 0;
#pragma unroll
  for (int e = 0; e < 32; ++e) {
    if constexpr (PASS == 0) hist_add_copies(lc, NB, key[e] >> 23, in);
    else hist_add_copies(lc, NB, (key[e] >> 17) & 63u, in && (key[e] >> 23) == want);
  }
  __syncthreads();
  for (int b = tid; b < NB; b += kThreads) {
    const uint32_t c = hist_sum_copies(lc, NB, b);  // local bins 0 .. NB-1 (both passes)
    if (c) atomicAdd(&hist[(blockIdx.x % kHistCopies) * kUHist + OFF + b], c);
    if constexpr (PASS == 1) {
      tie_counts[(size_t)blockIdx.x * kMantBins + b] = c;
      if (c && gridDim.x > kSuper)  // integer sums: any order
        atomicAdd(&super_counts[((blockIdx.x / kSuper) * kSuperCopies + blockIdx.x % kSuperCopies) * kMantBins + b], c);
    }
  }
}

// PMODE < 0: prune the codes in place (and write the keep mask).  PMODE >= 0: leave the codes
// and write S(Q(dX)) as fragment-major MFMA records (pack.hip layout, PackMode PMODE) to
// frag / fscale, including the zero records of rows past m (up to a multiple of 32) and of
// the missing half K step when d % 64 == 32.
template <int FMT, int PMODE>
__global__ __launch_bounds__(kThreads) void uapply_kernel(uint8_t* __restrict__ codes,
                                                          const void* __restrict__ scales, int64_t m,
                                                          int64_t d, uint32_t keep,
                                                          const uint32_t* __restrict__ hist,
                                                          const uint32_t* __restrict__ super_counts,
                                                          const uint32_t* __restrict__ tie_counts,
                                                          uint8_t* __restrict__ keep_mask,
                                                          uint8_t* __restrict__ frag,
                                                          uint8_t* __restrict__ fscale) {
  __shared__ uint32_t ch[4];
  __shared__ uint64_t wsum[kThreads / 64];
  __shared__ uint4 tab[PMODE == kPackHiA ? kHiSplitEntries : 1];
  if constexpr (PMODE == kPackHiA) hif4_load_split_tab(tab);  // published by load_choice's barrier
  const int64_t w0 = ((int64_t)blockIdx.x * kThreads + threadIdx.x) * kWordsPerThread;
  const bool in = w0 < m * (d / 8);
  ThreadWords tw{};
  if (in) tw = thread_words<FMT>(codes, scales, d, w0);
  load_choice(hist, keep, true, ch);
  const uint32_t T = ch[2], krem = ch[3];
  // ties of earlier workgroups: whole groups of kSuper workgroups, then this group's earlier
  // ones, from the second pass's counts of T's mantissa pattern
  const uint32_t tm = (T >> 17) & 63u, sb = blockIdx.x / kSuper;
  uint32_t before = 0;
  for (uint32_t w = threadIdx.x; w < sb * kSuperCopies; w += kThreads) before += super_counts[w * kMantBins + tm];
  for (uint32_t w = sb * kSuper + threadIdx.x; w < blockIdx.x; w += kThreads)
    before += tie_counts[(size_t)w * kMantBins + tm];
  uint32_t key[32];
  uint32_t ties = 0;
  if (in) {
    thread_keys<FMT>(tw, key);
#pragma unroll
    for (int e = 0; e < 32; ++e) ties += key[e] == T;
  }
  // one scan for both: this workgroup's ties in the low half (their exclusive prefix ranks
  // this thread's ties; at most 8192, no carry), the earlier workgroups' in the high half
  // (only their total is needed; at most m d <= 2^31)
  uint64_t total;
  const uint64_t pre = block_exclusive_scan<kThreads, uint64_t>(((uint64_t)before << 32) | ties, wsum, total);
  uint32_t rank = (uint32_t)(total >> 32) + (uint32_t)pre;
  if (!in) return;
  uint32_t kept = 0;  // 32 keep bits
#pragma unroll
  for (int e = 0; e < 32; ++e) {
    bool keep = key[e] > T;
    if (key[e] == T) keep = rank++ < krem;
    kept |= (uint32_t)keep << e;
  }
  uint4* cw = reinterpret_cast<uint4*>(codes + 4 * w0);
  uint4 v = tw.cw;
  v.x &= nibble_mask8(kept & 0xFFu);
  v.y &= nibble_mask8((kept >> 8) & 0xFFu);
  v.z &= nibble_mask8((kept >> 16) & 0xFFu);
  v.w &= nibble_mask8(kept >> 24);
  if constexpr (PMODE < 0) {
    *cw = v;
    if (keep_mask) *reinterpret_cast<uint32_t*>(keep_mask + w0) = kept;
  } else {
    // this thread's 32 elements are one lane record: row `row`, K elements j .. j+31
    const uint32_t e0 = (uint32_t)(8 * w0), row = e0 / (uint32_t)d, j = e0 - row * (uint32_t)d;
    const int64_t nkb = (d + 63) / 64, kb = j / 64;
    const int half = (int)((j / 32) & 1u);
    const uint32_t sc = tw.sc;  // the scale of this thread's block, loaded above
    const int64_t rec = ((int64_t)(row / 32) * nkb + kb) * 64 + (row & 31) + 32 * half;
    store_frag_record<PMODE>(frag, fscale, rec, v, sc, half, tab);
    const uint4 z = make_uint4(0, 0, 0, 0);
    if ((d & 63) == 32 && j + 32 == (uint32_t)d)  // the missing half K step: zero codes, scale 0
      store_frag_record<PMODE>(frag, fscale, rec + 32, z, 0u, 1, tab);
    if (row + 1 == (uint32_t)m)  // rows past m inside the last row tile: zero records
      for (uint32_t r = row + 1; r % 32 != 0; ++r) {
        const int64_t pr = ((int64_t)(r / 32) * nkb + kb) * 64 + (r & 31);
        store_frag_record<PMODE>(frag, fscale, pr + 32 * half, z, 0u, half, tab);
        if ((d & 63) == 32 && j + 32 == (uint32_t)d) store_frag_record<PMODE>(frag, fscale, pr + 32, z, 0u, 1, tab);
      }
  }
}

int64_t unstructured_wgs(int64_t m, int64_t d) {
  const int64_t per = (int64_t)kThreads * kWordsPerThread;
  return (m * (d / 8) + per - 1) / per;
}

// words cleared before an element-wise selection: the histogram copies and the group counts
int64_t hist_words(int64_t m, int64_t d) {
  return (int64_t)kHistCopies * kUHist + (unstructured_wgs(m, d) + kSuper - 1) / kSuper * kSuperCopies * kMantBins;
}

size_t a256(size_t x) { return (x + 255) & ~(size_t)255; }

int64_t n_blocks(int64_t m, int64_t d) { return ((m + 31) / 32) * (d / 64); }

}  // namespace

int64_t select_max_items() { return (int64_t)1 << 31; }

size_t select_ws_bytes(int sparsity, int fmt, int64_t m, int64_t d) {
  (void)fmt;
  switch (sparsity) {
    case 3:  // channel
      return a256((size_t)d * 8) + a256((size_t)(d + 31) / 32 * 4);
    case 4:  // block
      return a256((size_t)n_blocks(m, d) * 8) + a256((size_t)(n_blocks(m, d) + 31) / 32 * 4);
    case 5:  // element-wise
      return a256((size_t)hist_words(m, d) * 4) + a256((size_t)unstructured_wgs(m, d) * kMantBins * 4);
    default:
      return 0;
  }
}

void carve_select_ws(void* base, int sparsity, int fmt, int64_t m, int64_t d, SelectWs& ws) {
  (void)fmt;
  ws = SelectWs{};
  char* p = (char*)base;
  if (sparsity == 3 || sparsity == 4) {
    const int64_t n = sparsity == 3 ? d : n_blocks(m, d);
    ws.keys = (double*)p;
    ws.group_bits = (uint8_t*)(p + a256((size_t)n * 8));
  } else if (sparsity == 5) {
    ws.hist = (uint32_t*)p;
    ws.super_counts = ws.hist + kHistCopies * kUHist;
    ws.tie_counts = (uint32_t*)(p + a256((size_t)hist_words(m, d) * 4));
  }
}

void launch_select(int fmt, int sparsity, int64_t m, int64_t d, int64_t keep, uint8_t* qr_codes,
                   const void* qr_scales, const double* partials, uint8_t* keep_mask,
                   uint8_t* group_mask, const SelectWs& ws, hipStream_t s) {
  if (m == 0 || d == 0) return;
  const dim3 gw((unsigned)((d / 8 + kThreads - 1) / kThreads), (unsigned)(m < 65535 ? m : 65535));
  if (sparsity == 3) {
    launch_channel_top(fmt, qr_codes, qr_scales, m, d, keep, ws, group_mask, s);
    hipLaunchKernelGGL((apply_groups_kernel<0>), gw, dim3(kThreads), 0, s,
                       (uint32_t*)qr_codes, m, d, (const uint8_t*)ws.group_bits, keep_mask);
  } else if (sparsity == 4) {
    launch_block_top(fmt, partials, m, d, keep, ws, group_mask, s);
    hipLaunchKernelGGL((apply_groups_kernel<1>), gw, dim3(kThreads), 0, s,
                       (uint32_t*)qr_codes, m, d, (const uint8_t*)ws.group_bits, keep_mask);
  } else if (sparsity == 5) {
    const unsigned nwg = (unsigned)unstructured_wgs(m, d);
    hipLaunchKernelGGL(uzero_kernel, dim3(1), dim3(kThreads), 0, s, ws.hist, (int)hist_words(m, d));
    const uint32_t k = (uint32_t)keep;
#define RESQ_U(F)                                                                                          \
    hipLaunchKernelGGL((uhist_kernel<F, 0>), dim3(nwg), dim3(kThreads), 0, s, qr_codes, qr_scales, m, d, k, ws.hist,  \
                       ws.super_counts, ws.tie_counts);                                                               \
    hipLaunchKernelGGL((uhist_kernel<F, 1>), dim3(nwg), dim3(kThreads), 0, s, qr_codes, qr_scales, m, d, k, ws.hist,  \
                       ws.super_counts, ws.tie_counts);                                                               \
    hipLaunchKernelGGL((uapply_kernel<F, -1>), dim3(nwg), dim3(kThreads), 0, s, qr_codes, qr_scales, m, d, k,         \
                       (const uint32_t*)ws.hist, (const uint32_t*)ws.super_counts, (const uint32_t*)ws.tie_counts,    \
                       keep_mask, nullptr, nullptr);
    if (fmt == 0) { RESQ_U(0) } else { RESQ_U(1) }
#undef RESQ_U
  }
}

void launch_select_frag(int fmt, int sparsity, int64_t m, int64_t d, int64_t keep, uint8_t* qr_codes,
                        const void* qr_scales, const double* partials, const SelectWs& ws,
                        int pack_mode, uint8_t* frag, uint8_t* fscale, hipStream_t s) {
  if (m == 0 || d == 0) return;
  if (sparsity == 3 || sparsity == 4) {
    const bool chan = sparsity == 3;
    const int64_t n = chan ? d : n_blocks(m, d);
    if (chan) {
      launch_channel_top(fmt, qr_codes, qr_scales, m, d, keep, ws, nullptr, s);
    } else {
      if (partials) launch_block_top(fmt, partials, m, d, keep, ws, nullptr, s);
      else launch_top(ws.keys, n, keep, ws.group_bits, nullptr, s);  // keys from the residual pass
    }
    launch_pack(pack_mode, qr_codes, qr_scales, m, d, frag, fscale, s, chan ? 1 : 2, ws.group_bits);
  } else if (sparsity == 5) {
    // the histograms were cleared before the residual pass, which counted the exponent bins
    const unsigned nwg = (unsigned)unstructured_wgs(m, d);
    const uint32_t k = (uint32_t)keep;
#define RESQ_UF(F, P)                                                                                      \
    hipLaunchKernelGGL((uhist_kernel<F, 1>), dim3(nwg), dim3(kThreads), 0, s, qr_codes, qr_scales, m, d, k, ws.hist,  \
                       ws.super_counts, ws.tie_counts);                                                               \
    hipLaunchKernelGGL((uapply_kernel<F, P>), dim3(nwg), dim3(kThreads), 0, s, qr_codes, qr_scales, m, d, k,          \
                       (const uint32_t*)ws.hist, (const uint32_t*)ws.super_counts, (const uint32_t*)ws.tie_counts,    \
                       (uint8_t*)nullptr, frag, fscale);
    if (fmt == 0) { RESQ_UF(0, kPackMx) } else { RESQ_UF(1, kPackHiA) }
#undef RESQ_UF
  }
}

int select_hist_words(int64_t m, int64_t d) { return (int)hist_words(m, d); }

void launch_select_clear(const SelectWs& ws, int64_t m, int64_t d, hipStream_t s) {
  if (m == 0 || d == 0) return;
  hipLaunchKernelGGL(uzero_kernel, dim3(1), dim3(kThreads), 0, s, ws.hist, (int)hist_words(m, d));
}

}  // namespace resq
