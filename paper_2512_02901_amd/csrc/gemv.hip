// Decode product for 1..16 tokens on the vector units (Sec. 3.4, Algorithm 1,
// with the dequantisation of Eq. ifairy-dequant and the W conj(x) term):
// float32 activations, and bf16 or int8 where K % 64 != 0 keeps them off the
// matrix cores.
//
// Float activations (gemv_table_kernel).  In the layer's real form each
// (n, k) is a real 2 x 2 block acting on (Re x, Im x), and its 2T codes allow
// few different blocks: 4^(2T).  A thread block forms the blocks of every
// pair of stages once in LDS (256 of 16 bytes, summed over the stages in
// double and rounded once to float32); a code then costs one table index and
// one 16-byte LDS read a (n, k), and four multiply-adds a token, for any T.
// Block: kRows rows and TB tokens, its four waves split K; a lane takes four
// consecutive codes (one byte of every plane) of each row and their
// activations from memory in one round of loads, so that short rows still
// fill the lanes.  Sums run in float32 in a fixed order, lanes and waves as a
// tree.  (One wave per row, 16 codes a lane with a select and two adds per
// code, plane and token, and LDS reads of x for each, left 256 CUs with 250
// blocks of serial work: 1001 x 1500, T = 3, 5 tokens took 45.4 us, now 7.5;
// 128 x 128, T = 2, one token 9.5, now 4.0; 5504 x 5504, 16 tokens 829, now
// 97.  Two or eight rows a block instead of four: 10.9 and 9.9 against 8.7 us
// for 1001 x 1500, T = 2, 16 tokens, 147 and 107 for 5504 x 5504.)
// bf16 activations: entries and sums in double.  Signed adds of 8-bit
// significands round little (4e-8 to 9e-8 of the result for K 260 .. 16388 and
// T 1 .. 4, where float32 entries and sums are 8e-8 to 2e-7 off); in double it
// is 2.5e-8, the output's own rounding.  The tables are U's and W's 16 sums
// apart, 256 bytes each that random indexes read without bank conflicts, added
// per code: 5504 x 2052, T = 2, one token 11.7 us (256 blocks of 32 bytes 15.9),
// 16 tokens 66; in float32 8.9 and 42, by signed adds 22 and 439.
// A table entry of 0 times an infinite activation would be NaN where a code's
// sign flips and adds give a finite sum, so a block that meets one recomputes
// its outputs by those.
//
// Int8 activations (gemv_valu_kernel) keep the multiplication-free form, with
// exact int32 sums: for each matrix M in {U, W}, stage t and axis a in {re,
// im} one complex accumulator
//     A[M][t][a] = sum over codes k with (k & 1) == a of  (-1)^(k >> 1) x_j
// i.e. each 2-bit code costs one signed complex add of x_j into the
// accumulator its axis bit selects.  Both U and W accumulate x itself; the
// multiplication by i, the conjugation of the W term and the axis scales are
// applied once per output in the epilogue:
//     y = sum_t  s^U_re A[U][t][re] + i s^U_im A[U][t][im]
//              + s^W_re conj(A[W][t][re]) + i s^W_im conj(A[W][t][im]).
// One wave per output row, four rows per block; lane l owns the 32-bit code
// word (16 codes) l of every 1024-code chunk of the row, for each of the 2T
// code planes; the chunk of activations is staged in LDS (padded to spread
// banks).
#include "common.h"

namespace fairy2i {

namespace {

constexpr int kChunk = 1024;               // codes per LDS chunk
constexpr int kPad = kChunk + kChunk / 16;  // one float2 of padding every 16

__device__ inline int lds_index(int n) { return n + (n >> 4); }

template <int DT>
struct ActTraits;
template <>
struct ActTraits<FAIRY2I_ACT_F32> {
  using acc_t = float;
  __device__ static inline void load(const void* x, int64_t i, acc_t& re, acc_t& im) {
    const float2 v = static_cast<const float2*>(x)[i];
    re = v.x;
    im = v.y;
  }
};
template <>
struct ActTraits<FAIRY2I_ACT_BF16> {
  using acc_t = float;
  __device__ static inline void load(const void* x, int64_t i, acc_t& re, acc_t& im) {
    const uint32_t v = static_cast<const uint32_t*>(x)[i];
    re = __uint_as_float(v << 16);
    im = __uint_as_float(v & 0xFFFF0000u);
  }
};
template <>
struct ActTraits<FAIRY2I_ACT_I8> {
  using acc_t = int;
  __device__ static inline void load(const void* x, int64_t i, acc_t& re, acc_t& im) {
    const uint16_t v = static_cast<const uint16_t*>(x)[i];
    re = (int)(int8_t)(v & 0xFF);
    im = (int)(int8_t)(v >> 8);
  }
};

// 16 codes starting at code j0 of a row that has K codes, packed 4 per byte.
// Codes at or beyond K read as 0 (their activations are zero).
__device__ inline uint32_t load_code_word(const uint8_t* row, int64_t K, int64_t j0, bool aligned) {
  if (aligned) return *reinterpret_cast<const uint32_t*>(row + j0 / 4);
  uint32_t w = 0;
  for (int b = 0; b < 4; ++b)
    if (j0 + 4 * b < K) w |= (uint32_t)row[j0 / 4 + b] << (8 * b);
  return w;
}

template <typename A>
__device__ inline A wave_sum(A v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  return v;
}

template <int T, int TB, bool EXPORT>
__global__ __launch_bounds__(256) void gemv_valu_kernel(WlArgs a, bool aligned) {
  using Tr = ActTraits<FAIRY2I_ACT_I8>;
  using acc_t = typename Tr::acc_t;
  __shared__ acc_t xs[TB][kPad][2];

  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int64_t row = (int64_t)blockIdx.x * 4 + wave;
  const bool row_ok = row < a.N;
  const int64_t b0 = (int64_t)blockIdx.y * TB;
  const int64_t K = a.K;
  const int64_t plane = a.N * K / 4;  // bytes per stage plane

  acc_t acc[2][T][2][TB][2];
#pragma unroll
  for (int m = 0; m < 2; ++m)
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int ax = 0; ax < 2; ++ax)
#pragma unroll
        for (int tb = 0; tb < TB; ++tb) acc[m][t][ax][tb][0] = acc[m][t][ax][tb][1] = 0;

  for (int64_t c0 = 0; c0 < K; c0 += kChunk) {
    __syncthreads();
    for (int n = threadIdx.x; n < TB * kChunk; n += blockDim.x) {
      const int tb = n / kChunk, jj = n - tb * kChunk;
      const int64_t b = b0 + tb, j = c0 + jj;
      acc_t re = 0, im = 0;
      if (b < a.B && j < K) Tr::load(a.x, b * K + j, re, im);
      xs[tb][lds_index(jj)][0] = re;
      xs[tb][lds_index(jj)][1] = im;
    }
    __syncthreads();
    const int64_t j0 = c0 + 16 * lane;
    if (row_ok && j0 < K) {
#pragma unroll
      for (int m = 0; m < 2; ++m) {
#pragma unroll
        for (int t = 0; t < T; ++t) {
          const uint8_t* rowp = a.codes[m] + t * plane + row * (K / 4);
          const uint32_t w = load_code_word(rowp, K, j0, aligned);
#pragma unroll
          for (int cc = 0; cc < 16; ++cc) {
            const uint32_t k = (w >> (2 * cc)) & 3u;
            const int li = lds_index(16 * lane + cc);
#pragma unroll
            for (int tb = 0; tb < TB; ++tb) {
              acc_t re = xs[tb][li][0], im = xs[tb][li][1];
              if (k & 2u) {
                re = -re;
                im = -im;
              }
              if (k & 1u) {
                acc[m][t][1][tb][0] += re;
                acc[m][t][1][tb][1] += im;
              } else {
                acc[m][t][0][tb][0] += re;
                acc[m][t][0][tb][1] += im;
              }
            }
          }
        }
      }
    }
  }

#pragma unroll
  for (int m = 0; m < 2; ++m)
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int ax = 0; ax < 2; ++ax)
#pragma unroll
        for (int tb = 0; tb < TB; ++tb) {
          acc[m][t][ax][tb][0] = wave_sum(acc[m][t][ax][tb][0]);
          acc[m][t][ax][tb][1] = wave_sum(acc[m][t][ax][tb][1]);
        }
  if (!row_ok || lane != 0) return;

#pragma unroll
  for (int tb = 0; tb < TB; ++tb) {
    const int64_t b = b0 + tb;
    if (b >= a.B) break;
    if constexpr (EXPORT) {
      // acc[M][t][p][b][i][c]
#pragma unroll
      for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
          for (int ax = 0; ax < 2; ++ax) {
            int32_t* dst = a.acc + ((((int64_t)(m * T + t) * 2 + ax) * a.B + b) * a.N + row) * 2;
            dst[0] = (int32_t)acc[m][t][ax][tb][0];
            dst[1] = (int32_t)acc[m][t][ax][tb][1];
          }
    } else {
      float yr = 0.0f, yi = 0.0f;
#pragma unroll
      for (int t = 0; t < T; ++t) {
        const float su_re = a.scales[0][2 * t], su_im = a.scales[0][2 * t + 1];
        const float sw_re = a.scales[1][2 * t], sw_im = a.scales[1][2 * t + 1];
        const float ur0 = (float)acc[0][t][0][tb][0], ui0 = (float)acc[0][t][0][tb][1];
        const float ur1 = (float)acc[0][t][1][tb][0], ui1 = (float)acc[0][t][1][tb][1];
        const float wr0 = (float)acc[1][t][0][tb][0], wi0 = (float)acc[1][t][0][tb][1];
        const float wr1 = (float)acc[1][t][1][tb][0], wi1 = (float)acc[1][t][1][tb][1];
        yr += su_re * ur0 - su_im * ui1;
        yi += su_re * ui0 + su_im * ur1;
        yr += sw_re * wr0 + sw_im * wi1;
        yi += -sw_re * wi0 + sw_im * wr1;
      }
      const float f = a.x_scale[b];
      a.y[b * a.N + row] = make_float2(yr * f, yi * f);
    }
  }
}

// ------------------------------------------------------ table kernel ---
constexpr int kRows = 4;
constexpr int kTableThreads = 256;

// Four consecutive complex activations from element e0 on.
template <int DT>
__device__ inline void load_four(const void* x, int64_t e0, bool vec, float (&re)[4], float (&im)[4]) {
  if (!vec) {
#pragma unroll
    for (int e = 0; e < 4; ++e) ActTraits<DT>::load(x, e0 + e, re[e], im[e]);
  } else if constexpr (DT == FAIRY2I_ACT_F32) {
    const float4* p = reinterpret_cast<const float4*>(static_cast<const float2*>(x) + e0);
    const float4 a = p[0], b = p[1];
    re[0] = a.x; im[0] = a.y; re[1] = a.z; im[1] = a.w;
    re[2] = b.x; im[2] = b.y; re[3] = b.z; im[3] = b.w;
  } else {
    const uint4 w = *reinterpret_cast<const uint4*>(static_cast<const uint32_t*>(x) + e0);
    const uint32_t c[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      re[e] = __uint_as_float(c[e] << 16);
      im[e] = __uint_as_float(c[e] & 0xFFFF0000u);
    }
  }
}

// Sum of each of NV (a power of two up to 64) values over the wave, each step
// halving the values a lane carries: lane l ends with the sum of value
// l / (64 / NV).
// (Recursion, so that every index is a constant: a loop over the halvings
// became chains of selects, 9 us of a 128 x 128 call.)
template <int NV, int OFF = 32, typename A>
__device__ inline A wave_sums(const A (&v)[NV], int lane) {
  if constexpr (NV > 1) {
    const bool up = (lane & OFF) != 0;
    A h[NV / 2];
#pragma unroll
    for (int i = 0; i < NV / 2; ++i) {
      const A keep = up ? v[i + NV / 2] : v[i], send = up ? v[i] : v[i + NV / 2];
      h[i] = keep + __shfl_xor(send, OFF);
    }
    return wave_sums<NV / 2, OFF / 2>(h, lane);
  } else if constexpr (OFF > 0) {
    const A h[1] = {v[0] + __shfl_xor(v[0], OFF)};
    return wave_sums<1, OFF / 2>(h, lane);
  } else {
    return v[0];
  }
}

// What table entries and sums are held in.
template <int DT>
struct TableTraits {
  using acc_t = float;
};
template <>
struct TableTraits<FAIRY2I_ACT_BF16> {
  using acc_t = double;
};
// One output by signed adds (a token with infinite or undefined values): the
// lanes of a wave take every 64th column.
template <int DT, int T>
__device__ inline float2 signed_adds(const WlArgs& a, int64_t row, int64_t b, int lane) {
  float acc[2][T][2][2];
#pragma unroll
  for (int m = 0; m < 2; ++m)
#pragma unroll
    for (int t = 0; t < T; ++t) acc[m][t][0][0] = acc[m][t][0][1] = acc[m][t][1][0] = acc[m][t][1][1] = 0.0f;
  for (int64_t j = lane; j < a.K; j += 64) {
    float re, im;
    ActTraits<DT>::load(a.x, b * a.K + j, re, im);
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int t = 0; t < T; ++t) {
        const uint32_t k = (a.codes[m][((int64_t)t * a.N + row) * (a.K / 4) + j / 4] >> (2 * (j & 3))) & 3u;
        const float sr = k & 2u ? -re : re, si = k & 2u ? -im : im;
        if (k & 1u) {
          acc[m][t][1][0] += sr;
          acc[m][t][1][1] += si;
        } else {
          acc[m][t][0][0] += sr;
          acc[m][t][0][1] += si;
        }
      }
  }
  float yr = 0.0f, yi = 0.0f;
#pragma unroll
  for (int t = 0; t < T; ++t) {
    const float su_re = a.scales[0][2 * t], su_im = a.scales[0][2 * t + 1];
    const float sw_re = a.scales[1][2 * t], sw_im = a.scales[1][2 * t + 1];
    yr += su_re * wave_sum(acc[0][t][0][0]) - su_im * wave_sum(acc[0][t][1][1]);
    yi += su_re * wave_sum(acc[0][t][0][1]) + su_im * wave_sum(acc[0][t][1][0]);
    yr += sw_re * wave_sum(acc[1][t][0][0]) + sw_im * wave_sum(acc[1][t][1][1]);
    yi += -sw_re * wave_sum(acc[1][t][0][1]) + sw_im * wave_sum(acc[1][t][1][0]);
  }
  return make_float2(yr, yi);
}

template <int DT, int T, int TB>
__global__ __launch_bounds__(kTableThreads) void gemv_table_kernel(WlArgs a, bool vec) {
  using A = typename TableTraits<DT>::acc_t;
  constexpr int kTables = (T + 1) / 2;  // one per pair of stages
  constexpr int kWaves = kTableThreads / 64;
  constexpr int NV = kRows * (TB <= 1 ? 1 : TB <= 2 ? 2 : 4) * 2;  // sums of a lane, padded to a power of two
  // float: (R11, R12, R21, R22) by U's code of the pair's first stage (bits 0, 1)
  // and second (2, 3), W's (4, 5) and (6, 7); double: (Re, Im) of U's 16 sums and
  // of W's, whose 256 bytes a random index reads without bank conflicts
  constexpr bool kWide = sizeof(A) == 8;
  __shared__ float4 table[kWide ? 1 : kTables][kWide ? 1 : 256];
  __shared__ double2 half[kWide ? kTables : 1][2][kWide ? 16 : 1];
  __shared__ A part[kWaves][NV];
  __shared__ int odd_values;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t row0 = (int64_t)blockIdx.x * kRows, b0 = (int64_t)blockIdx.y * TB;
  if (threadIdx.x == 0) odd_values = 0;
#pragma unroll
  for (int p = 0; p < kTables; ++p) {
    double u[2] = {0.0, 0.0}, w[2] = {0.0, 0.0};
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int t = 2 * p + h;
      if (t < T) {
        const uint32_t ku = (threadIdx.x >> (2 * h)) & 3u, kw = (threadIdx.x >> (4 + 2 * h)) & 3u;
        const double su = a.scales[0][2 * t + (ku & 1u)], sw = a.scales[1][2 * t + (kw & 1u)];
        const double du = ku & 2u ? -su : su, dw = kw & 2u ? -sw : sw;
        u[0] += ku & 1u ? 0.0 : du;
        u[1] += ku & 1u ? du : 0.0;
        w[0] += kw & 1u ? 0.0 : dw;
        w[1] += kw & 1u ? dw : 0.0;
      }
    }
    if constexpr (kWide) {
      if (threadIdx.x < 16) half[p][0][threadIdx.x] = make_double2(u[0], u[1]);
      if (threadIdx.x % 16 == 0) half[p][1][threadIdx.x / 16] = make_double2(w[0], w[1]);
    } else {
      table[p][threadIdx.x] =
          make_float4((float)(u[0] + w[0]), (float)(w[1] - u[1]), (float)(u[1] + w[1]), (float)(u[0] - w[0]));
    }
  }
  __syncthreads();

  A acc[kRows][TB][2];
#pragma unroll
  for (int r = 0; r < kRows; ++r)
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) acc[r][tb][0] = acc[r][tb][1] = 0;
  float check = 0.0f;  // 0 times every activation: NaN if one is not finite
  const int64_t kb = a.K / 4, plane = a.N * kb;
  for (int64_t s = threadIdx.x; s < kb; s += kTableThreads) {
    uint32_t c[kRows][2 * T];
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
      const int64_t row = row0 + r < a.N ? row0 + r : a.N - 1;  // rows past the last repeat it, unstored
#pragma unroll
      for (int p = 0; p < 2 * T; ++p) c[r][p] = a.codes[p / T][(p % T) * plane + row * kb + s];
    }
    float re[TB][4], im[TB][4];
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) {
      const int64_t b = b0 + tb < a.B ? b0 + tb : a.B - 1;
      load_four<DT>(a.x, b * a.K + 4 * s, vec, re[tb], im[tb]);
#pragma unroll
      for (int e = 0; e < 4; ++e) check = fmaf(im[tb][e], 0.0f, fmaf(re[tb][e], 0.0f, check));
    }
    // (doubles a column at a time: all columns' conversions and blocks together
    // take up to 290 registers)
#pragma unroll
    for (int k = 0; k < 4 * kRows; ++k) {
      const int r = kWide ? k % kRows : k / 4, e = kWide ? k / kRows : k % 4;
      if (kWide && r == 0) __builtin_amdgcn_sched_barrier(0);
      A v[4];
#pragma unroll
      for (int p = 0; p < kTables; ++p) {
        const int p2 = 2 * p + 1 < T ? 2 * p + 1 : T - 1;  // the pair's second stage, where there is one
        A q[4];
        if constexpr (kWide) {
          uint32_t iu = (c[r][2 * p] >> (2 * e)) & 3u, iw = (c[r][T + 2 * p] >> (2 * e)) & 3u;
          if (2 * p + 1 < T) {
            iu |= ((c[r][p2] >> (2 * e)) & 3u) << 2;
            iw |= ((c[r][T + p2] >> (2 * e)) & 3u) << 2;
          }
          const double2 u = half[p][0][iu], w = half[p][1][iw];
          q[0] = u.x; q[1] = u.y; q[2] = w.x; q[3] = w.y;
        } else {
          uint32_t i = ((c[r][2 * p] >> (2 * e)) & 3u) | (((c[r][T + 2 * p] >> (2 * e)) & 3u) << 4);
          if (2 * p + 1 < T) i |= (((c[r][p2] >> (2 * e)) & 3u) << 2) | (((c[r][T + p2] >> (2 * e)) & 3u) << 6);
          const float4 t = table[p][i];
          q[0] = t.x; q[1] = t.y; q[2] = t.z; q[3] = t.w;
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = p == 0 ? q[j] : v[j] + q[j];
      }
      if constexpr (kWide) {
        const A u0 = v[0], u1 = v[1];
        v[0] = u0 + v[2]; v[1] = v[3] - u1;
        const A w0 = v[2];
        v[2] = u1 + v[3]; v[3] = u0 - w0;
      }
#pragma unroll
      for (int tb = 0; tb < TB; ++tb)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[r][tb][j] = fma(v[2 * j + 1], (A)im[tb][e], fma(v[2 * j], (A)re[tb][e], acc[r][tb][j]));
    }
  }
  if (check != check) odd_values = 1;

  A v[NV];
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int r = i / (NV / kRows), tb = (i / 2) % (NV / kRows / 2);
    v[i] = tb < TB ? acc[r][tb < TB ? tb : 0][i & 1] : (A)0;
  }
  const A sum = wave_sums<NV>(v, lane);
  if (lane % (64 / NV) == 0) part[wave][lane / (64 / NV)] = sum;
  __syncthreads();
  if (odd_values) {
    static_assert(kRows == kWaves, "one row a wave");
    const int64_t row = row0 + wave;
    if (row >= a.N) return;
    for (int tb = 0; tb < TB && b0 + tb < a.B; ++tb) {
      const float2 y = signed_adds<DT, T>(a, row, b0 + tb, lane);
      if (lane == 0) a.y[(b0 + tb) * a.N + row] = y;
    }
    return;
  }
  if (threadIdx.x < NV / 2) {
    const int r = threadIdx.x / (NV / kRows / 2), tb = threadIdx.x % (NV / kRows / 2);
    if (tb < TB && b0 + tb < a.B && row0 + r < a.N) {
      A yr = 0, yi = 0;
#pragma unroll
      for (int w = 0; w < kWaves; ++w) {
        yr += part[w][2 * threadIdx.x];
        yi += part[w][2 * threadIdx.x + 1];
      }
      a.y[(b0 + tb) * a.N + row0 + r] = make_float2((float)yr, (float)yi);
    }
  }
}

template <int DT, int T, int TB>
hipError_t launch_table_tb(const WlArgs& a, hipStream_t s) {
  // K % 4 == 0: every four activations start 16-byte aligned if the first do
  const bool vec = (reinterpret_cast<uintptr_t>(a.x) & 15) == 0;
  dim3 grid((unsigned)((a.N + kRows - 1) / kRows), (unsigned)((a.B + TB - 1) / TB));
  hipLaunchKernelGGL((gemv_table_kernel<DT, T, TB>), grid, dim3(kTableThreads), 0, s, a, vec);
  return hipGetLastError();
}

template <int DT, int T>
hipError_t launch_table_t(const WlArgs& a, hipStream_t s) {
  // up to four tokens a block, the blocks of a row group alike: 5 tokens are 3 + 2, not 4 + 1
  const int64_t groups = (a.B + 3) / 4;
  switch ((a.B + groups - 1) / groups) {
    case 1: return launch_table_tb<DT, T, 1>(a, s);
    case 2: return launch_table_tb<DT, T, 2>(a, s);
    case 3: return launch_table_tb<DT, T, 3>(a, s);
    default: return launch_table_tb<DT, T, 4>(a, s);
  }
}

template <int DT>
hipError_t launch_table(const WlArgs& a, hipStream_t s) {
  switch (a.T) {
    case 1: return launch_table_t<DT, 1>(a, s);
    case 2: return launch_table_t<DT, 2>(a, s);
    case 3: return launch_table_t<DT, 3>(a, s);
    default: return launch_table_t<DT, 4>(a, s);
  }
}

// ------------------------------------------------------- int8 launches ---
template <int T, int TB, bool EXPORT>
hipError_t launch_tb(const WlArgs& a, hipStream_t s) {
  const bool aligned = (a.K % 16) == 0;
  dim3 grid((unsigned)((a.N + 3) / 4), (unsigned)((a.B + TB - 1) / TB));
  hipLaunchKernelGGL((gemv_valu_kernel<T, TB, EXPORT>), grid, dim3(256), 0, s, a, aligned);
  return hipGetLastError();
}

template <int T, bool EXPORT>
hipError_t launch_t(const WlArgs& a, hipStream_t s) {
  if (a.B == 1) return launch_tb<T, 1, EXPORT>(a, s);
  if (a.B == 2) return launch_tb<T, 2, EXPORT>(a, s);
  return launch_tb<T, 4, EXPORT>(a, s);
}

template <bool EXPORT>
hipError_t launch_int8(const WlArgs& a, hipStream_t s) {
  switch (a.T) {
    case 1: return launch_t<1, EXPORT>(a, s);
    case 2: return launch_t<2, EXPORT>(a, s);
    case 3: return launch_t<3, EXPORT>(a, s);
    default: return launch_t<4, EXPORT>(a, s);
  }
}

}  // namespace

hipError_t launch_gemv(const WlArgs& a, hipStream_t s) {
  if (a.acc) return launch_int8<true>(a, s);
  switch (a.dtype) {
    case FAIRY2I_ACT_F32: return launch_table<FAIRY2I_ACT_F32>(a, s);
    case FAIRY2I_ACT_BF16: return launch_table<FAIRY2I_ACT_BF16>(a, s);
    default: return launch_int8<false>(a, s);
  }
}

}  // namespace fairy2i
