// Real form of a widely-linear layer for training (Sec. 3.1, Eq. UW-from-R
// read backwards, with Eq. realify-ops): y = U x + W conj(x) is one real
// linear map of the stacked (Re, Im) pairs, whose 2 x 2 block for output n
// and input k is
//     [ Re U + Re W    Im W - Im U ]
//     [ Im U + Im W    Re U - Re W ]
// (R11 = Re U + Re W, R12 = Im W - Im U, R21 = Im U + Im W, R22 = Re U - Re W
// of the half-split real matrix).  With R stored interleaved (row 2n + a,
// column 2k + b for the (a, b) entry of that block) and tokens stored as
// (re, im) pairs, the three products of a training step are plain real
// GEMMs of the same data in place:
//     Y   = X R^T        (M x 2N  =  M x 2K  .  2K x 2N)
//     G_X = G_Y R        (the gradient through the real map)
//     G_R = G_Y^T X      (2N x 2K)
// and G_U = G_Y^T conj(X), G_W = G_Y^T X are read off G_R's blocks:
//     Re G_U = G_R[2n][2k] + G_R[2n+1][2k+1],  Im G_U = G_R[2n+1][2k] - G_R[2n][2k+1],
//     Re G_W = G_R[2n][2k] - G_R[2n+1][2k+1],  Im G_W = G_R[2n][2k+1] + G_R[2n+1][2k].
// Against Gauss's three complex products per segment (six real products of
// M x N x K for the two segments) this is four real products' work, and the
// operands need no planes.
#include "common.h"

namespace fairy2i {

namespace {

__device__ inline uint16_t bf16_rne_bits(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

// A double rounded once to bf16 (nearest even).  Rounding to float32 first
// and then to bf16 goes wrong only where the float32 value is a bf16 tie
// that the double is not on (every bf16 tie is a float32 value, so
// elsewhere the float32 value lies on the same side of every tie as the
// double); there the sign of the float32 rounding's remainder decides.
// (Selects, no branches: at a float32 tie f is not zero, so a nonzero
// remainder rounds away from zero exactly when it has f's sign.)
__device__ inline uint16_t bf16_from_double(double v) {
  const float f = (float)v;  // nearest float32
  const double r = v - (double)f;
  const uint32_t u = __float_as_uint(f);
  const uint32_t low = u & 0xFFFFu;
  const uint32_t hi = u >> 16;
  const uint32_t away = r != 0.0 ? (uint32_t)((r > 0.0) == (f > 0.0f)) : (hi & 1u);
  return (uint16_t)(hi + ((uint32_t)(low > 0x8000u) | ((uint32_t)(low == 0x8000u) & away)));
}

__device__ inline float2 load_c(const void* p, int32_t dtype, int64_t i) {
  if (dtype == FAIRY2I_ACT_BF16) {
    const uint32_t w = static_cast<const uint32_t*>(p)[i];
    return make_float2(__uint_as_float(w << 16), __uint_as_float(w & 0xFFFF0000u));
  }
  return static_cast<const float2*>(p)[i];
}

// One thread per (n, k): the block's four entries as two 32-bit words, one
// in row 2n and one in row 2n + 1.
__global__ __launch_bounds__(256) void realify_kernel(const void* __restrict__ U, const void* __restrict__ W,
                                                      int32_t dtype, int64_t N, int64_t K,
                                                      uint32_t* __restrict__ R) {
  const int64_t total = N * K;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
    // N K <= 2^30 (checked by the host): 32-bit division
    const int64_t n = (int64_t)((uint32_t)i / (uint32_t)K), k = i - n * K;
    const float2 u = load_c(U, dtype, i), w = load_c(W, dtype, i);
    const double ur = u.x, ui = u.y, wr = w.x, wi = w.y;
    const uint32_t top = (uint32_t)bf16_from_double(ur + wr) | ((uint32_t)bf16_from_double(wi - ui) << 16);
    const uint32_t bot = (uint32_t)bf16_from_double(ui + wi) | ((uint32_t)bf16_from_double(ur - wr) << 16);
    R[(2 * n) * K + k] = top;      // row 2n: columns 2k, 2k + 1 (K words per row)
    R[(2 * n + 1) * K + k] = bot;  // row 2n + 1
  }
}

// One thread per (n, k): G_U and G_W from the block of G_R (float32 sums).
__global__ __launch_bounds__(256) void unrealify_grad_kernel(const float2* __restrict__ GR, int64_t N, int64_t K,
                                                             float2* __restrict__ GU, float2* __restrict__ GW) {
  const int64_t total = N * K;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t n = (int64_t)((uint32_t)i / (uint32_t)K), k = i - n * K;  // N K <= 2^30
    const float2 t = GR[(2 * n) * K + k];      // (G_R[2n][2k], G_R[2n][2k+1])
    const float2 b = GR[(2 * n + 1) * K + k];  // (G_R[2n+1][2k], G_R[2n+1][2k+1])
    GU[i] = make_float2(t.x + b.y, b.x - t.y);
    GW[i] = make_float2(t.x - b.y, t.y + b.x);
  }
}

// The block entries of one (n, k) from the codes of its stages (Eq.
// ifairy-dequant, Eq. res-sum): U^ and W^ are summed over the stages in
// increasing order in double (as the fake-quant dequantisation does), the
// entries formed in double and rounded once to bf16.  A stage adds s c with
// c in {1, 0, -1} as one fused multiply-add: the same rounding as adding or
// subtracting s, or nothing (a sum never holds -0, and the scales are not
// negative), without a branch on the code.
struct RealSum {
  double ur, ui, wr, wi;
};

__device__ inline void real_add(RealSum& a, int ku, int kw, double sur, double sui, double swr, double swi) {
  // i^k: 0 -> +1, 1 -> +i, 2 -> -1, 3 -> -i: real part 1 - k for even k, imaginary part 2 - k for odd k
  const int cur = (1 - ku) & ((ku & 1) - 1), cui = (2 - ku) & -(ku & 1);
  const int cwr = (1 - kw) & ((kw & 1) - 1), cwi = (2 - kw) & -(kw & 1);
  a.ur = fma(sur, (double)cur, a.ur);
  a.ui = fma(sui, (double)cui, a.ui);
  a.wr = fma(swr, (double)cwr, a.wr);
  a.wi = fma(swi, (double)cwi, a.wi);
}

// {row 2n, row 2n + 1} of the block, two bf16 entries each
__device__ inline uint2 real_block(const RealSum& a) {
  return make_uint2((uint32_t)bf16_from_double(a.ur + a.wr) | ((uint32_t)bf16_from_double(a.wi - a.ui) << 16),
                    (uint32_t)bf16_from_double(a.ui + a.wi) | ((uint32_t)bf16_from_double(a.ur - a.wr) << 16));
}

// R straight from the codes for T <= 2: a (n, k) has 2T codes, so at most 256
// different blocks exist.  Each thread block forms them all once in LDS (one
// a thread, by the sums above) and then only looks them up: a code byte of
// every plane in, two 16-byte stores out per four entries.  (Summing in
// double for every entry was bound by that arithmetic: 2048 x 2048, T = 2,
// 18.3 us, with the table 8.6 us for its 38 MB.)
template <int T>
__global__ __launch_bounds__(256) void realify_table_kernel(const uint8_t* __restrict__ cu,
                                                            const float* __restrict__ su,
                                                            const uint8_t* __restrict__ cw,
                                                            const float* __restrict__ sw, int64_t N, int64_t K,
                                                            uint4* __restrict__ R) {
  static_assert(T == 1 || T == 2, "2T codes index at most 256 blocks");
  __shared__ uint2 table[256];  // index: code of U's stage t at bits 2t, of W's at bits 4 + 2t
  {
    const int i = threadIdx.x;
    RealSum a{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int t = 0; t < T; ++t)
      real_add(a, (i >> (2 * t)) & 3, (i >> (4 + 2 * t)) & 3, (double)su[2 * t], (double)su[2 * t + 1],
               (double)sw[2 * t], (double)sw[2 * t + 1]);
    table[i] = real_block(a);
  }
  __syncthreads();
  const int64_t nbytes = N * K / 4, kb = K / 4, stride = (int64_t)gridDim.x * blockDim.x;
  constexpr int U = 4;  // bytes a thread loads before it looks them up
  for (int64_t b0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; b0 < nbytes; b0 += U * stride) {
    uint32_t u[U][T], w[U][T];
#pragma unroll
    for (int i = 0; i < U; ++i)
#pragma unroll
      for (int t = 0; t < T; ++t) {
        const int64_t bi = b0 + i * stride;
        u[i][t] = bi < nbytes ? cu[(int64_t)t * nbytes + bi] : 0u;
        w[i][t] = bi < nbytes ? cw[(int64_t)t * nbytes + bi] : 0u;
      }
#pragma unroll
    for (int i = 0; i < U; ++i) {
      const int64_t bi = b0 + i * stride;
      if (bi >= nbytes) break;
      uint2 v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        uint32_t idx = 0;
#pragma unroll
        for (int t = 0; t < T; ++t)
          idx |= (((u[i][t] >> (2 * e)) & 3u) << (2 * t)) | (((w[i][t] >> (2 * e)) & 3u) << (4 + 2 * t));
        v[e] = table[idx];
      }
      const int64_t n = (int64_t)((uint32_t)bi / (uint32_t)kb), j = bi - n * kb;  // N K / 4 <= 2^28
      R[(2 * n) * kb + j] = make_uint4(v[0].x, v[1].x, v[2].x, v[3].x);  // row 2n: K words, K / 4 uint4
      R[(2 * n + 1) * kb + j] = make_uint4(v[0].y, v[1].y, v[2].y, v[3].y);
    }
  }
}

// The same for T >= 3, whose tables (4096 blocks and more) cost more to form
// than the entries they would serve: every entry summed on its own.  One
// thread per packed byte, i.e. four entries (n, 4 j .. 4 j + 3).
__global__ __launch_bounds__(256) void realify_codes_kernel(const uint8_t* __restrict__ cu,
                                                            const float* __restrict__ su,
                                                            const uint8_t* __restrict__ cw,
                                                            const float* __restrict__ sw, int T, int64_t N,
                                                            int64_t K, uint4* __restrict__ R) {
  const int64_t nbytes = N * K / 4, kb = K / 4;
  for (int64_t bi = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; bi < nbytes;
       bi += (int64_t)gridDim.x * blockDim.x) {
    RealSum a[4] = {};
#pragma unroll
    for (int t = 0; t < FAIRY2I_MAX_STAGES; ++t) {
      if (t >= T) break;
      const uint32_t bu = cu[(int64_t)t * nbytes + bi], bw = cw[(int64_t)t * nbytes + bi];
      const double sur = (double)su[2 * t], sui = (double)su[2 * t + 1];
      const double swr = (double)sw[2 * t], swi = (double)sw[2 * t + 1];
#pragma unroll
      for (int e = 0; e < 4; ++e)
        real_add(a[e], (int)((bu >> (2 * e)) & 3u), (int)((bw >> (2 * e)) & 3u), sur, sui, swr, swi);
    }
    uint2 v[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = real_block(a[e]);
    const int64_t n = (int64_t)((uint32_t)bi / (uint32_t)kb), j = bi - n * kb;  // N K / 4 <= 2^28
    R[(2 * n) * kb + j] = make_uint4(v[0].x, v[1].x, v[2].x, v[3].x);
    R[(2 * n + 1) * kb + j] = make_uint4(v[0].y, v[1].y, v[2].y, v[3].y);
  }
}

// Eight values a thread, as two 16-byte loads and one 16-byte store, where
// both pointers are 16-byte aligned (`groups` of eight; the rest, and
// everything otherwise, one at a time).  One value a thread moved the 100 MB
// of 16.8 M values in 26 us (37 us from cold caches); this does in 15 (19).
__global__ __launch_bounds__(256) void f32_to_bf16_kernel(const float* __restrict__ in, int64_t n, int64_t groups,
                                                          uint16_t* __restrict__ out) {
  const int64_t t0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = t0; i < groups; i += stride) {
    const float4 a = reinterpret_cast<const float4*>(in)[2 * i], b = reinterpret_cast<const float4*>(in)[2 * i + 1];
    auto pair = [](float x, float y) { return (uint32_t)bf16_rne_bits(x) | ((uint32_t)bf16_rne_bits(y) << 16); };
    reinterpret_cast<uint4*>(out)[i] = make_uint4(pair(a.x, a.y), pair(a.z, a.w), pair(b.x, b.y), pair(b.z, b.w));
  }
  for (int64_t i = 8 * groups + t0; i < n; i += stride) out[i] = bf16_rne_bits(in[i]);
}

inline unsigned grid_for(int64_t n) {
  int64_t b = (n + 255) / 256;
  if (b > 65536) b = 65536;
  return (unsigned)(b < 1 ? 1 : b);
}

}  // namespace

}  // namespace fairy2i

using namespace fairy2i;

extern "C" {

fairy2i_status fairy2i_wl_realify(const void* U, const void* W, int32_t dtype, int64_t N, int64_t K, void* R,
                                  void* stream) {
  if (!U || !W || !R) return FAIRY2I_ERR_NULL;
  if (dtype != FAIRY2I_ACT_F32 && dtype != FAIRY2I_ACT_BF16) return FAIRY2I_ERR_DTYPE;
  if (N <= 0 || K <= 0 || N > ((int64_t)1 << 30) / K) return FAIRY2I_ERR_SHAPE;
  hipLaunchKernelGGL(realify_kernel, dim3(grid_for(N * K)), dim3(256), 0, static_cast<hipStream_t>(stream), U, W,
                     dtype, N, K, static_cast<uint32_t*>(R));
  return hipGetLastError() == hipSuccess ? FAIRY2I_OK : FAIRY2I_ERR_HIP;
}

fairy2i_status fairy2i_wl_realify_codes(const uint8_t* codes_U, const float* scales_U, const uint8_t* codes_W,
                                        const float* scales_W, int32_t T, int64_t N, int64_t K, void* R,
                                        void* stream) {
  if (!codes_U || !scales_U || !codes_W || !scales_W || !R) return FAIRY2I_ERR_NULL;
  if (T < 1 || T > FAIRY2I_MAX_STAGES) return FAIRY2I_ERR_STAGES;
  if (N <= 0 || K <= 0 || K % 4 != 0 || N > ((int64_t)1 << 30) / K) return FAIRY2I_ERR_SHAPE;
  if (reinterpret_cast<uintptr_t>(R) & 15) return FAIRY2I_ERR_SHAPE;
  const hipStream_t st = static_cast<hipStream_t>(stream);
  auto* out = static_cast<uint4*>(R);
  if (T <= 2) {
    // four bytes a thread, so a block's table serves 4096 entries
    auto* kernel = T == 1 ? realify_table_kernel<1> : realify_table_kernel<2>;
    hipLaunchKernelGGL(kernel, dim3(grid_for((N * K / 4 + 3) / 4)), dim3(256), 0, st, codes_U, scales_U, codes_W,
                       scales_W, N, K, out);
  } else {
    hipLaunchKernelGGL(realify_codes_kernel, dim3(grid_for(N * K / 4)), dim3(256), 0, st, codes_U, scales_U, codes_W,
                       scales_W, T, N, K, out);
  }
  return hipGetLastError() == hipSuccess ? FAIRY2I_OK : FAIRY2I_ERR_HIP;
}

fairy2i_status fairy2i_wl_unrealify_grad(const float* G_R, int64_t N, int64_t K, float* G_U, float* G_W,
                                         void* stream) {
  if (!G_R || !G_U || !G_W) return FAIRY2I_ERR_NULL;
  if (N <= 0 || K <= 0 || N > ((int64_t)1 << 30) / K) return FAIRY2I_ERR_SHAPE;
  hipLaunchKernelGGL(unrealify_grad_kernel, dim3(grid_for(N * K)), dim3(256), 0, static_cast<hipStream_t>(stream),
                     reinterpret_cast<const float2*>(G_R), N, K, reinterpret_cast<float2*>(G_U),
                     reinterpret_cast<float2*>(G_W));
  return hipGetLastError() == hipSuccess ? FAIRY2I_OK : FAIRY2I_ERR_HIP;
}

fairy2i_status fairy2i_f32_to_bf16(const float* in, int64_t n, void* out, void* stream) {
  if (!in || !out) return FAIRY2I_ERR_NULL;
  if (n <= 0) return FAIRY2I_ERR_SHAPE;
  const bool vec = ((reinterpret_cast<uintptr_t>(in) | reinterpret_cast<uintptr_t>(out)) & 15) == 0;
  const int64_t groups = vec ? n / 8 : 0;
  hipLaunchKernelGGL(f32_to_bf16_kernel, dim3(grid_for(vec ? (n + 7) / 8 : n)), dim3(256), 0,
                     static_cast<hipStream_t>(stream), in, n, groups, static_cast<uint16_t*>(out));
  return hipGetLastError() == hipSuccess ? FAIRY2I_OK : FAIRY2I_ERR_HIP;
}

}  // extern "C"
