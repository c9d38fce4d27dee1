// Per-token int8 activations: absmax over the 2K real components of a token,
// q = clamp(rint(x * (127 / g)), -127, 127), dequantisation factor g / 127,
// all in float32 with IEEE division (no fast-math).  One block per token;
// the absmax is a max, so its value does not depend on reduction order.
#include "common.h"

namespace fairy2i {

namespace {

template <int DT>
__device__ inline float load_act(const void* x, int64_t i) {
  if constexpr (DT == FAIRY2I_ACT_F32) {
    return static_cast<const float*>(x)[i];
  } else {
    const uint32_t bits = static_cast<const uint16_t*>(x)[i];
    return __uint_as_float(bits << 16);
  }
}

__device__ inline float block_max(float m, float* red) {
  for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  float g = red[0];
  for (int w = 1; w < (int)(blockDim.x >> 6); ++w) g = fmaxf(g, red[w]);
  return g;
}

__device__ inline int8_t quantise(float x, float inv) {
  return (int8_t)(int)fminf(fmaxf(rintf(__fmul_rn(x, inv)), -127.0f), 127.0f);
}

// Any size and alignment: one value at a time, the token read twice.
template <int DT>
__global__ __launch_bounds__(256) void act_quant_kernel(const void* __restrict__ x, int64_t K,
                                                        int8_t* __restrict__ q,
                                                        float* __restrict__ x_scale) {
  __shared__ float red[256 / 64];
  const int64_t b = blockIdx.x;
  const int64_t n = 2 * K;
  const int64_t base = b * n;
  float m = 0.0f;
  for (int64_t i = threadIdx.x; i < n; i += blockDim.x) m = fmaxf(m, fabsf(load_act<DT>(x, base + i)));
  const float g = block_max(m, red);
  if (g == 0.0f) {  // a branch per token: one per value keeps the loop's loads from going out together
    for (int64_t i = threadIdx.x; i < n; i += blockDim.x) q[base + i] = 0;
    if (threadIdx.x == 0) x_scale[b] = 0.0f;
    return;
  }
  const float inv = 127.0f / g;
  for (int64_t i = threadIdx.x; i < n; i += blockDim.x) q[base + i] = quantise(load_act<DT>(x, base + i), inv);
  if (threadIdx.x == 0) x_scale[b] = g / 127.0f;
}

// Tokens of whole, 16-byte aligned groups of eight values, up to
// GROUPS * NT of them: the token is read once, its values stay in
// registers from the maximum to the rounding.  What bounds it is the chain
// load - reduce - store, so all of a thread's loads go out together (one
// value at a time and two passes over the token: 11.6 us for 16 tokens of
// K = 5504 bf16, 9.4 and 31.8 us for 2048 of K = 2048 and 5504; now 4.0, 8.0
// and 13.3).  Short tokens take short blocks: with 512 threads for every K,
// most of them idle, many tokens were slower than one value at a time (bf16,
// one value at a time / 512 threads / now: 4096 tokens of K = 256 6.5 / 10.1 /
// 3.8 us, K = 512 8.3 / 10.6 / 4.5, K = 1024 11.1 / 11.6 / 6.9; 100,000 of
// K = 64 69 / 178 / 25; from K = 2048 on 512 threads are right: 22.7 / 14.2).
template <int DT, int NT, int GROUPS>
__global__ __launch_bounds__(NT) void act_quant_vec_kernel(const void* __restrict__ x, int groups,
                                                           uint2* __restrict__ q, float* __restrict__ x_scale) {
  __shared__ float red[NT / 64];
  const int64_t b = blockIdx.x;
  constexpr int W = DT == FAIRY2I_ACT_F32 ? 2 : 1;  // 16-byte words per group
  const uint4* src = static_cast<const uint4*>(x) + b * groups * W;
  uint4 w[GROUPS][W];
#pragma unroll
  for (int i = 0; i < GROUPS; ++i)
#pragma unroll
    for (int h = 0; h < W; ++h) {
      const int gi = threadIdx.x + i * NT;
      w[i][h] = gi < groups ? src[gi * W + h] : make_uint4(0u, 0u, 0u, 0u);
    }
  auto value = [&](int i, int e) -> float {  // e-th value of group i
    if constexpr (DT == FAIRY2I_ACT_F32) {
      const uint4 v = w[i][e >> 2];
      const uint32_t c[4] = {v.x, v.y, v.z, v.w};
      return __uint_as_float(c[e & 3]);
    } else {
      const uint32_t c[4] = {w[i][0].x, w[i][0].y, w[i][0].z, w[i][0].w};
      return __uint_as_float(e & 1 ? c[e >> 1] & 0xFFFF0000u : c[e >> 1] << 16);
    }
  };
  float m = 0.0f;
#pragma unroll
  for (int i = 0; i < GROUPS; ++i)
#pragma unroll
    for (int e = 0; e < 8; ++e) m = fmaxf(m, fabsf(value(i, e)));
  const float g = block_max(m, red);
  const float inv = g == 0.0f ? 0.0f : 127.0f / g;
#pragma unroll
  for (int i = 0; i < GROUPS; ++i) {
    const int gi = threadIdx.x + i * NT;
    if (gi >= groups) break;
    uint32_t out[2] = {0u, 0u};
#pragma unroll
    for (int e = 0; e < 8; ++e)
      if (g != 0.0f) out[e >> 2] |= (uint32_t)(uint8_t)quantise(value(i, e), inv) << (8 * (e & 3));
    q[b * groups + gi] = make_uint2(out[0], out[1]);
  }
  if (threadIdx.x == 0) x_scale[b] = g / 127.0f;
}

template <int DT, int NT, int GROUPS>
void launch_vec(const void* x, int64_t B, int64_t K, int8_t* q, float* x_scale, hipStream_t s) {
  hipLaunchKernelGGL((act_quant_vec_kernel<DT, NT, GROUPS>), dim3((unsigned)B), dim3(NT), 0, s, x, (int)(K / 4),
                     reinterpret_cast<uint2*>(q), x_scale);
}

template <int DT>
void launch_dt(const void* x, int64_t B, int64_t K, int8_t* q, float* x_scale, hipStream_t s) {
  // K % 4 == 0: a token is whole groups, every token starts on a group
  const bool vec = K % 4 == 0 && K <= 8192 &&
                   ((reinterpret_cast<uintptr_t>(x) & 15) | (reinterpret_cast<uintptr_t>(q) & 7)) == 0;
  if (!vec)
    hipLaunchKernelGGL(act_quant_kernel<DT>, dim3((unsigned)B), dim3(256), 0, s, x, K, q, x_scale);
  else if (K <= 256)
    launch_vec<DT, 64, 1>(x, B, K, q, x_scale, s);
  else if (K <= 512)
    launch_vec<DT, 64, 2>(x, B, K, q, x_scale, s);
  else if (K <= 1024)
    launch_vec<DT, 256, 1>(x, B, K, q, x_scale, s);
  else
    launch_vec<DT, 512, 4>(x, B, K, q, x_scale, s);
}

}  // namespace

hipError_t launch_quantize_act_int8(const void* x, int dtype, int64_t B, int64_t K, int8_t* q,
                                    float* x_scale, hipStream_t stream) {
  if (dtype == FAIRY2I_ACT_F32) launch_dt<FAIRY2I_ACT_F32>(x, B, K, q, x_scale, stream);
  else launch_dt<FAIRY2I_ACT_BF16>(x, B, K, q, x_scale, stream);
  return hipGetLastError();
}

}  // namespace fairy2i
