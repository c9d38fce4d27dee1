// One widely-linear decoder block for one decode token (Sec. 1: every linear
// layer of the LLaMA-style block becomes a widely-linear layer; Sec. 3.1,
// self-attention paragraph, Eq. hermitian-score: scores Re(q^H k) / sqrt(d_k),
// softmax and value aggregation acting on the real and imaginary parts alike,
// a widely-linear output projection).
//
// The seven projections run on the grouped fp8 x fp4 decode path (q, k, v in
// one call; o; gate and up in one call; down).  Between them:
//   add_rmsnorm   residual add, RMSNorm over the 2n real components, bf16 out
//   rope_append   rotary embedding as a complex rotation per head entry
//                 (angles in double), key and value written to the caches
//   attn_partial  per (head, run of 64 or more positions): scores, the run's
//                 maximum, softmax sum and weighted sum of values
//   attn_combine  the runs of a head merged in a fixed order, bf16 out
//   swiglu        silu(Re g) Re u + i silu(Im g) Im u, bf16 out
//   add           the final residual add
// For one token with two digit bands (every block this library plans, up to
// 8192 complex entries per token) the fused path runs instead: six launches
// in place of 19, one per product with the stages around it inside, and the
// attention's two:
//   norm, q k v product, rotary embedding, caches
//   attention
//   o product, first residual add
//   norm, gate and up product, SwiGLU
//   down product, second residual add
// Complex vectors are float2 (re, im); a head owns dc = n / n_heads
// consecutive complex entries (entry j: its real dims j and j + dc).  All
// reductions run in a fixed order, so results are bitwise reproducible.
#include <math.h>
#include <string.h>

#include "common.h"
#include "decode_dev.h"
#include "f4_operand.h"

namespace fairy2i {

namespace {

constexpr int kAttnRun = 64;  // positions of an attention block's shortest run
constexpr int64_t kMaxContext = (int64_t)1 << 18;
constexpr int kNormThreads = 256;

__device__ inline uint16_t bf16_rne(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

template <typename V>
__device__ inline V wave_sum(V v) {
  // butterfly: every lane ends with the same, commutatively formed sum
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  return v;
}

__device__ inline float wave_max(float v) {
  for (int off = 32; off > 0; off >>= 1) v = fmaxf(v, __shfl_xor(v, off));
  return v;
}

__device__ inline double wave_max(double v) {
  for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off));
  return v;
}

// v = x (+ a); h_out = v (if given); z = bf16(v / sqrt(mean(v^2) + eps) * gamma)
// over the 2n real components.  One block per token.
__global__ __launch_bounds__(kNormThreads) void add_rmsnorm_kernel(const float2* __restrict__ x,
                                                                   const float2* __restrict__ a,
                                                                   float2* __restrict__ h_out,
                                                                   const float* __restrict__ gamma, float eps,
                                                                   int n, uint16_t* __restrict__ z) {
  __shared__ float red[kNormThreads / 64];
  float ss = 0.0f;
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    float2 v = x[i];
    if (a) {
      const float2 w = a[i];
      v.x += w.x;
      v.y += w.y;
    }
    ss = fmaf(v.x, v.x, ss);
    ss = fmaf(v.y, v.y, ss);
  }
  ss = wave_sum(ss);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
  __syncthreads();
  float tot = 0.0f;
  for (int w = 0; w < kNormThreads / 64; ++w) tot += red[w];
  const float r = 1.0f / sqrtf(tot / (float)(2 * n) + eps);
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    float2 v = x[i];
    if (a) {
      const float2 w = a[i];
      v.x += w.x;
      v.y += w.y;
    }
    if (h_out) h_out[i] = v;
    z[2 * i] = bf16_rne((v.x * r) * gamma[i]);
    z[2 * i + 1] = bf16_rne((v.y * r) * gamma[n + i]);
  }
}

// Rotary embedding of q and k (entry j of a head turned by pos * theta_j,
// theta_j = base^(-2 j / dh), dh = 2 dc), then k and v stored at position pos
// of the caches [H][max_ctx][dc].
__global__ void rope_append_kernel(const float2* __restrict__ q, const float2* __restrict__ k,
                                   const float2* __restrict__ v, int n, int dc, int64_t pos, int64_t max_ctx,
                                   double base, float2* __restrict__ q_rot, float2* __restrict__ k_cache,
                                   float2* __restrict__ v_cache) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int h = i / dc, j = i - h * dc;
  const double ang = (double)pos * pow(base, -2.0 * (double)j / (double)(2 * dc));
  double s, c;
  sincos(ang, &s, &c);
  const float cf = (float)c, sf = (float)s;
  const float2 qv = q[i], kv = k[i];
  q_rot[i] = make_float2(fmaf(qv.x, cf, -qv.y * sf), fmaf(qv.x, sf, qv.y * cf));
  const int64_t at = ((int64_t)h * max_ctx + pos) * dc + j;
  k_cache[at] = make_float2(fmaf(kv.x, cf, -kv.y * sf), fmaf(kv.x, sf, kv.y * cf));
  v_cache[at] = v[i];
}

// One block of four waves per (run of positions, head).  Each wave takes every
// fourth step of 16 / R positions of the run and keeps the running maximum m,
// l = sum e^(s_t - m) and o = sum e^(s_t - m) v_t of its own, so nothing in the
// walk waits for another wave.  Scores: 8 R lanes per position, which take a
// key row's 16-byte chunks in turn (eight loads in flight a lane), summed
// across the lanes, times scale.  Values: 16 bytes a lane, eight loads in
// flight, asked for before the step's scores are formed, and the next step's
// keys before its values are needed.  At the end the four waves' sums are
// brought to one maximum and added in wave order.  From the scores on
// everything is in double: the output is rounded to bf16, and a sum in float
// puts a value next to a tie on the wrong side about once a token of 2048
// entries.  Partial record per (head, run): [m, l, o (2 dc doubles)].
// Bound by memory: 32 heads of 64 entries take 13.3 us for the 67 MB of context
// 2048, 180 us for the 1.07 GB of 32768 (6.0 TB/s).  One block per 64 positions,
// its waves meeting between scores and values, left four blocks a CU too few
// bytes in flight: 14.1 us at 2048; block calls, us, with it / now: context 32768
// 304 / 219, 262144 2172 / 1423, n = 4096 (64 heads) at 262144 4213 / 2826.
constexpr int kAttnThreads = 256;
template <int R>  // dc <= 64 R; R = 1, 2 or 4
__global__ __launch_bounds__(kAttnThreads, R == 1 ? 4 : 3) void attn_partial_kernel(
    const float2* __restrict__ q_rot, const float2* __restrict__ k_cache, const float2* __restrict__ v_cache, int dc,
    int n_ctx, int64_t max_ctx, int run, double scale, double2* __restrict__ part) {
#if defined(__HIP_DEVICE_COMPILE__)  // buffer-descriptor code: device pass only
  constexpr int W = kAttnThreads / 64;
  constexpr int LP = 8 * R, PR = 64 / LP, PS = 2 * PR;        // lanes a key row, rows a load, rows a step
  constexpr int RPI = R == 1 ? 2 : 1, NR = R == 4 ? 2 : 1;    // value rows a load, loads a row
  constexpr int VL = PS / RPI, LV = 64 / RPI;                 // loads a step (of NR), lanes a value row
  __shared__ double2 qs[32 * R][2];  // in registers over the walk it would spill
  __shared__ double es[W][PS];
  __shared__ double redm[W], redl[W];
  __shared__ double2 ow[W][64 * R];
  const int h = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);
  const int t_end = min((int)(blockIdx.x + 1) * run, n_ctx), nf4 = dc / 2;
  // Rows of the head from position t to the run's end (past it: zeros), each
  // load's own descriptor: scalar arithmetic in place of sixteen vector offsets
  const uint32_t row = 8u * (uint32_t)dc;  // at most 2 KB, positions below 2^18: 32 bits
  const float2* kh = k_cache + (int64_t)h * max_ctx * dc;
  const float2* vh = v_cache + (int64_t)h * max_ctx * dc;
  auto rows_from = [&](const float2* head, int t) {
    return make_rsrc(uniform_ptr(head + (int64_t)t * dc), t < t_end ? (uint32_t)(t_end - t) * row : 0u);
  };
  const int p = lane / LP, qd = lane % LP, vr = lane / LV, vj = lane % LV;
  uint32_t koff[4], voff[NR];  // of the lane's chunks
#pragma unroll
  for (int u = 0; u < 4; ++u) koff[u] = qd + LP * u < nf4 ? 16u * (uint32_t)(qd + LP * u) + (uint32_t)p * row : kOob;
#pragma unroll
  for (int r = 0; r < NR; ++r) voff[r] = vj + LV * r < nf4 ? 16u * (uint32_t)(vj + LV * r) + (uint32_t)vr * row : kOob;
  v4f kv[2][4], vv[VL][NR];
  auto load_keys = [&](int t) {
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int hf = 0; hf < 2; ++hf) kv[hf][u] = __builtin_bit_cast(v4f, buf_load16(rows_from(kh, t + PR * hf), koff[u]));
  };
  auto load_values = [&](int t) {
#pragma unroll
    for (int u = 0; u < VL; ++u)
#pragma unroll
      for (int r = 0; r < NR; ++r) vv[u][r] = __builtin_bit_cast(v4f, buf_load16(rows_from(vh, t + u * RPI), voff[r]));
  };
  int t0 = (int)blockIdx.x * run + PS * wave;
  if (t0 < t_end) load_keys(t0);
  for (int j = tid; j < 32 * R; j += kAttnThreads) {
    const float4 q = j < nf4 ? reinterpret_cast<const float4*>(q_rot + (int64_t)h * dc)[j] : make_float4(0.f, 0.f, 0.f, 0.f);
    qs[j][0] = make_double2(q.x, q.y);
    qs[j][1] = make_double2(q.z, q.w);
  }
  __syncthreads();
  double m = -INFINITY, l = 0.0, o[NR][4];
#pragma unroll
  for (int r = 0; r < NR; ++r) o[r][0] = o[r][1] = o[r][2] = o[r][3] = 0.0;
  while (t0 < t_end) {
    load_values(t0);
    double s[2] = {0.0, 0.0};
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const double2 q01 = qs[qd + LP * u][0], q23 = qs[qd + LP * u][1];
      const double q[4] = {q01.x, q01.y, q23.x, q23.y};
#pragma unroll
      for (int hf = 0; hf < 2; ++hf)
#pragma unroll
        for (int k = 0; k < 4; ++k) s[hf] = fma(q[k], (double)kv[hf][u][k], s[hf]);
    }
    const int t1 = t0 + W * PS;
    __builtin_amdgcn_sched_barrier(0);  // the keys' registers, for the next step's
    load_keys(t1);                      // past the run: zeros
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int hf = 0; hf < 2; ++hf) {
#pragma unroll
      for (int off = 1; off < LP; off <<= 1) s[hf] += __shfl_xor(s[hf], off);
      s[hf] = t0 + p + PR * hf < t_end ? s[hf] * scale : -INFINITY;
    }
    double mn = fmax(s[0], s[1]);
#pragma unroll
    for (int off = LP; off < 64; off <<= 1) mn = fmax(mn, __shfl_xor(mn, off));
    mn = fmax(m, mn);
    const double ref = mn == -INFINITY ? 0.0 : mn;  // no score above -infinity yet: every e is 0
    const double f = exp(m - ref);
    l *= f;
#pragma unroll
    for (int hf = 0; hf < 2; ++hf) {
      const double e = exp(s[hf] - ref);
      l += e;  // of the lane's positions, alike in the LP lanes of one
      if (qd == 0) es[wave][p + PR * hf] = e;
    }
    wave_sync();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
      for (int k = 0; k < 4; ++k) o[r][k] *= f;
#pragma unroll
    for (int u = 0; u < VL; ++u) {
      const double w = es[wave][u * RPI + vr];  // 0 past the run
#pragma unroll
      for (int r = 0; r < NR; ++r) {
#pragma unroll
        for (int k = 0; k < 4; ++k) o[r][k] = fma(w, (double)vv[u][r][k], o[r][k]);
      }
    }
    wave_sync();
    m = mn;
    t0 = t1;
  }
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    if constexpr (RPI == 2) {
#pragma unroll
      for (int k = 0; k < 4; ++k) o[r][k] += __shfl_xor(o[r][k], 32);
    }
    if (vr == 0) {
      ow[wave][2 * (vj + LV * r)] = make_double2(o[r][0], o[r][1]);
      ow[wave][2 * (vj + LV * r) + 1] = make_double2(o[r][2], o[r][3]);
    }
  }
  l = wave_sum(qd == 0 ? l : 0.0);
  if (lane == 0) {
    redm[wave] = m;
    redl[wave] = l;
  }
  __syncthreads();
  double M = redm[0];
#pragma unroll
  for (int w = 1; w < W; ++w) M = fmax(M, redm[w]);
  const double ref = M == -INFINITY ? 0.0 : M;
  double f[W], L = 0.0;
#pragma unroll
  for (int w = 0; w < W; ++w) {
    f[w] = exp(redm[w] - ref);  // 0 for a wave without positions
    L = fma(redl[w], f[w], L);
  }
  double2* rec = part + ((int64_t)h * gridDim.x + blockIdx.x) * (1 + dc);
  if (tid == 0) rec[0] = make_double2(M, L);
  for (int j = tid; j < dc; j += kAttnThreads) {
    double2 a = make_double2(0.0, 0.0);
#pragma unroll
    for (int w = 0; w < W; ++w) {
      a.x = fma(ow[w][j].x, f[w], a.x);
      a.y = fma(ow[w][j].y, f[w], a.y);
    }
    rec[1 + j] = a;
  }
#endif
}

// Per head: M = max_s m_s, f_s = e^(m_s - M) (in LDS), L = sum_s l_s f_s,
// o_j = sum_s o_{s,j} f_s / L over the runs s, wave w adding w, w + 4, ... and the
// waves' sums added in wave order; written as bf16 pairs at the head's
// entries.  (A kernel of its own: merged by the block that ends last for its
// head, every run's block waits for its record and for its count, 18.4 us
// at context 2048 and 36.3 at 4096 in all, against 14.2 + 4.7 and 25.4 + 4.7.)
template <int R>
__global__ __launch_bounds__(kAttnThreads) void attn_combine_kernel(const double2* __restrict__ part, int ns, int dc,
                                                                    uint32_t* __restrict__ o_out) {
  extern __shared__ double fs[];
  __shared__ double redm[kAttnThreads / 64], redl[kAttnThreads / 64];
  __shared__ double2 ow[kAttnThreads / 64][64 * R];
  const int h = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int rl = 1 + dc;
  const double2* ph = part + (int64_t)h * ns * rl;
  // every wave's first eight runs (of an entry a lane) and every thread's
  // first (m, l) in one round of loads
  double2 ov[8];
  auto load_runs = [&](int i0, int r) {
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int i = i0 + 4 * u, j = lane + 64 * r;
      ov[u] = i < ns && j < dc ? ph[(int64_t)i * rl + 1 + j] : make_double2(0.0, 0.0);
    }
  };
  const double2 ml0 = tid < ns ? ph[(int64_t)tid * rl] : make_double2(-INFINITY, 0.0);
  load_runs(wave, 0);
  double M = ml0.x;
  for (int i = tid + kAttnThreads; i < ns; i += kAttnThreads) M = fmax(M, ph[(int64_t)i * rl].x);
  M = wave_max(M);
  if (lane == 0) redm[wave] = M;
  __syncthreads();
  M = fmax(fmax(redm[0], redm[1]), fmax(redm[2], redm[3]));
  double lt = 0.0;
  for (int i = tid; i < ns; i += kAttnThreads) {
    const double2 ml = i == tid ? ml0 : ph[(int64_t)i * rl];
    const double f = exp(ml.x - M);
    fs[i] = f;
    lt = fma(ml.y, f, lt);
  }
  lt = wave_sum(lt);
  if (lane == 0) redl[wave] = lt;
  __syncthreads();
  const double L = ((redl[0] + redl[1]) + redl[2]) + redl[3];
#pragma unroll 1
  for (int r = 0; r < R; ++r) {
    double2 a = make_double2(0.0, 0.0);
    for (int i0 = wave; i0 < ns; i0 += 32) {
      if (r > 0 || i0 != wave) load_runs(i0, r);
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int i = i0 + 4 * u;
        const double f = i < ns ? fs[i] : 0.0;
        a.x = fma(ov[u].x, f, a.x);
        a.y = fma(ov[u].y, f, a.y);
      }
    }
    ow[wave][lane + 64 * r] = a;
  }
  __syncthreads();
  for (int j = tid; j < dc; j += kAttnThreads) {
    double2 a = ow[0][j];
    for (int w = 1; w < kAttnThreads / 64; ++w) {
      a.x += ow[w][j].x;
      a.y += ow[w][j].y;
    }
    o_out[h * dc + j] = (uint32_t)bf16_rne((float)(a.x / L)) | ((uint32_t)bf16_rne((float)(a.y / L)) << 16);
  }
}

__device__ inline float silu(float v) { return v / (1.0f + expf(-v)); }

__global__ void swiglu_kernel(const float2* __restrict__ g, const float2* __restrict__ u, int n,
                              uint16_t* __restrict__ act) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float2 gv = g[i], uv = u[i];
  act[2 * i] = bf16_rne(silu(gv.x) * uv.x);
  act[2 * i + 1] = bf16_rne(silu(gv.y) * uv.y);
}

__global__ void add_kernel(const float2* __restrict__ a, const float2* __restrict__ b, int n,
                           float2* __restrict__ out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float2 av = a[i], bv = b[i];
  out[i] = make_float2(av.x + bv.x, av.y + bv.y);
}

// ---------------------------------------------------------- fused path ---
// One product per launch, the stages around it inside.  What bounds a block
// of one token is latency: its codes (50 MB at n = 2048, n_ff = 5504, T = 2)
// and 2048 cached positions (67 MB) take 20 us at the rate of a large copy,
// while each launch of a chain costs 4-7 us whatever it does.  So a thread
// block owns 16 rows of a projection (of gate and of up for SwiGLU: M = 2
// matrices), its waves split K in 256-code steps (wave w of a matrix takes
// steps w, w + KW, ...) and add their shares of y in LDS, in double and in
// wave order; nothing is left for a reduction, and what follows the row
// (rotary embedding and caches, residual add, SwiGLU) is done by the thread
// that holds it.  The token is formed by every block: RMSNorm of x (the same
// fixed order in each) or the bf16 token as it stands; a wave then encodes
// the digits of its own steps (f4_operand.h), a lane per half run and
// component, while its codes, asked for before all this, arrive.  What is
// rounded to bf16 (the tokens, SwiGLU) is computed in double up to there,
// from the digits' sums on: the fewer roundings, the fewer values fall on the
// other side of a tie (products against 64 bits 6.5e-8 -> 2.5e-8).
// One token at the sizes above: 13 launches 78.6 us, now 51.7; the products
// with their stages 10.2 (q k v), 5.1 (o), 12.4 (gate, up) and 8.0 (down).
struct SplitMatrix {
  const uint8_t* codes[2];  // U, W, fp4 tiled
  const float* scales[2];
  float2* y;
};

struct SplitArgs {
  int32_t K, nk4, N;
  uint32_t code_bytes;  // of one matrix's codes
  SplitMatrix m[3];
  // kSrcNorm: the token z = bf16(x / sqrt(mean |x|^2 + eps) gamma); kSrcBf16: tok
  const float2* x;
  const float* gamma;
  float eps;
  uint32_t* z_out;
  const uint32_t* tok;
  // kOutRope
  const double* theta;
  int64_t pos, max_ctx;
  int32_t dc;
  float2 *q_rot, *k_cache, *v_cache;
  // kOutAdd: sum = base + y
  const float2* base;
  float2* sum;
  // kOutSwiglu
  uint32_t* act;
};

constexpr int kSrcNorm = 0, kSrcBf16 = 1;
constexpr int kOutRope = 0, kOutAdd = 1, kOutSwiglu = 2;
constexpr int kSplitMaxK = 8192;  // complex entries of a token the fused path takes

// M matrices with KW waves each; a token of K <= E * threads entries.  (T = 3:
// 128 registers, so that two blocks fit a CU: with the 164 of q, k and v past
// K = 2048 a block of n = 8192, n_ff = 1024 took 141 us, now 125.5.)
template <int T, int KW, int M, int SRC, int OUT, int E>
__global__ __launch_bounds__(64 * KW * M, T == 3 ? 4 : 1) void block_product_kernel(SplitArgs a) {
#if defined(__HIP_DEVICE_COMPILE__)  // buffer-descriptor code: device pass only
  constexpr int P = 2 * T, W = KW * M, NTH = 64 * W;
  __shared__ __attribute__((aligned(16))) uint32_t tokw[E * NTH];
  __shared__ __attribute__((aligned(16))) uint8_t xop[W][16 * 8 * 16];  // a step's operand: [run][column][16 bytes]
  __shared__ double red[W];
  __shared__ float redm[W];
  __shared__ double part[W][2][17];  // [wave][component][row]
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, li = lane & 15;
  const int wave = uniform(tid >> 6);
  const int mat = OUT == kOutRope ? (int)blockIdx.y : (M == 2 ? wave / KW : 0);
  const int kw = wave % KW;
  const int rb = blockIdx.x, K = a.K;
  const bool first = blockIdx.x == 0 && blockIdx.y == 0;

  // theta first: its wait then leaves the loads below in flight
  double theta = 0.0;
  if constexpr (OUT == kOutRope) {
    if (tid < 32 && mat < 2) theta = a.theta[(rb * 16 + li) % a.dc];
  }
  const __amdgpu_buffer_rsrc_t ru = make_rsrc(uniform_ptr(a.m[mat].codes[0]), a.code_bytes);
  const __amdgpu_buffer_rsrc_t rw = make_rsrc(uniform_ptr(a.m[mat].codes[1]), a.code_bytes);
  auto load = [&](int s, v4i(&c)[P]) {  // a step past the last reads zeros
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const uint32_t off = s < a.nk4 ? (uint32_t)((rb * a.nk4 + s) * T + t) * 1024u + 16u * (uint32_t)lane : kOob;
      c[t] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(ru, off, 0, kNonTemporal));
      c[T + t] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rw, off, 0, kNonTemporal));
    }
  };
  uint32_t zw[E];
  float2 v[E];
  if constexpr (SRC == kSrcNorm) {
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int i = tid + e * NTH;
      v[e] = i < K ? a.x[i] : make_float2(0.0f, 0.0f);
    }
  } else {
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int i = tid + e * NTH;
      zw[e] = i < K ? a.tok[i] : 0u;
    }
  }
  // gains with the token where the registers allow it; the residual
  constexpr bool kGainsFirst = SRC == kSrcNorm && E <= 4;
  float2 ga[kGainsFirst ? E : 1];
  if constexpr (kGainsFirst) {
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int i = tid + e * NTH;
      ga[e] = i < K ? make_float2(a.gamma[i], a.gamma[K + i]) : make_float2(0.0f, 0.0f);
    }
  }
  float base = 0.0f;  // of row li, component g (lanes 0 .. 31 write the outputs)
  if constexpr (OUT == kOutAdd) {
    if (tid < 32) base = reinterpret_cast<const float*>(a.base)[2 * (rb * 16 + li) + g];
  }
  v4i c[P];
  load(kw, c);
  float sc[2][T][2];  // one wait for the scalar loads, the vector loads in flight
  sload_scales<T>(uniform_ptr(a.m[mat].scales[0]), uniform_ptr(a.m[mat].scales[1]), sc);
  double cs = 0.0, sn = 0.0;
  if constexpr (OUT == kOutRope) {
    if (tid < 32 && mat < 2) sincos((double)a.pos * theta, &sn, &cs);
  }
  if constexpr (SRC == kSrcNorm) {
    // a thread's few squares in float, the rest and the root in double
    float s0 = 0.0f;
#pragma unroll
    for (int e = 0; e < E; ++e) {
      s0 = fmaf(v[e].x, v[e].x, s0);
      s0 = fmaf(v[e].y, v[e].y, s0);
    }
    const double ss = wave_sum((double)s0);
    if (lane == 0) red[wave] = ss;
    __syncthreads();
    double tot = 0.0;
#pragma unroll
    for (int w = 0; w < W; ++w) tot += red[w];
    const double ms = tot / (double)(2 * K) + (double)a.eps;
    const double r0 = (double)(1.0f / sqrtf((float)ms));
    const double r = r0 > 0.0 && isfinite(r0) ? r0 * (1.5 - 0.5 * ms * r0 * r0) : r0;  // one Newton step
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int i = tid + e * NTH;
      zw[e] = 0u;
      if (i < K) {
        const float2 gn = kGainsFirst ? ga[kGainsFirst ? e : 0] : make_float2(a.gamma[i], a.gamma[K + i]);
        zw[e] = (uint32_t)bf16_rne((float)((double)v[e].x * r * (double)gn.x)) |
                ((uint32_t)bf16_rne((float)((double)v[e].y * r * (double)gn.y)) << 16);
        if (first) a.z_out[i] = zw[e];
      }
    }
  }
  float gm = 0.0f;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    tokw[tid + e * NTH] = zw[e];
    gm = fmaxf(gm, fmaxf(fabsf(__uint_as_float(zw[e] << 16)), fabsf(__uint_as_float(zw[e] & 0xFFFF0000u))));
  }
  gm = wave_max(gm);
  if (lane == 0) redm[wave] = gm;
  __syncthreads();
  gm = redm[0];
#pragma unroll
  for (int w = 1; w < W; ++w) gm = fmaxf(gm, redm[w]);
  const int S = f4_token_shift(gm);

  v4f aS[P], aI[P];
#pragma unroll
  for (int p = 0; p < P; ++p) aS[p] = aI[p] = v4f{0.f, 0.f, 0.f, 0.f};
  for (int s = kw; s < a.nk4; s += KW) {
    v4i cn[P];
    load(s + KW, cn);
    {
      const int hr = lane >> 1, comp = lane & 1, k0 = 256 * s + 8 * hr;
      uint32_t w8[8] = {};
      if (k0 < K) {  // K % 64 == 0: the half run is in range or past K entirely
        const uint4 p0 = *reinterpret_cast<const uint4*>(&tokw[k0]);
        const uint4 p1 = *reinterpret_cast<const uint4*>(&tokw[k0 + 4]);
        w8[0] = p0.x; w8[1] = p0.y; w8[2] = p0.z; w8[3] = p0.w;
        w8[4] = p1.x; w8[5] = p1.y; w8[6] = p1.z; w8[7] = p1.w;
      }
      float xv[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) xv[e] = __uint_as_float(comp ? (w8[e] & 0xFFFF0000u) : (w8[e] << 16));
      uint32_t out[2][2][2];
      f4_unit_digits(xv, S, 2, out);
      f4_store_unit(xop[wave], hr >> 1, 8, 0, comp, hr & 1, 2, out);
    }
    wave_sync();  // the wave's operand: written above, read below
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
      v4i x0 = v4i{0, 0, 0, 0}, x1 = x0;
      if (li < 8) {  // columns 8 .. 15 hold no token
        x0 = *reinterpret_cast<const v4i*>(&xop[wave][((8 * kb + g) * 8 + li) * 16]);
        x1 = *reinterpret_cast<const v4i*>(&xop[wave][((8 * kb + 4 + g) * 8 + li) * 16]);
      }
      const v8i xa = v8i{x0[0], x0[1], x0[2], x0[3], x1[0], x1[1], x1[2], x1[3]};
#pragma unroll
      for (int p = 0; p < P; ++p) {
        v8i bs, bi;
        expand_f4((uint32_t)c[p][2 * kb], (uint32_t)c[p][2 * kb + 1], bs, bi);
        aS[p] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(xa, bs, aS[p], kFmtFp8, kFmtFp4, 0, 0, 0, 0);
        aI[p] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(xa, bi, aI[p], kFmtFp8, kFmtFp4, 0, 0, 0, 0);
      }
    }
    wave_sync();
#pragma unroll
    for (int p = 0; p < P; ++p) c[p] = cn[p];
  }

  // the wave's share of y (before the token factor): lane group 0 holds the
  // first band's digits of row li, group 1 the second's (times 2^8); what
  // follows is linear, so each group forms its share and they are added last
  {
    double yr = 0.0, yi = 0.0;
#pragma unroll
    for (int t = 0; t < T; ++t) {
      double re[2][2], im[2][2];  // [matrix][component]: products with b_re = S - I and b_im = I
#pragma unroll
      for (int mm = 0; mm < 2; ++mm)
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          const int p = mm * T + t;
          const double vS = fma((double)aS[p][2 + k], 1.0 / kLoScale, (double)aS[p][k]);
          im[mm][k] = fma((double)aI[p][2 + k], 1.0 / kLoScale, (double)aI[p][k]);
          re[mm][k] = vS - im[mm][k];
        }
      const double u_re = sc[0][t][0], u_im = sc[0][t][1], w_re = sc[1][t][0], w_im = sc[1][t][1];
      yr = fma(u_re, re[0][0], yr);
      yr = fma(-u_im, im[0][1], yr);
      yr = fma(w_re, re[1][0], yr);
      yr = fma(w_im, im[1][1], yr);
      yi = fma(u_re, re[0][1], yi);
      yi = fma(u_im, im[0][0], yi);
      yi = fma(-w_re, re[1][1], yi);
      yi = fma(w_im, im[1][0], yi);
    }
    yr = fma(__shfl_down(yr, 16), 1.0 / kBand2Scale, yr);
    yi = fma(__shfl_down(yi, 16), 1.0 / kBand2Scale, yi);
    if (lane < 16) {  // zero for a wave without steps
      part[wave][0][li] = yr;
      part[wave][1][li] = yi;
    }
  }
  __syncthreads();
  if (tid >= 32) return;
  const int row = rb * 16 + li;  // N % 64 == 0: every row of the block exists; this lane's component is g
  const double f = gm > 0.0f ? (double)ldexpf(1.0f, -S) : 0.0;
  double y[M];
#pragma unroll
  for (int q = 0; q < M; ++q) {
    y[q] = 0.0;
#pragma unroll
    for (int w = 0; w < KW; ++w) y[q] += part[q * KW + w][g][li];
    y[q] *= f;
    reinterpret_cast<float*>(a.m[M == 2 ? q : mat].y)[2 * row + g] = (float)y[q];
  }
  if constexpr (OUT == kOutRope) {
    const double other = __shfl_xor(y[0], 16);
    const float rot = (float)(g == 0 ? y[0] * cs - other * sn : other * sn + y[0] * cs);
    const int h = row / a.dc;
    const int64_t at = 2 * (((int64_t)h * a.max_ctx + a.pos) * a.dc + (row - h * a.dc)) + g;
    if (mat == 0) reinterpret_cast<float*>(a.q_rot)[2 * row + g] = rot;
    else if (mat == 1) reinterpret_cast<float*>(a.k_cache)[at] = rot;
    else reinterpret_cast<float*>(a.v_cache)[at] = (float)y[0];
  } else if constexpr (OUT == kOutAdd) {
    reinterpret_cast<float*>(a.sum)[2 * row + g] = (float)((double)base + y[0]);
  } else {
    reinterpret_cast<uint16_t*>(a.act)[2 * row + g] = bf16_rne((float)(y[0] / (1.0 + exp(-y[0])) * y[M - 1]));
  }
#endif
}

// Waves per matrix: 8 (a step of 256 codes each up to K = 2048); 4 for the
// two matrices of SwiGLU, so that two blocks fit a CU (with 8 each one does,
// and 344 blocks take two rounds: 16.2 us against 11.4); 16 where K is
// longer and one matrix's rows leave most of the chip idle (8 from T = 3 on,
// whose sums take the registers: with 16 the T = 3 kernel spills, blocks of
// n = n_ff = 8192 184 us against 176; 4096, 8192 85 and 82).  The token takes E entries a thread.
template <int T, int SRC, int OUT>
void launch_block_product(const SplitArgs& a, hipStream_t s) {
  constexpr int KW = OUT == kOutSwiglu ? 4 : 8, M = OUT == kOutSwiglu ? 2 : 1, KL = OUT == kOutAdd && T <= 2 ? 16 : KW;
  const dim3 grid((unsigned)(a.N / 16), OUT == kOutRope ? 3 : 1);
  if (a.K <= 2048)
    hipLaunchKernelGGL((block_product_kernel<T, KW, M, SRC, OUT, 4>), grid, dim3(512), 0, s, a);
  else
    hipLaunchKernelGGL((block_product_kernel<T, KL, M, SRC, OUT, kSplitMaxK / (64 * KL * M)>), grid, dim3(64 * KL * M), 0, s, a);
}

template <int SRC, int OUT>
void launch_block_product(const SplitArgs& a, int T, hipStream_t s) {
  switch (T) {
    case 1: launch_block_product<1, SRC, OUT>(a, s); break;
    case 2: launch_block_product<2, SRC, OUT>(a, s); break;
    case 3: launch_block_product<3, SRC, OUT>(a, s); break;
    default: launch_block_product<4, SRC, OUT>(a, s); break;
  }
}

inline size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

// Plan: header, rotary frequencies, then the four group tables (q k v; o;
// gate up; down).
constexpr uint32_t kBlockMagic = 0xFA11B10Du;
constexpr int kGroups = 4;
struct BlockPlanHeader {
  uint32_t magic, abi;
  int64_t n, n_ff, max_ctx;
  int32_t n_heads, T;
  float eps;
  int32_t fused;  // one-token fp4 groups: the fused path runs
  double rope_base;
  const float* norm_attn;
  const float* norm_mlp;
  // workspace buffers
  uint16_t* z;
  float2 *q, *k, *v, *q_rot;
  double2* part;
  uint16_t* o;
  float2 *a, *h1;
  uint16_t* z2;
  float2 *g, *u;
  uint16_t* act;
  float2* d;
  size_t theta_off;   // rotary frequencies base^(-j / dc), j < dc (double)
  size_t table_off[kGroups];
  size_t table_bytes[kGroups];
};

struct BlockLayout {
  size_t z, q, k, v, q_rot, part, o, a, h1, z2, g, u, act, d, groups[kGroups], total;
};

// the projections of each group call, as indices into desc->codes_*: q k v, o, gate up, down
const int kGroupLayers[kGroups][3] = {{0, 1, 2}, {3, -1, -1}, {4, 5, -1}, {6, -1, -1}};

bool block_desc_ok(const fairy2i_block_desc* d) {
  if (!d || d->n <= 0 || d->n_ff <= 0 || d->n_heads <= 0 || d->max_ctx <= 0) return false;
  if (d->n % d->n_heads != 0 || d->n / d->n_heads > 256 || (d->n / d->n_heads) % 2 != 0) return false;
  if (d->n % 64 != 0 || d->n_ff % 64 != 0) return false;
  if (d->n > (1 << 24) || d->n_ff > (1 << 24) || d->max_ctx > kMaxContext) return false;
  if (d->T < 1 || d->T > FAIRY2I_MAX_STAGES || !(d->eps >= 0.0f) || !(d->rope_base > 0.0)) return false;
  return true;
}

// The group's layer descriptors, pointing at the workspace buffers of `ws`
// (null: a layout pass that only needs the shapes).
int group_layers(const fairy2i_block_desc* d, int gi, char* ws, const BlockLayout& L, fairy2i_wl_layer* out) {
  const int64_t n = d->n, f = d->n_ff;
  int cnt = 0;
  for (int s = 0; s < 3; ++s) {
    const int p = kGroupLayers[gi][s];
    if (p < 0) continue;
    fairy2i_wl_layer l{};
    l.codes_U = d->codes_U[p];
    l.scales_U = d->scales_U[p];
    l.codes_W = d->codes_W[p];
    l.scales_W = d->scales_W[p];
    l.layout = FAIRY2I_LAYOUT_TILED_FP4;
    l.N = (p == 4 || p == 5) ? f : n;
    l.K = (p == 6) ? f : n;
    size_t xoff = 0, yoff = 0;
    switch (p) {
      case 0: xoff = L.z; yoff = L.q; break;
      case 1: xoff = L.z; yoff = L.k; break;
      case 2: xoff = L.z; yoff = L.v; break;
      case 3: xoff = L.o; yoff = L.a; break;
      case 4: xoff = L.z2; yoff = L.g; break;
      case 5: xoff = L.z2; yoff = L.u; break;
      default: xoff = L.act; yoff = L.d; break;
    }
    // placeholders keep the shape checks of the layout pass happy
    l.x = ws ? (const void*)(ws + xoff) : (const void*)d;
    l.y = ws ? reinterpret_cast<float*>(ws + yoff) : reinterpret_cast<float*>(const_cast<fairy2i_block_desc*>(d));
    out[cnt++] = l;
  }
  return cnt;
}

// Workspace layout; the group workspaces need the group shapes only.
bool block_layout(const fairy2i_block_desc* d, BlockLayout& L) {
  const size_t n = (size_t)d->n, f = (size_t)d->n_ff;
  const size_t H = (size_t)d->n_heads, dc = n / H;
  const size_t slices = ((size_t)d->max_ctx + kAttnRun - 1) / kAttnRun;
  size_t o = 0;
  auto take = [&](size_t bytes) { const size_t at = o; o += align256(bytes); return at; };
  L.z = take(n * 4);
  L.q = take(n * 8);
  L.k = take(n * 8);
  L.v = take(n * 8);
  L.q_rot = take(n * 8);
  L.part = take(H * slices * (2 + 2 * dc) * 8);
  L.o = take(n * 4);
  L.a = take(n * 8);
  L.h1 = take(n * 8);
  L.z2 = take(n * 4);
  L.g = take(f * 8);
  L.u = take(f * 8);
  L.act = take(f * 4);
  L.d = take(n * 8);
  for (int gi = 0; gi < kGroups; ++gi) {
    fairy2i_wl_layer ls[3];
    const int cnt = group_layers(d, gi, nullptr, L, ls);
    const size_t b = fairy2i_wl_group_workspace_bytes(ls, cnt, d->T, FAIRY2I_ACT_BF16, 1);
    if (b == 0) return false;
    L.groups[gi] = take(b);
  }
  L.total = o;
  return true;
}

inline fairy2i_status hip_st(hipError_t e) { return e == hipSuccess ? FAIRY2I_OK : FAIRY2I_ERR_HIP; }

// Positions a block takes: 64 while the heads' blocks are resident at once (four
// a CU, three of wide heads), at longer contexts what that many blocks walk, in
// whole steps; at most 256 runs a head, whose merge is one block's.
template <int R>
int attn_run(int64_t n_ctx, int H) {
  constexpr int kResident = 256 * (R == 1 ? 4 : 3);
  const int64_t most = H >= kResident ? 1 : kResident / H < 256 ? kResident / H : 256;
  const int64_t run = (n_ctx + most - 1) / most;
  return run <= kAttnRun ? kAttnRun : (int)((run + 15) / 16 * 16);
}

template <int R>
void launch_attention(const BlockPlanHeader* hdr, const float2* kc, const float2* vc, int64_t pos, hipStream_t s) {
  const int H = hdr->n_heads, dc = (int)hdr->n / H, n_ctx = (int)pos + 1;
  const int run = attn_run<R>(n_ctx, H), runs = (n_ctx + run - 1) / run;
  hipLaunchKernelGGL(attn_partial_kernel<R>, dim3(runs, H), dim3(kAttnThreads), 0, s, hdr->q_rot, kc, vc, dc, n_ctx,
                     hdr->max_ctx, run, 1.0 / sqrt((double)(2 * dc)), hdr->part);
  hipLaunchKernelGGL(attn_combine_kernel<R>, dim3(H), dim3(kAttnThreads), sizeof(double) * (size_t)runs, s, hdr->part,
                     runs, dc, reinterpret_cast<uint32_t*>(hdr->o));
}

void launch_attention(const BlockPlanHeader* hdr, const float2* kc, const float2* vc, int64_t pos, hipStream_t s) {
  const int dc = (int)hdr->n / hdr->n_heads;
  if (dc <= 64) launch_attention<1>(hdr, kc, vc, pos, s);
  else if (dc <= 128) launch_attention<2>(hdr, kc, vc, pos, s);
  else launch_attention<4>(hdr, kc, vc, pos, s);
}

// The fused path: six launches.
fairy2i_status block_decode_fused(const void* plan, const void* plan_device, const float2* xin, float2* kc,
                                  float2* vc, int64_t pos, float2* out, hipStream_t s) {
  const auto* hdr = static_cast<const BlockPlanHeader*>(plan);
  auto args = [&](int gi) {
    const auto* gt = reinterpret_cast<const GroupTableHeader*>(static_cast<const char*>(plan) + hdr->table_off[gi]);
    const auto* l = reinterpret_cast<const DecLayer*>(gt + 1);
    SplitArgs a{};
    a.K = l[0].K;
    a.nk4 = l[0].nk4;
    a.N = l[0].N;
    a.code_bytes = (uint32_t)((size_t)hdr->T * (size_t)l[0].nrb * (size_t)l[0].nk4 * 1024);
    for (int i = 0; i < gt->h.n_layers; ++i) {
      a.m[i].codes[0] = l[i].codes[0];
      a.m[i].codes[1] = l[i].codes[1];
      a.m[i].scales[0] = l[i].scales[0];
      a.m[i].scales[1] = l[i].scales[1];
      a.m[i].y = l[i].y;
    }
    return a;
  };
  SplitArgs a = args(0);
  a.x = xin;
  a.gamma = hdr->norm_attn;
  a.eps = hdr->eps;
  a.z_out = reinterpret_cast<uint32_t*>(hdr->z);
  a.theta = reinterpret_cast<const double*>(static_cast<const char*>(plan_device) + hdr->theta_off);
  a.pos = pos;
  a.max_ctx = hdr->max_ctx;
  a.dc = (int)(hdr->n / hdr->n_heads);
  a.q_rot = hdr->q_rot;
  a.k_cache = kc;
  a.v_cache = vc;
  launch_block_product<kSrcNorm, kOutRope>(a, hdr->T, s);
  launch_attention(hdr, kc, vc, pos, s);
  a = args(1);
  a.tok = reinterpret_cast<const uint32_t*>(hdr->o);
  a.base = xin;
  a.sum = hdr->h1;
  launch_block_product<kSrcBf16, kOutAdd>(a, hdr->T, s);
  a = args(2);
  a.x = hdr->h1;
  a.gamma = hdr->norm_mlp;
  a.eps = hdr->eps;
  a.z_out = reinterpret_cast<uint32_t*>(hdr->z2);
  a.act = reinterpret_cast<uint32_t*>(hdr->act);
  launch_block_product<kSrcNorm, kOutSwiglu>(a, hdr->T, s);
  a = args(3);
  a.tok = reinterpret_cast<const uint32_t*>(hdr->act);
  a.base = hdr->h1;
  a.sum = out;
  launch_block_product<kSrcBf16, kOutAdd>(a, hdr->T, s);
  return hip_st(hipGetLastError());
}

}  // namespace

}  // namespace fairy2i

using namespace fairy2i;

extern "C" {

size_t fairy2i_block_workspace_bytes(const fairy2i_block_desc* desc) {
  if (!block_desc_ok(desc)) return 0;
  BlockLayout L;
  return block_layout(desc, L) ? L.total : 0;
}

size_t fairy2i_block_plan_bytes(const fairy2i_block_desc* desc) {
  if (!block_desc_ok(desc)) return 0;
  size_t total = align256(sizeof(BlockPlanHeader)) + align256(sizeof(double) * (size_t)(desc->n / desc->n_heads));
  for (int gi = 0; gi < kGroups; ++gi) total += align256(fairy2i_wl_group_table_bytes(gi == 0 ? 3 : (gi == 2 ? 2 : 1)));
  return total;
}

fairy2i_status fairy2i_block_build_plan(const fairy2i_block_desc* desc, void* workspace, size_t workspace_bytes,
                                        void* plan, size_t plan_bytes) {
  if (!desc || !workspace || !plan) return FAIRY2I_ERR_NULL;
  if (!block_desc_ok(desc)) return FAIRY2I_ERR_SHAPE;
  for (int p = 0; p < 7; ++p)
    if (!desc->codes_U[p] || !desc->codes_W[p] || !desc->scales_U[p] || !desc->scales_W[p]) return FAIRY2I_ERR_NULL;
  if (!desc->norm_attn || !desc->norm_mlp) return FAIRY2I_ERR_NULL;
  BlockLayout L;
  if (!block_layout(desc, L)) return FAIRY2I_ERR_UNSUPPORTED;
  if (workspace_bytes < L.total) return FAIRY2I_ERR_WORKSPACE;
  if (plan_bytes < fairy2i_block_plan_bytes(desc)) return FAIRY2I_ERR_WORKSPACE;
  char* ws = static_cast<char*>(workspace);
  char* pl = static_cast<char*>(plan);
  auto* hdr = reinterpret_cast<BlockPlanHeader*>(pl);
  memset(hdr, 0, sizeof(BlockPlanHeader));
  hdr->magic = kBlockMagic;
  hdr->abi = (uint32_t)fairy2i_abi_version();
  hdr->n = desc->n;
  hdr->n_ff = desc->n_ff;
  hdr->max_ctx = desc->max_ctx;
  hdr->n_heads = desc->n_heads;
  hdr->T = desc->T;
  hdr->eps = desc->eps;
  hdr->rope_base = desc->rope_base;
  hdr->norm_attn = desc->norm_attn;
  hdr->norm_mlp = desc->norm_mlp;
  hdr->z = reinterpret_cast<uint16_t*>(ws + L.z);
  hdr->q = reinterpret_cast<float2*>(ws + L.q);
  hdr->k = reinterpret_cast<float2*>(ws + L.k);
  hdr->v = reinterpret_cast<float2*>(ws + L.v);
  hdr->q_rot = reinterpret_cast<float2*>(ws + L.q_rot);
  hdr->part = reinterpret_cast<double2*>(ws + L.part);
  hdr->o = reinterpret_cast<uint16_t*>(ws + L.o);
  hdr->a = reinterpret_cast<float2*>(ws + L.a);
  hdr->h1 = reinterpret_cast<float2*>(ws + L.h1);
  hdr->z2 = reinterpret_cast<uint16_t*>(ws + L.z2);
  hdr->g = reinterpret_cast<float2*>(ws + L.g);
  hdr->u = reinterpret_cast<float2*>(ws + L.u);
  hdr->act = reinterpret_cast<uint16_t*>(ws + L.act);
  hdr->d = reinterpret_cast<float2*>(ws + L.d);
  size_t off = align256(sizeof(BlockPlanHeader));
  hdr->theta_off = off;
  const int64_t dc = desc->n / desc->n_heads;
  for (int64_t j = 0; j < dc; ++j)
    reinterpret_cast<double*>(pl + off)[j] = pow(desc->rope_base, -2.0 * (double)j / (double)(2 * dc));
  off += align256(sizeof(double) * (size_t)dc);
  for (int gi = 0; gi < kGroups; ++gi) {
    fairy2i_wl_layer ls[3];
    const int cnt = group_layers(desc, gi, ws, L, ls);
    const size_t tb = fairy2i_wl_group_table_bytes(cnt);
    const size_t gws = fairy2i_wl_group_workspace_bytes(ls, cnt, desc->T, FAIRY2I_ACT_BF16, 1);
    const fairy2i_status st = fairy2i_wl_group_build_table(ls, cnt, desc->T, FAIRY2I_ACT_BF16, 1, ws + L.groups[gi],
                                                           gws, pl + off, tb);
    if (st != FAIRY2I_OK) return st;
    hdr->table_off[gi] = off;
    hdr->table_bytes[gi] = tb;
    off += align256(tb);
  }
  hdr->fused = desc->n <= kSplitMaxK && desc->n_ff <= kSplitMaxK;
  for (int gi = 0; gi < kGroups; ++gi) {
    const DecHeader& h = reinterpret_cast<const GroupTableHeader*>(pl + hdr->table_off[gi])->h;
    if (h.mode != kModeBf16F4 || h.B != 1 || h.bands != 2 || h.nc != 8 || h.ntile != 1) hdr->fused = 0;
  }
  return FAIRY2I_OK;
}

fairy2i_status fairy2i_block_intermediates(const void* plan, void** ptrs) {
  if (!plan || !ptrs) return FAIRY2I_ERR_NULL;
  const auto* hdr = static_cast<const BlockPlanHeader*>(plan);
  if (hdr->magic != kBlockMagic || hdr->abi != (uint32_t)fairy2i_abi_version()) return FAIRY2I_ERR_UNSUPPORTED;
  void* const p[12] = {hdr->z, hdr->q_rot, hdr->v, hdr->o, hdr->a, hdr->h1,
                       hdr->z2, hdr->g, hdr->u, hdr->act, hdr->d, hdr->k};
  for (int i = 0; i < 12; ++i) ptrs[i] = p[i];
  return FAIRY2I_OK;
}

fairy2i_status fairy2i_block_decode(const void* plan, const void* plan_device, const float* x, float* k_cache,
                                    float* v_cache, int64_t pos, float* out, void* stream) {
  if (!plan || !plan_device || !x || !k_cache || !v_cache || !out) return FAIRY2I_ERR_NULL;
  const auto* hdr = static_cast<const BlockPlanHeader*>(plan);
  if (hdr->magic != kBlockMagic || hdr->abi != (uint32_t)fairy2i_abi_version()) return FAIRY2I_ERR_UNSUPPORTED;
  if (pos < 0 || pos >= hdr->max_ctx) return FAIRY2I_ERR_SHAPE;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int n = (int)hdr->n, f = (int)hdr->n_ff, dc = n / hdr->n_heads;
  auto group = [&](int gi) -> fairy2i_status {
    return fairy2i_wl_matmul_group(static_cast<const char*>(plan) + hdr->table_off[gi],
                                   static_cast<const char*>(plan_device) + hdr->table_off[gi], stream);
  };
  const float2* xin = reinterpret_cast<const float2*>(x);
  float2* kc = reinterpret_cast<float2*>(k_cache);
  float2* vc = reinterpret_cast<float2*>(v_cache);
  hipError_t e;
  fairy2i_status st;
  if (hdr->fused) return block_decode_fused(plan, plan_device, xin, kc, vc, pos, reinterpret_cast<float2*>(out), s);
  hipLaunchKernelGGL(add_rmsnorm_kernel, dim3(1), dim3(kNormThreads), 0, s, xin, nullptr, nullptr, hdr->norm_attn,
                     hdr->eps, n, hdr->z);
  if ((e = hipGetLastError()) != hipSuccess) return hip_st(e);
  if ((st = group(0)) != FAIRY2I_OK) return st;
  hipLaunchKernelGGL(rope_append_kernel, dim3((n + 255) / 256), dim3(256), 0, s, hdr->q, hdr->k, hdr->v, n, dc, pos,
                     hdr->max_ctx, hdr->rope_base, hdr->q_rot, kc, vc);
  launch_attention(hdr, kc, vc, pos, s);
  if ((e = hipGetLastError()) != hipSuccess) return hip_st(e);
  if ((st = group(1)) != FAIRY2I_OK) return st;
  hipLaunchKernelGGL(add_rmsnorm_kernel, dim3(1), dim3(kNormThreads), 0, s, xin, hdr->a, hdr->h1, hdr->norm_mlp,
                     hdr->eps, n, hdr->z2);
  if ((e = hipGetLastError()) != hipSuccess) return hip_st(e);
  if ((st = group(2)) != FAIRY2I_OK) return st;
  hipLaunchKernelGGL(swiglu_kernel, dim3((f + 255) / 256), dim3(256), 0, s, hdr->g, hdr->u, f, hdr->act);
  if ((e = hipGetLastError()) != hipSuccess) return hip_st(e);
  if ((st = group(3)) != FAIRY2I_OK) return st;
  hipLaunchKernelGGL(add_kernel, dim3((n + 255) / 256), dim3(256), 0, s, hdr->h1, hdr->d, n,
                     reinterpret_cast<float2*>(out));
  return hip_st(hipGetLastError());
}

}  // extern "C"
