// Product of one layer on the int8 matrix cores for small token counts, in
// one launch, from the canonical packed codes (K % 64 == 0): int8 activations
// of up to a few hundred tokens, bf16 activations of up to 16.  Sec. 3.4 /
// Algorithm 1 with the dequantisation of Eq. (ifairy-dequant) and the
// W conj(x) term of Eq. (widely-linear).
//
// What bounds it is latency, not bytes or operations: a 2048 x 5504 layer is
// 11 MB of codes, 2 us at the HBM's rate, but a wave that walks K alone waits
// for memory dozens of times, and every launch around the product (an operand
// kernel before it, a reduction of K slices after it) costs 4-5 us.  So
//   * a block owns 16 rows and a few tokens, and its kWaves waves split K in
//     steps of 256 codes (wave w takes steps w, w + kWaves, ...); their shares
//     of y meet in LDS, in double and in wave order, so nothing is left for a
//     second kernel and y is rounded once;
//   * the activations are read as the caller has them: a lane splits the 16
//     (re, im) int8 pairs of its token into the two operands by byte
//     permutes, or turns 16 bf16 values into their three base-256 digits
//     (the block first finds its tokens' largest magnitudes).
// Measured, T = 2, one call, before (operand kernel, product, reduction of K
// slices; above 16 tokens the prefill GEMM and its operand kernel) and now:
//   2048 x 2048   bf16 1 token 15.3 -> 6.8 us, 16 tokens 32.6 -> 16.1 us;
//                 int8 1 token 13.3 -> 5.7, 16 tokens 21.0 -> 5.8, 64 20.5 -> 8.9
//   2048 x 5504   bf16 1 token 22.3 -> 11.0, 16 tokens 49.5 -> 30.2;
//                 int8 1 token 17.9 -> 10.5, 16 tokens 32.0 -> 10.7, 80 45.0 -> 24.3
//   5504 x 5504   int8 16 tokens 39.7 -> 17.3, 64 tokens 46.1 -> 44.4
// Many rows, long K and (T = 4) int8 layers of more blocks than CUs stay with
// the other kernels: one_launch_pays (api.hip).
//
// Products and recombination are those of the grouped int8 path: each code
// word of 16 codes expands in registers into the b_re and b_im int8 planes,
// v_mfma_i32_16x16x64_i8 sums them exactly, and the axis scales, the factor
// i, the conjugation of the W term and the token's factor are applied in
// double.
#include "common.h"
#include "decode_dev.h"

namespace fairy2i {

namespace {

constexpr uint32_t kTableRe = 0x00FF0001u;  // code 0 -> +1, 1 -> 0, 2 -> -1, 3 -> 0
constexpr uint32_t kTableIm = 0xFF000100u;  // code 0 -> 0, 1 -> +1, 2 -> 0, 3 -> -1

__device__ inline uint32_t perm(uint32_t hi, uint32_t lo, uint32_t sel) { return __builtin_amdgcn_perm(hi, lo, sel); }

// 16 codes -> the b_re and b_im planes; byte 4c + b holds code c + 4b.
__device__ inline void expand_codes(uint32_t w, v4i& bre, v4i& bim) {
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const uint32_t sel = (w >> (2 * c)) & 0x03030303u;
    bre[c] = (int)perm(0u, kTableRe, sel);
    bim[c] = (int)perm(0u, kTableIm, sel);
  }
}

// 16 interleaved (re, im) int8 pairs -> 16 re and 16 im bytes in the order
// the expanded codes use.
__device__ inline void split_pairs(const v4i a, const v4i b, v4i& re, v4i& im) {
  const uint32_t r02 = perm(a[2], a[0], 0x06020400u), r13 = perm(a[3], a[1], 0x06020400u);
  const uint32_t r46 = perm(b[2], b[0], 0x06020400u), r57 = perm(b[3], b[1], 0x06020400u);
  const uint32_t i02 = perm(a[2], a[0], 0x07030501u), i13 = perm(a[3], a[1], 0x07030501u);
  const uint32_t i46 = perm(b[2], b[0], 0x07030501u), i57 = perm(b[3], b[1], 0x07030501u);
  re = v4i{(int)perm(r46, r02, 0x05040100u), (int)perm(r46, r02, 0x07060302u), (int)perm(r57, r13, 0x05040100u),
           (int)perm(r57, r13, 0x07060302u)};
  im = v4i{(int)perm(i46, i02, 0x05040100u), (int)perm(i46, i02, 0x07060302u), (int)perm(i57, i13, 0x05040100u),
           (int)perm(i57, i13, 0x07060302u)};
}

// One wave's code loads: 16 bytes (64 codes) per lane and plane of step s;
// lane (g, li) holds codes 256 s + 64 g .. + 63 of row li of the block.
template <int T>
struct CodeLoader {
  __amdgpu_buffer_rsrc_t plane[2 * T];
  uint32_t base;
  int K, g;
  bool row_ok;
  __device__ CodeLoader(const WlArgs& a, int64_t row, int lane) {
    const uint32_t bytes = (uint32_t)(a.N * a.K / 4);
#pragma unroll
    for (int p = 0; p < 2 * T; ++p) plane[p] = make_rsrc(a.codes[p / T] + (int64_t)(p % T) * bytes, bytes);
    g = lane >> 4;
    K = (int)a.K;
    row_ok = row < a.N;
    base = (uint32_t)(row * (a.K / 4)) + 16u * (uint32_t)g;
  }
  __device__ void load(int s, v4i (&c)[2 * T]) const {
    const uint32_t off = row_ok && 256 * s + 64 * g < K ? base + 64u * (uint32_t)s : kOob;
#pragma unroll
    for (int p = 0; p < 2 * T; ++p) c[p] = buf_load16(plane[p], off);
  }
};

// ---------------------------------------------------------------- int8 ---
// A = codes (rows), B = activations: 16 tokens a block, their re and im parts
// two operands; acc lane (g, li) holds rows 4g .. 4g+3 of token li.
//
// A step's activations are 16 rows of 512 bytes.  A wave fetches them into
// its own LDS area two rows a load (a load of the operand's own layout, 16
// bytes of every row and lane group, touches 64 cache lines; these touch 8)
// and reads 32 bytes a lane and MFMA back.  Row t's 16-byte chunk c sits at
// chunk c ^ t of the row, so that the 16 rows' chunks a lane group reads
// together lie in different banks.
constexpr int kXBytes = 16 * 512;

template <int T, int kWaves>
__global__ __launch_bounds__(64 * kWaves, T <= 3 || kWaves > 4 ? 2 : 1) void split_i8_kernel(WlArgs a, bool vec) {
#if defined(__HIP_DEVICE_COMPILE__)  // buffer-descriptor and LDS-DMA code: device pass only
  constexpr int P = 2 * T;
  constexpr int kPartBytes = kWaves * 16 * 17 * (int)sizeof(double2), kRingBytes = kWaves * 2 * kXBytes;
  // the waves' activation buffers; after the last step their shares of y
  __shared__ __attribute__((aligned(16))) uint8_t lds[kPartBytes > kRingBytes ? kPartBytes : kRingBytes];
  const int lane = threadIdx.x & 63, g = lane >> 4, li = lane & 15;
  const int wave = uniform(threadIdx.x >> 6);
  const int64_t row0 = (int64_t)blockIdx.x * 16, tok0 = (int64_t)blockIdx.y * 16;
  const int K = (int)a.K, steps = (K + 255) / 256;
  const CodeLoader<T> codes(a, row0 + li, lane);
  const int ntok = (int)(a.B - tok0 < 16 ? a.B - tok0 : 16);
  const int8_t* q = static_cast<const int8_t*>(a.x) + tok0 * K * 2;
  const __amdgpu_buffer_rsrc_t qr = make_rsrc(q, (uint32_t)(ntok * K * 2));  // K <= 2^24: below 2^31
  uint8_t* buf0 = lds + wave * 2 * kXBytes;

  // Activations of step s into LDS: load i brings rows 2i and 2i + 1, half a
  // wave each; codes past K and rows past the last token read as zero.
  auto load_x = [&](int s, int b) {
    uint8_t* dst = buf0 + b * kXBytes;
    auto source = [&](int i) -> uint32_t {
      const int t = 2 * i + (lane >> 5), chunk = (lane & 31) ^ t;
      const bool ok = t < ntok && 256 * s + 8 * chunk < K;  // a chunk is 8 codes
      return ok ? (uint32_t)(t * K + 256 * s) * 2u + 16u * (uint32_t)chunk : kOob;
    };
    if (vec) {
#pragma unroll
      for (int i = 0; i < 8; ++i)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(qr, (lds_ptr_t)(dst + i * 1024), 16, source(i), 0, 0, 0);
    } else {
#pragma unroll 1
      for (int i = 0; i < 8; ++i) {
        const uint32_t off = source(i);
        uint32_t w[4] = {0u, 0u, 0u, 0u};
        if (off != kOob)
#pragma unroll
          for (int e = 0; e < 16; ++e) w[e >> 2] |= (uint32_t)(uint8_t)q[off + e] << (8 * (e & 3));
        *reinterpret_cast<uint4*>(dst + i * 1024 + lane * 16) = make_uint4(w[0], w[1], w[2], w[3]);
      }
    }
  };

  v4i acc[P][2][2];
#pragma unroll
  for (int p = 0; p < P; ++p)
#pragma unroll
    for (int ax = 0; ax < 2; ++ax) acc[p][ax][0] = acc[p][ax][1] = v4i{0, 0, 0, 0};
  v4i c[P];
  if (wave < steps) {
    codes.load(wave, c);
    load_x(wave, 0);
  }
  int b = 0;
  for (int s = wave; s < steps; s += kWaves) {
    __builtin_amdgcn_s_waitcnt(0);  // this step's codes and activations
    __builtin_amdgcn_wave_barrier();
    v4i cn[P];
    const bool more = s + kWaves < steps;
    if (more) {
      codes.load(s + kWaves, cn);
      load_x(s + kWaves, b ^ 1);
    }
    const uint32_t row = lds_addr(buf0 + b * kXBytes) + (uint32_t)li * 512u;
#pragma unroll
    for (int dd = 0; dd < 2; ++dd) {
      // chunks 8 g + 2 d, + 1 for d = 2 dd, 2 dd + 1
      v4i x[4];
      lds_read4(row + 16u * (uint32_t)((8 * g + 4 * dd) ^ li), row + 16u * (uint32_t)((8 * g + 4 * dd + 1) ^ li),
                row + 16u * (uint32_t)((8 * g + 4 * dd + 2) ^ li), row + 16u * (uint32_t)((8 * g + 4 * dd + 3) ^ li), x);
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        v4i xr, xi;
        split_pairs(x[2 * h], x[2 * h + 1], xr, xi);
#pragma unroll
        for (int p = 0; p < P; ++p) {
          v4i bre, bim;
          expand_codes((uint32_t)c[p][2 * dd + h], bre, bim);
          acc[p][0][0] = __builtin_amdgcn_mfma_i32_16x16x64_i8(bre, xr, acc[p][0][0], 0, 0, 0);
          acc[p][0][1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(bre, xi, acc[p][0][1], 0, 0, 0);
          acc[p][1][0] = __builtin_amdgcn_mfma_i32_16x16x64_i8(bim, xr, acc[p][1][0], 0, 0, 0);
          acc[p][1][1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(bim, xi, acc[p][1][1], 0, 0, 0);
        }
      }
    }
    if (more) {
#pragma unroll
      for (int p = 0; p < P; ++p) c[p] = cn[p];
    }
    b ^= 1;
  }

  // 17: the sums below read a token's rows, the stores here a row's tokens
  auto* part = reinterpret_cast<double2(*)[16][17]>(lds);
  float sc[2][T][2];
  sload_scales<T>(a.scales[0], a.scales[1], sc);
  __syncthreads();  // every wave is done with its activations
  if (wave < steps) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      double yr = 0.0, yi = 0.0;
#pragma unroll
      for (int t = 0; t < T; ++t) {
        const double su_re = sc[0][t][0], su_im = sc[0][t][1], sw_re = sc[1][t][0], sw_im = sc[1][t][1];
        const int pu = t, pw = T + t;
        yr += su_re * (double)acc[pu][0][0][r] - su_im * (double)acc[pu][1][1][r];
        yi += su_re * (double)acc[pu][0][1][r] + su_im * (double)acc[pu][1][0][r];
        yr += sw_re * (double)acc[pw][0][0][r] + sw_im * (double)acc[pw][1][1][r];
        yi += -sw_re * (double)acc[pw][0][1][r] + sw_im * (double)acc[pw][1][0][r];
      }
      part[wave][li][4 * g + r] = make_double2(yr, yi);
    }
  }
  __syncthreads();
  const int active = steps < kWaves ? steps : kWaves;
  for (int o = threadIdx.x; o < 256; o += 64 * kWaves) {
    const int t = o >> 4, r = o & 15;
    const int64_t tok = tok0 + t, row = row0 + r;
    if (tok >= a.B || row >= a.N) continue;
    double yr = 0.0, yi = 0.0;
    for (int w = 0; w < active; ++w) {
      yr += part[w][t][r].x;
      yi += part[w][t][r].y;
    }
    const double s = (double)a.x_scale[tok];
    a.y[tok * a.N + row] = make_float2((float)(yr * s), (float)(yi * s));
  }
#endif
}

// ---------------------------------------------------------------- bf16 ---
// A = activations: two tokens a block (more tokens a block, whose codes would
// expand once for all, measured no faster), 8 columns each (digit 0 re, im,
// digit 1 re, im, digit 2 re, im, two unused), B = codes (rows); acc lane
// (g, li) holds columns 4g .. 4g+3 of row li: digits 0 and 1 of token g / 2
// where g is even, digit 2 where it is odd.
template <int T, int kWaves>
__global__ __launch_bounds__(64 * kWaves) void split_bf16_kernel(WlArgs a, bool vec) {
#if defined(__HIP_DEVICE_COMPILE__)
  constexpr int P = 2 * T;
  __shared__ float tok_max[2][kWaves];
  // a step's operand: [d][g][column][16 bytes]; columns 6, 7, 14, 15 stay zero
  __shared__ __attribute__((aligned(16))) uint4 xop[kWaves][4][4][16];
  __shared__ double2 part[kWaves][2][17];
  const int lane = threadIdx.x & 63, g = lane >> 4, li = lane & 15;
  const int wave = uniform(threadIdx.x >> 6);
  const int64_t row0 = (int64_t)blockIdx.x * 16, tok0 = (int64_t)blockIdx.y * (2);
  const int K = (int)a.K, steps = (K + 255) / 256;
  const CodeLoader<T> codes(a, row0 + li, lane);
  v4i c[P];
  if (wave < steps) codes.load(wave, c);  // in flight while the tokens' magnitudes are found

  const uint16_t* x = static_cast<const uint16_t*>(a.x);
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    float m = 0.0f;
    if (tok0 + s < a.B) {
      const uint16_t* xb = x + (tok0 + s) * K * 2;
      if (vec) {
        const uint4* xv = reinterpret_cast<const uint4*>(xb);
        for (int i = threadIdx.x; i < K / 4; i += 64 * kWaves) {  // 8 bf16 (4 complex) per vector
          const uint4 w = xv[i];
          const uint32_t wd[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
          for (int j = 0; j < 4; ++j)
            m = fmaxf(m, fmaxf(fabsf(__uint_as_float(wd[j] << 16)), fabsf(__uint_as_float(wd[j] & 0xFFFF0000u))));
        }
      } else {
        for (int i = threadIdx.x; i < 2 * K; i += 64 * kWaves)
          m = fmaxf(m, fabsf(__uint_as_float((uint32_t)xb[i] << 16)));
      }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
    if (lane == 0) tok_max[s][wave] = m;
  }
  for (int i = lane; i < 256; i += 64) (&xop[wave][0][0][0])[i] = make_uint4(0u, 0u, 0u, 0u);
  __syncthreads();
  // fixed point of each token: X = rint(x 2^E), E from its largest magnitude
  int E[2];
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    float m = tok_max[s][0];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) m = fmaxf(m, tok_max[s][w]);
    // m in [2^(ex-1), 2^ex); m * 2^e in [2^21, 2^22): 3 base-256 digits;
    // e <= 149 keeps 2^-e representable in float32
    const int ex = __builtin_amdgcn_frexp_expf(m);
    E[s] = m > 0.0f ? (22 - ex < 149 ? 22 - ex : 149) : 0;
  }

  v4i acc[P][2];
#pragma unroll
  for (int p = 0; p < P; ++p) acc[p][0] = acc[p][1] = v4i{0, 0, 0, 0};

  for (int s = wave; s < steps; s += kWaves) {
    // this wave's operand of the step: a lane turns 16 values of one token
    // and component into their three digits (run = 4 d + g of the step)
    const int comp = lane & 1, run = (lane >> 1) & 15;
    const int rd = run >> 2, rg = run & 3;
    const int k0 = 256 * s + 64 * rg + 16 * rd;
    const int sl = lane >> 5;  // token of the block
    const int64_t tok = tok0 + sl;
    if (tok < a.B) {
      uint32_t dig[3][4] = {};
      if (k0 < K) {
        int v[16];
        load_run16<kModeBf16>(a.x, vec, (tok * K + k0) * 2, comp, v);
        const int e2 = sl ? E[1] : E[0];
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int dd = e >> 2, bb = e & 3;  // byte 4dd+bb holds code dd + 4bb of the run
          const int X = (int)rintf(ldexpf(__uint_as_float((uint32_t)v[dd + 4 * bb] << 16), e2));
          const int d0 = ((X + 128) & 255) - 128;
          const int X1 = (X - d0) >> 8;
          const int d1 = ((X1 + 128) & 255) - 128;
          const int d2 = (X1 - d1) >> 8;
          dig[0][dd] |= ((uint32_t)d0 & 0xFFu) << (8 * bb);
          dig[1][dd] |= ((uint32_t)d1 & 0xFFu) << (8 * bb);
          dig[2][dd] |= ((uint32_t)d2 & 0xFFu) << (8 * bb);
        }
      }
#pragma unroll
      for (int i = 0; i < 3; ++i)
        xop[wave][rd][rg][8 * sl + 2 * i + comp] = make_uint4(dig[i][0], dig[i][1], dig[i][2], dig[i][3]);
    }
    v4i cn[P];
    const bool more = s + kWaves < steps;
    if (more) codes.load(s + kWaves, cn);
    wave_sync();  // the wave's operand: written above, read below
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      const v4i xa = *reinterpret_cast<const v4i*>(&xop[wave][d][g][li]);
#pragma unroll
      for (int p = 0; p < P; ++p) {
        v4i bre, bim;
        expand_codes((uint32_t)c[p][d], bre, bim);
        acc[p][0] = __builtin_amdgcn_mfma_i32_16x16x64_i8(xa, bre, acc[p][0], 0, 0, 0);
        acc[p][1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(xa, bim, acc[p][1], 0, 0, 0);
      }
    }
    wave_sync();
    if (more) {
#pragma unroll
      for (int p = 0; p < P; ++p) c[p] = cn[p];
    }
  }

  float sc[2][T][2];
  sload_scales<T>(a.scales[0], a.scales[1], sc);
  {
    double yr = 0.0, yi = 0.0;
    // exact in double for any K <= 2^24; digit 2 is the next lane group's
    auto product = [&](int p, int ax, int comp) -> double {
      const int hi = __shfl_down(acc[p][ax][comp], 16);
      return (double)acc[p][ax][comp] + 256.0 * (double)acc[p][ax][2 + comp] + 65536.0 * (double)hi;
    };
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const double su_re = sc[0][t][0], su_im = sc[0][t][1], sw_re = sc[1][t][0], sw_im = sc[1][t][1];
      const double u00 = product(t, 0, 0), u01 = product(t, 0, 1), u10 = product(t, 1, 0), u11 = product(t, 1, 1);
      const double w00 = product(T + t, 0, 0), w01 = product(T + t, 0, 1);
      const double w10 = product(T + t, 1, 0), w11 = product(T + t, 1, 1);
      yr += su_re * u00 - su_im * u11;
      yi += su_re * u01 + su_im * u10;
      yr += sw_re * w00 + sw_im * w11;
      yi += -sw_re * w01 + sw_im * w10;
    }
    if (!(g & 1) && wave < steps) part[wave][g >> 1][li] = make_double2(yr, yi);
  }
  __syncthreads();
  const int active = steps < kWaves ? steps : kWaves;
  const int o = threadIdx.x;
  if (o < 32) {
    const int s = o >> 4, r = o & 15;
    const int64_t tok = tok0 + s, row = row0 + r;
    if (tok < a.B && row < a.N) {
      double yr = 0.0, yi = 0.0;
      for (int w = 0; w < active; ++w) {
        yr += part[w][s][r].x;
        yi += part[w][s][r].y;
      }
      float m = 0.0f;
      for (int w = 0; w < kWaves; ++w) m = fmaxf(m, tok_max[s][w]);
      const double f = m > 0.0f ? (double)ldexpf(1.0f, -(s ? E[1] : E[0])) : 0.0;
      a.y[tok * a.N + row] = make_float2((float)(yr * f), (float)(yi * f));
    }
  }
#endif
}

// Waves per block: four (two blocks on a CU hide each other's waits), eight
// where K is long and the blocks are too few for that.  2048 x 5504, T = 2,
// four against eight waves: int8 16 tokens (128 blocks) 11.3 / 10.6 us, 77
// tokens (640 blocks) 23.7 / 29.6 us; bf16 2 tokens (128) 14.0 / 11.8 us, 16
// tokens (1024) 30.2 / 33.8 us; K = 2048, one token, 5.8 / 6.0 and 6.8 / 7.2 us.
// (T = 4 int8 accumulators leave eight waves too few registers.)
bool eight_waves(const WlArgs& a, int64_t blocks, int64_t most) { return a.K > 2048 && blocks <= most; }

template <int T>
void launch_i8(const WlArgs& a, hipStream_t s) {
  const bool vec = (reinterpret_cast<uintptr_t>(a.x) & 15) == 0;
  const dim3 grid((unsigned)((a.N + 15) / 16), (unsigned)((a.B + 15) / 16));
  if constexpr (T <= 3) {
    if (eight_waves(a, (int64_t)grid.x * grid.y, 256)) {
      hipLaunchKernelGGL((split_i8_kernel<T, 8>), grid, dim3(512), 0, s, a, vec);
      return;
    }
  }
  hipLaunchKernelGGL((split_i8_kernel<T, 4>), grid, dim3(256), 0, s, a, vec);
}

template <int T>
void launch_bf16(const WlArgs& a, hipStream_t s) {
  const bool vec = (reinterpret_cast<uintptr_t>(a.x) & 15) == 0;
  const dim3 grid((unsigned)((a.N + 15) / 16), (unsigned)((a.B + 1) / 2));
  if (eight_waves(a, (int64_t)grid.x * grid.y, 512))
    hipLaunchKernelGGL((split_bf16_kernel<T, 8>), grid, dim3(512), 0, s, a, vec);
  else
    hipLaunchKernelGGL((split_bf16_kernel<T, 4>), grid, dim3(256), 0, s, a, vec);
}

}  // namespace

hipError_t launch_split(const WlArgs& a, hipStream_t s) {
  if (a.dtype == FAIRY2I_ACT_I8) {
    switch (a.T) {
      case 1: launch_i8<1>(a, s); break;
      case 2: launch_i8<2>(a, s); break;
      case 3: launch_i8<3>(a, s); break;
      default: launch_i8<4>(a, s); break;
    }
  } else {
    switch (a.T) {
      case 1: launch_bf16<1>(a, s); break;
      case 2: launch_bf16<2>(a, s); break;
      case 3: launch_bf16<3>(a, s); break;
      default: launch_bf16<4>(a, s); break;
    }
  }
  return hipGetLastError();
}

}  // namespace fairy2i
