// Grouped decode product of a few layers and up to four bf16 tokens on the
// fp8 x fp4 matrix cores, in one launch.  Sec. 3.4 / Algorithm 1 with the
// dequantisation of Eq. (ifairy-dequant) and the W conj(x) term of
// Eq. (widely-linear); the operands, products and recombination are those of
// the streaming kernel (fp4 tiled codes, two digit bands a token).
//
// What bounds a small group is latency: the q, k and v projections of one
// decoder block are 13 MB of codes, under 3 us at the rate of a large copy,
// but the operand kernel, the product over K slices and the reduction of the
// slices take 4 + 12 + 4 us.  Here a block owns 16 rows of a layer and its
// kWaves waves split K in 256-code steps (wave w takes steps w, w + kWaves,
// ...); their shares of y are recombined in double (in float one-step layers lost
// up to a fifth of their precision: 4.0e-8 -> 4.9e-8 of the result at K = 64,
// T = 1, now 2.7e-8), meet in LDS and are added in wave order, so y is rounded
// once.  A wave encodes the digits of its own steps from the tokens as the caller
// has them (a lane per half run and component), after the block has found the
// tokens' largest magnitudes; the layers come as kernel arguments, not from the
// table in memory, so that the first loads wait for nothing.
#include "common.h"
#include "decode_dev.h"
#include "f4_operand.h"

namespace fairy2i {

namespace {

constexpr int kWaves = 8;

struct SplitLayer {
  const uint8_t* codes[2];  // U, W
  const float* scales[2];
  const void* x;
  float2* y;
  int32_t N, K, nk4, gsteps, ngroups;
  uint32_t code_bytes, rb0;  // bytes of one matrix's codes; row blocks of the layers before
};

struct SplitGroup {
  SplitLayer l[kSplitLayers];
  int32_t n, B;
};

// TILES tiles of two tokens: wave w takes tile w % TILES and the K steps
// w / TILES, + kWaves / TILES, ... (one wave with both tiles' sums and tokens
// spills: the second tile's wave asks for the same codes and gets them from
// the cache).  GS: per-group scales.
template <int T, int TILES, bool GS>
__global__ __launch_bounds__(64 * kWaves, T <= 2 ? 4 : 2) void dec_split_f4_kernel(SplitGroup a) {
#if defined(__HIP_DEVICE_COMPILE__)  // buffer-descriptor code: device pass only
  constexpr int P = 2 * T, KW = kWaves / TILES;
  // a step's operand of one tile: [run][column][16 bytes]; the columns of a
  // token past the last stay zero
  __shared__ __attribute__((aligned(16))) uint8_t xop[kWaves][16 * 16 * 16];
  __shared__ float tok_max[2 * TILES][KW];
  __shared__ double2 part[KW][2 * TILES][17];
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, li = lane & 15;
  const int wave = uniform(tid >> 6), tile = wave % TILES, kw = wave / TILES;
  int idx = 0;
#pragma unroll
  for (int i = 1; i < kSplitLayers; ++i)
    if (i < a.n && blockIdx.x >= a.l[i].rb0) idx = i;
  idx = uniform(idx);
  const SplitLayer& L = a.l[idx];
  const int rb = (int)(blockIdx.x - L.rb0), K = L.K, N = L.N, nk4 = L.nk4, B = a.B;
  const int row = rb * 16 + li;

  const __amdgpu_buffer_rsrc_t ru = make_rsrc(uniform_ptr(L.codes[0]), L.code_bytes);
  const __amdgpu_buffer_rsrc_t rw = make_rsrc(uniform_ptr(L.codes[1]), L.code_bytes);
  const float* const su = uniform_ptr(L.scales[0]);
  const float* const sw = uniform_ptr(L.scales[1]);
  auto load = [&](int s, v4i(&c)[P]) {  // a step past the last reads zeros
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const uint32_t off = s < nk4 ? (uint32_t)((rb * nk4 + s) * T + t) * 1024u + 16u * (uint32_t)lane : kOob;
      c[t] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(ru, off, 0, kNonTemporal));
      c[T + t] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rw, off, 0, kNonTemporal));
    }
  };
  auto load_scales = [&](int s, float2(&gs)[GS ? P : 1]) {
    if constexpr (GS) {
#pragma unroll
      for (int p = 0; p < P; ++p) {
        gs[p] = make_float2(0.0f, 0.0f);
        if (row < N) {
          const int64_t at = (((int64_t)(p % T) * N + row) * L.ngroups + s / L.gsteps) * 2;
          const float* sp = (p < T ? su : sw) + at;
          gs[p] = make_float2(sp[0], sp[1]);
        }
      }
    }
  };
  // this lane's 8 (re, im) words of the tile's token sl in step s: half run lane / 2 (both
  // of its lanes load it and take a component each)
  const int hr = lane >> 1, comp = lane & 1;
  const uint16_t* const x = static_cast<const uint16_t*>(L.x);
  const bool vec = (reinterpret_cast<uintptr_t>(x) & 15) == 0;
  auto load_x = [&](int s, int sl, uint32_t(&w)[8]) {
    const int b = 2 * tile + sl;
#pragma unroll
    for (int e = 0; e < 8; ++e) w[e] = 0u;
    const int k0 = 256 * s + 8 * hr;
    if (b < B && k0 < K) {  // K % 64 == 0: the half run is in range or past K entirely
      const uint16_t* p = x + ((int64_t)b * K + k0) * 2;
      if (vec) {
        const uint4 v0 = reinterpret_cast<const uint4*>(p)[0], v1 = reinterpret_cast<const uint4*>(p)[1];
        w[0] = v0.x; w[1] = v0.y; w[2] = v0.z; w[3] = v0.w;
        w[4] = v1.x; w[5] = v1.y; w[6] = v1.z; w[7] = v1.w;
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) w[e] = (uint32_t)p[2 * e] | ((uint32_t)p[2 * e + 1] << 16);
      }
    }
  };
  auto largest = [](float m, const uint32_t(&w)[8]) {
#pragma unroll
    for (int e = 0; e < 8; ++e)
      m = fmaxf(m, fmaxf(fabsf(__uint_as_float(w[e] << 16)), fabsf(__uint_as_float(w[e] & 0xFFFF0000u))));
    return m;
  };

  // the first step's tokens stay in registers: K <= 256 KW is read once
  uint32_t xw[2][8];
#pragma unroll
  for (int sl = 0; sl < 2; ++sl) load_x(kw, sl, xw[sl]);
  v4i c[P];
  float2 gs[GS ? P : 1];
  load(kw, c);
  if (kw < nk4) load_scales(kw, gs);
  float sc[2][T][2];
  if constexpr (!GS) sload_scales<T>(su, sw, sc);
  float m[2];
#pragma unroll
  for (int sl = 0; sl < 2; ++sl) m[sl] = largest(0.0f, xw[sl]);
  for (int s = kw + KW; s < nk4; s += KW) {
    uint32_t w[2][8];
#pragma unroll
    for (int sl = 0; sl < 2; ++sl) load_x(s, sl, w[sl]);
#pragma unroll
    for (int sl = 0; sl < 2; ++sl) m[sl] = largest(m[sl], w[sl]);
  }
#pragma unroll
  for (int sl = 0; sl < 2; ++sl) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) m[sl] = fmaxf(m[sl], __shfl_xor(m[sl], off));
    if (lane == 0) tok_max[2 * tile + sl][kw] = m[sl];
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) reinterpret_cast<uint4*>(xop[wave])[lane + 64 * i] = make_uint4(0u, 0u, 0u, 0u);
  __syncthreads();
  int S[2];
#pragma unroll
  for (int sl = 0; sl < 2; ++sl) {
    float mb = tok_max[2 * tile + sl][0];
#pragma unroll
    for (int w = 1; w < KW; ++w) mb = fmaxf(mb, tok_max[2 * tile + sl][w]);
    S[sl] = f4_token_shift(mb);
  }

  // per-tensor scales: the products of all steps; per-group scales: those of
  // one step, folded into the scaled sums
  v4f aS[P], aI[P];
  float Are[GS ? P : 1][2], Aim[GS ? P : 1][2];
#pragma unroll
  for (int p = 0; p < P; ++p) {
    aS[p] = aI[p] = v4f{0.f, 0.f, 0.f, 0.f};
    if constexpr (GS) Are[p][0] = Are[p][1] = Aim[p][0] = Aim[p][1] = 0.0f;
  }
  for (int s = kw; s < nk4; s += KW) {
    v4i cn[P];
    if (s != kw) {
#pragma unroll
      for (int sl = 0; sl < 2; ++sl) load_x(s, sl, xw[sl]);
      load_scales(s, gs);
    }
    load(s + KW, cn);
#pragma unroll
    for (int sl = 0; sl < 2; ++sl)
      if (2 * tile + sl < B) {
        float xv[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) xv[e] = __uint_as_float(comp ? (xw[sl][e] & 0xFFFF0000u) : (xw[sl][e] << 16));
        uint32_t out[2][2][2];
        f4_unit_digits(xv, S[sl], 2, out);
        f4_store_unit(xop[wave], hr >> 1, 16, 8 * sl, comp, hr & 1, 2, out);
      }
    wave_sync();  // the wave's operand: written above, read below
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
      const v4i y0 = *reinterpret_cast<const v4i*>(&xop[wave][((8 * kb + g) * 16 + li) * 16]);
      const v4i y1 = *reinterpret_cast<const v4i*>(&xop[wave][((8 * kb + 4 + g) * 16 + li) * 16]);
      const v8i xa = v8i{y0[0], y0[1], y0[2], y0[3], y1[0], y1[1], y1[2], y1[3]};
#pragma unroll
      for (int p = 0; p < P; ++p) {
        v8i bs, bi;
        expand_f4((uint32_t)c[p][2 * kb], (uint32_t)c[p][2 * kb + 1], bs, bi);
        const v4f cS = (GS && kb == 0) ? v4f{0.f, 0.f, 0.f, 0.f} : aS[p];
        const v4f cI = (GS && kb == 0) ? v4f{0.f, 0.f, 0.f, 0.f} : aI[p];
        aS[p] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(xa, bs, cS, kFmtFp8, kFmtFp4, 0, 0, 0, 0);
        aI[p] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(xa, bi, cI, kFmtFp8, kFmtFp4, 0, 0, 0, 0);
      }
    }
    wave_sync();
    if constexpr (GS) {
#pragma unroll
      for (int p = 0; p < P; ++p)
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          const float vS = fmaf(aS[p][2 + k], 1.0f / kLoScale, aS[p][k]);
          const float vI = fmaf(aI[p][2 + k], 1.0f / kLoScale, aI[p][k]);
          Are[p][k] = fmaf(gs[p].x, vS - vI, Are[p][k]);
          Aim[p][k] = fmaf(gs[p].y, vI, Aim[p][k]);
        }
    }
#pragma unroll
    for (int p = 0; p < P; ++p) c[p] = cn[p];
  }

  // the wave's share of y before the token factor: lane group 2 sl holds the
  // first band's digits of token sl of the tile, 2 sl + 1 the second's (times
  // 2^8); what follows is linear, so each group forms its share and the two
  // are added last
  {
    double yr = 0.0, yi = 0.0;
#pragma unroll
    for (int st = 0; st < T; ++st) {
      float re[2][2], im[2][2];  // [matrix][component]
#pragma unroll
      for (int mm = 0; mm < 2; ++mm)
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          const int p = mm * T + st;
          if constexpr (GS) {
            re[mm][k] = Are[p][k];
            im[mm][k] = Aim[p][k];
          } else {
            const float vS = fmaf(aS[p][2 + k], 1.0f / kLoScale, aS[p][k]);
            im[mm][k] = fmaf(aI[p][2 + k], 1.0f / kLoScale, aI[p][k]);
            re[mm][k] = vS - im[mm][k];
          }
        }
      const double u_re = GS ? 1.0f : sc[0][st][0], u_im = GS ? 1.0f : sc[0][st][1];
      const double w_re = GS ? 1.0f : sc[1][st][0], w_im = GS ? 1.0f : sc[1][st][1];
      yr = fma(u_re, (double)re[0][0], yr);
      yr = fma(-u_im, (double)im[0][1], yr);
      yr = fma(w_re, (double)re[1][0], yr);
      yr = fma(w_im, (double)im[1][1], yr);
      yi = fma(u_re, (double)re[0][1], yi);
      yi = fma(u_im, (double)im[0][0], yi);
      yi = fma(-w_re, (double)re[1][1], yi);
      yi = fma(w_im, (double)im[1][0], yi);
    }
    yr = fma(__shfl_down(yr, 16), 1.0 / kBand2Scale, yr);
    yi = fma(__shfl_down(yi, 16), 1.0 / kBand2Scale, yi);
    if (!(g & 1)) part[kw][2 * tile + (g >> 1)][li] = make_double2(yr, yi);  // zero for a wave without steps
  }
  __syncthreads();
  if (tid >= 16 * B) return;
  const int b = tid >> 4, r = tid & 15;
  if (rb * 16 + r >= N) return;
  double yr = 0.0, yi = 0.0;
#pragma unroll
  for (int w = 0; w < KW; ++w) {
    yr += part[w][b][r].x;
    yi += part[w][b][r].y;
  }
  float mb = 0.0f;
#pragma unroll
  for (int w = 0; w < KW; ++w) mb = fmaxf(mb, tok_max[b][w]);
  const double f = mb > 0.0f ? (double)ldexpf(1.0f, -f4_token_shift(mb)) : 0.0;
  L.y[(int64_t)b * N + rb * 16 + r] = make_float2((float)(yr * f), (float)(yi * f));
#endif
}

template <int T, int TILES>
void launch_split_f4_n(const SplitGroup& a, bool gs, unsigned blocks, hipStream_t s) {
  if (gs) hipLaunchKernelGGL((dec_split_f4_kernel<T, TILES, true>), dim3(blocks), dim3(64 * kWaves), 0, s, a);
  else hipLaunchKernelGGL((dec_split_f4_kernel<T, TILES, false>), dim3(blocks), dim3(64 * kWaves), 0, s, a);
}

template <int T>
void launch_split_f4_t(const SplitGroup& a, bool gs, unsigned blocks, hipStream_t s) {
  if constexpr (T <= 3) {
    if (a.B > 2) {
      launch_split_f4_n<T, 2>(a, gs, blocks, s);
      return;
    }
  }
  launch_split_f4_n<T, 1>(a, gs, blocks, s);
}

}  // namespace

constexpr int64_t kCUs = 256;

// Every block encodes its tokens itself, over all of K, so the one launch costs
// more per row block and 256-code step than the streaming product, against the
// two launches it saves.  What it costs goes with the steps that the row blocks
// of a CU take together (row blocks x steps / 256 CUs), so the call's are
// bounded, by T, tokens and kind of scales; three and four tokens halve the
// waves on a row block's steps, which bounds the steps of a layer too.  One
// launch / streaming, us (n x k: rows x columns of a layer, w: steps a CU):
//   T = 1  8 x 2048 x 8192, w 128    1 token 26 / 27, 2 tokens 34 / 31
//          8192 x 8192, w 64         2 tokens 20 / 23, 3 30 / 31, 4 34 / 31
//          4 x 2048 x 5504, w 44     4 tokens 24 / 28
//   T = 2  8 x 2048 x 8192, w 128    1 token 37 / 37; 2 46 / 41, G = 256 52 / 53
//          8192 x 8192, w 64         2 tokens 25 / 30
//          4 x 2048 x 5504, w 44     4 tokens 30 / 28, G = 256 33 / 35
//          4 x 2048 x 4096, w 32     4 tokens 23 / 26
//          1024 x 8192, w 8, 32 steps, G = 256, 4 tokens 29 / 26; 2048 x 5504, 22 steps, 20 / 26
//   T = 3  8192 x 8192, w 64         1 token 29 / 28; 4 x 2048 x 5504, w 44, 23 / 25
//          4 x 2048 x 4096, w 32     4 tokens 30 / 26; 2 x 2048 x 5504, w 22, 22 / 26
//   T = 4  8192 x 8192, w 64         1 token 33 / 36, 2 38 / 38
//          4 x 2048 x 4096, w 32     2 tokens 24 / 25, G = 256 31 / 29
//          4096 x 8192, w 32 in one block a CU, G = 256, 2 tokens 27 / 31
//   16384 x 256, one step: the streaming product has no slices to reduce
//          T = 1 1 token 7.4 / 8.5; T = 2 1 token 9.5 / 9.3, 2 9.9 / 9.4
// and by the row blocks alone, whose fixed cost is the tokens' (q k v 384, gate
// and up 688, all seven layers of a 2048-wide block 1328):
//   T = 2  384 1 token 7.4 / 14.3, 4 tokens 12.0 / 18.7; 688 10.6 / 14.5, 17.1 / 19.5;
//          1024 (8 x 2048 x 2048) 14 / 19, 24 / 24; 1328 22.1 / 21.9, 43.4 / 30.7
//   T = 3  384 4 tokens 16.7 / 19.8; 688 (n = 1536) 2 tokens 19.2 / 17.6
//   T = 4  384 1 token 12.8 / 16.7; 688 (n = 1024) 2 tokens 17.7 / 16.7
// Blocks beyond those resident (two a CU, one from T = 3 on) wait for a second
// round, which costs a whole one however few they are; the streaming product
// spreads any number evenly.  What that wastes goes with the steps that the CUs
// idle in the last round (waste) and, where the waves on a row block are few, with
// all steps of the rounds (full), steps per CU:
//   T = 1  4 tokens  520 x 4096 columns (row blocks x columns), waste 31, 22.7 / 20.4; 640, 24, equal
//   T = 2  2 tokens  520 x 5504, waste 43, 23.1 / 21.3; 520 x 4096, 31, equal
//          4 tokens  520 x 4096, full 64, 29.1 / 21.3, G = 256 35.3 / 28.6; 2048, full 32, pays
//   T = 3  1, 2      260 x 5504, waste 22, 19.0 / 18.2, 21.9 / 19.1; 260 x 4096, 16, pays;
//                    G = 256 260 x 4096, 16, 20.2 / 18.6; 320 x 4096, 12, 20.9 / 20.3; 384 x 4096, 8, pays
//          4 tokens  260 x 3072, full 24, 20.9 / 19.9; 4096, 32, 27.1 / 20.4; 2048, 16, pays;
//                    G = 256 260 x 1984, waste 8, 18.7 / 17.0; 352, 5, 19.0 / 18.7; 384, 4, 19.1 / 20.1
//   T = 4  1 token   260 x 5504, waste 22, 21.5 / 20.9; 2 tokens 260 x 4096, 16, 19.3 / 18.7, 384 x 8192, 16, 33.0 / 31.8;
//                    G = 256 260 x 4096, 16 steps, 23.5 / 20.4, 384 x 4096, waste 8, 24.4 / 22.9; 260 x 3072 17.1 / 20.4
bool last_round_wasted(int T, int B, bool gs, int64_t blocks, int longest) {
  const int64_t resident = T >= 3 ? kCUs : 2 * kCUs, slots = (blocks + resident - 1) / resident * resident;
  if (slots == resident) return false;
  const int64_t waste = (slots - blocks) * longest / kCUs, full = slots * longest / kCUs;
  switch (T) {
    case 1: return B > 2 && waste >= 28;
    case 2: return B > 2 ? full > 32 : B == 2 && !gs && waste >= 40;
    case 3: return B > 2 ? full > 16 || (gs && waste >= 5) : waste >= (gs ? 12 : 15);
    default: return gs ? longest >= 16 && waste >= 8 : waste >= (B == 1 ? 20 : 15);
  }
}


bool f4_split_ok(const DecHeader& h, const DecLayer* tab) {
  if (h.mode != kModeBf16F4 || h.bands != 2 || h.n_layers > kSplitLayers) return false;
  if (h.B > (h.T <= 3 ? 4 : 2)) return false;
  int64_t blocks = 0, work = 0;
  int longest = 0;
  for (int i = 0; i < h.n_layers; ++i) {
    longest = tab[i].nk4 > longest ? tab[i].nk4 : longest;
    blocks += tab[i].nrb;
    work += (int64_t)tab[i].nrb * tab[i].nk4;
    // all tokens are read before any output is written only where there are
    // two launches: outputs in the memory of the call's tokens go there
    const auto y0 = reinterpret_cast<uintptr_t>(tab[i].y), y1 = y0 + (uintptr_t)h.B * (uintptr_t)tab[i].N * 8;
    for (int k = 0; k < h.n_layers; ++k) {
      const auto x0 = reinterpret_cast<uintptr_t>(tab[k].x), x1 = x0 + (uintptr_t)h.B * (uintptr_t)tab[k].K * 4;
      if (y0 < x1 && x0 < y1) return false;
    }
  }
  if (longest > kSplitMaxSteps) return false;
  if (longest > 24 && h.B > 2 && (h.T > 1 || blocks < 64)) return false;
  if (longest == 1 && blocks > 2 * kCUs && (h.T > 1 || h.B == 2)) return false;
  if (blocks > kCUs * (h.T >= 3 ? 2 : h.T == 2 && h.B > 2 ? 3 : 4)) return false;
  const bool gs = h.grouped != 0;
  if (last_round_wasted(h.T, h.B, gs, blocks, longest)) return false;
  int64_t most;  // steps per CU
  switch (h.T) {
    case 1: most = h.B == 1 ? 128 : h.B <= 3 ? 64 : 48; break;
    case 2: most = h.B == 1 ? 128 : h.B == 2 ? (gs ? 128 : 64) : (gs ? 48 : 40); break;
    case 3: most = h.B <= 2 ? 48 : 24; break;
    default: most = h.B == 1 ? 64 : gs && blocks > kCUs ? 24 : 48; break;
  }
  return work <= most * kCUs;
}

hipError_t launch_split_f4(const DecHeader& h, const DecLayer* tab, hipStream_t s) {
  SplitGroup a{};
  uint32_t blocks = 0;
  for (int i = 0; i < h.n_layers; ++i) {
    const DecLayer& d = tab[i];
    SplitLayer& l = a.l[i];
    l.codes[0] = d.codes[0];
    l.codes[1] = d.codes[1];
    l.scales[0] = d.scales[0];
    l.scales[1] = d.scales[1];
    l.x = d.x;
    l.y = d.y;
    l.N = d.N;
    l.K = d.K;
    l.nk4 = d.nk4;
    l.gsteps = d.gsteps;
    l.ngroups = d.gsteps ? (d.nk4 + d.gsteps - 1) / d.gsteps : 0;
    l.code_bytes = (uint32_t)((size_t)h.T * (size_t)d.nrb * (size_t)d.nk4 * 1024);
    l.rb0 = blocks;
    blocks += (uint32_t)d.nrb;
  }
  a.n = h.n_layers;
  a.B = h.B;
  const bool gs = h.grouped != 0;
  switch (h.T) {
    case 1: launch_split_f4_t<1>(a, gs, blocks, s); break;
    case 2: launch_split_f4_t<2>(a, gs, blocks, s); break;
    case 3: launch_split_f4_t<3>(a, gs, blocks, s); break;
    default: launch_split_f4_t<4>(a, gs, blocks, s); break;
  }
  return hipGetLastError();
}

}  // namespace fairy2i
