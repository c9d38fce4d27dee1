// Recursive residual PhaseQuant of one complex matrix (Sec. 3.3 formal
// definition, with the projection, axis scales and dequantisation of
// Sec. 3.2).
//
// Per-tensor scales: a fill kernel clears the per-stage totals; then stage t
// is one kernel on the caller's stream.  A thread takes packed bytes (4
// consecutive entries of a row): it rebuilds the float64 residual from M and
// the codes/scales of stages < t, projects it, writes the byte of stage-t
// codes, and adds |Re r| (k even) or |Im r| (k odd) into an exact sum.  Each
// block adds its sums into one of 16 copies of the stage total with 64-bit
// integer atomics (exact, so the total does not depend on the order blocks
// arrive in); the block that arrives last rounds each exact mean once to
// float32 -> scales[t].  Stage t+1 reads scales[t] from device memory;
// nothing returns to the host.
//
// The exact sums.  A double v is split by two float64 additions of large
// constants (M1, M2 below) into an integer multiple of 2^e and an integer
// multiple of 2^(e - 47), which the sums' bit patterns hold as integers: nine
// float64 / 64-bit instructions a value, no shifts and no branches.  e is
// chosen per wave from its first entries' largest magnitude 2^X, e = X - 40:
// every value below 2^(X+4) that is a multiple of 2^(X-87) is taken, which
// the residual of a float32 matrix always is unless its entries differ by
// more than 2^20 from the wave's first; anything else goes to the block's
// limbs in LDS one value at a time.  Either way the integer total is the
// same.  (The kernel that split every value into 32-bit limbs by shifts and
// kept five 64-bit limbs a lane was bound by that arithmetic, 28.6 us a stage
// of 2048 x 2048 entries, and rounding took a launch of 6.9 us more.  A T = 2
// call took 69 us, now 32: per stage 16.7 us under the profiler, of which
// the 34 MB of entries and codes are 7 at the rate of a large copy, the
// blocks' atomics about 4 and the last block's count, loads and rounding
// about 4.)
#include "common.h"
#include "superacc.h"

namespace fairy2i {

namespace {

constexpr int kPartWords = 2 * SA_LIMBS + 2;  // acc[2][SA_LIMBS], cnt[2]

// Eq. (ifairy-proj) by exact comparisons (floor-form ties, 0 -> +1): the
// codeword's axis is the larger component's, on the diagonal a = b != 0 the
// imaginary one (counter-clockwise), on a = -b the real one.
__device__ inline uint32_t project_code(double a, double b) {
  const double A = fabs(a), B = fabs(b);
  const bool odd = B > A || (a == b && a != 0.0);
  const bool neg = odd ? b < 0.0 : (a < 0.0 && A >= B);
  return (odd ? 1u : 0u) | (neg ? 2u : 0u);
}

// The fixed-point window of a wave's (or wave segment's) exact sums.
constexpr int kFxHigh = 44, kFxLow = 47;  // values < 2^(e + kFxHigh), multiples of 2^(e - kFxLow)
struct FxWindow {
  double M1, M2, lim;
  int e;
};

__device__ inline double pow2(int k) { return __longlong_as_double((long long)(k + 1023) << 52); }

// Window for magnitudes around m >= 0 (any float; m need not bound anything).
__device__ inline FxWindow fx_window(float m) {
  FxWindow w;
  const int X = (int)((__float_as_uint(m) >> 23) & 0xFFu) - 126;  // m < 2^X; within [-126, 129]
  w.e = X + 4 - kFxHigh;
  w.M1 = 1.5 * pow2(52 + w.e);
  w.M2 = 1.5 * pow2(52 + w.e - kFxLow);
  w.lim = pow2(w.e + kFxHigh);
  return w;
}

// One lane's sums: over all its values and over those on the imaginary axis
// (k odd), each as the bit patterns of v + M1 and of the remainder + M2.
struct FxSum {
  unsigned long long hi, lo, hi1, lo1;
};

// Adds v >= 0.  False, with nothing but the constants added, if the window
// does not hold v exactly.
__device__ inline bool fx_add(FxSum& s, const FxWindow& w, double v, bool odd) {
  double t1 = v + w.M1;
  const double rest = v - (t1 - w.M1);
  double t2 = rest + w.M2;
  const bool ok = v < w.lim && t2 - w.M2 == rest;
  t1 = ok ? t1 : w.M1;
  t2 = ok ? t2 : w.M2;
  const unsigned long long b1 = (unsigned long long)__double_as_longlong(t1);
  const unsigned long long b2 = (unsigned long long)__double_as_longlong(t2);
  s.hi += b1;
  s.lo += b2;
  s.hi1 += odd ? b1 : 0ull;
  s.lo1 += odd ? b2 : 0ull;
  return ok;
}

template <int WIDTH, typename V>
__device__ inline V segment_sum(V v) {
#pragma unroll
  for (int off = WIDTH / 2; off > 0; off >>= 1) v += __shfl_xor(v, off);
  return v;
}

// 128-bit totals of both axes over WIDTH lanes, in units of 2^(e - kFxLow):
// out[axis] = {low, high}.  n, n1: this lane's values and those of the
// imaginary axis (at most 1024 values a lane: the sums stay below 2^63).
template <int WIDTH>
__device__ inline void fx_totals(const FxSum& s, const FxWindow& w, uint32_t n, uint32_t n1,
                                 unsigned long long (&out)[2][2]) {
  const unsigned long long c1 = (unsigned long long)__double_as_longlong(w.M1);
  const unsigned long long c2 = (unsigned long long)__double_as_longlong(w.M2);
  const unsigned long long hi1 = segment_sum<WIDTH>(s.hi1 - n1 * c1);
  const long long lo1 = (long long)segment_sum<WIDTH>(s.lo1 - n1 * c2);
  const unsigned long long hi0 = segment_sum<WIDTH>(s.hi - n * c1) - hi1;
  const long long lo0 = (long long)segment_sum<WIDTH>(s.lo - n * c2) - lo1;
  auto join = [](unsigned long long h, long long l, unsigned long long (&o)[2]) {
    const unsigned long long a = h << kFxLow;
    o[0] = a + (unsigned long long)l;
    o[1] = (h >> (64 - kFxLow)) + (unsigned long long)(l >> 63) + (o[0] < a ? 1ull : 0ull);
  };
  join(hi0, lo0, out[0]);
  join(hi1, lo1, out[1]);
}

// Adds both axes' 128-bit totals to their limbs in LDS, one word a lane
// (lanes 0 .. 9; every lane of the wave holds the totals).
__device__ inline void fx_to_limbs(const unsigned long long (&v)[2][2], int e, unsigned long long* acc) {
  const int lane = threadIdx.x & 63;
  if (lane >= 10) return;
  const int axis = lane / 5, i = lane - 5 * axis;
  const int p = e - kFxLow + 1074, sh = p & 31;  // position of the unit in units of 2^-1074: 861 .. 1116
  const unsigned long long lo = axis ? v[1][0] : v[0][0], hi = axis ? v[1][1] : v[0][1];
  const uint32_t w[4] = {(uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32)};
  const uint32_t here = i == 0 ? w[0] : i == 1 ? w[1] : i == 2 ? w[2] : i == 3 ? w[3] : 0u;
  const uint32_t below = i == 1 ? w[0] : i == 2 ? w[1] : i == 3 ? w[2] : i == 4 ? w[3] : 0u;
  const uint32_t x = sh ? (here << sh) | (below >> (32 - sh)) : here;
  if (x) atomicAdd(&acc[axis * SA_LIMBS + (p >> 5) + i], (unsigned long long)x);
}

// One value straight to the limbs in LDS (the window does not hold it).
__device__ inline void limbs_add(unsigned long long* acc, double v) {
  if (v == 0.0) return;
  int limb;
  uint32_t lo, mid, hi;
  sa_split(v, &limb, &lo, &mid, &hi);
  if (lo) atomicAdd(&acc[limb], (unsigned long long)lo);
  if (mid) atomicAdd(&acc[limb + 1], (unsigned long long)mid);
  if (hi) atomicAdd(&acc[limb + 2], (unsigned long long)hi);
}

// The residual of one entry after a stage whose code for it is k.
__device__ inline void subtract_stage(double& re, double& im, uint32_t k, double s_re, double s_im) {
  const double s = (k & 1u) ? s_im : s_re;
  const double d = (k & 2u) ? -s : s;
  re = (k & 1u) ? re : re - d;
  im = (k & 1u) ? im - d : im;
}

// Range of nonzero limbs of one axis, found by the 64 lanes of a wave
// (hi = -1: all zero).
__device__ inline void limb_range(const unsigned long long* acc, int& lo, int& hi) {
  static_assert(SA_LIMBS > 64 && SA_LIMBS <= 128, "two ballots");
  const int lane = threadIdx.x & 63;
  const unsigned long long m0 = __ballot(acc[lane] != 0);
  const unsigned long long m1 = __ballot(64 + lane < SA_LIMBS && acc[64 + lane < SA_LIMBS ? 64 + lane : 0] != 0);
  hi = m1 ? 127 - __builtin_clzll(m1) : (m0 ? 63 - __builtin_clzll(m0) : -1);
  lo = m0 ? __builtin_ctzll(m0) : (m1 ? 64 + __builtin_ctzll(m1) : 0);
}

// Copies of a stage's total: block b adds into copy b % kTotCopies, so each
// total word takes 1/kTotCopies of the blocks' atomics; the last block adds
// the copies (integers: the order does not matter).
constexpr int kTotCopies = 16;
constexpr int kTotWords = kTotCopies * kPartWords;
// The blocks that have added their words to a copy are counted in the bits
// from 40 on of its last word (a count of entries, below 2^32), the copies
// that are complete from 52 on of copy 0's.  (Additions to one word queue up:
// one count of all 1024 blocks made a stage 5 us longer.  64 copies of the
// limbs in use instead of 16 changed nothing.)
constexpr int kArrivedBit = 40, kCompleteBit = 52;
constexpr int kQzUnroll = 2;      // bytes a thread loads before it quantises them
constexpr int kFlushRounds = 128;  // rounds of kQzUnroll bytes (1024 values) between flushes of a lane's sums

// Stage T0 (0-based) of the per-tensor quantiser.  Grid: up to kQzMaxBlocks
// blocks of 256, four per CU (512 blocks of 512 measured a tenth slower).
// kQzUnroll: with four bytes a round a thread took 132 registers or more, so
// three blocks fit a CU and the grid ended in a second, nearly empty round;
// with two the stages take 100, 106, 120 and (capped, two of them in memory;
// 130 without: a T = 4 call of 5504 x 2048 134 us, now 130) 128, and all 1024
// are resident.  2048 x 2048, T = 2, U and
// W with their conversion and repacking: 106.4 -> 96.1 us (four bytes capped
// at 128 registers spill: 113; one byte and the next round's loads ahead:
// 95.3, two bytes and those: 99.6).
template <int T0>
__global__ __launch_bounds__(kQzThreads, T0 == 3 ? 4 : 1) void qz_stage_kernel(const float2* __restrict__ M, int64_t nbytes,
                                                              uint8_t* __restrict__ codes,
                                                              float* __restrict__ scales,
                                                              unsigned long long* __restrict__ tot) {
  __shared__ unsigned long long acc[kPartWords];  // acc[2][SA_LIMBS], cnt[2]
  __shared__ bool last;
  const int lane = threadIdx.x & 63;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const bool al16 = (reinterpret_cast<uintptr_t>(M) & 15) == 0;  // a byte's 4 entries as two 16-byte loads
  float4 mv[kQzUnroll][2];
  uint32_t prev[kQzUnroll][T0 + 1];
  auto load_round = [&](int64_t b0) {
#pragma unroll
    for (int u = 0; u < kQzUnroll; ++u) {
      const int64_t bi = b0 + u * stride;
      const bool ok = bi < nbytes;
      mv[u][0] = mv[u][1] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (ok && al16) {
        const float4* m4 = reinterpret_cast<const float4*>(M + 4 * bi);
        mv[u][0] = m4[0];
        mv[u][1] = m4[1];
      } else if (ok) {
        const float2 a0 = M[4 * bi], a1 = M[4 * bi + 1], a2 = M[4 * bi + 2], a3 = M[4 * bi + 3];
        mv[u][0] = make_float4(a0.x, a0.y, a1.x, a1.y);
        mv[u][1] = make_float4(a2.x, a2.y, a3.x, a3.y);
      }
#pragma unroll
      for (int tp = 0; tp < T0; ++tp) prev[u][tp] = ok ? codes[(int64_t)tp * nbytes + bi] : 0u;
    }
  };
  // the first round is asked for before anything is waited for: a matrix of up
  // to kQzMaxBlocks * kQzThreads * kQzUnroll * 4 = 2 M entries has no other
  int64_t w0 = (int64_t)blockIdx.x * blockDim.x + (threadIdx.x - lane);
  load_round(w0 + lane);
  for (int i = threadIdx.x; i < kPartWords; i += blockDim.x) acc[i] = 0ull;
  __syncthreads();

  double s_re[T0 + 1], s_im[T0 + 1];
  float smax = 0.0f;
#pragma unroll
  for (int tp = 0; tp < T0; ++tp) {
    s_re[tp] = (double)scales[2 * tp];
    s_im[tp] = (double)scales[2 * tp + 1];
    smax = fmaxf(smax, fmaxf(scales[2 * tp], scales[2 * tp + 1]));
  }
  bool placed = false;
  FxWindow win = fx_window(1.0f);
  FxSum sum{0, 0, 0, 0};
  uint32_t n = 0, n1 = 0;
  auto flush = [&]() {
    unsigned long long v[2][2];
    fx_totals<64>(sum, win, n, n1, v);
    const uint32_t cn = segment_sum<64>(n), cn1 = segment_sum<64>(n1);
    fx_to_limbs(v, win.e, acc);
    if (lane < 2) atomicAdd(&acc[2 * SA_LIMBS + lane], (unsigned long long)(lane ? cn1 : cn - cn1));
    sum = FxSum{0, 0, 0, 0};
    n = n1 = 0;
  };
  // every lane of a wave runs the same number of rounds (the window and the
  // flushes are the wave's); lanes past the end load nothing
  int round = 0;
  while (w0 < nbytes) {
    const int64_t b0 = w0 + lane;
    if (!placed) {  // the wave's first entries that are not all zero place the window
      float m = 0.0f;
#pragma unroll
      for (int u = 0; u < kQzUnroll; ++u)
#pragma unroll
        for (int h = 0; h < 2; ++h)
          m = fmaxf(fmaxf(fmaxf(m, fabsf(mv[u][h].x)), fmaxf(fabsf(mv[u][h].y), fabsf(mv[u][h].z))), fabsf(mv[u][h].w));
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
      m = fmaxf(m, smax);
      placed = m > 0.0f;
      if (placed) {
        // nothing but zeros has been added so far: the sums restart with the
        // new window's constants of those
        win = fx_window(m);
        const unsigned long long c1 = (unsigned long long)__double_as_longlong(win.M1);
        const unsigned long long c2 = (unsigned long long)__double_as_longlong(win.M2);
        sum.hi = n * c1;
        sum.lo = n * c2;
        sum.hi1 = n1 * c1;
        sum.lo1 = n1 * c2;
      }
    }
#pragma unroll
    for (int u = 0; u < kQzUnroll; ++u) {
      const int64_t bi = b0 + u * stride;
      if (bi < nbytes) {
        const float2 m[4] = {make_float2(mv[u][0].x, mv[u][0].y), make_float2(mv[u][0].z, mv[u][0].w),
                             make_float2(mv[u][1].x, mv[u][1].y), make_float2(mv[u][1].z, mv[u][1].w)};
        uint32_t out = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          double re = (double)m[e].x, im = (double)m[e].y;
#pragma unroll
          for (int tp = 0; tp < T0; ++tp) subtract_stage(re, im, (prev[u][tp] >> (2 * e)) & 3u, s_re[tp], s_im[tp]);
          const uint32_t k = project_code(re, im);
          const bool odd = k & 1u;
          const double v = fabs(odd ? im : re);
          if (!fx_add(sum, win, v, odd)) limbs_add(acc + (odd ? SA_LIMBS : 0), v);
          out |= k << (2 * e);
        }
        n += 4;
        n1 += __builtin_popcount(out & 0x55u);
        codes[(int64_t)T0 * nbytes + bi] = (uint8_t)out;
      }
    }
    w0 += kQzUnroll * stride;
    if (w0 < nbytes) load_round(w0 + lane);
    if (++round % kFlushRounds == 0) flush();
  }
  flush();
  __syncthreads();
  // the block's words into its copy of the stage total: 64-bit integer
  // additions, exact and independent of the order in which blocks arrive
  // (a grid of one block has its total at hand)
  if (gridDim.x > 1) {
    const unsigned copy = blockIdx.x % kTotCopies;
    unsigned long long* tc = tot + (int64_t)copy * kPartWords;
    for (int i = threadIdx.x; i < kPartWords; i += blockDim.x)
      if (acc[i]) atomicAdd(&tc[i], acc[i]);
    // The totals are touched by device-scope atomics only, which are performed
    // at the device's point of coherence: once this block's have been performed
    // (the wait, which the compiler may move no memory access across), the
    // counts of arrived blocks and complete copies tell the last one that all
    // have.  A release fence would write back the codes in the L2 for each block.
    __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) {
      const unsigned in_copy = (gridDim.x - copy + kTotCopies - 1) / kTotCopies;  // blocks of this copy
      const unsigned copies = gridDim.x < kTotCopies ? gridDim.x : kTotCopies;
      const unsigned long long a = atomicAdd(&tc[kPartWords - 1], 1ull << kArrivedBit);
      bool end = ((a >> kArrivedBit) & 0xFFFu) + 1 == in_copy;
      if (end) end = (atomicAdd(&tot[kPartWords - 1], 1ull << kCompleteBit) >> kCompleteBit) + 1 == copies;
      last = end;
    }
    __syncthreads();
    if (!last) return;
    for (int i = threadIdx.x; i < kPartWords; i += blockDim.x) {
      unsigned long long c[kTotCopies], v = 0;
#pragma unroll
      for (int k = 0; k < kTotCopies; ++k)
        c[k] = __hip_atomic_load(&tot[(int64_t)k * kPartWords + i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
      for (int k = 0; k < kTotCopies; ++k) v += i == kPartWords - 1 ? c[k] & ((1ull << kArrivedBit) - 1) : c[k];
      acc[i] = v;
    }
    __syncthreads();
  }
  const int axis = threadIdx.x >> 6;  // one wave per axis finds the limbs in use, one lane rounds
  if (axis < 2) {
    int lo, hi;
    limb_range(acc + axis * SA_LIMBS, lo, hi);
    const uint64_t cnt = acc[2 * SA_LIMBS + axis];
    if (lane == 0)
      scales[2 * T0 + axis] = cnt ? sa_mean_range(reinterpret_cast<const uint64_t*>(acc) + axis * SA_LIMBS, lo, hi, cnt) : 0.0f;
  }
}

// Mean of a 128-bit total in units of 2^(e - kFxLow), rounded once.
__device__ inline float fx_mean(const unsigned long long (&v)[2], int e, uint64_t n) {
  if (!(v[0] | v[1]) || !n) return 0.0f;
  unsigned long long h = v[1], l = v[0];
  int E = e - kFxLow + 64;  // weight of h's unit
  if (!h) {
    h = l;
    l = 0;
    E -= 64;
  }
  const int z = __builtin_clzll(h);
  if (z) {
    h = (h << z) | (l >> (64 - z));
    l <<= z;
  }
  return sa_round_mean(h, l != 0, E - z, n);
}

// Per-group scales, groups of up to 1024 columns: LPG lanes (a power of two)
// per (row, group), 64 / LPG groups a wave, NB bytes (4 entries each) a lane.
// The entries stay in registers as residuals through all T stages, so M is
// read once and no stage waits for another kernel; each group's two exact
// means are rounded once to float32 into scales[t][row][g][axis].  (One block
// of 64 threads per group and a launch per stage, each with 134 words of LDS
// to clear and to round from, was bound by that fixed cost: 2752 x 2048,
// G = 256, T = 2 took 331 us, now 51, bound by the float64 arithmetic.)
constexpr int kQzgThreads = 256;

template <int LPG, int NB>
__global__ __launch_bounds__(kQzgThreads) void qzg_kernel(const float2* __restrict__ M, int64_t N, int64_t K, int64_t G,
                                                          int64_t ngroups, int T, uint8_t* __restrict__ codes,
                                                          float* __restrict__ scales) {
  __shared__ unsigned long long limbs[kQzgThreads / 64][2][SA_LIMBS];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int seg = lane / LPG, sl = lane % LPG;
  const int64_t gi = ((int64_t)blockIdx.x * (kQzgThreads / 64) + wave) * (64 / LPG) + seg;
  const bool live = gi < N * ngroups;
  const int64_t row = live ? gi / ngroups : 0;
  const int64_t g = live ? gi - row * ngroups : 0;
  const int64_t j0 = g * G, j1 = live ? (j0 + G < K ? j0 + G : K) : j0;  // columns of the group (multiples of 4)
  const int64_t nbytes = N * K / 4;
  const int64_t byte0 = (row * K + j0) / 4;
  const int gb = (int)((j1 - j0) / 4);  // bytes of the group; lane sl takes bytes sl, sl + LPG, ...
  const bool al16 = (reinterpret_cast<uintptr_t>(M) & 15) == 0;
  double re[NB][4], im[NB][4];
  float m = 0.0f;
  int nb = 0;
#pragma unroll
  for (int u = 0; u < NB; ++u) {
    const int bi = sl + u * LPG;
    float4 a = make_float4(0.f, 0.f, 0.f, 0.f), b = a;
    if (bi < gb) {
      ++nb;
      const float2* src = M + 4 * (byte0 + bi);
      if (al16) {
        a = reinterpret_cast<const float4*>(src)[0];
        b = reinterpret_cast<const float4*>(src)[1];
      } else {
        a = make_float4(src[0].x, src[0].y, src[1].x, src[1].y);
        b = make_float4(src[2].x, src[2].y, src[3].x, src[3].y);
      }
    }
    const float f[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      re[u][e] = (double)f[2 * e];
      im[u][e] = (double)f[2 * e + 1];
      m = fmaxf(m, fmaxf(fabsf(f[2 * e]), fabsf(f[2 * e + 1])));
    }
  }
#pragma unroll
  for (int off = LPG / 2; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
  // a residual is at most the entry plus the scales so far, each at most the
  // largest magnitude: the window's 2^4 above it holds all of a T <= 4 recursion
  const FxWindow win = fx_window(m);
  const uint32_t cnt_all = 4u * (uint32_t)gb;
  for (int t = 0; t < T; ++t) {
    FxSum sum{0, 0, 0, 0};
    uint32_t n1 = 0;
    bool ok = true;
    uint32_t out[NB];
#pragma unroll
    for (int u = 0; u < NB; ++u) {
      out[u] = 0;
      if (sl + u * LPG < gb) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint32_t k = project_code(re[u][e], im[u][e]);
          const bool odd = k & 1u;
          ok &= fx_add(sum, win, fabs(odd ? im[u][e] : re[u][e]), odd);
          out[u] |= k << (2 * e);
        }
        n1 += __builtin_popcount(out[u] & 0x55u);
        codes[(int64_t)t * nbytes + byte0 + sl + u * LPG] = (uint8_t)out[u];
      }
    }
    unsigned long long v[2][2];
    fx_totals<LPG>(sum, win, 4u * (uint32_t)nb, n1, v);
    const uint32_t odds = (uint32_t)segment_sum<LPG>(n1), evens = cnt_all - odds;
    float s[2] = {fx_mean(v[0], win.e, evens), fx_mean(v[1], win.e, odds)};
    // groups with a value that the window does not hold: all of the group's
    // values through the wave's limbs, one group at a time
    unsigned long long todo = __ballot(!ok);
    while (todo) {
      const int ts = __builtin_ctzll(todo) / LPG;
      unsigned long long* acc = &limbs[wave][0][0];
      for (int i = lane; i < 2 * SA_LIMBS; i += 64) acc[i] = 0ull;
      wave_sync();
      if (seg == ts) {
#pragma unroll
        for (int u = 0; u < NB; ++u)
          if (sl + u * LPG < gb) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const bool odd = (out[u] >> (2 * e)) & 1u;
              limbs_add(acc + (odd ? SA_LIMBS : 0), fabs(odd ? im[u][e] : re[u][e]));
            }
          }
      }
      wave_sync();
#pragma unroll
      for (int axis = 0; axis < 2; ++axis) {
        int lo, hi;
        limb_range(acc + axis * SA_LIMBS, lo, hi);
        const uint32_t c = axis ? odds : evens;
        if (seg == ts) s[axis] = c ? sa_mean_range(reinterpret_cast<const uint64_t*>(acc) + axis * SA_LIMBS, lo, hi, c) : 0.0f;
      }
      wave_sync();
      const unsigned long long mask = LPG == 64 ? ~0ull : ((1ull << (LPG % 64)) - 1) << (ts * LPG % 64);
      todo &= ~mask;
    }
    if (live && sl == 0) {
      float* dst = scales + ((t * N + row) * ngroups + g) * 2;
      dst[0] = s[0];
      dst[1] = s[1];
    }
    if (t + 1 < T) {
#pragma unroll
      for (int u = 0; u < NB; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e) subtract_stage(re[u][e], im[u][e], (out[u] >> (2 * e)) & 3u, (double)s[0], (double)s[1]);
    }
  }
}

// The same for groups of more than 1024 columns: one wave per (row, group)
// walks the group's bytes once per stage, rebuilding the residuals from M and
// the codes it wrote for the earlier stages.
__global__ __launch_bounds__(64) void qzg_long_kernel(const float2* __restrict__ M, int64_t N, int64_t K, int64_t G,
                                                      int64_t ngroups, int T, uint8_t* codes, float* __restrict__ scales) {
  __shared__ unsigned long long acc[2][SA_LIMBS];
  const int lane = threadIdx.x;
  const int64_t row = (int64_t)blockIdx.x / ngroups;
  const int64_t g = (int64_t)blockIdx.x - row * ngroups;
  const int64_t j0 = g * G, j1 = j0 + G < K ? j0 + G : K;
  const int64_t nbytes = N * K / 4;
  const int64_t byte0 = (row * K + j0) / 4, gb = (j1 - j0) / 4;
  double s_re[FAIRY2I_MAX_STAGES] = {0, 0, 0, 0}, s_im[FAIRY2I_MAX_STAGES] = {0, 0, 0, 0};
  float m0 = 0.0f;
  for (int64_t bi = lane; bi < gb && bi < 4 * 64; bi += 64)
    for (int e = 0; e < 4; ++e) {
      const float2 f = M[4 * (byte0 + bi) + e];
      m0 = fmaxf(m0, fmaxf(fabsf(f.x), fabsf(f.y)));
    }
  for (int off = 32; off > 0; off >>= 1) m0 = fmaxf(m0, __shfl_xor(m0, off));
  const FxWindow win = fx_window(m0);
#pragma unroll
  for (int t = 0; t < FAIRY2I_MAX_STAGES; ++t) {
    if (t >= T) break;
    for (int i = lane; i < 2 * SA_LIMBS; i += 64) (&acc[0][0])[i] = 0ull;
    __syncthreads();
    FxSum sum{0, 0, 0, 0};
    uint32_t n = 0, n1 = 0;
    uint64_t odds = 0;
    auto flush = [&]() {
      unsigned long long v[2][2];
      fx_totals<64>(sum, win, n, n1, v);
      odds += segment_sum<64>(n1);
      fx_to_limbs(v, win.e, &acc[0][0]);
      sum = FxSum{0, 0, 0, 0};
      n = n1 = 0;
    };
    int round = 0;
    for (int64_t w0 = 0; w0 < gb; w0 += 64) {
      const int64_t bi = byte0 + w0 + lane;
      if (w0 + lane < gb) {
        uint32_t out = 0;
        uint32_t prev[FAIRY2I_MAX_STAGES];
#pragma unroll
        for (int tp = 0; tp < FAIRY2I_MAX_STAGES; ++tp) prev[tp] = tp < t ? codes[(int64_t)tp * nbytes + bi] : 0u;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float2 f = M[4 * bi + e];
          double re = (double)f.x, im = (double)f.y;
#pragma unroll
          for (int tp = 0; tp < FAIRY2I_MAX_STAGES; ++tp)
            if (tp < t) subtract_stage(re, im, (prev[tp] >> (2 * e)) & 3u, s_re[tp], s_im[tp]);
          const uint32_t k = project_code(re, im);
          const bool odd = k & 1u;
          const double v = fabs(odd ? im : re);
          if (!fx_add(sum, win, v, odd)) limbs_add(acc[odd ? 1 : 0], v);
          out |= k << (2 * e);
        }
        n += 4;
        n1 += __builtin_popcount(out & 0x55u);
        codes[(int64_t)t * nbytes + bi] = (uint8_t)out;
      }
      if (++round % 256 == 0) flush();  // 1024 values a lane
    }
    flush();
    __syncthreads();
    float s[2];
#pragma unroll
    for (int axis = 0; axis < 2; ++axis) {
      int lo, hi;
      limb_range(acc[axis], lo, hi);
      const uint64_t c = axis ? odds : 4 * (uint64_t)gb - odds;
      s[axis] = c ? sa_mean_range(reinterpret_cast<const uint64_t*>(acc[axis]), lo, hi, c) : 0.0f;
    }
    if (lane == 0) {
      float* dst = scales + ((t * N + row) * ngroups + g) * 2;
      dst[0] = s[0];
      dst[1] = s[1];
    }
    s_re[t] = (double)s[0];
    s_im[t] = (double)s[1];
    __syncthreads();
  }
}

__global__ __launch_bounds__(256) void qz_zero_kernel(unsigned long long* __restrict__ p, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0ull;
}

int quantize_blocks(int64_t N, int64_t K) {
  const int64_t nbytes = N * K / 4;
  int64_t b = (nbytes + kQzThreads - 1) / kQzThreads;
  if (b > kQzMaxBlocks) b = kQzMaxBlocks;
  if (b < 1) b = 1;
  return (int)b;
}

template <int LPG, int NB>
void launch_qzg(const float2* M, int64_t N, int64_t K, int64_t G, int T, uint8_t* codes, float* scales, hipStream_t s) {
  const int64_t ngroups = (K + G - 1) / G;
  const int64_t per_block = kQzgThreads / LPG;
  hipLaunchKernelGGL((qzg_kernel<LPG, NB>), dim3((unsigned)((N * ngroups + per_block - 1) / per_block)),
                     dim3(kQzgThreads), 0, s, M, N, K, G, ngroups, T, codes, scales);
}

}  // namespace

hipError_t launch_quantize_grouped(const float2* M, int64_t N, int64_t K, int T, int64_t G, uint8_t* codes,
                                   float* scales, hipStream_t stream) {
  const int64_t b = G / 4;  // bytes of a whole group (the last of a row may be shorter)
  if (b <= 1) launch_qzg<1, 1>(M, N, K, G, T, codes, scales, stream);
  else if (b <= 2) launch_qzg<2, 1>(M, N, K, G, T, codes, scales, stream);
  else if (b <= 4) launch_qzg<4, 1>(M, N, K, G, T, codes, scales, stream);
  else if (b <= 8) launch_qzg<8, 1>(M, N, K, G, T, codes, scales, stream);
  else if (b <= 16) launch_qzg<16, 1>(M, N, K, G, T, codes, scales, stream);
  else if (b <= 32) launch_qzg<32, 1>(M, N, K, G, T, codes, scales, stream);
  else if (b <= 64) launch_qzg<64, 1>(M, N, K, G, T, codes, scales, stream);
  else if (b <= 128) launch_qzg<64, 2>(M, N, K, G, T, codes, scales, stream);
  else if (b <= 256) launch_qzg<64, 4>(M, N, K, G, T, codes, scales, stream);
  else {
    const int64_t ngroups = (K + G - 1) / G;
    hipLaunchKernelGGL(qzg_long_kernel, dim3((unsigned)(N * ngroups)), dim3(64), 0, stream, M, N, K, G, ngroups, T,
                       codes, scales);
  }
  return hipGetLastError();
}

size_t quantize_workspace_bytes(int64_t N, int64_t K) {
  (void)N;
  (void)K;
  return (size_t)FAIRY2I_MAX_STAGES * kTotWords * sizeof(unsigned long long);  // totals per stage
}

hipError_t launch_quantize(const float2* M, int64_t N, int64_t K, int T, uint8_t* codes,
                           float* scales, void* workspace, hipStream_t stream) {
  const int nblk = quantize_blocks(N, K);
  const int64_t nbytes = N * K / 4;
  auto* tot = static_cast<unsigned long long*>(workspace);
  const int words = T * kTotWords;
  hipLaunchKernelGGL(qz_zero_kernel, dim3((unsigned)((words + 255) / 256)), dim3(256), 0, stream, tot, words);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  for (int t = 0; t < T; ++t) {
    auto* kernel = t == 0 ? qz_stage_kernel<0> : t == 1 ? qz_stage_kernel<1> : t == 2 ? qz_stage_kernel<2> : qz_stage_kernel<3>;
    hipLaunchKernelGGL(kernel, dim3(nblk), dim3(kQzThreads), 0, stream, M, nbytes, codes, scales,
                       tot + (int64_t)t * kTotWords);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace fairy2i
