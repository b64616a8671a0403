// Gain estimation on the device, for frames whose gain is not supplied
// (Methods, "Main parameters": the gain is then estimated at each
// iteration).  The estimate of an iteration comes from the current image C:
//
//   1. sigma clipping: starting from every pixel, up to 5 rounds, each
//      keeping the values within 3 standard deviations (population) of the
//      lower median of the values kept so far; a round that keeps every value
//      ends the clipping;
//   2. the mean m and variance v (population) of the kept values;
//   3. g = (m + sqrt(m^2 + 4 v rn^2)) / (2 v): the gain for which the noise
//      model's variance of a pixel in ADU, m / g + rn^2 / g^2, equals v.
//
// All of it in binary64.  The sums are exact: each value x = M 2^(e-150)
// (M its 24-bit significand, e its biased exponent, at least 1) adds M to an
// integer accumulator of its exponent (positive and negative values apart),
// and M^2 = Mh^2 2^24 + Mh Ml 2^13 + Ml^2 (Mh, Ml the 12-bit halves) adds to
// three more, every partial sum below 2^55; the accumulators of all exponents
// are then added as one wide integer and rounded once to binary64.  So the
// sums, and everything computed from them, do not depend on the order in
// which the pixels were visited.  Nearly every value lies within a few powers
// of two of the median: those whose exponent is in a window of 8 from ebase
// are summed per thread in registers instead, as the integers M 2^(e - ebase)
// below 2^31 (their signed sum in 64 bits, their squares' in 96), and so are
// the counts of the 8 bins around the median (a byte each); the others take
// the accumulators and bins in LDS one by one.
//
// What bounds a pass: a read of the image (four 16-byte loads in flight per
// thread), then the last block's serial part, kept to the accumulators in
// use.  (With wave-wide sums per exponent and one pixel per load, the five
// rounds on a 2048^2 frame took 1.24 ms per iteration; now 0.30.)
//
// A clipping round keeps the values x with |x - median| <= 3 sd (in
// binary64), a set that is an interval of binary32 values (the test is
// monotone on either side of the median); the rounds intersect such
// intervals, so the kept set is always one interval [lo, hi] of
// order-preserving 32-bit keys, and every pass filters on it.
//
// The median is a radix selection over the keys in three passes (key bits
// 31-20, 19-10, 9-0), each a histogram of the values in the interval that
// share the digits found so far.  The first pass of a round also forms the
// sums.  Each pass is one launch over the frame's pixels; its last block to
// finish (a counter raised when its sums are published) reads the histogram
// and sums, takes the round's decisions and clears them for the next pass.
// From the second round on the median moves by little (the clipped values are
// few), so the first pass also counts the values at each of the 16384 keys
// around the previous median, one bin per key, and those below them: where
// the new median lies among them it is found at once and the two selection
// passes return at once.  (Small frames select: kGainNearPx.)
// The estimate ends after a round that keeps every value or after 5 rounds;
// the launches of the rounds not needed return at once.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "lacosmic_device.h"
#include "lacosmic_mem.h"

namespace lac {

// Order-preserving 32-bit key of a binary32 value (unsigned order).
__device__ __forceinline__ uint32_t gkey(float x) {
  const uint32_t b = __float_as_uint(x);
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__device__ __forceinline__ float gkey_value(uint32_t k) {
  return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}

__device__ __forceinline__ uint32_t gain_atomic_load(const uint32_t* p) {
  return __hip_atomic_load(gp(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long gain_atomic_load(const unsigned long long* p) {
  return __hip_atomic_load(gp(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The current image: the input in iteration 0 (float32 or uint16), the
// cleaned image after that.  (The launches of kFusedPingPong keep it in two
// places in turn: frames that estimate their gain do not run them.)  Pixels are
// taken canonical (-0 as +0).
struct GainImage {
  const float* f32;
  const uint16_t* u16;  // instead, if not null
  __device__ __forceinline__ GainImage(const FrameDev& f, int it) {
    u16 = it == 0 ? f.img16 : nullptr;
    f32 = it == 0 ? f.img : f.clean;
  }
  __device__ __forceinline__ float at(int64_t i) const {
    return u16 ? (float)ldg(u16, i) : ldg(f32, i) + 0.0f;
  }
};

// ---------------------------------------------------------- wide integers
// Adds v * 2^shift to the nl-limb unsigned integer L (little-endian limbs).
__device__ __forceinline__ void big_add(uint64_t* L, int nl, uint64_t v, int shift) {
  int w = shift >> 6;
  const int s = shift & 63;
  uint64_t lo = v << s, hi = s ? (v >> (64 - s)) : 0ull;
  uint64_t carry = 0;
  for (; w < nl; ++w) {
    const uint64_t a = L[w];
    const uint64_t add = lo;
    uint64_t t = a + add;
    uint64_t c1 = t < a ? 1ull : 0ull;
    const uint64_t t2 = t + carry;
    c1 += t2 < t ? 1ull : 0ull;
    L[w] = t2;
    carry = c1;
    lo = hi;
    hi = 0;
    if (!lo && !carry) break;
  }
}

// a <- a - b for a >= b.
__device__ __forceinline__ void big_sub(uint64_t* a, const uint64_t* b, int nl) {
  uint64_t borrow = 0;
  for (int w = 0; w < nl; ++w) {
    const uint64_t x = a[w], y = b[w];
    const uint64_t d = x - y;
    const uint64_t d2 = d - borrow;
    borrow = (x < y ? 1ull : 0ull) | (d < borrow ? 1ull : 0ull);
    a[w] = d2;
  }
}

__device__ __forceinline__ bool big_less(const uint64_t* a, const uint64_t* b, int nl) {
  for (int w = nl - 1; w >= 0; --w)
    if (a[w] != b[w]) return a[w] < b[w];
  return false;
}

__device__ __forceinline__ int big_bit(const uint64_t* L, int p) { return (int)((L[p >> 6] >> (p & 63)) & 1ull); }

// The value L * 2^lsb_exp rounded to the nearest binary64 (ties to even).
__device__ double big_to_double(const uint64_t* L, int nl, int lsb_exp) {
  int top = nl - 1;
  while (top >= 0 && L[top] == 0ull) --top;
  if (top < 0) return 0.0;
  int p = top * 64 + 63 - __clzll((long long)L[top]);  // most significant set bit
  if (p < 53) return ldexp((double)L[0], lsb_exp);
  const int lo = p - 52;  // the 53 bits [lo, p] form the significand
  uint64_t m = L[lo >> 6] >> (lo & 63);
  if ((lo & 63) && (lo >> 6) + 1 < nl) m |= L[(lo >> 6) + 1] << (64 - (lo & 63));
  m &= (1ull << 53) - 1ull;
  const int guard = big_bit(L, lo - 1);  // lo >= 1: p >= 53
  bool sticky = false;                   // any set bit in [0, lo - 2]
  const int last = lo - 2;
  if (last >= 0) {
    const int lw = last >> 6;
    for (int w = 0; w < lw; ++w) sticky = sticky || L[w] != 0ull;
    const uint64_t below = ((last & 63) == 63) ? ~0ull : ((2ull << (last & 63)) - 1ull);
    sticky = sticky || (L[lw] & below) != 0ull;
  }
  if (guard && (sticky || (m & 1ull))) {
    m += 1ull;
    if (m >> 53) {
      m >>= 1;
      p += 1;
    }
  }
  return ldexp((double)m, p - 52 + lsb_exp);
}

// ---------------------------------------------------------- noise coefficients
// The per-iteration constants of the noise model for gain g: the exact
// reciprocal when g is a power of two whose reciprocal is a normal number, and
// whether the variance at the median floor, fl(fl(g * 1e-4) + rn2), is at
// least 2^-96 (then the square root skips its small-argument path).
__device__ __forceinline__ NoiseCoef noise_coef_for(float g, float rn2) {
  NoiseCoef c;
  c.gain = g;
  const uint32_t b = __float_as_uint(g);
  const float r = 1.0f / g;
  const bool pow2 = (b & 0x007fffffu) == 0u && ((b >> 23) & 0xffu) != 0u;
  const uint32_t rb = __float_as_uint(r);
  const bool rnormal = ((rb >> 23) & 0xffu) != 0u && ((rb >> 23) & 0xffu) != 0xffu;
  c.inv_gain = (pow2 && rnormal && r * g == 1.0f) ? r : 0.0f;
  const float gm = g * 1e-4f;
  const float vmin = gm + rn2;
  c.fast_sqrt = vmin >= 0x1p-96f ? 1 : 0;
  c.valid = 1;
  return c;
}

// ---------------------------------------------------------- passes
constexpr int kGainBins0 = 4096;  // key bits 31-20
constexpr int kGainBins = 1024;   // key bits 19-10, then 9-0
constexpr int kGainRounds = 5;
constexpr int kGainThreads = 256;
// Passes launched per iteration: 5 rounds of three, then the sums of the
// values kept after the fifth.
constexpr int kGainLaunches = 3 * kGainRounds + 1;

struct GainShared {
  unsigned int hist[kGainBins0];
  unsigned long long acc[5][256];  // by exponent: sum M (x > 0), sum M (x < 0), Mh^2, Mh Ml, Ml^2
  unsigned long long wide[4];      // (GainWork::wide)
  unsigned long long below;        // (GainWork::below)
  unsigned long long used[4];      // exponents with a non-zero accumulator
  uint64_t pos[5], neg[5], sq[10]; // the sums as wide integers
  unsigned int part[kGainThreads / 64];
  double var;
  int last, done, bin;
  uint32_t rank;
};

// The bins and exponents that a pass counts and sums in registers, around a
// value near the median (its key).
constexpr int kGainRegBins = 8, kGainRegExps = 8;
__device__ __forceinline__ void gain_windows(GainWork* g, uint32_t key) {
  const int bin = (int)(key >> 20) - kGainRegBins / 2;
  g->kbin = (uint32_t)(bin < 0 ? 0 : bin > 4096 - kGainRegBins ? 4096 - kGainRegBins : bin);
  const int e = (int)((__float_as_uint(gkey_value(key)) >> 23) & 0xffu) - (kGainRegExps - 3);
  g->ebase = e < 1 ? 1 : e;
}

// The near histogram: one bin for each key from GainWork::near0 on, in the S
// plane.  Nothing is kept there over an estimate: the passes of an estimating
// frame's iteration rewrite S everywhere after it, the one-launch iteration
// stores there what it reads itself, and each estimate clears the bins first.
constexpr int kGainNear = 16384;
// Frames of fewer pixels select instead: their passes are all latency, and the
// search of the near histogram takes as long as the two passes it saves (about
// 12 us each; from 2^20 pixels on they read the image).  4096 keys held the
// median in the last of the four rounds only, 16384 in all (sky 200 e-).
constexpr int64_t kGainNearPx = int64_t(1) << 20;
static_assert(kGainNearPx >= kGainNear, "the S plane holds the bins");
__device__ __forceinline__ unsigned int* gain_near(const FrameDev& f) {
  return (int64_t)f.h * f.w >= kGainNearPx ? reinterpret_cast<unsigned int*>(f.splane) : nullptr;
}

// Resets the frame's estimator at the start of an iteration.
__device__ __forceinline__ void gain_reset(const FrameDev& f, int it) {
  GainWork* g = f.gw;
  for (int i = threadIdx.x; i < kGainBins0; i += blockDim.x) stg(g->hist, i, 0u);
  for (int i = threadIdx.x; i < 5 * 256; i += blockDim.x) stg(&g->acc[0][0], i, 0ull);
  if (threadIdx.x < 4) stg(g->wide, threadIdx.x, 0ull);
  if (unsigned int* near = gain_near(f)) {
    typedef uint32_t z4 __attribute__((ext_vector_type(4)));
    for (int i = threadIdx.x; i < kGainNear / 4; i += blockDim.x) stg(reinterpret_cast<z4*>(near), i, z4{0u, 0u, 0u, 0u});
  }
  if (threadIdx.x < 64) {
    // the register windows of the first round: around the median of 63
    // pixels spread over the frame (any choice gives the same sums)
    const GainImage img(f, it);
    const int64_t n = (int64_t)f.h * f.w;
    const int lane = threadIdx.x;
    const uint32_t k = lane < 63 ? gkey(img.at((n - 1) * lane / 62)) : 0xffffffffu;
    int below = 0;
    for (int j = 0; j < 64; ++j) {
      const uint32_t o = (uint32_t)__shfl((int)k, j);
      below += (o < k || (o == k && j < lane)) ? 1 : 0;
    }
    if (below == 31) gain_windows(g, k);
  }
  if (threadIdx.x == 0) {
    g->klo = 0u;
    g->khi = 0xffffffffu;
    g->prefix = 0u;
    g->rank = 0u;
    g->round = 0;
    g->done = 0;
    g->near0 = 0u;
    g->found = 0;
    g->below = 0ull;
    g->blocks_done = 0u;
    g->n_prev = -1;
    g->n_cur = 0;
    g->mean = 0.0;
    g->var = 0.0;
  }
}

// Adds one value's significand and its squares' parts to the accumulators of
// its exponent.
__device__ __forceinline__ void gain_sum_lds(GainShared& sh, float x) {
  const uint32_t b = __float_as_uint(x);
  const int ex = (int)((b >> 23) & 0xffu);
  const int e = ex ? ex : 1;
  const uint32_t M = (b & 0x007fffffu) | (ex ? 0x00800000u : 0u);
  if (!M) return;
  const uint32_t mh = M >> 12, ml = M & 0xfffu;
  atomicAdd(&sh.acc[b >> 31][e], (unsigned long long)M);
  atomicAdd(&sh.acc[2][e], (unsigned long long)(mh * mh));
  atomicAdd(&sh.acc[3][e], (unsigned long long)(mh * ml));
  atomicAdd(&sh.acc[4][e], (unsigned long long)(ml * ml));
}

__device__ __forceinline__ unsigned long long wave_sum_u64(unsigned long long v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  return v;
}

// A thread's counts of the register bins, a byte each, added to the block's
// histogram: wave sums in 16-bit fields (64 lanes of at most 255).
__device__ __forceinline__ void gain_flush_counts(GainShared& sh, uint32_t kbin, unsigned long long cnt) {
  const unsigned long long lo = wave_sum_u64(cnt & 0x00ff00ff00ff00ffull);
  const unsigned long long hi = wave_sum_u64((cnt >> 8) & 0x00ff00ff00ff00ffull);
  const int lane = threadIdx.x & 63;
  if (lane < kGainRegBins) {
    const unsigned int v = (unsigned int)(((lane & 1) ? hi : lo) >> (16 * (lane >> 1))) & 0xffffu;
    if (v) atomicAdd(&sh.hist[kbin + lane], v);
  }
}

// Block-wide search of the bin holding rank `rank` in a global histogram of
// kGainThreads x PER bins (read coherently): returns the bin, -1 if there are
// no more than `rank` values, and the rank within it in *rank_in.  Every
// thread of the block calls it.
template <int PER>
__device__ __forceinline__ int gain_find_bin(GainShared& sh, const unsigned int* hist, uint32_t rank,
                                             uint32_t* rank_in) {
  const int lane = threadIdx.x & 63;
  unsigned int v[PER], mine = 0;  // bins per thread
#pragma unroll
  for (int j = 0; j < PER; ++j) v[j] = gain_atomic_load(&hist[threadIdx.x * PER + j]);
#pragma unroll
  for (int j = 0; j < PER; ++j) mine += v[j];
  unsigned int incl = mine;  // inclusive sums over the wave, then over the waves
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const unsigned int o = __shfl_up(incl, off);
    if (lane >= off) incl += o;
  }
  if (lane == 63) sh.part[threadIdx.x >> 6] = incl;
  if (threadIdx.x == 0) sh.bin = -1;
  __syncthreads();
  for (int k = 0; k < (int)(threadIdx.x >> 6); ++k) incl += sh.part[k];
  uint32_t below = incl - mine;
  if (rank >= below && rank < incl) {  // one thread's bins hold the rank
    int bin = 0;
#pragma unroll
    for (int j = 0; j < PER - 1; ++j)
      if (bin == j && below + v[j] <= rank) {
        below += v[j];
        ++bin;
      }
    sh.bin = threadIdx.x * PER + bin;
    sh.rank = rank - below;
  }
  __syncthreads();
  *rank_in = sh.rank;
  const int bin = sh.bin;
  __syncthreads();  // the next search reuses them
  return bin;
}

// Smallest (dir < 0) or largest (dir > 0) key of a binary32 value x on that
// side of the median c with |x - c| <= lim in binary64: the clipping test is
// monotone on either side of c, so the kept values form an interval.
__device__ uint32_t clip_bound(float c, double lim, int dir) {
  auto keep = [&](uint32_t k) {
    const float x = gkey_value(k);
    return fabs((double)x - (double)c) <= lim;
  };
  const double t = dir > 0 ? (double)c + lim : (double)c - lim;
  uint32_t k = gkey((float)t);
  const uint32_t kc = gkey(c);
  if (dir > 0) {
    if (k < kc) k = kc;
    while (k > kc && !keep(k)) --k;
    while (k < 0xff800000u && keep(k + 1)) ++k;  // 0xff800000: the key of +inf
  } else {
    if (k > kc) k = kc;
    while (k < kc && !keep(k)) ++k;
    while (k > 0x007fffffu && keep(k - 1)) --k;  // 0x007fffff: the key of -inf
  }
  return k;
}

// The exact sums of a round from the accumulators in LDS (one thread; only
// the exponents in use), rounded once to binary64: *s1 = sum of the values,
// *s2 = sum of their squares.
__device__ void gain_exact_sums(GainShared& sh, int ebase, double* s1, double* s2) {
  if (!(sh.used[0] | sh.used[1] | sh.used[2] | sh.used[3])) {
    // every value lay in the window: a 64-bit and a 128-bit integer
    *s1 = ldexp((double)(long long)sh.wide[0], ebase - 150);
    const unsigned long long d0 = sh.wide[1], d1 = sh.wide[2], d2 = sh.wide[3];
    const unsigned long long lo = d0 + (d1 << 32);
    unsigned long long hi = d2 + (d1 >> 32) + (lo < d0 ? 1ull : 0ull);
    int sh2 = 0;
    unsigned long long top = lo;
    if (hi) {  // the top 64 bits, a set last bit standing for any below
      const int z = __clzll((long long)hi);
      sh2 = 64 - z;
      top = z ? (hi << z) | (lo >> (64 - z)) : hi;
      if (z ? (lo << z) != 0ull : lo != 0ull) top |= 1ull;
    }
    *s2 = ldexp((double)top, 2 * ebase - 300 + sh2);
    return;
  }
  // sum x: LSB 2^-149 (exponent 1); M 2^(e-150) is M << (e-1) of it
  // sum x^2: LSB 2^-298; M^2 2^(2e-300) = (Mh^2 << 24 + Mh Ml << 13 + Ml^2) << (2e-2)
  for (int k = 0; k < 5; ++k) sh.pos[k] = sh.neg[k] = 0ull;
  for (int k = 0; k < 10; ++k) sh.sq[k] = 0ull;
  for (int k = 0; k < 4; ++k)
    for (unsigned long long bits = sh.used[k]; bits; bits &= bits - 1) {
      const int e = 64 * k + __ffsll((long long)bits) - 1;
      if (sh.acc[0][e]) big_add(sh.pos, 5, sh.acc[0][e], e - 1);
      if (sh.acc[1][e]) big_add(sh.neg, 5, sh.acc[1][e], e - 1);
      if (sh.acc[2][e]) big_add(sh.sq, 10, sh.acc[2][e], 2 * e - 2 + 24);
      if (sh.acc[3][e]) big_add(sh.sq, 10, sh.acc[3][e], 2 * e - 2 + 13);
      if (sh.acc[4][e]) big_add(sh.sq, 10, sh.acc[4][e], 2 * e - 2);
    }
  const long long w = (long long)sh.wide[0];
  if (w > 0) big_add(sh.pos, 5, (uint64_t)w, ebase - 1);
  if (w < 0) big_add(sh.neg, 5, (uint64_t)(-w), ebase - 1);
  for (int k = 0; k < 3; ++k)
    if (sh.wide[1 + k]) big_add(sh.sq, 10, sh.wide[1 + k], 2 * ebase - 2 + 32 * k);
  if (big_less(sh.pos, sh.neg, 5)) {
    big_sub(sh.neg, sh.pos, 5);
    *s1 = -big_to_double(sh.neg, 5, -149);
  } else {
    big_sub(sh.pos, sh.neg, 5);
    *s1 = big_to_double(sh.pos, 5, -149);
  }
  *s2 = big_to_double(sh.sq, 10, -298);
}

// The noise-model constants of iteration it from the final mean and
// variance: the estimated gain, or gain 1 when there is no estimate (no
// spread, or a result that is not a positive normal binary32 number).
__device__ NoiseCoef gain_final(const FrameDev& f, double mean, double var) {
  double est = 1.0;
  bool ok = false;
  if (var > 0.0) {
    const double rn = (double)f.readnoise;
    const double rn2 = rn * rn;
    const double gg = (mean + sqrt(mean * mean + 4.0 * var * rn2)) / (2.0 * var);
    const uint32_t fb = __float_as_uint((float)gg);
    const uint32_t fe = (fb >> 23) & 0xffu;
    ok = isfinite(gg) && (fb >> 31) == 0u && fe != 0u && fe != 0xffu;
    if (ok) est = gg;
  }
  NoiseCoef c = noise_coef_for((float)est, f.rn2);
  c.valid = ok ? 1 : 0;
  return c;
}

// The lower median of a round's kept values is found (its key): the next
// round's interval.  Threads 0 and 1, each one side of it.
__device__ void gain_next_round(GainWork* g, uint32_t key, double var, uint32_t klo, uint32_t khi, bool near) {
  const float med = gkey_value(key);
  const double lim = 3.0 * (var > 0.0 ? sqrt(var) : 0.0);
  const uint32_t k = clip_bound(med, lim, threadIdx.x ? +1 : -1);
  if (threadIdx.x) {
    g->khi = k < khi ? k : khi;
    return;
  }
  g->klo = k > klo ? k : klo;
  g->n_prev = g->n_cur;
  g->round = g->round + 1;
  g->prefix = 0u;
  g->rank = 0u;
  gain_windows(g, key);
  // (keys of numbers lie within [0x007fffff, 0xff800000])
  g->near0 = near && key >= (uint32_t)kGainNear ? key - (uint32_t)(kGainNear / 2) : 0u;
}

// One pass of a clipping round (P = 0: count, sums and key bits 31-20;
// 1: bits 19-10; 2: bits 9-0) by block bx of nbx over frame f's pixels.
template <int P>
__device__ __forceinline__ void gain_pass(const FrameDev& f, int it, int bx, int nbx, GainShared& sh) {
  GainWork* g = f.gw;
  // every word of the state is loaded before the first is tested
  const int done = ldg(&g->done, 0), found = ldg(&g->found, 0);
  const uint32_t klo = ldg(&g->klo, 0), khi = ldg(&g->khi, 0), prefix = ldg(&g->prefix, 0);
  const uint32_t sel_rank = ldg(&g->rank, 0);
  const double var = ldg(&g->var, 0);
  const uint32_t kbin = ldg(&g->kbin, 0), near0 = P == 0 ? ldg(&g->near0, 0) : 0u;
  const int ebase = ldg(&g->ebase, 0);
  if (done || (P > 0 && found)) return;
  constexpr int NB = P == 0 ? kGainBins0 : kGainBins;
  for (int i = threadIdx.x; i < NB; i += blockDim.x) sh.hist[i] = 0u;
  if (P == 0) {
    for (int i = threadIdx.x; i < 5 * 256; i += blockDim.x) (&sh.acc[0][0])[i] = 0ull;
    if (threadIdx.x < 4) sh.wide[threadIdx.x] = 0ull;
    if (threadIdx.x == 0) sh.below = 0ull;
  }
  __syncthreads();
  const int64_t n = (int64_t)f.h * f.w;
  const GainImage img(f, it);
  unsigned long long cnt = 0ull;       // the register bins, a byte each
  long long sum = 0;                   // of M 2^(e - ebase)
  unsigned long long sq_lo = 0ull;     // of its square: 96 bits
  unsigned int sq_hi = 0u;
  unsigned int* near = near0 ? gain_near(f) : nullptr;
  unsigned int below = 0u;             // kept values below near0
  auto take = [&](float x) __attribute__((always_inline)) {
    const uint32_t k = gkey(x);
    bool in = k - klo <= khi - klo;
    if (P == 0) {
      if (!in) return;
      const uint32_t bin = k >> 20, b = bin - kbin;
      if (b < (uint32_t)kGainRegBins)
        cnt += 1ull << (8 * b);
      else
        atomicAdd(&sh.hist[bin], 1u);
      const uint32_t bits = __float_as_uint(x);
      const int ex = (int)((bits >> 23) & 0xffu);
      const uint32_t d = (uint32_t)(ex - ebase);  // (ebase >= 1: a denormal or 0 falls out)
      if (d < (uint32_t)kGainRegExps) {
        const uint32_t Y = ((bits & 0x007fffffu) | 0x00800000u) << d;  // < 2^31
        sum += (bits >> 31) ? -(long long)Y : (long long)Y;
        const unsigned long long p = (unsigned long long)Y * Y;
        sq_lo += p;
        sq_hi += sq_lo < p ? 1u : 0u;
      } else {
        gain_sum_lds(sh, x);
      }
      if (near) {  // (uniform)
        below += k < near0 ? 1u : 0u;
        const uint32_t r = k - near0;
        if (r < (uint32_t)kGainNear) atom_add(near + r, 1u);
      }
    } else if (P == 1) {
      if (in && (k >> 20) == prefix) atomicAdd(&sh.hist[(k >> 10) & 0x3ffu], 1u);
    } else {
      if (in && (k >> 10) == prefix) atomicAdd(&sh.hist[k & 0x3ffu], 1u);
    }
  };
  // four 4-pixel loads in flight per thread
  typedef float g4u __attribute__((ext_vector_type(4), aligned(4)));
  typedef uint16_t h4u __attribute__((ext_vector_type(4), aligned(2)));
  constexpr int kLoads = 4;
  const int64_t groups = n >> 2, span = (int64_t)kGainThreads * kLoads;
  int since = 0;
  for (int64_t base = (int64_t)bx * span; base < groups; base += (int64_t)nbx * span) {
    float v[kLoads][4];
    const int64_t g0 = base + threadIdx.x;
#pragma unroll
    for (int j = 0; j < kLoads; ++j) {
      const int64_t gi = min(g0 + (int64_t)j * kGainThreads, groups - 1);
      if (img.u16) {
        const h4u u = *(const __attribute__((address_space(1))) h4u*)(img.u16 + 4 * gi);
        v[j][0] = (float)u.x, v[j][1] = (float)u.y, v[j][2] = (float)u.z, v[j][3] = (float)u.w;
      } else {
        const g4u u = *(const __attribute__((address_space(1))) g4u*)(img.f32 + 4 * gi);
        v[j][0] = u.x, v[j][1] = u.y, v[j][2] = u.z, v[j][3] = u.w;
      }
    }
#pragma unroll
    for (int j = 0; j < kLoads; ++j)
      if (g0 + (int64_t)j * kGainThreads < groups) {
#pragma unroll
        for (int b = 0; b < 4; ++b) take(v[j][b] + 0.0f);
      }
    since += 4 * kLoads;
    if (P == 0 && since > 255 - 4 * kLoads) {  // a count's byte could overflow next time
      gain_flush_counts(sh, kbin, cnt);
      cnt = 0ull;
      since = 0;
    }
  }
  if (bx == 0 && threadIdx.x < (n & 3)) take(img.at((groups << 2) + threadIdx.x));
  if (P == 0) {
    gain_flush_counts(sh, kbin, cnt);
    const unsigned long long s64 = wave_sum_u64((unsigned long long)sum);
    const unsigned long long q0 = wave_sum_u64(sq_lo & 0xffffffffull), q1 = wave_sum_u64(sq_lo >> 32);
    const unsigned long long q2 = wave_sum_u64((unsigned long long)sq_hi);
    const unsigned long long bl = wave_sum_u64((unsigned long long)below);
    if ((threadIdx.x & 63) == 0) {
      atomicAdd(&sh.wide[0], s64);
      atomicAdd(&sh.wide[1], q0);
      atomicAdd(&sh.wide[2], q1);
      atomicAdd(&sh.wide[3], q2);
      if (bl) atomicAdd(&sh.below, bl);
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < NB; i += blockDim.x)
    if (sh.hist[i]) atom_add(&g->hist[i], sh.hist[i]);
  if (P == 0)
    for (int i = threadIdx.x; i < 5 * 256; i += blockDim.x) {
      const unsigned long long v = (&sh.acc[0][0])[i];
      if (v) atom_add(&(&g->acc[0][0])[i], v);
    }
  if (P == 0 && threadIdx.x < 4 && sh.wide[threadIdx.x]) atom_add(&g->wide[threadIdx.x], sh.wide[threadIdx.x]);
  if (P == 0 && threadIdx.x == 0 && sh.below) atom_add(&g->below, sh.below);
  // The last block of the frame to finish takes the round's decisions.  Blocks
  // share nothing but device-scope atomics, so a block has published its part
  // when they are answered; a device-scope fence would write the XCD's L2 back
  // as well, once for each block.
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0) sh.last = atom_add(&g->blocks_done, 1u) == (unsigned int)(nbx - 1) ? 1 : 0;
  __syncthreads();
  if (!sh.last) return;
  if (P == 0) {
    unsigned int c = 0;
#pragma unroll
    for (int j = 0; j < NB / kGainThreads; ++j) c += gain_atomic_load(&g->hist[threadIdx.x + j * kGainThreads]);
    unsigned long long a[5];
#pragma unroll
    for (int j = 0; j < 5; ++j) a[j] = gain_atomic_load(&g->acc[j][threadIdx.x]);
    bool any = false;
#pragma unroll
    for (int j = 0; j < 5; ++j) {
      sh.acc[j][threadIdx.x] = a[j];
      any |= a[j] != 0ull;
    }
    const unsigned long long used = __ballot(any);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) c += __shfl_xor(c, off);
    if ((threadIdx.x & 63) == 0) {
      sh.used[threadIdx.x >> 6] = used;
      sh.part[threadIdx.x >> 6] = c;
    }
    if (threadIdx.x < 4) sh.wide[threadIdx.x] = gain_atomic_load(&g->wide[threadIdx.x]);
    __syncthreads();
    if (threadIdx.x == 0) {
      long long cnt = 0;
      for (int t = 0; t < kGainThreads / 64; ++t) cnt += sh.part[t];
      double s1 = 0.0, s2 = 0.0;
      gain_exact_sums(sh, ebase, &s1, &s2);
      const double mean = s1 / (double)cnt;
      const double var = s2 / (double)cnt - mean * mean;  // (of this round)
      g->mean = mean;
      g->var = var;
      sh.var = var;
      g->n_cur = cnt;
      // final after a round that clipped nothing, or after the last round
      const bool fin = cnt == g->n_prev || g->round == kGainRounds;
      if (fin) {
        f.coef[it] = gain_final(f, mean, var);
        g->done = 1;
      }
      sh.done = fin ? 1 : 0;
      sh.rank = (uint32_t)((cnt - 1) / 2);  // rank of the lower median
    }
    __syncthreads();
    if (!sh.done) {
      const uint32_t rank = sh.rank;
      uint32_t r_in = 0;
      int bin = -1;
      if (near) {
        const unsigned long long nb = gain_atomic_load(&g->below);
        __syncthreads();  // (sh.rank is read)
        if ((unsigned long long)rank >= nb)
          bin = gain_find_bin<kGainNear / kGainThreads>(sh, near, rank - (uint32_t)nb, &r_in);
        typedef uint32_t z4 __attribute__((ext_vector_type(4)));
        for (int i = threadIdx.x; i < kGainNear / 4; i += blockDim.x)
          stg(reinterpret_cast<z4*>(near), i, z4{0u, 0u, 0u, 0u});
      }
      if (bin >= 0) {
        if (threadIdx.x < 2) gain_next_round(g, near0 + (uint32_t)bin, sh.var, klo, khi, true);
        if (threadIdx.x == 0) g->found = 1;
      } else {
        __syncthreads();
        bin = gain_find_bin<kGainBins0 / kGainThreads>(sh, g->hist, rank, &r_in);
        if (threadIdx.x == 0) {
          g->prefix = (uint32_t)bin;
          g->rank = r_in;
          g->found = 0;
        }
      }
    }
    if (threadIdx.x == 0) g->below = 0ull;
  } else {
    uint32_t r_in = 0;
    const int bin = gain_find_bin<kGainBins / kGainThreads>(sh, g->hist, sel_rank, &r_in);
    const uint32_t pre = (prefix << 10) | (uint32_t)bin;
    if (P == 1) {
      if (threadIdx.x == 0) {
        g->prefix = pre;
        g->rank = r_in;
      }
    } else if (threadIdx.x < 2) {
      gain_next_round(g, pre, var, klo, khi, gain_near(f) != nullptr);
    }
  }
  __syncthreads();
  // clear the global histogram (and sums) for the next pass
  for (int i = threadIdx.x; i < NB; i += blockDim.x) stg(g->hist, i, 0u);
  if (P == 0)
    for (int i = threadIdx.x; i < 5 * 256; i += blockDim.x) stg(&g->acc[0][0], i, 0ull);
  if (P == 0 && threadIdx.x < 4) stg(g->wide, threadIdx.x, 0ull);
  if (threadIdx.x == 0) stg(&g->blocks_done, 0, 0u);
}

}  // namespace lac
