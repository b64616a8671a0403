// One whole iteration of a frame in one launch, for runs whose workspace no
// caller can look into (the library's cached one, the static scratch, a
// batch's): only the mask and the cleaned image are results there, so S, S' and
// the candidate planes need not exist, and nothing is computed where a bound
// already decides.  (The server's steps share launches between frames at
// different iterations and run the passes.)
//
// One block per tile of TH x TW output pixels.  One iteration reads the
// previous image and mask within 8 pixels of an output pixel (replacement 2,
// growths 1 + 1, objlim test 4), so a block works alone from the tile plus an
// 8-pixel halo (the region) in LDS:
//
//   1. C_k over the region (clamped coordinates): the input, with the value
//      of every pixel of the mask M_k patched in.  The input is never
//      written, and the values of mask pixels lie in two planes used in
//      turn, so every block of a launch reads only what earlier launches
//      wrote.  (The cleaned image is written, never read: all of it in
//      iteration 0, then the pixels that changed.)
//   2. Candidates S > sigclip within 4 pixels of the tile.  A bound drops
//      nearly every pixel first: with v the smallest value of the region,
//      N >= N(v) (the noise model grows with the median, and a median of the
//      region's values is at least v), and L <= 2c - min(u, d) - min(l, r)
//      up to rounding, so a pixel where that is at most 2 sigclip N(v), less
//      a margin for the rounding, has S <= sigclip.  It costs 5 operations
//      per pixel where S costs 126.  The rest (about 1 % of the pixels of
//      the workloads, twice the number of true candidates) get S exactly.
//      Where they are too many, v being a defect's, a bound on the noise of
//      each pixel's own window takes its place.
//   3. S at the pixels within 3 of a candidate, by aligned 2x2 blocks
//      sharing one median network, kept in an LDS pool (S' at the pixels
//      within 1 of a candidate reads no other).  A tile with more of them
//      than the pool holds keeps S in the frame's S plane, and one with more
//      candidates than the list forms S everywhere.
//   4. S' = S - med5(S) at the candidates and, next to one, at the pixels
//      with S > sigfrac*sigclip: G1, G2.  (The growth reads G2 only within 1
//      of a pixel of B2, and B2 is a subset of the candidates.)  Where G1
//      holds, the objlim test: B1.
//   5. Both growths, M_(k+1), the pixels whose replacement can change (mask
//      pixels within 2 of a new one) and their values, on bit rows.
//
// A tile whose region no value or mask bit changed in during the previous
// iteration would repeat that iteration's result: it is skipped.  A tile that
// changes something stamps the tiles whose regions hold it for the next
// iteration, and the first to stamp one appends it to that iteration's list.
// (Iteration 1 works on every tile: nearly all hold a change of iteration 0.)
//
// Every value that decides anything is computed by the expressions of the
// sparse path, so the results are the same bit for bit.
//
// What bounds it: the latency of a block's phases.  A block's dozen phases are
// separated by barriers, and the sparse ones (64 bound hits, 110 blocks of S,
// 17 tests, 12 replacements in a 64 x 64 tile of a star field) keep one to
// three of its four waves busy: alone on a CU such a tile takes 44 k cycles in
// iteration 0, with three others beside it 49 k, and the issue slots are half
// used.  So the LDS is cut to 40 KB and the registers to 128 for four blocks
// per CU (three blocks: 179 -> 140 us for iteration 0 of a 4096^2 frame when
// that was done), the first loads of a tile are issued together, list places
// are reserved by a scan and one atomic per wave, and work too small for the
// block is split over more lanes.  Against the chain of about seven launches
// per iteration of the sparse passes (single frames, four iterations, the
// whole call): 512^2 0.173 -> 0.088 ms, 800^2 with eight times the cosmic rays
// 0.416 -> 0.107, 2049 x 3001 separable 0.406 -> 0.181, 4096^2 0.487 -> 0.263,
// 4000 x 6500 0.637 -> 0.347, 6400 x 9600 uint16 0.727 -> 0.512.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "lacosmic_device.h"
#include "lacosmic_tiles.h"

namespace lac {

constexpr int kIterHalo = 8;     // the iteration's dependency radius
constexpr int kIterThreads = 256;
constexpr int kIterWaves = 4;    // waves per SIMD the launch bounds ask for (blocks per CU, with its LDS)

// State word of a tile: bit 0, the plane (of two) that holds its mask bits
// and values; above it, it + 1 for the iteration `it` that wrote them.  A
// block that finds a neighbour written in its own iteration knows the plane
// before: the other one, which the neighbour does not touch.  Stamp word of a
// tile for iteration it, in one of two arrays used in turn: it + 1 if that
// iteration has work for it.
__device__ __forceinline__ uint32_t* iter_state(const FrameDev& f) {
  return reinterpret_cast<uint32_t*>(f.dirty);
}
__device__ __forceinline__ uint32_t* iter_stamp(const FrameDev& f, int it) {
  return reinterpret_cast<uint32_t*>((it & 1) ? f.rs : f.r4);
}
// The next iteration's list of tiles.
struct IterList {
  int* list;
  unsigned int* count;  // its length so far
  int base;             // added to the frame's tile index
};
__device__ __forceinline__ float* iter_values(const FrameDev& f, uint32_t plane) {
  return reinterpret_cast<float*>(plane ? f.conf : f.list);
}

// Bit rows of the region: 32 columns per word, each row between two zero
// words.  One thread per word: a word's neighbours in its row give the bits
// that a horizontal dilation shifts in.
struct BitSpan {  // words ww - 1, ww, ww + 1 of a row (or of several ORed)
  uint32_t l, c, r;
};
__device__ __forceinline__ BitSpan operator|(BitSpan x, BitSpan y) {
  return BitSpan{x.l | y.l, x.c | y.c, x.r | y.r};
}
// The middle word of the span dilated by R columns.
template <int R>
__device__ __forceinline__ uint32_t span_dil(BitSpan s) {
  uint32_t o = s.c;
#pragma unroll
  for (int k = 1; k <= R; ++k)
    o |= __builtin_amdgcn_alignbit(s.c, s.l, 32 - k) | __builtin_amdgcn_alignbit(s.r, s.c, k);
  return o;
}
// n shifted up by one, the sign of x below.
__device__ __forceinline__ uint32_t sign_into(uint32_t n, float x) {
  return __builtin_amdgcn_alignbit(n, __float_as_uint(x), 31);
}
// Where two or more of three bits are set.
__device__ __forceinline__ uint32_t majority(uint32_t x, uint32_t y, uint32_t z) {
  return (x & y) | (x & z) | (y & z);
}
// Columns [lo, hi) as bits of word ww.
__device__ __forceinline__ uint32_t col_bits(int ww, int lo, int hi) {
  const int a = clampi(lo - 32 * ww, 32), b = clampi(hi - 32 * ww, 32);
  const uint32_t below_b = b >= 32 ? ~0u : (1u << b) - 1u, below_a = a >= 32 ? ~0u : (1u << a) - 1u;
  return below_b & ~below_a;
}

// Minimum and largest magnitude over a wave, in lane 63 (DPP row shifts and
// broadcasts).
__device__ __forceinline__ float vmin(float a, float b) {
  float d;
  asm("v_min_f32 %0, %1, %2" : "=v"(d) : "v"(a), "v"(b));  // no NaN quieting of its inputs
  return d;
}
__device__ __forceinline__ float vmax(float a, float b) {
  float d;
  asm("v_max_f32 %0, %1, %2" : "=v"(d) : "v"(a), "v"(b));
  return d;
}
__device__ __forceinline__ float vmin3(float a, float b, float c) {
  float d;
  asm("v_min3_f32 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
  return d;
}
__device__ __forceinline__ float vmax3_abs(float a, float b, float c) {  // of |a|, |b|, |c|
  float d;
  asm("v_max3_f32 %0, |%1|, |%2|, |%3|" : "=v"(d) : "v"(a), "v"(b), "v"(c));
  return d;
}
template <int CTRL, int ROWS>
__device__ __forceinline__ float dpp_move(float v) {
  const int b = __float_as_int(v);
  return __int_as_float(__builtin_amdgcn_update_dpp(b, b, CTRL, ROWS, 0xf, false));
}
template <int CTRL, int ROWS>
__device__ __forceinline__ void dpp_step(float& mn, float& mx) {
  mn = vmin(mn, dpp_move<CTRL, ROWS>(mn));
  const float o = dpp_move<CTRL, ROWS>(mx);
  mx = vmax3_abs(mx, o, o);
}
__device__ __forceinline__ void wave_min_max(float& mn, float& mx) {
  dpp_step<0x111, 0xf>(mn, mx);  // row_shr:1, 2, 4, 8
  dpp_step<0x112, 0xf>(mn, mx);
  dpp_step<0x114, 0xf>(mn, mx);
  dpp_step<0x118, 0xf>(mn, mx);
  dpp_step<0x142, 0xa>(mn, mx);  // row_bcast:15, 31
  dpp_step<0x143, 0xc>(mn, mx);
}
// Sums over the lanes up to each one.
__device__ __forceinline__ int wave_scan(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);  // row_shr:1, 2, 4, 8
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);  // row_bcast:15, 31
  return v + __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);
}
// n places each from a counter in LDS, by a whole wave: one atomic.  (An
// atomicAdd of different amounts is a loop over the lanes, 40 cycles each: the
// lists waited up to 2000 cycles on it.)
__device__ __forceinline__ unsigned int wave_reserve(unsigned int* counter, unsigned int n) {
  const unsigned int upto = (unsigned int)wave_scan((int)n);
  const unsigned int total = (unsigned int)__builtin_amdgcn_readlane((int)upto, 63);
  unsigned int base = 0u;
  if (total) {  // (uniform)
    if ((threadIdx.x & 63) == 0) base = atomicAdd(counter, total);
    base = (unsigned int)__builtin_amdgcn_readfirstlane((int)base);
  }
  return base + upto - n;
}
// The OR over a wave.
__device__ __forceinline__ uint32_t wave_or(uint32_t v) {
  int x = (int)v;
  x |= __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);  // as wave_scan
  x |= __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);
  x |= __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);
  x |= __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);
  x |= __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);
  x |= __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);
  return (uint32_t)__builtin_amdgcn_readlane(x, 63);
}
// Keys of n staged values: where the region holds no negative value (a
// block-uniform choice) a value's bits are its key already.
template <int N>
__device__ __forceinline__ void keys_of(int* v, bool nonneg) {
  if (!nonneg) {
#pragma unroll
    for (int k = 0; k < N; ++k) v[k] ^= (v[k] >> 31) & 0x7fffffff;
  }
}

// Unsigned order-preserving keys (bisection over the floats).
__device__ __forceinline__ uint32_t gkey_of(float v) { return (uint32_t)fkey(v) ^ 0x80000000u; }
__device__ __forceinline__ float gkey_float(uint32_t k) { return funkey((int)(k ^ 0x80000000u)); }

// The thread's index, opaque to the optimiser: what a phase derives from it is
// computed there and not kept in registers across the phases (and the tiles)
// before, whose networks need them all.
__device__ __forceinline__ int phase_tid() {
  int t = (int)threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

// Bit planes of the region.
constexpr int kBitM = 0;   // M_k, then M_(k+1)
constexpr int kBitCd = 1;  // live candidates; then the new mask pixels
constexpr int kBitD1 = 2;  // pixels within 1 of a live candidate
constexpr int kBitG1 = 3, kBitG2 = 4, kBitB1 = 5;
constexpr int kBitDead = 6;  // candidates whose objlim test fails whatever their S'
constexpr int kBitPlanes = 7;

template <int TH, int TW_>
struct alignas(16) SmemIter {
  static constexpr int RH = TH + 2 * kIterHalo, RW = TW_ + 2 * kIterHalo;
  static constexpr int QR = (RH - 4) / 2, QC = (RW - 4) / 2;  // 2x2 blocks of the S area
  static constexpr int NW = (RW + 31) / 32;                   // words of a bit row
  // Rows of the bit planes: region rows 3 .. RH - 4 (nothing reads others),
  // NW words and a zero word each, and a zero word before the first row.
  static constexpr int BR0 = 3, BROWS = RH - 2 * BR0;
  static constexpr int kPlaneWords = (BROWS * (NW + 1) + 1 + 3) / 4 * 4;
  // 2x2 blocks of S and list items held at once: what the four blocks per CU
  // leave of its LDS (a denser tile keeps S in global memory), or, on small
  // tiles, every block there is
  static constexpr int kQuadCap = TW_ == 64 ? 256 : QR * QC, kItemCap = TW_ == 64 ? 512 : 1024;
  typedef typename std::conditional<(kQuadCap <= 256), uint8_t, uint16_t>::type QIndex;
  float c[RH][RW];        // C_k at the clamped region coordinates
  float s4[kQuadCap][4];  // S of the marked 2x2 blocks (before that: open candidates)
  uint32_t bits[kBitPlanes][kPlaneWords];
  uint64_t qbits[QR];      // the 2x2 blocks of the S area to evaluate, a bit row per block row
  uint16_t lst[kItemCap];  // items: region cell index
  QIndex qmap[QR * QC];    // a block's index in s4, by position
  float wmin[kIterThreads / 64], wmax[kIterThreads / 64];
  float mn, nmin, thr;  // the region's smallest value, the noise there, the candidates' bound
  float margin;         // of that bound; +inf where it does not apply
  unsigned int cnt, nopen, n2, fresh, unrep;
  unsigned int zones;  // bit 3 zy + zx: 3x3 zones of the tile (8 pixels along the edges) with a change
  int any_b1, live;
  __device__ __forceinline__ static int at(int r, int ww) { return (r - BR0) * (NW + 1) + 1 + ww; }
  __device__ __forceinline__ BitSpan span(int plane, int r, int ww) const {
    const uint32_t* p = bits[plane] + at(r, ww) - 1;
    return BitSpan{p[0], p[1], p[2]};
  }
  __device__ __forceinline__ uint32_t& word(int plane, int r, int ww) { return bits[plane][at(r, ww)]; }
  __device__ __forceinline__ uint32_t word(int plane, int r, int ww) const { return bits[plane][at(r, ww)]; }
  __device__ __forceinline__ bool bit(int plane, int r, int q) const {
    return ((word(plane, r, q >> 5) >> (q & 31)) & 1u) != 0u;
  }
  __device__ __forceinline__ void set(int plane, int r, int q) {
    atomicOr(&word(plane, r, q >> 5), 1u << (q & 31));
  }
  // The blocks within 3 pixels of live candidate (r, q), and the pixels
  // within 1 of it.
  __device__ __forceinline__ void mark_near(int r, int q) {
    const int c0 = (q - 3) >> 1;  // of 4 block columns, counted from region column 0
    const uint64_t m = ((0xfull << c0) >> 1) & ((1ull << QC) - 1ull);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int br = ((r - 3) >> 1) - 1 + k;
      if (br >= 0 && br < QR) atomicOr((unsigned long long*)&qbits[br], (unsigned long long)m);
    }
    const int c1 = q - 1, sh = c1 & 31;
#pragma unroll
    for (int k = -1; k <= 1; ++k) {
      uint32_t* p = &word(kBitD1, r + k, c1 >> 5);
      atomicOr(p, 7u << sh);
      if (sh > 29) atomicOr(p + 1, 7u >> (32 - sh));
    }
  }
};

// What 2c - min(u, d) - min(l, r) has to exceed for S > sigclip where the
// noise is at least n (step 2).
__device__ __forceinline__ float candidate_bound(float sigclip, float n, float margin) {
  return (2.0f * sigclip) * n * (1.0f - 0x1p-14f) - margin;
}

// S (and N) at one region cell (2 or more inside the region).
template <typename SM>
__device__ __forceinline__ float iter_s(const SM& s, const FrameDev& f, const NoiseCoef& nc, int y,
                                        int x, bool nonneg, float& N) {
  int v[25];
#pragma unroll
  for (int a = 0; a < 5; ++a)
#pragma unroll
    for (int b = 0; b < 5; ++b) v[a * 5 + b] = __float_as_int(s.c[y - 2 + a][x - 2 + b]);
  const float L = lap_edge(__int_as_float(v[12]), __int_as_float(v[7]), __int_as_float(v[17]),
                           __int_as_float(v[11]), __int_as_float(v[13]));
  keys_of<25>(v, nonneg);
  const int m = med25_of(v, f.sepmed);
  N = noise_fast(nc) ? noise_from_med<true>(m, nc, f.rn2) : noise_from_med<false>(m, nc, f.rn2);
  return L / (2.0f * N);
}

// Position of set bit n (from 0) of hi:lo.
__device__ __forceinline__ int nth_bit(uint32_t lo, uint32_t hi, int n) {
  const int c = __popc(lo);
  int pos = n >= c ? 32 : 0;
  uint32_t m = n >= c ? hi : lo;
  n -= n >= c ? c : 0;
#pragma unroll
  for (int k = 16; k > 0; k >>= 1) {
    const int below = __popc(m & ((1u << k) - 1u));
    const bool up = n >= below;
    n -= up ? below : 0;
    m >>= up ? k : 0;
    pos += up ? k : 0;
  }
  return pos;
}

// S at PX pixels from region cell (y, x) on (2 or more inside the region): the
// pixel, it and the next of the row, or the 2x2 block; cells outside the frame
// get values nothing reads.
template <int PX, typename SM>
__device__ __forceinline__ void iter_block(const SM& s, const FrameDev& f, const NoiseCoef& nc, int y,
                                           int x, bool nonneg, float* S) {
  if (PX == 1) {
    float N;
    S[0] = iter_s(s, f, nc, y, x, nonneg, N);
    return;
  }
  constexpr int ROWS = PX == 4 ? 6 : 5;
  int v[36];
#pragma unroll
  for (int a = 0; a < 6; ++a)
#pragma unroll
    for (int b = 0; b < 6; ++b) v[a * 6 + b] = a < ROWS ? __float_as_int(s.c[y - 2 + a][x - 2 + b]) : 0;
#pragma unroll
  for (int q = 0; q < PX; ++q) {
    const int k = ((q >> 1) + 2) * 6 + (q & 1) + 2;
    S[q] = lap_edge(__int_as_float(v[k]), __int_as_float(v[k - 6]), __int_as_float(v[k + 6]),
                    __int_as_float(v[k - 1]), __int_as_float(v[k + 1]));
  }
  keys_of<36>(v, nonneg);
  int m[4];  // (with PX == 2 nothing uses the second row's, which are not formed)
  med25_block(v, m, f.sepmed);
  if (noise_fast(nc)) {
#pragma unroll
    for (int q = 0; q < PX; ++q) S[q] = S[q] / (2.0f * noise_from_med<true>(m[q], nc, f.rn2));
  } else {
#pragma unroll
    for (int q = 0; q < PX; ++q) S[q] = S[q] / (2.0f * noise_from_med<false>(m[q], nc, f.rn2));
  }
}

// On tiles at the frame's edge a window clamps on the frame: its rows and
// columns outside take the values of the nearest one inside.  For the K x K
// window v around frame pixel (gy, gx).
template <int K>
__device__ __forceinline__ void clamp_window(int* v, const FrameDev& f, int gy, int gx) {
  constexpr int R = K / 2;
#pragma unroll
  for (int a = R - 1; a >= 0; --a) {  // from the centre outwards
    const bool up = gy - R + a < 0, dn = gy + R - a >= f.h;
    const bool lf = gx - R + a < 0, rt = gx + R - a >= f.w;
#pragma unroll
    for (int b = 0; b < K; ++b) {
      v[a * K + b] = up ? v[(a + 1) * K + b] : v[a * K + b];
      v[(K - 1 - a) * K + b] = dn ? v[(K - 2 - a) * K + b] : v[(K - 1 - a) * K + b];
    }
#pragma unroll
    for (int b = 0; b < K; ++b) {
      v[b * K + a] = lf ? v[b * K + a + 1] : v[b * K + a];
      v[b * K + K - 1 - a] = rt ? v[b * K + K - 2 - a] : v[b * K + K - 1 - a];
    }
  }
}

// S's 5x5 window around region cell (y, x), as keys (S >= +0: its bits are its
// key): from the pool, where it lies in 3x3 blocks, or from the S plane.
template <typename SM>
__device__ __forceinline__ void iter_pool_window(const SM& s, const FrameDev& f, int y, int x, int ry0, int rx0,
                                                 bool inner, int* v) {
  {
    const int q0 = (((y - 2) >> 1) - 1) * SM::QC + ((x - 2) >> 1) - 1;
    float w[36];
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        const float4 q = *reinterpret_cast<const float4*>(s.s4[s.qmap[q0 + a * SM::QC + b]]);
        w[(2 * a) * 6 + 2 * b] = q.x;
        w[(2 * a) * 6 + 2 * b + 1] = q.y;
        w[(2 * a + 1) * 6 + 2 * b] = q.z;
        w[(2 * a + 1) * 6 + 2 * b + 1] = q.w;
      }
    const bool oy = (y & 1) != 0, ox = (x & 1) != 0;  // the window starts at an odd cell
#pragma unroll
    for (int k = 0; k < 30; ++k) w[k] = oy ? w[k + 6] : w[k];
#pragma unroll
    for (int a = 0; a < 5; ++a)
#pragma unroll
      for (int b = 0; b < 5; ++b)
        v[a * 5 + b] = __float_as_int(ox ? w[a * 6 + b + 1] : w[a * 6 + b]);
  }
  if (!inner) clamp_window<5>(v, f, ry0 + y, rx0 + x);
}
__device__ __forceinline__ void iter_plane_window(const FrameDev& f, int gy, int gx, int* v) {
  const int* S = reinterpret_cast<const int*>(f.splane);
#pragma unroll
  for (int a = 0; a < 5; ++a) {
    const int64_t row = (int64_t)clampi(gy - 2 + a, f.h - 1) * f.w;
#pragma unroll
    for (int b = 0; b < 5; ++b) v[a * 5 + b] = ldg(S, row + clampi(gx - 2 + b, f.w - 1));
  }
}

// The objlim test's parts at region cell (y, x): med3 there, and the test's
// outcome for a given med7 and S'.  The outcome can only go from failing to
// holding as med7 grows or as S' grows (rounding keeps the order), so bounds
// on either decide it.
template <typename SM>
__device__ __forceinline__ float iter_med3(const SM& s, const FrameDev& f, int y, int x, bool nonneg) {
  int v9[9];
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) v9[a * 3 + b] = __float_as_int(s.c[y - 1 + a][x - 1 + b]);
  keys_of<9>(v9, nonneg);
  return funkey(med9_of(v9, f.sepmed));
}
__device__ __forceinline__ bool objlim_holds(const FrameDev& f, float m3, float m7, float N, float spv) {
  const float fr = (m3 - m7) / N;
  const float fn = (fr > 0.01f) ? fr : 0.01f;
  return (spv / fn) > f.objlim;
}
// Whether med7 of med3 at (y, x) is at most t, without forming any median, by
// the 4 lanes of a quad that share the arguments (all get the answer).  A
// median is at most t when more than half its values are, so the 9x9 patch
// becomes rows of bits [C <= t], the 3x3 majorities come from bit-sliced sums
// of three rows, and their number in the 7x7 window decides.  Lane k forms
// rows 2k to 2k + 2 of the patch and rows 2k and 2k + 1 of the majorities:
// about 140 operations, where one lane alone took 390 (and the medians
// themselves 1100) and the tile's other lanes waited for it.  A lane per row
// took 90, but 16 lanes each: a bright star's 100 pixels needed 7 rounds.
template <typename SM>
__device__ __forceinline__ bool iter_med7_le(const SM& s, const FrameDev& f, int y, int x, int ry0,
                                             int rx0, bool inner, float t) {
  const int lane = threadIdx.x & 63, k2 = 2 * (lane & 3);
  uint32_t one[4], two[4];  // per row and column: the sum of 3 neighbours' bits
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const float* p = &s.c[y - 4 + k2 + a][x - 4];
    uint32_t r = 0u;
#pragma unroll
    for (int b = 8; b >= 0; --b) r = r + r + (p[b] <= t ? 1u : 0u);
    const uint32_t r1 = r >> 1, r2 = r >> 2;
    one[a] = r ^ r1 ^ r2;
    two[a] = (r & r1) | (r & r2) | (r1 & r2);
  }
  // row 2k + 3 is the next lane's second (quad_perm 1, 2, 3, 3; lane 3 has no
  // use for it)
  one[3] = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)one[1], 0xf9, 0xf, 0xf, false);
  two[3] = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)two[1], 0xf9, 0xf, 0xf, false);
  uint32_t le[2];  // [med3 <= t] of the 7 positions of rows k2, k2 + 1, bit b: column b
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    const uint32_t p0 = two[a], p1 = two[a + 1], p2 = two[a + 2];
    const uint32_t mj = (p0 & p1) | (p0 & p2) | (p1 & p2);
    le[a] = mj;
    if (!f.sepmed) {  // (separable: the median of the three row medians)
      // 5 or more of 9: ones s1 + twos (p0 + p1 + p2 + c1) * 2
      const uint32_t o0 = one[a], o1 = one[a + 1], o2 = one[a + 2];
      const uint32_t s1 = o0 ^ o1 ^ o2, c1 = (o0 & o1) | (o0 & o2) | (o1 & o2);
      const uint32_t px = p0 ^ p1 ^ p2, par = px ^ c1, car = px & c1;
      le[a] = (mj & car) | ((mj ^ car) & (par | s1));
    }
  }
  if (!inner) {  // positions outside the frame take the nearest one inside
    const int gy = ry0 + y, gx = rx0 + x;
    const int up = max(0, 3 - gy), dn = 6 - max(0, gy + 3 - (f.h - 1));
    const uint32_t own0 = le[0], own1 = le[1];
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      const int row = min(max(k2 + a, up), dn), from = (lane & 60) + (row >> 1);
      const uint32_t e = (uint32_t)__shfl((int)own0, from), o = (uint32_t)__shfl((int)own1, from);
      le[a] = (row & 1) ? o : e;
    }
    const int lf = max(0, 3 - gx), rt = 6 - max(0, gx + 3 - (f.w - 1));  // first and last column inside
    const uint32_t lm = (1u << lf) - 1u, rm = 0x7fu & ~((2u << rt) - 1u);
#pragma unroll
    for (int a = 0; a < 2; ++a)
      le[a] = (le[a] & ~(lm | rm)) | (((le[a] >> lf) & 1u) ? lm : 0u) | (((le[a] >> rt) & 1u) ? rm : 0u);
  }
  int n0 = __popc(le[0] & 0x7fu), n1 = k2 == 6 ? 0 : __popc(le[1] & 0x7fu);
  if (f.sepmed) {
    n0 = n0 >= 4 ? 1 : 0;
    n1 = n1 >= 4 ? 1 : 0;
  }
  int n = n0 + n1;
  n += __builtin_amdgcn_update_dpp(0, n, 0xb1, 0xf, 0xf, false);  // quad_perm 1, 0, 3, 2
  n += __builtin_amdgcn_update_dpp(0, n, 0x4e, 0xf, 0xf, false);  // quad_perm 2, 3, 0, 1
  return n >= (f.sepmed ? 4 : 25);
}

// The objlim test at region cell (y, x) where the smallest med7 and N there
// can be do not decide it: it holds unless med7 <= limit.
template <typename SM>
__device__ __forceinline__ float iter_objlim(const SM& s, const FrameDev& f, const NoiseCoef& nc, int y,
                                             int x, bool nonneg, float m3, float spv) {
  float N;
  (void)iter_s(s, f, nc, y, x, nonneg, N);
  // the largest med7 for which the test still fails: its value without
  // rounding is m3 - d
  const float d = N * (spv / f.objlim), t = m3 - d, e = (fabsf(m3) + d) * 0x1p-21f;
  // (or, where that overflows, anywhere among the floats)
  const bool near = !objlim_holds(f, m3, t - e, N, spv) && objlim_holds(f, m3, t + e, N, spv);
  if (!near && objlim_holds(f, m3, s.mn, N, spv)) return __int_as_float(0xff800000);
  uint32_t fails = gkey_of(near ? t - e : s.mn), holds = near ? gkey_of(t + e) : 0xff800000u;
#pragma unroll 1
  while (holds - fails > 1u) {
    const uint32_t mid = fails + ((holds - fails) >> 1);
    if (objlim_holds(f, m3, gkey_float(mid), N, spv))
      holds = mid;
    else
      fails = mid;
  }
  return gkey_float(fails);
}

// The tiles of a frame.
template <int TH, int TW_>
struct IterGrid {
  int tiles_x, tiles_y;
  __device__ __forceinline__ explicit IterGrid(const FrameDev& f)
      : tiles_x((f.w + TW_ - 1) / TW_), tiles_y((f.h + TH - 1) / TH) {}
  // Index of neighbour k (0 .. 8, row-major) of tile (ty, tx), or -1.
  __device__ __forceinline__ int neighbour(int ty, int tx, int k) const {
    const int qy = ty + k / 3 - 1, qx = tx + k % 3 - 1;
    return qy >= 0 && qy < tiles_y && qx >= 0 && qx < tiles_x ? qy * tiles_x + qx : -1;
  }
};

// The iteration on one tile, by kIterThreads threads; every barrier is
// block-uniform.  news: 0 if the iteration does not run (looked at only when
// the first loads are on their way).
template <int TH, int TW_>
__device__ __forceinline__ void tile_iter(const FrameDev& f, int it, int tile, const IterList& next, unsigned long long news,
                                          SmemIter<TH, TW_>& s) {
  using SM = SmemIter<TH, TW_>;
  constexpr int NT = kIterThreads, RH = SM::RH, RW = SM::RW, QR = SM::QR, QC = SM::QC, NW = SM::NW;
  constexpr int HL = kIterHalo, QCAP = SM::kQuadCap, ICAP = SM::kItemCap;
  static_assert(TW_ == 32 || TW_ == 64, "a tile row is a half or a whole bit-plane word");
  static_assert(SM::BROWS * NW <= NT && TH % 2 == 0, "one thread per word of the bit rows");
  int tid = phase_tid();
  const int lane = tid & 63;
  const int h = f.h, w = f.w;
  const IterGrid<TH, TW_> grid(f);
  const int ty = tile / grid.tiles_x, tx = tile - ty * grid.tiles_x;
  const int y0 = ty * TH, x0 = tx * TW_;
  const int ry0 = y0 - HL, rx0 = x0 - HL;
  // Everything the tile starts from is read at once (each load is a round trip
  // to memory, and one that waits for another's answer makes two): the state
  // words, both planes' mask words, and the input.
  uint32_t state = 0u;
  if (it > 0) {
    const int n = grid.neighbour(ty, tx, lane < 9 ? lane : 4);
    state = __hip_atomic_load(gp(iter_state(f) + max(n, 0)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  const bool inner = ry0 >= 0 && rx0 >= 0 && ry0 + RH <= h && rx0 + RW <= w;
  const int fc0 = rx0 < 0 ? -rx0 : 0, fc1 = min(RW, w - rx0);  // region columns inside the frame
  auto row_in = [&](int r) __attribute__((always_inline)) { return ry0 + r >= 0 && ry0 + r < h; };
  int wr = tid / NW + SM::BR0, ww = tid % NW;  // this thread's word of the bit rows
  bool wt = tid < SM::BROWS * NW;
  auto next_phase = [&]() __attribute__((always_inline)) {
    tid = phase_tid();
    wr = tid / NW + SM::BR0;
    ww = tid % NW;
    wt = tid < SM::BROWS * NW;
  };

  // ---- 1. stage C_k and M_k
  const int mr = tid / NW, mq = tid - mr * NW;  // this thread's word of M_k
  static_assert(RH * NW <= NT, "one thread per word of M_k");
  typedef typename std::conditional<TW_ == 64, uint64_t, uint32_t>::type MWord;
  const bool mrow = it > 0 && mr < RH && row_in(mr);
  MWord mown[2] = {0, 0}, mside[2] = {0, 0};  // by plane: the tile's own columns, and 8 of a neighbour
  if (mrow) {
    const int side = mq == 0 ? tx - 1 : tx + 1;
    const bool beside = (mq == 0 || mq == NW - 1) && side >= 0 && side < grid.tiles_x;
    const int64_t at = (int64_t)(ry0 + mr) * f.wpr * (TW_ == 64 ? 1 : 2);
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const MWord* m = reinterpret_cast<const MWord*>(f.mbits[p]);
      mown[p] = ldg(m, at + tx);
      if (beside) mside[p] = ldg(m, at + side);
    }
  }
  // C4 threads per row of 4 pixels each, RP rows at a time
  constexpr int C4 = RW / 4, RP = NT / C4, K = (RH + RP - 1) / RP;
  typedef uint16_t h4u __attribute__((ext_vector_type(4), aligned(2)));
  const int r0 = tid / C4, q0 = 4 * (tid - r0 * C4);
  const float* src = f.img;
  const uint16_t* src16 = f.img16;
  uint4 raw[K];
  if (inner) {
    const uint32_t o0 = (uint32_t)(r0 * w + q0), step = (uint32_t)(RP * w);  // from the region's corner
    const int64_t corner = (int64_t)ry0 * w + rx0;
    // (threads and rows past the region load its first rows again)
    auto at = [&](int k) __attribute__((always_inline)) -> uint32_t {
      return (r0 + k * RP < RH) ? o0 + (uint32_t)k * step : o0;
    };
    if (src16) {
      const uint16_t* base = src16 + corner;
#pragma unroll
      for (int k = 0; k < K; ++k) {
        const h4u v = *(const __attribute__((address_space(1))) h4u*)(base + at(k));
        const uint2 u = __builtin_bit_cast(uint2, v);
        raw[k].x = u.x;
        raw[k].y = u.y;
      }
    } else {
      const float* base = src + corner;
#pragma unroll
      for (int k = 0; k < K; ++k)
        raw[k] = __builtin_bit_cast(uint4, (f4u) * (const __attribute__((address_space(1))) f4u*)(base + at(k)));
    }
  } else {  // clamped on the frame, pixel by pixel
    int cx[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) cx[b] = clampi(rx0 + q0 + b, w - 1);
    auto row = [&](int k) __attribute__((always_inline)) {
      return (int64_t)clampi(ry0 + min(r0 + k * RP, RH - 1), h - 1) * w;
    };
    if (src16) {  // (chosen per load instead, each load would wait for the one before)
#pragma unroll
      for (int k = 0; k < K; ++k) {
        const uint16_t* p = src16 + row(k);
        raw[k] = uint4{ldg(p, cx[0]), ldg(p, cx[1]), ldg(p, cx[2]), ldg(p, cx[3])};
      }
    } else {
#pragma unroll
      for (int k = 0; k < K; ++k) {
        const uint32_t* p = reinterpret_cast<const uint32_t*>(src + row(k));
        raw[k] = uint4{ldg(p, cx[0]), ldg(p, cx[1]), ldg(p, cx[2]), ldg(p, cx[3])};
      }
    }
  }
  if (tid == 0) {
    s.cnt = 0u;
    s.nopen = 0u;
    s.fresh = 0u;
    s.unrep = 0u;
    s.zones = 0u;
    s.any_b1 = 0;
    s.live = 0;
  }
  uint32_t st[9];  // planes of the 3x3 tiles after the previous iteration
  if (it > 0) {
    const uint32_t p = (state & 1u) ^ ((state >> 1) == (uint32_t)(it + 1) ? 1u : 0u);
#pragma unroll
    for (int k = 0; k < 9; ++k) st[k] = (uint32_t)__builtin_amdgcn_readlane((int)p, k);
  }
  const uint32_t plane = it > 0 ? st[4] : 1u;  // this iteration writes plane ^ 1
  if (news == 0ull) return;
  uint32_t mword = 0u;  // M_k: word mq of region row mr
  if (mrow) {
    const uint32_t sl = mr < HL ? st[0] : mr < HL + TH ? st[3] : st[6];
    const uint32_t sc = mr < HL ? st[1] : mr < HL + TH ? st[4] : st[7];
    const uint32_t sr = mr < HL ? st[2] : mr < HL + TH ? st[5] : st[8];
    const uint64_t cw = sc ? mown[1] : mown[0];
    const uint64_t dw = (mq == 0 ? sl : sr) ? mside[1] : mside[0];
    if (mq == 0) mword = (uint32_t)((dw >> (TW_ - 8)) & 0xffull) | ((uint32_t)cw << 8);
    if (mq == NW - 1) mword = (uint32_t)(cw >> (TW_ - 8)) | ((uint32_t)(dw & 0xffull) << 8);
    if (NW == 3 && mq == 1) mword = (uint32_t)(cw >> 24);
  }
  float mn = __int_as_float(0x7f800000), mx = 0.0f;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int r = r0 + k * RP;
    float a, b, c, d;
    if (!src16) {
      a = __uint_as_float(raw[k].x), b = __uint_as_float(raw[k].y);
      c = __uint_as_float(raw[k].z), d = __uint_as_float(raw[k].w);
    } else if (inner) {
      a = (float)(raw[k].x & 0xffffu), b = (float)(raw[k].x >> 16);
      c = (float)(raw[k].y & 0xffffu), d = (float)(raw[k].y >> 16);
    } else {
      a = (float)raw[k].x, b = (float)raw[k].y, c = (float)raw[k].z, d = (float)raw[k].w;
    }
    if (RP * C4 != NT && r0 >= RP) continue;
    if (K * RP != RH && r >= RH) continue;
    a += 0.0f;  // -0 becomes +0
    b += 0.0f;
    c += 0.0f;
    d += 0.0f;
    mn = vmin3(vmin3(mn, a, b), c, d);
    mx = vmax3_abs(vmax3_abs(mx, a, b), c, d);
    *reinterpret_cast<float4*>(&s.c[r][q0]) = float4{a, b, c, d};
  }
  if (!inner)  // edge tiles read blocks no one lists (and drop what they hold)
    for (int i = tid; i < QR * QC; i += NT) s.qmap[i] = 0;
  // the other planes start empty, the words beside each row stay zero
  for (int i = tid; i < kBitPlanes * SM::kPlaneWords / 4; i += NT)
    reinterpret_cast<uint4*>(&s.bits[0][0])[i] = uint4{0u, 0u, 0u, 0u};
  if (tid < QR) s.qbits[tid] = 0ull;
  __syncthreads();
  if (it > 0) {
    // the values of M_k's pixels replace the input's
    auto value_of = [&](int r, int q) __attribute__((always_inline)) -> float {  // a cell in the frame
      const int k = (r < HL ? 0 : r < HL + TH ? 3 : 6) + (q < HL ? 0 : q < HL + TW_ ? 1 : 2);
      uint32_t p = 0;
#pragma unroll
      for (int j = 0; j < 9; ++j) p = (j == k) ? st[j] : p;
      return ldg((const float*)iter_values(f, p), (int64_t)(ry0 + r) * w + rx0 + q);
    };
    if (mr >= SM::BR0 && mr < SM::BR0 + SM::BROWS) s.word(kBitM, mr, mq) = mword;
    const unsigned int mbase = wave_reserve(&s.cnt, (unsigned int)__popc(mword));
    __syncthreads();
    const unsigned int n = s.cnt;
    for (unsigned int c0 = 0; c0 < n; c0 += ICAP) {  // listed, then one thread each
      unsigned int at = mbase - c0;
      for (uint32_t bits = mword; bits; bits &= bits - 1, ++at)
        if (at < (unsigned int)ICAP) s.lst[at] = (uint16_t)(mr * RW + 32 * mq + __ffs((int)bits) - 1);
      __syncthreads();
      for (unsigned int j = tid; j < min(n - c0, (unsigned int)ICAP); j += NT) {
        const int i = s.lst[j], r = i / RW, q = i - r * RW;
        const float v = value_of(r, q);
        mn = vmin(mn, v);
        s.c[r][q] = v;
      }
      __syncthreads();
    }
    if (!inner && n) {  // a cell outside the frame holds the value of its clamped pixel
      for (int i = tid; i < RH * RW; i += NT) {
        const int r = i / RW, q = i - r * RW;
        const int cr = clampi(ry0 + r, h - 1) - ry0, cq = clampi(rx0 + q, w - 1) - rx0;
        if (cr != r || cq != q) s.c[r][q] = s.c[cr][cq];
      }
    }
  }
  wave_min_max(mn, mx);
  next_phase();
  if ((tid & 63) == 63) {
    s.wmin[tid >> 6] = mn;
    s.wmax[tid >> 6] = mx;
  }
  const NoiseCoef nc = noise_coef(f, it);
  const float sigclip = f.sigclip, lo = f.lo;
  __syncthreads();
  // ---- 2. candidates.  A pixel can have S > sigclip only where
  // 2c - min(u, d) - min(l, r) > thr.  The margin: L and the bound are sums
  // of a few values of magnitude at most 16 M (M the region's largest), each
  // rounded once, which moves them by less than 2^-18 M together; the
  // products of the noise model and of S round by less than 2^-20 each.
  // Where the bound's own arithmetic could over- or underflow, or a value is
  // not finite, every pixel is tested exactly (thr = -inf).
  if (tid < 64) {  // one wave for the block
    if (tid == 0) s.cnt = 0u;
    mn = vmin(vmin3(s.wmin[0], s.wmin[1], s.wmin[2]), s.wmin[3]);
    const float M = vmax3_abs(vmax3_abs(s.wmax[0], s.wmax[1], s.wmax[2]), s.wmax[3], s.wmax[3]);
    const float nmin = noise_from_med<false>(fkey(mn), nc, f.rn2);  // no noise in the region is smaller
    const bool sane = nc.fast_sqrt && nc.gain >= 0x1p-30f && nc.gain <= 0x1p30f && sigclip >= 0x1p-30f &&
                      sigclip <= 0x1p30f && M <= 0x1p90f && mn <= M;
    const float margin = M * 0x1p-16f, t = candidate_bound(sigclip, nmin, margin);
    if (tid == 0) {
      s.mn = mn;
      s.margin = sane ? margin : __int_as_float(0x7f800000);
      s.nmin = nmin;
      s.thr = (sane && t > 0.0f) ? t : __int_as_float(0xff800000);
      if (!(M <= 0x1.fffffep127f)) atom_or(f.status, 1);
    }
  }
  // A lane per group of 4 columns, whole rows of the region side by side in a
  // wave: the columns beside a group come from the lanes beside it.  (The
  // first and last group of a row have no pixel to test.)  Reading them from
  // LDS, a word in four of a bank, cost more than the rows themselves.
  // Each lane's rows are pairs far apart, so that a star's pixels, listed
  // lane by lane below, are spread over several lanes.
  constexpr int PG = RW / 4, PRUNS = 64 / PG, PALL = NT / 64 * PRUNS;  // row pairs at once
  constexpr int PP = (TH + 8) / (2 * PALL), PR = 2 * PP;               // a lane's pairs, rows
  static_assert(PR * PALL == TH + 8 && 4 * PR <= 32, "the waves share the rows evenly");
  uint32_t hits = 0;  // pixel b of row k: bit 4 PR - 1 - (4 k + b)
  const int run = min((tid & 63) / PG, PRUNS - 1), pg = (tid & 63) - run * PG;
  const int px0 = 4 * pg, py0 = 4 + 2 * ((tid >> 6) * PRUNS + run);
  auto prow = [&](int k) __attribute__((always_inline)) { return py0 + (k >> 1) * (2 * PALL) + (k & 1); };
  __syncthreads();
  const float thr = s.thr;
  const bool nonneg = s.mn >= 0.0f;
  {
#pragma unroll
    for (int j = 0; j < PP; ++j) {
      const int y = prow(2 * j);
      float4 up = *reinterpret_cast<const float4*>(&s.c[y - 1][px0]);
      float4 cu = *reinterpret_cast<const float4*>(&s.c[y][px0]);
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const float4 dn = *reinterpret_cast<const float4*>(&s.c[y + k + 1][px0]);
        const float l = dpp_move<0x138, 0xf>(cu.w), r = dpp_move<0x130, 0xf>(cu.x);  // wave_shr:1, wave_shl:1
        const float e0 = __builtin_fmaf(2.0f, cu.x, -(vmin(up.x, dn.x) + vmin(l, cu.y)));
        const float e1 = __builtin_fmaf(2.0f, cu.y, -(vmin(up.y, dn.y) + vmin(cu.x, cu.z)));
        const float e2 = __builtin_fmaf(2.0f, cu.z, -(vmin(up.z, dn.z) + vmin(cu.y, cu.w)));
        const float e3 = __builtin_fmaf(2.0f, cu.w, -(vmin(up.w, dn.w) + vmin(cu.z, r)));
        hits = hits + hits + (!(e0 <= thr) ? 1u : 0u);
        hits = hits + hits + (!(e1 <= thr) ? 1u : 0u);
        hits = hits + hits + (!(e2 <= thr) ? 1u : 0u);
        hits = hits + hits + (!(e3 <= thr) ? 1u : 0u);
        up = cu;
        cu = dn;
      }
    }
    if ((tid & 63) >= PG * PRUNS || pg == 0 || pg == PG - 1) hits = 0u;
    if (!inner && hits) {  // pixels of the frame only
#pragma unroll
      for (int k = 0; k < PR; ++k)
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          const int q = px0 + b;
          if (!row_in(prow(k)) || q < fc0 || q >= fc1) hits &= ~(1u << (4 * PR - 1 - (4 * k + b)));
        }
    }
  }
  unsigned int hbase = wave_reserve(&s.cnt, (unsigned int)__popc(hits));
  __syncthreads();
  unsigned int npc = s.cnt;
  // The smallest value says little where it is a dead pixel's or a border's:
  // one zero pixel among 1e4 of a CMOS sky raises the hits of a tile from 77 to
  // 950, and S at each costs a median.  So where the hits exceed the list, those
  // whose median must reach a level v typical of the tile -- 13 of the window's
  // 25 values do, or, separable, 3 values of 3 rows -- are held to the noise at
  // v.  Any v is right; a median of largest minima of 16 x 2 pixels passes dead
  // pixels, columns and borders by, and stars (950 -> 24 hits; 2050 -> 160 with
  // a dead column every 64).  About 7000 cycles of a tile with three others on
  // its CU, none on tiles without defects.  (6400 x 9600 uint16, 1e-3 of the
  // pixels zero: 1.11 -> 0.66 ms, the sparse passes 0.71.  Small tiles have few
  // pixels: their hits cost less than this.)
  if (TW_ == 64 && __builtin_expect(npc > (unsigned int)ICAP, 0)) {  // (uniform)
    // in the pool: a bit for each of the region's cells, the bit rows of the
    // medians below v, and the values v is taken from
    uint32_t* cells = reinterpret_cast<uint32_t*>(s.s4);
    uint32_t* low_med = cells + RH * RW / 32 + 4;
    float* levels = reinterpret_cast<float*>(low_med + RH * NW);
    static_assert(RH * RW / 32 <= NT && RH * RW / 8 + 16 + RH * NW * 4 + 64 <= (int)sizeof(s.s4), "they fit");
    next_phase();
    float v = __int_as_float(0xff800000);
#pragma unroll
    for (int j = 0; j < PP; ++j) {
      const float4 x = *reinterpret_cast<const float4*>(&s.c[prow(2 * j)][px0]);
      const float4 y = *reinterpret_cast<const float4*>(&s.c[prow(2 * j) + 1][px0]);
      float m = vmin3(vmin3(vmin3(x.x, x.y, x.z), x.w, y.x), vmin3(y.y, y.z, y.w), y.w);
      m = vmin(m, dpp_move<0xb1, 0xf>(m));  // quad_perm 1, 0, 3, 2
      m = vmin(m, dpp_move<0x4e, 0xf>(m));  // quad_perm 2, 3, 0, 1
      v = vmax(v, m);
    }
    if ((tid & 63) >= PG * PRUNS) v = __int_as_float(0xff800000);  // (a quad of its own)
    static_assert(PG * PRUNS == 60, "whole quads hold the region's columns");
    v = vmax(v, __shfl_xor(v, 4));
    v = vmax(v, __shfl_xor(v, 8));
    if ((tid & 15) == 0) levels[tid >> 4] = v;
    __syncthreads();
    {  // the median of the 16
      static_assert(NT == 256, "16 rows of lanes");
      v = levels[tid & 15];
      int rank = 0;
#pragma unroll
      for (int j = 0; j < 16; ++j) rank += levels[j] < v || (levels[j] == v && j < (tid & 15)) ? 1 : 0;
      const uint64_t at = __ballot(rank == 8);
      v = __shfl(v, at ? __ffsll((long long)at) - 1 : 0);
    }
    const float t = candidate_bound(sigclip, noise_from_med<false>(fkey(v), nc, f.rn2), s.margin);
    // (where it brings little, many hits stay too many; where the bound does
    // not apply, its margin is infinite)
    if (t > (npc > 2u * ICAP ? 1.5f : 1.1f) * s.thr) {  // (uniform; false for a NaN)
      if (tid == 0) s.cnt = 0u;
      // [C < v] of the region's cells, one after another: 32 each thread, read
      // from a different quarter row on in each lane (the banks)
      if (tid < RH * RW / 32) {
        uint32_t below = 0u;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const int part = (tid + j) & 7;
          const float4 x = *reinterpret_cast<const float4*>(&s.c[0][0] + 32 * tid + 4 * part);
          uint32_t n = sign_into(0u, x.w - v);
          n = sign_into(n, x.z - v);
          n = sign_into(n, x.y - v);
          n = sign_into(n, x.x - v);
          below |= n << (4 * part);
        }
        cells[tid] = below;
      }
      __syncthreads();
      // which medians lie below v: a word of 32 pixels each thread, the counts bit-sliced
      if (tid >= 4 * NW && tid < (RH - 4) * NW) {
        uint32_t one[5], two[5], four[5];  // per row of the window: how many of its 5 cells lie below
#pragma unroll
        for (int a = 0; a < 5; ++a) {
          const int i = (tid / NW - 2 + a) * RW + 32 * (tid % NW) - 2;
          const uint32_t* p = cells + (i >> 5);
          const uint32_t lo = __builtin_amdgcn_alignbit(p[1], p[0], i & 31);
          const uint32_t hi = __builtin_amdgcn_alignbit(p[2], p[1], i & 31);
          const uint32_t c1 = __builtin_amdgcn_alignbit(hi, lo, 1), c2 = __builtin_amdgcn_alignbit(hi, lo, 2);
          const uint32_t c3 = __builtin_amdgcn_alignbit(hi, lo, 3), c4 = __builtin_amdgcn_alignbit(hi, lo, 4);
          const uint32_t s1 = lo ^ c1 ^ c2, k1 = majority(lo, c1, c2), k2 = majority(s1, c3, c4);
          one[a] = s1 ^ c3 ^ c4;
          two[a] = k1 ^ k2;
          four[a] = k1 & k2;
        }
        uint32_t low;  // medians below v
        if (f.sepmed) {  // 3 rows with 3 cells below
#pragma unroll
          for (int a = 0; a < 5; ++a) one[a] = four[a] | (two[a] & one[a]);
          const uint32_t s1 = one[0] ^ one[1] ^ one[2], k1 = majority(one[0], one[1], one[2]);
          const uint32_t k2 = majority(s1, one[3], one[4]);
          low = (k1 & k2) | ((k1 ^ k2) & (s1 ^ one[3] ^ one[4]));
        } else {  // 13 cells below
          const uint32_t o1 = one[0] ^ one[1] ^ one[2], p0 = majority(one[0], one[1], one[2]);
          const uint32_t o = o1 ^ one[3] ^ one[4], p1 = majority(o1, one[3], one[4]);
          const uint32_t t1 = two[0] ^ two[1] ^ two[2], q0 = majority(two[0], two[1], two[2]);
          const uint32_t t2 = t1 ^ two[3] ^ two[4], q1 = majority(t1, two[3], two[4]);
          const uint32_t w = t2 ^ p0 ^ p1, q2 = majority(t2, p0, p1);
          const uint32_t f1 = four[0] ^ four[1] ^ four[2], e0 = majority(four[0], four[1], four[2]);
          const uint32_t f2 = f1 ^ four[3] ^ four[4], e1 = majority(f1, four[3], four[4]);
          const uint32_t f3 = q0 ^ q1 ^ q2, e2 = majority(q0, q1, q2);
          const uint32_t r = f2 ^ f3, e3 = f2 & f3;  // o + 2 w + 4 r + 8 (e0 + e1 + e2 + e3) cells
          const uint32_t x1 = e0 ^ e1 ^ e2, y1 = majority(e0, e1, e2);
          const uint32_t x = x1 ^ e3, y = y1 | (x1 & e3);  // (at most 3 of them)
          low = y | (x & r & (w | o));
        }
        low_med[tid] = low;
      }
      __syncthreads();
      uint32_t keep = 0u;  // the lane's pixels over the bound at v, and those whose median is below it
#pragma unroll
      for (int j = 0; j < PP; ++j) {
        const int y = prow(2 * j);
        float4 up = *reinterpret_cast<const float4*>(&s.c[y - 1][px0]);
        float4 cu = *reinterpret_cast<const float4*>(&s.c[y][px0]);
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          const float4 dn = *reinterpret_cast<const float4*>(&s.c[y + k + 1][px0]);
          const float l = dpp_move<0x138, 0xf>(cu.w), r = dpp_move<0x130, 0xf>(cu.x);
          const float e0 = __builtin_fmaf(2.0f, cu.x, -(vmin(up.x, dn.x) + vmin(l, cu.y)));
          const float e1 = __builtin_fmaf(2.0f, cu.y, -(vmin(up.y, dn.y) + vmin(cu.x, cu.z)));
          const float e2 = __builtin_fmaf(2.0f, cu.z, -(vmin(up.z, dn.z) + vmin(cu.y, cu.w)));
          const float e3 = __builtin_fmaf(2.0f, cu.w, -(vmin(up.w, dn.w) + vmin(cu.z, r)));
          keep = keep + keep + (!(e0 <= t) ? 1u : 0u);
          keep = keep + keep + (!(e1 <= t) ? 1u : 0u);
          keep = keep + keep + (!(e2 <= t) ? 1u : 0u);
          keep = keep + keep + (!(e3 <= t) ? 1u : 0u);
          const uint32_t low = low_med[(y + k) * NW + (px0 >> 5)] >> (px0 & 31);
          keep |= __brev(low) >> 28;
          up = cu;
          cu = dn;
        }
      }
      hits &= keep;
      hbase = wave_reserve(&s.cnt, (unsigned int)__popc(hits));
      __syncthreads();
      npc = s.cnt;
    }
  }
  uint2* open = reinterpret_cast<uint2*>(s.s4);  // candidates and their med7 bounds, before the pool's use
  constexpr int OCAP = (int)(sizeof(s.s4) / sizeof(uint2));
  const bool listed = npc <= (unsigned int)ICAP;  // (uniform) else every hit is evaluated below
  if (listed) {
    for (uint32_t hb = hits; hb; hb &= hb - 1, ++hbase) {
      const int b = 4 * PR - __ffs((int)hb);
      s.lst[hbase] = (uint16_t)(prow(b >> 2) * RW + px0 + (b & 3));
    }
    __syncthreads();
    for (unsigned int j = tid; j < npc; j += NT) {
      const int i = s.lst[j], r = i / RW, q = i - r * RW;
      // a NaN passes every bound, so it arrives here (and every pixel with an
      // infinite one in the region)
      if (!finite_bits(s.c[r][q])) atom_or(f.status, 1);
      float N;
      const float S = iter_s(s, f, nc, r, q, nonneg, N);
      if (S > sigclip) {
        // dead: the objlim test fails even for S' = S.  Not where it holds
        // for the smallest med7 there can be (cosmic rays); else where med7
        // lies below the value at which it would hold (stars): listed.
        const float m3 = iter_med3(s, f, r, q, nonneg);
        bool live = objlim_holds(f, m3, s.mn, s.nmin, S);
        if (!live) {
          const float d = N * (S / f.objlim), t = m3 - d - (fabsf(m3) + d) * 0x1p-18f;
          live = objlim_holds(f, m3, t, N, S);
          if (!live) {
            const unsigned int at = atomicAdd(&s.nopen, 1u);
            if (at < (unsigned int)OCAP)
              open[at] = uint2{__float_as_uint(t), (uint32_t)i};
            else
              live = true;  // (evaluated in full)
          }
        }
        if (live) {
          s.set(kBitCd, r, q);
          s.live = 1;
          s.mark_near(r, q);
        }
      }
    }
    __syncthreads();
    const unsigned int no = min(s.nopen, (unsigned int)OCAP);
    if (no) {  // (uniform)
      for (unsigned int j = tid >> 2; j < no; j += NT / 4) {
        const uint2 o = open[j];
        const int i = (int)o.y, r = i / RW, q = i - r * RW;
        const bool dead = iter_med7_le(s, f, r, q, ry0, rx0, inner, __uint_as_float(o.x));
        if ((tid & 3) == 0) {
          s.set(dead ? kBitDead : kBitCd, r, q);
          if (!dead) {
            s.live = 1;
            s.mark_near(r, q);
          }
        }
      }
      __syncthreads();
    }
  } else {
#pragma unroll 1
    for (int k = 0; k < PR; ++k) {  // (a NaN is a hit)
      const float4 x = *reinterpret_cast<const float4*>(&s.c[prow(k)][px0]);
      const bool bad = !finite_bits(x.x) || !finite_bits(x.y) || !finite_bits(x.z) || !finite_bits(x.w);
      if (bad && (hits >> (4 * (PR - 1 - k)) & 15u)) atom_or(f.status, 1);
    }
  }

  // ---- 3-4. S near the live candidates, S', G1, G2, B1.
  // S', G1, G2 and B1 at n listed pixels; window gives S's window there.
  auto evaluate = [&](const uint16_t* list, unsigned int n, auto window) __attribute__((always_inline)) {
#pragma unroll 1
    for (unsigned int j0 = 0; j0 < n; j0 += NT) {
      const unsigned int j = j0 + tid;
      int i = 0;
      float limit = 0.0f;
      bool open = false;
      if (j < n) {
        i = list[j];
        const int r = i / RW, q = i - r * RW;
        int v[25];
        window(r, q, v);
        const float spv = __int_as_float(v[12]) - funkey(med25_of(v, f.sepmed));
        if (spv > lo) s.set(kBitG2, r, q);
        if (spv > sigclip) {
          s.set(kBitG1, r, q);
          // holds for the smallest med7 and N there can be?
          const float m3 = iter_med3(s, f, r, q, nonneg);
          open = !objlim_holds(f, m3, s.mn, s.nmin, spv);
          if (open) {
            limit = iter_objlim(s, f, nc, r, q, nonneg, m3, spv);
          } else {
            s.set(kBitB1, r, q);
            s.any_b1 = 1;
          }
        }
      }
      const uint64_t left = __ballot(open);
      if (left) {  // (uniform) the wave's undecided ones, a quad each
        const int ln = tid & 63, total = __popcll(left);
        const int before = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(left >> 32),
                                                          __builtin_amdgcn_mbcnt_lo((uint32_t)left, 0u));
        // lane k gets the k-th one's lane
        const int nth = __builtin_amdgcn_ds_permute(4 * (open ? before : total + ln - before), ln);
#pragma unroll 1
        for (int k0 = 0; k0 < total; k0 += 16) {
          const int k = k0 + (ln >> 2), src = __shfl(nth, min(k, 63));
          const int ci = __shfl(i, src), r = ci / RW, q = ci - r * RW;
          const float lim = __shfl(limit, src);
          if (k < total && !iter_med7_le(s, f, r, q, ry0, rx0, inner, lim) && (ln & 3) == 0) {
            s.set(kBitB1, r, q);
            s.any_b1 = 1;
          }
        }
      }
    }
  };
  auto from_plane = [&](int r, int q, int* v) __attribute__((always_inline)) {
    iter_plane_window(f, ry0 + r, rx0 + q, v);
  };
  // By blocks near the candidates.  False (and no bit set) if the pixels to
  // evaluate exceed the list.
  auto detect = [&]() __attribute__((always_inline)) -> bool {
    next_phase();
    if (tid == 0) s.n2 = 0u;
    __syncthreads();
    // Every wave sums up the rows' blocks, a row each lane; block j of the
    // tile is then found from the sums, with no list.
    static_assert(QR <= 64 && QC <= 64, "a lane per row, a bit per column");
    const int ln = tid & 63;
    uint64_t row = ln < QR ? s.qbits[ln] : 0ull;
    if (!inner) {  // blocks that hold a pixel of the frame
      const int j0 = max(0, (fc0 - 2) >> 1), j1 = min(QC, (fc1 - 1) >> 1);
      const bool in = (row_in(2 + 2 * ln) || row_in(3 + 2 * ln)) && j0 < j1;
      row &= in ? ((1ull << j1) - 1ull) & ~((1ull << j0) - 1ull) : 0ull;
    }
    const int upto = wave_scan(__popcll(row));
    const unsigned int nq = (unsigned int)__builtin_amdgcn_readlane(upto, 63);
    // Where the pool does not hold them (a dense tile), S is kept in the frame's
    // S plane, which holds nothing else meanwhile -- tiles beside this one store
    // the same values there -- and the pool's place has the list.  (A small
    // tile's pool holds every block.)
    const bool big = QCAP < QR * QC && __builtin_expect(nq > (unsigned int)QCAP, 0);
    // S at the pixels of block j's part: PX of its pixels, in each of 4 / PX
    // lanes.  Those that are live candidates of the rows, or next to one with
    // S > lo (G2 off the candidates matters within 2 pixels of the tile), are
    // listed.  (Whole waves run this.)
    auto blocks = [&](auto px, auto in_plane) __attribute__((always_inline)) {
      constexpr int PX = decltype(px)::value, LANES = 4 / PX;
      constexpr bool PLANE = decltype(in_plane)::value;
      uint16_t* list = PLANE ? reinterpret_cast<uint16_t*>(s.s4) : s.lst;
      constexpr unsigned int cap = PLANE ? sizeof(s.s4) / 2 : ICAP;
#pragma unroll 1
      for (unsigned int j0 = 0; j0 < nq; j0 += NT / LANES) {
        const unsigned int j = j0 + tid / LANES;
        const int part = tid % LANES;
        const unsigned int jc = min(j, nq - 1u);
        int br = 0;  // the row that holds it: the first whose sum exceeds j
#pragma unroll
        for (int k = 32; k > 0; k >>= 1) br += __shfl(upto, br + k - 1) <= (int)jc ? k : 0;
        const uint32_t ml = (uint32_t)__shfl((int)(uint32_t)row, br);
        const uint32_t mh = QC > 32 ? (uint32_t)__shfl((int)(uint32_t)(row >> 32), br) : 0u;
        const int nth = (int)jc - (__shfl(upto, br) - __popc(ml) - __popc(mh));
        const int bc = nth_bit(ml, mh, nth);
        const int y = 2 + 2 * br + (PX == 4 ? 0 : part * PX / 2), x = 2 + 2 * bc + (PX == 1 ? part & 1 : 0);
        float S[PX];
        uint32_t want = 0u;  // bit k: pixel k listed
        if (j < nq) {
          constexpr int ROWS = PX == 4 ? 2 : 1, COLS = PX / ROWS;
          uint32_t cw[ROWS], dw[ROWS];
#pragma unroll
          for (int a = 0; a < ROWS; ++a) {
            const int rb = clampi(y + a - SM::BR0, SM::BROWS - 1) + SM::BR0;
            cw[a] = s.word(kBitCd, rb, x >> 5) >> (x & 31);
            dw[a] = s.word(kBitD1, rb, x >> 5) >> (x & 31);
            if (rb != y + a) cw[a] = 0u;
          }
          iter_block<PX>(s, f, nc, y, x, nonneg, S);
          if (PLANE) {
#pragma unroll
            for (int k = 0; k < PX; ++k) {
              const int r = y + (k >> 1), q = x + (k & 1);
              if (inner || (row_in(r) && q >= fc0 && q < fc1)) stg(f.splane, (int64_t)(ry0 + r) * w + rx0 + q, S[k]);
            }
          } else if (PX == 4)
            *reinterpret_cast<float4*>(s.s4[j]) = float4{S[0], S[1 % PX], S[2 % PX], S[3 % PX]};
          else if (PX == 2)
            *reinterpret_cast<float2*>(&s.s4[j][2 * part]) = float2{S[0], S[1 % PX]};
          else
            s.s4[j][part] = S[0];
          if (part == 0 && !PLANE) s.qmap[br * QC + bc] = (typename SM::QIndex)j;
#pragma unroll
          for (int k = 0; k < PX; ++k) {
            const int a = k / COLS, b = k % COLS, r = y + a, q = x + b;
            const bool cand = (cw[a] >> b) & 1u, by = (dw[a] >> b) & 1u;
            const bool here = r >= 6 && r < RH - 6 && q >= 6 && q < RW - 6 &&
                              (inner || (row_in(r) && q >= fc0 && q < fc1));
            if (cand || (by && here && S[k] > lo)) want |= 1u << k;
          }
        }
        unsigned int at = wave_reserve(&s.n2, (unsigned int)__popc(want));
#pragma unroll
        for (int k = 0; k < PX; ++k)
          if ((want >> k) & 1u) {
            if (at < cap) list[at] = (uint16_t)((y + k / 2 * (PX == 4 ? 1 : 0)) * RW + x + (PX == 1 ? 0 : k & 1));
            ++at;
          }
      }
    };
    // A block's four medians together take 308 operations, two of a row 212,
    // one alone 184: fewer blocks than lanes, less work per lane.
    if (4 * nq <= (unsigned int)NT)
      blocks(std::integral_constant<int, 1>{}, std::false_type{});
    else if (2 * nq <= (unsigned int)NT)
      blocks(std::integral_constant<int, 2>{}, std::false_type{});
    else if (!big)
      blocks(std::integral_constant<int, 4>{}, std::false_type{});
    else
      blocks(std::integral_constant<int, 4>{}, std::true_type{});
    __syncthreads();
    next_phase();
    const unsigned int n2 = s.n2;
    if (n2 > (big ? (unsigned int)sizeof(s.s4) / 2 : (unsigned int)ICAP)) {
      __syncthreads();  // (every wave has read the count before it is cleared)
      return false;
    }
    auto pool = [&](int r, int q, int* v) __attribute__((always_inline)) {
      iter_pool_window(s, f, r, q, ry0, rx0, inner, v);
    };
    if (!big)
      evaluate(s.lst, n2, pool);
    else
      evaluate(reinterpret_cast<const uint16_t*>(s.s4), n2, from_plane);
    __syncthreads();
    return true;
  };
  // By every block of the region, S in the S plane: every pixel with S > sigclip
  // is evaluated, whatever step 2 found.  Dense tiles are bound by the issue of
  // their medians.  (In bands of rows whose blocks fit the pool each band's
  // phases filled one or two of the four waves: a 4096^2 frame with its sky
  // subtracted took 2.24 ms, now 1.15, the sparse passes 1.34; one with 100
  // times the cosmic rays 1.51, 0.75 and 2.13.)
  auto detect_all = [&]() __attribute__((always_inline)) {
    next_phase();
    if (wt) {
      s.word(kBitCd, wr, ww) = 0u;
      s.word(kBitDead, wr, ww) = 0u;  // now the pixels with S > lo
    }
    if (tid == 0) s.n2 = 0u;
    __syncthreads();
#pragma unroll 1
    for (int j = tid; j < QR * QC; j += NT) {
      const int br = j / QC, y = 2 + 2 * br, x = 2 + 2 * (j - br * QC);
      float S[4];
      iter_block<4>(s, f, nc, y, x, nonneg, S);
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        uint32_t cd = 0u, g2 = 0u;
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          const int r = y + a, q = x + b;
          if (!inner && !(row_in(r) && q >= fc0 && q < fc1)) continue;
          stg(f.splane, (int64_t)(ry0 + r) * w + rx0 + q, S[2 * a + b]);
          cd |= S[2 * a + b] > sigclip ? 1u << b : 0u;
          g2 |= S[2 * a + b] > lo ? 1u << b : 0u;
        }
        const int r = y + a;  // (x is even: both bits in one word)
        if (r >= 4 && r < RH - 4 && x >= 4 && x < RW - 4) {
          if (cd) atomicOr(&s.word(kBitCd, r, x >> 5), cd << (x & 31));
          if (g2) atomicOr(&s.word(kBitDead, r, x >> 5), g2 << (x & 31));
        }
      }
    }
    __syncthreads();
    next_phase();
    // the list in the pool, and each thread's places in it after its end
    constexpr unsigned int LCAP = 1536;
    uint16_t* list = reinterpret_cast<uint16_t*>(s.s4);
    unsigned int* place = reinterpret_cast<unsigned int*>(list + LCAP);
    static_assert(2 * LCAP + 4 * NT <= sizeof(s.s4), "both fit");
    {
      uint32_t want = 0u;
      if (wt) {
        want = s.word(kBitCd, wr, ww);
        if (wr >= 6 && wr < RH - 6) {
          const BitSpan c = s.span(kBitCd, wr - 1, ww) | s.span(kBitCd, wr, ww) | s.span(kBitCd, wr + 1, ww);
          want |= span_dil<1>(c) & s.word(kBitDead, wr, ww) & col_bits(ww, 6, RW - 6);
        }
        s.word(kBitD1, wr, ww) = want;
      }
      place[tid] = wave_reserve(&s.n2, (unsigned int)__popc(want));
    }
    __syncthreads();
    const unsigned int n2 = s.n2;
#pragma unroll 1
    for (unsigned int c0 = 0; c0 < n2; c0 += LCAP) {
      next_phase();
      unsigned int at = place[tid] - c0;
      for (uint32_t want = wt ? s.word(kBitD1, wr, ww) : 0u; want; want &= want - 1, ++at)
        if (at < LCAP) list[at] = (uint16_t)(wr * RW + 32 * ww + __ffs((int)want) - 1);
      __syncthreads();
      evaluate(list, min(n2 - c0, LCAP), from_plane);
      __syncthreads();
    }
  };
  if (listed && s.live) {  // (uniform: written before a barrier, read after it)
    // B2 takes in candidates within 1 of a B1 pixel, dead ones too (a cosmic
    // ray beside a star): dead candidates within 1 of a live one are
    // evaluated with the live ones
    // (one that a promoted one brings in as well costs work, no more)
    const uint32_t up = wt ? s.word(kBitDead, wr, ww) & s.word(kBitD1, wr, ww) : 0u;
    if (up) {
      atomicOr(&s.word(kBitCd, wr, ww), up);
      for (uint32_t d = up; d; d &= d - 1) s.mark_near(wr, 32 * ww + __ffs((int)d) - 1);
    }
  }
  if (__builtin_expect(!listed || (s.live && !detect()), 0)) detect_all();

  // ---- 5. growth
  bool changed = false;
  next_phase();
  if (s.any_b1) {  // (uniform: written before a barrier, read after it)
    if (tid == 0) s.cnt = 0u;
    uint32_t fresh = 0u;
    if (wt) {
      uint32_t nw = 0u;
      if (wr >= 6 && wr < RH - 6) {
        // B2 of the rows above, of and below this one, each word with the
        // last column of the word before it and the first of the one after
        BitSpan b2 = {0u, 0u, 0u};
        BitSpan x0 = s.span(kBitB1, wr - 2, ww), x1 = s.span(kBitB1, wr - 1, ww);
#pragma unroll
        for (int k = -1; k <= 1; ++k) {
          const BitSpan x2 = s.span(kBitB1, wr + k + 1, ww), g = s.span(kBitG1, wr + k, ww);
          const BitSpan v = x0 | x1 | x2;
          b2 = b2 | BitSpan{(v.l | (v.l << 1) | (v.c << 31)) & g.l, span_dil<1>(v) & g.c,
                            (v.r | (v.r >> 1) | (v.c >> 31)) & g.r};
          x0 = x1;
          x1 = x2;
        }
        const uint32_t b3 = span_dil<1>(b2) & s.word(kBitG2, wr, ww) & col_bits(ww, 6, RW - 6);
        const uint32_t m = s.word(kBitM, wr, ww);
        nw = b3 & ~m;
        s.word(kBitM, wr, ww) = m | b3;
        const uint32_t own = nw & col_bits(ww, HL, HL + TW_);
        if (wr >= HL && wr < HL + TH) fresh = (uint32_t)__popc(own);
      }
      s.word(kBitCd, wr, ww) = nw;  // the new mask pixels
    }
    (void)wave_reserve(&s.fresh, fresh);
    __syncthreads();
    if (!inner) {  // the replacement's windows clamp on the frame too
      uint32_t m = 0u;
      if (wt) {
        const int cr = clampi(ry0 + wr, h - 1) - ry0;
        const uint32_t lo_out = col_bits(ww, 0, fc0), hi_out = col_bits(ww, fc1, RW);
        m = s.word(kBitM, cr, ww) & ~(lo_out | hi_out);
        if (lo_out && s.bit(kBitM, cr, fc0)) m |= lo_out;
        if (hi_out && s.bit(kBitM, cr, fc1 - 1)) m |= hi_out;
      }
      __syncthreads();
      if (wt) s.word(kBitM, wr, ww) = m;
    }
    // the tile's mask pixels: those within 2 of a new one are replaced anew,
    // the others keep their value
    uint32_t redo = 0u, keep = 0u, zone = 0u;
    if (wt && wr >= HL && wr < HL + TH && row_in(wr)) {
      const uint32_t own = s.word(kBitM, wr, ww) & col_bits(ww, HL, min(HL + TW_, fc1));
      if (own) {
        BitSpan o = s.span(kBitCd, wr - 2, ww);
#pragma unroll
        for (int k = -1; k <= 2; ++k) o = o | s.span(kBitCd, wr + k, ww);
        const uint32_t d = span_dil<2>(o);
        redo = own & d;
        keep = own & ~d;
        if (redo) {
          const int zy = wr < 2 * HL ? 0 : wr < TH ? 1 : 2;
          const uint32_t z = ((redo & col_bits(ww, HL, 2 * HL)) ? 1u : 0u) |
                             ((redo & col_bits(ww, 2 * HL, TW_)) ? 2u : 0u) |
                             ((redo & col_bits(ww, TW_, TW_ + HL)) ? 4u : 0u);
          zone = z << (3 * zy);
        }
      }
    }
    zone = wave_or(zone);
    if (zone && lane == 0) atomicOr(&s.zones, zone);
    const unsigned int rbase = wave_reserve(&s.cnt, (unsigned int)__popc(redo));
    __syncthreads();
    const unsigned int nredo = s.cnt;
    changed = nredo != 0u;  // (uniform)
    float* vals = iter_values(f, plane ^ 1u);
    if (changed) {
      while (keep) {  // carried values, plane to plane
        const int q = __ffs((int)keep) - 1 + 32 * ww;
        keep &= keep - 1;
        stg(vals, (int64_t)(ry0 + wr) * w + rx0 + q, s.c[wr][q]);
      }
    }
    unsigned int unrep = 0;
    for (unsigned int c0 = 0; c0 < nredo; c0 += ICAP) {
      unsigned int at = rbase;
      for (uint32_t bits = redo; bits; bits &= bits - 1) {
        const int b = __ffs((int)bits) - 1;
        if (at - c0 < (unsigned int)ICAP) s.lst[at - c0] = (uint16_t)(wr * RW + 32 * ww + b);
        ++at;
      }
      __syncthreads();
      const unsigned int n = min(nredo - c0, (unsigned int)ICAP);
      for (unsigned int j0 = 0; j0 < n; j0 += NT) {
        const unsigned int j = j0 + tid;
        float out = 0.0f;
        int r = 0, q = 0;
        if (j < n) {
          const int i = s.lst[j];
          r = i / RW;
          q = i - r * RW;
          out = s.c[r][q];  // (no mask pixel's value is below s.mn: the patches count in it)
          int v[25];
          int cnt = 0;
#pragma unroll
          for (int a = 0; a < 5; ++a) {
            // the window row's five mask bits, across a word boundary or not
            const uint32_t* mw = &s.word(kBitM, r - 2 + a, (q - 2) >> 5);
            const uint32_t bits = __builtin_amdgcn_alignbit(mw[1], mw[0], (q - 2) & 31);
            cnt += 5 - __popc(bits & 31u);
#pragma unroll
            for (int b = 0; b < 5; ++b)
              v[a * 5 + b] = __float_as_int(s.c[r - 2 + a][q - 2 + b]);
            if (!nonneg) {
#pragma unroll
              for (int b = 0; b < 5; ++b) v[a * 5 + b] ^= (v[a * 5 + b] >> 31) & 0x7fffffff;
            }
#pragma unroll
            for (int b = 0; b < 5; ++b) v[a * 5 + b] = ((bits >> b) & 1u) ? KEY_EXCLUDED : v[a * 5 + b];
          }
          if (cnt > 0) {
            int srt[13];
            sort25_lo13(v, srt);  // ranks 0..12: the lower median of cnt <= 25 values
            const int rk = (cnt - 1) >> 1;
            int sel = srt[0];
#pragma unroll
            for (int k = 1; k < 13; ++k) sel = (rk == k) ? srt[k] : sel;
            out = funkey(sel);
          } else {
            // counted when the previous mask still left an un-flagged cell in
            // the window (the pixel itself among them): one is new
            bool first = false;
            for (int a = 0; a < 5; ++a)
              for (int b = 0; b < 5; ++b)
                first |= s.bit(kBitCd, clampi(ry0 + r - 2 + a, h - 1) - ry0,
                               clampi(rx0 + q - 2 + b, w - 1) - rx0);
            unrep += first ? 1u : 0u;
          }
          const int64_t gi = (int64_t)(ry0 + r) * w + rx0 + q;
          stg(vals, gi, out);
          if (it > 0) {
            stg(f.clean, gi, out);
            stg(f.out_mask, gi, (uint8_t)1);
          } else {
            s.c[r][q] = out;  // the whole tile is stored below, from LDS; a mask pixel, so no window holds it
          }
        }
      }
      if (unrep) atomicAdd(&s.unrep, unrep);
      unrep = 0u;
      __syncthreads();  // the list is rebuilt
    }
    if (tid == 0) {
      if (s.fresh) atom_add(f.n_new + it, (unsigned long long)s.fresh);
      if (s.unrep) atom_add(f.n_new + f.niter, (unsigned long long)s.unrep);
    }
  }

  // ---- state, mask bits, and in iteration 0 the whole tile's outputs
  const bool write = changed || it == 0;
  next_phase();
  if (!write) return;
  if (tid == 0) {
    __hip_atomic_store(gp(iter_state(f) + tile), ((uint32_t)(it + 1) << 1) | (plane ^ 1u), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
    if (it == 0) {
      stg(iter_stamp(f, 0), tile, 0u);
      stg(iter_stamp(f, 1), tile, 0u);
    }
  }
  if (it > 0 && it + 1 < f.niter && !f.est_gain && tid < 9) {
    // the tiles whose region holds a change: this one, and those beside a
    // zone along its edge that holds one (a frame that estimates its gain runs
    // all its tiles)
    const uint32_t zr = tid < 3 ? 0x007u : tid < 6 ? 0x1ffu : 0x1c0u;
    const uint32_t zc = tid % 3 == 0 ? 0x049u : tid % 3 == 1 ? 0x1ffu : 0x124u;
    const int n = grid.neighbour(ty, tx, tid);
    if (n >= 0 && (s.zones & zr & zc)) {
      const uint32_t stamp = (uint32_t)(it + 2);
      if (__hip_atomic_exchange(gp(iter_stamp(f, it + 1) + n), stamp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) !=
          stamp)
        stg(next.list, atom_add(next.count, 1u), next.base + n);
    }
  }
  if (tid < TH && y0 + tid < h) {
    const uint32_t* m = &s.word(kBitM, tid + HL, 0);
    uint64_t word = (m[0] >> 8) | (m[1] << 24);
    if (TW_ == 64) word |= (uint64_t)((m[1] >> 8) | (m[2] << 24)) << 32;
    if (w - x0 < 64) word &= (1ull << (w - x0)) - 1ull;  // pixels of the frame only
    uint64_t* p = (plane ^ 1u) ? f.mbits[1] : f.mbits[0];
    if (TW_ == 64)
      stg(p, (int64_t)(y0 + tid) * f.wpr + tx, word);
    else
      stg(reinterpret_cast<uint32_t*>(p), (int64_t)(y0 + tid) * f.wpr * 2 + tx, (uint32_t)word);
  }
  if (it > 0) return;
  if (y0 + TH <= h && x0 + TW_ <= w) {
    constexpr int C4 = TW_ / 4, RP = NT / C4;  // C4 threads per row, RP rows at a time
    static_assert(TH % RP == 0, "whole passes");
    const int r0 = tid / C4, q0 = 4 * (tid - r0 * C4);
    float* cl = f.clean + (int64_t)y0 * w + x0;
#pragma unroll
    for (int k = 0; k < TH / RP; ++k) {
      const float4 v = *reinterpret_cast<const float4*>(&s.c[r0 + k * RP + HL][q0 + HL]);
      *(__attribute__((address_space(1))) f4u*)(cl + (uint32_t)((r0 + k * RP) * w + q0)) = f4u{v.x, v.y, v.z, v.w};
    }
    // 16 mask bytes per thread, wherever the row starts
    constexpr int M16 = TW_ / 16;
    typedef uint32_t u4u __attribute__((ext_vector_type(4), aligned(1)));
    if (tid < TH * M16) {
      const int r = tid / M16, q = 16 * (tid - r * M16);
      const uint32_t* m = &s.word(kBitM, r + HL, (HL + q) >> 5);
      const uint32_t b = __builtin_amdgcn_alignbit(m[1], m[0], (HL + q) & 31);
      *(__attribute__((address_space(1))) u4u*)(f.out_mask + (int64_t)(y0 + r) * w + x0 + q) =
          u4u{spread4(b & 15u), spread4((b >> 4) & 15u), spread4((b >> 8) & 15u), spread4((b >> 12) & 15u)};
    }
  } else {
    for (int i = tid; i < TH * TW_; i += NT) {
      const int r = i / TW_, q = i - r * TW_;
      if (y0 + r >= h || x0 + q >= w) continue;
      const int64_t gi = (int64_t)(y0 + r) * w + x0 + q;
      stg(f.clean, gi, s.c[r + HL][q + HL]);
      stg(f.out_mask, gi, (uint8_t)(s.bit(kBitM, r + HL, q + HL) ? 1 : 0));
    }
  }
}

// Whether iteration it has work for a tile (of one block per tile launches).
// A new gain changes the noise model everywhere.
__device__ __forceinline__ bool iter_due(const FrameDev& f, int it, int tile) {
  return it <= 1 || f.est_gain || ldg(iter_stamp(f, it), tile) == (uint32_t)(it + 1);
}

}  // namespace lac
