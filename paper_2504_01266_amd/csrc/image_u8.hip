// 8-bit image kernels: the paper's own image operations on its own data type.
//
// The paper filters 8-bit images read with OpenCV (interleaved channels, one
// pixel after another) with float taps: a 3x3 Laplacian sharpen that skips
// out-of-image neighbours (Section 4.2.4), run on images enlarged by nearest-
// neighbour upsampling (Section 4.2.3; the pipeline of Section 6.6), and a
// weighted RGB -> gray sum (Section 4.2.5).  Three kernels cover them:
//
//  k_u8_gather  one K x K filter (SHARED mode) on planar or interleaved 8-bit
//               images, clamp-to-edge or zero borders, optionally through a
//               nearest upsample by an integer factor s (output pixel (Y, X)
//               reads source pixel (Y / s, X / s)) that is never materialised.
//               A work-group owns a 32-row x 2048-element output tile (an
//               element is one channel of one pixel: for interleaved images a
//               row is W*s*C elements long and the tap offsets step C
//               elements).  It first stages the source rows the tile needs,
//               already expanded along the row (window element j holds the
//               source byte for output element e0 - rC + j, or 0 outside a
//               zero border) into LDS.  Each lane then walks down the tile's
//               rows producing 8 consecutive elements per row from its window
//               of 8 + 2rC bytes.  Rows whose K source rows are the same as the
//               previous row's (inside an upsampled block when s > 1) reuse
//               the previous values and only store.
//  k_u8_direct  the 3 x 3 filter into 8-bit outputs, upsampled by 1 to 4.
//  k_u8_mix     per-pixel channel mixing (BANK mode with K = 1, e.g. the
//               grayscale weights): up to 4 input and 4 output channels,
//               planar or interleaved, four pixels per lane.
//
// Arithmetic.  Float taps: binary32, accumulator +0, one fused multiply-add
// per term in the order input channel, tap row, tap column.  Integer taps:
// int32 sums (wrapping modulo 2^32).  8-bit outputs: the sum is clamped to
// [0, 255] and rounded to nearest, ties to even.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>

#include "f2d_host.hpp"
#include "f2d_internal.hpp"

namespace f2d {
namespace {

constexpr int kOutI32 = 0;
constexpr int kOutF32 = 1;
constexpr int kOutU8 = 2;

typedef uint32_t u32_a1 __attribute__((aligned(1)));
typedef uint32_t u32x2_a1 __attribute__((ext_vector_type(2), aligned(1)));
typedef uint32_t u32x4_a1 __attribute__((ext_vector_type(4), aligned(1)));

// N words from / to any byte address
template <int N>
__device__ __forceinline__ void load_words(const uint8_t* a, uint32_t (&w)[N]) {
  constexpr int N4 = N / 4 * 4, N2 = N4 + (N - N4) / 2 * 2;
#pragma unroll
  for (int i = 0; i < N4; i += 4) {
    const u32x4_a1 t = *reinterpret_cast<const u32x4_a1*>(a + 4 * i);
    w[i] = t[0];
    w[i + 1] = t[1];
    w[i + 2] = t[2];
    w[i + 3] = t[3];
  }
  if constexpr (N2 > N4) {
    const u32x2_a1 t = *reinterpret_cast<const u32x2_a1*>(a + 4 * N4);
    w[N4] = t[0];
    w[N4 + 1] = t[1];
  }
  if constexpr (N > N2) w[N2] = *reinterpret_cast<const u32_a1*>(a + 4 * N2);
}
template <int N>
__device__ __forceinline__ void store_words(uint8_t* a, const uint32_t (&w)[N]) {
  constexpr int N4 = N / 4 * 4, N2 = N4 + (N - N4) / 2 * 2;
#pragma unroll
  for (int i = 0; i < N4; i += 4)
    *reinterpret_cast<u32x4_a1*>(a + 4 * i) = u32x4_a1{w[i], w[i + 1], w[i + 2], w[i + 3]};
  if constexpr (N2 > N4) *reinterpret_cast<u32x2_a1*>(a + 4 * N4) = u32x2_a1{w[N4], w[N4 + 1]};
  if constexpr (N > N2) *reinterpret_cast<u32_a1*>(a + 4 * N2) = w[N2];
}

constexpr int kGThreads = 256;
// A lane produces E = 8 or 16 consecutive output elements per row (16 for
// 8-bit outputs of an image upsampled by 8 or more: one 16-byte store per
// lane and row);
// a tile row is 256 E elements, a staged row 256 E + 2rC bytes plus slack.
template <int E>
struct GTile {
  static constexpr int TW = kGThreads * E;
  static constexpr int PITCH_WORDS = (TW + 32) / 4;
};

struct GatherParams {
  const uint8_t* src;  // element (n, c, 0, 0): planar planes, or interleaved rows (stride_c 1)
  int64_t s_sn, s_sc, s_sh;
  void* dst;  // same layout as the source, in elements of the output type
  int64_t d_sn, d_sc, d_sh;
  const void* taps;  // K*K int32 or float
  int64_t H, W;      // source image, pixels
  int64_t Hout, Wout;  // H*s, W*s
  int64_t row0, out_rows;  // output rows [row0, row0 + out_rows) of the (upsampled) buffer
  int32_t s;         // nearest-upsample factor
  uint32_t s_magic;  // division by s: q = (t + ((x - t) >> 1)) >> s_shift, t = mulhi(x, s_magic)
  int32_t s_shift;   // (s >= 2; Granlund and Montgomery's method for invariant divisors)
  int32_t zero;      // zero borders (else clamp-to-edge)
  int32_t planes_c;  // planes per image on the grid: C (planar) or 1 (interleaved)
  int32_t th;        // output rows per tile
  int32_t lds_rows;  // staged source rows per tile (at most); one more zero row follows
  int32_t tiles_x, tiles_y;
  int64_t n_blocks;
};

// x / s for 0 <= x < 2^32 with the launch's invariant-divisor constants
__device__ __forceinline__ uint32_t div_s(uint32_t x, const GatherParams& p) {
  if (p.s == 1) return x;
  const uint32_t t = __umulhi(x, p.s_magic);
  return (t + ((x - t) >> 1)) >> p.s_shift;
}

template <int K, int P, bool TF, int OUT, int E>
__global__ __launch_bounds__(kGThreads) void k_u8_gather(GatherParams p) {
  constexpr int kGElems = E;
  constexpr int kGTW = GTile<E>::TW;
  constexpr int kGPitchWords = GTile<E>::PITCH_WORDS;
  constexpr int R = (K - 1) / 2;
  constexpr int RP = R * P;
  constexpr int WIN = kGTW + 2 * RP;          // staged elements per row
  constexpr int WORDS = (WIN + 3) / 4;
  constexpr int NW = (kGElems + 2 * RP + 3) / 4;  // words of a lane's window
  static_assert(WORDS <= kGPitchWords && (E / 4) * (kGThreads - 1) + NW <= kGPitchWords, "staged row too short");
  extern __shared__ uint32_t lds[];
  using Acc = typename std::conditional<TF, float, uint32_t>::type;
  const int zrow = p.lds_rows;                // an all-zero row for zero borders

  const int tid = threadIdx.x;
  const int64_t b = xcd_remap(blockIdx.x, p.n_blocks);
  const int64_t tiles = static_cast<int64_t>(p.tiles_x) * p.tiles_y;
  const int64_t plane = b / tiles;
  const int64_t t_in = b - plane * tiles;
  const int64_t ty = t_in / p.tiles_x;
  const int64_t tx = t_in - ty * p.tiles_x;
  const int64_t n = plane / p.planes_c;
  const int64_t c = plane - n * p.planes_c;
  const uint8_t* sp = p.src + n * p.s_sn + c * p.s_sc;
  const int64_t e0 = tx * kGTW;               // first output element of the tile
  const int64_t y0 = ty * p.th;               // first output row (band-relative)
  const int64_t L = p.Wout * P;               // elements per output row
  const int64_t nrow_out = min(static_cast<int64_t>(p.th), p.out_rows - y0);

  // source rows the tile reads: the upsampled rows t = row0 + y + u - R,
  // clamped to [0, Hout) (zero-border rows outside are the zero row);
  // indices fit in 32 bits (at most 2^30 rows and elements per row)
  auto clamp_out_row = [&](int64_t t) { return t < 0 ? int64_t{0} : (t >= p.Hout ? p.Hout - 1 : t); };
  const int32_t rlo = static_cast<int32_t>(div_s(static_cast<uint32_t>(clamp_out_row(p.row0 + y0 - R)), p));
  const int32_t rhi =
      static_cast<int32_t>(div_s(static_cast<uint32_t>(clamp_out_row(p.row0 + y0 + nrow_out - 1 + R)), p));
  const int nsrc = rhi - rlo + 1;  // <= lds_rows (host sizing)

  // ---- stage: row-expanded source bytes of every source row of the tile.
  // A thread owns window words tid + 256 k (k < NQ); their source offsets
  // are computed once, then the loads of two source rows for all its words
  // are issued before any of them is written, so a tile pays about nsrc / 2
  // load latencies.  Offsets < 0 are zero-border elements.
  constexpr int NQ = (WORDS + kGThreads - 1) / kGThreads;
  const int32_t wout = static_cast<int32_t>(p.Wout);
  int32_t off[NQ][4];
#pragma unroll
  for (int k = 0; k < NQ; ++k)
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) {
      const int32_t e = static_cast<int32_t>(e0) - RP + 4 * (tid + kGThreads * k) + jj;  // >= -RP
      const int32_t xu = (e + P * 4) / P - 4;                                          // floor(e / P)
      const int32_t ch = e - xu * P;
      int32_t xc = xu;
      bool inside = xu >= 0 && xu < wout;
      if (!inside && !p.zero) {
        xc = xu < 0 ? 0 : wout - 1;
        inside = true;
      }
      off[k][jj] = inside ? static_cast<int32_t>(div_s(static_cast<uint32_t>(xc), p)) * P + ch : -1;
    }
  // A window word whose four source bytes lie inside one 8-byte stretch of
  // the row (everywhere but zeroed border elements and the row's last bytes:
  // consecutive bytes without upsampling, at most two source pixels with it;
  // clamped edge pixels may repeat earlier offsets) is one or two 4-byte
  // loads from its lowest offset and a byte permute, instead of four byte
  // loads.
  const int32_t row_len = static_cast<int32_t>(p.W) * P;  // bytes of a source row
  bool dw[NQ], two_dw[NQ];
  int32_t dbase[NQ];
  uint32_t sel[NQ];
#pragma unroll
  for (int k = 0; k < NQ; ++k) {
    int32_t lo = off[k][0], hi = off[k][0];
#pragma unroll
    for (int jj = 1; jj < 4; ++jj) {
      lo = off[k][jj] < lo ? off[k][jj] : lo;
      hi = off[k][jj] > hi ? off[k][jj] : hi;
    }
    const int32_t span = hi - lo;
    two_dw[k] = span > 3;
    dw[k] = lo >= 0 && span <= 7 && lo + (two_dw[k] ? 7 : 3) < row_len;
    dbase[k] = lo < 0 ? 0 : lo;
    sel[k] = 0;
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) sel[k] |= static_cast<uint32_t>((off[k][jj] - lo) & 7) << (8 * jj);
  }
  typedef uint32_t u32_unaligned __attribute__((aligned(1)));
  for (int ri = 0; ri < nsrc; ri += 2) {
    const bool two = ri + 1 < nsrc;  // uniform
    const uint8_t* rp0 = sp + static_cast<int64_t>(rlo + ri) * p.s_sh;
    const uint8_t* rp1 = two ? rp0 + p.s_sh : rp0;
    uint32_t b[2][NQ][4];
#pragma unroll
    for (int k = 0; k < NQ; ++k) {
      if (dw[k]) {
        b[0][k][0] = *reinterpret_cast<const u32_unaligned*>(rp0 + dbase[k]);
        b[1][k][0] = *reinterpret_cast<const u32_unaligned*>(rp1 + dbase[k]);
        b[0][k][1] = two_dw[k] ? *reinterpret_cast<const u32_unaligned*>(rp0 + dbase[k] + 4) : 0u;
        b[1][k][1] = two_dw[k] ? *reinterpret_cast<const u32_unaligned*>(rp1 + dbase[k] + 4) : 0u;
      } else {
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
          const int32_t o = off[k][jj] < 0 ? 0 : off[k][jj];
          b[0][k][jj] = rp0[o];
          b[1][k][jj] = rp1[o];
        }
      }
    }
#pragma unroll
    for (int k = 0; k < NQ; ++k) {
      const int q = tid + kGThreads * k;
      if (q >= WORDS) continue;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        uint32_t w = 0;
        if (dw[k]) {
          w = __builtin_amdgcn_perm(b[h][k][1], b[h][k][0], sel[k]);  // bytes 0-3: first load, 4-7: second
        } else {
#pragma unroll
          for (int jj = 0; jj < 4; ++jj)
            if (off[k][jj] >= 0) w |= b[h][k][jj] << (8 * jj);
        }
        if (h == 0 || two) lds[(ri + h) * kGPitchWords + q] = w;
      }
    }
  }
#pragma unroll
  for (int k = 0; k < NQ; ++k)
    if (tid + kGThreads * k < WORDS) lds[zrow * kGPitchWords + tid + kGThreads * k] = 0u;
  __syncthreads();

  // ---- taps (uniform)
  Acc tap[K * K];
#pragma unroll
  for (int i = 0; i < K * K; ++i) tap[i] = static_cast<const Acc*>(p.taps)[i];

  // ---- walk the rows.  Tap row u of output row y reads upsampled row
  // t = row0 + y + u - R, i.e. source row q_u with t = q_u s + m_u; (q_u, m_u)
  // advance with y, so no division is needed inside the loop.
  int32_t qd[K], md[K];
#pragma unroll
  for (int u = 0; u < K; ++u) {
    const int64_t t = p.row0 + y0 + u - R;  // >= -R
    const uint32_t tp = static_cast<uint32_t>(t + 4 * p.s);  // shifted to stay non-negative
    qd[u] = static_cast<int32_t>(div_s(tp, p)) - 4;
    md[u] = static_cast<int32_t>(t - static_cast<int64_t>(qd[u]) * p.s);
  }
  const int32_t hlast = static_cast<int32_t>(p.H - 1);
  int32_t prev[K];
#pragma unroll
  for (int u = 0; u < K; ++u) prev[u] = -1;
  uint32_t outw[OUT == kOutU8 ? E / 4 : kGElems];
  const int64_t ebase = e0 + kGElems * tid;
  for (int64_t i = 0; i < nrow_out; ++i) {
    const int64_t y = y0 + i;
    int32_t ridx[K];
    bool same = i > 0;
#pragma unroll
    for (int u = 0; u < K; ++u) {
      const int64_t t = p.row0 + y + u - R;
      int32_t r;
      if (t < 0)
        r = p.zero ? zrow : -rlo;
      else if (t >= p.Hout)
        r = p.zero ? zrow : hlast - rlo;
      else
        r = qd[u] - rlo;
      ridx[u] = r;
      same = same && r == prev[u];
      prev[u] = r;
      if (++md[u] == p.s) {
        md[u] = 0;
        ++qd[u];
      }
    }
    if (!same) {
      Acc acc[kGElems];
#pragma unroll
      for (int j = 0; j < kGElems; ++j) acc[j] = Acc(0);
#pragma unroll
      for (int u = 0; u < K; ++u) {
        const uint32_t* row = lds + ridx[u] * kGPitchWords + (E / 4) * tid;
        uint32_t w[NW];
#pragma unroll
        for (int k2 = 0; k2 < NW; ++k2) w[k2] = row[k2];
#pragma unroll
        for (int v = 0; v < K; ++v)
#pragma unroll
          for (int j = 0; j < kGElems; ++j) {
            const int bi = j + v * P;
            const uint32_t byte = (w[bi >> 2] >> (8 * (bi & 3))) & 0xffu;
            if constexpr (TF)
              acc[j] = __builtin_fmaf(tap[u * K + v], static_cast<float>(byte), acc[j]);
            else
              acc[j] += byte * tap[u * K + v];
          }
      }
      if constexpr (OUT == kOutU8) {
        uint32_t q8[kGElems];
#pragma unroll
        for (int j = 0; j < kGElems; ++j) {
          if constexpr (TF) {
            const float v = __builtin_rintf(__builtin_amdgcn_fmed3f(acc[j], 0.0f, 255.0f));
            q8[j] = static_cast<uint32_t>(v);
          } else {
            const int32_t v = static_cast<int32_t>(acc[j]);
            q8[j] = static_cast<uint32_t>(v < 0 ? 0 : (v > 255 ? 255 : v));
          }
        }
#pragma unroll
        for (int w4 = 0; w4 < E / 4; ++w4)
          outw[w4] = q8[4 * w4] | (q8[4 * w4 + 1] << 8) | (q8[4 * w4 + 2] << 16) | (q8[4 * w4 + 3] << 24);
      } else {
#pragma unroll
        for (int j = 0; j < kGElems; ++j) outw[j] = __builtin_bit_cast(uint32_t, acc[j]);
      }
    }
    // ---- store the lane's 8 elements of row y
    if (ebase < L) {
      if constexpr (OUT == kOutU8) {
        uint8_t* dp = static_cast<uint8_t*>(p.dst) + n * p.d_sn + c * p.d_sc + y * p.d_sh + ebase;
        if (ebase + kGElems <= L) {
          store_words<E / 4>(dp, outw);
        } else {
#pragma unroll
          for (int j = 0; j < kGElems; ++j)
            if (ebase + j < L) dp[j] = static_cast<uint8_t>(outw[j >> 2] >> (8 * (j & 3)));
        }
      } else {
        uint32_t* dp = static_cast<uint32_t*>(p.dst) + n * p.d_sn + c * p.d_sc + y * p.d_sh + ebase;
        if (ebase + kGElems <= L) {
          store_words<kGElems>(reinterpret_cast<uint8_t*>(dp), outw);
        } else {
#pragma unroll
          for (int j = 0; j < kGElems; ++j)
            if (ebase + j < L) dp[j] = outw[j];
        }
      }
    }
  }
}

// ----------------------------------------------------- 3 x 3, 8-bit out --
//
// k_u8_direct: the paper's case (3 x 3 taps, 8-bit output, nearest upsample by
// 1 to 4).  k_u8_gather expands every row in LDS and then converts and
// multiplies each of an output's 9 bytes: 20 VALU and 14 scalar instructions
// per output byte, which held the 4K x2 sharpen at 78 us where its traffic
// takes 27.  Here a lane owns SPX neighbouring source pixels, loads each
// source row's (SPX + 2)-pixel window once, straight to registers, and
// produces the SPX * S output pixels of S output rows from the three windows
// around it: byte positions are compile-time constants, so a source byte is
// converted once for all its uses, equal outputs of the same source pixels are
// computed once, and there is no LDS, no barrier and no index arithmetic per
// output.  A wave walks down run_rows source rows of a 64 * SPX-pixel strip,
// its loads two rows ahead.  4K x2: 35 us, 3.5 TB/s of the 4.7 that a copy
// reaches.
//
// Whole-number taps (S <= 2; the paper's Laplacian) take 8-bit dot products:
// the sums are integers below 2^24, exact in any order, so taps that meet the
// same source byte are added first and four bytes go through one instruction.
// Larger factors repeat outputs, and the float chain is no slower there.
struct DirectParams {
  const uint8_t* src;
  int64_t s_sn, s_sc, s_sh;
  uint8_t* dst;
  int64_t d_sn, d_sc, d_sh;
  const void* taps;  // 9 int32 or float
  int64_t H, W;      // source image, pixels
  int64_t q0, q1;    // source rows whose output rows are produced (S = 1: the band; output row q*S - row_off)
  int64_t row_off;
  int32_t zero, planes_c, run_rows;
  int32_t strips, runs;
  int64_t n_waves;
};

// Source offset (-1, 0, 1) that tap t (0..2) of upsampled phase ph meets.
template <int S>
constexpr int phase_src(int ph, int t) {
  const int x = ph + t - 1;
  return x < 0 ? -1 : (x >= S ? 1 : 0);
}

template <int P, int S, int SPX>
struct DirectGeom {
  static constexpr int NE = SPX * S * P;             // output bytes of a lane and row
  static constexpr int NB = (SPX + 2) * P;           // window bytes of a source row
  static constexpr int NW = (NB + 3) / 4, NO = NE / 4;
  static constexpr bool DOT = S <= 2;
  static_assert(NE % 4 == 0, "whole words");
  // window byte of the source pixel at offset d from that of element e
  static constexpr int byte_of(int e, int d) { return (e / P / S + d + 1) * P + e % P; }
};

// One output row (phase r) of the lane from the windows of the source rows
// above, at and below it, in the order of the definition (taps u, then v).
template <int P, int S, int SPX, bool TF>
__device__ __forceinline__ void direct_row(const uint32_t (&w)[3][DirectGeom<P, S, SPX>::NW],
                                           const typename std::conditional<TF, float, uint32_t>::type (&tap)[9],
                                           int r, uint32_t (&o)[DirectGeom<P, S, SPX>::NO]) {
  using G = DirectGeom<P, S, SPX>;
  using Acc = typename std::conditional<TF, float, uint32_t>::type;
#pragma unroll
  for (int i = 0; i < G::NO; ++i) {
    uint32_t word = 0;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const int e = 4 * i + b;
      Acc acc = Acc(0);
#pragma unroll
      for (int u = 0; u < 3; ++u)
#pragma unroll
        for (int v = 0; v < 3; ++v) {
          const int at = G::byte_of(e, phase_src<S>(e / P % S, v));
          const uint32_t byte = (w[1 + phase_src<S>(r, u)][at / 4] >> (8 * (at % 4))) & 0xffu;
          if constexpr (TF)
            acc = __builtin_fmaf(tap[3 * u + v], static_cast<float>(byte), acc);
          else
            acc += byte * tap[3 * u + v];
        }
      uint32_t q;
      if constexpr (TF) {
        q = static_cast<uint32_t>(__builtin_rintf(__builtin_amdgcn_fmed3f(acc, 0.0f, 255.0f)));
      } else {
        const int32_t x = static_cast<int32_t>(acc);
        q = static_cast<uint32_t>(x < 0 ? 0 : (x > 255 ? 255 : x));
      }
      word |= q << (8 * b);
    }
    o[i] = word;
  }
}

// Tap words of the dot products: source row d (-1..1) of output phase r meets
// the sum of the tap rows u with phase_src(r, u) = d; within it, byte at of an
// element's window the sum of the taps v that meet it.
template <int P, int S>
struct DirectTaps {
  // [row phase][source row][column phase][byte alignment][word]
  uint32_t t[S][3][S][4][3];
  int32_t bias;
  bool fits;
  __device__ __forceinline__ void set(const int32_t (&tap)[9]) {
    fits = true;
    bias = 0;
#pragma unroll
    for (int i = 0; i < 9; ++i) bias += 128 * tap[i];
#pragma unroll
    for (int r = 0; r < S; ++r)
#pragma unroll
      for (int d = 0; d < 3; ++d)
#pragma unroll
        for (int c = 0; c < S; ++c) {
          int32_t sum[3];
#pragma unroll
          for (int x = 0; x < 3; ++x) {
            sum[x] = 0;
#pragma unroll
            for (int u = 0; u < 3; ++u)
#pragma unroll
              for (int v = 0; v < 3; ++v)
                if (phase_src<S>(r, u) == d - 1 && phase_src<S>(c, v) == x - 1) sum[x] += tap[3 * u + v];
            fits = fits && sum[x] >= -128 && sum[x] <= 127;
          }
#pragma unroll
          for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int q = 0; q < 3; ++q) {
              uint32_t word = 0;
#pragma unroll
              for (int x = 0; x < 3; ++x)
                if ((a + x * P) / 4 == q) word |= (static_cast<uint32_t>(sum[x]) & 0xffu) << (8 * ((a + x * P) % 4));
              t[r][d][c][a][q] = __builtin_amdgcn_readfirstlane(word);
            }
        }
  }
};

// direct_row through the dot products; the windows hold the bytes minus 128.
template <int P, int S, int SPX>
__device__ __forceinline__ void direct_row_dot(const uint32_t (&w)[3][DirectGeom<P, S, SPX>::NW],
                                               const DirectTaps<P, S>& tp, int r,
                                               uint32_t (&o)[DirectGeom<P, S, SPX>::NO]) {
  using G = DirectGeom<P, S, SPX>;
#pragma unroll
  for (int i = 0; i < G::NO; ++i) {
    uint32_t word = 0;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const int e = 4 * i + b, c = e / P % S, at = G::byte_of(e, -1);
      int32_t acc = tp.bias;
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        bool row = false;  // some tap row meets this source row
#pragma unroll
        for (int u = 0; u < 3; ++u) row = row || phase_src<S>(r, u) == d - 1;
        if (!row) continue;
#pragma unroll
        for (int q = 0; q < 3; ++q) {
          bool word_used = false;
#pragma unroll
          for (int v = 0; v < 3; ++v) word_used = word_used || (at % 4 + (phase_src<S>(c, v) + 1) * P) / 4 == q;
          if (word_used)
            acc = __builtin_amdgcn_sdot4(static_cast<int>(w[d][at / 4 + q]),
                                         static_cast<int>(tp.t[r][d][c][at % 4][q]), acc, false);
        }
      }
      word |= static_cast<uint32_t>(acc < 0 ? 0 : (acc > 255 ? 255 : acc)) << (8 * b);
    }
    o[i] = word;
  }
}

template <int P, int S, int SPX, bool TF>
__global__ __launch_bounds__(kGThreads) void k_u8_direct(DirectParams p) {
  using G = DirectGeom<P, S, SPX>;
  using Acc = typename std::conditional<TF, float, uint32_t>::type;
  const int lane = threadIdx.x % 64;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
  const int64_t item = xcd_remap(blockIdx.x, gridDim.x) * (kGThreads / 64) + wave;
  if (item >= p.n_waves) return;  // no barriers in this kernel
  const uint32_t it = static_cast<uint32_t>(item);
  const uint32_t rest = it / static_cast<uint32_t>(p.strips);
  const uint32_t strip = it - rest * p.strips;
  const uint32_t plane = rest / static_cast<uint32_t>(p.runs);
  const int64_t qa = p.q0 + static_cast<int64_t>(rest - plane * p.runs) * p.run_rows;
  const int64_t qb = qa + p.run_rows < p.q1 ? qa + p.run_rows : p.q1;
  const uint32_t n = plane / static_cast<uint32_t>(p.planes_c), c = plane - n * p.planes_c;
  const uint8_t* sp = p.src + n * p.s_sn + c * p.s_sc;
  uint8_t* dp = p.dst + n * p.d_sn + c * p.d_sc;
  const int64_t px = (static_cast<int64_t>(strip) * 64 + lane) * SPX;  // this lane's first source pixel
  if (px >= p.W) return;

  Acc tap[9];
#pragma unroll
  for (int i = 0; i < 9; ++i) tap[i] = static_cast<const Acc*>(p.taps)[i];
  bool dot = G::DOT;
  DirectTaps<P, G::DOT ? S : 1> tp;
  if constexpr (G::DOT) {
    int32_t ti[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) {
      if constexpr (TF) {
        const float t = tap[i] >= -128.0f && tap[i] <= 127.0f ? tap[i] : 0.5f;  // (also NaN)
        ti[i] = static_cast<int32_t>(t);
        dot = dot && static_cast<float>(ti[i]) == t;
      } else {
        ti[i] = static_cast<int32_t>(tap[i]);
        dot = dot && ti[i] >= -128 && ti[i] <= 127;
      }
    }
    if (!dot) {
#pragma unroll
      for (int i = 0; i < 9; ++i) ti[i] = 0;
    }
    tp.set(ti);
    dot = dot && tp.fits;
  }
  dot = __builtin_amdgcn_readfirstlane(dot) != 0;
  const uint32_t flip = dot ? 0x80808080u : 0u;

  // the window of source row q: clamped to the image, or zeros outside it
  auto clamp_row = [&](int64_t q) { return q < 0 ? 0 : (q >= p.H ? p.H - 1 : q); };
  auto finish = [&](int64_t q, uint32_t (&w)[G::NW]) {
    const uint32_t keep = p.zero && (q < 0 || q >= p.H) ? 0u : 0xffffffffu;  // uniform
#pragma unroll
    for (int i = 0; i < G::NW; ++i) w[i] = (w[i] & keep) ^ flip;
  };
  // every byte that load_words reads lies in the row, every pixel in the
  // image, for each lane of the wave (uniform)
  const bool mine = px >= 1 && (px - 1) * P + 4 * G::NW <= p.W * P && px + SPX <= p.W;
  const bool inside = __ballot(!mine) == 0;
  const uint8_t* wa = sp + (px - 1) * P;
  auto load = [&](int64_t q, uint32_t (&w)[G::NW]) { load_words<G::NW>(wa + clamp_row(q) * p.s_sh, w); };
  // at the ends of the rows: byte by byte, packed when the row is needed
  auto load_bytes = [&](int64_t q, uint32_t (&v)[G::NB]) {
    const uint8_t* row = sp + clamp_row(q) * p.s_sh;
#pragma unroll
    for (int x = 0; x < SPX + 2; ++x) {
      const int64_t g = px + x - 1, gc = g < 0 ? 0 : (g >= p.W ? p.W - 1 : g);
#pragma unroll
      for (int ch = 0; ch < P; ++ch) v[x * P + ch] = row[gc * P + ch];
    }
  };
  auto pack = [&](const uint32_t (&v)[G::NB], uint32_t (&w)[G::NW]) {
#pragma unroll
    for (int i = 0; i < G::NW; ++i) w[i] = 0;
#pragma unroll
    for (int x = 0; x < SPX + 2; ++x) {
      const int64_t g = px + x - 1;
      const bool out = p.zero && (g < 0 || g >= p.W);
#pragma unroll
      for (int ch = 0; ch < P; ++ch) {
        const int at = x * P + ch;
        w[at / 4] |= (out ? 0u : v[at]) << (8 * (at % 4));
      }
    }
  };
  auto row_out = [&](const uint32_t (&w)[3][G::NW], int r, uint32_t (&o)[G::NO]) {
    if constexpr (G::DOT) {
      if (dot) {  // uniform
        direct_row_dot<P, S, SPX>(w, tp, r, o);
        return;
      }
    }
    direct_row<P, S, SPX, TF>(w, tap, r, o);
  };

  uint32_t w[3][G::NW], nx[G::NW];
  if (inside) {
    load(qa - 1, w[0]);
    load(qa, w[1]);
    load(qa + 1, w[2]);
    load(qa + 2, nx);
    finish(qa - 1, w[0]);
    finish(qa, w[1]);
    finish(qa + 1, w[2]);
    uint8_t* d = dp + (qa * S - p.row_off) * p.d_sh + px * S * P;
    for (int64_t q = qa; q < qb; ++q) {
      uint32_t n2[G::NW];
      load(q + 3, n2);
#pragma unroll
      for (int r = 0; r < S; ++r) {
        uint32_t o[G::NO];
        row_out(w, r, o);
        store_words<G::NO>(d, o);
        d += p.d_sh;
      }
      finish(q + 2, nx);
#pragma unroll
      for (int i = 0; i < G::NW; ++i) {
        w[0][i] = w[1][i];
        w[1][i] = w[2][i];
        w[2][i] = nx[i];
        nx[i] = n2[i];
      }
    }
  } else {
    uint32_t v[G::NB];
    load_bytes(qa - 1, v);
    pack(v, w[0]);
    load_bytes(qa, v);
    pack(v, w[1]);
    load_bytes(qa + 1, v);
    pack(v, w[2]);
    finish(qa - 1, w[0]);
    finish(qa, w[1]);
    finish(qa + 1, w[2]);
    const int64_t bytes = (p.W - px) * S * P;  // of this lane inside the image
    for (int64_t q = qa; q < qb; ++q) {
      load_bytes(q + 2, v);
#pragma unroll
      for (int r = 0; r < S; ++r) {
        uint32_t o[G::NO];
        row_out(w, r, o);
        uint8_t* d = dp + (q * S + r - p.row_off) * p.d_sh + px * S * P;
        if (bytes >= G::NE) {
          store_words<G::NO>(d, o);
        } else {
#pragma unroll
          for (int e = 0; e < G::NE; ++e)
            if (e < bytes) d[e] = static_cast<uint8_t>(o[e / 4] >> (8 * (e % 4)));
        }
      }
      pack(v, nx);
      finish(q + 2, nx);
#pragma unroll
      for (int i = 0; i < G::NW; ++i) {
        w[0][i] = w[1][i];
        w[1][i] = w[2][i];
        w[2][i] = nx[i];
      }
    }
  }
}

// ------------------------------------------------------------- channel mix --

struct MixParams {
  const uint8_t* src;
  int64_t s_sn, s_sc, s_sh, s_sw;  // elements; interleaved: s_sc = 1, s_sw = CIN
  void* dst;
  int64_t d_sn, d_sc, d_sh, d_sw;  // elements of the output type
  const void* w;                   // [cout][CIN], int32 or float
  int32_t cout;
  int64_t W, row0, rows;  // output rows [row0, row0 + rows) of the buffer
  int32_t tiles_x;        // 1024-pixel segments per row
  int64_t n_blocks;
};

constexpr int kMixThreads = 256;
constexpr int kMixPx = 16;  // pixels per lane (measured: 8K gray 0.048 ms with 4)

// WHOLE: W is a multiple of a lane's 16 pixels (with the tests of the last lane
// in it the kernel took 23.6 us on the 8K frame, 22.2 without).
template <int CIN, bool TF, int OUT, bool WHOLE>
__global__ __launch_bounds__(kMixThreads) void k_u8_mix(MixParams p) {
  using Acc = typename std::conditional<TF, float, uint32_t>::type;
  const int64_t b = xcd_remap(blockIdx.x, p.n_blocks);
  const int64_t per_img = p.rows * p.tiles_x;
  const int64_t n = b / per_img;
  const int64_t rem = b - n * per_img;
  const int64_t y = rem / p.tiles_x;
  const int64_t x0 = (rem - y * p.tiles_x) * (kMixThreads * kMixPx) + kMixPx * threadIdx.x;
  if (x0 >= p.W) return;
  // the row's last lane loads the 16 pixels that end with the row, and stores
  // its own, [lo, hi) of them: a wave that also loaded by bytes paid for both
  // (8-bit gray of 62 x 62: 4.15 us, 3.95 by bytes alone)
  const bool full = WHOLE || p.W >= kMixPx;
  const int64_t xs = !WHOLE && full && x0 + kMixPx > p.W ? p.W - kMixPx : x0;
  const int lo = static_cast<int>(x0 - xs);
  const int hi = full ? kMixPx : static_cast<int>(p.W - xs);
  const uint8_t* rp = p.src + n * p.s_sn + (p.row0 + y) * p.s_sh;

  // x[i][k]: channel i of pixel x0 + k
  uint32_t x[CIN][kMixPx];
  if (p.s_sw == CIN && p.s_sc == 1 && CIN > 1) {  // interleaved
    if (full) {
      uint32_t wd[CIN * kMixPx / 4];
      load_words<CIN * kMixPx / 4>(rp + xs * CIN, wd);
#pragma unroll
      for (int k = 0; k < kMixPx; ++k)
#pragma unroll
        for (int i = 0; i < CIN; ++i) {
          const int bi = k * CIN + i;
          x[i][k] = (wd[bi >> 2] >> (8 * (bi & 3))) & 0xffu;
        }
    } else {
#pragma unroll
      for (int k = 0; k < kMixPx; ++k)
#pragma unroll
        for (int i = 0; i < CIN; ++i) x[i][k] = k < hi ? rp[(xs + k) * CIN + i] : 0u;
    }
  } else {  // planar
#pragma unroll
    for (int i = 0; i < CIN; ++i) {
      const uint8_t* cp = rp + i * p.s_sc;
      if (full) {
        uint32_t wd[kMixPx / 4];
        load_words<kMixPx / 4>(cp + xs, wd);
#pragma unroll
        for (int k = 0; k < kMixPx; ++k) x[i][k] = (wd[k >> 2] >> (8 * (k & 3))) & 0xffu;
      } else {
#pragma unroll
        for (int k = 0; k < kMixPx; ++k) x[i][k] = k < hi ? cp[(xs + k) * p.s_sw] : 0u;
      }
    }
  }

  const Acc* w = static_cast<const Acc*>(p.w);
#pragma unroll
  for (int o = 0; o < 4; ++o) {
    if (o >= p.cout) break;
    Acc acc[kMixPx];
#pragma unroll
    for (int k = 0; k < kMixPx; ++k) acc[k] = Acc(0);
#pragma unroll
    for (int i = 0; i < CIN; ++i) {
      const Acc wi = w[o * CIN + i];
#pragma unroll
      for (int k = 0; k < kMixPx; ++k) {
        if constexpr (TF)
          acc[k] = __builtin_fmaf(wi, static_cast<float>(x[i][k]), acc[k]);
        else
          acc[k] += x[i][k] * wi;
      }
    }
    const int64_t obase = n * p.d_sn + o * p.d_sc + (y)*p.d_sh;
    if constexpr (OUT == kOutU8) {
      uint32_t q8[kMixPx];
#pragma unroll
      for (int k = 0; k < kMixPx; ++k) {
        if constexpr (TF) {
          q8[k] = static_cast<uint32_t>(__builtin_rintf(__builtin_amdgcn_fmed3f(acc[k], 0.0f, 255.0f)));
        } else {
          const int32_t v = static_cast<int32_t>(acc[k]);
          q8[k] = static_cast<uint32_t>(v < 0 ? 0 : (v > 255 ? 255 : v));
        }
      }
      uint8_t* dp = static_cast<uint8_t*>(p.dst) + obase;
      if (full && lo == 0 && p.d_sw == 1) {
        uint32_t ow[kMixPx / 4];
#pragma unroll
        for (int q = 0; q < kMixPx / 4; ++q)
          ow[q] = q8[4 * q] | (q8[4 * q + 1] << 8) | (q8[4 * q + 2] << 16) | (q8[4 * q + 3] << 24);
        store_words<kMixPx / 4>(dp + x0, ow);
      } else {
#pragma unroll
        for (int k = 0; k < kMixPx; ++k)
          if (k >= lo && k < hi) dp[(xs + k) * p.d_sw] = static_cast<uint8_t>(q8[k]);
      }
    } else {
      uint32_t* dp = static_cast<uint32_t*>(p.dst) + obase;
      if (full && lo == 0 && p.d_sw == 1) {
        uint32_t ow[kMixPx];
#pragma unroll
        for (int k = 0; k < kMixPx; ++k) ow[k] = __builtin_bit_cast(uint32_t, acc[k]);
        store_words<kMixPx>(reinterpret_cast<uint8_t*>(dp + x0), ow);
      } else {
#pragma unroll
        for (int k = 0; k < kMixPx; ++k)
          if (k >= lo && k < hi) dp[(xs + k) * p.d_sw] = __builtin_bit_cast(uint32_t, acc[k]);
      }
    }
  }
}

// ------------------------------------------------------------------ host ----

int64_t eff_sw(const f2d_tensor& t) { return t.stride_w <= 0 ? 1 : t.stride_w; }

// Interleaved: channels adjacent (stride_c 1) and pixels C apart, C > 1.
bool interleaved(const f2d_tensor& t) { return t.c > 1 && t.stride_c == 1 && eff_sw(t) == t.c; }

template <int K, int P, bool TF, int OUT, int E>
hipError_t launch_gather_one(const GatherParams& g, hipStream_t s) {
  const void* kern = reinterpret_cast<const void*>(k_u8_gather<K, P, TF, OUT, E>);
  const size_t lds = static_cast<size_t>(g.lds_rows + 1) * GTile<E>::PITCH_WORDS * 4;
  if (lds > 64 * 1024) {
    hipError_t e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((k_u8_gather<K, P, TF, OUT, E>), dim3(static_cast<uint32_t>(g.n_blocks)), dim3(kGThreads), lds,
                     s, g);
  return hipGetLastError();
}

// 16 elements per lane for 8-bit outputs of images upsampled by 8 or more, else 8
template <int K, int P>
hipError_t launch_gather_kp(const GatherParams& g, bool tf, int out, int e, hipStream_t s) {
  if (out == kOutU8) {
    if (e == 16)
      return tf ? launch_gather_one<K, P, true, kOutU8, 16>(g, s) : launch_gather_one<K, P, false, kOutU8, 16>(g, s);
    return tf ? launch_gather_one<K, P, true, kOutU8, 8>(g, s) : launch_gather_one<K, P, false, kOutU8, 8>(g, s);
  }
  return tf ? launch_gather_one<K, P, true, kOutF32, 8>(g, s) : launch_gather_one<K, P, false, kOutI32, 8>(g, s);
}

template <int K>
hipError_t launch_gather_k(const GatherParams& g, int P, bool tf, int out, int e, hipStream_t s) {
  switch (P) {
    case 1: return launch_gather_kp<K, 1>(g, tf, out, e, s);
    case 3: return launch_gather_kp<K, 3>(g, tf, out, e, s);
    default: return launch_gather_kp<K, 4>(g, tf, out, e, s);
  }
}

int out_kind(int32_t dtype) { return dtype == F2D_U8 ? kOutU8 : (dtype == F2D_F32 ? kOutF32 : kOutI32); }

template <int P, int S, int SPX>
hipError_t launch_direct_one(DirectParams d, int64_t planes, bool tf, hipStream_t s) {
  d.strips = static_cast<int32_t>((d.W + 64 * SPX - 1) / (64 * SPX));
  const int64_t rows = d.q1 - d.q0;
  // 8 source rows per wave (two halo rows each), fewer where that leaves the
  // GPU's 8192 wave slots half empty
  int64_t run = 8;
  while (run > 2 && planes * d.strips * ((rows + run - 1) / run) < 4096) run /= 2;
  d.run_rows = static_cast<int32_t>(run);
  d.runs = static_cast<int32_t>((rows + run - 1) / run);
  d.n_waves = planes * d.strips * d.runs;
  const int64_t blocks = (d.n_waves + kGThreads / 64 - 1) / (kGThreads / 64);
  if (blocks <= 0) return hipSuccess;
  const dim3 grid(static_cast<uint32_t>(blocks)), block(kGThreads);
  if (tf) hipLaunchKernelGGL((k_u8_direct<P, S, SPX, true>), grid, block, 0, s, d);
  else hipLaunchKernelGGL((k_u8_direct<P, S, SPX, false>), grid, block, 0, s, d);
  return hipGetLastError();
}

// Source pixels per lane: whole words of output, and strips narrow enough that
// few of a row's waves hold its ends (those load by bytes: 16 planar pixels per
// lane at x1 took 35 us on three 4K planes, 8 take 25, 4 take 30).
hipError_t launch_direct(const DirectParams& d, int64_t planes, int P, int scale, bool tf, hipStream_t s) {
  switch (P * 8 + scale) {
    case 1 * 8 + 1: return launch_direct_one<1, 1, 8>(d, planes, tf, s);
    case 1 * 8 + 2: return launch_direct_one<1, 2, 4>(d, planes, tf, s);
    case 1 * 8 + 3: return launch_direct_one<1, 3, 4>(d, planes, tf, s);
    case 1 * 8 + 4: return launch_direct_one<1, 4, 4>(d, planes, tf, s);
    case 3 * 8 + 1: return launch_direct_one<3, 1, 4>(d, planes, tf, s);
    case 3 * 8 + 2: return launch_direct_one<3, 2, 4>(d, planes, tf, s);
    case 3 * 8 + 3: return launch_direct_one<3, 3, 4>(d, planes, tf, s);
    case 3 * 8 + 4: return launch_direct_one<3, 4, 1>(d, planes, tf, s);
    case 4 * 8 + 1: return launch_direct_one<4, 1, 4>(d, planes, tf, s);
    case 4 * 8 + 2: return launch_direct_one<4, 2, 2>(d, planes, tf, s);
    case 4 * 8 + 3: return launch_direct_one<4, 3, 4>(d, planes, tf, s);
    default: return launch_direct_one<4, 4, 1>(d, planes, tf, s);
  }
}

// SHARED filter on an 8-bit image, optional nearest upsample by `scale`.
f2d_status gather_forward(const Problem& pr, const f2d_tensor& out, int32_t scale, hipStream_t s) {
  const f2d_tensor& im = pr.image;
  const bool il = interleaved(im);
  if (!il && eff_sw(im) != 1) return fail(F2D_EUNSUPPORTED, "u8 images: planar or interleaved (stride_c 1, stride_w C) layouts");
  const int P = il ? static_cast<int>(im.c) : 1;
  if (il && P != 3 && P != 4) return fail(F2D_EUNSUPPORTED, "interleaved u8 images: 3 or 4 channels");
  if (il != interleaved(out) || (!il && eff_sw(out) != 1))
    return fail(F2D_EINVAL, "the output must have the image's layout (planar, or interleaved with the same channels)");
  if (pr.k > 7) return fail(F2D_EUNSUPPORTED, "u8 zero-border / u8-output / float-tap / upsampled filters: k <= 7 (got %d)", pr.k);
  const bool tf = pr.filter.dtype == F2D_F32;
  const int ok_out = out_kind(out.dtype);
  if ((tf && ok_out == kOutI32) || (!tf && ok_out == kOutF32))
    return fail(F2D_EINVAL, "u8 images: int32 taps give int32 or u8 outputs, float taps give f32 or u8 outputs");
  GatherParams g;
  std::memset(&g, 0, sizeof(g));
  g.src = static_cast<const uint8_t*>(im.data);
  g.s_sn = im.stride_n;
  g.s_sc = il ? 0 : im.stride_c;
  g.s_sh = im.stride_h;
  g.dst = out.data;
  g.d_sn = out.stride_n;
  g.d_sc = il ? 0 : out.stride_c;
  g.d_sh = out.stride_h;
  g.taps = pr.filter.data;
  g.H = im.h;
  g.W = im.w;
  g.s = scale;
  g.Hout = im.h * scale;
  g.Wout = im.w * scale;
  g.row0 = pr.row_begin;
  g.out_rows = scale == 1 ? pr.rows : g.Hout;
  g.zero = pr.opts.border == F2D_BORDER_ZERO ? 1 : 0;
  g.planes_c = il ? 1 : static_cast<int32_t>(im.c);
  const int64_t L = g.Wout * P;
  if (L > (int64_t{1} << 30) || g.Hout > (int64_t{1} << 30))
    return fail(F2D_EUNSUPPORTED, "u8 filter: output rows of at most 2^30 elements and 2^30 rows");
  // 3 x 3 into bytes, factors to 4: k_u8_direct (4K interleaved, gather /
  // direct: x1 36 / 28 us, x2 76 / 35, x3 134 / 75, x4 199 / 107).  Larger
  // factors are bound by their stores either way and stay with the gather, and
  // so do images of fewer than 32 columns, all of whose waves hold an end of
  // the rows and load by bytes (64 x 3 x 5^2 x1 8.9 / 11.4, 64 x 3 x 30^2 x3 22.4 /
  // 26.2, 64 x 4 x 30^2 x3 18.9 / 32.6; none slower from 33 on).
  if (pr.k == 3 && ok_out == kOutU8 && scale <= 4 && im.w >= 32) {
    DirectParams d;
    std::memset(&d, 0, sizeof(d));
    d.src = g.src;
    d.s_sn = g.s_sn;
    d.s_sc = g.s_sc;
    d.s_sh = g.s_sh;
    d.dst = static_cast<uint8_t*>(out.data);
    d.d_sn = g.d_sn;
    d.d_sc = g.d_sc;
    d.d_sh = g.d_sh;
    d.taps = g.taps;
    d.H = g.H;
    d.W = g.W;
    d.q0 = scale == 1 ? pr.row_begin : 0;
    d.q1 = scale == 1 ? pr.row_end : im.h;
    d.row_off = scale == 1 ? pr.row_begin : 0;
    d.zero = g.zero;
    d.planes_c = g.planes_c;
    const int64_t planes = im.n * g.planes_c;
    if (planes * ((im.h + 1) / 2) * ((im.w + 63) / 64) < (int64_t{1} << 31))  // wave numbers fit in 32 bits
      return hip_status(launch_direct(d, planes, P, scale, tf, s), "u8 3x3 filter launch");
  }
  // Tile height: 16 rows without upsampling; with it, about 8 source rows
  // per tile (rows inside an upsampled block repeat, so the work per tile is
  // set by its source rows), at most 512 rows.  LDS holds the tile's source
  // rows: at most (th + 2r - 1) / s + 2 of them.
  const int R = (pr.k - 1) / 2;
  g.th = scale == 1 ? 16 : static_cast<int32_t>(std::min<int64_t>(512, 8 * static_cast<int64_t>(scale)));
  g.lds_rows = std::min(g.th + 2 * R, (g.th + 2 * R - 1) / scale + 2);
  if (scale > 1) {
    int l = 0;
    while ((int64_t{1} << l) < scale) ++l;
    g.s_shift = l - 1;
    g.s_magic = static_cast<uint32_t>((((uint64_t{1} << 32) * ((uint64_t{1} << l) - scale)) / scale) + 1);
  }
  // 16-byte stores measured faster at x20 (1.93 against 2.28 ms on a 4K frame), 8-byte ones at x2 and x4
  const int elems = ok_out == kOutU8 && scale >= 8 ? 16 : 8;
  const int64_t tw = static_cast<int64_t>(kGThreads) * elems;
  g.tiles_x = static_cast<int32_t>((L + tw - 1) / tw);
  g.tiles_y = static_cast<int32_t>((g.out_rows + g.th - 1) / g.th);
  g.n_blocks = im.n * g.planes_c * static_cast<int64_t>(g.tiles_x) * g.tiles_y;
  if (g.n_blocks > kMaxBlocks) return fail(F2D_EUNSUPPORTED, "u8 filter: too many tiles for one launch");
  if (g.n_blocks == 0) return ok();
  hipError_t err;
  switch (pr.k) {
    case 1: err = launch_gather_k<1>(g, P, tf, ok_out, elems, s); break;
    case 3: err = launch_gather_k<3>(g, P, tf, ok_out, elems, s); break;
    case 5: err = launch_gather_k<5>(g, P, tf, ok_out, elems, s); break;
    default: err = launch_gather_k<7>(g, P, tf, ok_out, elems, s); break;
  }
  return hip_status(err, "u8 filter launch");
}

template <int CIN, bool WHOLE>
hipError_t launch_mix_w(const MixParams& m, bool tf, int out, hipStream_t s) {
  const dim3 grid(static_cast<uint32_t>(m.n_blocks)), block(kMixThreads);
  if (tf) {
    if (out == kOutU8) hipLaunchKernelGGL((k_u8_mix<CIN, true, kOutU8, WHOLE>), grid, block, 0, s, m);
    else hipLaunchKernelGGL((k_u8_mix<CIN, true, kOutF32, WHOLE>), grid, block, 0, s, m);
  } else {
    if (out == kOutU8) hipLaunchKernelGGL((k_u8_mix<CIN, false, kOutU8, WHOLE>), grid, block, 0, s, m);
    else hipLaunchKernelGGL((k_u8_mix<CIN, false, kOutI32, WHOLE>), grid, block, 0, s, m);
  }
  return hipGetLastError();
}
template <int CIN>
hipError_t launch_mix_c(const MixParams& m, bool tf, int out, hipStream_t s) {
  return m.W % kMixPx == 0 ? launch_mix_w<CIN, true>(m, tf, out, s) : launch_mix_w<CIN, false>(m, tf, out, s);
}

// BANK with K = 1 on an 8-bit image: per-pixel channel mixing.
f2d_status mix_forward(const Problem& pr, const f2d_tensor& out, hipStream_t s) {
  const f2d_tensor& im = pr.image;
  if (pr.k != 1) return fail(F2D_EUNSUPPORTED, "u8 images in BANK mode: k = 1 (per-pixel channel mixing) only");
  if (im.c > 4 || pr.c_out > 4) return fail(F2D_EUNSUPPORTED, "u8 channel mixing: at most 4 input and 4 output channels");
  const bool il = interleaved(im);
  if (!il && eff_sw(im) != 1) return fail(F2D_EUNSUPPORTED, "u8 images: planar or interleaved layouts");
  if (!interleaved(out) && eff_sw(out) != 1) return fail(F2D_EUNSUPPORTED, "u8 channel mixing: planar or interleaved outputs");
  const bool tf = pr.filter.dtype == F2D_F32;
  const int ok_out = out_kind(out.dtype);
  if ((tf && ok_out == kOutI32) || (!tf && ok_out == kOutF32))
    return fail(F2D_EINVAL, "u8 images: int32 weights give int32 or u8 outputs, float weights give f32 or u8 outputs");
  MixParams m;
  std::memset(&m, 0, sizeof(m));
  m.src = static_cast<const uint8_t*>(im.data);
  m.s_sn = im.stride_n;
  m.s_sc = im.stride_c;
  m.s_sh = im.stride_h;
  m.s_sw = eff_sw(im);
  m.dst = out.data;
  m.d_sn = out.stride_n;
  m.d_sc = out.stride_c;
  m.d_sh = out.stride_h;
  m.d_sw = eff_sw(out);
  m.w = pr.filter.data;
  m.cout = static_cast<int32_t>(pr.c_out);
  m.W = im.w;
  m.row0 = pr.row_begin;
  m.rows = pr.rows;
  m.tiles_x = static_cast<int32_t>((im.w + kMixThreads * kMixPx - 1) / (kMixThreads * kMixPx));
  m.n_blocks = im.n * m.rows * m.tiles_x;
  if (m.n_blocks > kMaxBlocks) return fail(F2D_EUNSUPPORTED, "u8 channel mixing: too many tiles for one launch");
  if (m.n_blocks == 0) return ok();
  hipError_t e;
  switch (im.c) {
    case 1: e = launch_mix_c<1>(m, tf, ok_out, s); break;
    case 2: e = launch_mix_c<2>(m, tf, ok_out, s); break;
    case 3: e = launch_mix_c<3>(m, tf, ok_out, s); break;
    default: e = launch_mix_c<4>(m, tf, ok_out, s); break;
  }
  return hip_status(e, "u8 channel mixing launch");
}

}  // namespace

// 8-bit images beyond the integer Sobel path: zero borders, float taps, u8
// outputs, interleaved layouts (SHARED), and channel mixing (BANK, K = 1).
f2d_status forward_u8_image(const Problem& pr, const f2d_tensor* outs, int32_t n_outs, hipStream_t s) {
  if (pr.mode == F2D_CH_DEPTHWISE)
    return fail(F2D_EUNSUPPORTED, "u8 DEPTHWISE filters: int32 taps, int32 outputs, clamp borders, planar layout");
  if (n_outs != 1) return fail(F2D_EINVAL, "expected one output");
  if (pr.mode == F2D_CH_BANK) return mix_forward(pr, outs[0], s);
  return gather_forward(pr, outs[0], 1, s);
}

f2d_status run_upsample_forward(const Problem& pr, int32_t scale, const f2d_tensor& out, hipStream_t s) {
  if (pr.image.n == 0 || pr.image.h == 0 || pr.image.w == 0 || pr.image.c == 0) return ok();
  return gather_forward(pr, out, scale, s);
}

}  // namespace f2d
