// FP32 filter banks on the matrix cores (v_mfma_f32_16x16x4_f32: FP32
// operands, FP32 products and sums, twice the rate of unpacked FP32 FMAs).
//
//  k_bank_f32_conv   Y[n][o] = sum_c corr(X[n][c], F[o][c]) (forward) or its
//                    adjoint in the image, as an implicit GEMM per tap: rows
//                    are 16 neighbouring pixels, columns 16 output channels,
//                    the contraction 4 source channels.  A wave holds the
//                    weights of its 16 outputs and 8 source channels in
//                    registers (one value per lane, tap and 4 channels); the
//                    source tile is in LDS as FP32 channel planes.
//
// Bound by the matrix cores: 154.6 TFLOP/s in a large FP32 product on this
// card (the clock falls to 2.2 GHz under it).  16 x 16 x 1024^2 -> 64, 3 x 3:
// forward 6.25 -> 2.88 ms (107 TFLOP/s; at 32 images 6.2 ms with the matrix
// cores busy 73% of the cycles at 2.1 GHz), grad_input 7.32 -> 3.1 ms,
// grad_filter 8.68 -> 2.95 ms against the VALU kernels, which stay for shapes
// that the padding to 4 x 16 channels makes slower here (bank_f32_conv_mfma,
// bank_f32_adjoint_mfma, bank_f32_wgrad_mfma).
//
//  k_bank_f32_wgrad  F-bar[o][c][u][v] = sum_p G[o][p] X[c][p + (u, v)]: per
//                    tap a 16 x 16 block of (output, source) channels
//                    contracted over pixels, rows of both operands streamed
//                    through LDS.
#include <hip/hip_runtime.h>

#include <cstring>
#include <mutex>

#include "bank_f32.hpp"
#include "f2d_host.hpp"
#include "f2d_internal.hpp"
#include "grad_internal.hpp"

namespace f2d {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4_u __attribute__((ext_vector_type(4), aligned(4)));  // any 4-byte aligned address
typedef float f32x2_u __attribute__((ext_vector_type(2), aligned(4)));

constexpr int kThreads = 256;

__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// ------------------------------------------------ forward and image adjoint --

// Four waves: OW of them take different blocks of 16 outputs, the 4 / OW
// others different column ranges (NCG groups of 16 pixels) of the 8-row tile.
template <int K, int OW>
struct ConvF32Geom {
  static constexpr int R = (K - 1) / 2;
  static constexpr int TH = 8;
  static constexpr int NCG = OW == 1 ? 1 : 2;
  static constexpr int TW = 16 * NCG * (4 / OW);
  static constexpr int HALO = R > 0 ? 4 : 0;  // staged columns left and right of the tile
  static constexpr int LW = TW + 2 * HALO;
  static constexpr int LH = TH + K - 1;
  static constexpr int CK = 8;     // source channels staged at a time
  // plane stride: the 4 planes that one operand read touches start 16 banks
  // apart, so its 4 x 16 words fall in 64 different banks
  static constexpr int plane_stride() {
    int p = LH * LW;
    while (p % 64 != 16 && p % 64 != 48) p += 4;
    return p;
  }
  static constexpr int PS = plane_stride();
  static constexpr int LWC = LW / 4;           // 16-byte chunks per staged row
  static constexpr int CPP = LH * LWC;         // chunks of a plane
  static constexpr int PPI = kThreads / CPP;   // planes staged by one load of every thread
  static_assert(PPI >= 1 && CK % PPI == 0, "every load of a thread is the same chunk of another plane");
  static constexpr int NT = CK / PPI;
};

struct ConvF32Tile {
  int64_t n, oy0, ox0;  // oy0: band-relative; ox0: output column (may be < 0 for the adjoint)
  int og;
};

template <int K, int OW>
__device__ __forceinline__ ConvF32Tile conv_tile(const BankF32Params& p, uint32_t t) {
  using G = ConvF32Geom<K, OW>;
  ConvF32Tile r;
  const uint32_t per_og = t / static_cast<uint32_t>(p.o_groups);
  r.og = static_cast<int>(t - per_og * p.o_groups);
  const uint32_t rows = per_og / static_cast<uint32_t>(p.tiles_x);
  r.ox0 = p.col0 + static_cast<int64_t>(per_og - rows * p.tiles_x) * G::TW;
  const uint32_t n = rows / static_cast<uint32_t>(p.tiles_y);
  r.n = n;
  r.oy0 = static_cast<int64_t>(rows - n * p.tiles_y) * G::TH;
  return r;
}

// This thread's chunk of every PPI-th staged plane,
// starting at plane `half`.
template <int K, int OW>
struct ConvF32Chunk {
  int half, ly, ch;
  bool act;
  __device__ __forceinline__ ConvF32Chunk() {
    using G = ConvF32Geom<K, OW>;
    const int tid = threadIdx.x;
    act = tid < G::PPI * G::CPP;
    const int idx = act ? tid : G::PPI * G::CPP - 1;
    half = idx / G::CPP;
    const int rest = idx - half * G::CPP;
    ly = rest / G::LWC;
    ch = rest - ly * G::LWC;
  }
};

// A thread's loads of channels c0 .. c0+CK-1 of a tile: one row address, and
// a uniform step of PPI planes from load to load.  The row is clamped to the
// image and the chunk to the nearest one inside the row (W >= 4); conv_write
// picks the clamped columns, or zeros, from it.
template <int K, int OW>
__device__ __forceinline__ void conv_load(const BankF32Params& p, const ConvF32Chunk<K, OW>& k, const ConvF32Tile& t,
                                          int c0, f32x4 (&v)[ConvF32Geom<K, OW>::NT]) {
  using G = ConvF32Geom<K, OW>;
  int64_t gy = p.row0 + t.oy0 - G::R + k.ly;
  gy = gy < 0 ? 0 : (gy >= p.H ? p.H - 1 : gy);
  int64_t gx = t.ox0 - G::HALO + 4 * k.ch;
  gx = gx < 0 ? 0 : (gx > p.W - 4 ? p.W - 4 : gx);
  const float* a = p.src + t.n * p.s_sn + gy * p.s_sh + gx;
  const int last = p.CI - 1;
#pragma unroll
  for (int i = 0; i < G::NT; ++i) {
    const int c = c0 + G::PPI * i + k.half;
    v[i] = *reinterpret_cast<const f32x4_u*>(a + (c < last ? c : last) * p.s_sc);
  }
}

template <int K, int OW>
__device__ __forceinline__ void conv_write(const BankF32Params& p, const ConvF32Chunk<K, OW>& k, const ConvF32Tile& t,
                                           int c0, const f32x4 (&v)[ConvF32Geom<K, OW>::NT],
                                           float* __restrict__ lds) {
  using G = ConvF32Geom<K, OW>;
  if (!k.act) return;
  const int64_t gy = p.row0 + t.oy0 - G::R + k.ly, gx0 = t.ox0 - G::HALO;
  const bool row_in = !p.zero || (gy >= 0 && gy < p.H);
  float* d = lds + k.half * G::PS + k.ly * G::LW + 4 * k.ch;
  if (gx0 >= 0 && gx0 + G::LW <= p.W) {  // uniform: every chunk inside the row
#pragma unroll
    for (int i = 0; i < G::NT; ++i) {
      const bool keep = row_in && c0 + G::PPI * i + k.half < p.CI;
      f32x4 w;
#pragma unroll
      for (int e = 0; e < 4; ++e) w[e] = keep ? v[i][e] : 0.0f;
      *reinterpret_cast<f32x4*>(d + i * G::PPI * G::PS) = w;
    }
  } else {
    const int64_t gx = gx0 + 4 * k.ch;
    const int64_t gl = gx < 0 ? 0 : (gx > p.W - 4 ? p.W - 4 : gx);  // the loaded chunk
    int from[4];
    bool in[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int64_t x = gx + e < 0 ? 0 : (gx + e >= p.W ? p.W - 1 : gx + e);
      from[e] = static_cast<int>(x - gl);
      in[e] = row_in && (!p.zero || x == gx + e);
    }
#pragma unroll
    for (int i = 0; i < G::NT; ++i) {
      const bool real = c0 + G::PPI * i + k.half < p.CI;
      f32x4 w;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float lo = from[e] == 0 ? v[i][0] : v[i][1], hi = from[e] == 2 ? v[i][2] : v[i][3];
        w[e] = real && in[e] ? (from[e] < 2 ? lo : hi) : 0.0f;
      }
      *reinterpret_cast<f32x4*>(d + i * G::PPI * G::PS) = w;
    }
  }
}

// acc[cg][y] += the staged channels' taps for NCG of the wave's 16-pixel
// column groups and 8 rows.  One operand read (4 channels x 16 pixels of
// staged row s at column shift v) feeds the MFMAs of every row y = s - u that
// it reaches; per output value the order is (4 channels, tap column v, tap
// row u), whatever the tile position, so bands equal the whole image bitwise.
template <int K, int OW, int NCG>
__device__ __forceinline__ void conv_compute(const float* __restrict__ base,
                                             const float (&wt)[ConvF32Geom<K, OW>::CK / 4][K * K], int channels,
                                             f32x4 (&acc)[ConvF32Geom<K, OW>::NCG][ConvF32Geom<K, OW>::TH]) {
  using G = ConvF32Geom<K, OW>;
#pragma unroll
  for (int c4 = 0; c4 < G::CK / 4; ++c4) {
    if (4 * c4 >= channels) break;  // uniform
    // step i = (tap column v, staged row s); step i + 1's operands are read
    // while step i's MFMAs run (the fences keep the compiler to that order)
    const float* cb = base + 4 * c4 * G::PS;
    float a[2][NCG];
#pragma unroll
    for (int g = 0; g < NCG; ++g) a[0][g] = cb[16 * g];
#pragma unroll
    for (int i = 0; i < K * G::LH; ++i) {
      const int v = i / G::LH, s = i % G::LH;
      if (i + 1 < K * G::LH) {
#pragma unroll
        for (int g = 0; g < NCG; ++g) a[(i + 1) % 2][g] = cb[(i + 1) % G::LH * G::LW + (i + 1) / G::LH + 16 * g];
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < K; ++u) {
        const int y = s - u;
        if (y < 0 || y >= G::TH) continue;
#pragma unroll
        for (int g = 0; g < NCG; ++g) acc[g][y] = mfma4(a[i % 2][g], wt[c4][u * K + v], acc[g][y]);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

template <int K, int OW, bool ADJ>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(K <= 3 ? 3 : 2))) void k_bank_f32_conv(BankF32Params p) {
  using G = ConvF32Geom<K, OW>;
  __shared__ f32x4 lds4[G::CK * G::PS / 4];
  float* lds = reinterpret_cast<float*>(lds4);
  const int lane = threadIdx.x % 64, l16 = lane % 16, q = lane / 16;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
  const int ow = wave % OW, xw = 16 * G::NCG * (wave / OW);
  const float* base = lds + q * G::PS + xw + l16 + G::HALO - G::R;
  const ConvF32Chunk<K, OW> ck;

  // a contiguous run of tiles per work-group, contiguous runs per XCD
  const int64_t b = xcd_remap(blockIdx.x, gridDim.x);
  const uint32_t t0 = static_cast<uint32_t>(p.n_tiles * b / gridDim.x);
  const uint32_t t1 = static_cast<uint32_t>(p.n_tiles * (b + 1) / gridDim.x);
  const bool one = p.CI <= G::CK && p.o_groups == 1;  // the weights never change
  float wt[G::CK / 4][K * K];
  f32x4 st[G::NT];
  if (t0 < t1) conv_load<K, OW>(p, ck, conv_tile<K, OW>(p, t0), 0, st);
  for (uint32_t ti = t0; ti < t1; ++ti) {
    const ConvF32Tile t = conv_tile<K, OW>(p, ti);
    const int o = (t.og * OW + ow) * 16 + l16;  // this lane's output channel
    f32x4 acc[G::NCG][G::TH];
#pragma unroll
    for (int g = 0; g < G::NCG; ++g)
#pragma unroll
      for (int y = 0; y < G::TH; ++y) acc[g][y] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int64_t left = p.xend - (t.ox0 + xw);  // columns of this wave that are produced

    for (int c0 = 0; c0 < p.CI; c0 += G::CK) {
      if (!one || ti == t0) {
        const float* wp = p.w + static_cast<int64_t>(o < p.CO ? o : p.CO - 1) * p.w_so;
#pragma unroll
        for (int c4 = 0; c4 < G::CK / 4; ++c4) {
          const int c = c0 + 4 * c4 + q;
          const float* wc = wp + static_cast<int64_t>(c < p.CI ? c : p.CI - 1) * p.w_sc;
#pragma unroll
          for (int e = 0; e < K * K; ++e) {
            const float x = wc[ADJ ? K * K - 1 - e : e];
            wt[c4][e] = c < p.CI ? x : 0.0f;
          }
        }
      }
      __syncthreads();  // the previous step's readers are done with the LDS
      conv_write<K, OW>(p, ck, t, c0, st, lds);
      __syncthreads();
      // the next step's loads are in flight while the matrix cores work
      const bool more = c0 + G::CK < p.CI;
      if (more || ti + 1 < t1)
        conv_load<K, OW>(p, ck, conv_tile<K, OW>(p, more ? ti : ti + 1), more ? c0 + G::CK : 0, st);
      __builtin_amdgcn_sched_barrier(0);
      if (left > 0) conv_compute<K, OW, G::NCG>(base, wt, p.CI - c0, acc);
      __builtin_amdgcn_sched_barrier(0);
    }

    // D rows are pixels 4q .. 4q+3 of a column group, columns the channels
    if (o >= p.CO || left <= 0) continue;
    float* dp = p.dst + t.n * p.d_sn + static_cast<int64_t>(o) * p.d_sc;
    const int64_t iy0 = (ADJ ? p.row0 : 0) + t.oy0;  // ADJ: image row; forward: band row
    const int64_t xl = t.ox0 + xw + 4 * q;
    const int64_t hlim = ADJ ? p.H : p.rows;
    const bool whole = t.oy0 + G::TH <= p.rows && iy0 >= 0 && iy0 + G::TH <= hlim && t.ox0 + xw >= 0 &&
                       t.ox0 + xw + 16 * G::NCG <= p.W;  // uniform: no border handling
    if (whole) {
      float* d = dp + iy0 * p.d_sh + xl;
#pragma unroll
      for (int y = 0; y < G::TH; ++y) {
#pragma unroll
        for (int g = 0; g < G::NCG; ++g) *reinterpret_cast<f32x4_u*>(d + 16 * g) = acc[g][y];
        d += p.d_sh;
      }
    } else {
      float* fp = ADJ ? p.frame + (t.n * p.CO + o) * p.frame_plane : nullptr;
#pragma unroll
      for (int y = 0; y < G::TH; ++y) {
        if (t.oy0 + y >= p.rows) break;
        const int64_t iy = iy0 + y;
        const bool row_in = iy >= 0 && iy < hlim;
#pragma unroll
        for (int g = 0; g < G::NCG; ++g)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int64_t ix = xl + 16 * g + e;
            if (row_in && ix >= 0 && ix < p.W)
              dp[iy * p.d_sh + ix] = acc[g][y][e];
            else if (ADJ && ix >= -p.fr && ix < p.xend)
              fp[frame_index(iy, ix, p.H, p.W, p.fr)] = acc[g][y][e];
          }
      }
    }
  }
}

// ------------------------------------------------------------- grad_filter --

// A lane quarter takes QC neighbouring columns of a 64-column strip, so the
// contraction index of MFMA step j is column QC*q + j.
template <int K>
struct WgradF32Geom {
  static constexpr int R = (K - 1) / 2;
  static constexpr int QC = 16;
  static constexpr int SW = 4 * QC;
  static constexpr int NX = QC + K - 1;  // X columns of a lane and row
  static constexpr int GP = SW + 4;      // LDS row pitches (floats, 16-byte aligned rows)
  static constexpr int XP = (SW + K - 1 + 7) / 4 * 4;
  // Error, not speed, sets these: with chains of 64 steps and one sum over a
  // unit the weights were further from the 64-bit ones than the VALU kernel's
  // (16 -> 64, 3x3, 2 x 44 x 40: 1.6e-7 against 1.1e-7, now 0.95e-7; 64 -> 64,
  // 1x1, 8 x 1000^2: 4.1e-7 against 3.1e-7, now 2.4e-7).  3x3 on 4 x 16 x
  // 1024^2 -> 64: 763 us then, 785 now (VALU 1950).
  static constexpr int FLUSH = K == 1 ? 4 : 8;  // MFMA steps (4 pixels each) of an accumulation chain
  static constexpr int SEG = K == 1 ? 32 : 64;  // rows of a wave before its sums go to memory
};

template <int K>
__device__ __forceinline__ void wgrad_row_x(const float* __restrict__ row, int64_t xb, int64_t W, bool inside,
                                            float (&x)[WgradF32Geom<K>::NX]) {
  using G = WgradF32Geom<K>;
  if (inside) {
    const float* a = row + xb - G::R;
#pragma unroll
    for (int i = 0; i < G::NX / 4; ++i) {
      const f32x4 t = *reinterpret_cast<const f32x4_u*>(a + 4 * i);
#pragma unroll
      for (int e = 0; e < 4; ++e) x[4 * i + e] = t[e];
    }
    if constexpr (G::NX % 4 != 0) {
      static_assert(G::NX % 4 == 2, "a two-column remainder");
      const f32x2_u t = *reinterpret_cast<const f32x2_u*>(a + G::NX - 2);
      x[G::NX - 2] = t[0];
      x[G::NX - 1] = t[1];
    }
  } else {
#pragma unroll
    for (int i = 0; i < G::NX; ++i) {
      int64_t c = xb - G::R + i;
      c = c < 0 ? 0 : (c >= W ? W - 1 : c);
      x[i] = row[c];
    }
  }
}

// A work-group (4 waves) takes obw x ibw blocks of 16 x 16 channels and 4 /
// (obw * ibw) row splits of its unit, one wave each, and walks down the rows.
// Per row every "slot" (16 planes x 64 columns of G, or of X with its halo)
// that the waves share is staged in LDS with row loads in column order, one
// row ahead in registers and double-buffered in LDS (one barrier a row).  A
// wave keeps the last K X rows of its windows in registers, so a row costs it
// one new X row and one G row from LDS for 16 K*K MFMAs.  Loading those
// operands straight from memory (a lane per plane: 16-byte pieces of 64 rows
// per instruction) held the 3 x 3 kernel at 5.2 ms on 16 x 16 x 1024^2 -> 64.
//
// One launch computes tap rows U0 .. U0+NU-1 (K = 5: 3 and 2 of them, since
// two accumulator sets of 25 taps leave one wave per SIMD).
template <int K, int U0, int NU>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2))) void k_bank_f32_wgrad(
    BankF32WgradParams p) {
  using G = WgradF32Geom<K>;
  constexpr int KK = K * K;
  constexpr int NT = NU * K;              // taps of this launch
  constexpr int LEAD = U0 + NU - 1 - G::R;  // the newest X row of G row y is y + LEAD
  extern __shared__ f32x4 shm[];
  float* lds = reinterpret_cast<float*>(shm);
  const int tid = threadIdx.x, lane = tid % 64, l16 = lane % 16, q = lane / 16;
  const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
  const int nbw = p.obw * p.ibw, splits = 4 / nbw;
  const int bw = wave % nbw, sp = wave / nbw;
  const int bo = bw / p.ibw, bi = bw % p.ibw;
  const int64_t b = xcd_remap(blockIdx.x, gridDim.x);
  const int64_t unit = b / p.block_groups;
  const int bg = static_cast<int>(b - unit * p.block_groups);
  const int ob0 = (bg / p.i_groups) * p.obw, ib0 = (bg % p.i_groups) * p.ibw;
  // unit = (image, row run, run of strips)
  const int64_t rest = unit / p.strip_runs, n = rest / p.runs;
  const int64_t ys = (rest - n * p.runs) * p.run_rows;
  const int64_t xs0 = (unit - rest * p.strip_runs) * p.run_strips * G::SW;
  const int64_t xs1 = xs0 + static_cast<int64_t>(p.run_strips) * G::SW < p.W
                          ? xs0 + static_cast<int64_t>(p.run_strips) * G::SW : p.W;
  const float* gn = p.g + n * p.g_sn;
  const float* xn = p.x + n * p.x_sn;
  const int64_t ye = ys + p.run_rows < p.H ? ys + p.run_rows : p.H;
  // of the current segment: first row, rows of a split, this wave's rows
  int64_t yseg, y0, y1;
  int rs;

  // staging: thread = (plane tid / 16 of a slot, 16-byte chunk tid % 16)
  const int gslots = p.obw * splits, xslots = p.ibw * splits;
  const int bufw = 16 * (gslots * G::GP + xslots * G::XP);  // floats per buffer
  const int pl = tid / 16, ch = tid % 16;
  auto inside = [&](int64_t c) { return c < 0 ? 0 : (c > p.W - 4 ? p.W - 4 : c); };
  // of the current strip (columns x0 .. x0+63): this thread's chunk of G and
  // of X (first column, and that of the nearest chunk inside the row, which
  // is loaded), its extra X column, and whether any chunk crosses the row's ends
  int64_t x0, gc, gl, xc, xl, el;
  bool gin, xin;
  constexpr int NE = K > 1 ? K - 1 : 1;
  const int epl = tid / NE, ee = tid % NE;  // X columns x0 - R + 64 .. : one value per thread
  auto set_strip = [&](int64_t x) {
    x0 = x;
    gin = x0 + G::SW <= p.W;
    xin = x0 >= G::R && x0 + G::SW + G::R <= p.W;
    gc = x0 + 4 * ch;
    xc = gc - G::R;
    gl = inside(gc);
    xl = inside(xc);
    el = x0 - G::R + G::SW + ee;
    el = el < p.W ? el : p.W - 1;
  };
  // (through an empty asm, or the compiler keeps every slot's address in
  // registers over the whole kernel and spills)
  auto fresh = [](int v) {
    asm volatile("" : "+v"(v));
    return v;
  };
  auto plane_g = [&](int i, int pp) {
    const int o = (ob0 + i % p.obw) * 16 + pp;
    return static_cast<int64_t>(o < p.CO ? o : p.CO - 1);
  };
  auto plane_x = [&](int i, int pp) {
    const int c = (ib0 + i % p.ibw) * 16 + pp;
    return static_cast<int64_t>(c < p.CI ? c : p.CI - 1);
  };
  auto row = [&](int64_t y) { return y < 0 ? 0 : (y >= p.H ? p.H - 1 : y); };
  f32x4 gv[4], xv[4];
  float xe[4];
  auto issue = [&](int it) {
    const int pln = fresh(pl), epn = fresh(epl);
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (i < gslots) {
        const int64_t y = row(yseg + (i / p.obw) * rs + it);
        gv[i] = *reinterpret_cast<const f32x4_u*>(gn + plane_g(i, pln) * p.g_sc + y * p.g_sh + gl);
      }
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (i < xslots) {
        const float* r = xn + row(yseg + (i / p.ibw) * rs + it + LEAD) * p.x_sh;
        xv[i] = *reinterpret_cast<const f32x4_u*>(r + plane_x(i, pln) * p.x_sc + xl);
        if (K > 1 && tid < 16 * NE) xe[i] = r[plane_x(i, epn) * p.x_sc + el];
      }
  };
  auto store = [&](float* buf) {
    const int pls = fresh(pl), chs = fresh(ch);
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (i < gslots) {
        f32x4 v = gv[i];
        if (!gin) {  // columns at or beyond W are zero; the loaded chunk may lie left of this one
          f32x4 w;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int f = static_cast<int>(gc + e - gl);
            w[e] = gc + e < p.W ? (f == 0 ? v[0] : (f == 1 ? v[1] : (f == 2 ? v[2] : v[3]))) : 0.0f;
          }
          v = w;
        }
        *reinterpret_cast<f32x4*>(buf + (i * 16 + pls) * G::GP + 4 * chs) = v;
      }
    float* xb = buf + gslots * 16 * G::GP;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (i < xslots) {
        f32x4 v = xv[i];
        if (!xin) {  // clamped columns
          f32x4 w;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            int64_t c = xc + e;
            c = c < 0 ? 0 : (c >= p.W ? p.W - 1 : c);
            const int f = static_cast<int>(c - xl);
            w[e] = f == 0 ? v[0] : (f == 1 ? v[1] : (f == 2 ? v[2] : v[3]));
          }
          v = w;
        }
        *reinterpret_cast<f32x4*>(xb + (i * 16 + pls) * G::XP + 4 * chs) = v;
        if (K > 1 && tid < 16 * NE) xb[(i * 16 + epl) * G::XP + G::SW + ee] = xe[i];
      }
  };

  float xr[NU][G::NX], g[G::QC];
  const float* gr = lds + ((sp * p.obw + bo) * 16 + l16) * G::GP + G::QC * q;
  const float* xw = lds + gslots * 16 * G::GP + ((sp * p.ibw + bi) * 16 + l16) * G::XP + G::QC * q;
  const int c = (ib0 + bi) * 16 + l16;
  bool first = true;
  for (int64_t xs = xs0; xs < xs1; xs += G::SW) {
    set_strip(xs);
    for (yseg = ys; yseg < ye; yseg += splits * G::SEG) {
      const int64_t yend = yseg + splits * G::SEG < ye ? yseg + splits * G::SEG : ye;
      rs = static_cast<int>((yend - yseg + splits - 1) / splits);
      y0 = yseg + sp * rs;
      y1 = y0 + rs < yend ? y0 + rs : yend;
      f32x4 sum[NT];
#pragma unroll
      for (int e = 0; e < NT; ++e) sum[e] = f32x4{0.f, 0.f, 0.f, 0.f};
      {
        // the NU - 1 X rows above the first one, straight from memory
        const float* xp = xn + static_cast<int64_t>(c < p.CI ? c : p.CI - 1) * p.x_sc;
#pragma unroll
        for (int u = 0; u + 1 < NU; ++u)
          wgrad_row_x<K>(xp + row(y0 - G::R + U0 + u) * p.x_sh, x0 + G::QC * q, p.W, xin, xr[u]);
      }
      issue(0);
      store(lds);
      __syncthreads();
      for (int it = 0; it < rs; ++it) {
        if (it + 1 < rs) issue(it + 1);
        const int off = (it & 1) * bufw;
#pragma unroll
        for (int i = 0; i < G::QC / 4; ++i) {
          const f32x4 t = *reinterpret_cast<const f32x4*>(gr + off + 4 * i);
#pragma unroll
          for (int e = 0; e < 4; ++e) g[4 * i + e] = t[e];
        }
#pragma unroll
        for (int i = 0; i < (G::NX + 3) / 4; ++i) {
          const f32x4 t = *reinterpret_cast<const f32x4*>(xw + off + 4 * i);
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (4 * i + e < G::NX) xr[NU - 1][4 * i + e] = t[e];
        }
        __builtin_amdgcn_sched_barrier(0);
        // short chains (the first MFMA of each starts from zero): see FLUSH
        if (y0 + it < y1) {
#pragma unroll
          for (int h = 0; h < G::QC; h += G::FLUSH) {
            f32x4 acc[NT];
#pragma unroll
            for (int j = h; j < h + G::FLUSH; ++j)
#pragma unroll
              for (int u = 0; u < NU; ++u)
#pragma unroll
                for (int v = 0; v < K; ++v)
                  acc[u * K + v] = mfma4(g[j], xr[u][j + v], j == h ? f32x4{0.f, 0.f, 0.f, 0.f} : acc[u * K + v]);
#pragma unroll
            for (int e = 0; e < NT; ++e) sum[e] += acc[e];
          }
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u + 1 < NU; ++u)
#pragma unroll
          for (int i = 0; i < G::NX; ++i) xr[u][i] = xr[u + 1][i];
        if (it + 1 < rs) store(lds + ((it + 1) & 1) * bufw);
        __syncthreads();
      }
      // the row splits are added in order
      for (int s = 1; s < splits; ++s) {
        if (sp == s) {
#pragma unroll
          for (int e = 0; e < NT; ++e) shm[(bw * NT + e) * 64 + lane] = sum[e];
        }
        __syncthreads();
        if (sp == 0) {
#pragma unroll
          for (int e = 0; e < NT; ++e) sum[e] += shm[(bw * NT + e) * 64 + lane];
        }
        __syncthreads();
      }
      // the unit's sums so far are in its partial (this lane's own entries)
      if (sp == 0 && c < p.CI) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int oo = (ob0 + bo) * 16 + 4 * q + j;
          if (oo >= p.CO) break;
          const int64_t f = static_cast<int64_t>(oo) * p.CI + c;
          float* dst = p.partial + (unit * p.CO * p.CI + f) * KK + U0 * K;
          if (!first) {
#pragma unroll
            for (int e = 0; e < NT; ++e) sum[e][j] += dst[e];
          }
#pragma unroll
          for (int e = 0; e < NT; ++e) dst[e] = sum[e][j];
        }
      }
      first = false;
    }
  }
}

// ---------------------------------------------------------------- dispatch --

// Resident work-groups of a kernel, looked up once per device.
struct Resident {
  std::mutex mu;
  int groups[64] = {};
};

hipError_t resident(const void* kern, Resident& r, int* out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  std::lock_guard<std::mutex> lk(r.mu);
  int cached = dev >= 0 && dev < 64 ? r.groups[dev] : 0;
  if (cached == 0) {
    int per_cu = 0, cus = 0;
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, kThreads, 0);
    if (e != hipSuccess) return e;
    e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return e;
    cached = (per_cu > 0 ? per_cu : 1) * (cus > 0 ? cus : 1);
    if (dev >= 0 && dev < 64) r.groups[dev] = cached;
  }
  *out = cached;
  return hipSuccess;
}

template <int K, int OW, bool ADJ>
hipError_t conv_go(BankF32Params p, hipStream_t s) {
  using G = ConvF32Geom<K, OW>;
  p.tiles_x = static_cast<int32_t>((p.xend - p.col0 + G::TW - 1) / G::TW);
  p.tiles_y = static_cast<int32_t>((p.rows + G::TH - 1) / G::TH);
  p.o_groups = (p.CO + 16 * OW - 1) / (16 * OW);
  p.n_tiles = p.n_img * p.o_groups * static_cast<int64_t>(p.tiles_x) * p.tiles_y;
  if (p.n_tiles <= 0) return hipSuccess;
  if (p.n_tiles > INT32_MAX) return hipErrorInvalidValue;
  static Resident res;
  int grid = 0;
  hipError_t e = resident(reinterpret_cast<const void*>(k_bank_f32_conv<K, OW, ADJ>), res, &grid);
  if (e != hipSuccess) return e;
  if (p.n_tiles < grid) grid = static_cast<int>(p.n_tiles);
  hipLaunchKernelGGL((k_bank_f32_conv<K, OW, ADJ>), dim3(grid), dim3(kThreads), 0, s, p);
  return hipGetLastError();
}

template <int K, bool ADJ>
hipError_t conv_by_out(const BankF32Params& p, hipStream_t s) {
  if (p.CO <= 16) return conv_go<K, 1, ADJ>(p, s);
  if (p.CO <= 32) return conv_go<K, 2, ADJ>(p, s);
  return conv_go<K, 4, ADJ>(p, s);
}

template <int K>
hipError_t conv_by_dir(const BankF32Params& p, bool adj, hipStream_t s) {
  return adj ? conv_by_out<K, true>(p, s) : conv_by_out<K, false>(p, s);
}

// Blocks of 16 x 16 channels per work-group (obw x ibw, at most 4; the other
// waves split rows) and the work-groups that cover every block of a unit.
struct WgradBlocks {
  int obw, ibw, i_groups;
  int64_t groups;
};
WgradBlocks wgrad_blocks(int64_t co, int64_t ci) {
  const int64_t ob = (co + 15) / 16, ib = (ci + 15) / 16;
  WgradBlocks w;
  w.ibw = ib == 1 ? 1 : (ob == 1 && ib > 2 ? 4 : 2);
  w.obw = ob == 1 ? 1 : (ib > 1 || ob == 2 ? 2 : 4);
  const int64_t ig = (ib + w.ibw - 1) / w.ibw, og = (ob + w.obw - 1) / w.obw;
  w.i_groups = static_cast<int>(ig);
  w.groups = ig * og;
  return w;
}

template <int K, int U0, int NU>
hipError_t wgrad_go(BankF32WgradParams p, hipStream_t s) {
  using G = WgradF32Geom<K>;
  const WgradBlocks w = wgrad_blocks(p.CO, p.CI);
  p.obw = w.obw;
  p.ibw = w.ibw;
  p.i_groups = w.i_groups;
  p.block_groups = static_cast<int32_t>(w.groups);
  const int64_t grid = p.n_img * p.runs * p.strip_runs * w.groups;
  if (grid <= 0) return hipSuccess;
  if (grid > kMaxBlocks) return hipErrorInvalidValue;
  const int splits = 4 / (w.obw * w.ibw);
  const size_t stage = 2 * 16 * (static_cast<size_t>(w.obw) * splits * G::GP + static_cast<size_t>(w.ibw) * splits * G::XP) * 4;
  const size_t red = splits > 1 ? static_cast<size_t>(w.obw) * w.ibw * NU * K * 64 * sizeof(f32x4) : 0;
  const size_t lds = stage > red ? stage : red;
  if (lds > 64 * 1024) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_bank_f32_wgrad<K, U0, NU>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((k_bank_f32_wgrad<K, U0, NU>), dim3(static_cast<uint32_t>(grid)), dim3(kThreads), lds, s, p);
  return hipGetLastError();
}

}  // namespace

// The matrix-core map pads the source channels to fours and the outputs to
// sixteens; the VALU kernels pad nothing at half the rate, but read the
// source again for every one to four outputs.  Measured at 8 x 512^2 (VALU /
// matrix time, forward): 1x1 3 -> 16 1.2, 16 -> 3 2.1, 4 -> 4 0.85; 3x3 3 ->
// 16 1.2, 8 -> 8 1.04, 16 -> 3 1.05, 4 -> 4 0.64, 1 -> 64 0.8, 64 -> 1 0.6,
// 16 -> 64 2.0; 5x5 8 -> 8 1.02, 16 -> 3 0.6, 1 -> 64 0.7, 16 -> 64 2.0.
//
// The VALU kernels take four outputs (of a multiple of four, and not with zero
// borders) from one staged tile, so on many tiles they win back some of these
// (VALU / matrix us):
// - 3x3 with less than half of the padded products real: 64 -> 4 8 x 512^2 220 /
//   345, 6 -> 8 45 / 54, 5 -> 12 4 x 1024^2 100 / 104, 64 -> 8 717 / 695; from two
//   channels 2 -> 32 144 / 159;
// - 1x1 on narrow images, whose tiles are mostly border: 64 x 512 x 24, 64 -> 4 74
//   / 119, 4 -> 64 90 / 113; 3 -> 32 at any width (8 x 512^2 65 / 69);
// - grad_input into many channels from few, bound by stores that start 4 columns
//   left of the lines: 8 x 512^2 3 -> 64 293 / 386, 4 -> 64 348 / 391, and of narrow
//   images: 64 x 512 x 48 16 -> 3 129 / 162, 8 -> 8 97 / 108.
// On few tiles the VALU leaves the GPU idle (64 -> 4, 4 x 224^2 150 / 54).  A
// forward takes one kernel for every height and batch all the same: row bands
// have the bits of the whole image.  A grad_input is of whole images.
bool bank_f32_conv_mfma(int mode, int K, int64_t src, int64_t out, int64_t w, bool zero) {
  if (mode != F2D_CH_BANK || w < 4 || src > 65536 || out > 65536) return false;
  const int64_t pairs = src * out, padded = (src + 3) / 4 * 4 * ((out + 15) / 16 * 16);
  const bool fours = out % 4 == 0 && !zero;
  if (K == 1)
    return src >= 3 && pairs >= 32 &&
           !(fours && ((w < 128 && pairs <= 256) || (src <= 4 && out > 16 && out <= 32)));
  if (K == 3)
    return src >= 2 && pairs >= 48 && 16 * pairs >= 3 * padded && !(fours && (src < 3 || 2 * pairs < padded));
  if (K == 5) return src >= 2 && pairs >= 48 && 2 * pairs >= padded;
  return false;
}

bool bank_f32_adjoint_mfma(int mode, int K, int64_t src, int64_t out, int64_t n, int64_t h, int64_t w) {
  if (mode != F2D_CH_BANK || w < 4 || src > 65536 || out > 65536) return false;
  const int64_t pairs = src * out, padded = (src + 3) / 4 * 4 * ((out + 15) / 16 * 16);
  const bool fours = out % 4 == 0;
  const double groups = static_cast<double>(n) * ((h + 63) / 64) * ((w + 63) / 64) * (fours ? out / 4 : out);
  const bool full = groups >= 256;  // the VALU's work-groups fill the GPU
  if (K == 1)
    return src >= 3 && pairs >= 32 &&
           !(fours && src <= 4 && w < 128) &&
           !(full && ((w < 128 && pairs <= 256) || (fours && src <= 4 && out > 16 && out <= 32)));
  if (K == 3)
    return src >= 2 && pairs >= 48 && 16 * pairs >= 3 * padded &&
           !(full && ((fours && 2 * pairs < padded) || (fours && src <= 4 && out >= 32) || (w < 128 && pairs <= 96)));
  if (K == 5) return src >= 2 && pairs >= 48 && 2 * pairs >= padded;
  return false;
}

// grad_filter pads both channel counts to sixteens.  Measured as above: 1x1
// 3 x 16 1.6, 8 x 8 1.1, 1 x 64 0.8; 3x3 8 x 16 1.24, 8 x 8 0.83, 16 x 64
// 2.8; 5x5 8 x 16 0.8, 16 x 16 1.2, 16 x 64 1.9.
// Small layers stay on the VALU, whose fewer partial sets are added sooner
// (VALU / matrix us):
// - 1x1 by multiply-adds: 0.4M 15.8 / 20.3, 0.9M 16.0 / 18.9, 13M 32.6 / 33.5,
//   18M 27.0 / 25.2, 28M 36.0 / 25.5.
// - 3x3 and 5x5 by the VALU kernel's work, 64 x 64 tiles times channel pairs
//   times images: it takes about as long up to 4096 of them as for 500, at any
//   number of pixels in them.  5x5: 1024 35 / 54 (16 -> 16, 112^2), 2304 41 / 75
//   (160^2), 4096 68 / 76 (16 -> 16) but 65 / 62 (16 -> 64, 112^2) and 65 / 43 (64
//   -> 64, 14^2), 6144 73 / 82 (48 -> 16) and 77 / 74 (12 -> 16), 8192 103 / 73.
//   3x3 likewise (2048 31 / 38, 16 -> 16; 4096 33 / 39, 16 -> 32; 6144 36 / 39, 48
//   -> 16, and 40 / 38, 12 -> 16; 8192 60 / 36), except where the rows and strips
//   of all images are few, and with them the partial sets: 14 rows 29 / 19, 224
//   rows 31 / 29 (16 -> 16; 400 rows 32 / 38).
bool bank_f32_wgrad_mfma(int mode, int K, int64_t co, int64_t ci, int64_t n, int64_t h, int64_t w) {
  if (mode != F2D_CH_BANK || w < 4 || ci > 65536 || co > 65536) return false;
  const int64_t pairs = ci * co, padded = (ci + 15) / 16 * 16 * ((co + 15) / 16 * 16);
  const double pixels = static_cast<double>(n) * h * w, rows = static_cast<double>(n) * h * ((w + 63) / 64);
  const double tiles = static_cast<double>(n) * ((h + 63) / 64) * ((w + 63) / 64) * pairs;
  if (K == 1) return 16 * pairs >= 3 * padded && pairs * pixels >= 16e6;
  if (K == 3) return 2 * pairs >= padded && (tiles >= 8192 || rows <= 256);
  if (K == 5) return 4 * pairs >= 3 * padded && (tiles >= 8192 || (tiles >= 4096 && pairs >= 1024));
  return false;
}

// Units of grad_filter: about 512 work-groups (two per CU), as whole-height
// runs of strips where the images have more strips than that, else as row
// runs of one strip; no more partial sets than max_sets (>= n).
void bank_f32_wgrad_plan(int64_t n, int64_t h, int64_t w, int64_t co, int64_t ci, int64_t max_sets,
                         BankF32WgradPlan* plan) {
  const int64_t groups = wgrad_blocks(co, ci).groups;
  const int64_t tx = (w + 63) / 64;
  int64_t want = (512 + groups - 1) / groups;  // sets
  if (want > max_sets) want = max_sets;
  int64_t spr = 1, runs = 1;
  if (n * tx > want && n > 0) {
    const int64_t per_image = want / n > 0 ? want / n : 1;
    spr = (tx + per_image - 1) / per_image;
  } else if (n * tx > 0) {
    runs = want / (n * tx);
    if (runs > h) runs = h;
    if (runs < 1) runs = 1;
  }
  const int64_t rows = h > 0 ? (h + runs - 1) / runs : 1;
  plan->run_strips = static_cast<int32_t>(spr);
  plan->strip_runs = static_cast<int32_t>((tx + spr - 1) / spr);
  plan->run_rows = static_cast<int32_t>(rows);
  plan->runs = static_cast<int32_t>(h > 0 ? (h + rows - 1) / rows : 1);
  plan->sets = n * plan->strip_runs * plan->runs;
}

hipError_t launch_bank_f32_conv(const BankF32Params& p, int K, bool adjoint, hipStream_t s) {
  switch (K) {
    case 1: return conv_by_dir<1>(p, adjoint, s);
    case 3: return conv_by_dir<3>(p, adjoint, s);
    case 5: return conv_by_dir<5>(p, adjoint, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_bank_f32_wgrad(const BankF32WgradParams& p, int K, hipStream_t s) {
  switch (K) {
    case 1: return wgrad_go<1, 0, 1>(p, s);
    case 3: return wgrad_go<3, 0, 3>(p, s);
    case 5: {
      const hipError_t e = wgrad_go<5, 0, 3>(p, s);
      return e != hipSuccess ? e : wgrad_go<5, 3, 2>(p, s);
    }
    default: return hipErrorInvalidValue;
  }
}

}  // namespace f2d
