// Parameter blocks and launchers of the FP32 filter-bank kernels (matrix cores).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace f2d {

// One map from CI source to CO output channels: the forward, or its adjoint
// in the image (zero = 1, taps flipped, the image plus an r-wide frame).
struct BankF32Params {
  const float* src;
  int64_t s_sn, s_sc, s_sh;
  float* dst;
  int64_t d_sn, d_sc, d_sh;
  const float* w;           // weight (output o, source c, tap e) at o * w_so + c * w_sc + e
  int64_t w_so, w_sc;
  int64_t H, W, row0, rows; // output rows [row0, row0 + rows) of the source frame
  int64_t col0, xend;       // output columns [col0, xend) (col0 4-aligned, <= -r for the adjoint)
  int64_t n_img;
  int32_t CI, CO;
  int32_t zero;             // out-of-range source pixels read as 0 (else clamp)
  // adjoint: values on the r-wide frame (frame_index(), frame_plane floats per output plane)
  int32_t fr;
  float* frame;
  int64_t frame_plane;
  // set by the launcher
  int32_t tiles_x, tiles_y, o_groups;
  int64_t n_tiles;
};

// grad_filter partial sums, one set [CO][CI][K*K] per unit = (image, run of
// run_rows rows, run of run_strips 64-column strips), units in that order.
struct BankF32WgradPlan {
  int32_t runs, run_rows, strip_runs, run_strips;
  int64_t sets;  // images * runs * strip_runs
};
struct BankF32WgradParams {
  const float* x;
  int64_t x_sn, x_sc, x_sh;
  const float* g;
  int64_t g_sn, g_sc, g_sh;
  float* partial;
  int64_t H, W, n_img;
  int32_t CI, CO;
  int32_t runs, run_rows, strip_runs, run_strips;
  // set by the launcher: 16 x 16 channel blocks per work-group (obw x ibw) and work-groups per unit
  int32_t obw, ibw, i_groups, block_groups;
};

// Whether a forward or its adjoint in the image, from src to out channels, or a
// grad_filter, of this shape takes these kernels (else the VALU ones).
bool bank_f32_conv_mfma(int mode, int K, int64_t src, int64_t out, int64_t w, bool zero);
bool bank_f32_adjoint_mfma(int mode, int K, int64_t src, int64_t out, int64_t n, int64_t h, int64_t w);
bool bank_f32_wgrad_mfma(int mode, int K, int64_t co, int64_t ci, int64_t n, int64_t h, int64_t w);
void bank_f32_wgrad_plan(int64_t n, int64_t h, int64_t w, int64_t co, int64_t ci, int64_t max_sets,
                         BankF32WgradPlan* plan);
hipError_t launch_bank_f32_conv(const BankF32Params& p, int K, bool adjoint, hipStream_t s);
hipError_t launch_bank_f32_wgrad(const BankF32WgradParams& p, int K, hipStream_t s);

}  // namespace f2d
