// Where a staged tile lies against its image (host and device; no HIP types,
// so that a host program can check it).
#pragma once

#include <cstdint>

namespace f2d {

// A tile's staged rows and columns start at image row row0 and column col0
// (both may be negative) of an image whose extents are below 2^31.  Corners
// and image positions fit in 32 bits; row0 + y and col0 + x pass 2^31 on
// images that end just below it, so they saturate (one instruction, and no
// register more than the plain sum: 64-bit bounds took 8 to 42 more).
struct ChunkWindow {
  int32_t row0, col0, H, W;
  bool inside;  // every staged column is an image column

  // Image row of staged row y, clamped.
  constexpr int32_t row(int32_t y) const {
    const int32_t r = __builtin_elementwise_add_sat(row0, y);
    return r < 0 ? 0 : (r >= H ? H - 1 : r);
  }
  // First of the four image columns nearest to staged columns x .. x + 3
  // (W >= 4), and where those start in them: staged column x + q is column
  // four(x) + clamp(shift + q, 0, 3).
  constexpr int32_t four(int32_t x, int32_t* shift) const {
    const int32_t c = __builtin_elementwise_add_sat(col0, x);  // saturated: beyond W, so shift >= 4
    const int32_t f = c < 0 ? 0 : (c > W - 4 ? W - 4 : c);
    *shift = c - f;
    return f;
  }
};

// row0 < H and col0 < W: the tile's first output lies in the image.
template <int PITCH>
constexpr ChunkWindow chunk_window(int32_t row0, int32_t col0, int32_t H, int32_t W) {
  return {row0, col0, H, W, col0 >= 0 && W - col0 >= PITCH};
}

}  // namespace f2d
