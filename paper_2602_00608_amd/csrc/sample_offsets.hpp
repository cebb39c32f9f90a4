// Element offsets of an epilogue's vectors inside one sample of h x w pixels of `cout` channels.
//
// The matrix-core kernels address a sample through a buffer with 32-bit byte offsets: a scalar one for the vector's position in
// the tile and a per-lane one, which is kOutside for a lane whose pixel is not in the image, so that its access is dropped.
// Samples have fewer than kOutside elements (checked on the host), at up to four bytes each; then base + kOutside stays below
// 2^32 bytes whether or not the hardware counts the scalar part in its range check.
#pragma once

namespace wmdec {

constexpr unsigned kOutside = 1u << 29;

// Channel co of pixel (row, col), the pixel that the lanes of a vector count from.  A tile overhangs the image by up to its own
// size less one; there every lane is outside and the pixel is taken from the last row or column instead: unclamped, an
// overhanging row of a short wide image is up to seven times the image further, past 2^31.
constexpr int vector_base(int row, int col, int h, int w, int cout, int co) {
  return ((row < h ? row : h - 1) * w + (col < w ? col : w - 1)) * cout + co;
}

}  // namespace wmdec
