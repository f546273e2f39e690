// Host-side packing of the weights into the tiled layout (tile_off).
#pragma once

#include <stddef.h>

#include <memory>

namespace fv {

// Rows of K values in the tiled order of a type with `piece` elements in 16
// bytes, as fp32.  Sixteen rows, one group of tiles, are gathered at a time
// from sixteen adjacent columns of the source, so that a source line is read
// once and the layout costs no pass of its own.  (4 M values of k 1024 in
// bf16: 45 ms when a row was gathered at a time and then repacked, 20 so.)
class TiledRows {
 public:
  // rows: a multiple of 16; K: of a tile's 4 pieces
  TiledRows(size_t rows, int K, int piece)
      : v_(new float[rows * K]), size_(rows * K), end_(v_.get()), K_(K), piece_(piece) {}
  // The next 16 rows: columns [col, col + 16) of W [n][out]; zero past its
  // columns (out) and past n.
  void append16(const float* W, int out, int col, int n) {
    const int cols = out - col < 16 ? out - col : 16;
    for (int k0 = 0; k0 < K_; k0 += piece_, end_ += 16 * piece_)
      for (int e = 0; e < piece_; ++e) {
        const float* src = W + (size_t)(k0 + e) * out + col;
        float* d = end_ + e;
        if (k0 + e < n && cols == 16)
          for (int r = 0; r < 16; ++r) d[r * piece_] = src[r];
        else
          for (int r = 0; r < 16; ++r) d[r * piece_] = k0 + e < n && r < cols ? src[r] : 0.f;
      }
  }
  // The next `count` rows (a multiple of 16) from column col on.
  void append(const float* W, int out, int col, int count) {
    for (int c = 0; c < count; c += 16) append16(W, out, col + c, K_);
  }
  const float* data() const { return v_.get(); }
  size_t size() const { return size_; }

 private:
  std::unique_ptr<float[]> v_;
  size_t size_;
  float* end_;
  int K_, piece_;
};

}  // namespace fv
