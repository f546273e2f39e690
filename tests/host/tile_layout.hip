// Offsets of the tiled operand layout, on the host: tile_off is a bijection of
// whole tiles, the kernels' shortcut for a block of k (tile_k) agrees with it,
// also where the offset passes 32 bits, and the packer (TiledRows) writes every
// value of a weight, and a zero everywhere else, where it says.
#include <cstdio>
#include <vector>

#include "fv_internal.h"
#include "fv_pack.h"

using namespace fv;

template <typename T>
int check(const char* name) {
  constexpr int KB = 64 / (int)sizeof(T);  // k of one tile
  for (int K : {KB, 2 * KB, 3 * KB, 16 * KB, 33 * KB}) {
    const int rows = 48;
    std::vector<char> seen((size_t)rows * K, 0);
    for (int r = 0; r < rows; ++r)
      for (int k = 0; k < K; ++k) {
        const size_t o = tile_off<T>(r, k, K);
        if (o >= seen.size() || seen[o]) return printf("%s: K %d row %d k %d -> %zu\n", name, K, r, k, o), 1;
        seen[o] = 1;
        const int kb = k / KB * KB;
        if (o != tile_off<T>(r, k - kb, K) + tile_k(kb)) return printf("%s: tile_k at K %d k %d\n", name, K, k), 1;
      }
  }
  for (int K : {1 << 22, (1 << 27) + 64, 0x7fffffc0})
    for (int r : {0, 5, 15})
      for (int kb : {0, K / 2 / KB * KB, K - KB}) {
        const int k = kb + r % KB;
        if (tile_off<T>(r, k, K) != tile_off<T>(r, k - kb, K) + tile_k(kb))
          return printf("%s: tile_k at K %d row %d k %d\n", name, K, r, k), 1;
      }
  // weights [n][out], with k past n and columns past out zero
  struct Shape { int n, out, K; };
  for (Shape s : {Shape{2 * KB, 48, 2 * KB}, Shape{5, 32, KB}, Shape{3 * KB, 7, 3 * KB}, Shape{1, 1, KB}}) {
    std::vector<float> W((size_t)s.n * s.out);
    for (size_t i = 0; i < W.size(); ++i) W[i] = (float)(i + 1);
    const int rows = (s.out + 15) / 16 * 16;
    TiledRows t(rows, s.K, 16 / (int)sizeof(T));
    for (int c = 0; c < rows; c += 16) t.append16(W.data(), s.out, c, s.n);
    if (t.size() != (size_t)rows * s.K) return printf("%s: size\n", name), 1;
    for (int r = 0; r < rows; ++r)
      for (int k = 0; k < s.K; ++k) {
        const float want = k < s.n && r < s.out ? W[(size_t)k * s.out + r] : 0.f;
        if (t.data()[tile_off<T>(r, k, s.K)] != want)
          return printf("%s: packed %dx%d at row %d k %d\n", name, s.n, s.out, r, k), 1;
      }
  }
  return 0;
}

int main() { return check<bf16_t>("bf16") | check<float>("fp32"); }
