// Index arithmetic of the convolution kernels against plain division, on the host.  Built and run by
// tests/test_host_sanitizers.py.
#include <cstdio>

#include "zeno_index.h"
#include "zeno.h"

#define CHECK(cond)                                                        \
  do {                                                                     \
    if (!(cond)) {                                                         \
      std::fprintf(stderr, "check failed at line %d: %s\n", __LINE__, #cond); \
      return 1;                                                            \
    }                                                                      \
  } while (0)

using namespace zeno;

// Both sides of a multiple of d: where a quotient goes wrong first.
static bool around(unsigned tile, unsigned d, unsigned magic) {
  for (unsigned v = tile * d - 1u; v != tile * d + 2u; ++v)
    if (v < (unsigned)kConvMostBlocks && div_any(v, d, magic) != v / d) return false;
  return true;
}

int main() {
  // blocks by candidates: every number of candidates, up to the largest grid that is launched
  for (unsigned d = 1; d <= ZENO_MAX_CANDIDATES; ++d) {
    const unsigned magic = magic_for(d), tiles = (unsigned)(kConvMostBlocks / d);
    for (unsigned t = 1; t <= tiles && t <= 5000; ++t) CHECK(around(t, d, magic));
    for (unsigned t = tiles > 3000 ? tiles - 3000 : 1; t <= tiles; ++t) CHECK(around(t, d, magic));
    for (unsigned t = 1; t < tiles; t += tiles / 3000 + 1) CHECK(around(t, d, magic));
  }
  // tiles by channel tiles: any number of channels
  for (unsigned d = 1; d < (unsigned)kConvMostBlocks / 3; d += d / 97 + 1) {
    const unsigned magic = magic_for(d), tiles = (unsigned)(kConvMostBlocks / d);
    for (unsigned t = 1; t <= tiles; t += tiles / 300 + 1) CHECK(around(t, d, magic));
    CHECK(around(tiles, d, magic));
  }
  // the multiplier alone: exact where the product of both is below 2^32, one too large beyond (1023 candidates, tile 4120)
  for (unsigned d = 1; d < 70000; d += d / 50 + 1) {
    const unsigned most = (unsigned)(((1ull << 32) - 1) / d), magic = magic_for(d);
    for (unsigned v = most < 3000 ? 0 : most - 3000; v < most; ++v) CHECK(div_magic(v, magic) == v / d);
  }
  CHECK(div_magic(4120u * 1023u + 1022u, magic_for(1023)) == 4121u && div_any(4120u * 1023u + 1022u, 1023u, magic_for(1023)) == 4120u);
  // columns of a wide operand row: the offsets pass 2^31 floats from column 2^26 on
  const int columns[] = {0, 3, 4, 7, 8, 175, (1 << 26) - 1, 1 << 26, (1 << 26) + 5, 0x7fffffff};
  for (int k : columns) {
    const long long group = k / 8, half = k % 8 / 4;
    CHECK(operand_column(k) == group * 8 * 32 + half * 4 * 32 + k % 4);
  }
  std::puts("index checks passed");
  return 0;
}
