// Index arithmetic of the convolution kernels.  Plain constexpr functions: the kernels and the host share them, and they can be
// checked without a GPU.
#ifndef ZENO_INDEX_H_
#define ZENO_INDEX_H_

namespace zeno {

constexpr long long kConvMostBlocks = 1ll << 30;   // workgroups of a launch

// Multiplier ceil(2^32 / d) of the quick divisions by d >= 1 (0: d = 1).
constexpr unsigned magic_for(long long d) {
  return d <= 1 ? 0u : (unsigned)(((1ull << 32) + (unsigned long long)d - 1) / (unsigned long long)d);
}
constexpr unsigned mul_high(unsigned a, unsigned b) { return (unsigned)(((unsigned long long)a * b) >> 32); }
// v / d for 0 <= v, v d < 2^32
constexpr unsigned div_magic(unsigned v, unsigned magic) { return magic == 0u ? v : mul_high(v, magic); }
// v / d for any v < 2^31: magic d exceeds 2^32 by less than d, so the product's high half is at most one too large.
constexpr unsigned div_any(unsigned v, unsigned d, unsigned magic) {
  const unsigned q = div_magic(v, magic);
  return q * d > v ? q - 1u : q;
}

// Floats between column 0 and column k of a row in float32 matrix-operand order (32 rows x 8 columns, half by half of the columns).
constexpr long long operand_column(int k) { return (long long)(k >> 3) * 256 + ((k >> 2) & 1) * 128 + (k & 3); }

}  // namespace zeno
#endif
