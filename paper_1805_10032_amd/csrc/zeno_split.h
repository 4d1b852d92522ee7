// Three-way split of float32 operands for the bf16 matrix cores, shared by the kernels that multiply at float32 accuracy.
#ifndef ZENO_SPLIT_H_
#define ZENO_SPLIT_H_

#include "zeno_internal.h"

namespace zeno {

namespace {

// Three-way split of eight floats into bf16 pieces, x = h + m + l + (at most 2^-25 |x|):
// h = bf16(x), m = bf16(x - h), l = bf16(x - h - m), round to nearest even each time;
// both subtractions are exact.
// The leading piece of a finite |x| from 0x1.ffp127 (3.396e38) on would be rounded to infinity: FINITE gives it the largest bf16
// value instead, and the other two pieces take up the rest (four maxima of three and a branch that is never taken on ordinary
// data: the steps of two convolutional models 157.2 -> 158.9 and 449 -> 454 us; one test for all values of a thread, with the
// staging code twice or with the result in a flag, took 160.3 and 458).  Below about 1e-33 the last pieces underflow, and
// products keep fewer than 24 bits.
template <bool FINITE = false>
__device__ inline void split3(const f32x4& v0, const f32x4& v1, bf16x8& h, bf16x8& m, bf16x8& l) {
  // Two floats at a time: one packed conversion gives both bf16 pieces in one register, and the exact remainder of
  // either float is one instruction, the bf16 dot product of that register with (-1, 0) or (0, -1) added to the
  // float (v_dot2c_f32_bf16: the product with -1 is exact, the product with 0 vanishes, and the sum x - h is
  // representable, so its single rounding changes nothing).  Seven instructions per two floats; taking the pieces'
  // float values out of the packed register with a shift or a mask and subtracting took eleven.
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
  const float x[8] = {v0[0], v0[1], v0[2], v0[3], v1[0], v1[1], v1[2], v1[3]};
  // The two constants go through registers: written as immediates, (-1, 0) is emitted as the inline constant -1.0,
  // which this instruction does not read as the bf16 pair (-1, 0) (measured: the remainders then come out wrong).
  unsigned first_bits = 0x0000bf80u, second_bits = 0xbf800000u;
  asm("" : "+s"(first_bits), "+s"(second_bits));
  const bf16x2 minus_first = __builtin_bit_cast(bf16x2, first_bits), minus_second = __builtin_bit_cast(bf16x2, second_bits);
  u32x4 hu, mu, lu;
  auto pack = [](float a, float b) {
    const f32x2 t = {a, b};
    return __builtin_convertvector(t, bf16x2);
  };
  unsigned lead[4];   // (an array: __builtin_bit_cast of a vector's element reads element 0, whatever its index)
#pragma unroll
  for (int i = 0; i < 4; ++i) lead[i] = __builtin_bit_cast(unsigned, pack(x[2 * i], x[2 * i + 1]));
  if (FINITE) {
    float top = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) top = __builtin_fmaxf(top, __builtin_fabsf(x[i]));
    if (__any(top >= 0x1.ffp127f)) {
      // (infinity has the next bit pattern after the largest finite value, in either half and with either sign)
      auto rounded_up = [](float v) { return (__builtin_bit_cast(unsigned, v) & 0x7fffffffu) - 0x7f7f8000u < 0x8000u; };
#pragma unroll
      for (int i = 0; i < 4; ++i) lead[i] -= (rounded_up(x[2 * i]) ? 1u : 0u) + (rounded_up(x[2 * i + 1]) ? 0x10000u : 0u);
    }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float a = x[2 * i], b = x[2 * i + 1];
    const bf16x2 hp = __builtin_bit_cast(bf16x2, lead[i]);
    const float ra = __builtin_amdgcn_fdot2_f32_bf16(hp, minus_first, a, false);
    const float rb = __builtin_amdgcn_fdot2_f32_bf16(hp, minus_second, b, false);
    const bf16x2 mp = pack(ra, rb);
    const float sa = __builtin_amdgcn_fdot2_f32_bf16(mp, minus_first, ra, false);
    const float sb = __builtin_amdgcn_fdot2_f32_bf16(mp, minus_second, rb, false);
    hu[i] = lead[i];
    mu[i] = __builtin_bit_cast(unsigned, mp);
    lu[i] = __builtin_bit_cast(unsigned, pack(sa, sb));
  }
  h = __builtin_bit_cast(bf16x8, hu);
  m = __builtin_bit_cast(bf16x8, mu);
  l = __builtin_bit_cast(bf16x8, lu);
}

// Eight consecutive k of one matrix operand as its three pieces.
struct Split8 {
  bf16x8 h, m, l;
};
__device__ inline Split8 split8(const f32x4& v0, const f32x4& v1) {
  Split8 s;
  split3<true>(v0, v1, s.h, s.m, s.l);
  return s;
}

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
// The same pieces of two floats, without the test for values that the leading piece would round to infinity: the caller's operands
// stay below 0x1.ffp127 (kScaleH in zeno_internal.h).
// The remainders are masks, shifts and subtractions, eleven instructions for two floats, not the bf16 dot products of split3 (seven):
// a dot product waits for the matrix cores (next to a wave that keeps them busy 328 cycles each, the others 11; alone 8 and 9).
__device__ inline void split_pair(float a, float b, unsigned& h, unsigned& m, unsigned& l) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  auto real = [](unsigned v) { return __builtin_bit_cast(float, v); };
  auto pack = [](float x, float y) {
    const f32x2 t = {x, y};
    return __builtin_bit_cast(unsigned, __builtin_convertvector(t, bf16x2));
  };
  h = pack(a, b);
  const float ra = a - real(h << 16), rb = b - real(h & 0xffff0000u);
  m = pack(ra, rb);
  l = pack(ra - real(m << 16), rb - real(m & 0xffff0000u));
}
// Eight floats pair by pair: a kernel that works on them between its matrix instructions keeps the pieces here.
struct SplitWords {
  u32x4 h, m, l;
  template <int I>
  __device__ void pair(float a, float b) {
    unsigned x, y, z;
    split_pair(a, b, x, y, z);
    h[I] = x;
    m[I] = y;
    l[I] = z;
  }
};

// One k-step of 16 of a 32 x 32 block of products at float32 accuracy: the six piece products down to 2^-17 of the leading
// one; what is dropped is about 2^-24 of |a||b| per product, one float32 rounding.  The leading products have an
// accumulator of their own: an operand that is not finite has no useful remainder (inf - inf), and the
// leading products alone say what the float32 product would have been (join_split).  A sum of leading products may overflow
// where the float32 sum ends within 1 % of its largest value (not in linear layers, whose operands are stored scaled).
__device__ inline void mfma_split(const Split8& a, const Split8& b, f32x16& lead, f32x16& rest) {
  rest = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.l, b.h, rest, 0, 0, 0);
  rest = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.h, b.l, rest, 0, 0, 0);
  rest = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.m, b.m, rest, 0, 0, 0);
  rest = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.m, b.h, rest, 0, 0, 0);
  rest = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.h, b.m, rest, 0, 0, 0);
  lead = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.h, b.h, lead, 0, 0, 0);
}
__device__ inline float join_split(float lead, float rest) {
  return __builtin_fabsf(lead) < __builtin_inff() ? lead + rest : lead;
}

}  // namespace

}  // namespace zeno
#endif
