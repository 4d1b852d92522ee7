// Marginal median (Definition 4) for more rows than the register-resident sorting
// networks of zeno_median.hip hold: 128 < m <= 1024.
//
// A workgroup of four or eight waves takes 32 adjacent columns at a time.  Their m x 32 values are copied global -> LDS (no
// registers), then every wave reads the columns it owns into registers, P (8 or 16) lanes per column and NK values per lane.
// From then on the LDS tile is free: the copies of the next tile are requested and arrive while this one is searched.
//
// Wanted is, per column, the value x of rank k = (m - 1) / 2, for even m also y of rank k + 1.  Counting the values below a pivot
// takes two instructions per value and a sum over the column's lanes.
//  * NaNs, where a wave meets any, become infinities, and the last ranks of their column are theirs.
//  * Every lane takes the median of medians of three of its own values; their mean over the lanes is the first pivot (at rank k
//    within about 0.7 sqrt(m)), their mean deviation tells how far apart ranks are, and with it the second pivot lies within a few
//    ranks of k.
//  * The third pivot aims kAim ranks below k, and the pass that counts the values below it also keeps each lane's four smallest
//    values from it on (seven instructions per value).  The lists, merged over the lanes by a bitonic network, are complete up to the
//    smallest of the fourth values, some thirteen values for P = 8: x and y are in there, or the next pivot is the successor of
//    that value, or lies lower.
//  * Lanes that agree on a median may have met a value that fills the middle of the column (the zero of an inactive unit, colluding
//    rows): that value and its successor are counted first.  Where lanes agree in most columns of a wave, these hold few values
//    (signs, quantised gradients): the lanes' other medians are tried in the same way, or, with some ten copies of a value only, the
//    bracket follows at once.
//  * Columns that three passes with lists do not finish, and waves whose second pivot is far off, go on
//    with a bracket lo <= x < hi of keys whose order is that of the values: the pivot is interpolated between the bounds (as
//    floats) at the rank wanted, one pass gives the number of keys below it and the keys next to it on either side (three
//    instructions per key), and the bounds move to these, so that a block of equal keys closes the bracket as well.  It ends when
//    exactly k keys lie below the pivot (x is the key above it), exactly k + 1 (x is the one below), or the bracket holds a single
//    value.  From the sixth pass on every third pivot is the middle of the bracket as integers, which bounds the number of passes.
// The result depends on the values only, not on the pivots; for even m it is the midpoint of x and y, formed in float64 and rounded
// once, as in the kernels for m <= 128.
//
// Layout of the tile: [row][column], the columns of a row permuted by an exclusive-or with a function of the row, so that the
// lanes of a wave (P rows x 64 / P columns) read 64 different banks; the copies write 64 consecutive words, so the
// permutation is applied to the addresses they read from, inside one 128-byte piece of a row.
// P = 8 up to m = 320 (the values then fit into 40 registers), P = 16 above; 32 columns either way, so that a workgroup that waits
// for its slowest wave leaves three others on the compute unit up to m = 320.  A workgroup takes kRun tiles, one after the other,
// and makes room for the next one: the tiles differ in their number of passes, and with as many workgroups as the chip
// holds, each with a fixed share of all tiles, the last ones ended 8-12 % after the others (kRun = 4, 8, 16, all: 481, 481, 486,
// 508 us for m = 300, 426 - 436, 423, 429, 410 us for m = 700, where the chip holds one per compute unit).  Neighbouring tiles run on
// the same XCD at about the same time, whose L2 then serves the memory lines that unaligned rows make them share.
//
// Bound by vector instructions: 26 per value for m = 300 (counted: 2.05e8 wave instructions on normally distributed columns, 39
// per value and 2.87e8 before, when four pivots were counted first and all further passes moved by one key).  Measured (MI355X, before ->
// now; calls in a series on buffers in turn): m = 300, d = 1.58 M, a worker's gradients around a common one, a third of the rows
// faulty 602 -> 510 us (3.7 TB/s), m = 129, d = 3.0 M 560 -> 468, m = 512, d = 0.8 M 548 -> 434, m = 1024, d = 0.4 M 629 -> 525; normally
// distributed columns 18-28 % shorter; a fifth of the rows NaN 576 -> 465 for m = 300; 40 % zeros 588 -> 372.  Columns of few values,
// normally distributed and rounded to a half, a quarter, an eighth, a sixteenth of their deviation (before -> lists alone -> now): m = 300
// 535 -> 568 -> 395, 538 -> 770 -> 530, 540 -> 707 -> 544, 547 -> 560 -> 550; m = 129 448 -> 621 -> 381, 450 -> 667 -> 492, 457 ->
// 506 -> 494, 463 -> 431 -> 458; m = 1024 486 -> 500 -> 370, 529 -> 829 -> 475, 529 -> 863 -> 617, 533 -> 788 -> 598: with one
// workgroup per compute unit its slowest wave decides.  A third to a half of the rows faulty, half of these equal and off the
// middle (lanes agree on them all the same): m = 436, d = 0.86 M 536 -> 560 -> 571, m = 236, d = 1.3 M 430 -> 388 -> 395, m = 130,
// d = 3 M 583 -> 603 -> 615, m = 700, d = 0.4 M 434 -> 460 -> 472.
#include <limits.h>
#include <stdint.h>

#include "zeno_internal.h"

namespace zeno {

namespace {

constexpr unsigned kNegInfKey = 0x807fffffu;            // signed-order key of -inf: subtracted, so that NaNs of either sign wrap to the top
constexpr unsigned kPosInf = 0x7f800000u - kNegInfKey;  // keys above this one are NaNs
constexpr unsigned kZero = 0u - kNegInfKey;             // key of +0; that of -0 is the one below

__device__ inline unsigned sel_key(float f) {
  const int k = __float_as_int(f);
  return (unsigned)(k ^ (int)((unsigned)(k >> 31) >> 1)) - kNegInfKey;
}
// every NaN becomes the one whose bits are 0x7fffffff
__device__ inline float sel_float(unsigned u) {
  const int k = (int)(u + kNegInfKey);
  return __int_as_float(u > kPosInf ? INT_MAX : k ^ (int)((unsigned)(k >> 31) >> 1));
}

__device__ inline unsigned umin(unsigned a, unsigned b) { return a < b ? a : b; }
__device__ inline unsigned umax(unsigned a, unsigned b) { return a < b ? b : a; }
__device__ inline unsigned umed3(unsigned a, unsigned b, unsigned c) { return umax(umin(a, b), umin(umax(a, b), c)); }

template <int CTRL>
__device__ inline unsigned dpp(unsigned v) {
  return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, true);
}
constexpr int kRun = 8;                                 // tiles a workgroup takes one after the other
constexpr int kAim = 5;                                 // ranks by which the collecting pivot aims below the one wanted
// Columns of few values, by the copies of the value that lanes agree on, squared, per row.  Up to 1 / kSome the lists find x sooner
// than the bracket (us, lists / bracket from the lanes' medians: m = 512, 3 copies 439 / 477; m = 700, 9 copies 577 / 543; m = 1024,
// 6 copies 556 / 582, 13 copies 670 / 606); from kMany on the lanes' medians, kTries of them after the first (bracket / tries:
// m = 300, 15 copies 535 / 590, 30 copies 523 / 496; m = 1024, 50 copies 600 / 642, 100 copies 593 / 459; one try less costs 2-6 %).
constexpr int kTries = 3;
constexpr unsigned kMany = 3, kSome = 10;
constexpr unsigned kNear = 7;                            // how far off the middle that value may be: a seventh of the rows
constexpr int kXor1 = 0xB1, kXor2 = 0x4E, kXor3 = 0x1B, kMirror8 = 0x141, kMirror16 = 0x140;  // lane permutations inside 4, 4, 8, 16 lanes
// Reductions over the P lanes of a column; every lane receives the result.
template <int P>
__device__ inline unsigned lanes_sum(unsigned v) {
  v += dpp<kXor1>(v);
  v += dpp<kXor2>(v);
  v += dpp<kMirror8>(v);
  if (P == 16) v += dpp<kMirror16>(v);
  return v;
}
template <int P>
__device__ inline float lanes_add(float v) {
  v += __uint_as_float(dpp<kXor1>(__float_as_uint(v)));
  v += __uint_as_float(dpp<kXor2>(__float_as_uint(v)));
  v += __uint_as_float(dpp<kMirror8>(__float_as_uint(v)));
  if (P == 16) v += __uint_as_float(dpp<kMirror16>(__float_as_uint(v)));
  return v;
}
template <int P>
__device__ inline unsigned lanes_min(unsigned v) {
  v = umin(v, dpp<kXor1>(v));
  v = umin(v, dpp<kXor2>(v));
  v = umin(v, dpp<kMirror8>(v));
  if (P == 16) v = umin(v, dpp<kMirror16>(v));
  return v;
}

template <int P>
__device__ inline float lanes_fmin(float v) {
  const float none = -__builtin_inff();
  v = __builtin_amdgcn_fmed3f(v, __uint_as_float(dpp<kXor1>(__float_as_uint(v))), none);
  v = __builtin_amdgcn_fmed3f(v, __uint_as_float(dpp<kXor2>(__float_as_uint(v))), none);
  v = __builtin_amdgcn_fmed3f(v, __uint_as_float(dpp<kMirror8>(__float_as_uint(v))), none);
  if (P == 16) v = __builtin_amdgcn_fmed3f(v, __uint_as_float(dpp<kMirror16>(__float_as_uint(v))), none);
  return v;
}

// Bitonic merge of the P lanes' ascending lists of four (no NaNs): afterwards lane i of the column holds its values
// 4 i .. 4 i + 3 in ascending order.  A step between lanes is a move and a median with +-inf (the minimum in the lower lane, the
// maximum in the upper one) per value.
template <int CTRL, bool REVERSED>
__device__ inline void merge_step(float (&v)[4], float side) {
  float o[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) o[i] = __uint_as_float(dpp<CTRL>(__float_as_uint(v[REVERSED ? 3 - i : i])));
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = __builtin_amdgcn_fmed3f(v[i], o[i], side);
}
__device__ inline void merge_inside(float (&v)[4]) {
  const float inf = __builtin_inff();
  auto exchange = [&](float& a, float& b) __attribute__((always_inline)) {
    const float lo = __builtin_amdgcn_fmed3f(a, b, -inf), hi = __builtin_amdgcn_fmed3f(a, b, inf);
    a = lo;
    b = hi;
  };
  exchange(v[0], v[2]);
  exchange(v[1], v[3]);
  exchange(v[0], v[1]);
  exchange(v[2], v[3]);
}
template <int P>
__device__ inline void merge_lanes(float (&v)[4], int part) {
  const float inf = __builtin_inff();
  const float s1 = part & 1 ? inf : -inf, s2 = part & 2 ? inf : -inf, s4 = part & 4 ? inf : -inf;
  merge_step<kXor1, true>(v, s1);
  merge_inside(v);
  merge_step<kXor3, true>(v, s2);
  merge_step<kXor1, false>(v, s1);
  merge_inside(v);
  merge_step<kMirror8, true>(v, s4);
  merge_step<kXor2, false>(v, s2);
  merge_step<kXor1, false>(v, s1);
  merge_inside(v);
  if (P == 16) {
    const float s8 = part & 8 ? inf : -inf;
    merge_step<kMirror16, true>(v, s8);
    float o[4];                                          // lanes four apart: the mirror image of eight, and of four
#pragma unroll
    for (int i = 0; i < 4; ++i) o[i] = __uint_as_float(dpp<kXor3>(dpp<kMirror8>(__float_as_uint(v[i]))));
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = __builtin_amdgcn_fmed3f(v[i], o[i], s4);
    merge_step<kXor2, false>(v, s2);
    merge_step<kXor1, false>(v, s1);
    merge_inside(v);
  }
}
// value j of the merged lists of a column (any value, if there is none)
template <int P>
__device__ inline float pick(const float (&v)[4], int part, int j) {
  const float a = j & 1 ? v[1] : v[0], b = j & 1 ? v[3] : v[2], c = j & 2 ? b : a;
  return lanes_fmin<P>(part == j >> 2 ? c : __builtin_inff());
}

// Copies of 64 words each global -> LDS: lane i's word of copy j, from p + j * step, lands at byte lds_off + STRIDE j + 4 i
// (lds_off wave-uniform).  m0, the copy's LDS base, is saved and restored: the compiler does not know that it changes.
__device__ inline void lds_copy(const float* p, unsigned lds_off) {
  unsigned saved_m0;
  asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %1, off\n\ts_mov_b32 m0, %0"
               : "=&s"(saved_m0)
               : "v"(p), "s"(lds_off)
               : "memory");
}
template <unsigned STRIDE>   // bytes between the copies: the waves take the copies of a tile in turn
__device__ inline void lds_copy4(const float* p, long long step, unsigned lds_off) {
  unsigned saved_m0;
  asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %5\n\ts_nop 0\n\tglobal_load_lds_dword %1, off\n\t"
               "s_add_u32 m0, m0, %6\n\ts_nop 0\n\tglobal_load_lds_dword %2, off\n\t"
               "s_add_u32 m0, m0, %6\n\ts_nop 0\n\tglobal_load_lds_dword %3, off\n\t"
               "s_add_u32 m0, m0, %6\n\ts_nop 0\n\tglobal_load_lds_dword %4, off\n\ts_mov_b32 m0, %0"
               : "=&s"(saved_m0)
               : "v"(p), "v"(p + step), "v"(p + 2 * step), "v"(p + 3 * step), "s"(lds_off), "n"(STRIDE)
               : "memory", "scc");
}

// The lane permutations read a register two instructions after it was written at the earliest; the compiler keeps that distance
// to its own instructions, but does not look into assembly for the write.
__device__ inline void settle(unsigned& v) { asm("s_nop 1" : "+v"(v)); }
__device__ inline void settle(unsigned& v, float& w) { asm("s_nop 1" : "+v"(v), "+v"(w)); }

// Number of values below p, two instructions per value, as floats or as keys.  The comparison results go through four scalar
// register pairs: left to itself the compiler sends all of them through vcc and has to wait two cycles between a comparison and
// the addition that reads it (a vector instruction that reads a scalar register written by the one before).  In groups of four the
// three instructions in between are that distance.
template <int NK>
__device__ inline unsigned count_below(const unsigned (&u)[NK], float p) {
  unsigned c = 0;
#pragma unroll
  for (int i = 0; i < NK; i += 4) {
    unsigned long long s0, s1, s2, s3;
    asm("v_cmp_lt_f32_e64 %1, %5, %9\n\tv_cmp_lt_f32_e64 %2, %6, %9\n\tv_cmp_lt_f32_e64 %3, %7, %9\n\tv_cmp_lt_f32_e64 %4, %8, %9\n\t"
        "v_addc_co_u32_e64 %0, %1, 0, %0, %1\n\tv_addc_co_u32_e64 %0, %2, 0, %0, %2\n\t"
        "v_addc_co_u32_e64 %0, %3, 0, %0, %3\n\tv_addc_co_u32_e64 %0, %4, 0, %0, %4"
        : "+v"(c), "=&s"(s0), "=&s"(s1), "=&s"(s2), "=&s"(s3)
        : "v"(u[i]), "v"(u[i + 1]), "v"(u[i + 2]), "v"(u[i + 3]), "v"(p));
  }
  settle(c);
  return c;
}
// The same together with the four smallest values at or above p (first <= ... <= fourth, +inf where there are fewer), seven
// instructions per value: those below p are taken as +inf, and a value enters the sorted list with three medians of three and a minimum.
template <int NK>
__device__ inline unsigned count_and_collect(const unsigned (&u)[NK], float p, float (&first)[4]) {
  unsigned c = 0;
  float inf = __builtin_inff(), m1 = inf, m2 = inf, m3 = inf, m4 = inf;
  asm("" : "+v"(inf));                                   // (in a vector register: the selection already reads a scalar one)
#pragma unroll
  for (int i = 0; i < NK; i += 4) {
    unsigned long long s0, s1, s2, s3;
    float t[4];
    asm("v_cmp_lt_f32_e64 %1, %9, %13\n\tv_cmp_lt_f32_e64 %2, %10, %13\n\tv_cmp_lt_f32_e64 %3, %11, %13\n\t"
        "v_cmp_lt_f32_e64 %4, %12, %13\n\t"
        "v_addc_co_u32_e64 %0, vcc, 0, %0, %1\n\tv_addc_co_u32_e64 %0, vcc, 0, %0, %2\n\t"
        "v_addc_co_u32_e64 %0, vcc, 0, %0, %3\n\tv_addc_co_u32_e64 %0, vcc, 0, %0, %4\n\t"
        "v_cndmask_b32_e64 %5, %9, %14, %1\n\tv_cndmask_b32_e64 %6, %10, %14, %2\n\t"
        "v_cndmask_b32_e64 %7, %11, %14, %3\n\tv_cndmask_b32_e64 %8, %12, %14, %4"
        : "+v"(c), "=&s"(s0), "=&s"(s1), "=&s"(s2), "=&s"(s3), "=&v"(t[0]), "=&v"(t[1]), "=&v"(t[2]), "=&v"(t[3])
        : "v"(u[i]), "v"(u[i + 1]), "v"(u[i + 2]), "v"(u[i + 3]), "v"(p), "v"(inf)
        : "vcc");
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      m4 = __builtin_amdgcn_fmed3f(m3, t[q], m4);
      m3 = __builtin_amdgcn_fmed3f(m2, t[q], m3);
      m2 = __builtin_amdgcn_fmed3f(m1, t[q], m2);
      asm("v_min_f32_e32 %0, %0, %1" : "+v"(m1) : "v"(t[q]));
    }
  }
  settle(c, m1);
  first[0] = m1, first[1] = m2, first[2] = m3, first[3] = m4;
  return c;
}
// Number of keys below p together with the neighbours of p: the differences u - p (modulo 2^32) of the keys at or above p are their
// distances, those of the keys below p lie above all of these, so the smallest difference belongs to the smallest key >= p
// and the largest one to the largest key < p (where there are any).  The borrow of the subtraction is the comparison.
template <int NK>
__device__ inline unsigned count_and_neighbours(const unsigned (&u)[NK], unsigned p, unsigned& d_min, unsigned& d_max) {
  unsigned c = 0, lo = UINT_MAX, hi = 0u;
#pragma unroll
  for (int i = 0; i < NK; i += 4) {
    unsigned long long s0, s1, s2, s3;
    unsigned d0, d1, d2, d3;
    asm("v_sub_co_u32_e64 %5, %1, %9, %13\n\tv_sub_co_u32_e64 %6, %2, %10, %13\n\tv_sub_co_u32_e64 %7, %3, %11, %13\n\t"
        "v_sub_co_u32_e64 %8, %4, %12, %13\n\t"
        "v_addc_co_u32_e64 %0, %1, 0, %0, %1\n\tv_addc_co_u32_e64 %0, %2, 0, %0, %2\n\t"
        "v_addc_co_u32_e64 %0, %3, 0, %0, %3\n\tv_addc_co_u32_e64 %0, %4, 0, %0, %4"
        : "+v"(c), "=&s"(s0), "=&s"(s1), "=&s"(s2), "=&s"(s3), "=&v"(d0), "=&v"(d1), "=&v"(d2), "=&v"(d3)
        : "v"(u[i]), "v"(u[i + 1]), "v"(u[i + 2]), "v"(u[i + 3]), "v"(p));
    lo = umin(umin(lo, d0), d1);
    lo = umin(umin(lo, d2), d3);
    hi = umax(umax(hi, d0), d1);
    hi = umax(umax(hi, d2), d3);
  }
  settle(c);
  d_min = lo;
  d_max = hi;
  return c;
}

template <int P, int NK, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void median_select_kernel(const float* __restrict__ G, int m, long long d,
                                                                   long long ldg, int step, float* __restrict__ out) {
  constexpr int COLS = WAVES * 64 / P;     // 64 / P columns a wave
  constexpr int ROWS = 64 / COLS;          // rows a copy of 64 words covers
  constexpr unsigned STRIDE = WAVES * 256;
  static_assert(COLS == 32 && (P == 8 || P == 16), "the permutation of a row's columns");
  extern __shared__ float tile[];          // [m rounded up to ROWS][COLS]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int part = lane & (P - 1);                       // rows part, part + P, ... of the column
  const int col = wave * (64 / P) + lane / P;
  // position of column c in row r of the tile: c ^ flip(r); the rows of a lane all have the same flip
  auto flip = [](int r) { return P == 8 ? 8 * ((r >> 1) & 3) : 4 * ((r >> 1) & 7); };
  const float* mine = tile + part * COLS + (col ^ flip(part));
  const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) void*)tile;
  const int n_copies = (m + ROWS - 1) / ROWS;
  const unsigned k = (unsigned)(m - 1) / 2, reach = (unsigned)m / kNear;
  const float rank_scale = __builtin_amdgcn_rsqf((float)(P * m)) * (1.f / (0.55f * P));   // mean deviation of the lanes' medians -> one rank

  // tiles of this workgroup: the XCD (blockIdx % 8) owns a contiguous range; `step` workgroups at a time take kRun tiles each in turn
  const long long n_tiles = (d + COLS - 1) / COLS;
  const int xcd = blockIdx.x & 7, nth = blockIdx.x >> 3;
  const long long first = n_tiles * xcd / 8, last = n_tiles * (xcd + 1) / 8;
  long long t = first + (long long)(nth / step) * step * kRun + nth % step;
  const long long run_end = first + (long long)(nth / step + 1) * step * kRun, t_end = run_end < last ? run_end : last;

  // the copies of a tile go to the waves in turn, so that all rows a wave copies have the same flip
  const int r0 = wave * ROWS + (lane >> 5), c0 = (lane & (COLS - 1)) ^ flip(r0);
  const long long row_step = WAVES * ROWS * ldg;
  auto copy_tile = [&](long long at) __attribute__((always_inline)) {
    long long c = at * COLS + c0;
    if (c >= d) c = d - 1;                               // columns beyond the end read the last one and are not written
    const float* p = G + (long long)r0 * ldg + c;
    unsigned off = lds0 + (unsigned)wave * 256u;
    int j = wave;
    for (; (j + 3 * WAVES + 1) * ROWS <= m; j += 4 * WAVES) {   // four copies, all of whose rows exist
      lds_copy4<STRIDE>(p, row_step, (unsigned)__builtin_amdgcn_readfirstlane((int)off));
      p += 4 * row_step;
      off += 4u * STRIDE;
    }
    for (; j < n_copies; j += WAVES) {
      const bool behind = j * ROWS + (lane >> 5) >= m;   // the odd row behind the last one: never read
      lds_copy(behind ? p - ldg : p, (unsigned)__builtin_amdgcn_readfirstlane((int)off));
      p += row_step;
      off += STRIDE;
    }
  };
  if (t < t_end) copy_tile(t);
  for (; t < t_end; t += step) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();                                     // every wave's copies have landed
    unsigned u[NK];
    bool no_number = false;
#pragma unroll
    for (int i = 0; i < NK; ++i) {
      // the rows beyond m hold +inf, which no pivot counts as below it
      const bool ok = i < NK - 4 || part + P * i < m;
      const float v = mine[ok ? P * COLS * i : 0];
      u[i] = ok ? __float_as_uint(v) : 0x7f800000u;
    }
#pragma unroll
    for (int i = 0; i < NK; i += 2) no_number |= __builtin_isunordered(__uint_as_float(u[i]), __uint_as_float(u[i + 1]));
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __syncthreads();                                     // every wave has its keys in registers
    if (t + step < t_end) copy_tile(t + step);

    // x: the key of rank k; y: the key of rank k + 1 (even m)
    unsigned lo = 0u, hi = UINT_MAX, c_lo = 0u, c_hi = (unsigned)m, x = 0u, y = 0u;
    bool have_x = false, have_y = (m & 1) != 0;
    unsigned nans = 0u;
    if (__ballot(no_number) != 0) {
      // NaNs are the highest values of their column: from here on they are infinities, and the last ranks
#pragma unroll
      for (int i = 0; i < NK; ++i) {
        const bool nan = __builtin_isnan(__uint_as_float(u[i]));
        nans += nan ? 1u : 0u;
        u[i] = nan ? 0x7f800000u : u[i];
      }
      nans = lanes_sum<P>(nans);
    }
    {
      float flo = -__builtin_inff(), fhi = __builtin_inff();
      auto bound = [&](float p, unsigned c) __attribute__((always_inline)) {
        const bool under = (c <= k) & (p > flo), above = (c > k) & (p < fhi);
        flo = under ? p : flo;
        c_lo = under ? c : c_lo;
        fhi = above ? p : fhi;
        c_hi = above ? c : c_hi;
      };
      // medians of medians of three in registers; their mean over the column's lanes is the first pivot, their mean deviation
      // from it the scale of a rank
      float w[NK - 4];                                   // (the last four may lie beyond m)
#pragma unroll
      for (int i = 0; i < NK - 4; ++i) w[i] = __uint_as_float(u[i]);
#pragma unroll
      for (int n = NK - 4; n >= 3; n /= 3)
#pragma unroll
        for (int i = 0; i < n / 3; ++i) w[i] = __builtin_amdgcn_fmed3f(w[3 * i], w[3 * i + 1], w[3 * i + 2]);
      const unsigned wb = __float_as_uint(w[0]);
      float p = lanes_add<P>(w[0]) * (1.f / P);
      const float slope = lanes_add<P>(__builtin_fabsf(w[0] - p)) * rank_scale;
      // lanes that agree on a value: it may fill the middle of the column (the zero of an inactive unit, colluding rows)
      const bool twin = (wb == dpp<kXor1>(wb)) | (wb == dpp<kXor2>(wb)) | (wb == dpp<kMirror8>(wb)) | (P == 16 && wb == dpp<kMirror16>(wb));
      unsigned after = 0u;                               // the key whose successor the pivot is, where no wanted key is below it
      bool behind = false;                               // whether the pivot is such a one
      bool few = false;                                  // columns of few values, which the slope does not find: no lists
      const unsigned long long twins = __ballot(twin);
      if (twins != 0) {
        // A lane's median and its successor are pivots: the values of rank k and k + 1 end here if they are that value.
        bool own = twin;                                 // lanes whose median is tried
        float aim_at = p;
#pragma unroll 1
        for (int tries = 0;; ++tries) {
          const float apart = own ? __builtin_fabsf(w[0] - aim_at) : __builtin_inff(), least = lanes_fmin<P>(apart);
          const unsigned key = ~lanes_min<P>((own & (apart == least)) ? ~sel_key(w[0] + 0.f) : UINT_MAX);   // 0: none
          const float tv = key != 0u ? sel_float(key) : p, tn = key != 0u ? sel_float(key + 1u) : p;
          const unsigned b = lanes_sum<P>(count_below(u, tv) | count_below(u, tn) << 16);
          const unsigned c0 = b & 0xffffu, c1 = b >> 16;
          bound(tv, c0);
          bound(tn, c1);
          // (no key: c0 and c1 are the same; a value above x: c0 is above k)
          const bool got_x = (c0 <= k) & (c1 > k), got_y = (c0 <= k + 1u) & (c1 > k + 1u);
          x = got_x ? key : x;
          y = got_y ? key : y;
          have_x |= got_x;
          have_y |= got_y;
          const bool left = !(have_x & have_y);
          if (__ballot(left) == 0) break;
          if (tries == 0) {
            behind = got_x;
            after = key;
            // Few values: lanes agree on one with some copies, not far from the middle, in (nearly) all columns, or in half of them and
            // not on account of a single value with many.
            const bool here = (c1 > c0) & (c0 <= k + reach) & (c1 > k - reach);
            const int agreed = __popcll(__ballot(here));
            int many = 0;
            if (agreed >= 32) {
              const unsigned copies = (c1 - c0) * (c1 - c0);
              const int some = __popcll(__ballot(here & (kSome * copies >= (unsigned)m)));
              many = __popcll(__ballot(here & (copies >= kMany * (unsigned)m)));
              few = 2 * some >= agreed && (agreed >= (P == 8 ? 48 : 64) || 2 * many < agreed);
            }
            const bool try_others = few & (many >= 32);
            few |= __popcll(twins) >= 32;                  // (half the lanes agreeing on a value far from the middle: the bracket, too)
            if (!few) {
              p = got_x ? tn : p;
              break;
            }
            if (!try_others) {
              // the bracket finds it sooner; its other end is the outermost of the lanes' medians
              const float side = c1 <= k ? -lanes_fmin<P>(-w[0]) : lanes_fmin<P>(w[0]);
              bound(side, lanes_sum<P>(count_below(u, side)));
              break;
            }
          }
          // the next one: for y the lowest above x, for x the one nearest to where the slope puts it
          aim_at = have_x ? sel_float(x) : c1 <= k ? tv + (float)(k - c1) * slope : tv - (float)(c0 - k) * slope;
          own = left & (have_x ? w[0] > aim_at : (w[0] >= flo) & (w[0] < fhi));
          if (__ballot(own) == 0 || tries == kTries) break;
        }
      }
      if ((__ballot(!(have_x & have_y)) != 0) & !few) {
        unsigned c = lanes_sum<P>(count_below(u, p));
        bound(p, c);
        // a second pivot, at rank k as far as the scale tells, and one a few ranks below it
        const float p1 = p;
        const unsigned c1 = c;
        p = have_x ? p : p + (float)((int)k - (int)c) * slope;
        c = lanes_sum<P>(count_below(u, p));
        bound(p, c);
        const int off = (int)c - (int)k;
        const bool far = !have_x & ((unsigned)(off < 0 ? -off : off) > k / 4u);
        const bool near = __popcll(__ballot(far)) < 24;
        // the slope between the two pivots, if they are far enough apart to tell, not too far from the first guess
        const float rise = __builtin_amdgcn_fmed3f((p - p1) * __builtin_amdgcn_rcpf((float)((int)c - (int)c1)), slope * (1.f / 3.f), slope * 3.f);
        const unsigned moved = c > c1 ? c - c1 : c1 - c;
        float q = p + (float)(-off - kAim) * (moved >= 4u ? rise : slope);
#pragma unroll 1
        for (int it = 0; near; ++it) {
          // between two bounds the pivot is interpolated; otherwise the slope leads to it
          const float between = flo + (float)((int)k - kAim - (int)c_lo) * (fhi - flo) * __builtin_amdgcn_rcpf((float)(c_hi - c_lo));
          const bool both = (flo > -__builtin_inff()) & (fhi < __builtin_inff());
          q = both ? ((int)k - kAim <= (int)c_lo ? flo : between) : q;
          p = behind ? sel_float(after + 1u) : q;
          float list[4];
          c = lanes_sum<P>(count_and_collect(u, p, list));
          bound(p, c);
          // up to the smallest of the lanes' fourth values the lists are complete; merged, they hold the column's values from p
          // on, four consecutive ones in every lane
          float last = lanes_fmin<P>(list[3]);
          merge_lanes<P>(list, part);
          const int want_x = (int)k - (int)c, want_y = want_x + 1;
          float kx = pick<P>(list, part, want_x), ky = kx;
          if ((m & 1) == 0) ky = pick<P>(list, part, want_y);
          const bool in_x = (want_x < 0) ? behind : (want_x < 4 * P) & (kx <= last);
          const bool in_y = (want_y < 0) ? behind : (want_y < 4 * P) & (ky <= last);
          const bool low = !behind & ((!have_x & (want_x < 0)) | (!have_y & (want_y < 0)));
          const bool got_x = !have_x & in_x, got_y = !have_y & in_y;
          x = got_x ? (want_x < 0 ? after : sel_key(kx + 0.f)) : x;   // (-0 + 0 is +0: one zero only, for now)
          y = got_y ? (want_y < 0 ? after : sel_key(ky + 0.f)) : y;
          const bool unreached = !low & !((have_x | got_x) & (have_y | got_y));
          have_x |= got_x;
          have_y |= got_y;
          if (__ballot(!(have_x & have_y)) == 0 || it == 2) break;
          // not in the lists: beyond all that they tell (then the next pivot is the successor of that), or below the pivot
          behind = unreached & (want_x < kAim + 16);
          after = sel_key(last + 0.f);
          const float from = unreached ? p : fhi;
          q = from + (float)((int)k - kAim - (int)(unreached ? c : c_hi)) * slope;
        }
      }
      // Comparisons of floats take the two zeros for one: a zero of some rank is the negative one where more values have their
      // sign set.
      const bool zero_x = have_x & (x == kZero), zero_y = have_y & (y == kZero);
      if (__ballot(zero_x | zero_y) != 0) {
        unsigned c = 0u, signs = 0u;
#pragma unroll
        for (int i = 0; i < NK; ++i) {                   // the signs of 32 values in a register
          signs = __builtin_amdgcn_alignbit(signs, u[i], 31);
          if (i % 32 == 31 || i == NK - 1) c += __builtin_popcount(signs), signs = 0u;
        }
        c = lanes_sum<P>(c);
        x = zero_x & (k < c) ? kZero - 1u : x;
        y = zero_y & (k + 1u < c) ? kZero - 1u : y;
      }
      // (keys tell the two zeros apart)
      lo = flo > -__builtin_inff() ? sel_key(flo == 0.f ? -0.f : flo) : 0u;
      hi = fhi < __builtin_inff() ? sel_key(fhi == 0.f ? -0.f : fhi) : UINT_MAX;
    }
    if (__ballot(!(have_x & have_y)) != 0) {
#pragma unroll
      for (int i = 0; i < NK; ++i) u[i] = sel_key(__uint_as_float(u[i]));
    }
    const float aim = (m & 1) != 0 ? 0.5f : 1.0f;          // even m: between the keys of rank k and k + 1
    for (int it = 1;; ++it) {
      const bool closed = !have_x & (hi - lo <= 1u);
      x = closed ? lo : x;
      have_x |= closed;
      if (__ballot(!(have_x & have_y)) == 0) break;
      // pivot: interpolated; a bound whose rank is already right, for its neighbour; or, for y, the successor of x
      const float lf = sel_float(lo), hf = sel_float(hi);
      float frac = ((float)(k - c_lo) + aim) * __builtin_amdgcn_rcpf((float)(c_hi - c_lo));
      frac = __builtin_amdgcn_fmed3f(frac, 0.02f, 0.98f);
      unsigned p = sel_key(lf + (hf - lf) * frac);
      const bool inside = (p - lo - 1u < hi - lo - 1u) & !(it >= 6 && it % 3 == 0);   // lo < p < hi
      p = inside ? p : lo + ((hi - lo) >> 1);
      p = c_hi == k + 1u ? hi : p;
      p = c_lo == k ? lo : p;
      p = have_x ? x + 1u : p;
      unsigned d_min, d_max;
      const unsigned c = lanes_sum<P>(count_and_neighbours(u, p, d_min, d_max));
      const unsigned above = p + lanes_min<P>(d_min), below = p - 1u - lanes_min<P>(~d_max);   // smallest key >= p, largest key < p
      const bool up = !have_x & (c <= k), down = !have_x & (c > k);
      y = (have_x & !have_y) ? (c > k + 1u ? x : above) : y;
      have_y |= have_x;
      lo = up ? above : lo;
      c_lo = up ? c : c_lo;
      hi = down ? below + 1u : hi;
      c_hi = down ? c : c_hi;
      const bool x_above = up & (c == k), x_below = down & (c == k + 1u);
      x = x_above ? above : (x_below ? below : x);
      y = x_below ? above : y;
      have_x |= x_above | x_below;
      have_y |= x_below;
    }
    float res = k + nans >= (unsigned)m ? __builtin_nanf("") : sel_float(x);
    if ((m & 1) == 0) res = (float)(0.5 * ((double)res + (double)(k + 1u + nans >= (unsigned)m ? __builtin_nanf("") : sel_float(y))));
    if (part == 0 && t * COLS + col < d) out[t * COLS + col] = res;
  }
}

int compute_units() {
  static const int n_cu = [] {
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v < 1)
      v = 256;
    return v;
  }();
  return n_cu;
}

template <int P, int NK, int WAVES = P / 2>
hipError_t launch_select(const float* G, long long ldg, int m, long long d, float* out, hipStream_t stream) {
  constexpr int COLS = WAVES * 64 / P, ROWS = 64 / COLS;
  const int lds_bytes = (m + ROWS - 1) / ROWS * 256;
  static const hipError_t attr_err = hipFuncSetAttribute(reinterpret_cast<const void*>(&median_select_kernel<P, NK, WAVES>),
                                                         hipFuncAttributeMaxDynamicSharedMemorySize, (P * NK / ROWS) * 256);
  if (attr_err != hipSuccess) return attr_err;
  if (m > P * NK || m <= P * (NK - 4)) return hipErrorInvalidValue;   // (not the instantiation for this m)
  const int by_lds = (160 * 1024) / lds_bytes;
  const long long resident = (long long)compute_units() * (by_lds < 1 ? 1 : by_lds > 32 / WAVES ? 32 / WAVES : by_lds);
  const long long n_tiles = (d + COLS - 1) / COLS;
  const long long per_xcd = (n_tiles + 7) / 8, step = per_xcd < resident / 8 ? per_xcd : resident / 8;
  const long long runs = (per_xcd + step * kRun - 1) / (step * kRun), rest = per_xcd - (runs - 1) * step * kRun;
  const long long grid = 8 * ((runs - 1) * step + (rest < step ? rest : step));
  hipLaunchKernelGGL((median_select_kernel<P, NK, WAVES>), dim3((unsigned)grid), dim3(64 * WAVES), lds_bytes, stream, G, m, d, ldg,
                     (int)step, out);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_median_select(const float* G, long long ldg, int m, long long d, float* out, hipStream_t stream) {
  // keys per lane: m / P rounded up to a multiple of four (the kernel looks at the row of the last four slots only)
  if (m <= 128 || m > 1024) return hipErrorInvalidValue;
  if (m <= 160) return launch_select<8, 20>(G, ldg, m, d, out, stream);
  if (m <= 192) return launch_select<8, 24>(G, ldg, m, d, out, stream);
  if (m <= 224) return launch_select<8, 28>(G, ldg, m, d, out, stream);
  if (m <= 256) return launch_select<8, 32>(G, ldg, m, d, out, stream);
  if (m <= 288) return launch_select<8, 36>(G, ldg, m, d, out, stream);
  if (m <= 320) return launch_select<8, 40>(G, ldg, m, d, out, stream);
  if (m <= 384) return launch_select<16, 24>(G, ldg, m, d, out, stream);
  if (m <= 448) return launch_select<16, 28>(G, ldg, m, d, out, stream);
  if (m <= 512) return launch_select<16, 32>(G, ldg, m, d, out, stream);
  if (m <= 576) return launch_select<16, 36>(G, ldg, m, d, out, stream);
  if (m <= 640) return launch_select<16, 40>(G, ldg, m, d, out, stream);
  if (m <= 704) return launch_select<16, 44>(G, ldg, m, d, out, stream);
  if (m <= 768) return launch_select<16, 48>(G, ldg, m, d, out, stream);
  if (m <= 832) return launch_select<16, 52>(G, ldg, m, d, out, stream);
  if (m <= 896) return launch_select<16, 56>(G, ldg, m, d, out, stream);
  if (m <= 960) return launch_select<16, 60>(G, ldg, m, d, out, stream);
  return launch_select<16, 64>(G, ldg, m, d, out, stream);
}

}  // namespace zeno
