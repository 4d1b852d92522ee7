// Marginal median (Definition 4) for more rows than the register-resident sorting
// networks of zeno_median.hip hold: 128 < m <= 1024.
//
// A workgroup of eight waves takes COLS (64 or 32) adjacent columns at a time.  Their m x COLS values are copied
// global -> LDS (no registers), then every wave reads the columns it owns into registers, P (8 or 16) lanes per column
// and NK keys per lane, as unsigned keys whose order is -inf < ... < -0 < +0 < ... < +inf < NaN.  From then on the LDS
// tile is free: the copies of the next tile are requested and arrive while this one is searched.
//
// The search keeps, per column, a bracket lo <= x < hi around the key x of rank k = (m - 1) / 2 and the number of
// keys below either bound, and narrows it with pivots: one pass of the lanes over their registers and lane shuffles
// give the number of keys below a pivot (two instructions per key) and, for one more, the keys next to it on
// either side.  It ends when exactly k keys lie below the pivot (x is the key above it), exactly k + 1 (x is the one
// below), or the bracket holds a single value.
//  * First pass: every lane takes the median of medians of three of its own keys; the smallest and the largest of
//    the column's P such values are two pivots, and one from their middle, together with its successor, is the third
//    pair (a value that fills the middle of the column, such as the zero of an inactive unit, ends the search here).
//  * Then the pivot is interpolated between the bounds (as floats) at the rank wanted, and the bounds move to the
//    nearest keys that occur, so that a block of equal keys (colluding rows) closes the bracket as well.
//  * From the sixth pass on every third pivot is the middle of the bracket as integers, which bounds the number of passes
//    whatever the values are.
// The result depends on the values only, not on the pivots.  For even m the key of rank k + 1 is the other neighbour of the
// pivot or takes one more pass; the result is the midpoint of the two, formed in float64 and rounded once, as in
// the kernels for m <= 128.
//
// Layout of the tile: [row][column], the columns of a row permuted by an exclusive-or with a function of the row, so that the
// lanes of a wave (P rows x 64 / P columns) read 64 different banks; the copies write 64 consecutive words, so the
// permutation is applied to the addresses they read from, inside one 256- or 128-byte piece of a row.
// P = 8 and COLS = 64 up to m = 320 (the tile then fits twice into a compute unit's LDS and the keys into 40
// registers), P = 16 and COLS = 32 above.  Neighbouring tiles run on the same XCD at about the same time, whose L2
// then serves the memory lines that unaligned rows make them share.
//
// Bound by vector instructions: 39 per key for m = 300 (4 to fetch and map it, 8 for the first four pivots, about 4 to 5
// passes of 3 plus some 70 per pass and lane for the pivots; counted: 2.87e8 wave instructions for 4.7e8 keys), which take
// 78 % of the issue slots of a call of 601 us.  Measured (MI355X; a worker's gradients around a common one, a third of the rows
// faulty, calls in a series on buffers in turn): m = 300, d = 1.58 M 601 us (3.2 TB/s), where the 32 counting passes over LDS
// that this kernel replaces took 2420; on repeated, normally distributed columns m = 129, d = 3.0 M 2970 -> 595 us; m = 512,
// d = 0.8 M 1820 -> 517 us; m = 1024, d = 0.4 M 2170 -> 569 us; 40 % zeros: the same or less; values spread over sixty
// binades, where interpolation helps little: 1.8-2.5 x faster.
#include <limits.h>
#include <stdint.h>

#include "zeno_internal.h"

namespace zeno {

namespace {

constexpr int kSelThreads = 512;
constexpr unsigned kNegInfKey = 0x807fffffu;            // signed-order key of -inf: subtracted, so that NaNs of either sign wrap to the top
constexpr unsigned kPosInf = 0x7f800000u - kNegInfKey;  // keys above this one are NaNs

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
constexpr int kXor1 = 0xB1, kXor2 = 0x4E, kMirror8 = 0x141, kMirror16 = 0x140;  // lane permutations inside 4, 4, 8, 16 lanes
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
__device__ inline unsigned lanes_min(unsigned v) {
  v = umin(v, dpp<kXor1>(v));
  v = umin(v, dpp<kXor2>(v));
  v = umin(v, dpp<kMirror8>(v));
  if (P == 16) v = umin(v, dpp<kMirror16>(v));
  return v;
}

// Copies of 64 words each global -> LDS: lane i's word of copy j, from p + j * step, lands at byte lds_off + kCopyStride j + 4 i
// (lds_off wave-uniform).  m0, the copy's LDS base, is saved and restored: the compiler does not know that it changes.
constexpr unsigned kCopyStride = 8 * 256;   // the eight waves take the copies of a tile in turn
__device__ inline void lds_copy(const float* p, unsigned lds_off) {
  unsigned saved_m0;
  asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %1, off\n\ts_mov_b32 m0, %0"
               : "=&s"(saved_m0)
               : "v"(p), "s"(lds_off)
               : "memory");
}
__device__ inline void lds_copy4(const float* p, long long step, unsigned lds_off) {
  unsigned saved_m0;
  asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %5\n\ts_nop 0\n\tglobal_load_lds_dword %1, off\n\t"
               "s_add_u32 m0, m0, %6\n\ts_nop 0\n\tglobal_load_lds_dword %2, off\n\t"
               "s_add_u32 m0, m0, %6\n\ts_nop 0\n\tglobal_load_lds_dword %3, off\n\t"
               "s_add_u32 m0, m0, %6\n\ts_nop 0\n\tglobal_load_lds_dword %4, off\n\ts_mov_b32 m0, %0"
               : "=&s"(saved_m0)
               : "v"(p), "v"(p + step), "v"(p + 2 * step), "v"(p + 3 * step), "s"(lds_off), "n"(kCopyStride)
               : "memory", "scc");
}

// Number of keys below p, two instructions per key.  The comparison results go through four scalar register pairs: left to
// itself the compiler sends all of them through vcc and has to wait two cycles between a comparison and the addition
// that reads it (a vector instruction that reads a scalar register written by the one before).  In groups of four the
// three instructions in between are that distance.
template <int NK>
__device__ inline unsigned count_below(const unsigned (&u)[NK], unsigned p) {
  unsigned c = 0;
#pragma unroll
  for (int i = 0; i < NK; i += 4) {
    unsigned long long s0, s1, s2, s3;
    asm("v_cmp_lt_u32_e64 %1, %5, %9\n\tv_cmp_lt_u32_e64 %2, %6, %9\n\tv_cmp_lt_u32_e64 %3, %7, %9\n\tv_cmp_lt_u32_e64 %4, %8, %9\n\t"
        "v_addc_co_u32_e64 %0, %1, 0, %0, %1\n\tv_addc_co_u32_e64 %0, %2, 0, %0, %2\n\t"
        "v_addc_co_u32_e64 %0, %3, 0, %0, %3\n\tv_addc_co_u32_e64 %0, %4, 0, %0, %4"
        : "+v"(c), "=&s"(s0), "=&s"(s1), "=&s"(s2), "=&s"(s3)
        : "v"(u[i]), "v"(u[i + 1]), "v"(u[i + 2]), "v"(u[i + 3]), "v"(p));
  }
  return c;
}
// The same together with the neighbours of p: the differences u - p (modulo 2^32) of the keys at or above p are their
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
  d_min = lo;
  d_max = hi;
  return c;
}

template <int P, int NK>
__global__ __launch_bounds__(kSelThreads) void median_select_kernel(const float* __restrict__ G, int m, long long d,
                                                                    long long ldg, float* __restrict__ out) {
  constexpr int COLS = 8 * 64 / P;         // eight waves, 64 / P columns each
  constexpr int ROWS = 64 / COLS;          // rows a copy of 64 words covers
  extern __shared__ float tile[];          // [m rounded up to ROWS][COLS]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int part = lane & (P - 1);                       // rows part, part + P, ... of the column
  const int col = wave * (64 / P) + lane / P;
  // position of column c in row r of the tile: c ^ flip(r); the rows of a lane all have the same flip
  auto flip = [](int r) { return P == 8 ? 8 * (r & 7) : 4 * ((r >> 1) & 7); };
  const float* mine = tile + part * COLS + (col ^ flip(part));
  const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) void*)tile;
  const int n_copies = (m + ROWS - 1) / ROWS;
  const unsigned k = (unsigned)(m - 1) / 2;

  // tiles of this workgroup: the XCD (blockIdx % 8) owns a contiguous range, its workgroups take it in turn
  const long long n_tiles = (d + COLS - 1) / COLS;
  const int xcd = blockIdx.x & 7, step = gridDim.x >> 3;
  const long long t_end = n_tiles * (xcd + 1) / 8;
  long long t = n_tiles * xcd / 8 + (blockIdx.x >> 3);

  // the copies of a tile go to the waves in turn, so that all rows a wave copies have the same flip
  const int r0 = wave * ROWS + (COLS == 64 ? 0 : lane >> 5), c0 = (lane & (COLS - 1)) ^ flip(r0);
  const long long row_step = 8 * ROWS * ldg;
  auto copy_tile = [&](long long at) __attribute__((always_inline)) {
    long long c = at * COLS + c0;
    if (c >= d) c = d - 1;                               // columns beyond the end read the last one and are not written
    const float* p = G + (long long)r0 * ldg + c;
    unsigned off = lds0 + (unsigned)wave * 256u;
    int j = wave;
    for (; (j + 25) * ROWS <= m; j += 32) {              // four copies, all of whose rows exist
      lds_copy4(p, row_step, (unsigned)__builtin_amdgcn_readfirstlane((int)off));
      p += 4 * row_step;
      off += 4u * kCopyStride;
    }
    for (; j < n_copies; j += 8) {
      const bool behind = j * ROWS + (COLS == 64 ? 0 : lane >> 5) >= m;   // the odd row behind the last one: never read
      lds_copy(behind ? p - ldg : p, (unsigned)__builtin_amdgcn_readfirstlane((int)off));
      p += row_step;
      off += kCopyStride;
    }
  };
  if (t < t_end) copy_tile(t);
  for (; t < t_end; t += step) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();                                     // every wave's copies have landed
    unsigned u[NK];
#pragma unroll
    for (int i = 0; i < NK; ++i) {
      // the rows beyond m hold the top key, which no pivot counts as below it
      const bool ok = i < NK - 4 || part + P * i < m;
      const float v = mine[ok ? P * COLS * i : 0];
      u[i] = ok ? sel_key(v) : UINT_MAX;
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __syncthreads();                                     // every wave has its keys in registers
    if (t + step < t_end) copy_tile(t + step);

    unsigned lo = 0u, hi = UINT_MAX, c_lo = 0u, c_hi = (unsigned)m;
    // (a top key can only be of rank k if it is a NaN: the bracket then closes on a NaN next to it)
    auto narrow = [&](unsigned p, unsigned c) __attribute__((always_inline)) {
      const bool at_or_above = (c <= k) & (p > lo), under = (c > k) & (p < hi);   // where the key of rank k lies
      lo = at_or_above ? p : lo;
      c_lo = at_or_above ? c : c_lo;
      hi = under ? p : hi;
      c_hi = under ? c : c_hi;
    };
    {
      // medians of medians of three, in registers, then over the lanes of the column
      unsigned w[NK];
#pragma unroll
      for (int i = 0; i < NK; ++i) w[i] = u[i];
#pragma unroll
      for (int n = NK; n >= 3; n /= 3)
#pragma unroll
        for (int i = 0; i < n / 3; ++i) w[i] = umed3(w[3 * i], w[3 * i + 1], w[3 * i + 2]);
      const unsigned s_min = lanes_min<P>(w[0]), s_max = ~lanes_min<P>(~w[0]);
      unsigned v = umed3(dpp<0x00>(w[0]), dpp<0x55>(w[0]), dpp<0xAA>(w[0]));   // of lanes 0, 1, 2 of every four
      v = umin(v, dpp<kMirror8>(v));
      if (P == 16) v = umax(v, dpp<kMirror16>(v));
      const unsigned v1 = v == UINT_MAX ? v : v + 1u;
      const unsigned a = lanes_sum<P>(count_below(u, s_min) | count_below(u, s_max) << 16);
      const unsigned b = lanes_sum<P>(count_below(u, v) | count_below(u, v1) << 16);
      narrow(s_min, a & 0xffffu);
      narrow(s_max, a >> 16);
      narrow(v, b & 0xffffu);
      narrow(v1, b >> 16);
    }
    // x: the key of rank k; y: the key of rank k + 1 (even m)
    unsigned x = 0u, y = 0u;
    bool have_x = false, have_y = (m & 1) != 0;
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
      p = have_x ? x + 1u : p;                           // (a NaN's key may wrap to 0: any y is one of no consequence then)
      unsigned d_min, d_max;
      const unsigned c = lanes_sum<P>(count_and_neighbours(u, p, d_min, d_max));
      const unsigned above = p + lanes_min<P>(d_min), below = p - 1u - lanes_min<P>(~d_max);   // smallest key >= p, largest key < p
      const bool up = !have_x & (c <= k), down = !have_x & (c > k);
      y = have_x & !have_y ? (c > k + 1u ? x : above) : y;
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
    float res = sel_float(x);
    if ((m & 1) == 0) res = (float)(0.5 * ((double)res + (double)sel_float(y)));
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

template <int P, int NK>
hipError_t launch_select(const float* G, long long ldg, int m, long long d, float* out, hipStream_t stream) {
  constexpr int COLS = 8 * 64 / P, ROWS = 64 / COLS;
  const int lds_bytes = (m + ROWS - 1) / ROWS * 256;
  static const hipError_t attr_err = hipFuncSetAttribute(reinterpret_cast<const void*>(&median_select_kernel<P, NK>),
                                                         hipFuncAttributeMaxDynamicSharedMemorySize, (P * NK / ROWS) * 256);
  if (attr_err != hipSuccess) return attr_err;
  if (m > P * NK || m <= P * (NK - 4)) return hipErrorInvalidValue;   // (not the instantiation for this m)
  const int by_lds = (160 * 1024) / lds_bytes;
  const long long resident = (long long)compute_units() * (by_lds < 1 ? 1 : by_lds > 4 ? 4 : by_lds);
  const long long n_tiles = (d + COLS - 1) / COLS;
  const int grid = (int)((n_tiles < resident ? n_tiles : resident) + 7) / 8 * 8;   // a multiple of the XCDs
  hipLaunchKernelGGL((median_select_kernel<P, NK>), dim3(grid), dim3(kSelThreads), lds_bytes, stream, G, m, d, ldg, out);
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
