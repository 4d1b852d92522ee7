// Convolutional f_r for the Stochastic Descendant Score (Definition 2; Section 6.1 evaluates
// Zeno on a network of convolutional layers followed by one fully connected layer).
//
// A 3 x 3 convolution with zero padding is a linear layer applied to every output position's
// patch, so the candidates are propagated exactly as through linear layers: for source s
//
//   pass at x:     Z0 = patches(H0) W^T + b,   H0_out = relu(Z0)
//   candidate s:   dZ = -gamma ( patches(H0) U_s^T + patches(D_s) (W - gamma U_s)^T + ub_s ),
//                  D_out = (relu(Z0 + dZ) - relu(Z0)) (-1/gamma)
//
// with W, U_s the kernels [c_out][ky][kx][c_in] of x and of candidate s, H0 the input map of
// the pass at x and D_s the scaled change of candidate s's input map (absent at the first
// convolution).  Nothing is unfolded in memory: a patch element (position, tap, channel) is
// gathered from the NHWC map when a lane needs it as a matrix operand.
//
// conv_packed_kernel (models whose first convolution has up to eight input channels and all others a multiple of eight above, where
// conv_fragments_cost expects a gain).  The products run on the bf16 matrix cores at float32 accuracy: both operands are split into
// three bf16 pieces each and the six leading piece products accumulated (zeno_split.h).  Six v_mfma_f32_32x32x16_bf16 cover 16 channels of a tap in 192 cycles
// where v_mfma_f32_32x32x2_f32 needs 512.  K is walked in units of (map of x or of the candidate) x (sixteen input channels), nine
// steps (taps) each.
//  * Every value is split once.  The first launch writes the kernels, U and W - gamma U, as fragments in the lanes' order (ConvPack),
//    and every launch writes its results as a split map for the next (split_map_bytes), from which a workgroup copies the
//    pixels that its positions touch, border included, straight to LDS: a copy is 64 lanes x 16 bytes without registers, the pixels'
//    offsets are computed once per workgroup.  With stride 2 even and odd pixels of a row are kept apart in LDS, so that
//    consecutive positions read consecutive 16-byte pieces.
//  * A workgroup is eight waves with 64 positions x 32 channels, which share out the steps, three fragments requested ahead, and
//    add their accumulators through LDS in a fixed order; two workgroups per compute unit.  The candidates' first convolution
//    (conv_flat) gives each wave 32 positions of its own instead.
//  * The launch of the candidates' convolution l carries the pass at x through convolution l + 1.
// Bound by latency: of the 12 us of a workgroup of 32 -> 32 channels with stride 2 (m = 20, n_r = 32) 2.6 pass before its first
// copies are requested, 1.9 and 2.4 waiting for the copies of its two stages, 1.2 in the products of each, 2 in the sums and results.
// Measured (MI355X, 32 x 32 x 3 images, convolutions 32-32-64-64 with strides 1-2-1-2, m = 20) against the kernels below:
// n_r = 32, candidates' convolutions 66 + 10 / 99 + 10 / 109 + 13 / 115 us with the pass at x on its own -> 64 / 79 / 109 / 65, fragments 6 us,
// the step 455 -> 343 us (331 with fc_sample); n_r = 4: 35 / 33 / 23 us for the last three -> 18 / 20 / 17, the step 159 -> 118 us
// (104).  Other models: conv_fragments_cost.  Models with other convolutions among them would alternate between both kinds of maps,
// in two launches for every one: 0.81-0.95 on 14 of 18, so they keep to the kernels below.  Splitting the maps in the workgroup that stages them (four times as many vector instructions): 106 us where the copies
// take 79; persistent workgroups that request the next candidate's copies ahead of their sums: 95.
//
// conv_wide_kernel, conv_deep_kernel (other models, the pass at x through the first convolution, and calls whose workspace holds no
// fragments).  The same products; a wave
// owns 32 output channels x 32 PB output positions (kernel values as the first operand, so that an accumulator lane is
// a position and its registers are channels).  K is walked in units of (map of x or of the candidate) x (chunk of eight or
// sixteen input channels), nine taps each; channels are padded to the chunk, and chunks of eight take two taps per step.
//  * Map values, which nine taps and all channel tiles use, are split once: a workgroup stages the rows of the
//    input map that its positions touch, with their zero border, as [piece][eight channels][pixel] in LDS, and every lane
//    reads its position's eight channels of a tap as one 128-bit piece at a fixed offset from the position: no masks,
//    and consecutive positions lie on consecutive 16-byte pieces (stride 1).
//  * Launches with many tiles (wide: four waves, 128 positions x 32 or 64 channels): kernel values are split once per
//    workgroup as well and staged next to the map; W - gamma U is formed in float32 first.  The next unit's values are
//    requested before the present one is multiplied.
//  * Launches with few tiles (deep: eight waves, 64 positions x 32 channels): up to four units are staged at once, the
//    waves share out the steps, each with its own kernel values straight from memory, and add their accumulators
//    through LDS in a fixed order; the results are finished by all of them.
// Where both are deep, a launch carries the candidates' convolution l and the pass at x through convolution l + 1, whose
// input map the launch before completed.  The first launch carries the pass at x through convolution 0 and two
// small jobs that nothing in it depends on (clearing the arrival counters of the fully connected layer, the squared norms of the
// kernels; before: two launches).
// Bound by latency: unit by unit a workgroup requests its values, waits for them, splits and multiplies; the matrix cores are
// busy for 5-26 % of the candidates' launches, the vector ALU for 17-54 % (counted).  Measured (MI355X, 32 x 32 x 3 images,
// convolutions 32-32-64-64 with strides 1-2-1-2, m = 20) against conv_layer_kernel for everything: n_r = 32, candidates'
// convolutions 109 / 134 / 251 / 120 -> 65 / 99 / 110 / 115 us, the whole step 682 -> 454 us; n_r = 4: 19 / 26 / 36 / 32 us and
// 47 us for the pass at x -> 22 (two launches) / 35 / 32 / 23 us including it and 9 us for its first convolution, the step 209 ->
// 159 us (both with the loss and the score in one launch).
//
// conv_layer_kernel serves what the staging does not cover (rows of the map too wide for LDS) or covers badly (channels that
// are no multiple of eight, see launch_conv): one wave owns 32 positions x 32
// channels in one fp32 accumulator block (v_mfma_f32_32x32x2_f32), and gathers every operand element from memory when it
// needs it (one 128-bit load per lane and operand feeds four matrix instructions; the tail of a channel
// count that is not a multiple of eight goes two at a time).  It carries the pass at x through the next layer as well, in its
// first row of workgroups (a launch of its own is 10-13 us; convolutions 33-33-8 with strides 2 on 32x32, m = 39, n_r = 4: the
// step 125 us with separate launches for everything, 114 us now).
// The last convolution writes its outputs straight into the matrix-operand
// order of the fully connected layer (rows = samples, columns = (y, x, c)), which the
// streaming layer kernel then consumes.
#include <cmath>

#include "zeno_index.h"
#include "zeno_layer_impl.h"
#include "zeno_split.h"

namespace zeno {

namespace {

__global__ __launch_bounds__(256) void fill_zero_kernel(uint4* __restrict__ p, long long n16) {
  const uint4 z = {0u, 0u, 0u, 0u};
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += (long long)gridDim.x * blockDim.x) p[i] = z;
}

// Results of one accumulator value: position r, channel fo (pre-activation of the pass at x, or its change).
__device__ inline float conv_result(const ConvArgs& a, bool cand, float val, float z0) {
  if (!cand) return relu_nan(val);
  const float dz = -a.gamma * val;
  const float hr = relu_nan(z0 + dz);
  // relu(z0 + dz) - relu(z0) without cancellation
  const float dd = (z0 > 0.f) ? ((dz < -z0) ? -z0 : dz) : hr;
  return dd * a.neg_inv_gamma;
}

constexpr int kDeepSteps = 36;   // matrix steps a workgroup of conv_deep_kernel stages at once

// Value `off` bytes behind a wave-uniform base (32-bit offsets: one register, no address arithmetic).
template <typename V>
__device__ inline V at_byte(const float* __restrict__ base, unsigned off) {
  return *reinterpret_cast<const V*>(reinterpret_cast<const char*>(base) + off);
}
// Eight consecutive floats `off` bytes behind base, of which the first nv exist (nv may be <= 0); the others are zero.  No
// branches, so that the loads of many items are in flight together: what does not exist is read from where something does.
// FULL: the channels are a multiple of eight, so that all eight exist or none.
template <bool FULL>
__device__ inline void load8(const float* __restrict__ base, unsigned off, int nv, f32x4& v0, f32x4& v1) {
  const unsigned p = nv > 0 ? off : 0u;
  if (FULL) {
    v0 = at_byte<f32x4_a4>(base, p);
    v1 = at_byte<f32x4_a4>(base, p + 16u);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v0[i] = nv > 0 ? v0[i] : 0.f;
      v1[i] = nv > 0 ? v1[i] : 0.f;
    }
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v0[i] = at_byte<float>(base, p + (i < nv ? 4u * i : 0u));
      v1[i] = at_byte<float>(base, p + (4 + i < nv ? 4u * (4 + i) : 0u));
      v0[i] = i < nv ? v0[i] : 0.f;
      v1[i] = 4 + i < nv ? v1[i] : 0.f;
    }
  }
}

// Squared norm of coordinates [0, count) of candidate s, piece blk of n_blocks, in a fixed order: a thread sums its
// strided elements in float64, lanes by xor-shuffle tree, waves in order.
__device__ void sumsq_piece(const ConvArgs& a, int s, int blk, double* red) {
  const int T = blockDim.x;
  const long long lo = a.aux_count * blk / a.aux_pieces, hi = a.aux_count * (blk + 1) / a.aux_pieces;
  const float* __restrict__ row = a.G + (long long)s * a.ldg;
  double t = 0.0;
  long long i = lo + threadIdx.x;
  for (; i + 7 * T < hi; i += 8 * T) {            // eight loads in flight
    float v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = row[i + q * T];
#pragma unroll
    for (int q = 0; q < 8; ++q) t += (double)v[q] * (double)v[q];
  }
  for (; i < hi; i += T) t += (double)row[i] * (double)row[i];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) t += __shfl_xor(t, off, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = t;
  __syncthreads();
  if (threadIdx.x == 0) {
    double sum = 0.0;
    for (int w = 0; w < T / 64; ++w) sum += red[w];
    a.aux_norm[(long long)s * a.aux_P + a.aux_p_off + blk] = sum;
  }
}

__device__ inline void store_split(unsigned char* o, unsigned piece_stride, const f32x4& v0, const f32x4& v1) {
  const Split8 p = split8(v0, v1);
  *reinterpret_cast<bf16x8*>(o) = p.h;
  *reinterpret_cast<bf16x8*>(o + piece_stride) = p.m;
  *reinterpret_cast<bf16x8*>(o + 2 * piece_stride) = p.l;
}
// Fragments of job `job` (channel tile, step of some layer) of source s, one wave: U and, for candidates of a layer with a
// second product, W - gamma U.
__device__ void pack_fragment(const ConvArgs& a, int s, int job) {
  int l = 0;
  while (l + 1 < a.pack_layers && job >= a.pack_layer[l + 1].first) ++l;
  const ConvPack& L = a.pack_layer[l];
  const int lane = threadIdx.x & 63, n = lane & 31, h = lane >> 5;
  const int ct = (job - L.first) / L.steps, i = (job - L.first) % L.steps;
  const int per_unit = L.groups == 2 ? 9 : 5, unit = i / per_unit, st = i - unit * per_unit;
  const int tap = L.groups == 2 ? st : 2 * st + h, c = unit * 8 * L.groups + (L.groups == 2 ? 8 * h : 0);
  const int f = ct * 32 + n;
  const int nv = tap < 9 && f < L.Cout ? L.Cin - c : 0;
  const float* __restrict__ P = (s == a.pack_x ? a.x : a.G + (long long)s * a.ldg) + L.w_off;
  const bool second = L.sets == 2 && s != a.pack_x;
  const unsigned off = 4u * (unsigned)((f * 9 + tap) * L.Cin + c);
  f32x4 u0, u1, w0, w1;
  if (L.Cin % 8 == 0) {
    load8<true>(P, off, nv, u0, u1);
    if (second) load8<true>(a.x + L.w_off, off, nv, w0, w1);
  } else {
    load8<false>(P, off, nv, u0, u1);
    if (second) load8<false>(a.x + L.w_off, off, nv, w0, w1);
  }
  unsigned char* o = a.pack + (long long)s * a.pack_stride + L.off + (long long)(ct * L.sets * L.steps + i) * kConvFragBytes + lane * 16;
  store_split(o, 1024, u0, u1);
  if (second) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      u0[e] = __builtin_fmaf(-a.gamma, u0[e], w0[e]);
      u1[e] = __builtin_fmaf(-a.gamma, u1[e], w1[e]);
    }
    store_split(o + (long long)L.steps * kConvFragBytes, 1024, u0, u1);
  }
}

// The pass at x through a narrow fully connected layer, next to the candidates' last convolution, which it does not depend on
// (a launch of the layer kernel behind it took 13 us, most of it latency; the step of 32-32-64-64 channels is 11 us shorter).  Eight
// outputs of one sample per workgroup: a thread sums its quads of columns in float32, lanes by xor-shuffle tree and waves in order in
// float64.  Against the launch of its own on 220 random models (64 to 9 M columns, 1 to 32 outputs, 1 to 128 samples): the step 1.13
// times as fast, two of them slower, with more than a million columns and few samples (conv_fc_rides).  With all
// outputs of a sample in one workgroup, which read up to 32 rows of the weights one after the other, 41 were slower, by up to 42 %
// (launch of its own -> one workgroup -> now, 32 outputs: 5000 columns 57 -> 65 -> 53 us, 123008 columns 322 -> 508 -> 290).
constexpr int kFcOutputs = 8;
inline __host__ __device__ int fc_groups(int N) { return (N + kFcOutputs - 1) / kFcOutputs; }
__device__ void fc_sample(const ConvArgs& a, int r, int n0, float* red) {
  const float* __restrict__ W = a.x + a.fc_w_off;
  const float* __restrict__ h = a.fc_h0 + tiled_index<false>(r, 0, a.fc_Kp);
  const int T = blockDim.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int quads = a.fc_K >> 2;
  f32x4 sum[kFcOutputs];
#pragma unroll
  for (int i = 0; i < kFcOutputs; ++i) sum[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 2
  for (int q = threadIdx.x; q < quads; q += T) {
    const f32x4 hv = *reinterpret_cast<const f32x4*>(h + operand_column(4 * q));
#pragma unroll
    for (int i = 0; i < kFcOutputs; ++i) {
      const f32x4 w = *reinterpret_cast<const f32x4_a4*>(W + (long long)(n0 + i < a.fc_N ? n0 + i : n0) * a.fc_K + 4 * q);
#pragma unroll
      for (int e = 0; e < 4; ++e) sum[i][e] = __builtin_fmaf(hv[e], w[e], sum[i][e]);
    }
  }
  const int k = 4 * quads + (int)threadIdx.x;        // up to three columns behind the quads
  const bool rest = k < a.fc_K;
  const float hr = rest ? h[operand_column(k)] : 0.f;
  double* sums = reinterpret_cast<double*>(red);
#pragma unroll
  for (int i = 0; i < kFcOutputs; ++i) {
    const int n = n0 + i < a.fc_N ? n0 + i : n0;
    double t = ((double)sum[i][0] + sum[i][1]) + ((double)sum[i][2] + sum[i][3]);
    if (rest) t += (double)hr * (double)W[(long long)n * a.fc_K + k];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) t += __shfl_xor(t, off, 64);
    if (lane == 0) sums[wave * kFcOutputs + i] = t;
  }
  __syncthreads();
  if (threadIdx.x < kFcOutputs && n0 + (int)threadIdx.x < a.fc_N) {
    const int n = n0 + (int)threadIdx.x;
    double t = a.fc_b_off >= 0 ? (double)a.x[a.fc_b_off + n] : 0.0;
    for (int w = 0; w < T / 64; ++w) t += (double)(1.f / kScaleH) * sums[w * kFcOutputs + threadIdx.x];
    a.fc_z0[(long long)r * a.fc_N + n] = (float)t;
  }
}
// The layer's weights in matrix-operand order (times kScaleW), columns beyond K zeros (rows beyond N only reach results that are discarded).
constexpr int kFcPieces = 4;   // 16-byte pieces a thread copies
__device__ void fc_weights(const ConvArgs& a, int block) {
  const long long pieces = (long long)a.fc_N * (a.fc_Kp >> 2);
#pragma unroll
  for (int i = 0; i < kFcPieces; ++i) {
    const long long at = ((long long)block * kFcPieces + i) * blockDim.x + threadIdx.x;
    if (at >= pieces) return;
    const int n = (int)(at / (a.fc_Kp >> 2)), k = 4 * (int)(at % (a.fc_Kp >> 2));
    const f32x4 v = load4_masked(a.x + a.fc_w_off + (long long)n * a.fc_K, k, a.fc_K, k < a.fc_K);
    *reinterpret_cast<f32x4*>(a.fc_wt + tiled_index<false>(n, k, a.fc_Kp)) = v * kScaleW;
  }
}

constexpr unsigned kNoPixel = 0xffffffffu;

// What a workgroup that owns NP consecutive output positions of a job needs of its input map, in rows of the map
// with a border of one zero pixel all around: sample smp's row iy is border row smp * (Hin + 2) + iy + 1.
template <int NP>
struct ConvTile {
  unsigned rows, r_first, v_first, Wv, Hv, plane;
  int pixels;
  __device__ inline ConvTile(const ConvArgs& a, const ConvJob& J, int pt) {
    const ConvLayer& L = J.L;
    rows = (unsigned)(a.n_r * L.Hout * L.Wout);
    Wv = (unsigned)L.Win + 2u;
    Hv = (unsigned)L.Hin + 2u;
    r_first = (unsigned)pt * NP;
    const unsigned r_last = (r_first + NP < rows ? r_first + NP : rows) - 1u;
    v_first = border_row(J, r_first);
    pixels = (int)((border_row(J, r_last) + 3u - v_first) * Wv);
    plane = (unsigned)(pixels | 1) * 16u;         // bytes of one (piece, group of eight channels) plane
  }
  // topmost border row position r reads
  __device__ inline unsigned border_row(const ConvJob& J, unsigned r) const {
    const unsigned orow = div_magic(r, J.magic_wout), smp = div_magic(orow, J.magic_hout);
    return smp * Hv + (orow - smp * (unsigned)J.L.Hout) * (unsigned)J.L.stride;
  }
  // byte offset inside a plane of the pixel that position r's first tap reads
  __device__ inline unsigned first_pixel(const ConvJob& J, unsigned r) const {
    const unsigned rc = r < rows ? r : rows - 1u;
    const unsigned ox = rc - div_magic(rc, J.magic_wout) * (unsigned)J.L.Wout;
    return ((border_row(J, rc) - v_first) * Wv + ox * (unsigned)J.L.stride) * 16u;
  }
  // position of the input map that border row `row` of the tile holds at column vx; behind the last one where it is border
  __device__ inline unsigned pixel_position(const ConvArgs& a, const ConvJob& J, unsigned row, unsigned vx) const {
    const ConvLayer& L = J.L;
    const unsigned v = v_first + row, smp = __umulhi(v, J.magic_hv), vy = v - smp * Hv;
    const bool inside = (vx - 1u < (unsigned)L.Win) & (vy - 1u < (unsigned)L.Hin) & (smp < (unsigned)a.n_r);
    const unsigned at = (smp * (unsigned)L.Hin + vy - 1u) * (unsigned)L.Win + (vx - 1u);
    return inside ? at : (unsigned)(a.n_r * L.Hin * L.Win);
  }
  // byte offset of border pixel px inside the input map, or kNoPixel where it is border
  __device__ inline unsigned pixel_offset(const ConvArgs& a, const ConvJob& J, unsigned px) const {
    const ConvLayer& L = J.L;
    const unsigned vr = div_magic(px, J.magic_wv), vx = px - vr * Wv, v = v_first + vr;
    const unsigned smp = div_magic(v, J.magic_hv), vy = v - smp * Hv;
    const bool inside = (vx - 1u < (unsigned)L.Win) & (vy - 1u < (unsigned)L.Hin) & (smp < (unsigned)a.n_r);
    return inside ? ((smp * (unsigned)L.Hin + vy - 1u) * (unsigned)L.Win + (vx - 1u)) * (unsigned)L.Cin * 4u : kNoPixel;
  }
};
// eight channels from c on of the pixel at byte offset off
template <bool FULL>
__device__ inline void load_pixel(const float* __restrict__ map, unsigned off, int c, int Cin, f32x4& v0, f32x4& v1) {
  load8<FULL>(map, off + 4u * (unsigned)c, off != kNoPixel ? Cin - c : 0, v0, v1);
}

// 64 lanes x 16 bytes, each lane's from its own address, to consecutive bytes of LDS from `to` (wave-uniform) on; no registers.
__device__ inline void copy_to_lds(const unsigned char* from, unsigned char* to) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)from,
                                   (__attribute__((address_space(3))) void*)to, 16, 0, 0);
}
__device__ inline Split8 load_split(const unsigned char* o, unsigned piece_stride) {
  Split8 p;
  p.h = *reinterpret_cast<const bf16x8*>(o);
  p.m = *reinterpret_cast<const bf16x8*>(o + piece_stride);
  p.l = *reinterpret_cast<const bf16x8*>(o + 2 * piece_stride);
  return p;
}

// Four consecutive channels fo .. fo + 3 (a multiple of four) of position r of a split map with C (a multiple of eight) channels.
__device__ inline void store_split_out(float* out, unsigned C, f32x4 v, unsigned r, unsigned rows, unsigned fo) {
  typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
  const unsigned groups = (C + 15u) / 16u * 2u, map_plane = (rows + 1u) * 16u;
  if (r >= rows || fo >= 8u * groups) return;
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  if (fo >= C) v = zero;
  const Split8 p = split8(v, zero);
  unsigned char* o = reinterpret_cast<unsigned char*>(out) + (unsigned long long)((fo >> 4) * 6u + ((fo >> 3) & 1u)) * map_plane +
                     r * 16u + (fo & 4u) * 2u;
  const unsigned long long piece = 2ull * map_plane;
  auto low = [](const bf16x8& x) { return __builtin_bit_cast(u32x2, __builtin_shufflevector(x, x, 0, 1, 2, 3)); };
  *reinterpret_cast<u32x2*>(o) = low(p.h);
  *reinterpret_cast<u32x2*>(o + piece) = low(p.m);
  *reinterpret_cast<u32x2*>(o + 2 * piece) = low(p.l);
  if (r + 1u == rows) {                           // the position of zeros behind the last one
    const u32x2 z = {0u, 0u};
#pragma unroll
    for (int i = 0; i < 3; ++i) *reinterpret_cast<u32x2*>(o + 16 + i * piece) = z;
  }
}

// What four consecutive channels fo .. fo + 3 of one position r need besides their sums, requested ahead of them.
struct ConvOut {
  f32x4 bias, z0;
};
__device__ inline ConvOut conv_out_request(const ConvArgs& a, const ConvJob& J, bool cand, const float* __restrict__ P, unsigned r,
                                           unsigned rows, unsigned fo) {
  const ConvLayer& L = J.L;
  const unsigned C = (unsigned)L.Cout, row = (r < rows ? r : rows - 1u) * C;
  ConvOut o;
  o.bias = o.z0 = f32x4{0.f, 0.f, 0.f, 0.f};
  if ((C & 3u) == 0u) {                           // the four channels exist together and lie 16-byte aligned
    const unsigned fc = fo < C ? fo : 0u;
    if (L.b_off >= 0) o.bias = at_byte<f32x4_a4>(P + L.b_off, 4u * fc);
    if (cand) o.z0 = at_byte<f32x4>(J.Z0, 4u * (row + fc));
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const unsigned fc = fo + i < C ? fo + i : 0u;
      if (L.b_off >= 0) o.bias[i] = at_byte<float>(P + L.b_off, 4u * fc);
      if (cand) o.z0[i] = at_byte<float>(J.Z0, 4u * (row + fc));
    }
  }
  return o;
}
// SPLIT: the output may be a split map.
template <bool SPLIT>
__device__ inline void conv_out_store(const ConvArgs& a, const ConvJob& J, bool cand, int s, const ConvOut& o, const f32x4& sum,
                                      unsigned r, unsigned rows, unsigned fo) {
  const unsigned C = (unsigned)J.L.Cout, row = r * C;
  f32x4 val, res;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    val[i] = sum[i] + o.bias[i];
    res[i] = conv_result(a, cand, val[i], o.z0[i]) * J.out_scale;
  }
  float* __restrict__ out = cand ? J.out + (long long)s * J.out_stride : J.out;
  if (SPLIT && J.split_out) {
    if (r < rows && fo < C && !cand) *reinterpret_cast<f32x4*>(J.Z0 + (row + fo)) = val;
    store_split_out(out, C, res, r, rows, fo);
    return;
  }
  if (r >= rows || fo >= C) return;
  unsigned smp = 0, k = row + fo;
  if (J.tiled_out) {                              // column of the fully connected layer's operand
    smp = div_magic(div_magic(r, J.magic_wout), J.magic_hout);
    k -= smp * (unsigned)(J.L.Hout * J.L.Wout) * C;
  }
  if ((C & 3u) == 0u) {
    if (!cand) *reinterpret_cast<f32x4*>(J.Z0 + (row + fo)) = val;
    *reinterpret_cast<f32x4*>(out + (J.tiled_out ? tiled_index<false>((int)smp, (int)k, J.Kp_fc) : (long long)k)) = res;
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (fo + i < C) {
        if (!cand) J.Z0[row + fo + i] = val[i];
        out[J.tiled_out ? tiled_index<false>((int)smp, (int)k + i, J.Kp_fc) : (long long)(k + i)] = res[i];
      }
  }
}

// TW = 3: three waves share one tile and take one kernel row (ky) each; their accumulators are added through
// LDS in the fixed order (0 + 1) + 2 and wave 0 finishes the tile.  Used when the launch has too few tiles
// to occupy the matrix cores otherwise (a wave's 9 c_in / 2 dependent matrix instructions set its pace).
// The first row of the grid is the pass at x, if the launch carries it.
template <int TW>
__global__ __launch_bounds__(64 * TW) void conv_layer_kernel(const ConvArgs a) {
  const bool cand = !a.has_base || blockIdx.y > 0;
  const ConvJob& J = cand ? a.cj : a.bj;
  const ConvLayer& L = J.L;
  const int lane = threadIdx.x & 63, n = lane & 31, h = lane >> 5;
  const int tw = TW > 1 ? __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) : 0;
  const int ftiles = (L.Cout + 31) / 32;
  const int ft = blockIdx.x % ftiles, rb = blockIdx.x / ftiles;
  const int s = (int)blockIdx.y - (a.has_base ? 1 : 0);
  const int K = 9 * L.Cin;
  const long long rows = (long long)a.n_r * L.Hout * L.Wout;
  if ((long long)rb * 32 >= rows) return;          // (the grid is as wide as the larger of two jobs)

  const float* __restrict__ P = cand ? a.G + (long long)s * a.ldg : a.x;
  const bool second = cand && J.D_in != nullptr;
  const float* __restrict__ Din = second ? J.D_in + (long long)s * J.D_in_stride : nullptr;

  // first operand: kernel row of output channel f, taps and channels contiguous
  const int f = ft * 32 + n;
  const bool f_ok = f < L.Cout;
  const float* __restrict__ Urow = P + L.w_off + (long long)(f_ok ? f : 0) * K;
  const float* __restrict__ Wrow = a.x + L.w_off + (long long)(f_ok ? f : 0) * K;
  // second operand: output position r = (sample, y, x)
  const long long r = (long long)rb * 32 + n;
  const bool r_ok = r < rows;
  const int hw = L.Hout * L.Wout;
  const int smp = (int)((r_ok ? r : 0) / hw), pos = (int)((r_ok ? r : 0) % hw);
  const int oy = pos / L.Wout, ox = pos % L.Wout;

  f32x16 acc;
#pragma unroll
  for (int j = 0; j < 16; ++j) acc[j] = 0.f;
  const float neg_gamma = -a.gamma;

  for (int tap = (TW > 1 ? 3 * tw : 0); tap < (TW > 1 ? 3 * tw + 3 : 9); ++tap) {
    const int ky = tap / 3, kx = tap % 3;
    const int iy = oy * L.stride + ky - 1, ix = ox * L.stride + kx - 1;
    const bool p_ok = r_ok && iy >= 0 && iy < L.Hin && ix >= 0 && ix < L.Win;
    const long long moff = (((long long)smp * L.Hin + (p_ok ? iy : 0)) * L.Win + (p_ok ? ix : 0)) * L.Cin;
    const float* __restrict__ hp = J.H0_in + moff;
    const float* __restrict__ dp = second ? Din + moff : nullptr;
    const float* __restrict__ up = Urow + tap * L.Cin;
    const float* __restrict__ wp = Wrow + tap * L.Cin;
    // channels two at a time: this lane's half h takes channel c0 + h
    int c0 = 0;
    // Eight channels at a time: each lane loads FOUR consecutive channels of its kernel row / its position with
    // one 128-bit load (half h takes channels c0 + 4h .. c0 + 4h + 3) and feeds four matrix instructions, the
    // i-th of which contracts the channel pair (c0 + i, c0 + 4 + i).  Two such groups are loaded ahead of
    // their instructions.  A wave walks its operands alone, so the loads in flight set its pace.
    auto group8 = [&](auto ng_c) __attribute__((always_inline)) {
      constexpr int NG = decltype(ng_c)::value;
      const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
      f32x4 u[NG], b1[NG], w[NG], b2[NG];
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        const int c = c0 + 8 * g + 4 * h;
        u[g] = f_ok ? *reinterpret_cast<const f32x4_a4*>(up + c) : zero;
        b1[g] = p_ok ? *reinterpret_cast<const f32x4_a4*>(hp + c) : zero;
        if (second) {
          w[g] = f_ok ? *reinterpret_cast<const f32x4_a4*>(wp + c) : zero;
          b2[g] = p_ok ? *reinterpret_cast<const f32x4_a4*>(dp + c) : zero;
        }
      }
#pragma unroll
      for (int g = 0; g < NG; ++g)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          acc = __builtin_amdgcn_mfma_f32_32x32x2f32(u[g][i], b1[g][i], acc, 0, 0, 0);
          if (second)
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__builtin_fmaf(neg_gamma, u[g][i], w[g][i]), b2[g][i], acc, 0, 0, 0);
        }
    };
    for (; c0 + 16 <= L.Cin; c0 += 16) group8(std::integral_constant<int, 2>{});
    for (; c0 + 8 <= L.Cin; c0 += 8) group8(std::integral_constant<int, 1>{});
    for (; c0 < L.Cin; c0 += 2) {
      const int c = c0 + h;
      const bool c_ok = c < L.Cin;
      const float u = (f_ok && c_ok) ? up[c] : 0.f;
      const float b1 = (p_ok && c_ok) ? hp[c] : 0.f;
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(u, b1, acc, 0, 0, 0);
      if (second) {
        const float w = (f_ok && c_ok) ? wp[c] : 0.f;
        const float b2 = (p_ok && c_ok) ? dp[c] : 0.f;
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__builtin_fmaf(neg_gamma, u, w), b2, acc, 0, 0, 0);
      }
    }
  }

  if (TW > 1) {
    __shared__ float red[2][16][64];
    if (tw > 0) {
#pragma unroll
      for (int j = 0; j < 16; ++j) red[tw - 1][j][lane] = acc[j];
    }
    __syncthreads();
    if (tw > 0) return;
#pragma unroll
    for (int j = 0; j < 16; ++j) acc[j] = (acc[j] + red[0][j][lane]) + red[1][j][lane];
  }
  // accumulator element j of lane (n, h): position r (this lane's), output channel ft*32 + 8 (j/4) + 4 h + j%4
  if (!r_ok) return;
  float* __restrict__ out = cand ? J.out + (long long)s * J.out_stride : J.out;
  if (J.split_out) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const unsigned fo = (unsigned)(ft * 32 + 8 * q + 4 * h);
      const f32x4 sum = {acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
      conv_out_store<true>(a, J, cand, s, conv_out_request(a, J, cand, P, (unsigned)r, (unsigned)rows, fo), sum, (unsigned)r, (unsigned)rows, fo);
    }
    return;
  }
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    const int fo = ft * 32 + 8 * (j >> 2) + 4 * h + (j & 3);
    if (fo >= L.Cout) continue;
    const float bias = L.b_off >= 0 ? P[L.b_off + fo] : 0.f;
    const float val = acc[j] + bias;
    float res;
    if (!cand) {
      J.Z0[r * L.Cout + fo] = val;
      res = relu_nan(val);
    } else {
      const float dz = -a.gamma * val;
      const float z0 = J.Z0[r * L.Cout + fo];
      const float hr = relu_nan(z0 + dz);
      // relu(z0 + dz) - relu(z0) without cancellation
      const float dd = (z0 > 0.f) ? ((dz < -z0) ? -z0 : dz) : hr;
      res = dd * a.neg_inv_gamma;
    }
    res *= J.out_scale;
    if (J.tiled_out) {
      out[tiled_index<false>(smp, pos * L.Cout + fo, J.Kp_fc)] = res;
    } else {
      out[r * L.Cout + fo] = res;
    }
  }
}

// Many tiles: four waves, 32 PB WP positions x 32 WC channels.  One (map, channel chunk) unit at a time: its map values and
// its kernel values are requested while the unit before is multiplied, split once and staged for all four waves.
// CG: groups of eight channels per unit.
template <int CG, bool FULL, int PB, int WP, int WC, bool SPLIT>
__device__ __forceinline__ void conv_wide(const ConvArgs& a, const ConvJob& J, bool cand, int s, int tile, unsigned char* lds) {
  static_assert(WP * WC == 4, "four waves");
  constexpr int THREADS = 256, NP = 32 * PB * WP;
  constexpr int STEPS = CG == 2 ? 9 : 5;                           // matrix steps of 16 k per unit (CG = 1: two taps each)
  constexpr int NI = 3;                                            // map items a thread requests ahead
  constexpr int KITEMS = 32 * WC * 9 * CG, NK = (KITEMS + THREADS - 1) / THREADS;   // kernel items: (channel, tap, group)
  constexpr unsigned KROW = (32 * WC + 1) * 16, KPIECE = 2 * STEPS * KROW;          // staged kernel: [piece][step, half][channel]
  const ConvLayer& L = J.L;
  const int tid = threadIdx.x, lane = tid & 63, n = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wc = wave % WC, wp = wave / WC;
  const int cgroups = (L.Cout + 32 * WC - 1) / (32 * WC);
  const int pt = tile / cgroups, f_base = (tile % cgroups) * 32 * WC;
  const float* __restrict__ P = cand ? a.G + (long long)s * a.ldg : a.x;
  const bool second = cand && J.D_in != nullptr;
  const float* __restrict__ Din = second ? J.D_in + (long long)s * J.D_in_stride : nullptr;
  const ConvTile<NP> T(a, J, pt);
  const unsigned plane = T.plane;
  unsigned char* klds = lds + 3 * CG * plane;
  const float neg_gamma = -a.gamma;

  unsigned pos_r[PB], pix[PB];
#pragma unroll
  for (int pb = 0; pb < PB; ++pb) {
    pos_r[pb] = T.r_first + (unsigned)((wp * PB + pb) * 32 + n);
    pix[pb] = T.first_pixel(J, pos_r[pb]);
  }
  // this thread's items of a unit: map values (pixel, group) and kernel values (channel, tap, group), groups fastest
  const int items = T.pixels * CG;
  unsigned m_off[NI];
#pragma unroll
  for (int q = 0; q < NI; ++q) {
    const int i = tid + q * THREADS;
    m_off[q] = i < items ? T.pixel_offset(a, J, (unsigned)i / CG) : kNoPixel;
  }
  const int g8 = CG == 2 ? 8 * (tid & 1) : 0;                      // first channel of this thread's group
  unsigned k_off[NK], k_at[NK];
#pragma unroll
  for (int q = 0; q < NK; ++q) {
    const unsigned t = (unsigned)(tid + q * THREADS) / CG, f = t / 9u, tap = t - 9u * f;
    k_off[q] = (((unsigned)f_base + f < (unsigned)L.Cout ? (unsigned)f_base + f : 0u) * 9u + tap) * (unsigned)L.Cin * 4u;
    k_at[q] = (CG == 2 ? 2u * tap + (tid & 1) : tap) * KROW + f * 16u;
  }
  if (CG == 1) {
    // the tenth tap of the last step: zeros
    for (int i = tid; i < 3 * 32 * WC; i += THREADS)
      *reinterpret_cast<f32x4*>(klds + (unsigned)(i / (32 * WC)) * KPIECE + 9 * KROW + (unsigned)(i % (32 * WC)) * 16u) = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  f32x16 lead[PB], rest[PB];
#pragma unroll
  for (int pb = 0; pb < PB; ++pb)
#pragma unroll
    for (int j = 0; j < 16; ++j) lead[pb][j] = rest[pb][j] = 0.f;

  const int chunks = (L.Cin + 8 * CG - 1) / (8 * CG), units = chunks * (second ? 2 : 1);
  auto stage_item = [&](int i, const f32x4 (&v)[2]) __attribute__((always_inline)) {
    store_split(lds + (CG == 2 ? (unsigned)(i & 1) * plane : 0u) + (unsigned)i / CG * 16u, CG * plane, v[0], v[1]);
  };
  const float* __restrict__ Pk = P + L.w_off;
  const float* __restrict__ Xk = a.x + L.w_off;
  // iteration u requests unit u, multiplies unit u - 1 meanwhile, and stages unit u
#pragma unroll 1
  for (int u = 0; u <= units; ++u) {
    const bool dmap = u >= chunks;
    const int ch = (u - (dmap ? chunks : 0)) * 8 * CG;
    const float* __restrict__ map = dmap ? Din : J.H0_in;
    f32x4 mv[NI][2], ku[NK][2], kv[NK][2];
    if (u < units) {
#pragma unroll
      for (int q = 0; q < NI; ++q) load_pixel<FULL>(map, m_off[q], ch + g8, L.Cin, mv[q][0], mv[q][1]);
#pragma unroll
      for (int q = 0; q < NK; ++q) {
        const int nv = KITEMS % THREADS == 0 || tid + q * THREADS < KITEMS ? L.Cin - ch - g8 : 0;
        load8<FULL>(Pk, k_off[q] + 4u * (unsigned)(ch + g8), nv, ku[q][0], ku[q][1]);
        if (dmap) load8<FULL>(Xk, k_off[q] + 4u * (unsigned)(ch + g8), nv, kv[q][0], kv[q][1]);
      }
    }
    if (u > 0) {
      const unsigned char* ka = klds + (unsigned)h * KROW + (unsigned)(wc * 32 + n) * 16u;
      // (not unrolled: a launch is short, and straight-line code costs it more instruction fetches than it saves)
#pragma unroll 1
      for (int st = 0; st < STEPS; ++st, ka += 2 * KROW) {
        const Split8 A = load_split(ka, KPIECE);
        const int tap = CG == 2 ? st : 2 * st + h, ky = (tap * 11) >> 5;
        const unsigned toff = (unsigned)(ky * (int)T.Wv + tap - 3 * ky) * 16u + (CG == 2 ? (unsigned)h * plane : 0u);
#pragma unroll
        for (int pb = 0; pb < PB; ++pb) {
          // (the tenth tap meets zero kernel values and reads pixel 0, which is border: 0 x inf would be NaN)
          const unsigned at = CG == 1 && tap > 8 ? 0u : toff + pix[pb];
          mfma_split(A, load_split(lds + at, CG * plane), lead[pb], rest[pb]);
        }
      }
      if (u == units) break;
      __syncthreads();                                             // everyone is done with unit u - 1
    }
#pragma unroll
    for (int q = 0; q < NI; ++q)
      if (tid + q * THREADS < items) stage_item(tid + q * THREADS, mv[q]);
#pragma unroll
    for (int q = 0; q < NK; ++q) {
      if (dmap) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          ku[q][0][e] = __builtin_fmaf(neg_gamma, ku[q][0][e], kv[q][0][e]);
          ku[q][1][e] = __builtin_fmaf(neg_gamma, ku[q][1][e], kv[q][1][e]);
        }
      }
      if (tid + q * THREADS < KITEMS) store_split(klds + k_at[q], KPIECE, ku[q][0], ku[q][1]);
    }
#pragma unroll 1
    for (int i = tid + NI * THREADS; i < items; i += THREADS) {    // tiles with more pixels than are requested ahead
      f32x4 v[2];
      load_pixel<FULL>(map, T.pixel_offset(a, J, (unsigned)i / CG), ch + g8, L.Cin, v[0], v[1]);
      stage_item(i, v);
    }
    __syncthreads();                                               // unit u is complete
  }
  // element j of lane (n, h) is position n of the block, channel 8 (j / 4) + 4 h + j % 4 of the tile
#pragma unroll
  for (int pb = 0; pb < PB; ++pb) {
    ConvOut o[4];
    const unsigned fo = (unsigned)(f_base + wc * 32 + 4 * h);
#pragma unroll
    for (int q = 0; q < 4; ++q) o[q] = conv_out_request(a, J, cand, P, pos_r[pb], T.rows, fo + 8u * q);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      f32x4 sum;
#pragma unroll
      for (int i = 0; i < 4; ++i) sum[i] = join_split(lead[pb][4 * q + i], rest[pb][4 * q + i]);
      conv_out_store<SPLIT>(a, J, cand, s, o[q], sum, pos_r[pb], T.rows, fo + 8u * q);
    }
  }
}

// Few tiles: 64 positions x 32 channels, eight waves that share out the matrix steps.  Up to stage_units units are staged at
// once; every wave requests the kernel values of all its steps of them before anything else.
template <int CG, bool FULL, bool SPLIT>
__device__ __forceinline__ void conv_deep(const ConvArgs& a, const ConvJob& J, bool cand, int s, int tile, unsigned char* lds) {
  constexpr int KW = 8, THREADS = 64 * KW, PB = 2, NP = 32 * PB;
  constexpr int STEPS = CG == 2 ? 9 : 5;
  constexpr int NA = (kDeepSteps + KW - 1) / KW;                   // steps of a wave per stage
  constexpr int NI = 2;
  const ConvLayer& L = J.L;
  const int tid = threadIdx.x, lane = tid & 63, n = lane & 31, h = lane >> 5;
  const int kw = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ctiles = (L.Cout + 31) / 32;
  const int pt = tile / ctiles, f0 = (tile % ctiles) * 32;
  const float* __restrict__ P = cand ? a.G + (long long)s * a.ldg : a.x;
  const bool second = cand && J.D_in != nullptr;
  const float* __restrict__ Din = second ? J.D_in + (long long)s * J.D_in_stride : nullptr;
  const float* __restrict__ Pk = P + L.w_off;
  const float* __restrict__ Xk = a.x + L.w_off;
  const ConvTile<NP> T(a, J, pt);
  const unsigned plane = T.plane;
  unsigned pix[PB];
#pragma unroll
  for (int pb = 0; pb < PB; ++pb) pix[pb] = T.first_pixel(J, T.r_first + (unsigned)(32 * pb + n));
  // the results this thread finishes at the end: wave kw takes quarter kw % 4 of block kw / 4
  const int opb = kw >> 2, oq = kw & 3;
  const unsigned r_out = T.r_first + (unsigned)(32 * opb + n), fo = (unsigned)(f0 + 8 * oq + 4 * h);
  const ConvOut o = conv_out_request(a, J, cand, P, r_out, T.rows, fo);
  const unsigned krow = (unsigned)(f0 + n < L.Cout ? f0 + n : 0) * 9u * (unsigned)L.Cin;
  const float neg_gamma = -a.gamma;

  f32x16 lead[PB], rest[PB];
#pragma unroll
  for (int pb = 0; pb < PB; ++pb)
#pragma unroll
    for (int j = 0; j < 16; ++j) lead[pb][j] = rest[pb][j] = 0.f;

  const int chunks = (L.Cin + 8 * CG - 1) / (8 * CG), units = chunks * (second ? 2 : 1);
  const unsigned unit_bytes = 3 * CG * plane;
  const unsigned per_unit = (unsigned)T.pixels * CG;
  const float inv_unit = 1.f / (float)per_unit;
#pragma unroll 1
  for (int u0 = 0; u0 < units; u0 += J.stage_units) {
    const int nu = units - u0 < J.stage_units ? units - u0 : J.stage_units;
    const int steps = nu * STEPS, items = nu * (int)per_unit;
    // channel and map of unit u of the stage
    auto unit_of = [&](int u, bool& dmap) {
      dmap = u0 + u >= chunks;
      return (u0 + u - (dmap ? chunks : 0)) * 8 * CG;
    };
    f32x4 ku[NA][2], kv[NA][2];
#pragma unroll
    for (int q = 0; q < NA; ++q) {
      const int i = kw + q * KW < steps ? kw + q * KW : steps - 1;  // (a step too many is not used)
      const int ul = i / STEPS, st = i - ul * STEPS;
      bool dmap;
      const int ch = unit_of(ul, dmap), tap = CG == 2 ? st : 2 * st + h, c = ch + (CG == 2 ? 8 * h : 0);
      const unsigned off = 4u * (krow + (unsigned)(tap * L.Cin + c));
      const int nv = tap < 9 ? L.Cin - c : 0;
      load8<FULL>(Pk, off, nv, ku[q][0], ku[q][1]);
      if (dmap) load8<FULL>(Xk, off, nv, kv[q][0], kv[q][1]);
    }
    if (u0 > 0) __syncthreads();                                   // everyone is done with the units before
#pragma unroll 1
    for (int i0 = tid; i0 < items; i0 += NI * THREADS) {
      f32x4 v[NI][2];
      unsigned at[NI];
#pragma unroll
      for (int q = 0; q < NI; ++q) {
        const int i = i0 + q * THREADS < items ? i0 + q * THREADS : items - 1;
        // (exact: i is below 2^21, and a quotient lies at least half an item from the next one's border)
        const unsigned u = (unsigned)(((float)i + 0.5f) * inv_unit), e = (unsigned)i - u * per_unit;
        bool dmap;
        const int ch = unit_of((int)u, dmap);
        const unsigned px = e / CG;
        at[q] = u * unit_bytes + (CG == 2 ? (e & 1) * plane : 0u) + px * 16u;
        const int c = ch + (CG == 2 ? 8 * (int)(e & 1) : 0);
        const unsigned off = T.pixel_offset(a, J, px);
        const float* map = dmap ? Din : J.H0_in;                   // (differs between lanes)
        load_pixel<FULL>(map, off, c, L.Cin, v[q][0], v[q][1]);
      }
#pragma unroll
      for (int q = 0; q < NI; ++q) store_split(lds + at[q], CG * plane, v[q][0], v[q][1]);
    }
    __syncthreads();                                               // the staged units are complete
#pragma unroll
    for (int q = 0; q < NA; ++q) {
      const int i = kw + q * KW;
      if (i < steps) {
        const int ul = i / STEPS, st = i - ul * STEPS;
        if (u0 + ul >= chunks) {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            ku[q][0][e] = __builtin_fmaf(neg_gamma, ku[q][0][e], kv[q][0][e]);
            ku[q][1][e] = __builtin_fmaf(neg_gamma, ku[q][1][e], kv[q][1][e]);
          }
        }
        const int tap = CG == 2 ? st : 2 * st + h, ky = (tap * 11) >> 5;
        // (a tenth tap meets zero kernel values and reads pixel 0, which is border: 0 x inf would be NaN)
        const unsigned toff = (unsigned)(ky * (int)T.Wv + tap - 3 * ky) * 16u + (CG == 2 ? (unsigned)h * plane : 0u);
        const Split8 A = split8(ku[q][0], ku[q][1]);
#pragma unroll
        for (int pb = 0; pb < PB; ++pb)
          mfma_split(A, load_split(lds + (unsigned)ul * unit_bytes + (CG == 1 && tap > 8 ? 0u : toff + pix[pb]), CG * plane),
                     lead[pb], rest[pb]);
      }
    }
  }
  // The waves' accumulators, added in wave order: quarter q of a block (registers 4q .. 4q + 3) is one 16-byte piece per lane.
  __syncthreads();                                                 // the staged units are no longer needed
  f32x4* red = reinterpret_cast<f32x4*>(lds);
#pragma unroll
  for (int pb = 0; pb < PB; ++pb)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      f32x4 v;
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = join_split(lead[pb][4 * q + i], rest[pb][4 * q + i]);
      red[((kw * PB + pb) * 4 + q) * 64 + lane] = v;
    }
  __syncthreads();
  f32x4 part[KW];
#pragma unroll
  for (int w = 0; w < KW; ++w) part[w] = red[((w * PB + opb) * 4 + oq) * 64 + lane];
#pragma unroll
  for (int w = 1; w < KW; ++w) part[0] += part[w];
  conv_out_store<SPLIT>(a, J, cand, s, o, part[0], r_out, T.rows, fo);
}

// The waves' accumulators of 64 positions x 32 channels, added in wave order; wave kw then finishes quarter kw % 4 of block kw / 4.
template <int KW, int PB>
__device__ __forceinline__ f32x4 sum_waves(const f32x16 (&lead)[PB], const f32x16 (&rest)[PB], unsigned char* lds, int kw, int lane) {
  // quarter q of a block (registers 4q .. 4q + 3) is one 16-byte piece per lane
  f32x4* red = reinterpret_cast<f32x4*>(lds);
#pragma unroll
  for (int pb = 0; pb < PB; ++pb)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      f32x4 v;
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = join_split(lead[pb][4 * q + i], rest[pb][4 * q + i]);
      red[((kw * PB + pb) * 4 + q) * 64 + lane] = v;
    }
  __syncthreads();
  f32x4 part[KW];
#pragma unroll
  for (int w = 0; w < KW; ++w) part[w] = red[((w * PB + (kw >> 2)) * 4 + (kw & 3)) * 64 + lane];
#pragma unroll
  for (int w = 1; w < KW; ++w) part[0] += part[w];
  return part[0];
}

// Kernel fragments and split maps from memory: 64 positions x 32 channels, eight waves that share out the matrix steps.
__device__ __forceinline__ void conv_packed(const ConvArgs& a, const ConvJob& J, bool cand, int s, int tile, unsigned char* lds) {
  constexpr int KW = 8, PB = 2, NP = 32 * PB, STEPS = 9, NA = 3;
  const ConvLayer& L = J.L;
  const int tid = threadIdx.x, lane = tid & 63, n = lane & 31, h = lane >> 5;
  const int kw = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ctiles = (L.Cout + 31) / 32;
  const int pt = (int)div_any((unsigned)tile, (unsigned)ctiles, J.magic_ctiles), ct = tile - pt * ctiles;
  const float* __restrict__ P = cand ? a.G + (long long)s * a.ldg : a.x;
  const bool second = cand && J.D_in != nullptr;
  const unsigned char* H0 = reinterpret_cast<const unsigned char*>(J.H0_in);
  const unsigned char* D = reinterpret_cast<const unsigned char*>(J.D_in) + (second ? (long long)s * J.D_in_stride * 4 : 0);
  const ConvTile<NP> T(a, J, pt);
  // With stride 2 a row of the staged map holds its even pixels first, then the odd ones, so that consecutive positions read
  // consecutive pieces.
  const unsigned Wv = T.Wv, even = L.stride == 2 ? (Wv + 1u) / 2u : Wv;
  const unsigned px_runs = ((unsigned)T.pixels + 63u) / 64u, plane = px_runs * 1024u, unit_bytes = 6u * plane;
  unsigned pix[PB];
#pragma unroll
  for (int pb = 0; pb < PB; ++pb) {
    const unsigned at = T.first_pixel(J, T.r_first + (unsigned)(32 * pb + n)) / 16u, row = div_magic(at, J.magic_wv);
    pix[pb] = (row * Wv + (at - row * Wv) / (unsigned)L.stride) * 16u;
  }
  const int chunks = (L.Cin + 15) / 16, units = chunks * (second ? 2 : 1);
  const unsigned positions = (unsigned)(a.n_r * L.Hin * L.Win), map_plane = (positions + 1u) * 16u;
  const unsigned char* __restrict__ frags = a.pack + (long long)(cand ? s : a.pack_x) * a.pack_stride + J.pack_off +
                                            (long long)ct * J.pack_sets * chunks * STEPS * kConvFragBytes + lane * 16;

  // offsets of the tile's pixels inside a plane of the map, once for all planes
  unsigned* offs = reinterpret_cast<unsigned*>(lds + J.offs_at);
  for (unsigned at = (unsigned)tid; at < px_runs * 64u; at += 64u * KW) {
    const unsigned row = __umulhi(at, J.magic_wv), k = at - row * Wv, odd = k >= even ? 1u : 0u;
    offs[at] = T.pixel_position(a, J, row, ((k - (odd ? even : 0u)) << (L.stride - 1)) + odd) * 16u;
  }
  f32x16 lead[PB], rest[PB];
#pragma unroll
  for (int pb = 0; pb < PB; ++pb)
#pragma unroll
    for (int j = 0; j < 16; ++j) lead[pb][j] = rest[pb][j] = 0.f;

#pragma unroll 1
  for (int u0 = 0; u0 < units; u0 += J.stage_units) {
    const int nu = units - u0 < J.stage_units ? units - u0 : J.stage_units;
    const int steps = nu * STEPS;
    const unsigned char* fr = frags + (long long)(u0 * STEPS + kw) * kConvFragBytes;
    __syncthreads();                                               // the offsets are there; everyone is done with the units before
    // copies of 64 pixels of one (unit, piece, group) plane each, the planes of a run of pixels one after the other
    const int planes = 6 * nu, copies = planes * (int)px_runs, of_x = 6 * (chunks - u0);   // planes from of_x on are the candidate's
    const unsigned char* from_x = H0 + (long long)(6 * u0) * map_plane;
    const unsigned char* from_cand = D + (long long)(6 * (u0 - chunks)) * map_plane;
    int run = 0, q = copies * kw / KW, left = copies * (kw + 1) / KW - q;
    while (q >= planes) {
      q -= planes;
      ++run;
    }
#pragma unroll 1
    while (left > 0) {
      const unsigned off = offs[run * 64 + lane];
      const int end = q + left < planes ? q + left : planes;
      left -= end - q;
#pragma unroll 2
      for (; q < end; ++q)
        copy_to_lds((q < of_x ? from_x : from_cand) + (unsigned long long)(unsigned)q * map_plane + off,
                    lds + (unsigned)q * plane + (unsigned)run * 1024u);
      q = 0;
      ++run;
    }
    // a wave's fragments three steps at a time, the first ones together with the copies
    Split8 A[NA];
    auto request = [&](int i0) __attribute__((always_inline)) {
#pragma unroll
      for (int j = 0; j < NA; ++j) A[j] = load_split(i0 + j * KW < steps ? fr + j * (KW * kConvFragBytes) : frags, 1024);
      fr += NA * KW * kConvFragBytes;
    };
    request(kw);
    __builtin_amdgcn_s_waitcnt(0x0f70);                            // vmcnt(0)
    __syncthreads();                                               // the staged units are complete
#pragma unroll 1
    for (int i0 = kw; i0 < steps; i0 += NA * KW) {
      if (i0 > kw) request(i0);
#pragma unroll
      for (int j = 0; j < NA; ++j) {
        const int i = i0 + j * KW;
        if (i < steps) {
          const int ul = i / STEPS, tap = i - ul * STEPS, ky = (tap * 11) >> 5, kx = tap - 3 * ky;
          const unsigned toff = (unsigned)(ky * (int)Wv) + (L.stride == 2 ? (kx == 1 ? even : (unsigned)kx >> 1) : (unsigned)kx);
          const unsigned char* m = lds + (unsigned)ul * unit_bytes + (unsigned)h * plane + toff * 16u;
#pragma unroll
          for (int pb = 0; pb < PB; ++pb) mfma_split(A[j], load_split(m + pix[pb], 2 * plane), lead[pb], rest[pb]);
        }
      }
    }
  }
  const unsigned r_out = T.r_first + (unsigned)(32 * (kw >> 2) + n), fo = (unsigned)(ct * 32 + 8 * (kw & 3) + 4 * h);
  const ConvOut o = conv_out_request(a, J, cand, P, r_out, T.rows, fo);
  __syncthreads();                                                 // the staged units are no longer needed
  const f32x4 sum = sum_waves<KW, PB>(lead, rest, lds, kw, lane);
  conv_out_store<true>(a, J, cand, s, o, sum, r_out, T.rows, fo);
}

// The candidates' first convolution, at most eight input channels, kernel fragments from memory: eight waves with 32 positions x
// 32 channels each, which all take every step.
__device__ __forceinline__ void conv_flat(const ConvArgs& a, const ConvJob& J, int s, int tile, unsigned char* lds) {
  constexpr int THREADS = 512, NP = 256, STEPS = 5;
  const ConvLayer& L = J.L;
  const int tid = threadIdx.x, lane = tid & 63, n = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ctiles = (L.Cout + 31) / 32;
  const int pt = (int)div_any((unsigned)tile, (unsigned)ctiles, J.magic_ctiles), ct = tile - pt * ctiles;
  const ConvTile<NP> T(a, J, pt);
  const unsigned plane = T.plane, r = T.r_first + (unsigned)(32 * wave + n), pix = T.first_pixel(J, r);
  const unsigned char* __restrict__ frags = a.pack + (long long)s * a.pack_stride + J.pack_off + (long long)ct * STEPS * kConvFragBytes + lane * 16;
#pragma unroll 1
  for (int i = tid; i < T.pixels; i += THREADS) {
    const unsigned off = T.pixel_offset(a, J, (unsigned)i);
    f32x4 v[2];
    if (L.Cin == 8) load_pixel<true>(J.H0_in, off, 0, 8, v[0], v[1]);   // (one by one: 2 us longer)
    else load_pixel<false>(J.H0_in, off, 0, L.Cin, v[0], v[1]);
    store_split(lds + (unsigned)i * 16u, plane, v[0], v[1]);
  }
  f32x16 lead, rest;
#pragma unroll
  for (int j = 0; j < 16; ++j) lead[j] = rest[j] = 0.f;
  Split8 A = load_split(frags, 1024);
  __syncthreads();
#pragma unroll 1
  for (int i = 0; i < STEPS; ++i) {
    const Split8 next = load_split(frags + (i + 1 < STEPS ? i + 1 : 0) * kConvFragBytes, 1024);
    const int tap = 2 * i + h, ky = (tap * 11) >> 5;
    const unsigned toff = (unsigned)(ky * (int)T.Wv + tap - 3 * ky) * 16u;
    // (the tenth tap meets zero kernel values and reads pixel 0, which is border: 0 x inf would be NaN)
    mfma_split(A, load_split(lds + (tap > 8 ? 0u : toff + pix), plane), lead, rest);
    A = next;
  }
  const float* __restrict__ P = a.G + (long long)s * a.ldg;
  const unsigned fo = (unsigned)(ct * 32 + 4 * h);
  ConvOut o[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) o[q] = conv_out_request(a, J, true, P, r, T.rows, fo + 8u * q);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    f32x4 sum;
#pragma unroll
    for (int i = 0; i < 4; ++i) sum[i] = join_split(lead[4 * q + i], rest[4 * q + i]);
    conv_out_store<true>(a, J, true, s, o[q], sum, r, T.rows, fo + 8u * q);
  }
}

// Blocks: [tiles of the pass at x] [tiles x candidates, candidate fastest] [squared norms: pieces x candidates] [one that
// clears the counters] [kernel fragments], or [samples of the fully connected layer x groups of its outputs] [its weights].  Returns
// whether the block is one of the small jobs, which it then has done.  EXTRA: the launch may have fragments to write, a fully connected
// layer or split maps; code for these costs other launches instruction fetches (wide tiles 62 -> 69 us, few tiles 9.8 -> 10.4).
template <bool EXTRA>
__device__ inline bool conv_block(const ConvArgs& a, unsigned char* lds, bool& is_base, int& s, int& tile) {
  int b = blockIdx.x;
  is_base = b < a.base_blocks;
  if (!is_base) b -= a.base_blocks;
  if (!is_base && b >= a.cand_blocks) {
    b -= a.cand_blocks;
    if (EXTRA && a.fc_N > 0) {                     // (a launch has these or the following)
      const int groups = fc_groups(a.fc_N);
      if (b < a.n_r * groups) fc_sample(a, b / groups, b % groups * kFcOutputs, reinterpret_cast<float*>(lds));
      else fc_weights(a, b - a.n_r * groups);
    } else if (b < a.aux_pieces * a.aux_m) {
      sumsq_piece(a, b / a.aux_pieces, b % a.aux_pieces, reinterpret_cast<double*>(lds));
    } else if (b == a.aux_pieces * a.aux_m) {
      const uint4 z = {0u, 0u, 0u, 0u};
      for (int i = threadIdx.x; i < a.aux_zero16; i += blockDim.x) reinterpret_cast<uint4*>(a.aux_zero)[i] = z;
    } else if (EXTRA) {
      const int waves = blockDim.x >> 6, job = (b - a.aux_pieces * a.aux_m - 1) * waves + (threadIdx.x >> 6);
      if (job < a.pack_jobs * (a.pack_x + 1)) pack_fragment(a, job / a.pack_jobs, job % a.pack_jobs);
    }
    return true;
  }
  // (blocks times candidates may exceed 2^32, and so may tiles times channel tiles)
  tile = is_base ? b : (int)div_any((unsigned)b, (unsigned)a.n_cand, a.magic_cand);
  s = is_base ? 0 : b - tile * a.n_cand;
  return false;
}

template <int CG, bool FULL, int PB, int WP, int WC, bool EXTRA>
__global__ __launch_bounds__(256, 2) void conv_wide_kernel(const ConvArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char conv_lds[];
  bool is_base;
  int s, tile;
  if (conv_block<EXTRA>(a, conv_lds, is_base, s, tile)) return;
  const ConvJob& J = is_base ? a.bj : a.cj;
  conv_wide<CG, FULL, PB, WP, WC, EXTRA>(a, J, !is_base, s, tile, conv_lds);
}

template <int CG, bool FULL, bool EXTRA>
__global__ __launch_bounds__(512, 2) void conv_deep_kernel(const ConvArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char conv_lds[];
  bool is_base;
  int s, tile;
  if (conv_block<EXTRA>(a, conv_lds, is_base, s, tile)) return;
  const ConvJob& J = is_base ? a.bj : a.cj;
  conv_deep<CG, FULL, EXTRA>(a, J, !is_base, s, tile, conv_lds);
}

__global__ __launch_bounds__(512, 4) void conv_packed_kernel(const ConvArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char conv_lds[];
  bool is_base;
  int s, tile;
  if (conv_block<true>(a, conv_lds, is_base, s, tile)) return;
  const ConvJob J = is_base ? a.bj : a.cj;
  if (J.flat) conv_flat(a, J, s, tile, conv_lds);
  else conv_packed(a, J, !is_base, s, tile, conv_lds);
}

// ---- host side
constexpr long long kConvLdsMost = 160 * 1024;
constexpr long long kConvLdsTwo = 80 * 1024;      // two workgroups per compute unit

// Most border rows that np consecutive positions touch.
long long most_border_rows(const ConvLayer& L, int np) {
  if (np % L.Wout == 0) {
    // tiles start at the beginning of a row: whole rows, and whole samples or parts of one where these numbers divide each other
    const long long n = np / L.Wout;
    if (L.Hout % n == 0) return (n - 1) * L.stride + 3;
    if (n % L.Hout == 0) return (n / L.Hout - 1) * (L.Hin + 2) + (long long)(L.Hout - 1) * L.stride + 3;
  }
  const long long out_rows = (np - 1 + L.Wout - 1) / L.Wout + 1;                 // output rows they can lie in
  const long long samples = (out_rows - 2 + L.Hout) / L.Hout;                    // sample boundaries among these
  const long long skip = (long long)L.Hin + 2 - (long long)L.Hout * L.stride;    // border rows beyond the stride at a boundary
  return (out_rows - 1) * L.stride + 3 + samples * (skip > 0 ? skip : 0);
}
// LDS bytes of the map values of one unit of `groups` groups of eight channels, upper bound for every tile of np positions.
long long map_bytes(const ConvLayer& L, int np, int groups) { return (most_border_rows(L, np) * (L.Win + 2) | 1) * 16 * 3 * groups; }
// ... of the kernel values (wide workgroups)
long long kernel_bytes(int wc, int groups) { return 3LL * 2 * (groups == 2 ? 9 : 5) * (32 * wc + 1) * 16; }

// The quick divisions want their products below 2^32, and so do the byte offsets inside one source's maps and kernels.
bool sizes_fit(const ConvLayer& L, int n_r, int np) {
  const long long rows = (long long)n_r * L.Hout * L.Wout, v = (long long)n_r * (L.Hin + 2) + 2, most = 1ll << 32;
  return rows < (1ll << 30) && rows * L.Wout < most && rows / L.Wout * L.Hout < most && v * (L.Hin + 2) < most &&
         most_border_rows(L, np) * (L.Win + 2) * (L.Win + 2) < most && most_border_rows(L, np) * (L.Win + 2) < (1ll << 18) &&
         4 * rows * L.Cout < most && 4ll * n_r * L.Hin * L.Win * L.Cin < most && 36ll * L.Cin * L.Cout < most;
}
// LDS bytes of a unit of a job with `groups` groups of eight channels.
long long wide_bytes(const ConvLayer& L, int np, int wc, int groups) { return map_bytes(L, np, groups) + kernel_bytes(wc, groups); }
long long deep_bytes(const ConvLayer& L, int groups) { return map_bytes(L, 64, groups); }
// LDS bytes of a unit of a split map (whole runs of 64 pixels)
long long split_unit_bytes(const ConvLayer& L) { return (most_border_rows(L, 64) * (L.Win + 2) + 63) / 64 * 1024 * 6; }
bool full_groups(const ConvLayer& L) { return L.Cin % 8 == 0; }

// What both kinds of launches prepare for each job; job_lds gives a job's LDS bytes and sets its groups and stage_units.
template <typename F>
hipError_t plan_tiles(ConvArgs& a, int np_most, int wc, F job_lds, long long* lds, long long* total) {
  long long blocks[2] = {0, 0};
  for (int q = 0; q < 2; ++q) {
    ConvJob& j = q == 0 ? a.bj : a.cj;
    if (q == 0 ? a.has_base == 0 : a.n_cand <= 0) continue;
    const ConvLayer& L = j.L;
    j.magic_wout = magic_for(L.Wout);
    j.magic_hout = magic_for(L.Hout);
    j.magic_wv = magic_for(L.Win + 2);
    j.magic_hv = magic_for(L.Hin + 2);
    j.magic_ctiles = magic_for((L.Cout + 31) / 32);
    const long long need = job_lds(j, q == 1 && j.D_in != nullptr ? 2 : 1);
    if (need > *lds) *lds = need;
    const int np = np_most > 0 ? np_most : j.flat ? 256 : 64;
    const long long rows = (long long)a.n_r * L.Hout * L.Wout;
    blocks[q] = (rows + np - 1) / np * ((L.Cout + 32 * wc - 1) / (32 * wc)) * (q == 1 ? a.n_cand : 1);
  }
  const int waves = wc > 0 && np_most == 128 ? 4 : 8;
  *total = blocks[0] + blocks[1] + (long long)a.aux_pieces * a.aux_m + (a.aux_zero16 > 0 ? 1 : 0) +
           ((long long)a.pack_jobs * (a.pack_x + 1) + waves - 1) / waves;
  if (a.fc_N > 0) *total += a.n_r * fc_groups(a.fc_N) + ((long long)a.fc_N * (a.fc_Kp / 4) + 64 * waves * kFcPieces - 1) / (64 * waves * kFcPieces);
  if (*total > kConvMostBlocks || *lds > kConvLdsMost) return hipErrorInvalidValue;
  a.base_blocks = (int)blocks[0];
  a.cand_blocks = (int)blocks[1];
  a.magic_cand = magic_for(a.n_cand);

  return hipSuccess;
}

// Whether a launch needs the kernels with everything in them.
bool has_extra(const ConvArgs& a) { return a.fc_N > 0 || a.pack_jobs > 0 || (a.has_base && a.bj.split_out) || (a.n_cand > 0 && a.cj.split_out); }

template <int CG, bool FULL, int PB, int WP, int WC, bool EXTRA>
hipError_t launch_wide(ConvArgs a, hipStream_t stream) {
  if (!EXTRA && has_extra(a)) return hipErrorInvalidValue;         // (not the instantiation for this launch)
  constexpr int NP = 32 * PB * WP;
  static const hipError_t attr_err = hipFuncSetAttribute(reinterpret_cast<const void*>(&conv_wide_kernel<CG, FULL, PB, WP, WC, EXTRA>),
                                                         hipFuncAttributeMaxDynamicSharedMemorySize, (int)kConvLdsMost);
  if (attr_err != hipSuccess) return attr_err;
  long long lds = 512, total = 0;                                  // (the small jobs' partial sums)
  const hipError_t e = plan_tiles(a, NP, WC, [](ConvJob& j, int) { return wide_bytes(j.L, NP, WC, CG); }, &lds, &total);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((conv_wide_kernel<CG, FULL, PB, WP, WC, EXTRA>), dim3((unsigned)total), dim3(256), (size_t)lds, stream, a);
  return hipGetLastError();
}

template <int CG, bool FULL, bool EXTRA>
hipError_t launch_deep(ConvArgs a, hipStream_t stream) {
  if (!EXTRA && has_extra(a)) return hipErrorInvalidValue;
  static const hipError_t attr_err = hipFuncSetAttribute(reinterpret_cast<const void*>(&conv_deep_kernel<CG, FULL, EXTRA>),
                                                         hipFuncAttributeMaxDynamicSharedMemorySize, (int)kConvLdsMost);
  if (attr_err != hipSuccess) return attr_err;
  long long lds = 8 * 8192, total = 0;                             // at least the accumulators of eight waves
  const hipError_t e = plan_tiles(a, 64, 1, [](ConvJob& j, int maps) {
    const int chunks = (j.L.Cin + 8 * CG - 1) / (8 * CG);
    const long long unit = deep_bytes(j.L, CG);
    long long n = kDeepSteps / (CG == 2 ? 9 : 5);
    if (n > kConvLdsMost / unit) n = kConvLdsMost / unit;
    j.stage_units = (int)(n > chunks * maps ? chunks * maps : n);
    return j.stage_units * unit;
  }, &lds, &total);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((conv_deep_kernel<CG, FULL, EXTRA>), dim3((unsigned)total), dim3(512), (size_t)lds, stream, a);
  return hipGetLastError();
}

// (channels that are no multiple of eight are staged up to one group of them only)
template <int PB, int WP, int WC, bool EXTRA>
hipError_t launch_wide_groups(int groups, bool full, const ConvArgs& a, hipStream_t stream) {
  if (groups == 2) return launch_wide<2, true, PB, WP, WC, EXTRA>(a, stream);
  return full ? launch_wide<1, true, PB, WP, WC, EXTRA>(a, stream) : launch_wide<1, false, PB, WP, WC, EXTRA>(a, stream);
}
template <bool EXTRA>
hipError_t launch_deep_groups(int groups, bool full, const ConvArgs& a, hipStream_t stream) {
  if (groups == 2) return launch_deep<2, true, EXTRA>(a, stream);
  return full ? launch_deep<1, true, EXTRA>(a, stream) : launch_deep<1, false, EXTRA>(a, stream);
}
template <int PB, int WP, int WC>
hipError_t launch_wide_as(int groups, bool full, const ConvArgs& a, hipStream_t stream) {
  return has_extra(a) ? launch_wide_groups<PB, WP, WC, true>(groups, full, a, stream) : launch_wide_groups<PB, WP, WC, false>(groups, full, a, stream);
}
hipError_t launch_deep_as(int groups, bool full, const ConvArgs& a, hipStream_t stream) {
  return has_extra(a) ? launch_deep_groups<true>(groups, full, a, stream) : launch_deep_groups<false>(groups, full, a, stream);
}

// More than eight channels that are no multiple of eight: the gathering kernel.  The staged tiles would read every channel by
// itself and test it (us per candidates' launch with the pass at x through the next layer, gathered / staged: 33 -> 33 on 16x16,
// stride 2, m = 39, n_r = 4: 30 / 56; on 14x14, m = 20, n_r = 32: 73 / 129; 20 -> 20 on 28x28, stride 1, m = 30, n_r = 48:
// 476 / 514; only the same with stride 2 is the other way round: 193 / 162).
bool few_channels(const ConvLayer& L) { return (L.Cin <= 2 && L.Cout <= 16) || (L.Cin <= 4 && L.Cout <= 8); }
bool gathered(const ConvLayer& L) { return !full_groups(L) && L.Cin > 8; }

// Tiles of 128 positions where they give every compute unit two workgroups or more.
bool wide_tiles(const ConvLayer& L, int n_r, int sources) {
  const long long rows = (long long)n_r * L.Hout * L.Wout;
  const int ctiles = (L.Cout + 31) / 32, wc = ctiles == 1 ? 1 : 2;
  return (rows + 127) / 128 * ((ctiles + wc - 1) / wc) * sources >= 512;
}

hipError_t launch_packed(ConvArgs a, hipStream_t stream) {
  static const hipError_t attr_err = hipFuncSetAttribute(reinterpret_cast<const void*>(&conv_packed_kernel),
                                                         hipFuncAttributeMaxDynamicSharedMemorySize, (int)kConvLdsTwo);
  if (attr_err != hipSuccess) return attr_err;
  long long lds = 8 * 8192, total = 0;                             // at least the accumulators of eight waves
  const hipError_t e = plan_tiles(a, 0, 1, [](ConvJob& j, int maps) {
    j.flat = j.L.Cin <= 8;
    if (j.flat) return map_bytes(j.L, 256, 1);
    const int chunks = (j.L.Cin + 15) / 16;
    const long long unit = split_unit_bytes(j.L);
    long long n = (kConvLdsTwo - unit / 24) / unit;
    j.stage_units = (int)(n > chunks * maps ? chunks * maps : n);
    const long long staged = j.stage_units * unit;
    j.offs_at = (int)(staged > 8 * 8192 ? staged : 8 * 8192);
    return j.offs_at + unit / 24;
  }, &lds, &total);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(conv_packed_kernel, dim3((unsigned)total), dim3(512), (size_t)lds, stream, a);
  return hipGetLastError();
}

hipError_t launch_gather(const ConvArgs& a, hipStream_t stream) {
  long long blocks = 0, tiles = 0;                 // of the wider job, of all sources
  for (const ConvJob* j : {&a.bj, &a.cj}) {
    const int sources = j == &a.bj ? (a.has_base ? 1 : 0) : a.n_cand;
    if (sources <= 0) continue;
    const long long rows = (long long)a.n_r * j->L.Hout * j->L.Wout;
    const long long n = (rows + 31) / 32 * ((j->L.Cout + 31) / 32);
    if (n > blocks) blocks = n;
    tiles += n * sources;
  }
  if (tiles == 0) return hipSuccess;
  const dim3 grid((unsigned)blocks, (a.has_base ? 1 : 0) + a.n_cand);
  // one wave per tile when there are tiles enough for every SIMD of the chip twice over, else three
  if (tiles >= 2048) hipLaunchKernelGGL(conv_layer_kernel<1>, grid, dim3(64), 0, stream, a);
  else hipLaunchKernelGGL(conv_layer_kernel<3>, grid, dim3(192), 0, stream, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_conv(const ConvArgs& a, hipStream_t stream) {
  if (a.pack != nullptr && a.pack_jobs == 0) return launch_packed(a, stream);
  // the job that dominates the launch decides its shape
  const ConvLayer& L = a.n_cand > 0 ? a.cj.L : a.bj.L;
  const int sources = a.n_cand > 0 ? a.n_cand : 1;
  const long long rows = (long long)a.n_r * L.Hout * L.Wout;
  const int ctiles = (L.Cout + 31) / 32;
  const bool full = full_groups(L);
  // groups of eight channels per unit: two, or one where the input has no more channels or where that makes room for two
  // workgroups per compute unit (stride 2, where a position has four pixels of its own); 0: neither fits
  auto pick_groups = [&](auto bytes, int np) {
    long long need[3] = {0, 0, 0};
    for (const ConvJob* j : {&a.cj, &a.bj}) {
      if (j == &a.cj ? a.n_cand <= 0 : !a.has_base) continue;
      if (!sizes_fit(j->L, a.n_r, np)) return 0;
      for (int g = 1; g <= 2; ++g)
        if (bytes(j->L, g) > need[g]) need[g] = bytes(j->L, g);
    }
    if (L.Cin > 8 && need[2] <= kConvLdsTwo) return 2;
    return need[1] <= kConvLdsMost ? 1 : 0;
  };
  const int wc = ctiles == 1 ? 1 : 2;
  const bool wide = wide_tiles(L, a.n_r, sources);
  // Channels that are no multiple of eight: the gathering kernel, but for wide tiles of one group of them (before those give every
  // compute unit two workgroups, gathered / staged with the pass at x through the next layer: 1 -> 33 on 32x32, stride 2, m = 39,
  // n_r = 4: 26 / 43 us; 3 -> 64 on 8x8, stride 2, m = 10, n_r = 2: 16 / 24; from there on 3 -> 32 on 32x32, m = 20: n_r = 4 25 / 23,
  // n_r = 32 136 / 68).
  // Neither where input and output channels are so few that a wide tile's products are mostly padding (time as wide tiles / gathered,
  // whole steps: up to 2 -> 16 or 4 -> 8 channels 1.04 on 21 random models, 19 of them slower as wide tiles, by up to 20 %; the
  // others 0.89 on 135).  The pass at x alone is staged up to 512 tiles of 64 positions x 32 channels, the small jobs of its launch
  // need as long (staged / gathered: 0.97 below 256 tiles, 1.01 on 38 up to 512, 1.02 on 32 beyond, 22 of them slower; measured
  // without fragments among the small jobs).
  const bool gather = gathered(L) || (!full && (a.n_cand > 0 ? !wide || few_channels(L) : (rows + 63) / 64 * ctiles >= 512));
  if (a.n_cand > 0 && a.has_base && !gather && (wide || gathered(a.bj.L) || (full && !full_groups(a.bj.L)))) {
    // The pass at x on its own: next to wide tiles its few workgroups, each with all of K to walk, would be the last ones to end
    // by far (n_r = 32, convolution 3 behind the candidates' convolution 2: 148 us together, 103 + 11 us apart); and one
    // staging kernel runs both jobs, so the channels of either have to be whole groups if the candidates' are.
    ConvArgs b = a, c = a;
    b.n_cand = 0;
    c.has_base = c.aux_m = c.aux_pieces = c.aux_zero16 = c.pack_jobs = 0;
    const hipError_t e = launch_conv(b, stream);
    return e != hipSuccess ? e : launch_conv(c, stream);
  }
  if (wide && !gather) {
    const int g = pick_groups([&](const ConvLayer& l, int gr) { return wide_bytes(l, 128, wc, gr); }, 128);
    if (g > 0) return wc == 1 ? launch_wide_as<1, 4, 1>(g, full, a, stream) : launch_wide_as<2, 2, 2>(g, full, a, stream);
  }
  const int g = pick_groups([&](const ConvLayer& l, int gr) { return deep_bytes(l, gr); }, 64);
  if (g > 0 && !gather) return launch_deep_as(g, full, a, stream);
  ConvArgs r = a;
  r.aux_pieces = r.aux_m = r.aux_zero16 = r.pack_jobs = r.fc_N = 0;
  const hipError_t e = launch_gather(r, stream);
  if (e != hipSuccess || (a.aux_m <= 0 && a.aux_zero16 <= 0 && a.pack_jobs <= 0 && a.fc_N <= 0)) return e;
  r = a;                                           // the small jobs alone
  r.has_base = r.n_cand = 0;
  return launch_wide_as<1, 4, 1>(1, true, r, stream);
}

bool conv_takes_fragments(const ConvLayer& L, int n_r, int index) {
  if (index == 0) return L.Cin <= 8 && !few_channels(L) && sizes_fit(L, n_r, 256) && map_bytes(L, 256, 1) <= kConvLdsTwo;
  return L.Cin > 8 && full_groups(L) && sizes_fit(L, n_r, 64) && split_unit_bytes(L) / 24 * 25 <= kConvLdsTwo;
}

// Fragments cost their launch 0.32 us per MB.  Where the kernels without them take large tiles (128 positions), the copies for 64
// positions cost more than they save, unless many input channels share them: per million positions x channel tiles 77 + 30 (one
// channel tile) + 30 (the last group of eight alone) - 40 us per sixteen channels with stride 1, 175 + 120 (the same) - 80 with
// stride 2; 15 us are saved where the pass at x had a launch of its own.  Few tiles gain: 1.6 us per sixteen channels and round of two
// workgroups per compute unit (0.2 where a position has so many pixels of its own that a stage holds one unit), and 60 per round
// after the first.  Fitted to 1539 random models of one to five convolutions (5 to 230 pixels wide, 16 to 256 channels, 1 to 128
// samples, 1 to 80 candidates), with fragments always / where this is negative: 1.14 times as fast as without in either case; slower
// than without by more than 3 % 87 / 26 of them, the slowest 0.72 / 0.89.
double conv_fragments_cost(const ConvLayer* layers, int n, int n_r, int m) {
  double us = 0.0, mb = 0.0;
  for (int l = 0; l < n; ++l) {
    const ConvLayer& L = layers[l];
    const double rows = (double)n_r * L.Hout * L.Wout, ctiles = (L.Cout + 31) / 32, units = (L.Cin + 15) / 16;
    const double millions = 1e-6 * m * rows * ctiles;
    mb += 1e-6 * (m + 1.0) * ctiles * conv_steps(L.Cin) * (l > 0 ? 2 : 1) * kConvFragBytes;
    const bool wide = wide_tiles(L, n_r, m);
    if (l == 0) {
      us -= 25.0 * millions + (!wide && L.Cin < 8 ? 1.0 : 0.0);   // (gathered without)
    } else if (wide) {
      const bool half = L.Cin % 16 != 0;
      us += millions * (L.stride == 1 ? 77.0 + (ctiles == 1 ? 30.0 : 0.0) + (half ? 30.0 : 0.0) - 40.0 * units
                                      : 175.0 + (half ? 120.0 : 0.0) - 80.0 * units);
      if (l + 1 < n) us -= 15.0;
    } else {
      const double tiles = m * std::ceil(rows / 64.0) * ctiles, rounds = tiles > 512.0 ? tiles / 512.0 : 1.0;
      us -= 60.0 * (rounds - 1.0) + rounds * units * (split_unit_bytes(L) <= 6 * 6144 ? 1.6 : 0.2);
    }
  }
  return us + 0.32 * mb;
}

hipError_t launch_fill_zero(void* p, size_t bytes, hipStream_t stream) {
  const long long n16 = (long long)(bytes / 16);   // the slots are multiples of 256 bytes
  if (n16 == 0) return hipSuccess;
  const long long want = (n16 + 255) / 256;
  hipLaunchKernelGGL(fill_zero_kernel, dim3((unsigned)(want > 4096 ? 4096 : want)), dim3(256), 0, stream,
                     reinterpret_cast<uint4*>(p), n16);
  return hipGetLastError();
}

}  // namespace zeno
