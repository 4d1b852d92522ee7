// The first launch of a model of several layers whose first layer has at most 1024 inputs, for up to 32 samples: the batch in
// matrix-operand order, and the pass at x through layer 0, which on its own would have to wait for it.
//
// Two launches cost 4-5 us each whatever they do.  Here every workgroup (a tile of 32 features) reads the rows of the batch as they
// are, straight into the registers that feed the matrix cores, and the workgroups share out the writing of the operand-order copy
// that the candidates' launches read.  The waves of a workgroup (four, eight or sixteen) take a chunk of 64 columns each and add their
// accumulators through LDS; there is no split over workgroups, whose arrival counters this launch clears.
// Bound by latency: the launch, one round trip for the loads, the reduction, the epilogue.  Measured (us, two launches / this one;
// n_r = 32): 1000 -> 700 17.9 / 13.8 (bf16 15.8 / 12.6), 784 -> 256 18.9 / 13.5, 500 -> 2000 16.5 / 11.2, 200 -> 300 11.3 / 9.7, 1024 -> 64
// line-aligned 10.7 / 7.5.  With two and four row blocks a wave's rows of the batch took so many registers and round trips that it lost
// (64 samples 17.3 / 14.5, 128 in bf16 27 / 36); beyond 16 chunks the K slices of the general path are worth more than the launch.
#include "zeno_layer_impl.h"

namespace zeno {

namespace {

constexpr int kFirstChunks = 16, kFirstRows = 32;

// WAVES: at least the chunks of K
template <bool BF16, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void first_layer_kernel(const FirstArgs a) {
  using T = Tr<BF16>;
  constexpr int STAGE_BYTES = 32 * 64 * T::ESIZE;
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  const int tid = threadIdx.x, lane = tid & 63, n = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  {
    const long long at = (long long)blockIdx.x * blockDim.x + tid, step = (long long)gridDim.x * blockDim.x;
    for (long long i = at; i < a.n_counters; i += step) a.counters[i] = 0u;
    for (long long i = at; i < a.n_zero; i += step) a.zero[i] = 0.0;
  }
  const LayerJob& J = a.job;
  const int N = J.N, K = J.K, n_chunks = J.Kp >> 6, n_tiles = (cover_rows(N, 0) + 31) / 32;
  const int nt = blockIdx.x;
  const int row0 = nt * 32;
  const float* __restrict__ U = a.x + J.w_off + (long long)row0 * K;
  unsigned char* st = lds + wave * STAGE_BYTES;
  float bias_lane = 0.f;
  if (J.b_off >= 0 && lane < 32 && row0 + lane < N) bias_lane = a.x[J.b_off + row0 + lane];

  f32x16 acc;
#pragma unroll
  for (int j = 0; j < 16; ++j) acc[j] = 0.f;
  const int c = wave;
  if (c < n_chunks) {
    f32x4 u[8], f[8];
    load_tile<0, false>(u, U + (c << 6), 0u, row0, c << 6, N, K, lane);
    // the lane's part of operand block i (8 columns; bf16: half a block of 16) of its sample; samples beyond the batch read the last
    // one and are zeroed
    const bool full = (c << 6) + 64 <= K;   // uniform
    const float* row = a.features + (long long)(n < a.n_r ? n : a.n_r - 1) * K;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int k = (c << 6) + (BF16 ? 16 * (i >> 1) + 8 * h + 4 * (i & 1) : 8 * i + 4 * h);
      if (full) f[i] = *reinterpret_cast<const f32x4_a4*>(row + k);
      else f[i] = load4_masked(row, k, K, true);
    }
    stage_tile<BF16>(u, st, lane);
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float v = n < a.n_r ? f[i][e] : 0.f;
        f[i][e] = BF16 ? v : v * kScaleH;
      }
    const bool copy = c % n_tiles == nt;    // this workgroup writes the chunk's operand-order copy
#pragma unroll
    for (int t = 0; t < (BF16 ? 4 : 8); ++t) {
      f32x4 op;
      if constexpr (BF16) {
        const f32x4 b = *reinterpret_cast<const f32x4*>(st + n * 128 + ((((2 * t + h) ^ (n >> 1)) & 7) << 4));
        bf16x8 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          o[e] = (__bf16)f[2 * t][e];
          o[4 + e] = (__bf16)f[2 * t + 1][e];
        }
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, b), o, acc, 0, 0, 0);
        op = __builtin_bit_cast(f32x4, o);
      } else {
        const f32x4 b = *reinterpret_cast<const f32x4*>(st + n * 256 + ((((2 * t + h) ^ n) & 15) << 4));
        op = f[t];
#pragma unroll
        for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(b[e], op[e], acc, 0, 0, 0);
      }
      if (copy)
        *reinterpret_cast<f32x4*>(reinterpret_cast<unsigned char*>(a.tiled) + ((long long)c * (BF16 ? 4 : 8) + t) * 1024 + lane * 16) = op;
    }
  }
  // the waves' accumulators in a fixed tree: wave w takes wave w + WAVES / 2's first, wave 1's last
  float* red = reinterpret_cast<float*>(lds);
  for (int step = WAVES / 2; step >= 1; step >>= 1) {
    __syncthreads();
    if (wave >= step && wave < 2 * step) {
#pragma unroll
      for (int j = 0; j < 16; ++j) red[((wave - step) * 16 + j) * 64 + lane] = acc[j];
    }
    __syncthreads();
    if (wave < step) {
#pragma unroll
      for (int j = 0; j < 16; ++j) acc[j] += red[(wave * 16 + j) * 64 + lane];
    }
  }
  if (wave != 0) return;
  // lane (n, h) holds sample n and features row0 + 8 q + 4 h + i
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int f0 = row0 + 8 * q + 4 * h;
    f32x4 val, hv;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float bias = __shfl(bias_lane, 8 * q + 4 * h + i, 64);
      val[i] = BF16 ? acc[4 * q + i] + bias : __builtin_fmaf(acc[4 * q + i], 1.f / kScaleH, bias);
      hv[i] = (n < a.n_r && f0 + i < N) ? relu_nan(val[i]) * (BF16 ? 1.f : kScaleH) : 0.f;
    }
    if (n < a.n_r) store4_masked(J.Z0 + (long long)n * N, f0, N, val);
    if (f0 < J.Np) store_tiled4<BF16>(J.H_base, n, f0, J.Np, hv);
  }
}

template <bool BF16, int WAVES>
hipError_t launch_first_inst(const FirstArgs& a, hipStream_t stream, LaunchShape* shape) {
  *shape = {1, WAVES, 1, 0, 1};
  constexpr int staging = WAVES * 32 * 64 * Tr<BF16>::ESIZE, reduction = WAVES / 2 * 16 * 64 * 4;
  constexpr int lds_bytes = staging > reduction ? staging : reduction;
  static const hipError_t attr_err =
      lds_bytes > 48 * 1024 ? hipFuncSetAttribute(reinterpret_cast<const void*>(&first_layer_kernel<BF16, WAVES>),
                                                  hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes)
                            : hipSuccess;
  if (attr_err != hipSuccess) return attr_err;
  const int tiles = (cover_rows(a.job.N, 0) + 31) / 32;
  hipLaunchKernelGGL((first_layer_kernel<BF16, WAVES>), dim3(tiles), dim3(64 * WAVES), lds_bytes, stream, a);
  return hipGetLastError();
}
template <bool BF16>
hipError_t launch_first(const FirstArgs& a, hipStream_t stream, LaunchShape* shape) {
  const int chunks = a.job.Kp >> 6;
  if (chunks <= 4) return launch_first_inst<BF16, 4>(a, stream, shape);
  if (chunks <= 8) return launch_first_inst<BF16, 8>(a, stream, shape);
  return launch_first_inst<BF16, 16>(a, stream, shape);
}

}  // namespace

bool first_layer_fits(int K, int n_r) { return K <= 64 * kFirstChunks && n_r <= kFirstRows; }

hipError_t launch_first_layer(const FirstArgs& a, bool bf16, hipStream_t stream, LaunchShape* shape) {
  if (!first_layer_fits(a.job.K, a.n_r) || a.job.last) return hipErrorInvalidValue;
  return bf16 ? launch_first<true>(a, stream, shape) : launch_first<false>(a, stream, shape);
}

}  // namespace zeno
