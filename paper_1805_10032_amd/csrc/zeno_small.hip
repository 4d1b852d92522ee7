// Stochastic Descendant Score (Definition 2) of small models in one launch: one workgroup per candidate.
//
// For a model of a few thousand parameters the launch sequence of the general path (pack the batch, the layers of the
// pass at x and of the candidates, loss, combine) costs 4-5 us per launch and does next to nothing in each.  Here the
// eight waves of a workgroup take one candidate through all layers: the pass at x is recomputed by every workgroup
// (it reads the same few KB from the caches), activations stay in LDS, and the loss differences, ||u||^2 and the
// score are formed at the end.  The arithmetic is the general path's (same change form, see zeno_layer_impl.h):
//     Z0 = H0 W^T + b,   dZ = -gamma ( H0 U^T + D (W - gamma U)^T + ub ),
// in fp32 on v_mfma_f32_32x32x2_f32, weights as the first operand; with the bf16 forward every operand is rounded to bf16
// where the general path rounds it, and products of two bf16 values are exact in fp32.
//
// A layer has at most four 32-feature tiles (widths after the input up to 128); each is shared by KP = 8 / 4 / 2 waves
// (1 / 2 / 3-4 tiles) that split K and add their accumulators through LDS in wave order.  A lane holds four consecutive k of
// its feature (weights) or its sample (activations) per step of 8 k and feeds four instructions, the i-th of which contracts
// k = i and 4 + i of the step; a step is requested one ahead of its products.
// Bound by latency: a dependent chain of round trips per layer, and instructions fetched as they are first run.  Measured (MI355X, wall time of score and update in a series
// of calls, m = 20, n_r = 32, float32; general path -> this one, four steps at a time -> one): 784 -> 10: 30.1 -> 25.9 -> 23.5 us,
// 784 -> 64 -> 10: 72.0 -> 43.1 -> 35.0; m = 40, n_r = 16: 256 -> 100 -> 50 -> 10: 47.8 -> 39.6; m = 8, n_r = 16: 64 -> 1: 28.8 -> 19.9.
#include <type_traits>

#include "zeno_layer_impl.h"

namespace zeno {

namespace {

constexpr int kWaves = 8, kThreads = 64 * kWaves;
constexpr int kMaxWidth = 128;   // widest layer output (four tiles)
constexpr int kRows = 32;        // samples
constexpr int kMaxClasses = 16;  // widest output layer: the threads of a workgroup take a class of a sample each
static_assert(kThreads == kRows * kMaxClasses, "one thread per sample and class");

template <bool BF16>
__device__ inline float operand(float v) {
  return BF16 ? (float)(__bf16)v : v;
}
template <bool BF16>
__device__ inline f32x4 operand(const f32x4& v) {
  f32x4 r;
#pragma unroll
  for (int i = 0; i < 4; ++i) r[i] = operand<BF16>(v[i]);
  return r;
}
// Four consecutive floats of a row of K >= 4 from k on, k < K + 8: requested from inside the row without a branch (paths that
// meet behind loads would wait for them), moved into place and zero-filled beyond the row's end when they are used.
__device__ inline f32x4 load_row4(const float* __restrict__ row, int k, int K) {
  return *reinterpret_cast<const f32x4_a4*>(row + (k < K - 4 ? k : K - 4));
}
__device__ inline f32x4 end_of_row4(const f32x4& v, int k, int K) {
  const int by = k - (k < K - 4 ? k : K - 4);
  f32x4 r;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    r[i] = 0.f;
#pragma unroll
    for (int j = i; j < 4; ++j) r[i] = by == j - i ? v[j] : r[i];
  }
  return r;
}
__device__ inline double sum_over(double v, int lanes) {
  for (int off = lanes / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}
__device__ inline double max_over(double v, int lanes) {
  for (int off = lanes / 2; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off, 64));
  return v;
}

template <bool BF16>
__global__ __launch_bounds__(kThreads) void score_small_kernel(const SmallArgs a) {
  extern __shared__ __attribute__((aligned(16))) float small_lds[];
  const int tid = threadIdx.x, lane = tid & 63, n = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int pitch = a.pitch;
  const float* __restrict__ P = a.G + (long long)blockIdx.x * a.ldg;
  // [activations of the pass at x, changes] x two layers in turn, each [32 samples][pitch], and the accumulators of the waves
  float* act[2] = {small_lds, small_lds + 2 * kRows * pitch};
  f32x4* red = reinterpret_cast<f32x4*>(small_lds + 4 * kRows * pitch);
  __shared__ double totals[2][kWaves];
  __shared__ int label[kRows];
  __shared__ float target[kRows];
  // requested now, stored behind the first layer's products (a wave would wait for them here)
  int label_mine = 0;
  float target_mine = 0.f;
  if (tid < a.n_r) {
    if (a.loss == ZENO_LOSS_SQUARED) target_mine = a.targets[tid];
    else label_mine = a.labels[tid];
  }
  const float neg_gamma = -a.gamma;
  double nrm = 0.0;

#pragma unroll 1
  for (int l = 0; l < a.L; ++l) {
    const int N = a.dims[l + 1], K = a.dims[l];
    const int tiles = (N + 31) / 32, kp_count = tiles == 1 ? 8 : tiles == 2 ? 4 : 2;
    const int tile = wave / kp_count, kp = wave % kp_count;
    const float* __restrict__ h_in = act[l & 1];
    const float* __restrict__ d_in = h_in + kRows * pitch;
    const int f = tile * 32 + n;
    const bool f_ok = f < N, second = l > 0;
    const float* __restrict__ wrow = a.x + a.w_off[l] + (long long)(f_ok ? f : 0) * K;
    const float* __restrict__ urow = P + a.w_off[l] + (long long)(f_ok ? f : 0) * K;
    const float* __restrict__ frow = a.features + (long long)(n < a.n_r ? n : 0) * a.dims[0];   // (layer 0; other rows are not used)
    // the biases of the tile, one feature per lane, requested ahead of everything else
    float bias_x = 0.f, bias_u = 0.f;
    if (a.b_off[l] >= 0 && f_ok) {
      bias_x = a.x[a.b_off[l] + f];
      bias_u = P[a.b_off[l] + f];
    }
    f32x16 z, c;
#pragma unroll
    for (int j = 0; j < 16; ++j) z[j] = c[j] = 0.f;
    if (tile < tiles) {
      const int steps = (K + 7) / 8, s_begin = steps * kp / kp_count, s_end = steps * (kp + 1) / kp_count;
      auto contract = [&](auto second_tag) {
        constexpr bool SECOND = decltype(second_tag)::value;
        // One step ahead of its products and hardly anything unrolled: the launch is short, its instructions come from memory as
        // they are first run, and straight-line code costs more than the round trips it hides (1, 2, 3, 4 steps a group, one
        // group ahead: 784 -> 10 23.7 / 24.8 / 25.7 / 26.3 us per score and update, 784 -> 64 -> 10 36.6 / 38.8 / 41.1 / 43.1).
        struct Step {
          f32x4 w, u, b, dv;
        };
        auto request = [&](Step& g, int s) {
          s = s < s_end ? s : s_end - 1;                             // (a step too many is not used)
          const int k = 8 * s + 4 * h;
          g.w = load_row4(wrow, k, K);
          g.u = load_row4(urow, k, K);
          if constexpr (SECOND) {
            g.b = *reinterpret_cast<const f32x4*>(h_in + n * pitch + k);
            g.dv = *reinterpret_cast<const f32x4*>(d_in + n * pitch + k);
          } else {
            g.b = load_row4(frow, k, K);
          }
        };
        auto multiply = [&](Step& g, int s) {
          if (s >= s_end) return;
          const int k = 8 * s + 4 * h;
          if (8 * s + 8 > K) {
            g.w = end_of_row4(g.w, k, K);
            g.u = end_of_row4(g.u, k, K);
            if constexpr (!SECOND) g.b = end_of_row4(g.b, k, K);
          }
          const f32x4 u = g.u;
          if (f_ok) nrm += (double)((u[0] * u[0] + u[1] * u[1]) + (u[2] * u[2] + u[3] * u[3]));
          const f32x4 wr = operand<BF16>(g.w), ur = operand<BF16>(u), b = SECOND ? g.b : operand<BF16>(g.b);
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            z = __builtin_amdgcn_mfma_f32_32x32x2f32(wr[i], b[i], z, 0, 0, 0);
            c = __builtin_amdgcn_mfma_f32_32x32x2f32(ur[i], b[i], c, 0, 0, 0);
            if constexpr (SECOND)
              c = __builtin_amdgcn_mfma_f32_32x32x2f32(operand<BF16>(__builtin_fmaf(neg_gamma, ur[i], wr[i])), g.dv[i], c, 0, 0, 0);
          }
        };
        if (s_begin >= s_end) return;
        Step even, odd;
        request(even, s_begin);
#pragma unroll 1
        for (int s = s_begin; s < s_end; s += 2) {
          request(odd, s + 1);
          multiply(even, s);
          request(even, s + 2);
          multiply(odd, s + 1);
        }
      };
      if (second) contract(std::true_type{});
      else contract(std::false_type{});
    }
    if (l == 0 && tid < kRows) {
      label[tid] = label_mine;
      target[tid] = target_mine;
    }
    // The accumulators of the waves that share a tile, added in wave order; the waves finish a quarter of the tile's
    // features each (two of two waves).  Quarter q: registers 4 q .. 4 q + 3, i.e. sample n, features 8 q + 4 h .. + 3.
    if (tile < tiles) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        red[(wave * 8 + q) * 64 + lane] = f32x4{z[4 * q], z[4 * q + 1], z[4 * q + 2], z[4 * q + 3]};
        red[(wave * 8 + 4 + q) * 64 + lane] = f32x4{c[4 * q], c[4 * q + 1], c[4 * q + 2], c[4 * q + 3]};
      }
    }
    __syncthreads();
    const int quarters = kp_count == 2 ? 2 : 1;
    if (tile < tiles && kp < 4) {
      if (kp == 0 && lane < 32) nrm += (double)(bias_u * bias_u);
      // The output layer leaves Z0 and dZ, hidden layers the operands of the next one (zeros in the padding of its last step)
      float* __restrict__ h_out = act[(l + 1) & 1];
      float* __restrict__ d_out = h_out + kRows * pitch;
      const bool last = l + 1 == a.L;
#pragma unroll 1
      for (int qq = 0; qq < quarters; ++qq) {
        const int q = kp * quarters + qq, f0 = tile * 32 + 8 * q + 4 * h;
        const f32x4* part = red + (tile * kp_count * 8 + q) * 64 + lane;
        f32x4 zs = part[0], cs = part[4 * 64];
#pragma unroll 1
        for (int w = 1; w < kp_count; ++w) {
          zs += part[w * 8 * 64];
          cs += part[(w * 8 + 4) * 64];
        }
        f32x4 hv, dd;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float bx = __shfl(bias_x, 8 * q + 4 * h + i, 64), bu = __shfl(bias_u, 8 * q + 4 * h + i, 64);
          const float z0 = zs[i] + bx, dz = -a.gamma * (cs[i] + bu);
          if (last) {
            hv[i] = z0;
            dd[i] = dz;
          } else {
            const bool ok = f0 + i < N;
            const float hr = relu_nan(z0 + dz);
            // relu(z0 + dz) - relu(z0) without cancellation
            const float change = (z0 > 0.f) ? ((dz < -z0) ? -z0 : dz) : hr;
            hv[i] = ok ? operand<BF16>(relu_nan(z0)) : 0.f;
            dd[i] = ok ? operand<BF16>(change * a.neg_inv_gamma) : 0.f;
          }
        }
        if (f0 < (N + 7) / 8 * 8) {
          *reinterpret_cast<f32x4*>(h_out + n * pitch + f0) = hv;
          *reinterpret_cast<f32x4*>(d_out + n * pitch + f0) = dd;
        }
      }
    }
    __syncthreads();
  }

  // per-sample loss differences in fp64 from (Z0, dZ), as in loss_diff_kernel; sixteen lanes (of up to sixteen classes) a sample
  const int C = a.dims[a.L];
  const float* __restrict__ z0 = act[a.L & 1];
  const float* __restrict__ dz = z0 + kRows * pitch;
  const int k = tid / kMaxClasses, q = tid % kMaxClasses;
  const bool live = k < a.n_r;
  const int r = live ? k : 0;
  double diff;
  if (a.loss == ZENO_LOSS_SQUARED) {
    const double zz = (double)z0[r * pitch], t = (double)dz[r * pitch], y = (double)target[r];
    diff = t * ((zz - y) + 0.5 * t);
  } else {
    const double v0 = q < C ? (double)z0[r * pitch + q] : -__builtin_inf();
    const double v1 = q < C ? v0 + (double)dz[r * pitch + q] : -__builtin_inf();
    const double m0 = max_over(v0, kMaxClasses), m1 = max_over(v1, kMaxClasses);
    const double s0 = sum_over(q < C ? exp(v0 - m0) : 0.0, kMaxClasses), s1 = sum_over(q < C ? exp(v1 - m1) : 0.0, kMaxClasses);
    // a label outside [0, C) has no logit: NaN instead of reading past the row
    const int y = label[r];
    const double dzy = (y >= 0 && y < C) ? (double)dz[r * pitch + y] : __builtin_nan("");
    diff = ((m1 + log(s1)) - (m0 + log(s0))) - dzy;
  }
  double diff_sum = live && q == 0 ? diff : 0.0;
  diff_sum = sum_over(diff_sum, 64);
  nrm = sum_over(nrm, 64);
  if (lane == 0) {
    totals[0][wave] = diff_sum;
    totals[1][wave] = nrm;
  }
  __syncthreads();
  if (tid == 0) {
    double sd = 0.0, sn = 0.0;
    for (int w = 0; w < kWaves; ++w) {
      sd += totals[0][w];
      sn += totals[1][w];
    }
    a.scores[blockIdx.x] = (float)(-(sd / (double)a.n_r) - (double)a.rho * sn);
  }
}

int small_pitch(const int* dims, int L) {
  int width = 8;
  for (int l = 1; l <= L; ++l) width = dims[l] > width ? dims[l] : width;
  return (width + 7) / 8 * 8 + 4;      // rows 16 bytes further round the banks each
}

}  // namespace

// One workgroup per candidate pays while a workgroup's matrix steps (8 k of a tile; the second product counts) stay below what
// the general path spends on its 2 L + 3 launches.  Measured on 962 random models with up to 400 steps a layer, time of score and
// update on the general path / this one: float32 up to 300 steps a layer 1.60, none of 471 more than 2 % slower; 300 to 350 1.50, 1 of 32;
// beyond that 9 of 27, by up to 8 %; 600 to 800 steps in all 1.82, 800 to 1300 1.50, 1 of 29.  bf16 operands, whose general path
// multiplies eight times as fast: up to 200 steps a layer 1.40, none of 366, but for four layers of that length.  Single layers, with
// the fewest launches to save, are among the slower ones from 350 (222) steps on and change sides at 250 (125).
// More classes would put several rounds of exponentials behind each other (784 -> 32: 37.8 / 32.4, 59.2 / 46.8).  Beyond 256
// candidates the workgroups of a CU follow each other (random models, 257 to 1024 candidates: 1.06, 49 of 216 slower, by up to
// 18 %).  Rows shorter than four floats cannot be read four at a time.
bool small_model_fits(const int* dims, int L, int m, int n_r, bool bf16) {
  if (n_r > kRows || dims[L] > kMaxClasses || m > 256) return false;
  long long steps = 0;
  for (int l = 0; l < L; ++l) {
    if (dims[l] < 4 || dims[l + 1] > kMaxWidth) return false;
    steps += (long long)((dims[l + 1] + 31) / 32) * ((dims[l] + 7) / 8) * (l > 0 ? 3 : 2);
  }
  if (L == 1) return steps <= (bf16 ? 125 : 250);
  return steps <= (bf16 ? 180LL : 300LL) * L && steps <= (bf16 ? 600 : 1000);
}

hipError_t launch_score_small(SmallArgs a, bool bf16, int m, hipStream_t stream) {
  a.pitch = small_pitch(a.dims, a.L);
  const int lds = (4 * kRows * a.pitch + kWaves * 8 * 64 * 4) * (int)sizeof(float);
  constexpr int most = (4 * kRows * (kMaxWidth + 4) + kWaves * 8 * 64 * 4) * (int)sizeof(float);
  static const hipError_t attr_err = [] {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&score_small_kernel<true>), hipFuncAttributeMaxDynamicSharedMemorySize, most);
    if (e == hipSuccess)
      e = hipFuncSetAttribute(reinterpret_cast<const void*>(&score_small_kernel<false>), hipFuncAttributeMaxDynamicSharedMemorySize, most);
    return e;
  }();
  if (attr_err != hipSuccess) return attr_err;
  if (lds > most || !small_model_fits(a.dims, a.L, m, a.n_r, bf16)) return hipErrorInvalidValue;
  if (bf16) hipLaunchKernelGGL(score_small_kernel<true>, dim3(m), dim3(kThreads), lds, stream, a);
  else hipLaunchKernelGGL(score_small_kernel<false>, dim3(m), dim3(kThreads), lds, stream, a);
  return hipGetLastError();
}

}  // namespace zeno
