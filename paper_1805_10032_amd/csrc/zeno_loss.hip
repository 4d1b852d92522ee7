// Loss head and score combine of the Stochastic Descendant Score (Definition 2).
//
// The layer kernels deliver, for the output layer, the pre-activations at x (Z0)
// and, per candidate, their change dZ_i caused by moving to x - gamma u_i.
// Per sample k this file forms f(x - gamma u_i; z_k) - f(x; z_k) in fp64
// directly from (Z0, dZ_i), then
//     score_i = -(1/n_r) sum_k diff_ik - rho ||u_i||^2 .
#include "zeno_internal.h"

namespace zeno {

namespace {

template <int LANES = 64>
__device__ inline double wave_sum(double v) {
#pragma unroll
  for (int off = LANES / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}
template <int LANES = 64>
__device__ inline double wave_max(double v) {
#pragma unroll
  for (int off = LANES / 2; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off, 64));
  return v;
}

// Loss difference of one sample by LANES lanes, lane `lane` of them.  Softmax cross-entropy:
//   diff = logsumexp(z0 + dz) - logsumexp(z0) - dz[label]
// squared loss (output width 1):
//   diff = 1/2 (z0 + dz - y)^2 - 1/2 (z0 - y)^2 = dz ((z0 - y) + dz/2).
// A NaN anywhere in dz reaches the sum of exponentials and makes diff NaN.
template <int LANES>
__device__ inline double loss_diff(const float* __restrict__ z0, const float* __restrict__ dz, const int32_t* __restrict__ label,
                                   const float* __restrict__ target, int loss, int C, int lane) {
  if (loss == ZENO_LOSS_SQUARED) {
    const double z = (double)z0[0], t = (double)dz[0], y = (double)*target;
    return t * ((z - y) + 0.5 * t);
  }
  const int y = *label;
  double m0 = -__builtin_inf(), m1 = -__builtin_inf();
  for (int c = lane; c < C; c += LANES) {
    const double a = (double)z0[c], b = a + (double)dz[c];
    m0 = fmax(m0, a);
    m1 = fmax(m1, b);
  }
  m0 = wave_max<LANES>(m0);
  m1 = wave_max<LANES>(m1);
  double s0 = 0.0, s1 = 0.0;
  for (int c = lane; c < C; c += LANES) {
    const double a = (double)z0[c], b = a + (double)dz[c];
    s0 += exp(a - m0);
    s1 += exp(b - m1);
  }
  s0 = wave_sum<LANES>(s0);
  s1 = wave_sum<LANES>(s1);
  // a label outside [0, C) has no logit: the sample's loss difference becomes NaN (and with it
  // every score) instead of reading past the row
  const double dzy = (y >= 0 && y < C) ? (double)dz[y] : __builtin_nan("");
  return ((m1 + log(s1)) - (m0 + log(s0))) - dzy;
}

// One wave per (sample, candidate).
__global__ __launch_bounds__(64) void loss_diff_kernel(const float* __restrict__ Z0, const float* __restrict__ dZ,
                                                       const int32_t* __restrict__ labels,
                                                       const float* __restrict__ targets, int loss, int n_r_total,
                                                       int chunk_begin, int chunk_rows, int C,
                                                       double* __restrict__ sample_diff) {
  const int kk = blockIdx.x, i = blockIdx.y, lane = threadIdx.x;
  const double diff = loss_diff<64>(Z0 + (long long)kk * C, dZ + ((long long)i * chunk_rows + kk) * C, labels + chunk_begin + kk,
                                    targets + chunk_begin + kk, loss, C, lane);
  if (lane == 0) sample_diff[(long long)i * n_r_total + chunk_begin + kk] = diff;
}

// One workgroup per candidate: the loss differences of all its samples, sixteen lanes each, and the score, in one launch (two
// cost 4-5 us each, whatever they do).  Every sum is formed in the order of the two kernels, so the bits are the same: lanes
// beyond the classes hold the sum's zeros in either.
constexpr int kScoreClasses = 16;
constexpr int kScoreRows = 64;
constexpr int kScoreThreads = kScoreClasses * kScoreRows;
__global__ __launch_bounds__(kScoreThreads) void loss_score_kernel(const float* __restrict__ Z0, const float* __restrict__ dZ,
                                                                   const int32_t* __restrict__ labels,
                                                                   const float* __restrict__ targets, int loss, int n_r, int C,
                                                                   const double* __restrict__ norm_partials, int P_stride, int P,
                                                                   float rho, float* __restrict__ scores) {
  __shared__ double diffs[kScoreRows], norm;
  const int i = blockIdx.x, tid = threadIdx.x;
  if (tid >= kScoreThreads - 64) {       // the last wave, whose samples are the last
    const int lane = tid & 63;
    double sn = 0.0;
    for (int p = lane; p < P; p += 64) sn += norm_partials[(long long)i * P_stride + p];
    sn = wave_sum(sn);
    if (lane == 0) norm = sn;
  }
  const int k = tid / kScoreClasses, lane = tid % kScoreClasses;
  if (k < n_r) {                         // (uniform over the sixteen lanes of a sample)
    const double diff = loss_diff<kScoreClasses>(Z0 + (long long)k * C, dZ + ((long long)i * n_r + k) * C, labels + k, targets + k,
                                                 loss, C, lane);
    if (lane == 0) diffs[k] = diff;
  }
  __syncthreads();
  if (tid >= 64) return;
  const double sd = wave_sum(tid < n_r ? diffs[tid] : 0.0);
  if (tid == 0) scores[i] = (float)(-(sd / (double)n_r) - (double)rho * norm);
}

// One wave per candidate: mean over the n_r samples, sum of the partial squared
// norms, and the three-term combine, all in fp64, rounded once to fp32.
// A candidate's partial norms lie P_stride apart, of which the first P are in use.
__global__ __launch_bounds__(64) void score_combine_kernel(const double* __restrict__ sample_diff,
                                                           const double* __restrict__ norm_partials, int P_stride, int P,
                                                           int n_r_total, float rho, float* __restrict__ scores) {
  const int i = blockIdx.x, lane = threadIdx.x;
  double sd = 0.0, sn = 0.0;
  for (int k = lane; k < n_r_total; k += 64) sd += sample_diff[(long long)i * n_r_total + k];
  for (int p = lane; p < P; p += 64) sn += norm_partials[(long long)i * P_stride + p];
  sd = wave_sum(sd);
  sn = wave_sum(sn);
  if (lane == 0) scores[i] = (float)(-(sd / (double)n_r_total) - (double)rho * sn);
}

}  // namespace

hipError_t launch_loss(const float* Z0, const float* dZ, const int32_t* labels, const float* targets, int loss,
                       int m, int n_r_total, int chunk_begin, int chunk_rows, int C, double* sample_diff,
                       hipStream_t stream) {
  hipLaunchKernelGGL(loss_diff_kernel, dim3(chunk_rows, m), dim3(64), 0, stream, Z0, dZ, labels, targets, loss,
                     n_r_total, chunk_begin, chunk_rows, C, sample_diff);
  return hipGetLastError();
}

hipError_t launch_score_combine_strided(const double* sample_diff, const double* norm_partials, int P_stride, int P,
                                        int m, int n_r_total, float rho, float* scores, hipStream_t stream) {
  hipLaunchKernelGGL(score_combine_kernel, dim3(m), dim3(64), 0, stream, sample_diff, norm_partials, P_stride, P,
                     n_r_total, rho, scores);
  return hipGetLastError();
}

hipError_t launch_score_combine(const double* sample_diff, const double* norm_partials, int P, int m,
                                int n_r_total, float rho, float* scores, hipStream_t stream) {
  return launch_score_combine_strided(sample_diff, norm_partials, P, P, m, n_r_total, rho, scores, stream);
}

// One launch for what its 1024 threads take at a time.  Measured (us per score of 512 -> 256 -> C, m = 20, one launch / two):
// C = 10, n_r = 32: 54.4 / 55.6, n_r = 64: 72.4 / 74; n_r = 128 (two samples after each other): 100.0 / 99; a wave per sample
// for more classes: C = 17, n_r = 4: 54.4 / 55.9, n_r = 16: 56.5 / 55.8, n_r = 32: 59.8 / 55.9.
bool loss_score_fits(int n_r, int C) { return n_r <= kScoreRows && C <= kScoreClasses; }

hipError_t launch_loss_score(const float* Z0, const float* dZ, const int32_t* labels, const float* targets, int loss, int m, int n_r,
                             int C, const double* norm_partials, int P_stride, int P, float rho, float* scores, hipStream_t stream) {
  if (!loss_score_fits(n_r, C)) return hipErrorInvalidValue;
  hipLaunchKernelGGL(loss_score_kernel, dim3(m), dim3(kScoreThreads), 0, stream, Z0, dZ, labels, targets, loss, n_r, C, norm_partials,
                     P_stride, P, rho, scores);
  return hipGetLastError();
}

}  // namespace zeno
