// Trainer-side consumer of the recorded behaviour log-probs (Sec. 2.1 of the paper): truncated
// token-level importance weights w = min(c, pi / mu) and the normalised effective sample size
// (sum w)^2 / (N sum w^2), per packed sequence and over the whole batch.  A stream of 8 bytes in and
// 4 bytes out per token; all arithmetic in fp64, reductions in a fixed order (no atomics), so the
// result does not depend on scheduling.
#include "pl_common.h"

namespace pl {
namespace {

template <int NW>
__device__ inline void block_sum2(double &a, double &b, double *red) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    a += __shfl_xor(a, o, 64);
    b += __shfl_xor(b, o, 64);
  }
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) { red[2 * wave] = a; red[2 * wave + 1] = b; }
  __syncthreads();
  a = 0.0; b = 0.0;
  for (int w = 0; w < NW; ++w) { a += red[2 * w]; b += red[2 * w + 1]; }
}

// One workgroup per sequence: tokens [offsets[s], offsets[s + 1]).  Bound by latency and by the compute unit that
// gets the most tokens, not by bytes or by the fp64 exp (one of half the operations changed nothing).  A thread
// takes four tokens with 16-byte accesses wherever the three arrays are aligned alike (the tokens before the first
// aligned one and after the last go one by one).  1024 sequences (4096 tokens on average, 16384 at most), whole call:
// 24.1 us with 256 threads and 4-byte accesses; 16-byte: 17.4 us with 1024 threads, one quad in flight each; 18.9 with
// 512 and four; 21.6 with 1024 and two; 22.6 with 256 and four.
constexpr int IS_NT = 1024;
__device__ inline float is_weight(float pi, float mu, double c, double &s1, double &s2) {
  const double w = fmin(c, exp((double)pi - (double)mu));
  s1 += w;
  s2 = __builtin_fma(w, w, s2);
  return (float)w;
}
__global__ __launch_bounds__(IS_NT) void is_seq_kernel(const float *__restrict__ lp_pi, const float *__restrict__ lp_mu,
                                                       const int64_t *__restrict__ offsets, double c,
                                                       float *__restrict__ w_out, double *__restrict__ seq_sums,
                                                       double *__restrict__ ess_seq) {
  __shared__ double red[2 * IS_NT / 64];
  const int s = blockIdx.x;
  const int64_t a = offsets[s], b = offsets[s + 1];
  const uintptr_t off = (uintptr_t)(lp_pi + a) & 15;
  const bool alike = ((uintptr_t)(lp_mu + a) & 15) == off && (!w_out || ((uintptr_t)(w_out + a) & 15) == off);
  const int64_t first = alike ? min(b, a + (int64_t)((16 - off) & 15) / 4) : b;   // [first, last): whole aligned quads
  const int64_t last = first + (b - first) / 4 * 4;
  double s1 = 0.0, s2 = 0.0;
  for (int64_t i = first + 4 * (int64_t)threadIdx.x; i < last; i += 4 * IS_NT) {
    const f32x4 p = *(const f32x4 *)(lp_pi + i), m = *(const f32x4 *)(lp_mu + i);
    f32x4 w;
#pragma unroll
    for (int e = 0; e < 4; ++e) w[e] = is_weight(p[e], m[e], c, s1, s2);
    if (w_out) *(f32x4 *)(w_out + i) = w;
  }
  // what is left: [a, first) and [last, b)
  const int64_t head = first - a;
  for (int64_t k = threadIdx.x; k < head + (b - last); k += IS_NT) {
    const int64_t i = k < head ? a + k : last + (k - head);
    const float w = is_weight(lp_pi[i], lp_mu[i], c, s1, s2);
    if (w_out) w_out[i] = w;
  }
  block_sum2<IS_NT / 64>(s1, s2, red);
  if (threadIdx.x == 0) {
    seq_sums[2 * s] = s1;
    seq_sums[2 * s + 1] = s2;
    ess_seq[s] = b > a ? s1 * s1 / ((double)(b - a) * s2) : __longlong_as_double(0x7FF8000000000000LL);
  }
}

// totals[0..2] = sum w, sum w^2, normalised ESS over all tokens; one workgroup, fixed order
__global__ __launch_bounds__(1024) void is_total_kernel(const double *__restrict__ seq_sums,
                                                        const int64_t *__restrict__ offsets, int n_seq,
                                                        double *__restrict__ totals) {
  __shared__ double red[32];
  double s1 = 0.0, s2 = 0.0;
  for (int s = threadIdx.x; s < n_seq; s += 1024) { s1 += seq_sums[2 * s]; s2 += seq_sums[2 * s + 1]; }
  block_sum2<16>(s1, s2, red);
  if (threadIdx.x == 0) {
    const int64_t n = offsets[n_seq] - offsets[0];
    totals[0] = s1;
    totals[1] = s2;
    totals[2] = n > 0 ? s1 * s1 / ((double)n * s2) : __longlong_as_double(0x7FF8000000000000LL);
  }
}

}  // namespace

int launch_is_ess(const float *lp_pi, const float *lp_mu, const int64_t *offsets, int n_seq, double c, float *w_out,
                  double *seq_sums, double *ess_seq, double *totals, hipStream_t s) {
  if (n_seq < 1) return -1;
  hipLaunchKernelGGL(is_seq_kernel, dim3(n_seq), dim3(IS_NT), 0, s, lp_pi, lp_mu, offsets, c, w_out, seq_sums, ess_seq);
  hipLaunchKernelGGL(is_total_kernel, dim3(1), dim3(1024), 0, s, seq_sums, offsets, n_seq, totals);
  return hipGetLastError() == hipSuccess ? 0 : -7;
}

}  // namespace pl
