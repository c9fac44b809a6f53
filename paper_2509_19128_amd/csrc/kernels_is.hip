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
// A sequence's sums are added up in an order that its own length decides, not the number of sequences in the call: one of more than
// IS_SHORT tokens as IS_LANES lanes would, lane l taking the quads l, l + IS_LANES, ..., wavefront by wavefront, however many of
// these lanes a thread takes over; a shorter one as IS_SHORT_LANES lanes, a token at a time.
constexpr int IS_LANES = 1024, IS_SHORT = 1024, IS_SHORT_LANES = 256;
__device__ inline float is_weight(float pi, float mu, double c, double &s1, double &s2) {
  const double w = fmin(c, exp((double)pi - (double)mu));
  s1 += w;
  s2 = __builtin_fma(w, w, s2);
  return (float)w;
}
template <int NT>
__global__ __launch_bounds__(NT) void is_seq_kernel(const float *__restrict__ lp_pi, const float *__restrict__ lp_mu,
                                                    const int64_t *__restrict__ offsets, double c,
                                                    float *__restrict__ w_out, double *__restrict__ seq_sums,
                                                    double *__restrict__ ess_seq) {
  constexpr int V = IS_LANES / NT, NW = IS_LANES / 64;   // lanes of a thread: threadIdx.x + v * NT
  __shared__ double red[2 * NW];
  const int s = blockIdx.x;
  const int64_t a = offsets[s], b = offsets[s + 1];
  double s1[V] = {}, s2[V] = {};
  int nw = NW;   // wavefronts of lanes that have tokens
  if (b - a <= IS_SHORT) {
    nw = (int)min((int64_t)IS_SHORT_LANES, b - a + 63) / 64;
    for (int64_t i0 = a + threadIdx.x; threadIdx.x < IS_SHORT_LANES && i0 < b; i0 += 4 * IS_SHORT_LANES) {
      float p[4], m[4];   // the loads of four tokens are issued together
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (i0 + u * IS_SHORT_LANES < b) { p[u] = lp_pi[i0 + u * IS_SHORT_LANES]; m[u] = lp_mu[i0 + u * IS_SHORT_LANES]; }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (i0 + u * IS_SHORT_LANES >= b) continue;
        const float w = is_weight(p[u], m[u], c, s1[0], s2[0]);
        if (w_out) w_out[i0 + u * IS_SHORT_LANES] = w;
      }
    }
  } else {
    const uintptr_t off = (uintptr_t)(lp_pi + a) & 15;
    const bool alike = ((uintptr_t)(lp_mu + a) & 15) == off && (!w_out || ((uintptr_t)(w_out + a) & 15) == off);
    const int64_t first = alike ? a + (int64_t)((16 - off) & 15) / 4 : b;   // [first, last): whole aligned quads
    const int64_t last = first + (b - first) / 4 * 4;
    for (int64_t i0 = first + 4 * (int64_t)threadIdx.x; i0 < last; i0 += 4 * IS_LANES) {
#pragma unroll
      for (int v = 0; v < V; ++v) {
        const int64_t i = i0 + v * 4 * NT;
        if (i >= last) continue;
        const f32x4 p = *(const f32x4 *)(lp_pi + i), m = *(const f32x4 *)(lp_mu + i);
        f32x4 w;
#pragma unroll
        for (int e = 0; e < 4; ++e) w[e] = is_weight(p[e], m[e], c, s1[v], s2[v]);
        if (w_out) *(f32x4 *)(w_out + i) = w;
      }
    }
    // what is left: [a, first) and [last, b)
    const int64_t head = first - a, left = head + (b - last);
    nw = (int)min((int64_t)NW, (max((last - first) / 4, left) + 63) / 64);
    for (int64_t k0 = threadIdx.x; k0 < left; k0 += IS_LANES) {
#pragma unroll
      for (int v = 0; v < V; ++v) {
        const int64_t k = k0 + v * NT;
        if (k >= left) continue;
        const int64_t i = k < head ? a + k : last + (k - head);
        const float w = is_weight(lp_pi[i], lp_mu[i], c, s1[v], s2[v]);
        if (w_out) w_out[i] = w;
      }
    }
  }
#pragma unroll
  for (int v = 0; v < V; ++v) {
    const int wave = (int)(threadIdx.x >> 6) + v * (NT / 64);   // of the lanes
    if (wave >= nw) continue;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      s1[v] += __shfl_xor(s1[v], o, 64);
      s2[v] += __shfl_xor(s2[v], o, 64);
    }
    if ((threadIdx.x & 63) == 0) { red[2 * wave] = s1[v]; red[2 * wave + 1] = s2[v]; }
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double t1 = 0.0, t2 = 0.0;
    for (int w = 0; w < nw; ++w) { t1 += red[2 * w]; t2 += red[2 * w + 1]; }
    seq_sums[2 * s] = t1;
    seq_sums[2 * s + 1] = t2;
    ess_seq[s] = b > a ? t1 * t1 / ((double)(b - a) * t2) : __longlong_as_double(0x7FF8000000000000LL);
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
  // 1024 threads finish the longest sequences sooner, 256 let more workgroups run: whole call with 256 / 1024, 1536 sequences of 16
  // tokens on average 9.7 / 9.7 us, of 1000 16.2 / 15.1, of 4096 31 / 25; 2048 of 1000 14.0 / 15.7; 8192 of 16 13.4 / 27, of
  // 1000 31 / 49, of 4096 94 / 91.
  if (n_seq <= 1536)
    hipLaunchKernelGGL(is_seq_kernel<1024>, dim3(n_seq), dim3(1024), 0, s, lp_pi, lp_mu, offsets, c, w_out, seq_sums, ess_seq);
  else
    hipLaunchKernelGGL(is_seq_kernel<256>, dim3(n_seq), dim3(256), 0, s, lp_pi, lp_mu, offsets, c, w_out, seq_sums, ess_seq);
  hipLaunchKernelGGL(is_total_kernel, dim3(1), dim3(1024), 0, s, seq_sums, offsets, n_seq, totals);
  return hipGetLastError() == hipSuccess ? 0 : -7;
}

}  // namespace pl
