// Trainer-side consumer of the recorded behaviour log-probs (Sec. 2.1 of the paper): truncated
// token-level importance weights w = min(c, pi / mu) and the normalised effective sample size
// (sum w)^2 / (N sum w^2), per packed sequence and over the whole batch.  A stream of 8 bytes in and
// 4 bytes out per token; all arithmetic in fp64, reductions in a fixed order (no atomics), so the
// result does not depend on scheduling.
#include "pl_common.h"

namespace pl {
namespace {

// Sum over the wavefront in a fixed order; every lane ends with it.
__device__ inline double wave_sum(double v) {
#ifdef __HIP_DEVICE_COMPILE__
  auto other = [&](auto CTRL) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, decltype(CTRL)::value, 0xF, 0xF, true),
                   hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), decltype(CTRL)::value, 0xF, 0xF, true);
    return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
  };
  v += other(std::integral_constant<int, DPP_XOR1>{});
  v += other(std::integral_constant<int, DPP_XOR2>{});
  v += other(std::integral_constant<int, DPP_HALF_MIRROR>{});
  v += other(std::integral_constant<int, DPP_MIRROR>{});
  v += __shfl_xor(v, 16, 64);
  v += __shfl_xor(v, 32, 64);
#endif
  return v;
}

// e^x: 2^(j / 64) from a table, 2^i by the exponent, and e^r - 1 by its power series to r^5 with the next term spread over the even ones
// (Chebyshev's r^6 on |r| <= ln 2 / 128), which leaves 2^-59.6.  19 fp64 operations where the library's exp has 28: a compute unit with more than its share of tokens
// is busy with them (1024 sequences 14.4 -> 13.6 us).  At most 0.53 units in the last place: half of one from the last addition, 0.01 from the series,
// 0.02 from what is added to the table's value (with the table rounded to one number, an operation and 0.5 us less, it was 1.0).
__device__ const double EXP2_64[64] = {
    0x1.0000000000000p+0, 0x1.02c9a3e778061p+0, 0x1.059b0d3158574p+0, 0x1.0874518759bc8p+0,
    0x1.0b5586cf9890fp+0, 0x1.0e3ec32d3d1a2p+0, 0x1.11301d0125b51p+0, 0x1.1429aaea92de0p+0,
    0x1.172b83c7d517bp+0, 0x1.1a35beb6fcb75p+0, 0x1.1d4873168b9aap+0, 0x1.2063b88628cd6p+0,
    0x1.2387a6e756238p+0, 0x1.26b4565e27cddp+0, 0x1.29e9df51fdee1p+0, 0x1.2d285a6e4030bp+0,
    0x1.306fe0a31b715p+0, 0x1.33c08b26416ffp+0, 0x1.371a7373aa9cbp+0, 0x1.3a7db34e59ff7p+0,
    0x1.3dea64c123422p+0, 0x1.4160a21f72e2ap+0, 0x1.44e086061892dp+0, 0x1.486a2b5c13cd0p+0,
    0x1.4bfdad5362a27p+0, 0x1.4f9b2769d2ca7p+0, 0x1.5342b569d4f82p+0, 0x1.56f4736b527dap+0,
    0x1.5ab07dd485429p+0, 0x1.5e76f15ad2148p+0, 0x1.6247eb03a5585p+0, 0x1.6623882552225p+0,
    0x1.6a09e667f3bcdp+0, 0x1.6dfb23c651a2fp+0, 0x1.71f75e8ec5f74p+0, 0x1.75feb564267c9p+0,
    0x1.7a11473eb0187p+0, 0x1.7e2f336cf4e62p+0, 0x1.82589994cce13p+0, 0x1.868d99b4492edp+0,
    0x1.8ace5422aa0dbp+0, 0x1.8f1ae99157736p+0, 0x1.93737b0cdc5e5p+0, 0x1.97d829fde4e50p+0,
    0x1.9c49182a3f090p+0, 0x1.a0c667b5de565p+0, 0x1.a5503b23e255dp+0, 0x1.a9e6b5579fdbfp+0,
    0x1.ae89f995ad3adp+0, 0x1.b33a2b84f15fbp+0, 0x1.b7f76f2fb5e47p+0, 0x1.bcc1e904bc1d2p+0,
    0x1.c199bdd85529cp+0, 0x1.c67f12e57d14bp+0, 0x1.cb720dcef9069p+0, 0x1.d072d4a07897cp+0,
    0x1.d5818dcfba487p+0, 0x1.da9e603db3285p+0, 0x1.dfc97337b9b5fp+0, 0x1.e502ee78b3ff6p+0,
    0x1.ea4afa2a490dap+0, 0x1.efa1bee615a27p+0, 0x1.f50765b6e4540p+0, 0x1.fa7c1819e90d8p+0,
};
__device__ const double EXP2_64_REST[64] = {   // what the values above lack
    0x0.0p+0, -0x1.19083535b085dp-56, 0x1.d73e2a475b465p-55, 0x1.186be4bb284ffp-57,
    0x1.8a62e4adc610bp-54, 0x1.03a1727c57b53p-59, -0x1.6c51039449b3ap-54, -0x1.32fbf9af1369ep-54,
    -0x1.19041b9d78a76p-55, 0x1.e5b4c7b4968e4p-55, 0x1.e016e00a2643cp-54, 0x1.dc775814a8495p-55,
    0x1.9b07eb6c70573p-54, 0x1.2bd339940e9d9p-55, 0x1.612e8afad1255p-55, 0x1.0024754db41d5p-54,
    0x1.6f46ad23182e4p-55, 0x1.32721843659a6p-54, -0x1.63aeabf42eae2p-54, -0x1.5e436d661f5e3p-56,
    0x1.ada0911f09ebcp-55, -0x1.ef3691c309278p-58, 0x1.89b7a04ef80d0p-59, 0x1.3c1a3b69062f0p-56,
    0x1.d4397afec42e2p-56, -0x1.4b309d25957e3p-54, -0x1.07abe1db13cadp-55, 0x1.9bb2c011d93adp-54,
    0x1.6324c054647adp-54, 0x1.ba6f93080e65ep-54, -0x1.383c17e40b497p-54, -0x1.bb60987591c34p-54,
    -0x1.bdd3413b26456p-54, -0x1.bbe3a683c88abp-57, -0x1.16e4786887a99p-55, -0x1.0245957316dd3p-54,
    -0x1.41577ee04992fp-55, 0x1.05d02ba15797ep-56, -0x1.d4c1dd41532d8p-54, -0x1.fc6f89bd4f6bap-54,
    0x1.6e9f156864b27p-54, 0x1.5cc13a2e3976cp-55, -0x1.75fc781b57ebcp-57, -0x1.d185b7c1b85d1p-54,
    0x1.c7c46b071f2bep-56, -0x1.359495d1cd533p-54, -0x1.d2f6edb8d41e1p-54, 0x1.0fac90ef7fd31p-54,
    0x1.7a1cd345dcc81p-54, -0x1.2805e3084d708p-57, -0x1.5584f7e54ac3bp-56, 0x1.23dd07a2d9e84p-55,
    0x1.11065895048ddp-55, 0x1.2884dff483cadp-54, 0x1.503cbd1e949dbp-56, -0x1.cbc3743797a9cp-54,
    0x1.2ed02d75b3707p-55, 0x1.c2300696db532p-54, -0x1.1a5cd4f184b5cp-54, 0x1.39e8980a9cc8fp-55,
    -0x1.e9c23179c2893p-54, 0x1.dc7f486a4b6b0p-54, 0x1.9d3e12dd8a18bp-54, 0x1.74853f3a5931ep-55,
};
__device__ inline double exp_table(double x, const double *t) {   // t: EXP2_64, then EXP2_64_REST
  x = fmax(fmin(x, 710.0), -746.0);   // infinity and zero beyond; a NaN goes with infinity, as fmin(c, NaN) is c
  const double shifted = __builtin_fma(x, 0x1.71547652b82fep+6, 0x1.8p52), k = shifted - 0x1.8p52;   // k = rint(64 x / ln 2), also in the low bits
  const int n = (int)(uint32_t)__builtin_bit_cast(uint64_t, shifted);
  const double r = __builtin_fma(-k, 0x1.473de6af278edp-40, __builtin_fma(-k, 0x1.62e42fef00000p-7, x));
  const double q = __builtin_fma(__builtin_fma(__builtin_fma(r, 1.0 / 120, 0x1.55557621dbbb3p-5), r, 1.0 / 6), r, 0x1.fffffffffd0bap-2);
  const double p = __builtin_fma(r * r, q, r), e = t[n & 63];
  return __builtin_ldexp(e + __builtin_fma(e, p, t[64 + (n & 63)]), n >> 6);
}

// One workgroup per sequence: tokens [offsets[s], offsets[s + 1]).  A thread takes four tokens with 16-byte accesses wherever the
// three arrays are aligned alike (the tokens before the first aligned one and after the last go one by one), the loads of its next four under the
// exponentials of those at hand.  Bound by the compute unit that gets the most tokens (its fp64 exponentials and what it can read): 1024 sequences
// (4096 tokens on average, 16384 at most) 13.6 us, 9.5 if all were as long as the average; their tokens without sequences 9.4 with the library's
// exp.  With that exp 14.4; and with a question per quad whether weights are wanted 15.1; with 1024 threads 15.4; and with no load under way
// meanwhile 16.5.  Sequences ranked by length, so that long and short ones share a unit: finding the rank takes what the balance gains.
// A sequence's sums are added up in an order that its own length decides, not the number of sequences in the call: one of more than
// IS_SHORT tokens as IS_LANES lanes would, lane l taking the quads l, l + IS_LANES, ..., wavefront by wavefront, however many of
// these lanes a thread takes over; a shorter one as IS_SHORT_LANES lanes, a token at a time.
constexpr int IS_MANY = 1536;   // most sequences of a call that have 512 threads each
constexpr int IS_LANES = 512, IS_SHORT = 1024, IS_SHORT_LANES = 256;
__device__ inline float is_weight(float pi, float mu, double c, const double *t, double &s1, double &s2) {
  const double w = fmin(c, exp_table((double)pi - (double)mu, t));
  s1 += w;
  s2 = __builtin_fma(w, w, s2);
  return (float)w;
}
template <int NT, bool W>   // W: weights are wanted
__global__ __launch_bounds__(NT) void is_seq_kernel(const float *__restrict__ lp_pi, const float *__restrict__ lp_mu,
                                                    const int64_t *__restrict__ offsets, double c,
                                                    float *__restrict__ w_out, double *__restrict__ seq_sums,
                                                    double *__restrict__ ess_seq) {
  constexpr int V = IS_LANES / NT, NW = IS_LANES / 64;   // lanes of a thread: threadIdx.x + v * NT
  __shared__ double red[2 * NW], exp2_64[128];
  if (threadIdx.x < 64) {
    exp2_64[threadIdx.x] = EXP2_64[threadIdx.x];
    exp2_64[64 + threadIdx.x] = EXP2_64_REST[threadIdx.x];
  }
  const int s = blockIdx.x;
  const int64_t a = offsets[s], b = offsets[s + 1];
  double s1[V] = {}, s2[V] = {};
  __syncthreads();
  int nw = NW;   // wavefronts of lanes that have tokens
  if (b - a <= IS_SHORT) {
    nw = (int)min((int64_t)IS_SHORT_LANES, b - a + 63) / 64;
    const int64_t i0 = a + threadIdx.x;
    if (threadIdx.x < IS_SHORT_LANES && i0 < b) {
      float p[4], m[4];   // the loads of four tokens are issued together
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (i0 + u * IS_SHORT_LANES < b) { p[u] = lp_pi[i0 + u * IS_SHORT_LANES]; m[u] = lp_mu[i0 + u * IS_SHORT_LANES]; }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (i0 + u * IS_SHORT_LANES >= b) continue;
        const float w = is_weight(p[u], m[u], c, exp2_64, s1[0], s2[0]);
        if (W) w_out[i0 + u * IS_SHORT_LANES] = w;
      }
    }
  } else {
    const uintptr_t off = (uintptr_t)(lp_pi + a) & 15;
    const bool alike = ((uintptr_t)(lp_mu + a) & 15) == off && (!W || ((uintptr_t)(w_out + a) & 15) == off);
    const int64_t first = alike ? a + (int64_t)((16 - off) & 15) / 4 : b;   // [first, last): whole aligned quads
    const int64_t last = first + (b - first) / 4 * 4;
    f32x4 p[V], m[V];
    auto load = [&](int64_t i0) {
#pragma unroll
      for (int v = 0; v < V; ++v)
        if (i0 + v * 4 * NT < last) { p[v] = *(const f32x4 *)(lp_pi + i0 + v * 4 * NT); m[v] = *(const f32x4 *)(lp_mu + i0 + v * 4 * NT); }
    };
    int64_t i0 = first + 4 * (int64_t)threadIdx.x;
    load(i0);
    // what is outside the quads, [a, first) and [last, b): ahead of them, as a round trip behind them would be one more
    const int64_t head = first - a, left = head + (b - last);
    nw = (int)min((int64_t)NW, (max((last - first) / 4, left) + 63) / 64);
    for (int64_t k0 = threadIdx.x; k0 < left; k0 += IS_LANES) {
#pragma unroll
      for (int v = 0; v < V; ++v) {
        const int64_t k = k0 + v * NT;
        if (k >= left) continue;
        const int64_t i = k < head ? a + k : last + (k - head);
        const float w = is_weight(lp_pi[i], lp_mu[i], c, exp2_64, s1[v], s2[v]);
        if (W) w_out[i] = w;
      }
    }
    for (; i0 < last; i0 += 4 * IS_LANES) {
      f32x4 ph[V], mh[V];
#pragma unroll
      for (int v = 0; v < V; ++v) { ph[v] = p[v]; mh[v] = m[v]; }
      load(i0 + 4 * IS_LANES);
#pragma unroll
      for (int v = 0; v < V; ++v) {
        const int64_t i = i0 + v * 4 * NT;
        if (i >= last) continue;
        f32x4 w;
#pragma unroll
        for (int e = 0; e < 4; ++e) w[e] = is_weight(ph[v][e], mh[v][e], c, exp2_64, s1[v], s2[v]);
        if (W) *(f32x4 *)(w_out + i) = w;
      }
    }
  }
#pragma unroll
  for (int v = 0; v < V; ++v) {
    const int wave = (int)(threadIdx.x >> 6) + v * (NT / 64);   // of the lanes
    if (wave >= nw) continue;
    s1[v] = wave_sum(s1[v]);
    s2[v] = wave_sum(s2[v]);
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
template <int NT>
__global__ __launch_bounds__(NT) void is_total_kernel(const double *__restrict__ seq_sums,
                                                      const int64_t *__restrict__ offsets, int n_seq,
                                                      double *__restrict__ totals) {
  __shared__ double red[2 * (NT / 64)];
  const int64_t n = offsets[n_seq] - offsets[0];
  double s1 = 0.0, s2 = 0.0;
  for (int s = threadIdx.x; s < n_seq; s += 4 * NT) {
    double v1[4], v2[4];   // the loads of four sequences are issued together
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const double *sums = seq_sums + 2 * (int64_t)min(s + u * NT, n_seq - 1);
      v1[u] = sums[0];
      v2[u] = sums[1];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (s + u * NT < n_seq) { s1 += v1[u]; s2 += v2[u]; }
  }
  s1 = wave_sum(s1);
  s2 = wave_sum(s2);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (lane == 0) { red[2 * wave] = s1; red[2 * wave + 1] = s2; }
  __syncthreads();
  if (threadIdx.x != 0) return;
  s1 = s2 = 0.0;
#pragma unroll
  for (int w = 0; w < NT / 64; ++w) { s1 += red[2 * w]; s2 += red[2 * w + 1]; }
  totals[0] = s1;
  totals[1] = s2;
  totals[2] = n > 0 ? s1 * s1 / ((double)n * s2) : __longlong_as_double(0x7FF8000000000000LL);
}

}  // namespace

int launch_is_ess(const float *lp_pi, const float *lp_mu, const int64_t *offsets, int n_seq, double c, float *w_out,
                  double *seq_sums, double *ess_seq, double *totals, hipStream_t s) {
  if (n_seq < 1) return -1;
  // 512 threads finish the longest sequences sooner, 256 let more workgroups run: 512 and 256, first kernel, 1500 sequences of 4096 tokens on average
  // 17.3 and 20.2 us, 2048 of 1000 8.9 and 9.6, 4096 of 100 7.0 and 6.7, 8192 of 100 11.7 and 10.1
  auto launch = [&](auto kernel, int nt) { hipLaunchKernelGGL(kernel, dim3(n_seq), dim3(nt), 0, s, lp_pi, lp_mu, offsets, c, w_out, seq_sums, ess_seq); };
  if (n_seq <= IS_MANY) {
    if (w_out) launch(is_seq_kernel<512, true>, 512); else launch(is_seq_kernel<512, false>, 512);
  } else {
    if (w_out) launch(is_seq_kernel<256, true>, 256); else launch(is_seq_kernel<256, false>, 256);
  }
  if (n_seq <= 2048) hipLaunchKernelGGL(is_total_kernel<256>, dim3(1), dim3(256), 0, s, seq_sums, offsets, n_seq, totals);
  else hipLaunchKernelGGL(is_total_kernel<1024>, dim3(1), dim3(1024), 0, s, seq_sums, offsets, n_seq, totals);
  return hipGetLastError() == hipSuccess ? 0 : -7;
}

}  // namespace pl
