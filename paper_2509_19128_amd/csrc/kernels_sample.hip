// Fused log-softmax + Gumbel-max sampler over fp32 logits.
//
// Each step draws y ~ softmax(logits / T) (Sec. 2.1 eq. 1 of the paper) and records
// log softmax(logits / T)[y], the behaviour log-prob the trainer's truncated importance weights
// divide by.  The draw is argmax_i (z_i + g_i) with g_i = -log(-log u_i) and u_i from
// Philox4x32-10 keyed by (seed; vocabulary index / 4, position, sequence id).  The decision is made
// in fp32 with a fixed operation order (plain multiplies and adds, no fused multiply-add: this file
// is compiled with floating-point contraction off), so it can be reproduced exactly elsewhere:
//   u = (2 (bits >> 9) + 1) 2^-24;  z = logit * inv_T;  y = z + -LOG(-LOG(u));  lowest index wins ties
//   LOG(x): e = exponent - 127, m = mantissa in [1,2); if bits(m) > 0x3FB504F3 { m *= 0.5; e += 1 }
//           f = m - 1; p = C8; p = p f + Cj (j = 7..0); f2 = f f; r = (f2 f) p; r += -0.5 f2;
//           r += e LN2_LO; r += f; LOG = e LN2_HI + r
// One pass over the logits: every workgroup scans a slice of one row keeping (max z, sum exp,
// best y, its index); a second small kernel merges the slices of a row in a fixed order (a vocabulary
// of one slice needs none).
#include "pl_common.h"

#include <mutex>
#pragma clang fp contract(off)

namespace pl {
namespace {

constexpr int SLICE = 8192;   // vocabulary entries per workgroup

__device__ inline void philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0,
                                     uint32_t k1, uint32_t out[4]) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    if (r) { k0 += 0x9E3779B9u; k1 += 0xBB67AE85u; }
    const uint32_t hi0 = __umulhi(0xD2511F53u, c0), lo0 = 0xD2511F53u * c0;
    const uint32_t hi1 = __umulhi(0xCD9E8D57u, c2), lo1 = 0xCD9E8D57u * c2;
    c0 = hi1 ^ c1 ^ k0; c1 = lo1; c2 = hi0 ^ c3 ^ k1; c3 = lo0;
  }
  out[0] = c0; out[1] = c1; out[2] = c2; out[3] = c3;
}

__device__ inline float spec_log(float x) {
#pragma clang fp contract(off)
  const uint32_t bits = __float_as_uint(x);
  int e = (int)(bits >> 23) - 127;
  uint32_t mb = (bits & 0x007FFFFFu) | 0x3F800000u;
  float m = __uint_as_float(mb);
  if (mb > 0x3FB504F3u) { m = m * 0.5f; e += 1; }
  const float f = m - 1.0f;
  const float C[9] = {__uint_as_float(0x3EAAAAAAu), __uint_as_float(0xBE7FFFFEu), __uint_as_float(0x3E4CCEADu),
                      __uint_as_float(0xBE2AADA5u), __uint_as_float(0x3E11E90Du), __uint_as_float(0xBDFE7A63u),
                      __uint_as_float(0x3DEF5141u), __uint_as_float(0xBDEB1ADEu), __uint_as_float(0x3D8EC753u)};
  float p = C[8];
#pragma unroll
  for (int j = 7; j >= 0; --j) {
    p = __fmul_rn(p, f);
    p = __fadd_rn(p, C[j]);
  }
  const float f2 = __fmul_rn(f, f);
  float r = __fmul_rn(__fmul_rn(f2, f), p);
  r = __fadd_rn(r, __fmul_rn(-0.5f, f2));
  const float ef = (float)e;
  r = __fadd_rn(r, __fmul_rn(ef, __uint_as_float(0x35BFBE8Eu)));
  r = __fadd_rn(r, f);
  return __fadd_rn(__fmul_rn(ef, __uint_as_float(0x3F317200u)), r);
}

__device__ inline float gumbel(uint32_t bits) {
  const float k = (float)(bits >> 9);
  const float u = __fmul_rn(__fadd_rn(__fmul_rn(k, 2.0f), 1.0f), 5.9604644775390625e-08f);
  return -spec_log(-spec_log(u));
}

struct Part { float mx, sum, besty; int32_t besti; };

__device__ inline void merge_best(float &by, int &bi, float y, int i) {
  if (y > by || (y == by && i < bi)) { by = y; bi = i; }
}

// Upper bound of gumbel(bits) from one hardware logarithm.  With t = 1 - u (exact: 2 k' + 1 with k' the
// complement of k) -log u >= t, so -log(-log u) <= -log t.  The slack covers the rounding of the specified
// logarithm (2e-6 at the largest value, 16.6) and of the hardware's.
__device__ inline float gumbel_bound(uint32_t bits) {
  const float k = (float)((bits >> 9) ^ 0x7FFFFFu);
  const float t = __fmul_rn(__fadd_rn(__fmul_rn(k, 2.0f), 1.0f), 5.9604644775390625e-08f);
  return __builtin_amdgcn_logf(t) * -0.693147180559945f + 1.0e-3f;
}

// All 64 lanes' parts in one, in a fixed order; every lane ends with the result.  A part without a finite or
// infinite maximum (all entries -inf) contributes nothing to the sum.
__device__ inline Part merge_wave(const Part &v) {
  Part r;
  r.mx = wave_max(v.mx);
  r.sum = wave_sum(v.mx > -INFINITY ? v.sum * __expf(v.mx - r.mx) : 0.f);
  r.besty = wave_max(v.besty);
  r.besti = wave_min(v.besty == r.besty ? v.besti : 0x7FFFFFFF);
  return r;
}
constexpr Part NO_PART = {-INFINITY, 0.f, -INFINITY, 0x7FFFFFFF};

__device__ inline void finish_row(const SampleParams &p, int row, const Part &v) {
  int tok = p.forced ? p.forced[row] : -1;
  if (tok < 0) tok = v.besti;
  tok = min(max(tok, 0), p.vocab - 1);
  const float z = __fmul_rn(p.logits[(int64_t)row * p.vocab + tok], p.inv_t[row]);
  p.token[row] = tok;
  p.logprob[row] = (z - v.mx) - logf(v.sum);
  if (p.last_tok) p.last_tok[p.row_slot[row]] = tok;
}

// One slice of one row; NT threads keep its logits and random words in registers (SLICE / NT of each).
// Bound: vector arithmetic, not the 4 bytes per entry.  Philox takes 40 quarter-rate multiplies per four
// entries; the two specified logarithms of the noise (about 60 operations) are therefore evaluated only
// where they can matter: each lane first takes the entry with the largest upper bound z + gumbel_bound,
// computes that one exactly, the wavefront's largest exact value becomes the bar, and only entries whose
// bound reaches the bar (about one in a thousand) are computed as well.  An entry below the bar cannot
// win or tie: bound >= exact value entry by entry, rounding included (rounding is monotone).
// The sum of exponentials does not depend on NT, so a row's log-prob does not depend on how many rows share the
// call: all exponentials are relative to the slice's maximum, and they are added up as SUM_LANES threads of
// SUM_LANES / 64 wavefronts would, whatever number of these a thread takes over (1.6 us of the next line's 52).
// 256 x 152064, whole call: 52 us (3.0 TB/s) against 82-93 us with every entry's noise evaluated and a branchy online sum;
// 4 x 4096: 5 us against 8.6.  One 64-bit multiply-add per product (v_mad_u64_u32) is slower than the
// high/low pair (73 against 61 us before the reductions below), four wavefronts per SIMD spill (69), 16 entries
// per thread cost 63.
constexpr int SUM_LANES = 1024;
template <int NT>
__global__ __launch_bounds__(NT) void sample_slice_kernel(SampleParams p, int nslice) {
  constexpr int Q = SLICE / NT / 4;   // groups of four entries per thread
  constexpr int V = SUM_LANES / NT;   // lanes of the sum per thread: lane threadIdx.x + v * NT has groups v, v + V, ...
  constexpr int NW = NT / 64;
  const int row = blockIdx.y, sl = blockIdx.x;
  const float *lg = p.logits + (int64_t)row * p.vocab;
  const float inv_t = p.inv_t[row];
  const uint64_t sid = p.seq_id[row];
  const uint32_t pos = (uint32_t)p.position[row];
  const uint32_t k0 = (uint32_t)p.seed, k1 = (uint32_t)(p.seed >> 32);
  const int beg4 = sl * (SLICE / 4) + threadIdx.x, end4 = min(p.vocab, (sl + 1) * SLICE) / 4;   // vocab is a multiple of 4
  float z[Q][4];
  uint32_t rnd[Q][4];
  float mx = -INFINITY, first = -INFINITY, second = -INFINITY;   // largest two upper bounds
  int fi = -1;
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int i4 = beg4 + q * NT;
    float4 v = make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
    if (i4 < end4) v = *(const float4 *)(lg + (int64_t)i4 * 4);
    z[q][0] = v.x; z[q][1] = v.y; z[q][2] = v.z; z[q][3] = v.w;
  }
  uint32_t best_bits = 0;
  float best_z = 0.f;
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int i4 = beg4 + q * NT;
    philox4x32_10((uint32_t)i4, pos, (uint32_t)sid, (uint32_t)(sid >> 32), k0, k1, rnd[q]);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      z[q][e] = __fmul_rn(z[q][e], inv_t);
      mx = fmaxf(mx, z[q][e]);
      const float ub = __fadd_rn(z[q][e], gumbel_bound(rnd[q][e]));
      second = fmaxf(second, fminf(first, ub));
      if (ub > first) { first = ub; fi = i4 * 4 + e; best_bits = rnd[q][e]; best_z = z[q][e]; }
    }
  }
  __shared__ float s_max[NW], s_besty[NW], s_sum[SUM_LANES / 64];
  __shared__ int s_besti[NW];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  mx = wave_max(mx);
  if (lane == 0) s_max[wave] = mx;
  float by = -INFINITY;
  int bi = 0x7FFFFFFF;
  if (fi >= 0) merge_best(by, bi, __fadd_rn(best_z, gumbel(best_bits)), fi);
  const float bar = wave_max(by);
  if (second >= bar) {
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int i4 = beg4 + q * NT;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (i4 < end4 && __fadd_rn(z[q][e], gumbel_bound(rnd[q][e])) >= bar)
          merge_best(by, bi, __fadd_rn(z[q][e], gumbel(rnd[q][e])), i4 * 4 + e);
    }
  }
  const float besty = wave_max(by);
  const int besti = wave_min(by == besty ? bi : 0x7FFFFFFF);
  __syncthreads();
  mx = s_max[0];
#pragma unroll
  for (int w = 1; w < NW; ++w) mx = fmaxf(mx, s_max[w]);
#pragma unroll
  for (int v = 0; v < V; ++v) {
    float sum = 0.f;
#pragma unroll
    for (int q = v; q < Q; q += V)
#pragma unroll
      for (int e = 0; e < 4; ++e) sum += __expf(z[q][e] - mx);   // (entries beyond the slice: exp(-inf) = 0; mx = -inf: unused)
    sum = wave_sum(sum);
    if (lane == 0) s_sum[v * NW + wave] = sum;
  }
  if (lane == 0) { s_besty[wave] = besty; s_besti[wave] = besti; }
  __syncthreads();
  if (threadIdx.x >= 64) return;
  Part v;
  v.mx = mx;
  v.sum = wave_sum(lane < SUM_LANES / 64 ? s_sum[lane] : 0.f);
  by = lane < NW ? s_besty[lane] : -INFINITY;
  v.besty = wave_max(by);
  v.besti = wave_min(lane < NW && by == v.besty ? s_besti[lane] : 0x7FFFFFFF);
  if (threadIdx.x != 0) return;
  if (nslice == 1) finish_row(p, row, v);   // the whole vocabulary: nothing to merge
  else ((Part *)p.workspace)[(int64_t)row * nslice + sl] = v;
}

// Merge of a row's slices, one wavefront per row: lane s takes slice s (and s + 64, ...), then the fixed
// tree: 4.5 us for 256 x 19 slices against 11 us for one thread per row walking its slices.
__global__ __launch_bounds__(64) void sample_merge_kernel(SampleParams p, int nslice) {
  const int row = blockIdx.x;
  const Part *pp = (const Part *)p.workspace + (int64_t)row * nslice;
  Part v = NO_PART;
  for (int s = threadIdx.x; s < nslice; s += 64) {
    const Part w = pp[s];
    const float M = fmaxf(v.mx, w.mx);
    float sum = v.mx > -INFINITY ? v.sum * __expf(v.mx - M) : 0.f;
    if (w.mx > -INFINITY) sum += w.sum * __expf(w.mx - M);
    v.mx = M;
    v.sum = sum;
    merge_best(v.besty, v.besti, w.besty, w.besti);
  }
  v = merge_wave(v);
  if (threadIdx.x == 0) finish_row(p, row, v);
}

}  // namespace

// ---- slice partials kept in the library's own device memory, for callers that cannot allocate ------
namespace {
constexpr int STATIC_MAX_ROWS = 512, STATIC_MAX_VOCAB = 262144;
constexpr int64_t STATIC_SCRATCH_BYTES = (int64_t)STATIC_MAX_ROWS * (STATIC_MAX_VOCAB / SLICE) * (int64_t)sizeof(Part);   // 256 KiB
// One copy per GPU the library runs on, held until the process ends.  In host code this name is only a
// handle for hipGetSymbolAddress: the address kernels use is looked up once per device below.
static __device__ __align__(256) unsigned char scratch[STATIC_SCRATCH_BYTES];
constexpr int MAX_DEVICES = 64;
void *g_scratch_ptr[MAX_DEVICES] = {};
std::mutex g_scratch_mu;
}  // namespace

// Device address of the current device's scratch array (looked up on the first call on that device)
// and the largest launch it serves.  Returns 0, -1 if the shape does not fit, -7 on a HIP error.
int sample_static_workspace(int n, int vocab, void **ptr) {
  if (n < 1 || n > STATIC_MAX_ROWS || vocab < 1 || vocab > STATIC_MAX_VOCAB ||
      sample_workspace_bytes(n, vocab) > STATIC_SCRATCH_BYTES)
    return -1;
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return -7;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void *p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return -7;
    g_scratch_ptr[dev] = p;
  }
  *ptr = g_scratch_ptr[dev];
  return 0;
}
void sample_static_limits(int *max_rows, int *max_vocab) { *max_rows = STATIC_MAX_ROWS; *max_vocab = STATIC_MAX_VOCAB; }

int64_t sample_workspace_bytes(int n, int vocab) {
  return (int64_t)n * ((vocab + SLICE - 1) / SLICE) * (int64_t)sizeof(Part);
}

int launch_sample(const SampleParams &p, hipStream_t s) {
  if (p.n <= 0) return 0;
  if (p.vocab % 4) return -1;
  const int nslice = (p.vocab + SLICE - 1) / SLICE;
  // Few slices leave most of the chip idle whatever the workgroup does: 1024 threads of 8 entries each shorten
  // the chain of a slice; with two workgroups per compute unit or more, 32 entries per thread share the fixed
  // work (exact value of the lane's best entry, reductions) among more of them.
  if ((int64_t)nslice * p.n < 512)
    hipLaunchKernelGGL(sample_slice_kernel<1024>, dim3(nslice, p.n), dim3(1024), 0, s, p, nslice);
  else
    hipLaunchKernelGGL(sample_slice_kernel<256>, dim3(nslice, p.n), dim3(256), 0, s, p, nslice);
  if (nslice > 1) hipLaunchKernelGGL(sample_merge_kernel, dim3(p.n), dim3(64), 0, s, p, nslice);
  return hipGetLastError() == hipSuccess ? 0 : -7;
}

}  // namespace pl
