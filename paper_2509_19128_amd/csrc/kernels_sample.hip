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
#include <type_traits>
#pragma clang fp contract(off)

namespace pl {
namespace {

constexpr int SLICE = 8192;   // vocabulary entries per workgroup

// a ^ b ^ c as one instruction
__device__ inline uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
#ifdef __HIP_DEVICE_COMPILE__
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
#else
  return a ^ b ^ c;
#endif
}
__device__ inline void philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0,
                                     uint32_t k1, uint32_t out[4]) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    if (r) { k0 += 0x9E3779B9u; k1 += 0xBB67AE85u; }
    const uint64_t p0 = (uint64_t)c0 * 0xD2511F53u, p1 = (uint64_t)c2 * 0xCD9E8D57u;   // one instruction each
    const uint32_t hi0 = (uint32_t)(p0 >> 32), lo0 = (uint32_t)p0, hi1 = (uint32_t)(p1 >> 32), lo1 = (uint32_t)p1;
    c0 = xor3(hi1, c1, k0); c1 = lo1; c2 = xor3(hi0, c3, k1); c3 = lo0;
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

__device__ inline void finish_row(const SampleParams &p, int row, const Part &v, int forced, float inv_t) {
  const int tok = min(max(forced < 0 ? v.besti : forced, 0), p.vocab - 1);
  const float z = __fmul_rn(p.logits[(int64_t)row * p.vocab + tok], inv_t);
  const float lp = (z - v.mx) - logf(v.sum);
  if (p.results) {   // the host is waiting for these words
    __hip_atomic_store(&p.results[row].time, (uint64_t)wall_clock64(), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(&p.results[row].token_logprob, (uint64_t)__float_as_uint(lp) << 32 | (uint32_t)tok, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  } else {
    p.token[row] = tok;
    p.logprob[row] = lp;
  }
  if (p.last_tok) p.last_tok[p.row_slot[row]] = tok;
}

// One slice of one row; NT threads keep its entries in registers (SLICE / NT of each).
// Bound: vector arithmetic, then the 4 bytes per entry.  The two specified logarithms of the noise (about 60 operations)
// are evaluated only where they can matter.  y = z + g is largest where x / -log u is, with x = e^(z - max), and with
// t = 1 - u (exact) t <= -log u <= t / (1 - t): so x / t bounds an entry from above, and the slice's best is no less than
// the largest x / t minus 1, nor than 1 / 16.7 (the entry with x = 1 and the least noise).  x / t is compared by `key`, the difference
// of the two floats' bits, which is 2^23 log2(x / t) within KEY_ERROR.  Only entries whose key can reach that bar are
// computed as specified (about one per slice; their random words are drawn again).  KEY_SLACK covers the rounding of x and of y
// as long as |max| <= BOUND_MAX; slices beyond that, whose maximum is infinite or that hold NaNs compute every entry.
// The sum of exponentials does not depend on NT, so a row's log-prob does not depend on how many rows share the
// call: all exponentials are relative to the slice's maximum, and they are added up as SUM_LANES threads of
// SUM_LANES / 64 wavefronts would, whatever number of these a thread takes over.
// 256 x 152064, whole call, the merge launch included: 35 us (4.4 TB/s) against 54 with the bounds by logarithms, the best entry of every lane
// computed, and two multiplications per product (a product is one instruction now, v_mad_u64_u32, 5.6 cycles where the two
// took 9.7; fused multiply-adds in double precision, three per product, gave 55 us); 82-93 us with every entry's noise evaluated.
constexpr float KEY_ERROR = 0.088f, KEY_SLACK = 0.004f;   // of log2: 0.0861 per difference of bits and logarithm
constexpr int KEY_MOST = 25 << 23;                        // beyond any key of numbers: x <= 1, t >= 2^-24
constexpr int SUM_LANES = 1024;
constexpr float BOUND_MAX = 1024.f;
template <int NT, bool ONE, int Q = SLICE / NT / 4>   // ONE: a row is one slice; Q: groups of four entries per thread (half of them: a row of half a slice)
__global__ __launch_bounds__(NT) void sample_slice_kernel(SampleParams p, int nslice) {
  constexpr int V = SUM_LANES / NT;   // lanes of the sum per thread: lane threadIdx.x + v * NT has groups v, v + V, ...
  constexpr int NW = NT / 64;
  const int row = blockIdx.y, sl = blockIdx.x;
  const float *lg = p.logits + (int64_t)row * p.vocab;
  const float inv_t = p.inv_t[row];
  const uint64_t sid = p.seq_id[row];
  const uint32_t pos = (uint32_t)p.position[row];
  const uint32_t k0 = (uint32_t)p.seed, k1 = (uint32_t)(p.seed >> 32);
  const int forced = ONE && p.forced ? p.forced[row] : -1;
  const int beg4 = sl * (SLICE / 4) + threadIdx.x, end4 = min(p.vocab, (sl + 1) * SLICE) / 4;   // vocab is a multiple of 4
  float z[Q][4];
  auto load = [&](auto WHOLE) {   // a whole slice asks for no end
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int i4 = beg4 + q * NT;
      f32x4 v = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
      if (decltype(WHOLE)::value || i4 < end4) v = __builtin_nontemporal_load((const f32x4 *)(lg + (int64_t)i4 * 4));
      z[q][0] = v[0]; z[q][1] = v[1]; z[q][2] = v[2]; z[q][3] = v[3];
    }
  };
  if ((Q * NT * 4 == SLICE ? (sl + 1) * SLICE : Q * NT * 4) <= p.vocab) load(std::true_type{}); else load(std::false_type{});
  int key[Q][4];   // the bits of t, later the keys
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    uint32_t rnd[4];
    philox4x32_10((uint32_t)(beg4 + q * NT), pos, (uint32_t)sid, (uint32_t)(sid >> 32), k0, k1, rnd);
#pragma unroll
    for (int e = 0; e < 4; ++e)   // t = 1 - (2 k + 1) 2^-24 is exact
      key[q][e] = __float_as_int(__builtin_fmaf((float)(rnd[e] >> 9), -1.1920928955078125e-07f, 0.999999940395355224609375f));
  }
  float mx = -INFINITY;
#pragma unroll
  for (int q = 0; q < Q; ++q)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      z[q][e] = __fmul_rn(z[q][e], inv_t);
      mx = fmaxf(mx, z[q][e]);
    }
  __shared__ float s_max[NW], s_besty[NW], s_sum[SUM_LANES / 64];
  __shared__ int s_key[NW], s_besti[NW];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  mx = wave_max(mx);
  if (lane == 0) s_max[wave] = mx;
  __syncthreads();
  mx = s_max[0];
#pragma unroll
  for (int w = 1; w < NW; ++w) mx = fmaxf(mx, s_max[w]);
  int most[Q];   // largest key of a group
#pragma unroll
  for (int v = 0; v < V; ++v) {
    float sum = 0.f;
#pragma unroll
    for (int q = v; q < Q; q += V) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float x = __expf(z[q][e] - mx);   // (entries beyond the slice: exp(-inf) = 0; mx = -inf: unused)
        sum += x;
        key[q][e] = __float_as_int(x) - key[q][e];
      }
      most[q] = max(max(key[q][0], key[q][1]), max(key[q][2], key[q][3]));
    }
    sum = wave_sum(sum);
    if (lane == 0) s_sum[v * NW + wave] = sum;
  }
  int top = most[0];
#pragma unroll
  for (int q = 1; q < Q; ++q) top = max(top, most[q]);
  const int wave_top = wave_max(top);
  if (lane == 0) s_key[wave] = wave_top;
  __syncthreads();
  int slice_top = s_key[0];
#pragma unroll
  for (int w = 1; w < NW; ++w) slice_top = max(slice_top, s_key[w]);
  const float least = __builtin_amdgcn_exp2f((float)slice_top * 1.1920928955078125e-07f - KEY_ERROR) - 1.f;   // of the best's x / t
  const int bar = (int)((__builtin_amdgcn_logf(fmaxf(least, 0.0598f)) - KEY_ERROR - KEY_SLACK) * 8388608.f);
  uint32_t todo = 0;   // entries (q, e) that any lane of the wavefront has to compute
  if (wave_top >= bar) {
#pragma unroll
    for (int q = 0; q < Q; ++q)
      if (__builtin_amdgcn_ballot_w64(most[q] >= bar)) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (__builtin_amdgcn_ballot_w64(key[q][e] >= bar)) todo |= 1u << (4 * q + e);
      }
  }
  if (!(fabsf(mx) <= BOUND_MAX) || slice_top > KEY_MOST) todo = (uint32_t)((1ull << (4 * Q)) - 1);
  float by = -INFINITY;
  int bi = 0x7FFFFFFF;
  for (; todo; todo &= todo - 1) {
    const int at = __builtin_ctz(todo), i4 = beg4 + (at >> 2) * NT, e = at & 3;
    if (i4 >= end4) continue;
    const float z = __fmul_rn(lg[(int64_t)i4 * 4 + e], inv_t);
    uint32_t rnd[4];
    philox4x32_10((uint32_t)i4, pos, (uint32_t)sid, (uint32_t)(sid >> 32), k0, k1, rnd);
    const uint32_t bits = e == 0 ? rnd[0] : e == 1 ? rnd[1] : e == 2 ? rnd[2] : rnd[3];
    merge_best(by, bi, __fadd_rn(z, gumbel(bits)), i4 * 4 + e);
  }
  const float besty = wave_max(by);
  const int besti = wave_min(by == besty ? bi : 0x7FFFFFFF);
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
  if constexpr (ONE) finish_row(p, row, v, forced, inv_t);   // the whole vocabulary: nothing to merge
  else ((Part *)p.workspace)[(int64_t)row * nslice + sl] = v;
}

// Merge of a row's slices, one wavefront per row: lane s takes slice s (and s + 64, ...), then the fixed
// tree: 4.5 us for 256 x 19 slices against 11 us for one thread per row walking its slices.
__global__ __launch_bounds__(64) void sample_merge_kernel(SampleParams p, int nslice) {
  const int row = blockIdx.x;
  const Part *pp = (const Part *)p.workspace + (int64_t)row * nslice;
  const int forced = p.forced ? p.forced[row] : -1;
  const float inv_t = p.inv_t[row];
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
  if (threadIdx.x == 0) finish_row(p, row, v, forced, inv_t);
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
  // the chain of a slice as long as all workgroups run at once (two per compute unit); beyond that, 32 entries per thread share the
  // fixed work (reductions, the scan for candidates) among more of them.  1024 and 256 threads, whole call: 512 x 4096 7.7 and 9.0 us,
  // 128 x 32000 10.5 and 12.7, 26 x 152064 10.1 both, 30 x 152064 11.1 and 10.3, 128 x 152064 26.6 and 21.4.
  // A vocabulary of half a slice or less: no thread takes a group that has no entries, and a row of one slice
  // has its forced token before the draw (1 x 4096 4.2 -> 3.6 us, 64 x 4096 4.8 -> 4.2; the missing zeros of a sum change nothing).
  auto launch = [&](auto kernel, int nt) { hipLaunchKernelGGL(kernel, dim3(nslice, p.n), dim3(nt), 0, s, p, nslice); };
  const bool few = (int64_t)nslice * p.n <= 512;
  if (p.vocab <= SLICE / 2) {
    if (few) launch(sample_slice_kernel<1024, true, 1>, 1024); else launch(sample_slice_kernel<256, true, 4>, 256);
  } else if (nslice == 1) {
    if (few) launch(sample_slice_kernel<1024, true>, 1024); else launch(sample_slice_kernel<256, true>, 256);
  } else {
    if (few) launch(sample_slice_kernel<1024, false>, 1024); else launch(sample_slice_kernel<256, false>, 256);
  }
  if (nslice > 1) hipLaunchKernelGGL(sample_merge_kernel, dim3(p.n), dim3(64), 0, s, p, nslice);
  return hipGetLastError() == hipSuccess ? 0 : -7;
}

}  // namespace pl
