// Small row-wise kernels of the decode step: the kernel that begins a step (metadata, work list, rotary tables,
// embedding gather + RMSNorm), residual add (summing split-K partials) + RMSNorm, rotary + KV-cache append.
#include "attn_worklist.h"
#include "pl_common.h"

namespace pl {
namespace {

constexpr int BEGIN_LIST = 512;   // most sequences of a step (threads of the workgroup that builds its list)


// Root mean square of a row, inverted.  A row's squares are added up in an order that its length decides: in every group of 64 values (one per lane) lanes
// 32, 16, ... 1 apart, then the groups in order.  v: the lane's values of N groups, number n * waves + its wavefront; at most G.
// (The root and the divisions in full: the instruction for an inverted root and a product with 1 / d, each up to an ulp off, take 0.15 us less at rows of
// 1536 values and 0.27 at 3584.)
template <int G, int N>
__device__ inline float inverse_rms(const float (&v)[N], int waves, int d, float eps) {
  __shared__ __attribute__((aligned(16))) float red[G];
#pragma unroll
  for (int n = 0; n < N; ++n) {
    float s = with_xor16(with_xor32(v[n], OpSum{}), OpSum{});
    s += dpp<DPP_ROR8>(s);
    s += dpp<DPP_ROR4>(s);   // (what is 8 apart is the same by now)
    s += dpp<DPP_XOR2>(s);
    s += dpp<DPP_XOR1>(s);
    if ((threadIdx.x & 63) == 0) red[n * waves + (threadIdx.x >> 6)] = s;
  }
  __syncthreads();
  float ss = 0.f;
#pragma unroll
  for (int i = 0; i < G; i += 4) {
    const f32x4 r = *(const f32x4 *)&red[i];
#pragma unroll
    for (int e = 0; e < 4; ++e) ss += i + e < N * waves ? r[e] : 0.f;
  }
  return 1.0f / sqrtf(ss / (float)d + eps);
}

// theta^(-2i/hd), and cos/sin of pos times that: in double so that long positions lose nothing
__device__ inline double rope_freq(int i, int hd, float theta) { return pow((double)theta, -2.0 * (double)i / (double)hd); }
__device__ inline void rope_angle(float *cs, int pos, int i, int hd, double freq) {
  double sn, c;
  sincos((double)pos * freq, &sn, &c);
  cs[i] = (float)c;
  cs[hd / 2 + i] = (float)sn;
}
__global__ void rope_freqs_kernel(double *freqs, int hd, float theta) { freqs[threadIdx.x] = rope_freq(threadIdx.x, hd, theta); }

__device__ inline uint64_t pass_word(uint64_t mark) { return mark << PASS_CLOCK_BITS | ((uint64_t)wall_clock64() & PASS_CLOCK); }
// The end of a pass: its mark goes to the host, who may be waiting for it.
__global__ void pass_end_kernel(const uint64_t *mark_at, uint64_t *word) {
  __hip_atomic_store(word, pass_word(*mark_at), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// The beginning of a step or pass, one launch: everything the layers need that depends on the metadata alone.
// Workgroup 0 applies a decode step's page-table changes (a pass's: brings its slot's pages and its groups of rows) and builds the attention work
// list; workgroup r + 1 brings row r: its metadata (read from the host's pinned image in a decode step and in a pass that its caller waits for,
// where a copy would be a launch of its own ahead of this one), cos/sin of its position, h = E[token], a = rmsnorm(h) * g.
// Bound by latency: one round trip to the host's memory (all of what a thread wants from there at once), one to the table or the row, the row's sum.
// Decode steps, the frequencies' powers taken anew, scans through LDS and 1024 threads: 4 rows of the tiny shape 6.3 us, 64 of the 1.5B shape 7.6, 256 of the
// 7B shape 13.1; 4.1, 5.2 and 7.4 with an approximate root, which is 0.1 to 0.5 us less than the full one (under a trace 4.8, 7.0 and 11.9, now 4.8, 7.2 and 12.4).
// ONE: a pass over one slot's rows, whose metadata is the token alone: six reads per row over the bus held 3000 rows of the 1.5B shape up
// for 33 us, one leaves 14.5 (512 rows of the 7B shape 11.3 -> 10.0).
template <int NT, int NV, bool ONE>   // NV: pieces of eight elements per thread
__global__ __launch_bounds__(NT) void step_begin_kernel(StepBegin q, AttnParams p, int cap) {
  if (blockIdx.x == 0) {
    if (q.time && threadIdx.x == 0)
      __hip_atomic_store(q.time, q.mark_at ? pass_word(q.mark) : (uint64_t)wall_clock64(), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    if (q.mark_at && threadIdx.x == 0) *q.mark_at = q.mark;
    for (int i = threadIdx.x; i < q.n_pairs; i += NT) q.pairs_dst[i] = q.pairs_src[i];
    for (int i = threadIdx.x; i < q.n_table; i += NT) q.table_dst[i] = q.table_src[i];
    if (NT < BEGIN_LIST || !p.work) return;   // a pass
    const int b = min((int)threadIdx.x, p.n_seq - 1);   // (no branch between the loads)
    int n_upd = 0, at = 0, page = 0;
    const int pos = q.src.pos[b], slot = q.src.row_slot[b];
    if (q.updates) {   // one per sequence at most
      at = q.updates[2 + 2 * b];
      page = q.updates[3 + 2 * b];
      n_upd = q.updates[0];
    }
    const bool has = (int)threadIdx.x < p.n_seq;
    const int ctx = has ? pos + 1 : 0;
    if ((int)threadIdx.x < n_upd) q.page_table[at] = page;
    __syncthreads();   // the list is built from the table
    build_worklist<NT>(ctx, has ? slot : 0, q.page_table, p.work, p.tickets, p.first_item, p.n_seq, p.Hkv, p.item_tokens, p.page_tokens, p.pages_per_seq, cap,
                       p.item_tokens < p.chunk);
    return;
  }
  const int row = blockIdx.x - 1, d8 = q.d >> 3;
  int tok = q.src.input_tok[row], pos = q.first_pos + row, slot = q.one_slot, forced = -1;
  float inv_t = 0.f;
  uint64_t seq_id = 0;
  if constexpr (!ONE) {
    pos = q.src.pos[row];
    slot = q.src.row_slot[row];
    forced = q.src.forced[row];
    inv_t = q.src.inv_t[row];
    seq_id = q.src.seq_id[row];
#ifdef __HIP_DEVICE_COMPILE__
    asm volatile("" : "+s"(pos), "+s"(tok), "+s"(slot), "+s"(forced), "+s"(inv_t), "+s"(seq_id));   // one round trip for all of them
#endif
  }
  tok = min(max(tok, 0), q.vocab - 1);
  const int i = NT - 1 - (int)threadIdx.x;   // the last wavefronts, which have least of the row, take the angles
  const double freq = i < p.hd / 2 ? q.freqs[i] : 0.0;
  bf16x8 e[NV], g[NV];
  bool mine[NV];
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const int at = threadIdx.x + k * NT;
    mine[k] = at < d8;
    e[k] = g[k] = bf16x8{};
    if (mine[k]) {
      e[k] = ((const bf16x8 *)(q.embed + (int64_t)tok * q.d))[at];
      g[k] = ((const bf16x8 *)q.g)[at];
    }
  }
  if (i < p.hd / 2) rope_angle(q.cs + (int64_t)row * p.hd, pos, i, p.hd, freq);
  if (threadIdx.x == 0) {
    q.ctx_len[row] = pos + 1;
    if (q.dst.pos) {
      q.dst.row_slot[row] = slot;
      q.dst.pos[row] = pos;
      if constexpr (!ONE) {   // (nothing of a pass is sampled)
        q.dst.forced[row] = forced;
        q.dst.inv_t[row] = inv_t;
        q.dst.seq_id[row] = seq_id;
      }
    }
  }
  float ss[NV] = {};
#pragma unroll
  for (int k = 0; k < NV; ++k)
#pragma unroll
    for (int j = 0; j < 8; ++j) ss[k] += (float)e[k][j] * (float)e[k][j];
  const float r = inverse_rms<NV * NT / 64>(ss, NT / 64, q.d, q.eps);
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const int at = threadIdx.x + k * NT;
    if (!mine[k]) continue;
    bf16x8 o;
    f32x4 h0, h1;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const float v = (float)e[k][j];
      o[j] = (__bf16)(v * r * (float)g[k][j]);
      if (j < 4) h0[j] = v; else h1[j - 4] = v;
    }
    f32x4 *h = (f32x4 *)(q.h + (int64_t)row * q.d) + 2 * at;
    h[0] = h0;
    h[1] = h1;
    ((bf16x8 *)(q.a + (int64_t)row * q.d))[at] = o;
  }
}

// h[row] += sum_s parts[s][row]; a[row] = rmsnorm(h[row]) * g.  The slices are added up in slice order, their
// sum to h (a product that comes as one slice, added up the same way before, gives the same bits).
// One workgroup per row, NV 16-byte pieces per thread, as many threads as that takes; the row stays in registers between the two passes.
// Bound by its own chain (a kernel of a graph that does nothing takes 1.7 us): loads, a sum over the row, stores, and by the instructions
// on the way, so every number of slices has a kernel without branches and the sum goes through lanes.  Rows
// of 3584 floats, nine slices: 1 row 3.7 -> 3.0 us, 64 rows 4.1 -> 3.3, 256 rows 6.7 -> 5.8; of 1536, six slices, 64 rows 2.7 -> 2.2.
// JOIN: a thread's two pieces count as one of a group's 64 values.
template <int SL, int NV, bool JOIN>
__global__ __launch_bounds__(JOIN ? 1024 : 512) void resid_rmsnorm_kernel(float *h, const float *parts, int splits, const bf16_t *g, bf16_t *a, int n,
                                                                         int d, float eps, int waves) {
  const int row = blockIdx.x, d4 = d >> 2, threads = waves * 64;
  f32x4 *h4 = (f32x4 *)(h + (int64_t)row * d);
  const f32x4 *p4 = (const f32x4 *)(parts + (int64_t)row * d);
  f32x4 v[NV];
  bf16x4 gg[NV];
  float ss[JOIN ? 1 : NV] = {};
#pragma unroll
  for (int it = 0; it < NV; ++it) {
    const int idx = threadIdx.x + it * threads;
    if (it == 0 || idx < d4) {   // (NV = 1: a thread per piece)
      v[it] = h4[idx];
      gg[it] = ((const bf16x4 *)g)[idx];
      v[it] += sum_slices<SL>(p4 + idx, splits, (int64_t)n * d4);
      h4[idx] = v[it];
      float sq = v[it][0] * v[it][0];
#pragma unroll
      for (int e = 1; e < 4; ++e) sq = __builtin_fmaf(v[it][e], v[it][e], sq);
      ss[JOIN ? 0 : it] += sq;
    }
  }
  const float r = inverse_rms<NV == 1 ? 8 : 16>(ss, waves, d, eps);
#pragma unroll
  for (int it = 0; it < NV; ++it) {
    const int idx = threadIdx.x + it * threads;
    if (it == 0 || idx < d4) {
      bf16x4 o;
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = (__bf16)(v[it][e] * r * (float)gg[it][e]);
      ((bf16x4 *)(a + (int64_t)row * d))[idx] = o;
    }
  }
}

// The rotary tables alone, and the attention length of the step (pos + 1): fp32 test build.
__global__ void rope_tables_kernel(const int32_t *pos, float *cs, int32_t *ctx_len, int n, int hd, float theta) {
  const int half = hd / 2;
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= n * half) return;
  const int row = idx / half, i = idx % half;
  rope_angle(cs + (int64_t)row * hd, pos[row], i, hd, rope_freq(i, hd, theta));
  if (i == 0) ctx_len[row] = pos[row] + 1;
}

// qkv (fp32, split-K partials) -> rotated q (bf16), rotated k and v into the row's cache page.
// One thread per four consecutive rotated pairs (i .. i + 3 with their partners half + i ..) of a row, 16-byte
// loads.  The page is looked up by scalar loads while the vectors are on their way.
// BLOCKS (a pass): v goes eight rows at a time where they are eight consecutive positions from a multiple of eight on, whose elements
// of one dimension are 16 bytes of the V block: grid rows n .. n + groups - 1, a thread per four dimensions of the eight.
// 1.5B shape, 3000 rows 13.4 us with 2-byte stores of v.
template <int SL, bool BLOCKS>
__global__ __launch_bounds__(256) void rope_append_kernel(const float *qkv, int splits, const float *cs, const int32_t *pos,
                                                          const int32_t *row_slot, const int32_t *page_table, bf16_t *q_out,
                                                          bf16_t *kv_layer, int n, int Hq, int Hkv, int hd, int page_tokens,
                                                          int pages_per_seq) {
  const int half = hd / 2, quads = half / 4, width = (Hq + 2 * Hkv) * hd;
  const int64_t page_elems = (int64_t)2 * page_tokens * hd, stride = (int64_t)n * (width / 4);
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  int row = blockIdx.y;
  bool v_alone = true;   // this row's v goes by itself
  if constexpr (BLOCKS) {
    const bool group = row >= n;
    const int r0 = group ? (row - n) * 8 : row & ~7;
    bool eight = r0 + 8 <= n && pos[r0] % 8 == 0;
    if (eight)
#pragma unroll
      for (int r = 1; r < 8; ++r) eight &= pos[r0 + r] == pos[r0] + r && row_slot[r0 + r] == row_slot[r0];
    v_alone = !eight;
    if (group) {
      if (!eight || idx >= Hkv * hd / 4) return;
      const int p = pos[r0], page = page_table[(int64_t)row_slot[r0] * pages_per_seq + p / page_tokens], hv = idx / (hd / 4), dim = idx % (hd / 4) * 4;
      const f32x4 *src = (const f32x4 *)(qkv + (int64_t)r0 * width + (Hq + Hkv + hv) * hd + dim);
      bf16x8 o[4];
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        const f32x4 x = sum_slices<SL>(src + r * (width / 4), splits, stride);
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e][r] = (__bf16)x[e];
      }
      bf16_t *vb = kv_layer + ((int64_t)page * Hkv + hv) * page_elems + (int64_t)page_tokens * hd + v_elem_offset(p % page_tokens, dim, hd);
#pragma unroll
      for (int e = 0; e < 4; ++e) *(bf16x8 *)(vb + e * 8) = o[e];
      return;
    }
  }
  if (idx >= (Hq + (v_alone ? 2 : 1) * Hkv) * quads) return;
  const int hh = idx / quads, i = (idx % quads) * 4;
  const int p = pos[row], page = page_table[(int64_t)row_slot[row] * pages_per_seq + p / page_tokens], t = p % page_tokens;
  const f32x4 *src = (const f32x4 *)(qkv + (int64_t)row * width + hh * hd + i);
  const f32x4 c = *(const f32x4 *)(cs + (int64_t)row * hd + i), sn = *(const f32x4 *)(cs + (int64_t)row * hd + half + i);
  const f32x4 x1 = sum_slices<SL>(src, splits, stride), x2 = sum_slices<SL>(src + half / 4, splits, stride);
  bf16x4 lo, hi;   // elements i .. i + 3 and half + i .. half + i + 3 of the head
  if (hh < Hq + Hkv) {
    rotate_pairs(x1, x2, c, sn, lo, hi);
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) { lo[e] = (__bf16)x1[e]; hi[e] = (__bf16)x2[e]; }
  }
  if (hh < Hq) {
    bf16_t *q = q_out + ((int64_t)row * Hq + hh) * hd;
    *(bf16x4 *)(q + i) = lo;
    *(bf16x4 *)(q + half + i) = hi;
    return;
  }
  if (hh < Hq + Hkv) {
    // four consecutive dims of a token (i is a multiple of 4) are contiguous in the K block
    bf16_t *kb = kv_layer + ((int64_t)page * Hkv + (hh - Hq)) * page_elems;
    *(bf16x4 *)(kb + k_elem_offset(t, i, hd)) = lo;
    *(bf16x4 *)(kb + k_elem_offset(t, half + i, hd)) = hi;
  } else {
    bf16_t *vb = kv_layer + ((int64_t)page * Hkv + (hh - Hq - Hkv)) * page_elems + (int64_t)page_tokens * hd;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      vb[v_elem_offset(t, i + e, hd)] = lo[e];
      vb[v_elem_offset(t, half + i + e, hd)] = hi[e];
    }
  }
}

// Read-only stream over a buffer (16-byte loads, 8 independent loads in flight per lane): measures
// what HBM delivers to a kernel that does nothing but read.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
template <bool NT>
__global__ __launch_bounds__(256) void stream_read_kernel(const u32x4 *__restrict__ p, uint32_t *sink, int64_t n_per_wg) {
  const u32x4 *base = p + (int64_t)blockIdx.x * n_per_wg;
  u32x4 acc = {0, 0, 0, 0};
  for (int64_t i = threadIdx.x; i < n_per_wg; i += 256 * 8) {
    u32x4 v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = NT ? __builtin_nontemporal_load(&base[i + u * 256]) : base[i + u * 256];
#pragma unroll
    for (int u = 0; u < 8; ++u) acc ^= v[u];
  }
  if ((acc.x ^ acc.y ^ acc.z ^ acc.w) == 0x9E3779B9u && sink) sink[0] = 1;   // keeps the loads alive
}

// LM head tied to the embedding table: dst = the [vocab, d] row-major table in the layout the LM-head
// GEMM streams (bf16: MFMA operand order, 16-byte pieces of 8 consecutive columns; fp32 build: a plain copy).
__global__ void tie_lm_head_kernel(const bf16x8 *__restrict__ embed, bf16x8 *__restrict__ dst, int vocab, int d) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;   // one 8-column piece
  const int d8 = d >> 3;
  if (idx >= (int64_t)vocab * d8) return;
  const int r = (int)(idx / d8), c = (int)(idx % d8) * 8;
  const int64_t o = ((int64_t)(c / 64) * (vocab / 32) + r / 32) * 2048 + ((c % 32) / 8) * 512 + ((c % 64) / 32) * 256 + (r % 32) * 8;
  dst[o >> 3] = embed[idx];
}

__global__ void fill_u32_kernel(uint32_t *p, uint32_t v, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) p[i] = v;
}

}  // namespace

static inline int ok() { return hipGetLastError() == hipSuccess ? 0 : -7; }

int launch_step_begin(const StepBegin &q, const AttnParams &p, int cap, hipStream_t s) {
  if (p.n_seq <= 0) return 0;
  if ((p.work && p.n_seq > BEGIN_LIST) || q.d > 8192 || ((uintptr_t)p.work & 31)) return -1;
  // the work list's threads; the rows of a pass no more than they have pieces (1536 wide: 1000 rows 11 us by 1024 threads, 3000 rows 14 by 256)
  auto launch = [&](auto kernel, int nt) { hipLaunchKernelGGL(kernel, dim3(p.n_seq + 1), dim3(nt), 0, s, q, p, cap); };
  auto shape = [&](auto ONE) {
    constexpr bool one = decltype(ONE)::value;
    if (q.d > 4096) launch(step_begin_kernel<512, 2, one>, 512);
    else if (p.work || q.d > 2048) launch(step_begin_kernel<512, 1, one>, 512);
    else launch(step_begin_kernel<256, 1, one>, 256);
  };
  if (q.pairs_src) shape(std::true_type{}); else shape(std::false_type{});
  return ok();
}

int launch_pass_end(const uint64_t *mark_at, uint64_t *word, hipStream_t s) {
  hipLaunchKernelGGL(pass_end_kernel, dim3(1), dim3(1), 0, s, mark_at, word);
  return ok();
}

int launch_rope_freqs(double *freqs, int hd, float theta, hipStream_t s) {
  hipLaunchKernelGGL(rope_freqs_kernel, dim3(1), dim3(hd / 2), 0, s, freqs, hd, theta);
  return ok();
}

int launch_resid_rmsnorm(float *h, const float *parts, int splits, const bf16_t *g, bf16_t *a, int n, int d,
                         float eps, hipStream_t s) {
  if (n <= 0) return 0;
  if (d % 256 || d > 8192 || splits < 1) return -1;
  // a piece per thread up to rows of 2048 floats, two beyond, 1024 apart from 4096 on, where they join (the order in which squares are added up depends on it) (3584 floats, nine slices, 256 rows: 5.6 us by 896 threads, 5.5 by 448)
  const int nv = d <= 2048 ? 1 : 2, waves = d > 4096 ? 16 : (d / 4 / nv + 63) / 64;
  with_slices(splits, [&](auto SL) {
    constexpr int sl = decltype(SL)::value;
    auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3(n), dim3(waves * 64), 0, s, h, parts, splits, g, a, n, d, eps, waves); };
    if (nv == 1) launch(resid_rmsnorm_kernel<sl, 1, false>);
    else if (d <= 4096) launch(resid_rmsnorm_kernel<sl, 2, false>);
    else launch(resid_rmsnorm_kernel<sl, 2, true>);
  });
  return ok();
}

int launch_rope_tables(const int32_t *pos, float *cs, int32_t *ctx_len, int n, int hd, float theta,
                       hipStream_t s) {
  if (n <= 0) return 0;
  int total = n * (hd / 2);
  hipLaunchKernelGGL(rope_tables_kernel, dim3((total + 255) / 256), dim3(256), 0, s, pos, cs, ctx_len, n, hd,
                     theta);
  return ok();
}

int launch_rope_append(const float *qkv, int splits, const float *cs, const int32_t *pos,
                       const int32_t *row_slot, const int32_t *page_table, bf16_t *q_out, bf16_t *kv_layer,
                       int n, int Hq, int Hkv, int hd, int page_tokens, int pages_per_seq, bool pass, hipStream_t s) {
  if (n <= 0) return 0;
  const int threads = (Hq + 2 * Hkv) * (hd / 8), blocks = (threads + 255) / 256, nt = ((threads + blocks - 1) / blocks + 63) / 64 * 64;
  with_slices(splits, [&](auto SL) {
    auto launch = [&](auto kernel, int rows) {
      hipLaunchKernelGGL(kernel, dim3(blocks, rows), dim3(nt), 0, s, qkv, splits, cs, pos, row_slot, page_table, q_out, kv_layer, n, Hq, Hkv, hd,
                         page_tokens, pages_per_seq);
    };
    if (pass) launch(rope_append_kernel<decltype(SL)::value, true>, n + n / 8);
    else launch(rope_append_kernel<decltype(SL)::value, false>, n);
  });
  return ok();
}

int64_t launch_stream_read(const void *p, int64_t nbytes, uint32_t *sink, bool nontemporal, hipStream_t s) {
  const int wgs = 8192;
  int64_t n_per_wg = nbytes / 16 / wgs / 2048 * 2048;
  if (n_per_wg <= 0) return 0;
  if (nontemporal)
    hipLaunchKernelGGL(stream_read_kernel<true>, dim3(wgs), dim3(256), 0, s, (const u32x4 *)p, sink, n_per_wg);
  else
    hipLaunchKernelGGL(stream_read_kernel<false>, dim3(wgs), dim3(256), 0, s, (const u32x4 *)p, sink, n_per_wg);
  return hipGetLastError() == hipSuccess ? n_per_wg * 16 * wgs : -7;
}

int launch_tie_lm_head(const void *embed, void *lm_head, int vocab, int d, bool f32, hipStream_t s) {
  if (f32) return hipMemcpyAsync(lm_head, embed, (size_t)vocab * d * 4, hipMemcpyDeviceToDevice, s) == hipSuccess ? 0 : -7;
  const int64_t pieces = (int64_t)vocab * (d / 8);
  hipLaunchKernelGGL(tie_lm_head_kernel, dim3((unsigned)((pieces + 255) / 256)), dim3(256), 0, s, (const bf16x8 *)embed,
                     (bf16x8 *)lm_head, vocab, d);
  return ok();
}

int launch_fill_u32(uint32_t *p, uint32_t v, int64_t n, hipStream_t s) {
  if (n <= 0) return 0;
  int64_t blocks = (n + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(fill_u32_kernel, dim3((unsigned)blocks), dim3(256), 0, s, p, v, n);
  return ok();
}

}  // namespace pl
