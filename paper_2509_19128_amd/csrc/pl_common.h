// Internal declarations shared by the engine's host code and its kernels (not part of the ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

typedef __bf16 bf16_t;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;

namespace pl {

// ---- wavefront reductions: lanes of 16 by data-parallel primitives that the combining instruction reads through, the four
// rows of 16 by row swaps (a few cycles a step, no LDS round trips); fixed order, every lane ends with the result -------------
template <typename T>
__device__ inline uint32_t lane_bits(T v) { return __builtin_bit_cast(uint32_t, v); }
#ifdef __HIP_DEVICE_COMPILE__
template <int CTRL, typename T>
__device__ inline T dpp(T v) {   // (every lane has a source: the old value and the bounds play no part)
  return __builtin_bit_cast(T, __builtin_amdgcn_update_dpp(0, (int)lane_bits(v), CTRL, 0xF, 0xF, true));
}
// op of a lane's value with that of the lane 16 (32) away
template <typename T, typename F>
__device__ inline T with_xor16(T v, F op) {
  const auto r = __builtin_amdgcn_permlane16_swap(lane_bits(v), lane_bits(v), false, false);
  const uint32_t a = r[0], b = r[1];
  return op(__builtin_bit_cast(T, a), __builtin_bit_cast(T, b));
}
template <typename T, typename F>
__device__ inline T with_xor32(T v, F op) {
  const auto r = __builtin_amdgcn_permlane32_swap(lane_bits(v), lane_bits(v), false, false);
  const uint32_t a = r[0], b = r[1];
  return op(__builtin_bit_cast(T, a), __builtin_bit_cast(T, b));
}
#else
template <int CTRL, typename T>
__device__ inline T dpp(T v) { return v; }
template <typename T, typename F>
__device__ inline T with_xor16(T v, F op) { return op(v, v); }
template <typename T, typename F>
__device__ inline T with_xor32(T v, F op) { return op(v, v); }
#endif
constexpr int DPP_XOR1 = 0xB1, DPP_XOR2 = 0x4E, DPP_HALF_MIRROR = 0x141, DPP_MIRROR = 0x140, DPP_ROR4 = 0x124, DPP_ROR8 = 0x128;
struct OpSum { __device__ float operator()(float a, float b) const { return a + b; } };
struct OpMax {
  __device__ float operator()(float a, float b) const { return fmaxf(a, b); }
  __device__ int operator()(int a, int b) const { return max(a, b); }
};
struct OpMin { __device__ int operator()(int a, int b) const { return min(a, b); } };
template <typename T, typename F>
__device__ inline T wave_reduce(T v, F op) {
  v = op(v, dpp<DPP_XOR1>(v));
  v = op(v, dpp<DPP_XOR2>(v));
  v = op(v, dpp<DPP_HALF_MIRROR>(v));
  v = op(v, dpp<DPP_MIRROR>(v));
  v = with_xor16(v, op);
  return with_xor32(v, op);
}
__device__ inline float wave_sum(float v) { return wave_reduce(v, OpSum{}); }
__device__ inline float wave_max(float v) { return wave_reduce(v, OpMax{}); }
__device__ inline int wave_max(int v) { return wave_reduce(v, OpMax{}); }
__device__ inline int wave_min(int v) { return wave_reduce(v, OpMin{}); }

// Sum of `splits` partial sums, `stride` vectors apart, in slice order.  SL > 0: exactly that many, all loads issued together and no branch between
// them; SL = 0: any number, eight loads at a time.
template <int SL>
__device__ __forceinline__ f32x4 sum_slices(const f32x4 *p, int splits, int64_t stride) {
  f32x4 y = {0.f, 0.f, 0.f, 0.f};   // (from zero, as a folded product: slices of -0 add up to 0)
  if constexpr (SL > 0) {
    f32x4 v[SL];
#pragma unroll
    for (int u = 0; u < SL; ++u) v[u] = p[u * stride];
#pragma unroll
    for (int u = 0; u < SL; ++u) y += v[u];
  } else {
    for (int s0 = 0; s0 < splits; s0 += 8) {
      f32x4 v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (s0 + u < splits) v[u] = p[(s0 + u) * stride];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (s0 + u < splits) y += v[u];
    }
  }
  return y;
}
constexpr int SLICES_MOST = 12;   // slices that have a kernel of their own
// calls f(integral constant): the number of slices, or 0 beyond MOST
template <int SL = 1, int MOST = SLICES_MOST, typename F>
void with_slices(int splits, F f) {
  if constexpr (SL > MOST) f(std::integral_constant<int, 0>{});
  else if (splits == SL) f(std::integral_constant<int, SL>{});
  else with_slices<SL + 1, MOST>(splits, f);
}

// SwiGLU of a gate and an up value, one rounding rule for every kernel that has both.  By a division: a reciprocal saves nine instructions per element
// (tiny shape, one row, 4.0 -> 3.6 us), but is up to an ulp off, and zero where the divisor is beyond 2^126 (gates below -87.3).
__device__ inline __bf16 swiglu(float g, float u) {
#ifdef __HIP_DEVICE_COMPILE__
  return (__bf16)(g / (1.f + __expf(-g)) * u);
#else
  return (__bf16)0.f;
#endif
}

// ---- KV page geometry (one layer, one page, one kv head: K block then V block) ---------------
// Tokens of a page are grouped in runs of 32 (t = 32 r + u).  Both blocks are laid out so that the
// 64 lanes of a wavefront read one MFMA operand with a single fully contiguous 1 KiB load.
__host__ __device__ inline int64_t k_elem_offset(int t, int d, int hd) {
  int r = t >> 5, u = t & 31;
  int T = (u >> 2) & 1, R = ((u >> 3) << 2) | (u & 3);
  return ((int64_t)((r * 2 + T) * (hd / 8) + d / 8)) * 128 + R * 8 + (d & 7);
}
__host__ __device__ inline int64_t v_elem_offset(int t, int d, int hd) {
  int r = t >> 5, u = t & 31;
  return ((int64_t)((r * (hd / 16) + d / 16) * 4 + (u >> 3))) * 128 + (d & 15) * 8 + (u & 7);
}

constexpr int ATTN_SUB = 512;            // tokens of a sub of an attention chunk (chunks are powers of two)
constexpr int ATTN_ML = 32;              // floats of the soft-max statistics of one part: (m, l) of up to 16 heads, one cache line
constexpr int ATTN_SPLIT_PARTS = 2048;   // most (sub, kv head) pairs of a launch whose items are subs
// Four rotated pairs (elements i .. i + 3 of the first half with the same of the second), rounded the same way by
// every kernel that rotates.
__device__ inline void rotate_pairs(f32x4 x1, f32x4 x2, f32x4 c, f32x4 s, bf16x4 &lo, bf16x4 &hi) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    lo[e] = (__bf16)__builtin_fmaf(x1[e], c[e], -__fmul_rn(x2[e], s[e]));
    hi[e] = (__bf16)__builtin_fmaf(x2[e], c[e], __fmul_rn(x1[e], s[e]));
  }
}

constexpr int ATTN_ROTATE_SLICES = 8;    // most QKV slices the attention kernel adds up itself
struct AttnParams {
  const bf16_t *q;          // [n_seq, Hq, hd], or null: the kernel rotates the QKV product's slices and appends k and v itself
  const float *qkv;         // [splits, n_seq, (Hq + 2 Hkv) hd] (q null)
  const float *cs;          // [n_seq, hd] cos | sin of the row's position (q null)
  int32_t splits;
  bf16_t *kv;               // page pool of one layer (written only with q null)
  const int32_t *page_table;// [n_slots, pages_per_seq], row = slot_of_row[row] (or row if null)
  const int32_t *ctx_len;   // [n_seq]
  const int32_t *row_slot;  // [n_seq] or null
  int32_t *work;            // work list built by launch_attention_worklist for these ctx_len, row_slot and page_table;
                            // null: none (row_slot null; max_items = n_seq * max_chunks)
  int32_t *tickets;         // [n_seq, Hkv], zero between launches (the work-list kernel clears them), or null: see attention_tickets
  int32_t *first_item;      // [n_seq] list index of a row's first item (item_tokens < chunk)
  const int32_t *groups;    // rows of a pass: {count, -, (first row, rows) ...}, each group consecutive positions of one slot
  int32_t max_items;        // upper bound on the list length, or on the number of groups (sizes the grid)
  bf16_t *out;              // [n_seq, Hq, hd]
  float *part_o;            // [n_seq, Hkv, max_chunks, G, hd]; item_tokens < chunk: [item, Hkv, 4, G, hd]
  float *part_ml;           // [n_seq, Hkv, max_chunks, ATTN_ML]; item_tokens < chunk: [item, Hkv, 4, 16, 2]
  int32_t n_seq, Hq, Hkv, hd, page_tokens, pages_per_seq, chunk, max_chunks;
  int32_t merge;            // rows span several items and the decode kernel does not merge them: launch the merge kernel
  int32_t item_tokens;      // tokens of a work item: chunk, or ATTN_SUB where attention_split says so
};
int launch_attention(const AttnParams &p, hipStream_t s, int part = 0);
bool attention_tickets(int max_chunks);
bool attention_rotates(int items, int64_t tokens, int Hq, int Hkv, int hd, int splits);
int launch_attention_rows(const AttnParams &p, hipStream_t s);
int attention_rows_per_group(int Hq, int Hkv);
int attention_apart_rows(int Hkv, int hd);
int64_t attention_worklist_ints(int64_t max_items);
bool attention_split(int chunk, int64_t total_tokens, int64_t longest_item, int64_t n_subs, int Hkv);
int launch_attention_worklist(const AttnParams &p, int cap, hipStream_t s);
int attention_chunk_tokens(int n_seq, int Hkv, int max_ctx);

// x and W are each addressed through one buffer descriptor with 32-bit byte offsets kept in signed
// registers: an operand must stay below 2 GiB (launch_gemm returns -1 beyond that).
constexpr int64_t GEMM_MAX_OPERAND_BYTES = (int64_t)1 << 31;
// tile configurations of the GEMM kernel: rows x columns of a workgroup's tile ("P": the four wavefronts
// stacked along the rows, each holding a gate and an up tile; "R": side by side along the columns)
enum { GEMM_32x256, GEMM_64x256, GEMM_128x256, GEMM_64x128, GEMM_128x128, GEMM_256x128, GEMM_64x64, GEMM_128x64,
       GEMM_32x128, GEMM_128x64P, GEMM_256x64P, GEMM_64x128R, GEMM_128x128R, GEMM_256x128R, GEMM_256x256 };
// How K is split: columns [0, n_main) in `splits` slices, columns [n_main, N) in `rem_splits` (mode 1
// only; mode 0 has n_main = N).  Chosen once per product from the largest row count (gemm_pick_split),
// so that every call adds up an output element in the same order whatever its row count.
struct GemmSplit { int splits, n_main, rem_splits; };
GemmSplit gemm_pick_split(int M_max, int N, int K, int mode);
int64_t gemm_workspace_elems(int M_max, int N, const GemmSplit &ks);
// Bytes that are read again and again but do not stay in the 256 MB last-level cache in between (a matrix a little
// larger than the cache is still mostly there: 271 MB, 76 rows, 45 us against 53 with non-temporal loads).
inline bool gemm_cold(int64_t bytes) { return bytes > (int64_t)384 << 20; }
// cold: gemm_cold of all the weights that pass between two uses of this matrix (kernels_gemm.hip: W_CACHE)
// ws: fp32 workspace of gemm_workspace_elems (mode 1 with split K, up to 128 rows), else may be null
int launch_gemm(const bf16_t *x, const bf16_t *w, void *y, float *ws, int M, int N, int K, int mode,
                const GemmSplit &ks, bool cold, hipStream_t s);
// Rows of launch_gemm_folded and of a pass.  A prompt in one pass instead of several has its tiles in few full rounds and its short
// kernels' fixed time once: 3000 rows of a layer of the 1.5B shape 530 us in three passes of 1000, 475 in one.
constexpr int GEMM_MAX_ROWS = 4096;
int launch_gemm_folded(const bf16_t *x, const bf16_t *w, void *y, int M, int N, int K, int mode, const GemmSplit &ks, hipStream_t s);
int gemm_pass_slices(int M, int N, int K, const GemmSplit &ks);
int64_t gemm_pass_elems(int R, int N, int K, const GemmSplit &ks);
// room: fp32 elements that y holds (mode 0); -1 where the call would need more
int launch_gemm_pass(const bf16_t *x, const bf16_t *w, void *y, int64_t room, int M, int N, int K, int mode, const GemmSplit &ks,
                     hipStream_t s);
int launch_gemm_cfg(int cfg, const bf16_t *x, const bf16_t *w, void *y, float *ws, int M, int N, int K, int mode,
                    int splits, int n_begin, int n_end, bool paired, bool cold, hipStream_t s);
int gemm_pick_splits(int M, int N, int K);

// A row's result as the host polls for it in pinned memory: both words differ from RESULT_PENDING once they have arrived.
struct StepResult { uint64_t token_logprob, time; };   // token | log-prob's bits << 32; wall clock
constexpr uint64_t RESULT_PENDING = ~(uint64_t)0;
struct SampleParams {
  const float *logits; int32_t n, vocab;
  const uint64_t *seq_id; const int32_t *position; const float *inv_t; const int32_t *forced;
  uint64_t seed; int32_t *token; float *logprob; void *workspace;
  int32_t *last_tok; const int32_t *row_slot;   // optional: last_tok[row_slot[row]] = token
  StepResult *results;      // optional, instead of token and logprob
};
int64_t sample_workspace_bytes(int n, int vocab);
int launch_sample(const SampleParams &p, hipStream_t s);
int sample_static_workspace(int n, int vocab, void **ptr);
void sample_static_limits(int *max_rows, int *max_vocab);

// per-step metadata, one row per occupied slot
struct StepMeta {
  int32_t *row_slot, *pos, *input_tok, *forced;
  float *inv_t;
  uint64_t *seq_id;
};
struct StepBegin {
  StepMeta src;             // where the rows' metadata is read: the host's pinned image, or the device's
  StepMeta dst;             // device copies for the kernels that follow (pos null: src is the device's)
  const int32_t *updates;   // null, or {count, -, (element of the page table, page id) ...}
  int32_t *page_table;
  const bf16_t *embed, *g;
  float *h, *cs;
  bf16_t *a;
  int32_t *ctx_len;
  const double *freqs;      // [hd / 2] rotary frequencies (launch_rope_freqs)
  int32_t d, vocab;
  float eps;
  uint64_t *time;           // null, or where the wall clock goes when the step begins (host)
  // A pass that fetches everything itself: rows of pairs and of the page table as the host has them, and a mark that launch_pass_end hands on.
  const int32_t *pairs_src, *table_src;   // null: they are on the device already
  int32_t *pairs_dst, *table_dst;
  int32_t n_pairs, n_table;
  uint64_t mark, *mark_at;                // mark_at: device
  int32_t one_slot, first_pos;            // with pairs_src: the rows are this slot's, at consecutive positions from first_pos on
};
// Words of a pass in the host's memory: its mark's low bits above the wall clock's.
constexpr int PASS_CLOCK_BITS = 40;
constexpr uint64_t PASS_CLOCK = ((uint64_t)1 << PASS_CLOCK_BITS) - 1;
int launch_pass_end(const uint64_t *mark_at, uint64_t *word, hipStream_t s);
int launch_rope_freqs(double *freqs, int hd, float theta, hipStream_t s);
int launch_step_begin(const StepBegin &q, const AttnParams &p, int cap, hipStream_t s);
int launch_resid_rmsnorm(float *h, const float *parts, int splits, const bf16_t *g, bf16_t *a, int n,
                         int d, float eps, hipStream_t s);
int launch_rope_tables(const int32_t *pos, float *cs, int32_t *ctx_len, int n, int hd, float theta,
                       hipStream_t s);
int launch_rope_append(const float *qkv, int splits, const float *cs, const int32_t *pos,
                       const int32_t *row_slot, const int32_t *page_table, bf16_t *q_out, bf16_t *kv_layer,
                       int n, int Hq, int Hkv, int hd, int page_tokens, int pages_per_seq, bool pass, hipStream_t s);
// fp32 test build (kernels_f32.hip)
int f32_launch_norm(const float *embed, const int32_t *input_tok, int vocab, const float *y, const float *g, float *h,
                    float *a, int n, int d, float eps, hipStream_t s);
int f32_launch_gemm(const float *x, const float *w, float *y, int M, int N, int K, hipStream_t s);
int f32_launch_swiglu(const float *gu, float *mid, int M, int F, hipStream_t s);
int f32_launch_rope_append(const float *qkv, const float *cs, const int32_t *pos, const int32_t *row_slot,
                           const int32_t *page_table, float *q_out, float *kv_layer, int n, int Hq, int Hkv, int hd,
                           int page_tokens, int pages_per_seq, hipStream_t s);
int f32_launch_attention(const float *q, const float *kv_layer, const int32_t *page_table, const int32_t *pos,
                         const int32_t *row_slot, float *out, int n, int Hq, int Hkv, int hd, int page_tokens,
                         int pages_per_seq, hipStream_t s);
int64_t launch_stream_read(const void *p, int64_t nbytes, uint32_t *sink, bool nontemporal, hipStream_t s);
int launch_fill_u32(uint32_t *p, uint32_t v, int64_t n, hipStream_t s);
int launch_tie_lm_head(const void *embed, void *lm_head, int vocab, int d, bool f32, hipStream_t s);
int launch_is_ess(const float *lp_pi, const float *lp_mu, const int64_t *offsets, int n_seq, double c, float *w_out,
                  double *seq_sums, double *ess_seq, double *totals, hipStream_t s);

}  // namespace pl
