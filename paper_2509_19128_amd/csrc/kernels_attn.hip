// Ragged grouped-query decode attention over the paged bf16 KV cache (gfx950).
//
// One decode step of "generate next tokens" (Alg. 2 of the paper) attends one new query per
// sequence over that sequence's whole cached history; the work is a stream of K and V bytes at a
// few flops per byte, so the kernel is built around HBM reads: every load instruction of a
// wavefront fetches one contiguous KiB that is already in MFMA operand order (the page layout is
// chosen for that), the query heads that share a kv head ride along as the 16 columns of one
// 16x16x32 MFMA so each K/V byte is read once for the whole group, and soft-max statistics are
// reduced by row swaps between lanes.  Work is split over (sequence, kv head, item of tokens).
//
// The order of a result's additions is fixed by the chunk length alone, whatever is launched: a chunk is
// cut into subs of ATTN_SUB tokens; wavefront w takes the 32-token runs w, w + 4, ... of a sub with an
// online soft-max, folds its subs in order, the four wavefronts are merged, and the chunks of a sequence
// are folded in order.  An item is a chunk, or one sub where few sequences would leave the chip idle
// (the wavefronts' partial results then go to a merge kernel that does the same folds).
#include "attn_worklist.h"
#include "pl_common.h"

#include <algorithm>
#include <type_traits>

#ifndef PL_ATTN_NS
#define PL_ATTN_NS 2   // register stages of K/V runs per wavefront where the kernel does not rotate
#endif
#ifndef PL_ATTN_CHUNK
#define PL_ATTN_CHUNK 8192   // largest number of tokens one workgroup handles
#endif

namespace pl {
namespace {

constexpr int SUB_RUNS = ATTN_SUB / 32;
static_assert(PL_ATTN_CHUNK <= 1 << 20, "a work list's keys");
typedef __attribute__((address_space(4))) int32_t scalar_i32;   // read by scalar loads

// of the four lanes that hold a column's tokens
__device__ inline float column_sum(float v) { return with_xor32(with_xor16(v, OpSum{}), OpSum{}); }
__device__ inline float column_max(float v) { return with_xor32(with_xor16(v, OpMax{}), OpMax{}); }

// (m, l, o) <- (m, l, o) folded with a later part (mi, li, oi); m is in log2 units.  A part without tokens
// has mi = -inf and changes nothing; the first part is taken over as it is.
// The operations are spelled out so that every kernel rounds them alike.
__device__ inline float fold_value(float o, float e0, float oi, float e1) { return __builtin_fmaf(o, e0, __fmul_rn(oi, e1)); }
__device__ inline f32x4 fold_value(f32x4 o, float e0, f32x4 oi, float e1) {
  f32x4 r;
#pragma unroll
  for (int i = 0; i < 4; ++i) r[i] = fold_value(o[i], e0, oi[i], e1);
  return r;
}
__device__ inline f32x4 fma4(f32x4 a, float b, f32x4 c) {
  f32x4 r;
#pragma unroll
  for (int i = 0; i < 4; ++i) r[i] = __builtin_fmaf(a[i], b, c[i]);
  return r;
}
__device__ inline void fold_factors(float m, float mi, float &M, float &e0, float &e1) {
  M = fmaxf(m, mi);
  e0 = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m - M);
  e1 = mi == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mi - M);
}
template <typename V>
__device__ inline void fold_part(float &m, float &l, V &o, float mi, float li, V oi) {
  float M, e0, e1;
  fold_factors(m, mi, M, e0, e1);
  o = fold_value(o, e0, oi, e1);
  l = fold_value(l, e0, li, e1);
  m = M;
}

// One run of scores, 8 per lane: its largest, and its exponentials relative to m with their sum.
__device__ inline float run_max(const float (&s)[8]) {
  float v = s[0];
#pragma unroll
  for (int e = 1; e < 8; ++e) v = fmaxf(v, s[e]);
  return column_max(v);
}
__device__ inline bf16x8 run_exp(const float (&s)[8], float m, float &sum) {
  bf16x8 p;
  sum = 0.f;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const float v = __builtin_amdgcn_exp2f(s[e] - m);
    sum += v;
    p[e] = (__bf16)v;
  }
  return p;
}

// A result from its sums, the quotients rounded as a division rounds them: with the product of o and a reciprocal alone, up to an ulp off, means that bf16 holds or
// that lie half-way between two of its values come out as their neighbours.  The four quotients share the reciprocal and its refinement, and the steps
// are those of the division without its scaling, which sums of weights (1 at least) and results that are no smaller than 2^-100 do not call for.
// (Rows of a pass, 3000 of the 1.5B shape: 65.4 us, by four divisions 67.9, by the reciprocal 64.7.  A decode launch takes 0.1 to 0.2 us more than by the reciprocal.)
__device__ inline bf16x4 finish(f32x4 o, float l) {
  bf16x4 q = {};
#ifdef __HIP_DEVICE_COMPILE__
  float r = __builtin_amdgcn_rcpf(l);
  r = __builtin_fmaf(__builtin_fmaf(-l, r, 1.f), r, r);
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    float x = o[e] * r;
    x = __builtin_fmaf(__builtin_fmaf(-l, x, o[e]), r, x);
    x = __builtin_fmaf(__builtin_fmaf(-l, x, o[e]), r, x);
    q[e] = (__bf16)__builtin_amdgcn_div_fixupf(x, l, o[e]);   // (infinities and NaN)
  }
#endif
  return q;
}

// Values that another workgroup of the same launch reads: written through to the memory all XCDs share and
// read from there (agent scope), so that no L2 has to be written back or invalidated.
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
#ifdef __HIP_DEVICE_COMPILE__
constexpr int AGENT_SCOPE = 16;   // of a buffer instruction
struct Shared {
  __amdgpu_buffer_rsrc_t r;
  __device__ Shared(const float *p, int64_t n) : r(__builtin_amdgcn_make_buffer_rsrc((void *)p, 0, (int)(n * 4), 0x00020000)) {}
  __device__ void store4(int at, f32x4 v) const { __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), r, at * 4, 0, AGENT_SCOPE); }
  __device__ void store2(int at, float2 v) const { __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, at * 4, 0, AGENT_SCOPE); }
  __device__ f32x4 load4(int at) const { return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, at * 4, 0, AGENT_SCOPE)); }
  __device__ float2 load2(int at) const { return __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(r, at * 4, 0, AGENT_SCOPE)); }
};
#else
struct Shared {
  __device__ Shared(const float *, int64_t) {}
  __device__ void store4(int, f32x4) const {}
  __device__ void store2(int, float2) const {}
  __device__ f32x4 load4(int) const { return {}; }
  __device__ float2 load2(int) const { return {}; }
};
#endif

// The chunks of one (sequence, kv head), written through, folded in order into the output row: four elements of a head per thread,
// the loads of eight chunks together.  256 threads.
template <int HD>
__device__ inline void merge_chunks(const AttnParams &p, const Shared &po, const Shared &pml, int b, int g, int nchunk) {
  const int G = p.Hq / p.Hkv;
  for (int i = threadIdx.x; i < G * (HD / 4); i += 256) {
    const int h = i / (HD / 4);
    float M = -INFINITY, L = 0.f;
    f32x4 O = {0.f, 0.f, 0.f, 0.f};
    for (int c0 = 0; c0 < nchunk; c0 += 8) {
      float2 ml[8];
      f32x4 o[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int c = min(c0 + u, nchunk - 1);
        ml[u] = pml.load2(c * ATTN_ML + h * 2);
        o[u] = po.load4(c * G * HD + i * 4);
      }
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (c0 + u < nchunk) fold_part(M, L, O, ml[u].x, ml[u].y, o[u]);
    }
    *(bf16x4 *)(p.out + ((int64_t)b * p.Hq + g * G) * HD + i * 4) = finish(O, L);
  }
}

// ROTATE: q, k and v of the step come as the QKV product's slices of partial sums; the workgroup adds them up and
// rotates its group's heads, and the item that holds the step's own position also appends k and v to the cache
// and patches them into the run it has loaded.  Saves a launch per layer, but the rotation is a dependent round
// trip ahead of the first scores: worth it in launches of few workgroups (attention_rotates).  Those launches do better with three
// workgroups per compute unit of one register stage than with two of two (7B shape, 19 rows: a step 2450 -> 2425 us, others the same; the large
// launches lose by it: 512 ragged sequences 680 -> 690).
template <int HD, int NS, bool ROTATE, int SP>   // SP: slices of the product (ROTATE)
__global__ __launch_bounds__(256, ROTATE ? 3 : 2) void attn_decode_kernel(AttnParams p) {
  static_assert(NS >= 1 && SUB_RUNS % (4 * NS) == 0, "a sub is whole rounds of the stages");
  constexpr int NJ = HD / 32;   // QK MFMAs per 16-token tile
  constexpr int NV = HD / 16;   // PV MFMAs per 32-token run
  // Work items come from a compact list built on the device for this step: every launched workgroup
  // up to the list's length has work (full chunks first, then the last chunks, longest first), so
  // consecutive workgroup ids, which the hardware deals round-robin to the 8 XCDs, load all XCDs
  // evenly whatever the mix of context lengths.  An item is one 32-byte record (sequence, chunk,
  // context length, slot, and the first four page ids of the chunk), so that the first K/V loads of
  // a workgroup are one dependent scalar load away (its record; records beyond the list's end say so
  // themselves) instead of five: with the memory system saturated each such load takes about a
  // microsecond during which the workgroup has nothing in flight.
  // Calls whose items all run at once whatever their order need no list (work null): item i is chunk
  // i % max_chunks of sequence i / max_chunks.
  const int item = blockIdx.x / p.Hkv, g = blockIdx.x % p.Hkv;
  int b, c, ctx, slot;
  int4 r1;   // page ids
  if (p.work) {
    const int4 *rec = (const int4 *)(p.work + 8 * (int64_t)item);
    const int4 r0 = rec[0];
    r1 = rec[1];
    b = r0.x; c = r0.y; ctx = r0.z; slot = r0.w;
    if (ctx <= 0) return;   // beyond the end of the list (the list kernel clears the records up to the grid's end)
  } else {
    b = slot = item / p.max_chunks;
    c = item % p.max_chunks;
    ctx = p.ctx_len[b];
    const int32_t *row = p.page_table + (int64_t)slot * p.pages_per_seq;
    const int p0 = (int)((int64_t)c * p.item_tokens / p.page_tokens), last = p.pages_per_seq - 1;
    r1 = make_int4(row[min(p0, last)], row[min(p0 + 1, last)], row[min(p0 + 2, last)], row[min(p0 + 3, last)]);
    if (c * p.item_tokens >= ctx) return;
  }
  const int t0 = c * p.item_tokens;
  const int t1 = min(ctx, t0 + p.item_tokens);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63;   // uniform: page ids by scalar loads
  const int head = l & 15, qg = l >> 4;
  const int G = p.Hq / p.Hkv;
  // The launch does not write the page table: reads through the constant address space stay scalar loads.  As ordinary
  // reads behind the stores of k and v (ROTATE) they became vector loads, each of which waited for every K/V load in
  // flight, from the fifth page of an item on (7B shape, 34 sequences of 6000 tokens: 13 us per launch).
  const scalar_i32 *pt = (const scalar_i32 *)(p.page_table + (int64_t)slot * p.pages_per_seq);
  const int page_first = t0 / p.page_tokens;   // r1 holds the ids of pages page_first .. page_first + 3
  const float scale = 1.4426950408889634f / sqrtf((float)HD);   // log2(e) / sqrt(hd)
  const int64_t page_elems = (int64_t)2 * p.page_tokens * HD;   // K block + V block of one kv head

  __shared__ __attribute__((aligned(16))) bf16_t s_qkv[ROTATE ? 18 * HD : 8];   // rotated q of the group's heads (16), k, v
  const bool appends = ROTATE && t1 == ctx;   // this item holds the step's own position, ctx - 1
  // ROTATE: one thread per four rotated pairs of a head of the group, of k or of v
  constexpr int QUADS = HD / 8;
  const int n_rot = ROTATE ? (G + (appends ? 2 : 0)) * QUADS : 0, hh = threadIdx.x / QUADS, pair = threadIdx.x % QUADS * 4;
  const bool rotates = (int)threadIdx.x < n_rot;
  f32x4 f1[SP], f2[SP], rc = {}, rs = {};
  int own_page = 0;
  if (ROTATE && rotates) {
    // everything the rotation reads is requested before the first K/V loads: loads return in order
    const int width = (p.Hq + 2 * p.Hkv) * HD;
    const float *src = p.qkv + (int64_t)b * width + (hh < G ? g * G + hh : hh == G ? p.Hq + g : p.Hq + p.Hkv + g) * HD + pair;
#pragma unroll
    for (int u = 0; u < SP; ++u) {
      f1[u] = *(const f32x4 *)(src + (int64_t)u * p.n_seq * width);
      f2[u] = *(const f32x4 *)(src + (int64_t)u * p.n_seq * width + HD / 2);
    }
    rc = *(const f32x4 *)(p.cs + (int64_t)b * HD + pair);
    rs = *(const f32x4 *)(p.cs + (int64_t)b * HD + HD / 2 + pair);
    if (appends) own_page = pt[(ctx - 1) / p.page_tokens];
  }
  if constexpr (ROTATE) __builtin_amdgcn_sched_barrier(0);

  // Query operand: column = head of the group (zero for the padding columns), k = head-dim slice.
  bf16x8 qf[NJ];
  auto read_q = [&](const bf16_t *q) {
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      if (head < G) {
        qf[j] = *(const bf16x8 *)(q + head * HD + j * 32 + qg * 8);
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) qf[j][e] = (__bf16)0.0f;
      }
    }
  };
  if constexpr (!ROTATE) read_q(p.q + ((int64_t)b * p.Hq + g * G) * HD);

  f32x4 o[NV];
#pragma unroll
  for (int i = 0; i < NV; ++i) o[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY, lsum = 0.f;

  const int nblk = (t1 - t0 + 31) >> 5;
  // page id of a run, and the address of its K fragments given that id: the id of the run a stage will
  // hold next is fetched one refill ahead, so that no K/V load waits for a page-table load
  auto page_of = [&](int blk) -> int {
    const int t = t0 + blk * 32;
    const int rel = t / p.page_tokens - page_first;
    return rel == 0 ? r1.x : rel == 1 ? r1.y : rel == 2 ? r1.z : rel == 3 ? r1.w : pt[t / p.page_tokens];
  };
  auto run_base = [&](int blk, int page) -> const bf16_t * {
    const int r = ((t0 + blk * 32) % p.page_tokens) >> 5;
    return p.kv + ((int64_t)page * p.Hkv + g) * page_elems + (int64_t)r * 32 * HD + l * 8;
  };

  // NS register stages per wavefront: stage s holds the K and V fragments of run (it * NS + s) * 4 +
  // wave.  As soon as a stage's K fragments have gone through the QK MFMAs they are reloaded for the
  // run NS rounds later, likewise the V fragments after the PV MFMAs, so about NS runs (16 KiB each)
  // per wavefront are always in flight.
  // K and V are read once per step and never again before they are evicted: non-temporal loads keep
  // them from displacing each other in L2 on the way (measured +6 to 10 % bandwidth).
  bf16x8 kf[NS][2][NJ], vf[NS][NV];
  auto load_k = [&](int st, const bf16_t *kb) {
#pragma unroll
    for (int T = 0; T < 2; ++T)
#pragma unroll
      for (int j = 0; j < NJ; ++j) kf[st][T][j] = __builtin_nontemporal_load((const bf16x8 *)(kb + (T * NJ + j) * 512));
  };
  auto load_v = [&](int st, const bf16_t *kb) {
    const bf16_t *vb = kb + (int64_t)p.page_tokens * HD;
#pragma unroll
    for (int i = 0; i < NV; ++i) vf[st][i] = __builtin_nontemporal_load((const bf16x8 *)(vb + i * 512));
  };
  // The first loads of stage 0 carry no condition (a wavefront without a run loads the last one), so that the wait
  // counts of the rotation stay exact.  ROTATE: stage 0 is requested right behind the rotation's input, the others
  // when that has arrived and freed its registers.
  int page_next[NS];   // page of the run stage st takes after the one it holds
  auto load_first = [&](int st) {
    const int b0 = wave + 4 * st, bl = min(b0, nblk - 1);
    if (st == 0 || b0 < nblk) {
      const bf16_t *kb = run_base(bl, page_of(bl));
      load_k(st, kb);
      load_v(st, kb);
    }
    page_next[st] = b0 + 4 * NS < nblk ? page_of(b0 + 4 * NS) : 0;
  };
  load_first(0);
  f32x4 x1 = {0.f, 0.f, 0.f, 0.f}, x2 = {0.f, 0.f, 0.f, 0.f};
  if constexpr (ROTATE) {
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < SP; ++u) { x1 += f1[u]; x2 += f2[u]; }   // slices are added in order
    __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll
  for (int st = 1; st < NS; ++st) load_first(st);
  if constexpr (ROTATE) {
    __builtin_amdgcn_sched_barrier(0);
    if (rotates) {
      bf16x4 lo, hi;   // elements pair .. pair + 3 and half + pair .. half + pair + 3 of the head
      if (hh <= G) {
        rotate_pairs(x1, x2, rc, rs, lo, hi);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) { lo[e] = (__bf16)x1[e]; hi[e] = (__bf16)x2[e]; }
      }
      bf16_t *to = s_qkv + (hh < G ? hh : hh - G + 16) * HD + pair;
      *(bf16x4 *)to = lo;
      *(bf16x4 *)(to + HD / 2) = hi;
      if (hh >= G) {   // the step's own k or v goes to the cache
        const int tok = (ctx - 1) % p.page_tokens;
        bf16_t *kb = p.kv + ((int64_t)own_page * p.Hkv + g) * page_elems;
        if (hh == G) {
          *(bf16x4 *)(kb + k_elem_offset(tok, pair, HD)) = lo;
          *(bf16x4 *)(kb + k_elem_offset(tok, HD / 2 + pair, HD)) = hi;
        } else {
          bf16_t *vb = kb + (int64_t)p.page_tokens * HD;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            vb[v_elem_offset(tok, pair + e, HD)] = lo[e];
            vb[v_elem_offset(tok, HD / 2 + pair + e, HD)] = hi[e];
          }
        }
      }
    }
    // Only LDS passes between the wavefronts here: a full barrier would also wait for every K/V load in flight.
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    read_q(s_qkv);
  }
  // The run that holds the step's own position was loaded before (or while) the position was written: its operands
  // are patched from LDS.
  const int blk_own = appends ? nblk - 1 : -1;
  auto patch_own = [&](int st) {
    const int u = (ctx - 1) & 31, T = (u >> 2) & 1, R = ((u >> 3) << 2) | (u & 3);
#pragma unroll
    for (int j = 0; j < NJ; ++j)
      if (head == R) {
        const bf16x8 kn = *(const bf16x8 *)(s_qkv + 16 * HD + j * 32 + qg * 8);
        if (T == 0) kf[st][0][j] = kn; else kf[st][1][j] = kn;
      }
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const bf16_t vn = s_qkv[17 * HD + i * 16 + head];
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (qg == (u >> 3) && e == (u & 7)) vf[st][i][e] = vn;
    }
  };
  // Results of this wavefront's finished subs, folded in order; o is kept in the wavefront's own part of sm_o.
  __shared__ __attribute__((aligned(16))) float sm_o[4][16][HD + 4];   // (the columns of a store start at banks of their own)
  __shared__ float sm_m[4][16], sm_l[4][16];
  float m_all = -INFINITY, l_all = 0.f;
  bool folded = false;
  auto fold_sub = [&](bool first) {
    lsum = column_sum(lsum);
    float *mine = &sm_o[wave][head][qg * 4];
    if (first) {
      if (head < G) {
#pragma unroll
        for (int i = 0; i < NV; ++i) *(f32x4 *)(mine + i * 16) = o[i];
      }
      m_all = m; l_all = lsum;
      return;
    }
    float M, e0, e1;
    fold_factors(m_all, m, M, e0, e1);
    if (head < G) {
#pragma unroll
      for (int i = 0; i < NV; ++i) *(f32x4 *)(mine + i * 16) = fold_value(*(const f32x4 *)(mine + i * 16), e0, o[i], e1);
    }
    l_all = fold_value(l_all, e0, lsum, e1);
    m_all = M;
  };
  for (int base = wave; base < nblk; base += 4 * NS) {
#pragma unroll
    for (int st = 0; st < NS; ++st) {
      const int blk = base + 4 * st;
      if (blk < nblk) {
        if (ROTATE && blk == blk_own) patch_own(st);
        // scores of the 32 tokens of this run: two 16-token tiles
        f32x4 s4[2];
#pragma unroll
        for (int T = 0; T < 2; ++T) {
          s4[T] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int j = 0; j < NJ; ++j)
            s4[T] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[st][T][j], qf[j], s4[T], 0, 0, 0);
        }
        const int nxt = blk + 4 * NS;
        const bf16_t *nb = nullptr;
        if (nxt < nblk) {
          nb = run_base(nxt, page_next[st]);
          load_k(st, nb);
          page_next[st] = nxt + 4 * NS < nblk ? page_of(nxt + 4 * NS) : 0;
        }
        float s[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) s[e] = s4[e >> 2][e & 3] * scale;
        if (t0 + blk * 32 + 32 > t1) {   // the item's last run
          const int left = t1 - (t0 + blk * 32 + qg * 8);
#pragma unroll
          for (int e = 0; e < 8; ++e) s[e] = e < left ? s[e] : -INFINITY;
        }
        const float m_new = fmaxf(m, run_max(s));
        const float alpha = __builtin_amdgcn_exp2f(m - m_new);
        float psum;
        const bf16x8 pf = run_exp(s, m_new, psum);
        lsum = __builtin_fmaf(lsum, alpha, psum);
        m = m_new;
        if (__builtin_amdgcn_ballot_w64(!(alpha == 1.f))) {   // a maximum has moved (a factor of 1 changes nothing)
#pragma unroll
          for (int i = 0; i < NV; ++i) o[i] *= alpha;
        }
#pragma unroll
        for (int i = 0; i < NV; ++i) o[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[st][i], pf, o[i], 0, 0, 0);
        if (nb) load_v(st, nb);
      }
    }
    // end of a sub: SUB_RUNS runs, of which this wavefront took every fourth
    if ((base & (SUB_RUNS - 1)) + 4 * NS >= SUB_RUNS && base + 4 * NS < nblk) {
      fold_sub(!folded);
      folded = true;
      m = -INFINITY;
      lsum = 0.f;
#pragma unroll
      for (int i = 0; i < NV; ++i) o[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  }

  if (p.item_tokens < p.chunk && ctx > p.item_tokens) {   // an item is one sub: the wavefronts' results, for the merge kernel
    lsum = column_sum(lsum);
    const int64_t part = ((int64_t)item * p.Hkv + g) * 4 + wave;
    if (head < G) {
#pragma unroll
      for (int i = 0; i < NV; ++i) *(f32x4 *)(p.part_o + (part * G + head) * HD + i * 16 + qg * 4) = o[i];
      if (qg == 0) *(float2 *)(p.part_ml + (part * 16 + head) * 2) = make_float2(m, lsum);
    }
    return;
  }
  fold_sub(!folded);   // (the loop leaves the last sub of a wavefront open)
  if (head < G && qg == 0) { sm_m[wave][head] = m_all; sm_l[wave][head] = l_all; }
  __syncthreads();
  // merge the four wavefronts of the workgroup
  const int nchunk = (ctx + p.chunk - 1) / p.chunk;
  // (1.5B shape, 64 rows: the last workgroup ended 6.6 us behind the last run, merging an element at a time in three rounds of loads; four elements per
  // thread: 32.5 -> 30.0 us for the launch)
  auto merged = [&](auto put) {   // four elements of a head per thread
    for (int i = threadIdx.x; i < G * (HD / 4); i += 256) {
      const int h = i / (HD / 4), d = i % (HD / 4) * 4;
      const float M = fmaxf(fmaxf(sm_m[0][h], sm_m[1][h]), fmaxf(sm_m[2][h], sm_m[3][h]));
      float L = 0.f;
      f32x4 O = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const float f = __builtin_amdgcn_exp2f(sm_m[w][h] - M);
        L = __builtin_fmaf(sm_l[w][h], f, L);
        O = fma4(*(const f32x4 *)&sm_o[w][h][d], f, O);
      }
      put(i, h, d, M, L, O);
    }
  };
  if (nchunk == 1) {
    merged([&](int i, int, int, float, float L, f32x4 O) { *(bf16x4 *)(p.out + ((int64_t)b * p.Hq + g * G) * HD + i * 4) = finish(O, L); });
    return;
  }
  const int64_t row_parts = ((int64_t)b * p.Hkv + g) * p.max_chunks;
  const Shared po(p.part_o + row_parts * G * HD, (int64_t)p.max_chunks * G * HD), pml(p.part_ml + row_parts * ATTN_ML, (int64_t)p.max_chunks * ATTN_ML);
  merged([&](int i, int h, int d, float M, float L, f32x4 O) {
    po.store4(c * G * HD + i * 4, O);
    if (d == 0) pml.store2(c * ATTN_ML + h * 2, make_float2(M, L));
  });
  if (!p.tickets) return;
  // The workgroup that finishes a (sequence, kv head) last folds its chunks: no merge launch (a 5 us kernel and
  // a launch gap per layer).  Every store above has reached the shared memory (the wait) before the
  // ticket is taken; partial results of different workgroups share no cache line (128 bytes), so the last one
  // cannot have an old copy.  Release and acquire fences in their place would write back and invalidate the XCD's L2
  // in every workgroup (2.5 times the launch's time).
  __shared__ int s_last;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0) {
    int32_t *ticket = p.tickets + (int64_t)b * p.Hkv + g;
    const int before = __hip_atomic_fetch_add(ticket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    s_last = before == nchunk - 1;
    if (before == nchunk - 1) __hip_atomic_store(ticket, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // for the next launch
  }
  __syncthreads();
  if (s_last) merge_chunks<HD>(p, po, pml, b, g, nchunk);
}

// Merge of rows that span several items, where the decode kernel does not do it itself: one workgroup per (row, query head), four output
// elements per thread.  Latency bound (a few KiB per thread group): the loads of PARTS parts are issued together, no branch between them (19
// rows of 7300 tokens, 7B shape, 8.0 -> 6.6 us).
// SUBS: items are subs.  Two chunks at a time, HD threads for each; thread group w of a chunk folds wavefront w's subs, then the four
// wavefronts are merged as the decode kernel does it and the chunks folded in order.
template <int HD, bool SUBS, int PARTS>
__global__ __launch_bounds__(SUBS ? 2 * HD : 64) void attn_merge_kernel(AttnParams p) {
  constexpr int QUADS = HD / 4;
  const int b = blockIdx.y, hq = blockIdx.x, at = threadIdx.x % HD, w = at / QUADS, d = at % QUADS * 4;
  const int G = p.Hq / p.Hkv, g = hq / G, h = hq % G;
  const int ctx = p.ctx_len[b], first = SUBS ? p.first_item[b] : 0;   // (list index of the row's first item)
  if (ctx <= p.item_tokens) return;   // the decode kernel wrote the row
  const int nchunk = (ctx + p.chunk - 1) / p.chunk;
  float M = -INFINITY, L = 0.f;
  f32x4 O = {0.f, 0.f, 0.f, 0.f};
  // fold of n parts, part i at index at(i)
  auto fold_parts = [&](float &m, float &l, f32x4 &o, int n, int ml_floats, auto index) {
    for (int j0 = 0; j0 < n; j0 += PARTS) {
      float2 ml[PARTS];
      f32x4 op[PARTS];
#pragma unroll
      for (int u = 0; u < PARTS; ++u) {
        const int64_t part = index(min(j0 + u, n - 1));
        ml[u] = *(const float2 *)(p.part_ml + part * ml_floats + h * 2);
        op[u] = *(const f32x4 *)(p.part_o + (part * G + h) * HD + d);
      }
#pragma unroll
      for (int u = 0; u < PARTS; ++u) {
        float m1 = m, l1 = l;   // (selects, not branches: parts beyond the last change nothing)
        f32x4 o1 = o;
        fold_part(m1, l1, o1, ml[u].x, ml[u].y, op[u]);
        const bool in = j0 + u < n;
        m = in ? m1 : m;
        l = in ? l1 : l;
        o = in ? o1 : o;
      }
    }
  };
  if constexpr (!SUBS) {
    if ((int)threadIdx.x >= QUADS) return;
    const int64_t base = ((int64_t)b * p.Hkv + g) * p.max_chunks;
    fold_parts(M, L, O, nchunk, ATTN_ML, [&](int c) { return base + c; });
  } else {
    __shared__ f32x4 so[2][4][QUADS];
    __shared__ float sml[2][4][2];
    const int half = threadIdx.x / HD, per = p.chunk / p.item_tokens;
    for (int c0 = 0; c0 < nchunk; c0 += 2) {
      const int c = c0 + half;
      float mw = -INFINITY, lw = 0.f;
      f32x4 ow = {0.f, 0.f, 0.f, 0.f};
      if (c < nchunk)
        fold_parts(mw, lw, ow, min(per, (ctx - c * p.chunk + p.item_tokens - 1) / p.item_tokens), 32,
                   [&](int j) { return ((int64_t)(first + c * per + j) * p.Hkv + g) * 4 + w; });
      __syncthreads();
      so[half][w][at % QUADS] = ow;
      if (d == 0) { sml[half][w][0] = mw; sml[half][w][1] = lw; }
      __syncthreads();
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        if (c0 + k >= nchunk) continue;
        const float Mc = fmaxf(fmaxf(sml[k][0][0], sml[k][1][0]), fmaxf(sml[k][2][0], sml[k][3][0]));
        float Lc = 0.f;
        f32x4 Oc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const float f = __builtin_amdgcn_exp2f(sml[k][v][0] - Mc);
          Lc = __builtin_fmaf(sml[k][v][1], f, Lc);
          Oc = fma4(so[k][v][at % QUADS], f, Oc);
        }
        fold_part(M, L, O, Mc, Lc, Oc);
      }
    }
    if ((int)threadIdx.x >= QUADS) return;
  }
  *(bf16x4 *)(p.out + ((int64_t)b * p.Hq + hq) * HD + d) = finish(O, L);
}

// Attention of the rows of a cache-only pass: consecutive positions of one sequence, each over the positions up to its
// own.  One workgroup per (group of rows, kv head) walks all keys of the group's longest row; the columns of an MFMA
// are the heads of 16 CB / G rows, and every K/V operand serves CB blocks of 16 columns, where one row per workgroup
// (as in a decode step) reads the sequence once per row.  Operation by operation the same sums as the decode kernel
// for every row: runs, subs, wavefronts and chunks in the same order; a run that lies beyond a row's positions
// leaves its column as it was (factor 1, product not taken: 0 times an infinity would not be 0).
// Bound by vector arithmetic (about 80 instructions per run and column block, 32 more where a maximum moves; positions are masked only
// in runs that some row does not see whole), then by L2.  3000 rows of the 1.5B shape in one launch: 65 us, 84 with results at a
// stride of HD in LDS, 100 with whole rows per column block too.  As nine launches of 1000 rows before those two: 346 us, 365 with every run
// masked, maxima by shuffles through LDS and page ids by vector loads; 960 row by row.
template <int HD, int CB>
__global__ __launch_bounds__(256, 2) void attn_rows_kernel(AttnParams p) {
  constexpr int NJ = HD / 32, NV = HD / 16, COLS = CB * 16, PER = COLS * HD / 1024;
  const int g = blockIdx.x % p.Hkv, n_groups = p.groups[0], index = n_groups - 1 - (int)(blockIdx.x / p.Hkv);   // longest rows first
  if (index < 0) return;
  const int row0 = p.groups[2 + 2 * index], nrows = p.groups[3 + 2 * index];
  const int G = p.Hq / p.Hkv;   // column c of all CB blocks: head c % G of row c / G
  // (constant address space: the loop's stores to LDS would turn the page ids into vector loads that wait for the keys in flight)
  const scalar_i32 *pt = (const scalar_i32 *)(p.page_table + (int64_t)p.row_slot[row0] * p.pages_per_seq);
  const int ctx0 = p.ctx_len[row0], ctx_max = ctx0 + nrows - 1;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63, col = l & 15, qg = l >> 4;
  const float scale = 1.4426950408889634f / sqrtf((float)HD);   // log2(e) / sqrt(hd)
  const int64_t page_elems = (int64_t)2 * p.page_tokens * HD;

  // queries in operand order: element (column block, slice j, lane); in LDS, as the registers are taken by the results
  __shared__ __attribute__((aligned(16))) bf16x8 sq[CB * NJ * 64];
  for (int i = threadIdx.x; i < CB * NJ * 64; i += 256) {
    const int ln = i & 63, j = i / 64 % NJ, c = i / (64 * NJ) * 16 + (ln & 15), r = c / G;
    bf16x8 v = {};
    if (r < nrows) v = *(const bf16x8 *)(p.q + ((int64_t)(row0 + r) * p.Hq + g * G + c % G) * HD + j * 32 + (ln >> 4) * 8);
    sq[i] = v;
  }
  __shared__ int s_ctx[COLS];   // context of a column; columns without a row see no position
  if (threadIdx.x < COLS) {
    const int r = threadIdx.x / G;
    s_ctx[threadIdx.x] = r < nrows ? ctx0 + r : 0;
  }

  // (rows of HD + 4: the 16 columns of a store start at banks of their own; with HD, 70 % of the LDS's cycles were conflicts)
  __shared__ __attribute__((aligned(16))) float sm_o[4][COLS][HD + 4];
  __shared__ float sm_m[4][COLS], sm_l[4][COLS];
  // Result of the chunks so far: a thread owns the quads threadIdx.x + 256 k of [COLS][HD].
  f32x4 run_o[PER];
  __shared__ float run_m[COLS], run_l[COLS], s_f[4][COLS], s_e[2][COLS];
#pragma unroll
  for (int k = 0; k < PER; ++k) run_o[k] = f32x4{0.f, 0.f, 0.f, 0.f};
  if (threadIdx.x < COLS) { run_m[threadIdx.x] = -INFINITY; run_l[threadIdx.x] = 0.f; }

  __syncthreads();
  int ctx[CB];
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) ctx[cb] = s_ctx[cb * 16 + col];
  bf16x8 kf[2][NJ], vf[NV];
  auto run_at = [&](int tok) {   // the run that starts at token tok, or the sequence's last one
    tok = min(tok, (ctx_max - 1) & ~31);
    return p.kv + ((int64_t)pt[tok / p.page_tokens] * p.Hkv + g) * page_elems + (int64_t)(tok % p.page_tokens) * HD + l * 8;
  };
  auto load_k = [&](const bf16_t *kb) {
#pragma unroll
    for (int T = 0; T < 2; ++T)
#pragma unroll
      for (int j = 0; j < NJ; ++j) kf[T][j] = *(const bf16x8 *)(kb + (T * NJ + j) * 512);
  };
  auto load_v = [&](const bf16_t *kb) {
    const bf16_t *vb = kb + (int64_t)p.page_tokens * HD;
#pragma unroll
    for (int i = 0; i < NV; ++i) vf[i] = *(const bf16x8 *)(vb + i * 512);
  };
  load_k(run_at(wave * 32));
  load_v(run_at(wave * 32));
  for (int t0 = 0; t0 < ctx_max; t0 += p.chunk) {
    const int t1 = min(ctx_max, t0 + p.chunk), nblk = (t1 - t0 + 31) >> 5;
    f32x4 o[CB][NV];
    float m[CB], lsum[CB], m_all[CB], l_all[CB];
    auto reset = [&]() {
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) {
        m[cb] = -INFINITY;
        lsum[cb] = 0.f;
#pragma unroll
        for (int i = 0; i < NV; ++i) o[cb][i] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
    };
    reset();
    bool folded = false;
    auto fold_sub = [&]() {
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) {
        lsum[cb] = column_sum(lsum[cb]);
        float *mine = &sm_o[wave][cb * 16 + col][qg * 4];
        if (!folded) {
#pragma unroll
          for (int i = 0; i < NV; ++i) *(f32x4 *)(mine + i * 16) = o[cb][i];
          m_all[cb] = m[cb];
          l_all[cb] = lsum[cb];
          continue;
        }
        float Mx, e0, e1;
        fold_factors(m_all[cb], m[cb], Mx, e0, e1);
#pragma unroll
        for (int i = 0; i < NV; ++i) *(f32x4 *)(mine + i * 16) = fold_value(*(const f32x4 *)(mine + i * 16), e0, o[cb][i], e1);
        l_all[cb] = fold_value(l_all[cb], e0, lsum[cb], e1);
        m_all[cb] = Mx;
      }
    };
    // ENDED: rows of the group end before this run and have no part in it, whatever its values are
    auto take_run = [&](auto ENDED, int blk) {
      asm volatile("" ::: "memory");   // the queries stay in LDS: read anew for every run
      f32x4 s4[CB][2];
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) {
        bf16x8 qf[NJ];
#pragma unroll
        for (int j = 0; j < NJ; ++j) qf[j] = sq[(cb * NJ + j) * 64 + l];
#pragma unroll
        for (int T = 0; T < 2; ++T) {
          s4[cb][T] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int j = 0; j < NJ; ++j) s4[cb][T] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[T][j], qf[j], s4[cb][T], 0, 0, 0);
        }
      }
      const bf16_t *nb = run_at(blk + 4 < nblk ? t0 + (blk + 4) * 32 : t0 + p.chunk + wave * 32);   // (of the next chunk)
      load_k(nb);
      const bool whole = t0 + blk * 32 + 32 <= ctx0;   // every row sees every position of the run
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) {
        float s[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) s[e] = s4[cb][e >> 2][e & 3] * scale;
        if (!whole) {
          const int left = ctx[cb] - (t0 + blk * 32 + qg * 8);
#pragma unroll
          for (int e = 0; e < 8; ++e) s[e] = e < left ? s[e] : -INFINITY;
        }
        const float m_new = fmaxf(m[cb], run_max(s)), m_ref = m_new == -INFINITY ? 0.f : m_new;
        const float alpha = __builtin_amdgcn_exp2f(m[cb] - m_ref);
        float psum;
        const bf16x8 pf = run_exp(s, m_ref, psum);
        lsum[cb] = __builtin_fmaf(lsum[cb], alpha, psum);
        m[cb] = m_new;
        if (__builtin_amdgcn_ballot_w64(!(alpha == 1.f))) {   // a maximum has moved (a factor of 1 changes nothing)
#pragma unroll
          for (int i = 0; i < NV; ++i) o[cb][i] *= alpha;
        }
#pragma unroll
        for (int i = 0; i < NV; ++i) {
          const f32x4 r = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[i], pf, o[cb][i], 0, 0, 0);
          if (!decltype(ENDED)::value || t0 + blk * 32 < ctx[cb]) o[cb][i] = r;
        }
      }
      load_v(nb);
      if ((blk & (SUB_RUNS - 1)) + 4 >= SUB_RUNS && blk + 4 < nblk) {   // end of a sub
        fold_sub();
        folded = true;
        reset();
      }
    };
    int blk = wave;
    for (; blk < nblk && t0 + blk * 32 < ctx0; blk += 4) take_run(std::false_type{}, blk);
    for (; blk < nblk; blk += 4) take_run(std::true_type{}, blk);
    fold_sub();
    if (qg == 0) {
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) { sm_m[wave][cb * 16 + col] = m_all[cb]; sm_l[wave][cb * 16 + col] = l_all[cb]; }
    }
    __syncthreads();
    // merge of the four wavefronts and fold of the chunk: the factors of a column once, then its elements; a
    // column that ends before this chunk keeps what it has (factors 1 and 0)
    if (threadIdx.x < COLS) {
      const int cc = threadIdx.x;
      const bool here = s_ctx[cc] > t0;
      const float Mc = fmaxf(fmaxf(sm_m[0][cc], sm_m[1][cc]), fmaxf(sm_m[2][cc], sm_m[3][cc]));
      float Lc = 0.f;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const float f = here ? __builtin_amdgcn_exp2f(sm_m[w][cc] - Mc) : 0.f;
        Lc = __builtin_fmaf(sm_l[w][cc], f, Lc);
        s_f[w][cc] = f;
      }
      float M = run_m[cc], e0 = 1.f, e1 = 0.f;
      if (here) {
        fold_factors(run_m[cc], Mc, M, e0, e1);
        run_l[cc] = fold_value(run_l[cc], e0, Lc, e1);
        run_m[cc] = M;
      }
      s_e[0][cc] = e0;
      s_e[1][cc] = e1;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int at = threadIdx.x + 256 * k, cc = at / (HD / 4), d = at % (HD / 4) * 4;
      f32x4 Oc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int w = 0; w < 4; ++w) Oc = fma4(*(const f32x4 *)&sm_o[w][cc][d], s_f[w][cc], Oc);
      run_o[k] = fold_value(run_o[k], s_e[0][cc], Oc, s_e[1][cc]);
    }
    __syncthreads();   // the next chunk's results go to the same place
  }
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int at = threadIdx.x + 256 * k, cc = at / (HD / 4), d = at % (HD / 4) * 4;
    const int r = cc / G, h = cc % G;
    if (r >= nrows) continue;
    *(bf16x4 *)(p.out + ((int64_t)(row0 + r) * p.Hq + g * G + h) * HD + d) = finish(run_o[k], run_l[cc]);
  }
}

__global__ __launch_bounds__(1024) void attn_worklist_kernel(AttnParams p, int cap) {
  const int b = threadIdx.x;
  build_worklist<1024>(b < p.n_seq ? p.ctx_len[b] : 0, b < p.n_seq ? (p.row_slot ? p.row_slot[b] : b) : 0, p.page_table, p.work, p.tickets,
                 p.first_item, p.n_seq, p.Hkv, p.item_tokens, p.page_tokens, p.pages_per_seq, cap, p.item_tokens < p.chunk);
}

}  // namespace

int attention_chunk_tokens(int n_seq, int Hkv, int max_ctx) {
  // Tokens per workgroup: large enough that the merge is a small fraction of the bytes, small
  // enough that a few hundred compute units all get work.  A function of the launch shape only,
  // never of the contexts, so a sequence's result does not depend on its neighbours' lengths.
  int chunk = PL_ATTN_CHUNK;
  while (chunk > 128 && (int64_t)n_seq * Hkv * ((max_ctx + chunk - 1) / chunk) < 2048) chunk >>= 1;
  return chunk;
}

// A step in which one item would outlast the rest: an item is then one sub.  A compute unit alone streams about
// 1/128 of what the chip does, so a launch lasts at least longest_item x 128 of total bytes; cutting pays from
// about three subs on (the merge launch takes 5 to 7 us, a sub 5).  7B shape, 19 sequences of 7000 tokens in an engine of
// 256 slots (8192-token chunks): 82 + 5 (merge) -> 34 + 8 us per layer.  The result's bits do not depend on the choice.
bool attention_split(int chunk, int64_t total_tokens, int64_t longest_item, int64_t n_subs, int Hkv) {
  return chunk > ATTN_SUB && longest_item >= 3 * ATTN_SUB && n_subs * Hkv <= ATTN_SPLIT_PARTS && longest_item * 128 > total_tokens * Hkv;
}

// Whether the workgroup that finishes a row last merges its chunks.  One workgroup folds them eight at a time, each a
// round trip to the shared memory: 118 chunks (5 rows of up to 15000 tokens in 128-token chunks) 41 us against 37 with the
// merge launch, which has a workgroup per head; up to 17 (1.5B shape, 64 rows) the same or better.
bool attention_tickets(int max_chunks) { return max_chunks <= 32; }

// Whether a step's attention rotates and appends by itself, for `items` work items over `tokens` positions.  It saves the
// launch (3 us per layer where nothing else changes), but every workgroup begins with a round trip to the slices: in workgroups
// that start later, and the more the longer the memory system is saturated, that costs more.  Microseconds per layer won by
// rotating inside (a step's time with it and without):
//   bytes: 7B shape, 192 workgroups of 6000 tokens +2.5, 256 -1.7; 384 of 3000 +0.1, 416 -1.4; 768 of 1300 +0.6, of 1600 -0.6;
//     32B shape, 384 of 2000 +1.4, 512 -2.3; head dimension 64, 448 of 6000 +1.2, 512 -1.1: 400 to 600 MB of keys and values.
//   workgroups: 7B (four slices) 768 of 800 tokens +2.3; 1.5B (six slices), 512-token chunks, 768 +1.3; head dimension 64, 768 of
//     800 +1.1, 1024 -1.2; 32B (seven slices) 512 of 500 +3.2, 768 -2.9.
// Slices and rotated quads have to fit the registers and threads of one workgroup.
bool attention_rotates(int items, int64_t tokens, int Hq, int Hkv, int hd, int splits) {
  return items * Hkv <= (splits <= 6 ? 768 : 512) && tokens * Hkv * hd * 4 <= (int64_t)448 << 20 && splits <= ATTN_ROTATE_SLICES &&
         (Hq / Hkv + 2) * (hd / 8) <= 256;
}

// ints of the work buffer (which must be 32-byte aligned): one 8-int record per item
int64_t attention_worklist_ints(int64_t max_items) { return 8 * max_items; }

int launch_attention_worklist(const AttnParams &p, int cap, hipStream_t s) {
  if (p.n_seq <= 0 || p.n_seq > 1024 || ((uintptr_t)p.work & 31)) return -1;
  hipLaunchKernelGGL(attn_worklist_kernel, dim3(1), dim3(1024), 0, s, p, cap);
  return hipGetLastError() == hipSuccess ? 0 : -7;
}

template <int HD>
static void launch_attention_hd(const AttnParams &p, hipStream_t s, int part) {
  if (part != 2) {
    const dim3 grid((unsigned)(p.max_items * p.Hkv));
    if (p.q)
      hipLaunchKernelGGL((attn_decode_kernel<HD, PL_ATTN_NS, false, 1>), grid, dim3(256), 0, s, p);
    else
      with_slices<1, ATTN_ROTATE_SLICES>(p.splits, [&](auto SP) {
        if constexpr (decltype(SP)::value > 0) hipLaunchKernelGGL((attn_decode_kernel<HD, 1, true, decltype(SP)::value>), grid, dim3(256), 0, s, p);
      });
  }
  if (part != 1 && p.merge) {
    // (whole chunks: 101 sequences of at most two, head dimension 32, 2.7 us a call by 16 parts at a time, 2.5 by four; three of up to 128 5.4 by 16, 6.4
    // by 16 with a branch for each)
    if (p.item_tokens < p.chunk) hipLaunchKernelGGL((attn_merge_kernel<HD, true, 16>), dim3(p.Hq, p.n_seq), dim3(2 * HD), 0, s, p);
    else if (p.max_chunks <= 4) hipLaunchKernelGGL((attn_merge_kernel<HD, false, 4>), dim3(p.Hq, p.n_seq), dim3(64), 0, s, p);
    else hipLaunchKernelGGL((attn_merge_kernel<HD, false, 16>), dim3(p.Hq, p.n_seq), dim3(64), 0, s, p);
  }
}

// part: 0 = the decode kernel and, where it does not merge the items of a row itself, the merge kernel; 1 = the
// decode kernel alone; 2 = the merge kernel alone (so that a caller can time the two separately)
int launch_attention(const AttnParams &p, hipStream_t s, int part) {
  if (p.n_seq <= 0) return 0;
  switch (p.hd) {
    case 128: launch_attention_hd<128>(p, s, part); break;
    case 64: launch_attention_hd<64>(p, s, part); break;
    case 32: launch_attention_hd<32>(p, s, part); break;
    default: return -1;
  }
  return hipGetLastError() == hipSuccess ? 0 : -7;
}

// Rows of a group of attn_rows_kernel: as many as have their G heads in the columns of CB blocks (six heads: five rows in 32 columns,
// where whole rows per block would be four).
constexpr int ATTN_ROWS_CB = 2;
int attention_rows_per_group(int Hq, int Hkv) { return ATTN_ROWS_CB * 16 / (Hq / Hkv); }

// Most rows of a pass that attend one by one in the decode kernel, which takes the chunks of a row side by side,
// instead of in groups that walk the whole context (2.2 us per 128 tokens, whatever the number of groups while they all
// run at once).  One by one the time grows with the bytes of all rows together.  GPU time of a pass of four layers
// of the 1.5B (256 elements of k per position), 7B (512) and of two of the 32B (1024) shape, one by one against in groups:
// 4 rows at position 8000 209 / 568, 521 / 646, 261 / 309 us; 192, 96 and 48 rows there 624 / 642, 919 / 856, 403 / 380.  With 64
// elements of k per position what a workgroup costs decides: 128 rows at 300 and at 8000 208 / 202, 316 / 435; 256 rows
// 168 / 156, 353 / 390; 512 rows 184 / 152, 525 / 385.
int attention_apart_rows(int Hkv, int hd) { return std::min(128, 32768 / (Hkv * hd)); }

int launch_attention_rows(const AttnParams &p, hipStream_t s) {
  if (p.n_seq <= 0) return 0;
  const dim3 grid((unsigned)(p.max_items * p.Hkv));
  switch (p.hd) {
    case 128: hipLaunchKernelGGL((attn_rows_kernel<128, ATTN_ROWS_CB>), grid, dim3(256), 0, s, p); break;
    case 64: hipLaunchKernelGGL((attn_rows_kernel<64, ATTN_ROWS_CB>), grid, dim3(256), 0, s, p); break;
    case 32: hipLaunchKernelGGL((attn_rows_kernel<32, ATTN_ROWS_CB>), grid, dim3(256), 0, s, p); break;
    default: return -1;
  }
  return hipGetLastError() == hipSuccess ? 0 : -7;
}

}  // namespace pl
