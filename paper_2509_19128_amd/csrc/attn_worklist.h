// The attention work list, built by one workgroup: alone (pl_attention_decode) or as part of the kernel that
// begins a step (kernels_misc.hip).
#pragma once
#include "pl_common.h"

namespace pl {
namespace {

// Inclusive prefix sum over the wavefront, through lanes.
__device__ inline int wave_scan(int v) {
#ifdef __HIP_DEVICE_COMPILE__
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);   // rows of 16: the lane 1, 2, 4, 8 before
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);   // the last lane of rows 0 and 2 to rows 1 and 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);   // lane 31 to the upper half
#endif
  return v;
}
// Inclusive prefix sums of two values over the NT threads of the workgroup, and their totals.
template <int NT>
__device__ inline int2 block_scan(int2 v, int2 *total) {
  __shared__ int2 wsum[NT / 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  v = make_int2(wave_scan(v.x), wave_scan(v.y));
  if (lane == 63) wsum[wave] = v;
  __syncthreads();
  int2 before = make_int2(0, 0), all = make_int2(0, 0);
#pragma unroll
  for (int w = 0; w < NT / 64; ++w) {
    const int2 x = wsum[w];
    all.x += x.x; all.y += x.y;
    before.x += w < wave ? x.x : 0; before.y += w < wave ? x.y : 0;
  }
  *total = all;
  return make_int2(v.x + before.x, v.y + before.y);
}

// The list's items are 8-int records: {sequence, chunk, context length, slot, ids of the
// chunk's first four pages}.  All full chunks come first, then each sequence's last (partial or full) chunk,
// longest first, so that the workgroups still running when the grid drains are the short ones.  With
// `contiguous` a sequence's items follow one another instead, from first_item[sequence] on (what the merge
// kernel of single subs needs; those launches run all items at once).  Records up to index `cap` beyond the
// list's end say "no item".  One workgroup of NT threads; thread b < n_seq
// brings sequence b's context length and slot, the others zeros.  Each record has a thread of its own that finds its
// sequence in the prefix sums: a thread per sequence that walks its chunks takes 10 us where sequences have 15.
template <int NT>
__device__ inline void build_worklist(int ctx, int slot, const int32_t *page_table, int32_t *work, int32_t *tickets,
                                      int32_t *first_item, int n_seq, int Hkv, int item_tokens, int page_tokens, int pages_per_seq,
                                      int cap, bool contiguous) {
  __shared__ __attribute__((aligned(16))) int tail[NT];
  __shared__ int pre[NT], s_ctx[NT], s_slot[NT];
  const int b = threadIdx.x;
  const int n = (ctx + item_tokens - 1) / item_tokens;
  const int listed = contiguous ? n : n > 0 ? n - 1 : 0;   // items of this sequence in the first part of the list
  auto pages = [&](int c, int cx, int sl) {   // the first four of a chunk
    const int32_t *pt = page_table + (int64_t)sl * pages_per_seq;
    const int last_page = (cx - 1) / page_tokens, p0 = (int)((int64_t)c * item_tokens / page_tokens);
    return make_int4(pt[min(p0, last_page)], pt[min(p0 + 1, last_page)], pt[min(p0 + 2, last_page)], pt[min(p0 + 3, last_page)]);
  };
  auto put = [&](int i, int4 r0, int4 r1) {
    if (i >= cap) return;
    int4 *rec = (int4 *)(work + 8 * (int64_t)i);
    rec[0] = r0;
    rec[1] = r1;
  };
  int4 own_pages = make_int4(0, 0, 0, 0);   // of this sequence's last chunk, on their way while its place in the list is found
  if (!contiguous && n > 0) own_pages = pages(n - 1, ctx, slot);
  int2 totals;
  pre[b] = block_scan<NT>(make_int2(listed, !contiguous && n > 0), &totals).x - listed;
  const int total = totals.x, n_last = totals.y;
  s_ctx[b] = ctx;
  s_slot[b] = slot;
  const int rem = n > 0 ? ctx - (n - 1) * item_tokens : 0;
  // of its last chunk's place: longer first, lower sequence index first among equals; 0 for empty rows and for threads at or beyond n_seq
  const int key = n > 0 ? rem << 10 | (1023 - b) : 0;
  tail[b] = key;
  __syncthreads();
  if (contiguous && b < n_seq) first_item[b] = pre[b];
  for (int i = b; i < total; i += NT) {   // last sequence whose items start at or before i
    int lo = 0;
#pragma unroll
    for (int step = NT / 2; step > 0; step >>= 1)
      if (pre[lo + step] <= i) lo += step;   // lo + step < NT
    const int c = i - pre[lo];
    put(i, make_int4(lo, c, s_ctx[lo], s_slot[lo]), pages(c, s_ctx[lo], s_slot[lo]));
  }
  if (!contiguous && n > 0) {
    int rank = 0;
    const int4 *t4 = (const int4 *)tail;
    for (int o = 0; o < n_seq; o += 32) {   // (eight reads under way; the zeros behind the last sequence outrank nothing)
      int4 t[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) t[u] = t4[o / 4 + u];
#pragma unroll
      for (int u = 0; u < 8; ++u) rank += (t[u].x > key) + (t[u].y > key) + (t[u].z > key) + (t[u].w > key);
    }
    put(total + rank, make_int4(b, n - 1, ctx, slot), own_pages);
  }
  for (int i = b; tickets && i < n_seq * Hkv; i += NT) tickets[i] = 0;
  for (int i = total + n_last + b; i < cap; i += NT) ((int4 *)(work + 8 * (int64_t)i))[0] = make_int4(0, 0, 0, 0);
}

}  // namespace
}  // namespace pl
