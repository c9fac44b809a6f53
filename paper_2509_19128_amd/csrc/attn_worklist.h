// The attention work list, built by one workgroup: alone (pl_attention_decode) or as part of the kernel that
// begins a step (kernels_misc.hip).
#pragma once
#include "pl_common.h"

namespace pl {
namespace {

// Inclusive prefix sum over the 1024 threads of the workgroup (wave shuffles, then the 16 wave totals).
__device__ inline int block_scan_1024(int v, int *wsum, int *total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int t = __shfl_up(v, o, 64);
    if (lane >= o) v += t;
  }
  __syncthreads();   // wsum may still be read from a previous call
  if (lane == 63) wsum[wave] = v;
  __syncthreads();
  int before = 0, all = 0;
#pragma unroll
  for (int w = 0; w < 16; ++w) {
    const int x = wsum[w];
    all += x;
    if (w < wave) before += x;
  }
  *total = all;
  return v + before;
}

// The list's items are 8-int records: {sequence, chunk, context length, slot, ids of the
// chunk's first four pages}.  All full chunks come first, then each sequence's last (partial or full) chunk,
// longest first, so that the workgroups still running when the grid drains are the short ones.  With
// `contiguous` a sequence's items follow one another instead, from first_item[sequence] on (what the merge
// kernel of single subs needs; those launches run all items at once).  Records up to index `cap` beyond the
// list's end say "no item".  One workgroup of 1024 threads; thread b < n_seq
// brings sequence b's context length and slot, the others zeros.  Each record has a thread of its own that finds its
// sequence in the prefix sums: a thread per sequence that walks its chunks takes 10 us where sequences have 15.
__device__ inline void build_worklist(int ctx, int slot, const int32_t *page_table, int32_t *work, int32_t *tickets,
                                      int32_t *first_item, int n_seq, int Hkv, int item_tokens, int page_tokens, int pages_per_seq,
                                      int cap, bool contiguous) {
  __shared__ int wsum[16];
  __shared__ __attribute__((aligned(16))) int tail[1024];
  __shared__ int pre[1024], s_ctx[1024], s_slot[1024];
  const int b = threadIdx.x;
  const int n = (ctx + item_tokens - 1) / item_tokens;
  const int listed = contiguous ? n : n > 0 ? n - 1 : 0;   // items of this sequence in the first part of the list
  auto put = [&](int i, int bb, int c, int cx, int sl) {
    if (i >= cap) return;
    const int32_t *pt = page_table + (int64_t)sl * pages_per_seq;
    const int last_page = (cx - 1) / page_tokens, p0 = (int)((int64_t)c * item_tokens / page_tokens);
    int4 *rec = (int4 *)(work + 8 * (int64_t)i);
    rec[0] = make_int4(bb, c, cx, sl);
    rec[1] = make_int4(pt[min(p0, last_page)], pt[min(p0 + 1, last_page)], pt[min(p0 + 2, last_page)], pt[min(p0 + 3, last_page)]);
  };
  int total, n_last = 0;
  pre[b] = block_scan_1024(listed, wsum, &total) - listed;
  s_ctx[b] = ctx;
  s_slot[b] = slot;
  const int rem = n > 0 ? ctx - (n - 1) * item_tokens : 0;
  tail[b] = rem;   // 0 for empty rows and for threads at or beyond n_seq
  if (!contiguous) (void)block_scan_1024(n > 0, wsum, &n_last);
  __syncthreads();
  if (contiguous && b < n_seq) first_item[b] = pre[b];
  for (int i = b; i < total; i += 1024) {   // last sequence whose items start at or before i
    int lo = 0;
#pragma unroll
    for (int step = 512; step > 0; step >>= 1)
      if (pre[lo + step] <= i) lo += step;   // lo + step <= 1023
    put(i, lo, i - pre[lo], s_ctx[lo], s_slot[lo]);
  }
  if (!contiguous && n > 0) {   // rank among the last chunks: longer first, lower sequence index first among equals
    int rank = 0;
    const int4 *t4 = (const int4 *)tail;
    for (int o4 = 0; o4 < (n_seq + 3) / 4; ++o4) {
      const int4 t = t4[o4];
      const int o = o4 * 4;
      rank += (t.x > rem) || (t.x == rem && o < b);
      rank += (t.y > rem) || (t.y == rem && o + 1 < b);
      rank += (t.z > rem) || (t.z == rem && o + 2 < b);
      rank += (t.w > rem) || (t.w == rem && o + 3 < b);
    }
    put(total + rank, b, n - 1, ctx, slot);
  }
  for (int i = b; tickets && i < n_seq * Hkv; i += 1024) tickets[i] = 0;
  for (int i = total + n_last + b; i < cap; i += 1024) ((int4 *)(work + 8 * (int64_t)i))[0] = make_int4(0, 0, 0, 0);
}

}  // namespace
}  // namespace pl
