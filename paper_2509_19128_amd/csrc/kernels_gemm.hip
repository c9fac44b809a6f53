// Skinny-M bf16 GEMM y = x W^T for the decode projections (QKV, O, gate/up + SwiGLU, down, LM head).
//
// With M = batch <= 256 rows these products are bound by streaming W once from HBM; W is never
// reused across workgroups, so it bypasses LDS: every wavefront loads the W rows it owns straight
// into the registers of the MFMA's first operand.  W is stored in operand order (blocks of 32 rows x 64 k, see
// pl_weight_layout in pl.h), so each of those loads is one contiguous KiB per wavefront.  The small activation tile x is what all
// workgroups share; it goes to LDS by direct loads and feeds the other operand.  32x32x16 bf16 MFMAs
// accumulate in fp32.  K can be split across workgroups (partials summed by the consumer in a
// fixed order) so that narrow outputs still occupy every compute unit.
#include "pl_common.h"

#include <algorithm>
#include <type_traits>

namespace pl {
namespace {

constexpr int BK = 64;          // k elements per main-loop step
constexpr int STAGES = 4;       // k-steps held: one is multiplied while three are on their way
typedef __attribute__((address_space(3))) void lds_void;
// Cache policy of the W loads: non-temporal (2) for weights that are COLD, that is, cannot be in the 256 MB last-level cache
// from the pass before, in tiles whose W one wavefront reads (WM = 1): they have no second reader, and ordinary loads
// evict each other from L2 on the way.  SwiGLU of the 32B shape, 128 rows: 111.8 -> 98.7 us (5.7 TB/s); 7B shape, 19 rows,
// whole step -4 %; products at 256 rows -1 % (the second row tile's reader still finds W in L2; not where that tile
// or one of more is short: launch_gemm, launch_gemm_folded).  Where two wavefronts
// share W through the caches (WM = 2; 1.5B shape, 64 rows) they cost 3.5 % of the step, and a matrix that stays in the
// last-level cache between calls 5 to 30 % (55 MB, 3 rows: 11 -> 16 us).
template <int WM, bool COLD>
constexpr int W_CACHE = WM == 1 && COLD ? 2 : 0;

// A tile of the product: a workgroup of 4 wavefronts arranged WM x WN, each of which owns (AT*32) x (BT*32) outputs.
// W fragments go from memory to a ring of register stages, x tiles by direct loads to a ring of LDS stages (no registers
// and no store instructions on the way), both three k-steps ahead of the products that use them; nothing waits for
// younger loads, as loads complete in order and each wait names the number that may stay in flight.  What bounds a k-step is the
// larger of its MFMA time and of its bytes at what one compute unit gets from the caches (about 100 KB/us from L2, 45
// from HBM): cycles per k-step of a lone workgroup with W in L2, and of its MFMAs alone, 256x256 2260 and 2048, 128x256 1100 and 1024,
// 128x128 790 and 512 (with x through registers, a double-buffered LDS tile and a full wait at each barrier: 128x256 1680).
// On the full chip with random operands the clock settles so that about 1.5 PFLOP/s are left at the margin (256x256 tiles, 1024 rows:
// 1.42 us per k-step, 1.01 with operands of zeros).
// Row r of an LDS stage holds its eight 16-byte chunks at slots chunk ^ (r & 7): a direct load fills a KiB in lane order, 8 whole rows,
// and the reads of a fragment (one chunk of 32 rows) meet every bank once.
// The products are taken with W as the first operand: a lane ends with one row and groups of four consecutive columns.
template <int WM, int WN, int AT, int BT, bool COLD>
struct Tile {
  static constexpr int BM = WM * AT * 32, BN = WN * BT * 32;
  static constexpr int XI = BM / 32, XH = (XI + 1) / 2, WI = BT * 4;   // loads of a wavefront per k-step: x (half of them XH), W
  static constexpr int STAGE = BM * BK, LDS = STAGES * STAGE;          // elements
  static_assert(WM * WN == 4 && BT <= 2, "tile");

  // where a tile's operands are
  struct Part {
    int x_lane[XI];        // per lane: byte offset of its row and chunk (rows beyond M repeat the last one)
    int x_k;               // byte offset of the first k
    uint32_t w_blk[BT];    // byte offset of the first W block
  };
  // Operand-ordered W: block (k-step, n / 32) is 4096 bytes: [j][lane][16 B], lane = half * 32 + row.
  // Blocks are k-step-major: workgroups walk K in step, so at any moment the whole chip reads one
  // contiguous plane of W and the traffic spreads over every HBM channel (with row-block-major
  // order all streams sit a multiple of 8 blocks apart and camp on a fraction of the channels).
  __amdgpu_buffer_rsrc_t rw, rx;   // one resource per operand; what is uniform across a wavefront is in scalar registers
  uint32_t w_plane;
  int wave, wm, wn, l, lrow, half, a_off[4];
  bf16_t *xs;
  f32x16 acc[AT][BT];
  bf16x8 wf[STAGES][BT][4], af[2][AT];

  __device__ __forceinline__ void init(bf16_t *xs_, const bf16_t *X, const bf16_t *W, int M, int N, int K) {
    xs = xs_;
    l = threadIdx.x & 63;
    wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    wm = wave / WN; wn = wave % WN;
    lrow = l & 31; half = l >> 5;
    w_plane = (uint32_t)(N >> 5) * 4096u;
    rw = __builtin_amdgcn_make_buffer_rsrc((void *)W, 0, (int)((int64_t)N * K * 2), 0x00020000);
    rx = __builtin_amdgcn_make_buffer_rsrc((void *)X, 0, (int)((int64_t)M * K * 2), 0x00020000);
#pragma unroll
    for (int j = 0; j < 4; ++j) a_off[j] = (wm * AT * 32 + lrow) * BK + ((half * 4 + j) ^ (lrow & 7)) * 8;
  }
  __device__ __forceinline__ Part part(int n_tile0, int m0, int ks0, int M, int N, int K) const {
    Part p;
#pragma unroll
    for (int i = 0; i < XI; ++i)
      p.x_lane[i] = (min(m0 + (wave * XI + i) * 8 + (l >> 3), M - 1) * K + ((l & 7) ^ (l >> 3)) * 8) * 2;
    p.x_k = ks0 * BK * 2;
#pragma unroll
    for (int b = 0; b < BT; ++b)
      p.w_blk[b] = (uint32_t)ks0 * w_plane + (uint32_t)min(((n_tile0 + wn * BT * 32) >> 5) + b, (N >> 5) - 1) * 4096u;
    return p;
  }
  __device__ __forceinline__ void zero() {
#pragma unroll
    for (int a = 0; a < AT; ++a)
#pragma unroll
      for (int b = 0; b < BT; ++b)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[a][b][i] = 0.f;
  }
  __device__ __forceinline__ void load_x(const Part &p, int st, int ks, int i0, int i1) {
#ifdef __HIP_DEVICE_COMPILE__
#pragma unroll
    for (int i = i0; i < i1; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (lds_void *)(xs + st * STAGE + (wave * XI + i) * 512), 16, p.x_lane[i], p.x_k + ks * (BK * 2), 0, 0);
#endif
  }
  __device__ __forceinline__ void load_w(const Part &p, int st, int ks, int b) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
      wf[st][b][j] = __builtin_bit_cast(
          bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rw, l * 16 + j * 1024, (int)(p.w_blk[b] + (uint32_t)ks * w_plane), W_CACHE<WM, COLD>));
  }
  __device__ __forceinline__ void load(const Part &p, int st, int ks) {
    load_x(p, st, ks, 0, XI);
#pragma unroll
    for (int b = 0; b < BT; ++b) load_w(p, st, ks, b);
  }
  __device__ __forceinline__ void read_a(int st, int j) {
#pragma unroll
    for (int a = 0; a < AT; ++a) af[j & 1][a] = *(const bf16x8 *)(xs + st * STAGE + a_off[j] + a * 32 * BK);
  }
  __device__ __forceinline__ void mma(int st, int j) {
#pragma unroll
    for (int a = 0; a < AT; ++a)
#pragma unroll
      for (int b = 0; b < BT; ++b)
        acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[st][b][j], af[j & 1][a], acc[a][b], 0, 0, 0);
  }
  // all but the LEFT youngest loads have arrived, and this wavefront has its operands out of LDS; then the others too
  template <int LEFT>
  __device__ __forceinline__ void meet() {
#ifdef __HIP_DEVICE_COMPILE__
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"i"(LEFT) : "memory");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
#endif
  }
  // no load is on its way to LDS any more
  __device__ __forceinline__ void drain() {
#ifdef __HIP_DEVICE_COMPILE__
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#endif
  }
  // Issue order of a quarter of a k-step: LDS reads (for the next quarter) and VM loads one by one between the products.
  template <int VM, bool READS>
  __device__ __forceinline__ void order() {
    constexpr int per = VM >= AT ? VM / AT : 1;
#pragma unroll
    for (int i = 0; i < AT; ++i) {
      if (READS) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, BT, 0);
      if (VM >= AT || i * VM / AT != (i + 1) * VM / AT) __builtin_amdgcn_sched_group_barrier(0x020, per, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  // First three k-steps of a part into stages 0 .. 2, and the first operands out of LDS.
  __device__ __forceinline__ void begin(const Part &p) {
#pragma unroll
    for (int st = 0; st < STAGES - 1; ++st) load(p, st, st);
    meet<2 * (XI + WI) + WI>();
    read_a(0, 0);
  }
  // One k-step in stage U (k-step index mod 4).  LOAD: k-step ks of part p goes to the stage that the last one freed.
  // AFTER: k-steps that follow (3: three or more), whose loads stay in flight while the next stage is waited for.
  // The operands of the last quarter are read before that wait, those of the next k-step's first quarter behind it, so that the matrix
  // pipeline has a quarter's products to work on meanwhile.
  template <int U, bool LOAD, int AFTER>
  __device__ __forceinline__ void kstep(const Part &p, int ks) {
    constexpr int TO = (U + 3) & 3;
    read_a(U, 1);
    if (LOAD) load_x(p, TO, ks, 0, XH);
    mma(U, 0);
    order<LOAD ? XH : 0, true>();
    read_a(U, 2);
    if (LOAD) load_x(p, TO, ks, XH, XI);
    mma(U, 1);
    order<LOAD ? XI - XH : 0, true>();
    read_a(U, 3);
    if (LOAD) load_w(p, TO, ks, 0);
    mma(U, 2);
    order<LOAD ? 4 : 0, true>();
    if (AFTER > 0) {
      meet<AFTER == 1 ? WI : AFTER == 2 ? XI + 2 * WI : 2 * (XI + WI) + 4>();
      read_a((U + 1) & 3, 0);
    }
    if (LOAD && BT > 1) load_w(p, TO, ks, BT - 1);
    mma(U, 3);
    if (AFTER > 0) {
#pragma unroll
      for (int i = 0; i < AT; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, BT, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        if (LOAD && BT > 1 && (4 >= AT || i * 4 / AT != (i + 1) * 4 / AT)) __builtin_amdgcn_sched_group_barrier(0x020, 4 >= AT ? 4 / AT : 1, 0);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  // k-steps ks .. ks + 3 of a part of more than ks + 7, and its last four
  __device__ __forceinline__ void four(const Part &p, int ks) {
    kstep<0, true, 3>(p, ks + 3);
    kstep<1, true, 3>(p, ks + 4);
    kstep<2, true, 3>(p, ks + 5);
    kstep<3, true, 3>(p, ks + 6);
  }
  __device__ __forceinline__ void last_four(const Part &p, int ks) {
    kstep<0, true, 3>(p, ks + 3);
    kstep<1, false, 2>(p, 0);
    kstep<2, false, 1>(p, 0);
    kstep<3, false, 0>(p, 0);
  }
  // accumulator register i of lane l is column (i / 4) * 8 + (l / 32) * 4 + i % 4, row l % 32
  // a 32 x 32 block so that the four lanes of a quad hold 64 bytes of a row: v[t] is row (l % 32 & ~3) + t, columns l / 32 * 16 + l % 4 * 4 on
  static __device__ __forceinline__ void by_rows(f32x4 (&v)[4], const f32x16 &c) {
#ifdef __HIP_DEVICE_COMPILE__
    const int odd = threadIdx.x & 1, high = threadIdx.x >> 1 & 1;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
      auto halves = [&](float x, float y, uint32_t &a, uint32_t &b) {   // lanes 32 .. 63 of x against 0 .. 31 of y
        const u32x2 r = __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false));
        a = r[0]; b = r[1];
      };
      uint32_t q[4];   // 16 columns of a row, in groups of four
      halves(c[e], c[8 + e], q[0], q[1]);
      halves(c[4 + e], c[12 + e], q[2], q[3]);
      // each lane reads its neighbour's registers before it chooses (a choice between reads would be a branch that leaves the neighbour out)
      uint32_t x[4], y[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) x[k] = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)q[k ^ 1], 0xB1, 0xf, 0xf, true);   // quad_perm 1 0 3 2
#pragma unroll
      for (int k = 0; k < 4; ++k) y[k] = odd != (k & 1) ? x[k] : q[k];
#pragma unroll
      for (int k = 0; k < 4; ++k) x[k] = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)y[k ^ 2], 0x4E, 0xf, 0xf, true);   // quad_perm 2 3 0 1
#pragma unroll
      for (int k = 0; k < 4; ++k) v[k][e] = __uint_as_float(high != (k >> 1) ? x[k] : y[k]);
    }
#endif
  }
  // fp32 sums: row stride ldy, columns counted from y_col0, columns below n_end (a multiple of 32).
  // Stores of 64 bytes of a row instead of 32 (a lane's own columns): LM head of the 7B shape, 256 rows, 322 -> 306 us, 7B QKV 22.6 -> 20.9,
  // 32B QKV, 128 rows, 22.3 -> 21.4.  Up to 64 rows the exchange costs more than it saves (1.5B QKV, 64 rows, 4.8 -> 5.0; a step of the tiny
  // shape 3 %).
  __device__ __forceinline__ void store(float *Y, int n_tile0, int m0, int M, int n_end, int64_t ldy, int y_col0) const {
    const int n0 = n_tile0 + wn * BT * 32;
#pragma unroll
    for (int a = 0; a < AT; ++a) {
      const int m = m0 + (wm * AT + a) * 32;
      if (m >= M) continue;
#pragma unroll
      for (int b = 0; b < BT; ++b) {
        if (n0 + b * 32 >= n_end) continue;
        if (M <= 64) {
          float *y = Y + (m + lrow) * ldy + (n0 + b * 32 + half * 4 - y_col0);
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (m + lrow < M) *(f32x4 *)(y + i * 8) = f32x4{acc[a][b][4 * i], acc[a][b][4 * i + 1], acc[a][b][4 * i + 2], acc[a][b][4 * i + 3]};
          continue;
        }
        f32x4 v[4];
        by_rows(v, acc[a][b]);
        float *y = Y + (m + (lrow & ~3)) * ldy + (n0 + b * 32 + half * 16 + (lrow & 3) * 4 - y_col0);
#pragma unroll
        for (int t = 0; t < 4; ++t)
          if (m + (lrow & ~3) + t < M) *(f32x4 *)(y + t * ldy) = v[t];
#ifdef __HIP_DEVICE_COMPILE__
        __builtin_amdgcn_sched_barrier(0);   // (one block's registers at a time)
#endif
      }
    }
  }
  // SwiGLU of a 64-row block's gate and up halves: the two column tiles of a wavefront, or (BT = 1) the tiles of two
  // neighbours, which swap half of them through the LDS stages that nothing reads any more and take half of the block each.
  __device__ __forceinline__ void store_swiglu(bf16_t *Y, int n_tile0, int m0, int M, int n_end, int N) {
    static_assert(BT == 2 || WM == 1, "pairs");
    constexpr int NI = BT == 2 ? 4 : 2;   // groups of four columns per lane
    const int n0 = BT == 2 ? n_tile0 + wn * 64 : n_tile0 + (wn >> 1) * 64, i0 = BT == 2 ? 0 : (wn & 1) * 2;
    f32x4 *swap = (f32x4 *)xs + l;        // [wavefront][a][2][lane]: two stages at most, and the last k-step reads the fourth
    if (BT == 1) {
#pragma unroll
      for (int a = 0; a < AT; ++a)
#pragma unroll
        for (int i = 0; i < 2; ++i) {   // an even wavefront (gate) hands on its groups 2 and 3, an odd one (up) 0 and 1
          f32x4 v;
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = wn & 1 ? acc[a][0][4 * i + e] : acc[a][0][4 * (i + 2) + e];
          swap[((wn * AT + a) * 2 + i) * 64] = v;
        }
      __syncthreads();
    }
    if (n0 >= n_end) return;
#pragma unroll
    for (int a = 0; a < AT; ++a) {
      const int m = m0 + (wm * AT + a) * 32 + lrow;
      bf16_t *y = Y + (int64_t)m * (N / 2) + (n0 >> 1) + half * 4;
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        f32x4 gte, up;
        if (BT == 2) {
#pragma unroll
          for (int e = 0; e < 4; ++e) { gte[e] = acc[a][0][4 * i + e]; up[e] = acc[a][BT - 1][4 * i + e]; }
        } else {
          const f32x4 other = swap[(((wn ^ 1) * AT + a) * 2 + i) * 64];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float mine = wn & 1 ? acc[a][0][4 * (i + 2) + e] : acc[a][0][4 * i + e];
            gte[e] = wn & 1 ? other[e] : mine;
            up[e] = wn & 1 ? mine : other[e];
          }
        }
        bf16x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = swiglu(gte[e], up[e]);
        if (m < M) *(bf16x4 *)(y + (i0 + i) * 8) = o;
      }
    }
  }
};

// One tile (column tile at n_tile0, rows from m0, K slice `split`) with the whole workgroup; the kernels below are thin
// wrappers that pick the tile(s) of a workgroup.  K slices are multiples of four k-steps (the host sees to it).
// FOLD: all K slices of `ksteps` k-steps in one go: every slice's sum starts from zero and is added to the
// running total in slice order, so the one result equals the sum a consumer makes of separate slices bit for bit.
template <int WM, int WN, int AT, int BT, int MODE, bool COLD, bool FOLD = false>
__device__ __forceinline__ void gemm_tile(bf16_t *xs, const bf16_t *__restrict__ X,
                                          const bf16_t *__restrict__ W, void *__restrict__ Yv, int M, int N, int K,
                                          int ksteps, int n_tile0, int m0, int split, int n_end, int ldy, int y_col0) {
  Tile<WM, WN, AT, BT, COLD> t;
  t.init(xs, X, W, M, N, K);
  const int nks = FOLD ? K / BK : min(ksteps, K / BK - split * ksteps);
  const auto p = t.part(n_tile0, m0, split * ksteps, M, N, K);
  t.zero();
  t.begin(p);
  f32x16 tot[FOLD ? AT : 1][FOLD ? BT : 1];
  int slice_end = ksteps;
  if constexpr (FOLD) {
#pragma unroll
    for (int a = 0; a < AT; ++a)
#pragma unroll
      for (int b = 0; b < BT; ++b)
#pragma unroll
        for (int i = 0; i < 16; ++i) tot[a][b][i] = 0.f;
  }
  auto fold = [&]() {
    if constexpr (FOLD) {
#pragma unroll
      for (int a = 0; a < AT; ++a)
#pragma unroll
        for (int b = 0; b < BT; ++b)
#pragma unroll
          for (int i = 0; i < 16; ++i) { tot[a][b][i] += t.acc[a][b][i]; t.acc[a][b][i] = 0.f; }
    }
  };
  int ks = 0;
  for (; ks < nks - 4; ks += 4) {
    if (FOLD && ks == slice_end) { fold(); slice_end += ksteps; }
    t.four(p, ks);
  }
  if (FOLD && ks == slice_end) fold();
  t.last_four(p, ks);
  if constexpr (FOLD) {
#pragma unroll
    for (int a = 0; a < AT; ++a)
#pragma unroll
      for (int b = 0; b < BT; ++b)
#pragma unroll
        for (int i = 0; i < 16; ++i) t.acc[a][b][i] += tot[a][b][i];
  }
  if constexpr (MODE == 0) t.store((float *)Yv + (int64_t)split * M * ldy, n_tile0, m0, M, n_end, ldy, y_col0);
  else t.store_swiglu((bf16_t *)Yv, n_tile0, m0, M, n_end, N);
}

template <int WM, int WN, int AT, int BT, int MODE, bool COLD>
__global__ __launch_bounds__(256) void gemm_kernel(const bf16_t *__restrict__ X, const bf16_t *__restrict__ W,
                                                   void *__restrict__ Yv, int M, int N, int K, int ksteps,
                                                   int n_base, int n_end, int nrow, int ldy, int y_col0) {
  constexpr int BM = WM * AT * 32, BN = WN * BT * 32;
  __shared__ __attribute__((aligned(1024))) bf16_t xs[Tile<WM, WN, AT, BT, false>::LDS];
  // Tile and K slice of this workgroup.  nrow = 0: (column tile, slice, row tile) = the block index.  nrow > 0:
  // a flat grid in which the row tiles of one column tile and slice sit 8 workgroup ids apart, so the hardware's
  // round-robin deal of consecutive ids to the 8 XCDs puts them on the same XCD at the same moment
  // and the second reader of a W tile finds it in that XCD's L2.
  int ctile = blockIdx.x, split = blockIdx.y, rtile = blockIdx.z;
  if (nrow > 0) {
    const int item = (blockIdx.x / (8 * nrow)) * 8 + (blockIdx.x & 7), nct = (n_end - n_base + BN - 1) / BN;
    rtile = (blockIdx.x >> 3) % nrow;
    ctile = item % nct;
    split = item / nct;
    if (split * ksteps * BK >= K) return;   // padding of the flat grid (uniform for the workgroup)
  }
  gemm_tile<WM, WN, AT, BT, MODE, COLD>(xs, X, W, Yv, M, N, K, ksteps, n_base + ctile * BN, rtile * BM, split, n_end, ldy, y_col0);
}

// Many rows (prompt passes): all K slices of a tile in one workgroup (FOLD; one slice: the plain sum).
// A flat grid of which the hardware deals consecutive ids to the 8 XCDs in turn: XCD i takes the i-th eighth of the tiles, so that all units
// have the same number whatever the shape (groups of 8 column tiles gave 12 of them as 2 and 1 per XCD), column tile by column tile or, ROWS,
// row tile by row tile: the order in which an eighth shares more of its operands.  us, groups of 8 column tiles -> so, same tiles: 1.5B O, 3000 rows,
// 160 x 128 33.7 -> 19.8, 1.5B down, 3000 rows, 140 -> 88, 2000 rows, 96 x 128 94 -> 57; 7B QKV, 1024 rows, 160 x 128 56 -> 36; 3000 rows, 128 x 256 128 -> 101.
// (128 x 256 tiles: the second set of accumulators leaves no register free and each fold moves 256; still the fastest where
// launch_gemm_folded takes it: down product of the 32B shape, 1536 rows, 375 us, 418 with the best of the 128-wide tiles.)
__device__ __forceinline__ void deal(int nrow, int ncol, bool rows, int &rtile, int &ctile) {
  const int tiles = nrow * ncol, xcd = blockIdx.x & 7;
  const int t = xcd * (tiles >> 3) + min(xcd, tiles & 7) + (blockIdx.x >> 3);
  const int slow = t / (rows ? ncol : nrow), fast = t - slow * (rows ? ncol : nrow);
  rtile = rows ? slow : fast;
  ctile = rows ? fast : slow;
}
template <int WM, int WN, int AT, int BT, bool FOLD>
__global__ __launch_bounds__(256) void gemm_fold_kernel(const bf16_t *__restrict__ X, const bf16_t *__restrict__ W,
                                                        void *__restrict__ Yv, int M, int N, int K, int ksteps, int nrow, bool rows) {
  constexpr int BM = WM * AT * 32, BN = WN * BT * 32;
  __shared__ __attribute__((aligned(1024))) bf16_t xs[Tile<WM, WN, AT, BT, false>::LDS];
  int rtile, ctile;
  deal(nrow, (N + BN - 1) / BN, rows, rtile, ctile);
  gemm_tile<WM, WN, AT, BT, 0, false, FOLD>(xs, X, W, Yv, M, N, K, ksteps, ctile * BN, rtile * BM, 0, N, N, 0);
}
// The SwiGLU product (MODE 1) of a pass over columns [n_begin, n_end), dealt like that; FOLD: columns whose K is in slices elsewhere.
template <int WM, int WN, int AT, int BT, int MODE, bool FOLD>
__global__ __launch_bounds__(256) void gemm_pass_kernel(const bf16_t *__restrict__ X, const bf16_t *__restrict__ W, void *__restrict__ Yv,
                                                        int M, int N, int K, int ksteps, int nrow, bool rows, int n_begin, int n_end) {
  constexpr int BM = WM * AT * 32, BN = WN * BT * 32;
  __shared__ __attribute__((aligned(1024))) bf16_t xs[Tile<WM, WN, AT, BT, false>::LDS];
  int rtile, ctile;
  deal(nrow, (n_end - n_begin + BN - 1) / BN, rows, rtile, ctile);
  gemm_tile<WM, WN, AT, BT, MODE, false, FOLD>(xs, X, W, Yv, M, N, K, ksteps, n_begin + ctile * BN, rtile * BM, 0, n_end, N, 0);
}

// Products of more 256 x 256 tiles than compute units: a workgroup of each takes tiles one after the other and loads the first
// k-steps of the next one under the last products of the tile at hand, so that the pipeline fills once and not
// once per round (one tile fills a compute unit: no other workgroup could work meanwhile).  Tiles below n_big are those of columns
// [0, n_cut), all K slices (mode 0); the columns behind, which would be a nearly empty last round, go in 256 x 128 tiles.
// One launch of a workgroup per tile and this kernel: gate/up of the 1.5B shape, 3000 rows (840 tiles), 166 and 154 us, its down product
// (648) 112 and 104; LM head of the 7B shape, 256 rows (594), 337 and 322, 129 rows 303 and 279; 7B down as one slice, 512 rows, 171 and 146.
template <int MODE, bool COLD>
__global__ __launch_bounds__(256) void gemm_rounds_kernel(const bf16_t *__restrict__ X, const bf16_t *__restrict__ W,
                                                          void *__restrict__ Yv, int M, int N, int K, int ksteps, int n_cut, int n_big, int n_left) {
  using Big = Tile<1, 4, 8, 2, COLD>;
  __shared__ __attribute__((aligned(1024))) bf16_t xs[Big::LDS];
  const int nrow = (M + 255) / 256, per = MODE == 0 ? ksteps : K / BK;
  struct At { int m0, n0, split; };
  // tile `i` of column tiles `width` wide from `n_begin`: row tiles of a column tile and slice 8 apart, padded as everywhere
  auto at = [&](int i, int n_begin, int n_end, int width) {
    const int item = (i / (8 * nrow)) * 8 + (i & 7), nct = (n_end - n_begin + width - 1) / width;
    return At{(i >> 3) % nrow * 256, n_begin + item % nct * width, item / nct};
  };
  const int slices = MODE == 0 ? (K / BK + per - 1) / per : 1;
  auto next = [&](int i) {   // the first tile from i on that is none of the grid's padding
    while (i < n_big && at(i, 0, n_cut, 256).split >= slices) i += gridDim.x;
    return i;
  };
  int i = next(blockIdx.x);
  if (i < n_big) {   // (all of this is uniform for the workgroup)
    Big t;
    t.init(xs, X, W, M, N, K);
    At c = at(i, 0, n_cut, 256);
    auto p = t.part(c.n0, c.m0, c.split * per, M, N, K);
    t.zero();
    t.begin(p);
    for (;;) {
      const int nks = min(per, K / BK - c.split * per), n = next(i + gridDim.x);
      const At d = n < n_big ? at(n, 0, n_cut, 256) : c;   // behind the last tile: its own first k-steps again, which nothing reads
      int ks = 0;
      for (; ks < nks - 4; ks += 4) t.four(p, ks);
      t.template kstep<0, true, 3>(p, ks + 3);
      p = t.part(d.n0, d.m0, d.split * per, M, N, K);
      t.template kstep<1, true, 3>(p, 0);
      t.template kstep<2, true, 3>(p, 1);
      t.template kstep<3, true, 3>(p, 2);
      if constexpr (MODE == 0) t.store((float *)Yv + (int64_t)c.split * M * N, c.n0, c.m0, M, n_cut, N, 0);
      else t.store_swiglu((bf16_t *)Yv, c.n0, c.m0, M, n_cut, N);
      if (n >= n_big) break;
      t.zero();
      c = d;
      i = n;
    }
    t.drain();
    __syncthreads();
  }
  for (int j = blockIdx.x; j < n_left; j += gridDim.x) {
    const At c = at(j, n_cut, N, 128);
    if (c.split >= slices) continue;
    gemm_tile<1, 4, 8, 1, MODE, COLD>(xs, X, W, Yv, M, N, K, per, c.n0, c.m0, c.split, N, N, 0);
    __syncthreads();   // (the next tile's first stages, and the halves that neighbours swap, share the LDS)
  }
}

// The SwiGLU product of a 129..256-row batch in one launch.  Main tiles (128 x 256, row tiles paired on an XCD as above) fill the chip once; the columns left
// over beyond them, [n_main, N), whose K is added up in slices by batches of fewer rows, are 64 x 128 tiles with the slices added up in the workgroup, ahead of the main
// tiles: a unit that has one takes its main tile when it is done, and nothing is written and read again.  Bound by what a compute unit gets from the caches (48 KB per k-step at
// 45 KB/us) in both.  7B shape, 256 / 129 rows: 80 / 81 us; the K slices of the remainder behind the main tiles, written as partial sums for a launch that adds them up, 85 / 85.
template <int WM, int WN, int AT, int BT, int MODE, bool COLD>
__global__ __launch_bounds__(256) void gemm_ahead_kernel(const bf16_t *__restrict__ X, const bf16_t *__restrict__ W, void *__restrict__ mid, int M, int N,
                                                         int K, int ksteps, int n_main, int n_ahead) {
  constexpr int BM = WM * AT * 32, BN = WN * BT * 32;
  __shared__ __attribute__((aligned(1024))) bf16_t xs[Tile<WM, WN, AT, BT, false>::LDS];
  if ((int)blockIdx.x < n_ahead) {   // uniform for the workgroup
    const int nr = (M + 63) / 64, nc = (N - n_main + 127) / 128, tiles = nr * nc;
    if ((int)(blockIdx.x >> 3) >= (tiles >> 3) + ((int)(blockIdx.x & 7) < (tiles & 7) ? 1 : 0)) return;   // padding of the grid
    int rtile, ctile;
    deal(nr, nc, false, rtile, ctile);
    gemm_tile<1, 4, 2, 1, MODE, false, true>(xs, X, W, mid, M, N, K, ksteps, n_main + ctile * 128, rtile * 64, 0, N, N, 0);
    return;
  }
  const int nrow = (M + BM - 1) / BM, i = blockIdx.x - n_ahead;
  const int rtile = (i >> 3) % nrow, ctile = (i / (8 * nrow)) * 8 + (i & 7);
  if (ctile * BN < n_main) gemm_tile<WM, WN, AT, BT, MODE, COLD>(xs, X, W, mid, M, N, K, K / BK, ctile * BN, rtile * BM, 0, n_main, N, 0);
}

// The same product in calls of at most one row tile: workgroups
// below n_tiles take the main tiles, the others the K slices of the remainder, in one launch.  Tiles of 128 columns: 7B shape, 19 / 64 / 128
// rows 45 / 48 / 60 us with the reduction, by 256 (64 rows: 128) columns 49 / 56 / 68.  The two launches
// in a row each left part of the chip idle: 7B shape, 19 rows, 43 + 11 us and a gap; joined 50.
template <int WM, int WN, int AT, int BT, bool COLD>
__global__ __launch_bounds__(256) void gemm_gu_joint_kernel(const bf16_t *__restrict__ X, const bf16_t *__restrict__ W,
                                                            bf16_t *__restrict__ mid, float *__restrict__ ws, int M, int N,
                                                            int K, int n_main, int n_tiles, int rem_splits, int rem_ksteps) {
  constexpr int BN = WN * BT * 32;
  __shared__ __attribute__((aligned(1024))) bf16_t xs[Tile<WM, WN, AT, BT, false>::LDS];
  const int item = (int)blockIdx.x - n_tiles;
  if (item < 0)   // uniform for the workgroup
    gemm_tile<WM, WN, AT, BT, 1, COLD>(xs, X, W, mid, M, N, K, K / BK, (int)blockIdx.x * BN, 0, 0, n_main, 0, 0);
  else
    gemm_tile<WM, WN, AT, BT, 0, COLD>(xs, X, W, ws, M, N, K, rem_ksteps, n_main + item / rem_splits * BN, 0, item % rem_splits, N,
                                 N - n_main, n_main);
}

// SwiGLU over K-split partial sums: parts [splits][M][ld] holds columns [col0, col0 + ld) of the
// interleaved gate/up product (blocks of 64 columns: 32 gate, then the 32 matching up columns);
// mid[m][(col0 + c) / 2 ...] = silu(sum_s gate) * (sum_s up), slices added in order.
// Four outputs of a row per thread.
template <int SL>
__global__ __launch_bounds__(256) void swiglu_reduce_kernel(const float *__restrict__ parts, int splits, int M, int ld,
                                                            int col0, bf16_t *__restrict__ mid, int F) {
  const int j = (blockIdx.x * blockDim.x + threadIdx.x) * 4, m = blockIdx.y;   // (ld is a multiple of 64)
  if (j >= ld / 2) return;
  const f32x4 *row = (const f32x4 *)(parts + (int64_t)m * ld + (j >> 5) * 64 + (j & 31));
  const int64_t stride = (int64_t)M * (ld / 4);
  const f32x4 g = sum_slices<SL>(row, splits, stride), u = sum_slices<SL>(row + 8, splits, stride);
  bf16x4 o;
#pragma unroll
  for (int i = 0; i < 4; ++i) o[i] = swiglu(g[i], u[i]);
  *(bf16x4 *)(mid + (int64_t)m * F + (col0 >> 1) + j) = o;
}

struct Launch {
  const bf16_t *x, *w;
  void *y;
  int M, N, K, mode, splits, n_begin, n_end, ldy, y_col0;
  bool paired, cold;
  hipStream_t s;
};

// calls f(bool constant), true where the tile shape has a kernel of its own for cold weights
template <int WM, typename F>
void with_cold(bool cold, F f) {
  if (WM == 1 && cold) f(std::bool_constant<WM == 1>{}); else f(std::false_type{});
}

// Launch over output columns [n_begin, n_end) (multiples of the tile width, except the matrix edge).
template <int WM, int WN, int AT, int BT>
int launch_cfg(const Launch &L) {
  constexpr int BM = WM * AT * 32, BN = WN * BT * 32;
  if (L.n_end <= L.n_begin) return 0;
  if (BT == 1 && WM > 1 && L.mode == 1) return -1;   // gate and up tiles of a block: in one wavefront or in neighbours
  dim3 grid((L.n_end - L.n_begin + BN - 1) / BN, L.splits, (L.M + BM - 1) / BM);
  int nrow = 0;
  if (L.paired) {   // flat grid, column tiles and slices padded to a multiple of 8 (see the kernel)
    nrow = grid.z;
    grid.x = ((grid.x * L.splits + 7) / 8) * 8 * nrow;
    grid.y = grid.z = 1;
  }
  int ksteps = 4 * ((L.K / (4 * BK) + L.splits - 1) / L.splits);
  with_cold<WM>(L.cold, [&](auto COLD) {
    constexpr bool cold = decltype(COLD)::value;
    if (L.mode == 0)
      hipLaunchKernelGGL((gemm_kernel<WM, WN, AT, BT, 0, cold>), grid, dim3(256), 0, L.s, L.x, L.w, L.y, L.M, L.N, L.K, ksteps,
                         L.n_begin, L.n_end, nrow, L.ldy, L.y_col0);
    else
      hipLaunchKernelGGL((gemm_kernel<WM, WN, AT, (BT > 1 || WM == 1 ? BT : 2), 1, cold>), grid, dim3(256), 0, L.s, L.x, L.w, L.y, L.M, L.N,
                         L.K, ksteps, L.n_begin, L.n_end, nrow, L.ldy, L.y_col0);
  });
  return hipGetLastError() == hipSuccess ? 0 : -7;
}

int launch_by_id(int cfg, const Launch &L) {
  switch (cfg) {
    case GEMM_32x256: return launch_cfg<1, 4, 1, 2>(L);
    case GEMM_64x256: return launch_cfg<1, 4, 2, 2>(L);
    case GEMM_128x256: return launch_cfg<1, 4, 4, 2>(L);
    case GEMM_64x128: return launch_cfg<2, 2, 1, 2>(L);
    case GEMM_128x128: return launch_cfg<2, 2, 2, 2>(L);
    case GEMM_256x128: return launch_cfg<2, 2, 4, 2>(L);
    case GEMM_64x64: return launch_cfg<2, 2, 1, 1>(L);
    case GEMM_128x64: return launch_cfg<2, 2, 2, 1>(L);
    case GEMM_32x128: return launch_cfg<1, 4, 1, 1>(L);
    case GEMM_128x64P: return launch_cfg<4, 1, 1, 2>(L);
    case GEMM_256x64P: return launch_cfg<4, 1, 2, 2>(L);
    case GEMM_128x128R: return launch_cfg<1, 4, 4, 1>(L);
    case GEMM_256x128R: return launch_cfg<1, 4, 8, 1>(L);
    case GEMM_64x128R: return launch_cfg<1, 4, 2, 1>(L);
    case GEMM_256x256: return launch_cfg<1, 4, 8, 2>(L);
    default: return -1;
  }
}

// A plain product of many rows, K in `splits` slices added up in the workgroup (one slice: no second set of accumulators).  An eighth of the tiles
// reads all rows and an eighth of the columns or the other way round; the line between the orders lies where both take the same time (128 x 256 tiles, column /
// row order: 7B O, 2000 / 3000 / 4096 rows 47.8 / 85.8 / 103.9 and 48.8 / 87.9 / 101.2 us; 32B QKV, 3000 rows, 216 and 239; 1.5B O, 3000 rows, 96 x 128, 23.1 and 20.5).
template <int WM, int WN, int AT, int BT>
int launch_fold_cfg(const Launch &L) {
  constexpr int BM = WM * AT * 32, BN = WN * BT * 32;
  const int nrow = (L.M + BM - 1) / BM, grid = (L.N + BN - 1) / BN * nrow;
  const int ksteps = 4 * ((L.K / (4 * BK) + L.splits - 1) / L.splits);
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(256), 0, L.s, L.x, L.w, L.y, L.M, L.N, L.K, ksteps, nrow, (int64_t)L.M * 5 >= (int64_t)L.N * 4);
  };
  if (L.splits == 1) launch(gemm_fold_kernel<WM, WN, AT, BT, false>);
  else launch(gemm_fold_kernel<WM, WN, AT, BT, true>);
  return hipGetLastError() == hipSuccess ? 0 : -7;
}

template <int AT, int BT, bool FOLD>
int launch_pass_cfg(const Launch &L, int slices) {
  constexpr int BM = AT * 32, BN = BT * 128;
  const int nrow = (L.M + BM - 1) / BM, cols = L.n_end - L.n_begin, ksteps = 4 * ((L.K / (4 * BK) + slices - 1) / slices);
  hipLaunchKernelGGL((gemm_pass_kernel<1, 4, AT, BT, 1, FOLD>), dim3(nrow * ((cols + BN - 1) / BN)), dim3(256), 0, L.s, L.x, L.w, L.y, L.M, L.N, L.K,
                     ksteps, nrow, (int64_t)L.M * 5 >= (int64_t)cols * 4, L.n_begin, L.n_end);
  return hipGetLastError() == hipSuccess ? 0 : -7;
}

// Columns [0, n_cut) by 256 x 256 tiles, a workgroup per compute unit, the rest by 256 x 128 tiles in the same launch.
int launch_rounds(const Launch &L, int n_cut) {
  const int nrow = (L.M + 255) / 256, splits = L.mode == 0 ? L.splits : 1;
  if (n_cut >= L.N && (L.N + 255) / 256 * splits * nrow <= 256) return launch_cfg<1, 4, 8, 2>(L);   // a tile each
  const int big = ((n_cut + 255) / 256 * splits + 7) / 8 * 8 * nrow, left = ((L.N - n_cut + 127) / 128 * splits + 7) / 8 * 8 * nrow;
  const int ksteps = 4 * ((L.K / (4 * BK) + splits - 1) / splits);
  with_cold<1>(L.cold, [&](auto COLD) {
    auto launch = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, dim3(256), dim3(256), 0, L.s, L.x, L.w, L.y, L.M, L.N, L.K, ksteps, n_cut, big, n_cut < L.N ? left : 0);
    };
    constexpr bool cold = decltype(COLD)::value;
    if (L.mode == 1) launch(gemm_rounds_kernel<1, cold>); else launch(gemm_rounds_kernel<0, cold>);
  });
  return hipGetLastError() == hipSuccess ? 0 : -7;
}

bool splits_valid(int K, int splits) {
  const int total = K / (4 * BK);
  return splits >= 1 && splits <= total && (splits - 1) * ((total + splits - 1) / splits) < total;   // no empty slice
}

int swiglu_reduce(const float *parts, int splits, int M, int ld, int col0, bf16_t *mid, int F, hipStream_t s) {
  const int quads = ld / 8, blocks = (quads + 255) / 256, nt = ((quads + blocks - 1) / blocks + 63) / 64 * 64;
  with_slices(splits, [&](auto SL) {
    hipLaunchKernelGGL(swiglu_reduce_kernel<decltype(SL)::value>, dim3(blocks, M), dim3(nt), 0, s, parts, splits, M, ld, col0, mid, F);
  });
  return hipGetLastError() == hipSuccess ? 0 : -7;
}

}  // namespace


// Microseconds of a product by tiles of one shape, as measured: fixed + out * MB written + k-steps of a workgroup * (base + load *
// (fraction of the compute units at work) + round * (workgroups on the fullest unit - 1) + more * (average beyond one)).
// Fits by hand to 10000 launches (the products of the 1.5B, 7B and 32B shapes, 1 to 512 rows, 1 to 9 slices, weights in and out of the
// last-level cache): the shape with the least is the best measured one within 2.5 % on average (11 % in 95 of 100).
struct ShapeTime { int cfg, log_rows, log_cols; float fixed, base, load, round, more, out; };
constexpr ShapeTime SHAPES[] = {
    {GEMM_32x128, 5, 7, 5.2f, 0.23f, 0.13f, 0.42f, 0.26f, 0.f},   {GEMM_64x128R, 6, 7, 5.3f, 0.24f, 0.20f, 0.53f, 0.30f, 0.05f},
    {GEMM_64x64, 6, 6, 5.1f, 0.22f, 0.05f, 0.20f, 0.20f, 0.15f},   {GEMM_128x64, 7, 6, 4.9f, 0.26f, 0.12f, 0.28f, 0.25f, 0.13f},
    {GEMM_128x128R, 7, 7, 5.3f, 0.31f, 0.31f, 0.80f, 0.10f, 0.15f}, {GEMM_128x128, 7, 7, 5.5f, 0.40f, 0.35f, 0.f, 0.60f, 0.15f},
    {GEMM_32x256, 5, 8, 6.0f, 0.40f, 0.55f, 0.70f, 0.50f, 0.f},   {GEMM_64x256, 6, 8, 6.3f, 0.50f, 0.55f, 0.80f, 0.65f, 0.f},
    {GEMM_128x256, 7, 8, 6.3f, 0.59f, 0.41f, 1.0f, 0.40f, 0.16f}, {GEMM_256x128R, 8, 7, 5.5f, 0.50f, 0.39f, 0.90f, 0.28f, 0.25f},
    {GEMM_256x256, 8, 8, 7.7f, 0.84f, 0.62f, 1.45f, 0.50f, 0.23f}};

int gemm_tile_rows(int cfg) {
  for (const ShapeTime &t : SHAPES)
    if (t.cfg == cfg) return 1 << t.log_rows;
  return 0;
}

// us per k-step of this many 256 x 256 tiles
float big_rounds(int64_t tiles) { return tiles / 256 * 1.45f + (tiles % 256 ? 1.05f + tiles % 256 * (0.4f / 256) : 0.f); }

// Columns that launch_rounds gives to 256 x 256 tiles: all, or full rounds of them where what is left fits one round of 256 x 128 tiles
// (0.89 us per k-step when they fill the chip, 0.5 when few) in less time; *us: per k-step.
int rounds_cut(int M, int N, int splits, float *us) {
  const int per = (M + 255) / 256 * splits, ncol = (N + 255) / 256, cut = ncol * per / 256 * 256 / per, left = (N - cut * 256 + 127) / 128 * per;
  *us = big_rounds((int64_t)ncol * per);
  if (cut == 0 || cut == ncol || left > 256) return N;
  const float with = big_rounds((int64_t)cut * per / 256 * 256) + (cut * per % 256 ? 1.45f : 0.f) + 0.5f + left * (0.39f / 256);
  if (with >= *us) return N;
  *us = with;
  return cut * 256;
}

// Tile shape of a call.  Shapes whose wavefronts stack rows have no SwiGLU pairs (64 x 64, 128 x 64); 64 x 64 tiles for up to 32 rows
// pay only where W comes from memory (7B down in one slice, 16 rows: 75 us, by 32 x 128 tiles 95; O from the cache 10.6 and 10.0); 128 x 128
// tiles in two rows of two are a second choice where two of them share a unit.  256 x 256 tiles in rounds only from 129 rows on: half of a tile's
// products would be of rows that are not there (LM head of the 7B / 32B / 1.5B shape, 128 rows, 256 / 348 / 125 us, by 128 x 256 226 / 304 / 116; 96 rows 246 / 361 / 116
// and 213 / 291 / 110; 160 rows 261 / 360 / 129 and 291 / 402 / 145).
int pick_shape(int M, int N, int K, int mode, int splits, bool cold) {
  const float ksteps = 4 * ((K / (4 * BK) + splits - 1) / splits), out_mb = 4e-6f * M * N * (mode == 0 ? splits : 0.25f);
  const float floor_us = 2e-6f / 6.6f * N * K + 3;
  int best = -1;
  float best_us = 0;
  for (const ShapeTime &t : SHAPES) {   // (in a caller's launch path: no divisions)
    const int rows = 1 << t.log_rows;
    if ((rows > 64 && rows >= 4 * M) || rows * 5 < M) continue;
    const int n = ((M + rows - 1) >> t.log_rows) * ((N + (1 << t.log_cols) - 1) >> t.log_cols) * splits;
    if (t.cfg == GEMM_64x64 && (mode == 1 || (M <= 32 && !cold))) continue;
    if ((t.cfg == GEMM_128x64 && mode == 1) || (t.cfg == GEMM_128x128 && n > 512) || (t.cfg == GEMM_256x256 && n > 256 && M <= 128)) continue;
    const float r = n * (1.f / 256);
    float us = t.fixed + t.out * out_mb + ksteps * (t.base + t.load * std::min(r, 1.f) + t.round * ((n + 255) / 256 - 1) + t.more * std::max(r - 1, 0.f));
    if (t.cfg == GEMM_256x256 && n > 256) {
      rounds_cut(M, N, splits, &us);
      us = t.fixed + ksteps * us;   // (what earlier rounds write goes out under later ones)
    }
    const float bound = std::max(us, floor_us + r * 0.128f);
    if (best < 0 || bound < best_us) { best = t.cfg; best_us = bound; }
  }
  return best;
}

// One launch of one tile configuration over a column range (tuning and tests).  mode 1 with
// splits > 1 writes fp32 partials to ws and finishes with the SwiGLU reduction.
int launch_gemm_cfg(int cfg, const bf16_t *x, const bf16_t *w, void *y, float *ws, int M, int N, int K, int mode,
                    int splits, int n_begin, int n_end, bool paired, bool cold, hipStream_t s) {
  if (M < 1 || M > 512 || K % (4 * BK) || N % 32 || !splits_valid(K, splits)) return -1;
  if (mode != 0 && mode != 1) return -1;
  if (mode == 1 && (N % 64 || n_begin % 64 || n_end % 64)) return -1;
  if (n_begin < 0 || n_end > N || n_begin % 32 || n_end % 32) return -1;
  if ((int64_t)N * K * 2 >= GEMM_MAX_OPERAND_BYTES || (int64_t)M * K * 2 >= GEMM_MAX_OPERAND_BYTES) return -1;
  if (paired && splits != 1 && mode == 1) return -1;
  Launch L{x, w, y, M, N, K, mode, splits, n_begin, n_end, N, 0, paired, cold, s};
  if (mode == 1 && splits > 1) {
    if (!ws) return -1;
    L.mode = 0; L.y = ws; L.ldy = n_end - n_begin; L.y_col0 = n_begin;
    int rc = launch_by_id(cfg, L);
    return rc ? rc : swiglu_reduce(ws, splits, M, n_end - n_begin, n_begin, (bf16_t *)y, N / 2, s);
  }
  return launch_by_id(cfg, L);
}

// K split of a mode-0 product for calls of up to M rows.  The tile shapes named here are the ones
// launch_gemm uses for such calls; the counts come from sweeps over tile shape and split count at the
// benchmark's shapes (weights cold, launches back to back): a launch costs a fixed 3-9 us (first
// loads, drain, partial sums written) plus its weight bytes at 3.5-4.5 TB/s, so narrow outputs want
// about one workgroup per compute unit and as few slices as that allows.
int gemm_pick_splits(int M, int N, int K) {
  auto largest = [&](int tiles, int cap) {
    int best = 1;
    for (int sp = 2; sp <= 32 && tiles * sp <= cap; ++sp)
      if (splits_valid(K, sp)) best = sp;
    return best;
  };
  if (M <= 32 && N < 16384) return largest((N + 127) / 128, 256);               // 32 x 128 tiles
  if (M <= 64 && N < 16384) return largest((N + 63) / 64, 256);                 // 64 x 64 tiles
  if (M <= 128) return largest((N + 255) / 256, 256);                           // 128 x 256 tiles
  // 129..256 rows: at these rows two, three or four slices of the short-K products (QKV, O) and eight or
  // nine of the long one (down) take the same time within a microsecond; the larger counts are kept
  // because an engine sized for 256 rows also runs steps of a few rows (a batch that is not refilled
  // decays), and with few rows the bytes in flight, hence the weight bandwidth, grow with the slices.
  if (M <= 256 && K <= 4096 && splits_valid(K, 4)) return 4;                    // 128 x 128 tiles
  return largest(((N + 127) / 128) * ((M + 255) / 256), 256);                   // 256 x 128 tiles
}

// How K is split for a product, as a function of the LARGEST row count the caller will ever pass
// (so that every pass, whatever its row count, adds up each output element in the same order).
// mode 0: one split count for all columns (the caller's output holds that many slices).
// mode 1: columns [0, n_main) with `splits` slices, columns [n_main, N) with `rem_splits`; wherever a
// count exceeds 1 the partial sums go through the workspace and the SwiGLU is applied by a reduction.
// Launched on their own, no SwiGLU product gained from a K split in the sweeps (64 x 128 tiles fill the
// chip for narrow batches).  The one split chosen is the column remainder of a wide product at 129..256
// rows, whose slices ride in the launch of the main tiles (gemm_gu_joint_kernel; 129 to 256 rows add them up in the workgroup, gemm_ahead_kernel).
GemmSplit gemm_pick_split(int M_max, int N, int K, int mode) {
  GemmSplit ks{1, N, 1};
  if (mode == 0) {
    ks.splits = gemm_pick_splits(M_max, N, K);
    return ks;
  }
  if (M_max > 128 && M_max <= 256 && N >= 128 * 256) {
    // 128 x 256 tiles, two row tiles: what is left over a multiple of 256 tiles is split along K so that
    // every compute unit gets one slice on top of its main tile
    const int ctiles = (N + 255) / 256, tiles = 2 * ctiles, rem = tiles % 256;
    if (tiles > 256 && rem > 0 && rem <= 96) {
      int best = 1;
      for (int sp = 2; sp <= 16 && rem * sp <= 256; ++sp)
        if (splits_valid(K, sp)) best = sp;
      if (best > 1) {
        ks.n_main = ((tiles - rem) / 2) * 256;
        ks.rem_splits = best;
      }
    }
  }
  return ks;
}

// fp32 elements of workspace a mode-1 product of up to M_max rows needs (0 if K is not split)
int64_t gemm_workspace_elems(int M_max, int N, const GemmSplit &ks) {
  int64_t need = 0;
  if (ks.splits > 1) need = (int64_t)ks.splits * M_max * ks.n_main;
  if (ks.n_main < N && ks.rem_splits > 1) need = std::max<int64_t>(need, (int64_t)ks.rem_splits * M_max * (N - ks.n_main));
  return need;
}

int launch_gemm(const bf16_t *x, const bf16_t *w, void *y, float *ws, int M, int N, int K, int mode,
                const GemmSplit &ks, bool cold, hipStream_t s) {
  if (M < 1 || M > 512 || K % (4 * BK) || N % 32 || !splits_valid(K, ks.splits)) return -1;
  if (mode != 0 && mode != 1) return -1;
  if (mode == 1 && (N % 64 || ks.n_main % 64 || !splits_valid(K, ks.rem_splits))) return -1;
  if (mode == 0 && ks.n_main != N) return -1;
  if (ks.n_main < 0 || ks.n_main > N) return -1;
  if ((int64_t)N * K * 2 >= GEMM_MAX_OPERAND_BYTES || (int64_t)M * K * 2 >= GEMM_MAX_OPERAND_BYTES) return -1;
  if (mode == 1 && M <= 256 && ks.n_main < N && ks.rem_splits > 1 && ks.splits == 1 && (ws || M > 128)) {
    // main tiles and K slices of the remainder in one launch; up to 128 rows the SwiGLU over the slices follows
    const int rem_ksteps = 4 * ((K / (4 * BK) + ks.rem_splits - 1) / ks.rem_splits);
    if (M > 128) {
      const int ahead = ((M + 63) / 64 * ((N - ks.n_main + 127) / 128) + 7) / 8 * 8, nrow = (M + 127) / 128;
      with_cold<1>(cold && M >= 192, [&](auto COLD) {
        hipLaunchKernelGGL((gemm_ahead_kernel<1, 4, 4, 2, 1, decltype(COLD)::value>), dim3(ahead + ((ks.n_main + 255) / 256 + 7) / 8 * 8 * nrow), dim3(256), 0, s, x,
                           w, y, M, N, K, rem_ksteps, ks.n_main, ahead);
      });
      return hipGetLastError() == hipSuccess ? 0 : -7;
    } else {
      const int n_tiles = (ks.n_main + 127) / 128;
      const dim3 grid(n_tiles + (N - ks.n_main + 127) / 128 * ks.rem_splits);
      with_cold<1>(cold, [&](auto COLD) {
        constexpr bool c = decltype(COLD)::value;
        auto launch = [&](auto kernel) {
          hipLaunchKernelGGL(kernel, grid, dim3(256), 0, s, x, w, (bf16_t *)y, ws, M, N, K, ks.n_main, n_tiles, ks.rem_splits, rem_ksteps);
        };
        if (M <= 32) launch(gemm_gu_joint_kernel<1, 4, 1, 1, c>);
        else if (M <= 64) launch(gemm_gu_joint_kernel<1, 4, 2, 1, c>);
        else launch(gemm_gu_joint_kernel<1, 4, 4, 1, c>);
      });
    }
    if (hipGetLastError() != hipSuccess) return -7;
    return swiglu_reduce(ws, ks.rem_splits, M, N - ks.n_main, ks.n_main, (bf16_t *)y, N / 2, s);
  }
  if (ks.n_main != N) return -1;
  const int cfg = pick_shape(M, N, K, mode, ks.splits, cold);
  const bool paired = M > gemm_tile_rows(cfg);
  // A second row tile of a few rows runs through its W ahead of the first one's loads, which then find nothing in L2 if they
  // are non-temporal: LM head of the 7B / 32B shape by 128 x 256 tiles, 129 rows 287 / 474 us with ordinary, 318 / 550 with non-temporal
  // loads, 160 rows 295 / 473 and 301 / 502, 192 rows 303 / 457 and 300 / 438.
  if (paired && (M - 1) % gemm_tile_rows(cfg) < gemm_tile_rows(cfg) / 2) cold = false;
  if (cfg == GEMM_256x256 && (mode == 0 || ks.splits == 1) && (M + 255) / 256 * ((N + 255) / 256) * ks.splits > 256) {
    float us;
    return launch_rounds(Launch{x, w, y, M, N, K, mode, ks.splits, 0, N, N, 0, true, cold, s}, rounds_cut(M, N, ks.splits, &us));
  }
  return launch_gemm_cfg(cfg, x, w, y, ws, M, N, K, mode, ks.splits, 0, N, paired && (mode == 0 || ks.splits == 1), cold, s);
}

// Microseconds of a folded product by tiles of one shape: fixed + k-steps * (base + load * (fraction of the compute units at work) + round * (tiles of
// the fullest unit - 1) + more * (average beyond one)).  Fits to 1264 launches (the products of the 1.5B, 7B and 32B shapes, 260 to 4096 rows): the shape with the
// least takes 0.3 % more than the best measured one on average, 1.4 % in 95 of 100.  128-wide tiles by four wavefronts side by side, which load no W twice.
// Before tiles were dealt evenly and with six shapes, us: 1.5B O, 3000 rows, 24.8, now 20; 7B QKV, 511 / 1024 / 3000 rows 24 / 42 / 126, now 23 / 36 / 101; 7B O, 511
// / 3000 rows 21 / 93, now 18 / 82; 32B QKV, 4096 rows, 382, now 301 (all of the sweep 11 % less on average).
struct FoldTime { int rows, cols; float fixed, base, load, round, more; };
constexpr FoldTime FOLDS[] = {{64, 64, 2.7f, 0.180f, 0.063f, 0.146f, 0.114f},  {64, 128, 3.0f, 0.230f, 0.107f, 0.167f, 0.183f},
                              {96, 128, 4.1f, 0.290f, 0.110f, 0.203f, 0.279f}, {128, 128, 5.8f, 0.308f, 0.172f, 0.295f, 0.323f},
                              {160, 128, 6.7f, 0.361f, 0.188f, 0.353f, 0.361f}, {192, 128, 8.1f, 0.406f, 0.224f, 0.443f, 0.374f},
                              {128, 256, 8.8f, 0.522f, 0.271f, 0.511f, 0.473f}};
static int least(const FoldTime *f0, int from, int to, int M, int N, int K, float *us) {
  int best = from;
  for (int i = from; i < to; ++i) {
    const FoldTime &f = f0[i];
    const int n = (M + f.rows - 1) / f.rows * ((N + f.cols - 1) / f.cols);
    const float r = n * (1.f / 256);
    const float t = f.fixed + K / BK * (f.base + f.load * std::min(r, 1.f) + f.round * ((n + 255) / 256 - 1) + f.more * std::max(r - 1, 0.f));
    if (i == from || t < *us) { best = i; *us = t; }
  }
  return best;
}
static int fold_shape(int M, int N, int K, float *us) { return least(FOLDS, 0, 7, M, N, K, us); }

// The same of a pass's SwiGLU product: fits to 512 launches (1.5B, 7B and 32B shapes, 260 to 4096 rows); the shape with the least takes 0.2 % more than
// the best measured one on average.  Against 128 x 256 and 128 x 128 tiles in groups of eight column tiles or rounds of 256 x 256, us: 1.5B 300 / 511 / 640 / 1024 / 1300 rows
// 33 / 41 / 44 / 72 / 84, now 25 / 33 / 38 / 57 / 68, 3000 rows 159 -> 155; 7B 511 / 640 / 1300 143 / 175 / 328, now 132 / 154 / 298; 32B 260 / 640 / 1300 214 / 366 / 726,
// now 161 / 315 / 567.
constexpr FoldTime PASSES[] = {{128, 256, 11.3f, 0.f, 0.769f, 0.546f, 0.347f},   {160, 256, 12.9f, 0.354f, 0.447f, 0.767f, 0.270f},
                               {192, 256, 15.8f, 0.294f, 0.610f, 0.917f, 0.293f}, {224, 256, 18.7f, 0.110f, 0.912f, 0.933f, 0.481f},
                               {256, 256, 23.6f, 0.028f, 1.126f, 1.124f, 0.491f}};

// A product of up to GEMM_MAX_ROWS rows with all K slices of an element added up in the workgroup, in slice
// order: y is ONE slice (mode 0: [M][N]; mode 1: the SwiGLU result), equal bit for bit to what a consumer of
// launch_gemm's slices gets by adding them in order.  From 257 rows on the tiles alone fill the chip, and the
// partial sums that a K split writes and its consumer reads (33 MB per 256 rows of the 7B down projection)
// are saved.  Measured at 1024 rows against four 256-row launches, consumers' reads not counted: QKV / O / gate-up
// / down of the 1.5B shape 14 / 13 / 73 / 52 against 50 / 43 / 116 / 100 us, of the 7B shape 53 / 37 / 288 / 189
// against 82 / 71 / 350 / 200 us.
int launch_gemm_folded(const bf16_t *x, const bf16_t *w, void *y, int M, int N, int K, int mode, const GemmSplit &ks, hipStream_t s) {
  if (M < 1 || M > GEMM_MAX_ROWS || K % (4 * BK) || N % 32 || !splits_valid(K, ks.splits)) return -1;
  if (mode != 0 && mode != 1) return -1;
  if (mode == 1 && (N % 64 || ks.n_main % 64 || !splits_valid(K, ks.rem_splits))) return -1;
  if (mode == 0 && ks.n_main != N) return -1;
  if (ks.n_main < 0 || ks.n_main > N) return -1;
  if ((int64_t)N * K * 2 >= GEMM_MAX_OPERAND_BYTES || (int64_t)M * K * 2 >= GEMM_MAX_OPERAND_BYTES) return -1;
  Launch L{x, w, y, M, N, K, mode, ks.splits, 0, ks.n_main, N, 0, true, false, s};
  float us;
  if (mode == 1) {
    if (ks.splits > 1) return -1;   // (gemm_pick_split leaves the main columns whole)
    auto narrow = [&](int n_begin, int n_end, int slices, auto FOLD) {   // by 128-wide tiles
      constexpr bool fold = decltype(FOLD)::value;
      L.n_begin = n_begin;
      L.n_end = n_end;
      switch (least(FOLDS, 1, 6, M, n_end - n_begin, K, &us)) {
        case 1: return launch_pass_cfg<2, 1, fold>(L, slices);
        case 2: return launch_pass_cfg<3, 1, fold>(L, slices);
        case 3: return launch_pass_cfg<4, 1, fold>(L, slices);
        case 4: return launch_pass_cfg<5, 1, fold>(L, slices);
        default: return launch_pass_cfg<6, 1, fold>(L, slices);
      }
    };
    int rc = 0;
    // Few tiles leave the chip idle: 2048 x 256, 260 / 2000 rows, by 128 x 256 tiles 7.8 / 9.0 us, by 64 x 128 5.1 / 7.1; 5632 x 1024, 384 / 640 rows, 14.8 / 16.0, by 96 and 128 x 128 9.6 / 11.7,
    // 1024 rows (176 tiles) 17.3, by 128-wide ones 16.9.
    if ((M + 127) / 128 * ((ks.n_main + 255) / 256) <= 128) {
      if (ks.n_main > 0) rc = narrow(0, ks.n_main, 1, std::false_type{});
    } else {
      switch (least(PASSES, 0, 5, M, ks.n_main, K, &us)) {
        case 0: rc = launch_pass_cfg<4, 2, false>(L, 1); break;
        case 1: rc = launch_pass_cfg<5, 2, false>(L, 1); break;
        case 2: rc = launch_pass_cfg<6, 2, false>(L, 1); break;
        case 3: rc = launch_pass_cfg<7, 2, false>(L, 1); break;
        default: rc = ks.n_main < N ? launch_pass_cfg<8, 2, false>(L, 1) : launch_rounds(L, rounds_cut(M, N, 1, &us));
      }
    }
    // A remainder's columns, whose K a step adds up in slices, behind the main ones (7B shape, 640 / 1024 / 2000 rows, as leftovers of rounds of 256 x 256 tiles
    // 204 / 271 / 488 us, so 160 / 237 / 457).
    return rc || ks.n_main == N ? rc : narrow(ks.n_main, N, ks.rem_splits, std::true_type{});
  }
  switch (fold_shape(M, N, K, &us)) {
    case 0: return launch_fold_cfg<2, 2, 1, 1>(L);
    case 1: return launch_fold_cfg<1, 4, 2, 1>(L);
    case 2: return launch_fold_cfg<1, 4, 3, 1>(L);
    case 3: return launch_fold_cfg<1, 4, 4, 1>(L);
    case 4: return launch_fold_cfg<1, 4, 5, 1>(L);
    case 5: return launch_fold_cfg<1, 4, 6, 1>(L);
    default: return launch_fold_cfg<1, 4, 4, 2>(L);
  }
}

// How many slices a pass of M rows leaves a plain product in: 1 (launch_gemm_folded) or all ks.splits, as a step does.  A long K in one
// workgroup after the other leaves the chip to small tiles, at half the rate; by slices there are enough 256 x 256
// tiles (few: 128 x 256), for the price of the slices' way to memory (0.24 us per MB) and back (0.14).  Folded weights that are far (48 MB on) take an eighth
// more than fold_shape says.  Down products with the residual + RMSNorm behind them, random operands, us folded / in slices: 1.5B shape 511 rows 41 / 28, 1024 54 / 46,
// 1200 56 / 65, 2000 74 / 91, 3000 96 / 133; 7B 511 118 / 76, 900 130 / 139, 1024 165 / 145, 1200 163 / 199, 3000 446 / 463; 32B 511 208 / 145, 1024 320 / 296, 1200
// 344 / 372, 1500 373 / 455; 4096 x 14336, 8 slices, 511 94 / 69, 1200 136 / 173.  QKV and O: 7B, 511 rows, 38 / 33 and 25 / 31; 32B, 1024 rows, 77 / 112.
// Over 216 points (12 shapes, 300 to 1500 rows, random operands) the choice takes 0.5 % more than the better of the two on average.
int gemm_pass_slices(int M, int N, int K, const GemmSplit &ks) {
  if (ks.splits == 1 || K < 8192) return 1;
  const int ksteps = 4 * ((K / (4 * BK) + ks.splits - 1) / ks.splits);
  const int64_t tiles = (int64_t)((M + 255) / 256) * ((N + 255) / 256) * ks.splits;
  float fold;
  fold_shape(M, N, K, &fold);
  const int64_t halves = (int64_t)((M + 127) / 128) * ((N + 255) / 256) * ks.splits;
  const float step = tiles <= 128 ? 0.5f + 0.4f * std::min(halves * (1.f / 256), 1.f) : big_rounds(tiles);
  const float sliced = ksteps * step + 4e-6f * M * N * (0.24f * ks.splits + 0.14f * (ks.splits - 1));
  return sliced < fold * ((int64_t)N * K > 24 << 20 ? 1.125f : 1.f) ? ks.splits : 1;
}

// fp32 elements of a plain product of a pass of up to R rows.  Slices come and go with the row count (fold_shape steps at the rows of its
// tile shapes), so every row count is asked, from the most down to the first that keeps them.
int64_t gemm_pass_elems(int R, int N, int K, const GemmSplit &ks) {
  int r = R;
  while (r > 0 && gemm_pass_slices(r, N, K, ks) == 1) --r;
  return std::max((int64_t)R, (int64_t)r * ks.splits) * N;
}

// The product of a pass of more than 256 rows in gemm_pass_slices(...) slices.
// Those of a SwiGLU product's remainder are added up in the workgroup (7B shape, 257 / 384 / 511 rows, by slices behind 256 x 256 tiles 138 / 125 / 135 us, so 88 / 99 / 126).
int launch_gemm_pass(const bf16_t *x, const bf16_t *w, void *y, int64_t room, int M, int N, int K, int mode, const GemmSplit &ks,
                     hipStream_t s) {
  const int slices = mode == 0 ? gemm_pass_slices(M, N, K, ks) : 1;
  if (mode == 0 && (int64_t)slices * M * N > room) return -1;
  if (slices == 1) return launch_gemm_folded(x, w, y, M, N, K, mode, ks, s);
  if (M < 1 || M > GEMM_MAX_ROWS || K % (4 * BK) || N % 32 || !splits_valid(K, ks.splits) || ks.n_main != N) return -1;
  if ((int64_t)N * K * 2 >= GEMM_MAX_OPERAND_BYTES || (int64_t)M * K * 2 >= GEMM_MAX_OPERAND_BYTES) return -1;
  const Launch L{x, w, y, M, N, K, 0, ks.splits, 0, N, N, 0, true, false, s};
  float us;
  // few tiles: 128 x 256 ones (1.5B shape, 511 rows: 32 -> 23 us; 1024 rows 41 -> 44)
  return (M + 255) / 256 * ((N + 255) / 256) * ks.splits <= 128 ? launch_cfg<1, 4, 4, 2>(L) : launch_rounds(L, rounds_cut(M, N, ks.splits, &us));
}

}  // namespace pl
