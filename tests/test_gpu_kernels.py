"""Kernel-level parity (GPU): the HIP kernels, called through the C ABI, against the CPU oracle on the
same seeded inputs."""
import numpy as np
import pytest
import torch

import paper_2509_19128_amd as pl
import synth
from oracle import decoder, sampler

from gpu_util import close, dev_bf16, to_np

pytestmark = pytest.mark.gpu

# spec tolerance for bf16 results
ATOL, RTOL = 2e-2, 1e-2


def _paged_inputs(rng, ctx, Hq, Hkv, hd, page_tokens, check_rows):
    """Random page pool on the device; rows in `check_rows` get host-known K/V written into their pages."""
    n = len(ctx)
    pages_per_seq = (int(max(ctx)) + page_tokens - 1) // page_tokens
    need = [(int(c) + page_tokens - 1) // page_tokens for c in ctx]
    n_pages = sum(need) + 3
    perm = rng.permutation(n_pages).astype(np.int32)
    table = np.zeros((n, pages_per_seq), np.int32)
    k = 0
    for b in range(n):
        table[b, :need[b]] = perm[k:k + need[b]]
        k += need[b]
    page_elems = Hkv * 2 * page_tokens * hd
    g = torch.Generator(device="cuda").manual_seed(int(rng.integers(1 << 30)))
    pool = torch.randn(n_pages * page_elems, generator=g, device="cuda", dtype=torch.float32).to(torch.bfloat16)
    known = {}
    for b in check_rows:
        c = int(ctx[b])
        K = synth.bf16_round(rng.standard_normal((c, Hkv, hd)).astype(np.float32))
        V = synth.bf16_round(rng.standard_normal((c, Hkv, hd)).astype(np.float32))
        img = np.zeros(need[b] * page_elems, np.uint16)
        pl.pl_kv_pack_host(img, np.arange(need[b], dtype=np.int32), K, V, 0, Hkv, hd, page_tokens)
        dst = pool.view(torch.int16).view(n_pages, page_elems)
        dst[torch.from_numpy(table[b, :need[b]].astype(np.int64)).cuda()] = torch.from_numpy(
            img.view(np.int16).reshape(need[b], page_elems)).cuda()
        known[b] = (K, V)
    return pool, table, pages_per_seq, known


def _run_attention(q_np, pool, table, ctx, Hq, Hkv, hd, page_tokens, pages_per_seq, max_ctx):
    n = len(ctx)
    q = dev_bf16(q_np)
    out = torch.zeros(n, Hq, hd, device="cuda", dtype=torch.bfloat16)
    ws = torch.empty(max(pl.pl_attention_workspace_bytes(n, Hq, Hkv, hd, max_ctx), 16), device="cuda", dtype=torch.uint8)
    tb = torch.from_numpy(table).cuda()
    cl = torch.from_numpy(np.asarray(ctx, np.int32)).cuda()
    torch.cuda.synchronize()
    pl.pl_attention_decode(q.data_ptr(), pool.data_ptr(), tb.data_ptr(), cl.data_ptr(), out.data_ptr(), ws.data_ptr(),
                           n, Hq, Hkv, hd, page_tokens, pages_per_seq, max_ctx, 0)
    torch.cuda.synchronize()
    return to_np(out)


@pytest.mark.parametrize("Hq,Hkv,hd,page_tokens", [(28, 4, 128, 64), (8, 2, 32, 64), (12, 2, 128, 32),
                                                    (40, 8, 128, 128), (16, 1, 64, 64)])
def test_attention_matches_oracle_on_ragged_contexts(Hq, Hkv, hd, page_tokens):
    rng = np.random.default_rng(hd + Hq)
    ctx = np.array([1, 31, 32, 33, 64, 127, 129, 700, 1500, 0, 5], np.int32)   # a zero-length row is skipped
    pool, table, pps, known = _paged_inputs(rng, np.maximum(ctx, 1), Hq, Hkv, hd, page_tokens, range(len(ctx)))
    q = synth.bf16_round(rng.standard_normal((len(ctx), Hq, hd)).astype(np.float32))
    got = _run_attention(q, pool, table, ctx, Hq, Hkv, hd, page_tokens, pps, int(ctx.max()))
    for b, c in enumerate(ctx):
        if c == 0:
            assert np.all(got[b] == 0)
            continue
        K, V = known[b]
        ref = decoder.attend_one(q[b].astype(np.float64), K[:c].astype(np.float64), V[:c].astype(np.float64))
        ok, err = close(got[b], ref, ATOL, RTOL)
        assert ok, (b, c, err)


def test_attention_closed_forms_on_device():
    """q = 0 gives the mean of V; one cached token gives its value."""
    rng = np.random.default_rng(5)
    Hq, Hkv, hd, pt = 28, 4, 128, 64
    ctx = np.array([300, 1], np.int32)
    pool, table, pps, known = _paged_inputs(rng, ctx, Hq, Hkv, hd, pt, [0, 1])
    q = synth.bf16_round(rng.standard_normal((2, Hq, hd)).astype(np.float32))
    q[0] = 0
    got = _run_attention(q, pool, table, ctx, Hq, Hkv, hd, pt, pps, 300)
    for h in range(Hq):
        assert close(got[0, h], known[0][1][:, h // 7].mean(0), ATOL, RTOL)[0]
        assert close(got[1, h], known[1][1][0, h // 7], 1e-6, 4e-3)[0]


def test_attention_full_microbench_shape_on_sampled_rows():
    """The launch shape of the attention microbenchmark (batch 512, 28 q / 4 kv heads, head_dim 128,
    log-normal contexts clipped to [128, 16384]); 12 sampled rows, shortest and longest included, are
    checked against the oracle, the others only for being finite."""
    rng = np.random.default_rng(1236)
    Hq, Hkv, hd, pt = 28, 4, 128, 64
    ctx = synth.attention_microbench_lengths(1236).astype(np.int32)
    rows = sorted(set([int(ctx.argmin()), int(ctx.argmax())] + rng.choice(512, 10, replace=False).tolist()))
    pool, table, pps, known = _paged_inputs(rng, ctx, Hq, Hkv, hd, pt, rows)
    q = synth.bf16_round(rng.standard_normal((512, Hq, hd)).astype(np.float32))
    got = _run_attention(q, pool, table, ctx, Hq, Hkv, hd, pt, pps, 16384)
    assert np.isfinite(got).all()
    for b in rows:
        K, V = known[b]
        ref = decoder.attend_one(q[b].astype(np.float64), K.astype(np.float64), V.astype(np.float64))
        ok, err = close(got[b], ref, ATOL, RTOL)
        assert ok, (b, int(ctx[b]), err)


def test_attention_chunk_boundaries_in_the_benchmark_launch_shape():
    """Batch 256, 28 q / 4 kv heads, head_dim 128, 128-token pages, contexts up to 512 + 16384: the launch
    shape of the 7B benchmark, where one workgroup handles up to 8192 tokens.  Contexts on both sides of
    one and two full chunks, and the maximum, against the oracle; the merge of two and three chunks is on
    the path of the last five."""
    rng = np.random.default_rng(99)
    Hq, Hkv, hd, pt = 28, 4, 128, 128
    edges = [8191, 8192, 8193, 16383, 16384, 16385, 16896, 1, 128, 129]
    ctx = np.concatenate([edges, rng.integers(200, 3000, 256 - len(edges))]).astype(np.int32)
    rows = list(range(len(edges)))
    pool, table, pps, known = _paged_inputs(rng, ctx, Hq, Hkv, hd, pt, rows)
    q = synth.bf16_round(rng.standard_normal((256, Hq, hd)).astype(np.float32))
    got = _run_attention(q, pool, table, ctx, Hq, Hkv, hd, pt, pps, 16896)
    assert np.isfinite(got).all()
    for b in rows:
        K, V = known[b]
        ref = decoder.attend_one(q[b].astype(np.float64), K.astype(np.float64), V.astype(np.float64))
        ok, err = close(got[b], ref, ATOL, RTOL)
        assert ok, (b, int(ctx[b]), err)


def test_attention_of_a_sequence_does_not_depend_on_its_neighbours():
    """The chunk length is a function of the launch shape only, and the merge order is fixed: the same
    sequence gives bit-identical output whatever the other rows' contexts are and wherever it sits in
    the work list (which is sorted by length)."""
    rng = np.random.default_rng(321)
    Hq, Hkv, hd, pt, n = 28, 4, 128, 128, 64
    ctx_a = rng.integers(100, 12000, n).astype(np.int32)
    ctx_b = rng.integers(100, 12000, n).astype(np.int32)
    keep = [3, 17, 40]
    ctx_a[keep] = ctx_b[keep] = [9000, 700, 16896]
    both = np.maximum(ctx_a, ctx_b)
    pool, table, pps, _ = _paged_inputs(rng, both, Hq, Hkv, hd, pt, [])
    q = synth.bf16_round(rng.standard_normal((n, Hq, hd)).astype(np.float32))
    out_a = _run_attention(q, pool, table, ctx_a, Hq, Hkv, hd, pt, pps, 16896)
    out_b = _run_attention(q, pool, table, ctx_b, Hq, Hkv, hd, pt, pps, 16896)
    for b in keep:
        assert np.array_equal(out_a[b], out_b[b]), b
    assert not np.array_equal(out_a[0], out_b[0])        # the other rows did change


@pytest.mark.parametrize("n,Hq,Hkv,hd,page,max_ctx", [
    (5, 28, 4, 128, 128, 900),       # no list, chunks merged by a launch of their own
    (300, 40, 8, 128, 32, 300),      # no list, one chunk per row
    (212, 28, 4, 128, 64, 480),      # list, chunks of 128 merged by the last workgroup
    (3, 28, 4, 128, 64, 24000)])     # list, more chunks than one workgroup merges
def test_attention_on_every_route_of_a_launch(n, Hq, Hkv, hd, page, max_ctx):
    """With and without a work list, chunks merged by the last workgroup of a row or by the merge launch: sampled rows
    (the longest, one chunk and a little, an empty one) against the oracle, twice over the same workspace (what
    one call leaves there must not disturb the next)."""
    rng = np.random.default_rng(n + max_ctx)
    ctx = rng.integers(1, max_ctx + 1, n).astype(np.int32)
    ctx[0], ctx[1], ctx[2] = max_ctx, 129, 0
    rows = [0, 1] + ([n - 1] if n > 3 else [])
    pool, table, pps, known = _paged_inputs(rng, np.maximum(ctx, 1), Hq, Hkv, hd, page, rows)
    qs = [synth.bf16_round(rng.standard_normal((n, Hq, hd)).astype(np.float32)) for _ in range(2)]
    ws = torch.full((pl.pl_attention_workspace_bytes(n, Hq, Hkv, hd, max_ctx) + 64,), 0xA5, device="cuda", dtype=torch.uint8)
    tb, cl = torch.from_numpy(table).cuda(), torch.from_numpy(ctx).cuda()
    for q in qs:
        qd, out = dev_bf16(q), torch.zeros(n, Hq, hd, device="cuda", dtype=torch.bfloat16)
        pl.pl_attention_decode(qd.data_ptr(), pool.data_ptr(), tb.data_ptr(), cl.data_ptr(), out.data_ptr(), ws.data_ptr() + 16,
                               n, Hq, Hkv, hd, page, pps, max_ctx, 0)
        torch.cuda.synchronize()
        got = to_np(out)
        assert np.isfinite(got).all() and np.all(got[2] == 0)
        for b in rows:
            K, V = known[b]
            ref = decoder.attend_one(q[b].astype(np.float64), K.astype(np.float64), V.astype(np.float64))
            ok, err = close(got[b], ref, ATOL, RTOL)
            assert ok, (b, int(ctx[b]), err)


@pytest.mark.parametrize("n,Hq,Hkv,hd,page,max_ctx", [
    (300, 40, 8, 128, 32, 300),      # one chunk per row
    (5, 28, 4, 128, 128, 900),       # chunks merged by a launch of their own
    (212, 28, 4, 128, 64, 480),      # chunks merged by the last workgroup
    (3, 28, 4, 64, 64, 24000), (17, 8, 2, 32, 32, 2000)])
def test_attention_divides_by_the_sum_of_the_weights(n, Hq, Hkv, hd, page, max_ctx):
    """q = 0 makes every weight 1, so sums over an even number of tokens whose values alternate are exact and their means lie half-way between two bf16
    values (1 + 2^-8 and 1 + 3 2^-8): rounded once, to even, whatever the number of tokens; and what is
    infinite or not a number stays so."""
    pages = -(-max_ctx // page)
    V = np.empty((pages * page, Hkv, hd), np.float32)
    V[0::2, :, 0::2], V[1::2, :, 0::2] = 1, 1 + 2.0 ** -7
    V[0::2, :, 1::2], V[1::2, :, 1::2] = 1 + 2.0 ** -7, 1 + 2.0 ** -6
    V[0, :, 0], V[1, :, 1], V[0, :, 2], V[1, :, 2], V[0, :, 3] = np.inf, -np.inf, np.inf, -np.inf, np.nan
    img = np.zeros(pages * Hkv * 2 * page * hd, np.uint16)
    pl.pl_kv_pack_host(img, np.arange(pages, dtype=np.int32), np.zeros_like(V), V, 0, Hkv, hd, page)
    pool = torch.from_numpy(img.view(np.int16)).cuda()
    table = np.broadcast_to(np.arange(pages, dtype=np.int32), (n, pages)).copy()
    for seed in range(5):
        ctx = (2 * np.random.default_rng(seed).integers(1, max_ctx // 2 + 1, n)).astype(np.int32)
        ctx[0] = max_ctx - 2 * seed
        got = _run_attention(np.zeros((n, Hq, hd), np.float32), pool, table, ctx, Hq, Hkv, hd, page, pages, max_ctx)
        assert (got[:, :, 4::2] == 1).all() and (got[:, :, 5::2] == 1 + 2.0 ** -6).all(), seed
        assert (got[:, :, 0] == np.inf).all() and (got[:, :, 1] == -np.inf).all() and np.isnan(got[:, :, 2:4]).all(), seed


def test_attention_rejects_bad_arguments():
    t = torch.zeros(1 << 16, device="cuda", dtype=torch.bfloat16)
    p = t.data_ptr()
    good = dict(n=2, Hq=8, Hkv=2, hd=32, pt=32, pps=4, mx=128)
    for bad in [dict(Hq=7), dict(hd=48), dict(pt=48), dict(pt=16), dict(mx=129), dict(mx=0), dict(n=0), dict(n=2000), dict(Hq=40, Hkv=2)]:
        a = dict(good, **bad)
        with pytest.raises(pl.PlError) as ex:
            pl.pl_attention_decode(p, p, p, p, p, p, a["n"], a["Hq"], a["Hkv"], a["hd"], a["pt"], a["pps"], a["mx"], 0)
        assert ex.value.code == pl.PL_E_INVAL, bad
    with pytest.raises(pl.PlError):
        pl.pl_attention_decode(0, p, p, p, p, p, 2, 8, 2, 32, 32, 4, 128, 0)
    assert pl.pl_attention_workspace_bytes(0, 8, 2, 32, 128) == 0


GEMM_SHAPES = [(4, 384, 256, 1), (4, 4096, 1024, 4), (3, 256, 1024, 2), (33, 320, 256, 1), (64, 2048, 1536, 3),
               (130, 1536, 8960, 7), (256, 4608, 3584, 7), (200, 3584, 18944, 8), (256, 3584, 18944, 9), (256, 2560, 3584, 1),
               (300, 640, 512, 2), (256, 33792, 256, 1), (130, 34000 // 32 * 32, 256, 1),
               (256, 43552, 256, 1), (129, 32768, 512, 1), (200, 3584, 3584, 4), (256, 2048, 1536, 3)]   # the last four take the paired 128 x 256 tiles


@pytest.mark.parametrize("M,N,K,splits", GEMM_SHAPES)
def test_gemm_partials_sum_to_the_product(M, N, K, splits):
    rng = np.random.default_rng(M * 7 + N)
    x = synth.bf16_round(rng.standard_normal((M, K)).astype(np.float32))
    w = synth.bf16_round((rng.standard_normal((N, K)) * 0.05).astype(np.float32))
    xd, wd = dev_bf16(x), dev_bf16(pl.operand_order(w))
    y = torch.full((splits, M, N), float("nan"), device="cuda", dtype=torch.float32)
    pl.pl_gemm_bf16(xd.data_ptr(), wd.data_ptr(), y.data_ptr(), M, N, K, 0, splits, 0)
    torch.cuda.synchronize()
    got = to_np(y).astype(np.float64).sum(0)
    ref = x.astype(np.float64) @ w.astype(np.float64).T
    ok, err = close(got, ref, 1e-4 * np.sqrt(K) * 0.05, 1e-4)      # fp32 accumulation of exact bf16 products
    assert ok, err


@pytest.mark.parametrize("M,F,K", [(4, 1024, 256), (64, 2240, 1536), (256, 1280, 3584), (129, 320, 512), (200, 16640, 256),
                                   (200, 18944, 256)])
def test_gemm_swiglu_epilogue(M, F, K):
    rng = np.random.default_rng(F + M)
    x = synth.bf16_round(rng.standard_normal((M, K)).astype(np.float32))
    wg = synth.bf16_round((rng.standard_normal((F, K)) * 0.05).astype(np.float32))
    wu = synth.bf16_round((rng.standard_normal((F, K)) * 0.05).astype(np.float32))
    inter = np.stack([wg.reshape(F // 32, 32, K), wu.reshape(F // 32, 32, K)], axis=1).reshape(2 * F, K)
    y = torch.full((M, F), float("nan"), device="cuda", dtype=torch.bfloat16)
    xd, wd = dev_bf16(x), dev_bf16(pl.operand_order(inter))          # keep the device tensors alive across the launch
    pl.pl_gemm_bf16(xd.data_ptr(), wd.data_ptr(), y.data_ptr(), M, 2 * F, K, 1, 1, 0)
    torch.cuda.synchronize()
    x64 = x.astype(np.float64)
    ref = decoder.silu(x64 @ wg.astype(np.float64).T) * (x64 @ wu.astype(np.float64).T)
    ok, err = close(to_np(y), ref, 2e-3, RTOL)
    assert ok, err


@pytest.mark.parametrize("F,K", [(352, 512), (96, 1024), (8960, 256)])
def test_swiglu_of_every_row_count_gives_the_same_rows(F, K):
    """Row counts on both sides of every tile height, a last tile of one gate/up pair and of two: shapes whose wavefronts hold both
    halves of a pair and shapes whose neighbours swap them, against fp64 and bit for bit against one another."""
    g = torch.Generator(device="cuda").manual_seed(F)
    x = torch.empty(512, K, device="cuda", dtype=torch.bfloat16).normal_(generator=g)
    w = synth.bf16_round(np.random.default_rng(F).standard_normal((2 * F, K), dtype=np.float32) * 0.05)
    wd = dev_bf16(pl.operand_order(w))
    p = to_np(x).astype(np.float64) @ w.astype(np.float64).T
    gate, up = (p.reshape(512, F // 32, 2, 32)[:, :, i].reshape(512, F) for i in (0, 1))
    want, widest = decoder.silu(gate) * up, None
    for M in (512, 511, 385, 257, 256, 160, 129, 128, 97, 65, 64, 33, 32, 9, 1):
        y = torch.full((M + 1, F), float("nan"), device="cuda", dtype=torch.bfloat16)
        pl.pl_gemm_bf16(x.data_ptr(), wd.data_ptr(), y.data_ptr(), M, 2 * F, K, 1, 1, 0)
        torch.cuda.synchronize()
        if widest is None:
            widest = y.clone()
            ok, err = close(to_np(y[:M]), want, 2e-3, RTOL)
            assert ok, err
        assert torch.equal(y[:M], widest[:M]) and bool(y[M].isnan().all()), M


@pytest.mark.parametrize("splits", [1, 2])
def test_swiglu_of_a_saturated_gate_is_the_quotient(splits):
    """Gates down to where 1 + e^-g is near the largest float (its reciprocal is subnormal), up values that bring the results back among
    ordinary numbers: within a rounding to bf16 (2^-8) and the exponential's error (2^-24 of an exponent of up to 128, 2^-17) of the definition, by the
    epilogue and by the reduction over K slices."""
    F, K = 320, 512
    coarse, fine = np.linspace(0, -87, F // 32)[:, None].round(), -np.arange(32, dtype=np.float32)[None] / 20
    w = np.zeros((F // 32, 2, 32, K), np.float32)
    w[:, 0, :, 0], w[:, 0, :, K // 2] = coarse, synth.bf16_round(np.broadcast_to(fine, (F // 32, 32)).astype(np.float32))
    up = 2.0 ** np.clip(np.round(-coarse / np.log(2)) - 1, 0, 125)
    w[:, 1, :, 0] = up
    gate = (w[:, 0, :, 0].astype(np.float64) + w[:, 0, :, K // 2]).reshape(F)
    x = np.zeros((1, K), np.float32)
    x[0, 0] = x[0, K // 2] = 1
    xd, wd = dev_bf16(x), dev_bf16(pl.operand_order(w.reshape(2 * F, K)))
    y, ws = torch.full((1, F), float("nan"), device="cuda", dtype=torch.bfloat16), torch.empty(splits * 2 * F, device="cuda")
    pl.pl_debug_gemm_cfg(8, xd.data_ptr(), wd.data_ptr(), y.data_ptr(), ws.data_ptr(), 1, 2 * F, K, 1, splits, 0, 2 * F, False, 0)
    torch.cuda.synchronize()
    assert gate.min() < -88.5
    want = gate / (1 + np.exp(-gate)) * np.broadcast_to(up, (F // 32, 32)).reshape(F)
    assert (np.abs(to_np(y)[0] - want) <= (2.0 ** -8 + 2.0 ** -16) * np.abs(want)).all()


CFG_TILES = {0: (32, 256), 1: (64, 256), 2: (128, 256), 3: (64, 128), 4: (128, 128), 5: (256, 128), 6: (64, 64),
             7: (128, 64), 8: (32, 128), 9: (128, 64), 10: (256, 64), 11: (64, 128), 12: (128, 128), 13: (256, 128), 14: (256, 256)}


@pytest.mark.parametrize("cfg", sorted(CFG_TILES))
def test_every_gemm_tile_configuration_against_fp64(cfg):
    """Each tile configuration of the kernel on shapes with several row tiles, a ragged last row tile,
    a column range that starts and ends inside the matrix, with and without a K split; the SwiGLU
    product also with its K split (partials + reduction)."""
    rows, cols = CFG_TILES[cfg]
    rng = np.random.default_rng(100 + cfg)
    M, N, K = min(2 * rows + 7, 300), 5 * 128, 768
    x = synth.bf16_round(rng.standard_normal((M, K), dtype=np.float32))
    w = synth.bf16_round(rng.standard_normal((N, K), dtype=np.float32) * 0.05)
    xd, wd = dev_bf16(x), dev_bf16(pl.operand_order(w))
    ref = x.astype(np.float64) @ w.astype(np.float64).T
    for splits, nb, ne, paired in [(1, 0, N, False), (3, 128, N - 64, False), (1, 64, N, True), (3, 64, N - 32, True)]:
        y = torch.full((splits, M, N), float("nan"), device="cuda", dtype=torch.float32)
        pl.pl_debug_gemm_cfg(cfg, xd.data_ptr(), wd.data_ptr(), y.data_ptr(), 0, M, N, K, 0, splits, nb, ne, paired, 0)
        torch.cuda.synchronize()
        got = to_np(y)
        assert np.isnan(got[:, :, :nb]).all() and np.isnan(got[:, :, ne:]).all()       # nothing outside the range
        tol = 1e-4 * (np.sqrt(K) * 0.05 + np.abs(ref[:, nb:ne]))
        assert (np.abs(got[:, :, nb:ne].astype(np.float64).sum(0) - ref[:, nb:ne]) <= tol).all(), (splits, nb, ne)
    if cfg in (6, 7):                                 # wavefronts of one column tile in two rows: no gate/up pair
        with pytest.raises(pl.PlError):
            pl.pl_debug_gemm_cfg(cfg, xd.data_ptr(), wd.data_ptr(), xd.data_ptr(), 0, M, N, K, 1, 1, 0, N, False, 0)
        return
    F = N // 2
    gate = ref.reshape(M, N // 64, 2, 32)[:, :, 0].reshape(M, F)
    up = ref.reshape(M, N // 64, 2, 32)[:, :, 1].reshape(M, F)
    want = gate / (1.0 + np.exp(-gate)) * up
    with pytest.raises(pl.PlError):
        pl.pl_debug_gemm_cfg(cfg, xd.data_ptr(), wd.data_ptr(), xd.data_ptr(), wd.data_ptr(), M, N, K, 1, 2, 0, N, True, 0)
    for splits, nb, ne in [(1, 0, N), (3, 0, N), (2, 128, N - 64), (1, 64, N - 64)]:
        mid = torch.full((M, F), float("nan"), device="cuda", dtype=torch.bfloat16)
        ws = torch.empty(splits * M * (ne - nb), device="cuda", dtype=torch.float32)
        pl.pl_debug_gemm_cfg(cfg, xd.data_ptr(), wd.data_ptr(), mid.data_ptr(), ws.data_ptr(), M, N, K, 1, splits, nb, ne, False, 0)
        torch.cuda.synchronize()
        got = to_np(mid)
        assert np.isnan(got[:, :nb // 2]).all() and np.isnan(got[:, ne // 2:]).all()
        ok, err = close(got[:, nb // 2:ne // 2], want[:, nb // 2:ne // 2], 2e-3, RTOL)
        assert ok, (splits, nb, ne, err)


@pytest.mark.parametrize("F,K", [(18944, 3584), (18976, 768)])
def test_swiglu_product_of_a_256_row_engine_is_the_same_for_every_row_count(F, K):
    """An engine of 256 slots at a wide SwiGLU product: passes of 129..256 rows take the launch that gives every
    compute unit a main tile and a K slice of the leftover columns, narrower passes separate launches with
    the same slices.  Every row count against fp64, and the rows of a narrower pass bit-equal to the same
    rows of the widest one.  The second shape ends in a ragged column tile."""
    N, M_max = 2 * F, 256
    splits, n_main, rem_splits, ws_elems = pl.pl_debug_gemm_plan(M_max, N, K, 1)
    assert splits == 1 and 0 < n_main < N and rem_splits > 1 and ws_elems == rem_splits * M_max * (N - n_main)
    rng = np.random.default_rng(F + K)
    x = synth.bf16_round(rng.standard_normal((M_max, K), dtype=np.float32))
    w = synth.bf16_round(rng.standard_normal((N, K), dtype=np.float32) * 0.05)
    xd, wd = dev_bf16(x), dev_bf16(pl.operand_order(w))
    ref = x.astype(np.float64) @ w.astype(np.float64).T
    gate = ref.reshape(M_max, N // 64, 2, 32)[:, :, 0].reshape(M_max, F)
    up = ref.reshape(M_max, N // 64, 2, 32)[:, :, 1].reshape(M_max, F)
    want = gate / (1.0 + np.exp(-gate)) * up
    ws = torch.empty(ws_elems, device="cuda", dtype=torch.float32)
    widest = None
    for M in (256, 255, 200, 129, 128, 65, 64, 20, 1):
        mid = torch.full((M, F), float("nan"), device="cuda", dtype=torch.bfloat16)
        ws.fill_(float("nan"))
        pl.pl_debug_gemm_planned(xd.data_ptr(), wd.data_ptr(), mid.data_ptr(), ws.data_ptr(), M_max, M, N, K, 1, 0)
        torch.cuda.synchronize()
        got = to_np(mid)
        ok, err = close(got, want[:M], 2e-3, RTOL)
        assert ok, (M, err)
        if widest is None:
            widest = got
        else:
            assert np.array_equal(got, widest[:M]), M
    with pytest.raises(pl.PlError):
        pl.pl_debug_gemm_planned(xd.data_ptr(), wd.data_ptr(), mid.data_ptr(), 0, M_max, 200, N, K, 1, 0)


@pytest.mark.parametrize("M_max,N,K", [(256, 4608, 3584), (256, 3584, 18944), (64, 2048, 1536), (128, 7168, 5120)])
def test_plain_products_of_an_engine_are_the_same_for_every_row_count(M_max, N, K):
    """QKV- and down-shaped products as an engine of M_max slots launches them: the tile shape follows the rows
    of the call, the K split is fixed, so every slice of the partial sums of a narrow pass is bit-equal to the
    same rows of the widest pass; their sum is the product."""
    splits, n_main, rem_splits, ws_elems = pl.pl_debug_gemm_plan(M_max, N, K, 0)
    assert n_main == N and ws_elems == 0
    rng = np.random.default_rng(N + K)
    x = synth.bf16_round(rng.standard_normal((M_max, K), dtype=np.float32))
    w = synth.bf16_round(rng.standard_normal((N, K), dtype=np.float32) * 0.05)
    xd, wd = dev_bf16(x), dev_bf16(pl.operand_order(w))
    ref = x.astype(np.float64) @ w.astype(np.float64).T
    widest = None
    for M in sorted({M_max, M_max - 1, 200, 129, 128, 65, 64, 33, 32, 5, 1}, reverse=True):
        if M > M_max:
            continue
        y = torch.full((splits, M, N), float("nan"), device="cuda", dtype=torch.float32)
        pl.pl_debug_gemm_planned(xd.data_ptr(), wd.data_ptr(), y.data_ptr(), 0, M_max, M, N, K, 0, 0)
        torch.cuda.synchronize()
        got = to_np(y)
        if widest is None:
            widest = got
            ok, err = close(got.astype(np.float64).sum(0), ref, 1e-4 * np.sqrt(K) * 0.05, 1e-4)
            assert ok, err
        else:
            assert np.array_equal(got, widest[:, :M]), M


@pytest.mark.parametrize("M_max,N,K,mode", [(64, 2048, 1536, 0), (64, 1536, 8960, 0), (256, 4608, 3584, 0), (128, 7168, 5120, 0),
                                            (2, 96, 256, 0), (64, 2 * 8960, 256, 1), (256, 2 * 18944, 768, 1), (256, 2 * 18976, 768, 1),
                                            (256, 2 * 18944, 3584, 1)])   # (256 x 256 tiles of the main columns at 511, 1024, 2000 and 4096 rows)
def test_products_of_many_rows_equal_the_slices_of_few_added_in_order(M_max, N, K, mode):
    """The products of a prompt pass of more than 256 rows add up the K slices in the workgroup: bit-equal to the
    slices a narrow pass of the same engine gives its consumer, added in slice order, at the row counts where a tile or
    the choice of a tile shape ends.  (Row counts and shapes between them reach every tile shape of the choice.)"""
    splits, n_main, _, ws_elems = pl.pl_debug_gemm_plan(M_max, N, K, mode)
    g = torch.Generator(device="cuda").manual_seed(N + K)
    rows_most = 4096
    x = torch.empty(rows_most, K, device="cuda", dtype=torch.bfloat16).normal_(generator=g)
    w = torch.empty(N * K, device="cuda", dtype=torch.bfloat16).normal_(0, 0.05, generator=g)
    want = torch.empty(rows_most, N if mode == 0 else N // 2, device="cuda", dtype=torch.float32)
    ws = torch.empty(max(ws_elems, 1), device="cuda", dtype=torch.float32)
    for r in range(0, rows_most, M_max):
        rows = min(M_max, rows_most - r)
        y = torch.empty(splits, rows, N, device="cuda") if mode == 0 else torch.empty(rows, N // 2, device="cuda", dtype=torch.bfloat16)
        pl.pl_debug_gemm_planned(x[r:].data_ptr(), w.data_ptr(), y.data_ptr(), ws.data_ptr(), M_max, rows, N, K, mode, 0)
        if mode == 0:
            for s in range(1, splits):
                y[0] += y[s]
            want[r:r + rows] = y[0]
        else:
            want[r:r + rows] = y.float()
        torch.cuda.synchronize()
    for M in (257, 300, 384, 511, 512, 513, 1023, 1024, 1025, 1537, 2000, 3001, 4095, 4096):
        y = torch.full((M + 1, want.shape[1]), float("nan"), device="cuda", dtype=torch.float32 if mode == 0 else torch.bfloat16)
        pl.pl_debug_gemm_folded(x.data_ptr(), w.data_ptr(), y.data_ptr(), M_max, M, N, K, mode, 0)
        torch.cuda.synchronize()
        assert torch.equal(y[:M].float(), want[:M]), M
        assert bool(y[M].isnan().all()), M             # nothing written beyond the rows
    for bad in [(rows_most + 1, N, K), (0, N, K), (300, N, K + 64), (300, N + 16, K)]:
        with pytest.raises(pl.PlError):
            pl.pl_debug_gemm_folded(x.data_ptr(), w.data_ptr(), y.data_ptr(), M_max, *bad, mode, 0)


@pytest.mark.parametrize("N,K", [(17920, 1536), (4160, 2048), (5632, 512)])
def test_swiglu_products_of_passes_give_the_rows_of_steps(N, K):
    """Every tile shape of a pass's SwiGLU product (few tiles: 128 wide; 128 to 256 x 256), full and ragged: the rows that calls of 64 give, to the last bit."""
    g = torch.Generator(device="cuda").manual_seed(N)
    x = torch.empty(4096, K, device="cuda", dtype=torch.bfloat16).normal_(generator=g)
    w = torch.empty(N * K, device="cuda", dtype=torch.bfloat16).normal_(0, 0.05, generator=g)
    want, ws = torch.empty(4096, N // 2, device="cuda", dtype=torch.bfloat16), torch.empty(1, device="cuda")
    for r in range(0, 4096, 64):
        pl.pl_debug_gemm_planned(x[r:].data_ptr(), w.data_ptr(), want[r:].data_ptr(), ws.data_ptr(), 64, 64, N, K, 1, 0)
    torch.cuda.synchronize()
    for M in (1, 257, 384, 511, 640, 673, 900, 1025, 1281, 1537, 2017, 3001, 4096):
        y = torch.full((M + 1, N // 2), float("nan"), device="cuda", dtype=torch.bfloat16)
        pl.pl_debug_gemm_folded(x.data_ptr(), w.data_ptr(), y.data_ptr(), 64, M, N, K, 1, 0)
        torch.cuda.synchronize()
        assert torch.equal(y[:M], want[:M]), M
        assert bool(y[M].isnan().all()), M


def test_rows_of_a_wide_product_do_not_depend_on_the_row_count():
    """A product of more 256-wide column tiles than compute units at the row counts where its tiles change: close to fp64, and the same rows
    whatever their number."""
    N, K = 257 * 256 + 32, 256
    g = torch.Generator(device="cuda").manual_seed(3)
    x = torch.empty(160, K, device="cuda", dtype=torch.bfloat16).normal_(generator=g)
    w = torch.empty(N, K, device="cuda", dtype=torch.bfloat16).normal_(0, 0.05, generator=g)
    packed = w.view(N // 32, 32, K // 64, 2, 4, 8).permute(2, 0, 4, 3, 1, 5).contiguous()   # [k-step][row block][j][half][row][8]
    ref = x.double() @ w.double().T
    widest = None
    for M in (160, 129, 128, 127, 96, 65, 64):
        y = torch.full((M + 1, N), float("nan"), device="cuda")
        pl.pl_gemm_bf16(x.data_ptr(), packed.data_ptr(), y.data_ptr(), M, N, K, 0, 1, 0)
        torch.cuda.synchronize()
        assert bool(y[M].isnan().all()), M
        if widest is None:
            widest = y[:M].clone()
            assert float((widest.double() - ref).abs().max()) <= K * 2.0 ** -24 * float((x.double().abs() @ w.double().abs().T).max())   # fp32 sums of K products
        assert torch.equal(y[:M], widest[:M]), M


@pytest.mark.parametrize("N,K", [(32, 512), (96, 1536), (352, 768), (1312, 1536), (2080, 256)])
def test_every_tile_of_a_folded_product_is_dealt_to_one_workgroup(N, K):
    """Fewer tiles than XCDs, counts that eight does not divide, and both orders of the deal (by rows where 5 M >= 4 N): every element once,
    bit-equal to the slices of a narrow pass added in order."""
    splits = pl.pl_debug_gemm_plan(64, N, K, 0)[0]
    g = torch.Generator(device="cuda").manual_seed(N + K)
    x = torch.empty(2050, K, device="cuda", dtype=torch.bfloat16).normal_(generator=g)
    w = torch.empty(N * K, device="cuda", dtype=torch.bfloat16).normal_(0, 0.05, generator=g)
    want = torch.empty(2050, N, device="cuda")
    ws = torch.empty(1, device="cuda")
    for r in range(0, 2050, 64):
        rows = min(64, 2050 - r)
        y = torch.empty(splits, rows, N, device="cuda")
        pl.pl_debug_gemm_planned(x[r:].data_ptr(), w.data_ptr(), y.data_ptr(), ws.data_ptr(), 64, rows, N, K, 0, 0)
        for s in range(1, splits):
            y[0] += y[s]
        want[r:r + rows] = y[0]
        torch.cuda.synchronize()
    for M in (1, 31, 65, 259, 4 * N // 5, 4 * N // 5 + 1, 2050):
        y = torch.full((M + 1, N), float("nan"), device="cuda")
        pl.pl_debug_gemm_folded(x.data_ptr(), w.data_ptr(), y.data_ptr(), 64, M, N, K, 0, 0)
        torch.cuda.synchronize()
        assert torch.equal(y[:M], want[:M]), M
        assert bool(y[M].isnan().all()), M


@pytest.mark.parametrize("cfg", sorted(CFG_TILES))
def test_every_gemm_tile_configuration_for_cold_weights_gives_the_same_bits(cfg):
    """Weights that do not stay in the cache between two steps are loaded with another cache policy, by kernels of their
    own: equal bit for bit to the others, which the test above holds to float64, in both modes, with and without a K split."""
    rows, _ = CFG_TILES[cfg]
    M, N, K = min(2 * rows + 7, 300), 5 * 128, 768
    g = torch.Generator(device="cuda").manual_seed(cfg)
    x = torch.empty(M, K, device="cuda", dtype=torch.bfloat16).normal_(generator=g)
    w = torch.empty(N * K, device="cuda", dtype=torch.bfloat16).normal_(0, 0.05, generator=g)
    ws = torch.empty(3 * M * N, device="cuda", dtype=torch.float32)
    for mode, splits, nb, ne, paired in [(0, 1, 0, N, False), (0, 3, 128, N - 64, False), (0, 1, 64, N, True), (0, 3, 64, N - 32, True), (1, 1, 0, N, False),
                                         (1, 3, 0, N, False), (1, 2, 128, N - 64, False)]:
        if mode == 1 and cfg in (6, 7):
            continue
        got = []
        for cold in (0, pl.PL_GEMM_COLD):
            y = torch.zeros(splits, M, N, device="cuda") if mode == 0 else torch.zeros(M, N // 2, device="cuda", dtype=torch.bfloat16)
            pl.pl_debug_gemm_cfg(cfg, x.data_ptr(), w.data_ptr(), y.data_ptr(), ws.data_ptr(), M, N, K, mode | cold, splits, nb, ne, paired, 0)
            torch.cuda.synchronize()
            got.append(y)
        assert bool(got[0].abs().sum() > 0) and torch.equal(got[0], got[1]), (mode, splits, nb, ne, paired)


@pytest.mark.parametrize("M_max,N,K,mode", [(64, 2048, 1536, 0), (256, 4608, 3584, 0), (256, 3584, 18944, 0), (128, 7168, 5120, 0), (256, 32800, 256, 0),
                                            (64, 2 * 8960, 256, 1), (128, 2 * 27648, 256, 1), (256, 2 * 18944, 768, 1), (256, 2 * 18976, 768, 1)])
def test_products_of_an_engine_with_cold_weights_give_the_same_bits(M_max, N, K, mode):
    """The same for the launches of a step (at every row count that chooses another kernel); and a pass of many rows, which loads cold weights like
    others, gives the planned slices added in order."""
    splits, _, _, ws_elems = pl.pl_debug_gemm_plan(M_max, N, K, mode)
    g = torch.Generator(device="cuda").manual_seed(N + K)
    x = torch.empty(1024, K, device="cuda", dtype=torch.bfloat16).normal_(generator=g)
    w = torch.empty(N * K, device="cuda", dtype=torch.bfloat16).normal_(0, 0.05, generator=g)
    ws = torch.empty(max(ws_elems, 1), device="cuda", dtype=torch.float32)

    def both(M, slices, launch):
        got = []
        for cold in (0, pl.PL_GEMM_COLD):
            y = torch.full((slices, M, N), float("nan"), device="cuda") if mode == 0 else torch.full((M, N // 2), float("nan"), device="cuda", dtype=torch.bfloat16)
            ws.fill_(float("nan"))
            launch(y, M, mode | cold)
            torch.cuda.synchronize()
            got.append(y)
        assert bool(got[0].isfinite().all()) and torch.equal(got[0], got[1]), M
    for M in (1, 20, 33, 64, 65, 128, 129, 200, 256):
        if M <= M_max:
            both(M, splits, lambda y, M, md: pl.pl_debug_gemm_planned(x.data_ptr(), w.data_ptr(), y.data_ptr(), ws.data_ptr(), M_max, M, N, K, md, 0))
    want = torch.empty(1024, N, device="cuda") if mode == 0 else torch.empty(1024, N // 2, device="cuda", dtype=torch.bfloat16)
    for r in range(0, 1024, M_max):
        y = torch.empty(splits, M_max, N, device="cuda") if mode == 0 else want[r:]
        pl.pl_debug_gemm_planned(x[r:].data_ptr(), w.data_ptr(), y.data_ptr(), ws.data_ptr(), M_max, M_max, N, K, mode | pl.PL_GEMM_COLD, 0)
        if mode == 0:
            want[r:r + M_max] = 0
            for s in range(splits):
                want[r:r + M_max] += y[s]
        torch.cuda.synchronize()
    for M in (300, 511, 1024):
        y = torch.full_like(want[:M], float("nan"))
        pl.pl_debug_gemm_folded(x.data_ptr(), w.data_ptr(), y.data_ptr(), M_max, M, N, K, mode | pl.PL_GEMM_COLD, 0)
        torch.cuda.synchronize()
        assert torch.equal(y, want[:M]), M


@pytest.mark.parametrize("M,N,K,mode,splits", [(130, 66048, 256, 0, 1), (200, 78112, 512, 0, 1), (256, 65600, 768, 1, 1), (256, 131136, 256, 1, 1),
                                              (300, 33792, 256, 0, 1), (512, 36896, 1280, 0, 2), (511, 33856, 512, 1, 1), (129, 152064, 256, 0, 1)])
def test_products_of_more_tiles_than_compute_units(M, N, K, mode, splits):
    """A workgroup takes 256 x 256 tiles one after the other, whatever is left behind full rounds by narrower ones: with and without
    leftover columns, short last column tiles and rows, K of four k-steps (the ring never runs within a tile) and slices.  Against the
    float64 product (sums of K products of N(0, 1) and N(0, 0.05): the bound of the tests above), and nothing written beyond the rows."""
    g = torch.Generator(device="cuda").manual_seed(N + K)
    x = torch.empty(M, K, device="cuda", dtype=torch.bfloat16).normal_(generator=g)
    w = torch.empty(N, K, device="cuda", dtype=torch.bfloat16).normal_(0, 0.05, generator=g)
    packed = w.view(N // 32, 32, K // 64, 2, 4, 8).permute(2, 0, 4, 3, 1, 5).contiguous()   # [k-step][row block][j][half][row][8]
    shape = (splits, M, N) if mode == 0 else (1, M, N // 2)
    y = torch.full((shape[0] * M + 1, shape[2]), float("nan"), device="cuda", dtype=torch.float32 if mode == 0 else torch.bfloat16)
    pl.pl_gemm_bf16(x.data_ptr(), packed.data_ptr(), y.data_ptr(), M, N, K, mode, splits, 0)
    torch.cuda.synchronize()
    assert bool(y[-1].isnan().all())
    got = y[:-1].view(shape).double().sum(0)
    ref = x.double() @ w.double().T
    if mode == 1:
        r = ref.view(M, N // 64, 2, 32)
        ref = (torch.nn.functional.silu(r[:, :, 0]) * r[:, :, 1]).reshape(M, N // 2)
        assert bool((got - ref).abs().le(2 ** -8 * ref.abs() + 1e-3).all())   # rounded to bf16; sums of up to 768 products, both factors
    else:
        assert bool((got - ref).abs().le(1e-4 * np.sqrt(K) * 0.05 + 1e-4 * ref.abs()).all())


@pytest.mark.parametrize("M,mode", [(1, 0), (37, 0), (200, 0), (200, 1)])
def test_products_of_operands_at_any_alignment(M, mode):
    """16-byte accesses, direct loads to LDS among them, on operands that start at any element."""
    N, K = 640, 512
    g = torch.Generator(device="cuda").manual_seed(M)
    x = torch.empty(M * K, device="cuda", dtype=torch.bfloat16).normal_(generator=g)
    w = torch.empty(N * K, device="cuda", dtype=torch.bfloat16).normal_(0, 0.05, generator=g)
    n, dtype = (M * N, torch.float32) if mode == 0 else (M * N // 2, torch.bfloat16)
    want = None
    for ox, ow, oy in [(0, 0, 0), (1, 0, 0), (2, 0, 0), (0, 1, 0), (0, 6, 0), (0, 0, 1), (3, 5, 2)]:
        xs, ws, ys = (torch.zeros(k + 8, device="cuda", dtype=t) for k, t in ((M * K, x.dtype), (N * K, w.dtype), (n, dtype)))
        xs[ox:ox + M * K], ws[ow:ow + N * K] = x, w
        pl.pl_gemm_bf16(xs[ox:].data_ptr(), ws[ow:].data_ptr(), ys[oy:].data_ptr(), M, N, K, mode, 1, 0)
        torch.cuda.synchronize()
        got = ys[oy:oy + n]
        want = got.clone() if want is None else want
        assert bool(want.abs().sum() > 0) and torch.equal(got, want), (ox, ow, oy)
        assert bool((ys[:oy] == 0).all()) and bool((ys[oy + n:] == 0).all())


def test_gemm_rejects_bad_shapes():
    t = torch.zeros(600 * 512, device="cuda", dtype=torch.bfloat16)
    for args in [(4, 64, 192, 0, 1), (0, 64, 256, 0, 1), (4, 64, 512, 0, 3), (4, 96, 256, 1, 1), (4, 64, 512, 1, 2),
                 (4, 64, 256, 2, 1), (600, 64, 256, 0, 1), (4, 48, 256, 0, 1)]:
        with pytest.raises(pl.PlError) as ex:
            pl.pl_gemm_bf16(t.data_ptr(), t.data_ptr(), t.data_ptr(), args[0], args[1], args[2], args[3], args[4], 0)
        assert ex.value.code == pl.PL_E_INVAL


def _gpu_sample(logits, seq_id, pos, temps, forced, seed):
    n, V = logits.shape
    lg = torch.from_numpy(logits).cuda()
    sid = torch.from_numpy(np.asarray(seq_id, np.uint64).view(np.int64)).cuda()
    ps = torch.from_numpy(np.asarray(pos, np.int32)).cuda()
    it = torch.from_numpy((np.float32(1.0) / np.asarray(temps, np.float32)).astype(np.float32)).cuda()
    fr = torch.from_numpy(np.asarray(forced, np.int32)).cuda()
    tok = torch.zeros(n, device="cuda", dtype=torch.int32)
    lp = torch.zeros(n, device="cuda", dtype=torch.float32)
    ws = torch.empty(pl.pl_sample_workspace_bytes(n, V), device="cuda", dtype=torch.uint8)
    pl.pl_sample(lg.data_ptr(), n, V, sid.data_ptr(), ps.data_ptr(), it.data_ptr(), fr.data_ptr(), seed,
                 tok.data_ptr(), lp.data_ptr(), ws.data_ptr(), 0)
    torch.cuda.synchronize()
    return tok.cpu().numpy(), lp.cpu().numpy()


@pytest.mark.parametrize("n,V", [(7, 4096), (4, 152064), (3, 151936), (5, 8)])
def test_sampler_tokens_bit_exact_and_logprobs_close(n, V):
    rng = np.random.default_rng(V + n)
    logits = (rng.standard_normal((n, V)) * 2).astype(np.float32)
    seq_id = rng.integers(0, 2**63, size=n, dtype=np.uint64) * np.uint64(2) + np.uint64(1)
    pos = rng.integers(0, 16384, size=n).astype(np.int32)
    temps = np.array([1.0, 0.7, 1.3, 1.0, 0.5, 2.0, 1.0][:n], np.float32)
    forced = np.full(n, -1, np.int32)
    forced[n - 1] = V // 3
    seed = 0x1234567890ABCDEF
    tok, lp = _gpu_sample(logits, seq_id, pos, temps, forced, seed)
    for r in range(n):
        t_ref, lp_ref = sampler.sample_row(logits[r], float(temps[r]), seed, int(seq_id[r]), int(pos[r]), int(forced[r]))
        assert tok[r] == t_ref, (r, tok[r], t_ref)
        assert abs(lp[r] - lp_ref) <= 1e-4 * max(1.0, abs(lp_ref))


@pytest.mark.parametrize("n,V", [(1, 4), (2, 8188), (2, 8192), (3, 8196), (26, 152064), (27, 152064), (512, 4096), (513, 4096)])
def test_sampler_at_slice_and_launch_boundaries_with_masked_entries(n, V):
    """One slice and a little more or less, both sides of the choice of threads per slice (512 workgroups), and rows
    with masked entries: -inf, the lowest float, a whole masked slice, equal logits."""
    rng = np.random.default_rng(V * 5 + n)
    logits = (rng.standard_normal((n, V)) * 3).astype(np.float32)
    logits[0, : V // 2] = -np.inf
    if n > 1:
        logits[1] = np.float32(-1.25)
    if n > 2:
        logits[2, ::3] = np.finfo(np.float32).min
        logits[2, : min(8192, V // 2)] = -np.inf
    seq_id = rng.integers(0, 2**63, size=n, dtype=np.uint64)
    pos = rng.integers(0, 16384, size=n).astype(np.int32)
    temps = rng.choice([1.0, 0.7, 1.5], n).astype(np.float32)
    tok, lp = _gpu_sample(logits, seq_id, pos, temps, np.full(n, -1, np.int32), 77)
    for r in list(range(min(n, 6))) + [n - 1]:
        with np.errstate(over="ignore"):             # the lowest float at T < 1 becomes -inf
            t_ref, lp_ref = sampler.sample_row(logits[r], float(temps[r]), 77, int(seq_id[r]), int(pos[r]))
        assert tok[r] == t_ref, (r, tok[r], t_ref)
        assert abs(lp[r] - lp_ref) <= 1e-4 * max(1.0, abs(lp_ref))


@pytest.mark.parametrize("n", [3, 513])
@pytest.mark.parametrize("V", [4, 4092, 4096, 4100])
def test_sampler_around_half_a_slice(n, V):
    """Vocabularies of half a slice and a little more or less, on both sides of the choice of threads: the definition's
    tokens, with the last entries drawn and forced and with masked rows; a vocabulary that ends in masked entries
    gives the same bits as one without them."""
    rng = np.random.default_rng(V + n)
    logits = (rng.standard_normal((n, V)) * 3).astype(np.float32)
    logits[0, -1] = 40.0
    logits[1, : V - 2] = -np.inf
    seq_id = rng.integers(0, 2**63, size=n, dtype=np.uint64)
    pos = rng.integers(0, 16384, size=n).astype(np.int32)
    temps = rng.choice([1.0, 0.7, 1.5], n).astype(np.float32)
    forced = np.full(n, -1, np.int32)
    forced[2] = V - 1
    tok, lp = _gpu_sample(logits, seq_id, pos, temps, forced, 5)
    for r in list(range(3)) + [n - 1]:
        t_ref, lp_ref = sampler.sample_row(logits[r], float(temps[r]), 5, int(seq_id[r]), int(pos[r]), int(forced[r]))
        assert tok[r] == t_ref, (r, tok[r], t_ref)
        assert abs(lp[r] - lp_ref) <= 1e-4 * max(1.0, abs(lp_ref))
    masked = np.concatenate([logits, np.full((n, 8192 - V), -np.inf, np.float32)], 1)
    tok2, lp2 = _gpu_sample(masked, seq_id, pos, temps, forced, 5)
    assert np.array_equal(tok, tok2) and np.array_equal(lp.view(np.uint32), lp2.view(np.uint32))


@pytest.mark.parametrize("n,V", [(10, 8), (10, 8196), (60, 152064)])
def test_sampler_where_bounds_say_little_or_nothing(n, V):
    """Rows in which the bounds on the noise decide little (one dominating logit, two far apart from the rest) and rows
    beyond their use, where every entry is computed (large magnitudes, infinities, NaNs): the tokens of the definition."""
    rng = np.random.default_rng(V + 3 * n)
    logits = (rng.standard_normal((n, V)) * 2).astype(np.float32)
    at = rng.integers(0, V, n)
    logits[0, at[0]] = 30.0                     # the others are e^-30 of it
    logits[1, at[1]] = 300.0                    # e^-300 = 0 in fp32
    logits[2, at[2]], logits[2, (at[2] + V // 2) % V] = 40.0, 40.5
    logits[3] += np.float32(1000.0)             # on both sides of the largest magnitude that the bounds are used for
    logits[4] -= np.float32(1030.0)
    logits[5] *= np.float32(3000.0)
    logits[6] = np.float32(65536.0)             # the sum with the noise keeps two binary places
    logits[7, [at[7], V - 1]] = np.inf
    logits[8, ::2] = np.nan
    logits[9] = -np.inf
    seq_id = rng.integers(0, 2**63, size=n, dtype=np.uint64)
    pos = rng.integers(0, 16384, size=n).astype(np.int32)
    tok, lp = _gpu_sample(logits, seq_id, pos, np.ones(n, np.float32), np.full(n, -1, np.int32), 99)
    for r in range(10):
        z = np.where(np.isnan(logits[r]), -np.inf, logits[r])     # a NaN is never drawn
        t_ref = sampler.sample_row(z, 1.0, 99, int(seq_id[r]), int(pos[r]), -1)[0] if r not in (7, 9) else int(np.argmax(z))
        assert tok[r] == t_ref, (r, tok[r], t_ref)
        if r < 7:
            lp_ref = sampler.log_softmax(logits[r])[tok[r]]
            assert abs(lp[r] - lp_ref) <= 1e-4 * max(1.0, abs(lp_ref))


@pytest.mark.parametrize("few,many,V", [(26, 27, 152064), (512, 513, 4096), (128, 129, 32000), (3, 300, 8200)])
def test_a_row_is_sampled_alike_whatever_rows_share_the_call(few, many, V):
    """Both sides of the choice of threads per slice: the same rows' tokens and log-probs are bit-identical."""
    rng = np.random.default_rng(V + few)
    logits = (rng.standard_normal((many, V)) * 3).astype(np.float32)
    logits[0, : V // 2] = -np.inf
    seq_id = rng.integers(0, 2**63, size=many, dtype=np.uint64)
    pos = rng.integers(0, 16384, size=many).astype(np.int32)
    temps = rng.choice([1.0, 0.7, 1.5], many).astype(np.float32)
    forced = np.full(many, -1, np.int32)
    forced[::2] = rng.integers(V // 2, V, len(forced[::2]))
    a = _gpu_sample(logits[:few], seq_id[:few], pos[:few], temps[:few], forced[:few], 77)
    b = _gpu_sample(logits, seq_id, pos, temps, forced, 77)
    assert np.array_equal(a[0], b[0][:few])
    assert np.array_equal(a[1].view(np.uint32), b[1][:few].view(np.uint32))


def test_sampler_ties_resolve_to_the_lowest_index_like_the_oracle():
    """Constant logits: the winner is decided by the noise alone, and with 2^23 distinct uniforms over
    152064 entries equal maxima do occur; both sides must pick the lowest index."""
    n, V = 96, 152064
    logits = np.zeros((n, V), np.float32)
    seq_id = np.arange(n, dtype=np.uint64) + np.uint64(1 << 33)
    pos = np.arange(n, dtype=np.int32) * 3
    tok, lp = _gpu_sample(logits, seq_id, pos, np.ones(n, np.float32), np.full(n, -1, np.int32), 42)
    ties = 0
    for r in range(n):
        g = sampler.gumbel_from_bits(__import__("oracle.philox", fromlist=["x"]).sampler_bits(42, int(seq_id[r]), int(pos[r]), V))
        ties += int((g == g.max()).sum() > 1)
        assert tok[r] == int(np.argmax(g))
        assert abs(lp[r] + np.log(V)) < 1e-4
    print("rows with tied maxima:", ties)
