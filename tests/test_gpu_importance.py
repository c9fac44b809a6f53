"""Parity (GPU): truncated importance weights and normalised ESS over packed sequences, through the C
ABI, against the CPU oracle.  The kernel computes in fp64: weights are compared after their rounding to
fp32 (rel 1e-6), sums and ESS values to rel 1e-11 (only the summation order differs)."""
import numpy as np
import pytest
import torch

import paper_2509_19128_amd as pl
from oracle import importance

pytestmark = pytest.mark.gpu


def _run(lp_pi, lp_mu, off, c, want_w=True):
    n_seq = len(off) - 1
    n = int(off[-1])
    d_pi = torch.from_numpy(np.asarray(lp_pi, np.float32)).cuda()
    d_mu = torch.from_numpy(np.asarray(lp_mu, np.float32)).cuda()
    d_off = torch.from_numpy(np.asarray(off, np.int64)).cuda()
    w = torch.full((max(n, 1),), float("nan"), device="cuda", dtype=torch.float32)
    sums = torch.full((n_seq, 2), float("nan"), device="cuda", dtype=torch.float64)
    ess = torch.full((n_seq,), -1.0, device="cuda", dtype=torch.float64)
    tot = torch.full((3,), float("nan"), device="cuda", dtype=torch.float64)
    pl.pl_is_ess(d_pi.data_ptr(), d_mu.data_ptr(), d_off.data_ptr(), n_seq, c, w.data_ptr() if want_w else 0,
                 sums.data_ptr(), ess.data_ptr(), tot.data_ptr(), 0)
    torch.cuda.synchronize()
    return w.cpu().numpy()[:n], sums.cpu().numpy(), ess.cpu().numpy(), tot.cpu().numpy()


def _case(rng, lens, spread):
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    n = int(off[-1])
    mu = (-rng.random(n) * 6).astype(np.float32)
    pi = (mu + rng.normal(0, spread, n)).astype(np.float32)
    return pi, mu, off


@pytest.mark.parametrize("lens,spread,c", [
    ([5], 0.5, 5.0), ([1, 1, 1], 1.0, 5.0), ([0, 7, 0, 300, 1025, 0], 0.8, 5.0), ([4096, 16384, 513, 2], 0.3, 5.0),
    ([255, 256, 257, 1023, 1024, 1025], 2.5, 5.0), ([100] * 1500, 0.7, 2.0), ([3000], 3.0, 1e9)])
def test_weights_and_ess_match_the_oracle(lens, spread, c):
    rng = np.random.default_rng(len(lens) * 1000 + int(spread * 10))
    pi, mu, off = _case(rng, lens, spread)
    w, sums, ess, tot = _run(pi, mu, off, c)
    w_ref, ess_ref, tot_ref = importance.packed_is_ess(pi, mu, off, c)
    assert np.allclose(w, w_ref, rtol=1e-6, atol=0)
    for s, L in enumerate(lens):
        seg = w_ref[off[s]:off[s + 1]]
        assert np.isclose(sums[s, 0], seg.sum(), rtol=1e-11) and np.isclose(sums[s, 1], (seg * seg).sum(), rtol=1e-11)
        if L:
            assert np.isclose(ess[s], ess_ref[s], rtol=1e-11), (s, ess[s], ess_ref[s])
        else:
            assert np.isnan(ess[s])
    assert np.isclose(tot[2], tot_ref, rtol=1e-11)
    assert np.isclose(tot[0], w_ref.sum(), rtol=1e-11) and np.isclose(tot[1], (w_ref * w_ref).sum(), rtol=1e-11)


@pytest.mark.parametrize("shift_pi,shift_mu,shift_w", [(0, 0, 0), (1, 1, 1), (3, 3, 3), (2, 2, 1), (0, 1, 0)])
def test_weights_at_every_alignment_of_the_arrays_and_of_the_sequences(shift_pi, shift_mu, shift_w):
    """Arrays that start on the same and on different positions of a 16-byte line, sequences that begin and end
    anywhere in one, lengths around one round of the workgroup; masked (-inf), infinite and NaN differences as
    fmin(c, exp(.)) has them."""
    rng = np.random.default_rng(5)
    lens = [1, 2, 3, 4, 5, 7, 0, 4095, 4096, 4097, 8191, 4 * 4096 + 3, 6]
    pi, mu, off = _case(rng, lens, 1.5)
    pi[20:26] = [-np.inf, np.inf, np.nan, 800.0, -800.0, 3.0]
    mu[20:26] = [0.0, 0.0, 0.0, 0.0, 0.0, np.nan]

    def shifted(x, k):
        t = torch.zeros(len(x) + 4, device="cuda", dtype=torch.float32)
        t[k:k + len(x)] = torch.from_numpy(x)
        return t
    a, b, w = shifted(pi, shift_pi), shifted(mu, shift_mu), shifted(np.full(len(pi), -7, np.float32), shift_w)
    o = torch.from_numpy(off.astype(np.int64)).cuda()
    sums, ess, tot = (torch.empty(k, device="cuda", dtype=torch.float64) for k in (2 * len(lens), len(lens), 3))
    pl.pl_is_ess(a[shift_pi:].data_ptr(), b[shift_mu:].data_ptr(), o.data_ptr(), len(lens), 5.0, w[shift_w:].data_ptr(), sums.data_ptr(),
                 ess.data_ptr(), tot.data_ptr(), 0)
    torch.cuda.synchronize()
    with np.errstate(over="ignore", invalid="ignore"):
        ref = np.fmin(5.0, np.exp(pi.astype(np.float64) - mu.astype(np.float64)))
    got = w.cpu().numpy()
    assert np.allclose(got[shift_w:shift_w + len(pi)], ref, rtol=1e-6, atol=0)
    assert (got[:shift_w] == 0).all() and (got[shift_w + len(pi):] == 0).all()
    for s in range(len(lens)):
        seg = ref[off[s]:off[s + 1]]
        assert np.isclose(sums[2 * s].item(), seg.sum(), rtol=1e-11) and np.isclose(sums[2 * s + 1].item(), (seg * seg).sum(), rtol=1e-11)


def test_a_weight_is_the_exponential_to_the_last_bits():
    """Sequences of one token and a cap beyond every number: their sums are the exponentials themselves.  The kernel's may be off by 1.1 units in the
    last place (half of one from its table, half from its last addition), numpy's by less than one; subnormal results by one unit of
    their own more."""
    rng = np.random.default_rng(8)
    pi = np.concatenate([rng.uniform(-745, 709, 6000), rng.normal(0, 1, 6000), rng.normal(0, 1e-3, 2000), [0.0, -0.0, 709.78, 710.0, -745.1, -746.5, 1e30,
                         -1e30, np.inf, -np.inf]]).astype(np.float32)
    n = len(pi)
    a, b, o = torch.from_numpy(pi).cuda(), torch.zeros(n, device="cuda"), torch.arange(n + 1, device="cuda")
    sums, ess, tot = (torch.empty(k, device="cuda", dtype=torch.float64) for k in (2 * n, n, 3))
    pl.pl_is_ess(a.data_ptr(), b.data_ptr(), o.data_ptr(), n, np.inf, 0, sums.data_ptr(), ess.data_ptr(), tot.data_ptr(), 0)
    got = sums.cpu().numpy()[::2]
    with np.errstate(over="ignore"):
        ref = np.exp(pi.astype(np.float64))
    fin = np.isfinite(ref)
    assert np.array_equal(got[~fin], ref[~fin])
    off = np.abs(got[fin] - ref[fin]) / np.spacing(ref[fin])
    print("most units in the last place:", off.max())
    assert off.max() <= 2 + (ref[fin][off.argmax()] < 2.3e-308)


def test_a_weight_is_as_near_to_the_exponential_as_the_last_addition_allows():
    """Against 64-bit mantissas, over ordinary results: half a unit in the last place from the rounding of the last addition, 0.03 from what it adds."""
    rng = np.random.default_rng(9)
    x = np.concatenate([rng.uniform(-700, 700, 200000), rng.normal(0, 1, 200000), rng.normal(0, 1e-2, 100000), np.arange(-64, 65) * np.log(2) / 64,
                        (np.arange(-64, 65) + 0.5) * np.log(2) / 64])
    pi = x.astype(np.float32)
    mu = (pi.astype(np.float64) - x).astype(np.float32)   # (the kernel's argument is a difference of two floats)
    n = len(pi)
    a, b, o = torch.from_numpy(pi).cuda(), torch.from_numpy(mu).cuda(), torch.arange(n + 1, device="cuda")
    sums, ess, tot = (torch.empty(k, device="cuda", dtype=torch.float64) for k in (2 * n, n, 3))
    pl.pl_is_ess(a.data_ptr(), b.data_ptr(), o.data_ptr(), n, np.inf, 0, sums.data_ptr(), ess.data_ptr(), tot.data_ptr(), 0)
    assert np.finfo(np.longdouble).nmant >= 63
    ref = np.exp(pi.astype(np.longdouble) - mu.astype(np.longdouble))
    got = sums.cpu().numpy()[::2]
    off = np.abs(got - ref) / np.spacing(ref.astype(np.float64))
    print("most units in the last place:", off.max())
    assert off.max() <= 0.53


@pytest.mark.parametrize("with_w", [True, False])
def test_a_sequences_sums_do_not_depend_on_the_number_of_sequences(with_w):
    """Both sides of the choice of threads (1536 sequences): weights and sums of the same sequences are bit-identical, at the
    lengths where the order of their sums changes (1024 tokens) and a round of it ends."""
    rng = np.random.default_rng(6)
    lens = [1, 5, 255, 257, 1023, 1024, 1025, 2049, 0, 4096, 4099, 8200, 16384]
    got = []
    for n_seq in (len(lens), 1536, 1537, 4000):
        r = np.random.default_rng(6)
        pi, mu, off = _case(r, lens + [3] * (n_seq - len(lens)), 1.5)
        n = int(off[len(lens)])
        if not got:
            first = pi[:n].copy(), mu[:n].copy()
        pi[:n], mu[:n] = first
        a, b, o = torch.from_numpy(pi).cuda(), torch.from_numpy(mu).cuda(), torch.from_numpy(off.astype(np.int64)).cuda()
        w = torch.empty(len(pi), device="cuda") if with_w else None
        sums, ess, tot = (torch.empty(k, device="cuda", dtype=torch.float64) for k in (2 * n_seq, n_seq, 3))
        pl.pl_is_ess(a.data_ptr(), b.data_ptr(), o.data_ptr(), n_seq, 5.0, w.data_ptr() if with_w else 0, sums.data_ptr(), ess.data_ptr(), tot.data_ptr(), 0)
        torch.cuda.synchronize()
        got.append((sums[:2 * len(lens)].cpu().numpy().view(np.int64), ess[:len(lens)].cpu().numpy().view(np.int64), w[:n].cpu().numpy().view(np.int32) if with_w else 0))
    ref = np.fmin(5.0, np.exp(first[0].astype(np.float64) - first[1]))
    ends = np.cumsum([0] + lens)
    for s in range(len(lens)):
        assert np.isclose(got[0][0].view(np.float64)[2 * s], ref[ends[s]:ends[s + 1]].sum(), rtol=1e-11)
    for other in got[1:]:
        assert all(np.array_equal(x, y) for x, y in zip(got[0], other))


def test_many_short_sequences_do_not_take_a_workgroup_of_a_long_one_each():
    """32768 sequences of 16 tokens against 1024 of them, best of several runs: 4 times the time (43 and 10 us), with workgroups
    of 1024 threads for each of them 15 times."""
    def best(n_seq):
        pi, mu, off = _case(np.random.default_rng(1), [16] * n_seq, 1.5)
        a, b, o = torch.from_numpy(pi).cuda(), torch.from_numpy(mu).cuda(), torch.from_numpy(off.astype(np.int64)).cuda()
        sums, ess, tot = (torch.empty(k, device="cuda", dtype=torch.float64) for k in (2 * n_seq, n_seq, 3))
        times = []
        for _ in range(8):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            for _ in range(20):
                pl.pl_is_ess(a.data_ptr(), b.data_ptr(), o.data_ptr(), n_seq, 5.0, 0, sums.data_ptr(), ess.data_ptr(), tot.data_ptr(),
                             torch.cuda.current_stream().cuda_stream)
            e1.record()
            torch.cuda.synchronize()
            times.append(e0.elapsed_time(e1))
        return min(times)
    few, many = best(1024), best(32768)
    assert many < 8 * few, (few, many)


def test_on_policy_batch_is_exactly_one_and_weights_are_optional():
    rng = np.random.default_rng(8)
    lp = (-rng.random(5000) * 9).astype(np.float32)
    off = np.array([0, 17, 17, 4000, 5000])
    w, sums, ess, tot = _run(lp, lp, off, 5.0)
    assert np.array_equal(w, np.ones(5000, np.float32))
    assert ess[0] == 1.0 and np.isnan(ess[1]) and ess[2] == 1.0 and ess[3] == 1.0 and tot[2] == 1.0
    assert tot[0] == 5000.0 and tot[1] == 5000.0
    _, sums2, ess2, tot2 = _run(lp, lp, off, 5.0, want_w=False)            # NULL weight output
    assert np.array_equal(sums, sums2) and np.array_equal(tot, tot2)


def test_runs_are_bit_reproducible_and_bad_arguments_are_rejected():
    rng = np.random.default_rng(9)
    pi, mu, off = _case(rng, [777, 12000, 31], 1.2)
    a, b = _run(pi, mu, off, 5.0), _run(pi, mu, off, 5.0)
    for x, y in zip(a, b):
        assert np.array_equal(x, y, equal_nan=True)
    t = torch.zeros(16, device="cuda", dtype=torch.float64)
    for n_seq, c in [(0, 5.0), (1, 0.0), (1, -1.0)]:
        with pytest.raises(pl.PlError) as ex:
            pl.pl_is_ess(t.data_ptr(), t.data_ptr(), t.data_ptr(), n_seq, c, 0, t.data_ptr(), t.data_ptr(), t.data_ptr(), 0)
        assert ex.value.code == pl.PL_E_INVAL


def test_engine_logprobs_rescored_under_the_same_weights_give_ess_one():
    """Closes the loop of Sec. 2.1 on the GPU path: the behaviour log-probs the engine records, fed
    back as both pi and mu (what an on-policy trainer would compute), give weights 1 and ESS 1."""
    import synth
    M = synth.CONFIGS["tiny"]
    eng = pl.Engine.from_model(M, max_batch=4, max_context=128, kv_pool_tokens=512, kv_page_tokens=32, seed=3, device=0)
    eng.load_weights(eng.pack_weights(synth.make_weights(M, seed=1235), synth.f32_to_bf16_bits))
    prompts = synth.random_prompts(np.random.default_rng(2), 4, 8, M.vocab)
    for i in range(4):
        eng.add_sequence(i, prompts[i], 20)
    lps = {i: [] for i in range(4)}
    for _ in range(8 + 20 - 1):
        o = eng.decode_step()
        for i in range(o["n"]):
            if o["emitted"][i]:
                lps[int(o["slot"][i])].append(float(o["logprob"][i]))
    eng.close()
    flat = np.concatenate([lps[i] for i in range(4)]).astype(np.float32)
    off = np.concatenate([[0], np.cumsum([len(lps[i]) for i in range(4)])])
    assert off[-1] == 80 and np.isfinite(flat).all() and (flat < 0).all()
    w, _, ess, tot = _run(flat, flat, off, 5.0)
    assert np.array_equal(w, np.ones(80, np.float32)) and np.all(ess == 1.0) and tot[2] == 1.0
