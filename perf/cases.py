"""Timed cases of the decode framework: what a user of it has the GPU do, through its public entry points.

Engine cases drive slices of the benchmark's decoder shapes (their widths, a few of their layers and a small
vocabulary, so that the logits a pass returns are a small part of it): decode steps of a full batch and of a
batch that has decayed, prompt reading, and whole short rollouts.  The kernel-level cases are the paged
attention, the LM head, the SwiGLU product, the sampler and the trainer-side importance weights.

Every pass forces the tokens it decodes (teacher forcing is part of the step's interface), so that logits of
two implementations can be compared: a sampled near-tie would send the rest of a sequence elsewhere.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2509_19128_amd as pl
import synth

PAGE = 128          # the engine's default page size
VOCAB = 4096        # vocabulary of the engine slices (that of the tiny configuration)
HEADS = {"tiny": (8, 2, 32), "64": (16, 4, 64), "1p5b": (12, 2, 128), "7b": (28, 4, 128), "32b": (40, 8, 128)}
GROW = 512          # positions a decode case's sequences may grow before they are replaced


# ---- the cases -----------------------------------------------------------------------------------------

def listed():
    return [
        # the smallest whole call: admit 4 short prompts, read them, generate, retire (launch and host latency)
        dict(name="rollout tiny b4", kind="rollout", model="tiny", layers=2, batch=4, prompt=16, new=16),
        # decode steps of the 1.5B shape at its benchmark batch: every kernel of a layer is short
        dict(name="decode 1.5b b64", kind="decode", model="1p5b", layers=8, slots=64, batch=64, max_context=8448,
             prompt=256, mean=2048, gmax=7000, steps=4),
        # decode steps of the 7B shape at its benchmark batch and stationary context mix (the headline workload)
        dict(name="decode 7b b256", kind="decode", model="7b", layers=4, slots=256, batch=256, max_context=16896,
             prompt=512, mean=4096, gmax=15000, steps=4),
        # the same engine late in a stage that is not refilled: a few long sequences are left
        dict(name="decode 7b b19 of 256", kind="decode", model="7b", layers=4, slots=256, batch=19, max_context=16896,
             prompt=512, mean=7000, gmax=15000, steps=4),
        # a refilled slot's 512-token prompt, read in batched passes, and its first generated token
        dict(name="prompt 7b 512", kind="prompt", model="7b", layers=4, slots=256, prompt=512, max_context=16896),
        # a long prompt (also what a cache recomputation replays): thousands of positions attend to one another
        dict(name="prompt 1.5b 3001", kind="prompt", model="1p5b", layers=4, slots=64, prompt=3001, max_context=8448),
        # the attention microbenchmark's launch: 512 ragged sequences over one layer's pages
        dict(name="attention 7b b512", kind="attention", heads="7b", n=512, mean=4096, lo=128, hi=16384, page=128),
        # the smallest attention call
        dict(name="attention tiny b5", kind="attention", heads="tiny", n=5, mean=48, lo=1, hi=80, page=32),
        # LM head of the 7B shape at batch 256 (fp32 logits out)
        dict(name="head 7b 256 rows", kind="gemm", M=256, N=152064, K=3584, mode=0, splits=1),
        # gate/up product + SwiGLU of the 32B shape at its batch of 128
        dict(name="swiglu 32b 128 rows", kind="gemm", M=128, N=55296, K=5120, mode=1, splits=1),
        # the sampler over a step's logits
        dict(name="sample 256 x 152064", kind="sample", n=256, vocab=152064),
        # importance weights and effective sample size of one optimizer batch of recorded log-probs
        dict(name="ess 1024 sequences", kind="ess", n=1024, mean=4096, hi=16384),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["decode", "decode", "prompt", "rollout", "attention", "gemm", "gemm", "sample", "ess"])
    if kind == "rollout":
        return dict(kind=kind, model="tiny", layers=rng.randint(1, 3), batch=rng.randint(1, 12), prompt=_log(rng, 2, 80),
                    new=rng.randint(4, 24))
    if kind == "decode":
        model = rng.choice(["tiny", "1p5b", "7b", "32b"])
        slots = rng.choice([16, 64, 96, 128, 200, 256])
        if model == "32b":
            slots = min(slots, 128)
        return dict(kind=kind, model=model, layers=rng.randint(2, 4) if model != "32b" else 2, slots=slots,
                    batch=_log(rng, 1, slots), max_context=8448, prompt=_log(rng, 2, 512), mean=_log(rng, 64, 3500), gmax=7000,
                    steps=rng.randint(2, 4))
    if kind == "prompt":
        model = rng.choice(["tiny", "1p5b", "7b"])
        return dict(kind=kind, model=model, layers=rng.randint(2, 4), slots=rng.choice([16, 64, 128, 256]),
                    prompt=_log(rng, 2, 3500 if model != "7b" else 1500), max_context=8448)
    if kind == "attention":
        hi = _log(rng, 64, 16384)
        return dict(kind=kind, heads=rng.choice(sorted(HEADS)), n=_log(rng, 1, 300), mean=max(16, hi // rng.choice([2, 3, 4])),
                    lo=1, hi=hi, page=rng.choice([32, 64, 128]))
    if kind == "gemm":
        model = rng.choice(["tiny", "1p5b", "7b", "32b"])
        m = synth.CONFIGS[model]
        which = rng.choice(["qkv", "o", "gu", "down", "head"])
        n, k = {"qkv": (m.q_dim + 2 * m.kv_dim, m.d_model), "o": (m.d_model, m.q_dim), "gu": (2 * m.d_ffn, m.d_model),
                "down": (m.d_model, m.d_ffn), "head": (m.vocab, m.d_model)}[which]
        mode = 1 if which == "gu" else 0
        most = k // 256
        ok = [s for s in range(1, 10) if s <= most and (s - 1) * -(-most // s) < most]
        rows = _log(rng, 1, 256) if which == "head" else _log(rng, 1, 512)
        return dict(kind=kind, M=rows, N=n, K=k, mode=mode, splits=rng.choice(ok) if which in ("qkv", "o", "down") else 1)
    if kind == "sample":
        return dict(kind=kind, n=_log(rng, 1, 256), vocab=rng.choice([4096, 32000, 151936, 152064]))
    return dict(kind=kind, n=_log(rng, 1, 1024), mean=_log(rng, 16, 4096), hi=16384)


# ---- shapes --------------------------------------------------------------------------------------------

def _shape(case):
    """The decoder slice of an engine case."""
    m = synth.CONFIGS[case["model"]]
    return synth.ModelCfg(case["layers"], m.d_model, m.n_q_heads, m.n_kv_heads, m.head_dim, m.d_ffn, VOCAB)


def _tensors(m):
    """The weight blob, as documented in pl.h: (name, element offset, rows, columns); columns 1 for gains."""
    out, off = [], 0

    def add(name, r, c):
        nonlocal off
        out.append((name, off, r, c))
        off += r * c

    add("embed", m.vocab, m.d_model)
    for l in range(m.n_layers):
        add(f"{l}.g1", m.d_model, 1)
        add(f"{l}.qkv", m.q_dim + 2 * m.kv_dim, m.d_model)
        add(f"{l}.o", m.d_model, m.q_dim)
        add(f"{l}.g2", m.d_model, 1)
        add(f"{l}.gu", 2 * m.d_ffn, m.d_model)
        add(f"{l}.d", m.d_model, m.d_ffn)
    add("gf", m.d_model, 1)
    add("head", m.vocab, m.d_model)
    return out, off


def _contexts(case):
    """Positions already cached per sequence of a decode case, or lengths of an attention / ESS case: sizes, so
    a function of the case alone."""
    r = np.random.default_rng([case.get("n", case.get("batch")), case["mean"], case.get("hi", case.get("gmax"))])
    if case["kind"] == "decode":
        _, age = synth.stationary_ages(r, case["batch"], case["mean"], 1, case["gmax"])
        return (case["prompt"] - 1 + age).astype(np.int64)
    return synth.lognormal_lengths(r, case["n"], case["mean"], case.get("lo", 1), case["hi"])


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _weights(m, seed):
    tensors, n = _tensors(m)
    blob = torch.empty(n, device="cuda", dtype=torch.bfloat16).normal_(0, 0.02, generator=_gen(seed))
    for name, off, r, c in tensors:
        if c == 1:
            blob[off:off + r] = 1.0
    return blob


def _fill_kv(pool, seed):
    pool.normal_(0, 1, generator=_gen(seed + 1))


class _Device:
    """A device buffer that the library owns, for torch.as_tensor."""

    def __init__(self, ptr, n):
        self.__cuda_array_interface__ = dict(shape=(n,), typestr="<i2", data=(ptr, False), version=2)


def _cache(eng):
    """The engine's KV pages as a tensor."""
    ptr, nbytes = eng.debug_kv_pool()
    return torch.as_tensor(_Device(ptr, nbytes // 2), device="cuda").view(torch.bfloat16)


def _pages(tokens):
    return -(-int(tokens) // PAGE)


def _decode_pool_pages(ctx):
    return sum(_pages(c + GROW + 1) for c in ctx)


def _tokens(case, seed):
    """Tokens of an engine case: prompts [batch, prompt], forced tokens [steps, batch]."""
    r = np.random.default_rng(seed)
    batch = case.get("batch", 1)
    steps = case.get("new", case.get("steps", 1))
    return (r.integers(0, VOCAB, (batch, case["prompt"]), dtype=np.int32), r.integers(0, VOCAB, (steps, batch), dtype=np.int32),
            r.integers(0, VOCAB, batch, dtype=np.int32))


# ---- prepare -------------------------------------------------------------------------------------------

def _engine(case, m, slots, max_context, pool_tokens, seed):
    eng = pl.Engine.from_model(m, max_batch=slots, max_context=max_context, kv_pool_tokens=pool_tokens, n_weight_buffers=1,
                               seed=seed & 0xFFFF, device=0)
    blob = _weights(m, seed)
    torch.cuda.synchronize()
    eng.load_weights(blob.data_ptr(), blob.numel() * 2)
    return eng


def _admit(st):
    case = st["case"]
    for i, c in enumerate(st["ctx"]):
        c = int(c)
        st["eng"].debug_add_sequence_at(i, st["prompts"][i], case["prompt"], case["max_context"] - case["prompt"], 1.0, c,
                                        max(0, c - (case["prompt"] - 1)), int(st["last"][i]))
    st["grown"] = 0


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("rollout", "decode", "prompt"):
        m = _shape(case)
        prompts, forced, last = _tokens(case, seed)
        st = dict(case=case, prompts=prompts, last=last)
        if kind == "rollout":
            ctx = case["prompt"] + case["new"]
            st["eng"] = _engine(case, m, case["batch"], ctx, case["batch"] * _pages(ctx) * PAGE, seed)
            st["forced"] = forced
        elif kind == "prompt":
            st["eng"] = _engine(case, m, case["slots"], case["max_context"], _pages(case["prompt"]) * PAGE, seed)
            st["forced"] = np.full((1, case["slots"]), -1, np.int32)
            st["forced"][:, 0] = forced[:, 0]
        else:
            st["ctx"] = _contexts(case)
            st["eng"] = _engine(case, m, case["slots"], case["max_context"], _decode_pool_pages(st["ctx"]) * PAGE, seed)
            _fill_kv(_cache(st["eng"]), seed)
            st["forced"] = np.full((case["steps"], case["slots"]), -1, np.int32)
            st["forced"][:, :case["batch"]] = forced
            _admit(st)
        if kind != "decode":
            st["cache"] = _cache(st["eng"])
        torch.cuda.synchronize()
        return st

    g = _gen(seed)
    if kind == "attention":
        hq, hkv, hd = HEADS[case["heads"]]
        ctx, page = _contexts(case), case["page"]
        per_seq = -(-case["hi"] // page)
        need = -(-ctx // page)
        total = int(need.sum())
        pool = torch.empty(total * hkv * 2 * page * hd, device="cuda", dtype=torch.bfloat16).normal_(0, 1, generator=g)
        ids = np.random.default_rng(seed).permutation(total).astype(np.int32)
        table = np.zeros((case["n"], per_seq), np.int32)
        at = 0
        for b, k in enumerate(need):
            table[b, :k] = ids[at:at + k]
            at += k
        ws = pl.pl_attention_workspace_bytes(case["n"], hq, hkv, hd, case["hi"])
        return dict(case=case, dims=(case["n"], hq, hkv, hd, page, per_seq, case["hi"]), pool=pool,
                    q=torch.empty(case["n"], hq, hd, device="cuda", dtype=torch.bfloat16).normal_(0, 1, generator=g),
                    table=torch.from_numpy(table).cuda(), ctx=torch.from_numpy(ctx.astype(np.int32)).cuda(),
                    out=torch.empty(case["n"], hq, hd, device="cuda", dtype=torch.bfloat16),
                    ws=torch.empty(ws, device="cuda", dtype=torch.uint8))
    if kind == "gemm":
        M, N, K = case["M"], case["N"], case["K"]
        y = (torch.empty(case["splits"], M, N, device="cuda") if case["mode"] == 0 else
             torch.empty(M, N // 2, device="cuda", dtype=torch.bfloat16))
        return dict(case=case, y=y, x=torch.empty(M, K, device="cuda", dtype=torch.bfloat16).normal_(0, 1, generator=g),
                    w=torch.empty(N * K, device="cuda", dtype=torch.bfloat16).normal_(0, 0.02, generator=g))
    if kind == "sample":
        n, v = case["n"], case["vocab"]
        r = np.random.default_rng(seed)
        return dict(case=case, seed=seed, logits=torch.empty(n, v, device="cuda").normal_(0, 2, generator=g),
                    seq_id=torch.from_numpy(r.integers(0, 1 << 40, n)).cuda(),
                    pos=torch.from_numpy(r.integers(0, 16384, n).astype(np.int32)).cuda(),
                    inv_t=torch.from_numpy(r.choice([1.0, 1.0 / 0.7], n).astype(np.float32)).cuda(),
                    forced=torch.full((n,), -1, device="cuda", dtype=torch.int32),
                    token=torch.empty(n, device="cuda", dtype=torch.int32), logprob=torch.empty(n, device="cuda"),
                    ws=torch.empty(pl.pl_sample_workspace_bytes(n, v), device="cuda", dtype=torch.uint8))
    lens = _contexts(case)
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    mu = -6 * torch.rand(int(off[-1]), device="cuda", generator=g)
    pi = mu + 0.3 * torch.randn(int(off[-1]), device="cuda", generator=g)
    return dict(case=case, mu=mu, pi=pi, off=torch.from_numpy(off).cuda(), w=torch.empty_like(mu),
                sums=torch.empty(case["n"], 2, device="cuda", dtype=torch.float64),
                ess=torch.empty(case["n"], device="cuda", dtype=torch.float64),
                tot=torch.empty(3, device="cuda", dtype=torch.float64))


# ---- run -----------------------------------------------------------------------------------------------

def _steps(eng, forced):
    """Decode steps with these forced tokens: logits of the last one, log-probs and tokens of all."""
    logprob, token = [], []
    for f in forced:
        out = eng.decode_step(f)
        logprob.append(out["logprob"].copy())
        token.append(out["token"].copy())
    return dict(logits=eng.debug_get_logits(out["n"]), logprob=np.stack(logprob), token=np.stack(token))


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "decode":
        if st["grown"] + case["steps"] > GROW:          # every sequence is replaced by one of its original age
            for s in range(case["batch"]):
                st["eng"].retire_sequence(s)
            _admit(st)
        st["grown"] += case["steps"]
        return _steps(st["eng"], st["forced"])
    if kind in ("rollout", "prompt"):
        eng = st["eng"]
        slots = [eng.add_sequence(i, p, len(st["forced"]), 1.0) for i, p in enumerate(st["prompts"])]
        for s in slots:
            eng.prefill(s)
        out = _steps(eng, st["forced"])
        for s in slots:
            eng.retire_sequence(s)
        out["cache"] = st["cache"].clone()      # the pages end with the engine
        return out
    stream = torch.cuda.current_stream().cuda_stream
    if kind == "attention":
        pl.pl_attention_decode(st["q"].data_ptr(), st["pool"].data_ptr(), st["table"].data_ptr(), st["ctx"].data_ptr(),
                               st["out"].data_ptr(), st["ws"].data_ptr(), *st["dims"], stream)
        return st["out"]
    if kind == "gemm":
        pl.pl_gemm_bf16(st["x"].data_ptr(), st["w"].data_ptr(), st["y"].data_ptr(), case["M"], case["N"], case["K"],
                        case["mode"], case["splits"], stream)
        return st["y"]
    if kind == "sample":
        pl.pl_sample(st["logits"].data_ptr(), case["n"], case["vocab"], st["seq_id"].data_ptr(), st["pos"].data_ptr(),
                     st["inv_t"].data_ptr(), st["forced"].data_ptr(), st["seed"], st["token"].data_ptr(),
                     st["logprob"].data_ptr(), st["ws"].data_ptr(), stream)
        return dict(token=st["token"], logprob=st["logprob"])
    pl.pl_is_ess(st["pi"].data_ptr(), st["mu"].data_ptr(), st["off"].data_ptr(), case["n"], 5.0, st["w"].data_ptr(),
                 st["sums"].data_ptr(), st["ess"].data_ptr(), st["tot"].data_ptr(), stream)
    return dict(w=st["w"], sums=st["sums"], ess=st["ess"], tot=st["tot"])


# ---- what a pass cannot do without ----------------------------------------------------------------------

def work(case):
    kind = case["kind"]
    if kind in ("rollout", "decode", "prompt"):
        m = _shape(case)
        layer = sum(r * c for _, _, r, c in _tensors(m)[0] if c > 1) - 2 * m.vocab * m.d_model
        head, kv = m.vocab * m.d_model, 2 * m.n_layers * m.kv_dim * 2
        if kind == "decode":
            total, steps, b = float(_contexts(case).sum()), case["steps"], case["batch"]
            seen = steps * total + b * steps * (steps + 1) / 2
            return dict(bytes=steps * (2 * (layer + head) + b * m.vocab * 4) + (seen + steps * b) * kv,
                        flops=2.0 * steps * b * (layer + head) + 4.0 * seen * m.n_layers * m.q_dim)
        b, p, new = case.get("batch", 1), case["prompt"], case.get("new", 1)
        end = p - 1 + new
        reads = sum(range(p, end + 1)) * b                  # positions the decode steps attend to
        return dict(bytes=(new + (p > 1)) * 2.0 * layer + new * (2.0 * head + b * m.vocab * 4) + (reads + b * end) * kv,
                    flops=2.0 * b * end * layer + 2.0 * new * b * head + 2.0 * b * end * (end + 1) * m.n_layers * m.q_dim)
    if kind == "attention":
        hq, hkv, hd = HEADS[case["heads"]]
        total = float(_contexts(case).sum())
        return dict(bytes=total * 4 * hkv * hd + case["n"] * hq * hd * 4, flops=4.0 * total * hq * hd)
    if kind == "gemm":
        M, N, K = case["M"], case["N"], case["K"]
        return dict(bytes=2.0 * (N * K + M * K) + (4.0 * case["splits"] * M * N if case["mode"] == 0 else 1.0 * M * N),
                    flops=2.0 * M * N * K)
    if kind == "sample":
        return dict(bytes=4.0 * case["n"] * case["vocab"], flops=0)
    return dict(bytes=12.0 * float(_contexts(case).sum()), flops=0)


def tolerance(case):
    kind = case["kind"]
    if kind in ("rollout", "decode", "prompt"):
        return {"rel": 0.03, "max": 0.2, "differ": 0.0}     # bf16 activations and cache, rounded in every layer
    if kind == "attention":
        return {"rel": 0.01, "max": 0.05}                   # bf16 probabilities and result
    if kind == "gemm":
        return {"rel": 1e-5, "max": 2e-5} if case["mode"] == 0 else {"rel": 0.008, "max": 0.02}
    if kind == "sample":
        return {"rel": 1e-5, "max": 1e-4, "differ": 0.0}    # the draw is specified bit by bit
    return {"rel": 1e-6, "max": 1e-6}


# ---- the same in 64 bits ---------------------------------------------------------------------------------

def _unpack(w, n, k):
    """Operand order -> [n, k], float64."""
    return w.view(k // 64, n // 32, 4, 2, 32, 8).permute(1, 4, 0, 3, 2, 5).reshape(n, k).double()


def _unpack_kv(pages, hd):
    """[pages, K|V, page * hd] of one kv head in operand order -> keys, values [tokens, hd], float64."""
    n = pages.shape[0]
    k = pages[:, 0].reshape(n, -1, 2, hd // 8, 4, 4, 8).permute(0, 1, 4, 2, 5, 3, 6).reshape(-1, hd)
    v = pages[:, 1].reshape(n, -1, hd // 16, 4, 16, 8).permute(0, 1, 3, 5, 2, 4).reshape(-1, hd)
    return k.double(), v.double()


def _pack_kv(k, v, pages):
    """Keys, values [tokens, Hkv, hd] -> pages [pages, Hkv, K|V, page * hd] in operand order, zeros beyond the tokens."""
    n, hkv, hd = k.shape
    pad = lambda x: torch.cat([x, x.new_zeros(pages * PAGE - n, hkv, hd)]).transpose(0, 1)   # noqa: E731
    k = pad(k).reshape(hkv, pages, -1, 4, 2, 4, hd // 8, 8).permute(1, 0, 2, 4, 6, 3, 5, 7).reshape(pages, hkv, -1)
    v = pad(v).reshape(hkv, pages, -1, 4, 8, hd // 16, 16).permute(1, 0, 2, 5, 3, 6, 4).reshape(pages, hkv, -1)
    return torch.stack([k, v], 2)


class _Decoder:
    """The decoder in float64 on the blob's weights; one growing cache per sequence and layer."""

    def __init__(self, m, blob):
        self.m, self.w = m, {}
        for name, off, r, c in _tensors(m)[0]:
            t = blob[off:off + r * c]
            self.w[name] = t.double() if c == 1 else t.view(r, c).double() if name == "embed" else _unpack(t, r, c)

    def norm(self, h, g):
        return h / torch.sqrt((h * h).mean(-1, keepdim=True) + self.m.rms_eps) * g

    def rope(self, x, pos):
        hd = self.m.head_dim
        inv = self.m.rope_theta ** (-2.0 * torch.arange(hd // 2, device="cuda", dtype=torch.float64) / hd)
        ang = (pos.double()[:, None] * inv)[:, None, :]
        a, b = x[..., :hd // 2], x[..., hd // 2:]
        return torch.cat([a * ang.cos() - b * ang.sin(), b * ang.cos() + a * ang.sin()], -1)

    def forward(self, tokens, pos, attend):
        """Rows (token, position) -> logits; attend(layer, q, k, v) appends the rows' keys and values and attends."""
        m = self.m
        h = self.w["embed"][tokens]
        for l in range(m.n_layers):
            a = self.norm(h, self.w[f"{l}.g1"])
            q, k, v = (a @ self.w[f"{l}.qkv"].T).split([m.q_dim, m.kv_dim, m.kv_dim], -1)
            q = self.rope(q.view(-1, m.n_q_heads, m.head_dim), pos)
            k = self.rope(k.view(-1, m.n_kv_heads, m.head_dim), pos)
            o = attend(l, q, k, v.view(-1, m.n_kv_heads, m.head_dim))
            h = h + o.reshape(len(tokens), -1) @ self.w[f"{l}.o"].T
            gu = (self.norm(h, self.w[f"{l}.g2"]) @ self.w[f"{l}.gu"].T).view(len(tokens), -1, 2, 32)
            mid = torch.nn.functional.silu(gu[:, :, 0]) * gu[:, :, 1]
            h = h + mid.reshape(len(tokens), -1) @ self.w[f"{l}.d"].T
        return self.norm(h, self.w["gf"]) @ self.w["head"].T


def _attend_one(q, k, v, first=None):
    """q [rows, Hq, hd], k/v [tokens, Hkv, hd]; row i sees tokens 0 .. first + i (all of them if first is None)."""
    group = q.shape[1] // k.shape[1]
    q, k, v = q.transpose(0, 1), k.transpose(0, 1).repeat_interleave(group, 0), v.transpose(0, 1).repeat_interleave(group, 0)
    s = torch.matmul(q, k.transpose(1, 2).contiguous()) / math.sqrt(q.shape[-1])
    if first is not None:
        i = torch.arange(q.shape[1], device="cuda")[:, None] + first
        s = s.masked_fill(torch.arange(k.shape[1], device="cuda")[None, :] > i, -math.inf)
    return torch.matmul(s.softmax(-1), v).transpose(0, 1)


def _exact_engine(case, seed):
    m = _shape(case)
    prompts, forced, last = _tokens(case, seed)
    dec = _Decoder(m, _weights(m, seed))
    batch = len(prompts)
    cache = [[None] * m.n_layers for _ in range(batch)]
    if case["kind"] == "decode":
        # a new engine hands out its pages in ascending order, admission by admission
        ctx = _contexts(case)
        pages = _decode_pool_pages(ctx)
        pool = torch.empty(m.n_layers * pages * m.n_kv_heads * 2 * PAGE * m.head_dim, device="cuda", dtype=torch.bfloat16)
        _fill_kv(pool, seed)
        pool = pool.view(m.n_layers, pages, m.n_kv_heads, 2, -1)
        at = 0
        for b, c in enumerate(ctx):
            c, need = int(c), _pages(max(int(c), case["prompt"]))
            for l in range(m.n_layers):
                kv = [_unpack_kv(pool[l, at:at + need, g], m.head_dim) for g in range(m.n_kv_heads)]
                cache[b][l] = tuple(torch.stack([x[i][:c] for x in kv], 1).bfloat16() for i in (0, 1))   # bf16 values: kept as such
            at += need
        pos = torch.from_numpy(ctx).cuda()
        token = torch.tensor([int(prompts[b][c]) if c < case["prompt"] else int(last[b]) for b, c in enumerate(ctx)], device="cuda")
    else:
        # prompts up to the last token; all rows of a sequence at once, causal
        for b in range(batch):
            n = case["prompt"] - 1
            if not n:
                continue

            def read(l, q, k, v, b=b):
                cache[b][l] = (k, v)
                return torch.cat([_attend_one(q[i:i + 512], k[:i + 512], v[:i + 512], i) for i in range(0, len(q), 512)])
            dec.forward(torch.from_numpy(prompts[b][:n].astype(np.int64)).cuda(), torch.arange(n, device="cuda"), read)
        pos = torch.full((batch,), case["prompt"] - 1, device="cuda")
        token = torch.from_numpy(prompts[:, -1].astype(np.int64)).cuda()

    new = [[None] * m.n_layers for _ in range(batch)]     # keys and values of the steps, float64

    def attend(l, q, k, v):
        out = []
        for b in range(batch):
            kv = (k[b:b + 1], v[b:b + 1])
            new[b][l] = kv if new[b][l] is None else tuple(torch.cat(t) for t in zip(new[b][l], kv))
            old = cache[b][l]
            kk, vv = new[b][l] if old is None else tuple(torch.cat([o.double(), n]) for o, n in zip(old, new[b][l]))
            out.append(_attend_one(q[b:b + 1], kk, vv))
        return torch.cat(out)

    logprob = []
    for f in forced:
        logits = dec.forward(token, pos, attend)
        token = torch.from_numpy(f.astype(np.int64)).cuda()
        logprob.append(logits.log_softmax(-1).gather(1, token[:, None])[:, 0])
        pos = pos + 1
    got = dict(logits=logits, logprob=torch.stack(logprob), token=None)
    if case["kind"] != "decode":     # admitted in order, each sequence's pages follow the last one's
        dense = lambda b, l, i: torch.cat([t[b][l][i] for t in (cache, new) if t[b][l] is not None])   # noqa: E731
        got["cache"] = torch.stack([torch.cat([_pack_kv(dense(b, l, 0), dense(b, l, 1), _pages(case["prompt"] + len(forced) - 1))
                                               for b in range(batch)]) for l in range(m.n_layers)]).reshape(-1)
    return got


def _exact_sample(case, st):
    """Philox4x32-10 keyed by (seed; vocabulary index / 4, position, sequence id), Gumbel-max, log-softmax."""
    n, v, mask = case["n"], case["vocab"], 0xFFFFFFFF

    def mul(c, x):       # high and low half of the 32 x 32 bit product
        lo, hi = (x & 0xFFFF) * c, (x >> 16) * c
        t = hi + (lo >> 16)
        return t >> 16, ((t & 0xFFFF) << 16) | (lo & 0xFFFF)

    shape = (n, v // 4)
    c = [torch.arange(v // 4, device="cuda").expand(shape), st["pos"].long()[:, None].expand(shape),
         (st["seq_id"] & mask)[:, None].expand(shape), (st["seq_id"] >> 32)[:, None].expand(shape)]
    k0, k1 = st["seed"] & mask, st["seed"] >> 32
    for r in range(10):
        if r:
            k0, k1 = (k0 + 0x9E3779B9) & mask, (k1 + 0xBB67AE85) & mask
        (h0, l0), (h1, l1) = mul(0xD2511F53, c[0]), mul(0xCD9E8D57, c[2])
        c = [h1 ^ c[1] ^ k0, l1, h0 ^ c[3] ^ k1, l0]
    u = (torch.stack(c, -1).reshape(n, v) >> 9).double().mul_(2).add_(1).mul_(2.0 ** -24)
    z = st["logits"].double() * st["inv_t"].double()[:, None]
    token = (z - torch.log(-torch.log(u))).argmax(1)
    return dict(token=token.int(), logprob=z.log_softmax(1).gather(1, token[:, None])[:, 0])


def exact(case, seed):
    kind = case["kind"]
    if kind in ("rollout", "decode", "prompt"):
        return _exact_engine(case, seed)
    st = prepare(case, seed)
    if kind == "attention":
        n, hq, hkv, hd, page, _, _ = st["dims"]
        pool = st["pool"].view(-1, hkv, 2, page * hd)
        out = []
        for b, c in enumerate(st["ctx"].tolist()):
            ids = st["table"][b, :-(-c // page)].long()
            kv = [_unpack_kv(pool[ids, g], hd) for g in range(hkv)]
            k, v = (torch.stack([x[i][:c] for x in kv], 1) for i in (0, 1))
            out.append(_attend_one(st["q"][b:b + 1].double(), k, v))
        return torch.cat(out)
    if kind == "gemm":
        x, w = st["x"].double(), _unpack(st["w"], case["N"], case["K"])
        if case["mode"] == 1:
            y = (x @ w.T).view(case["M"], -1, 2, 32)
            return (torch.nn.functional.silu(y[:, :, 0]) * y[:, :, 1]).reshape(case["M"], -1)
        c = 256 * -(-(case["K"] // 256) // case["splits"])
        return torch.stack([x[:, s * c:(s + 1) * c] @ w[:, s * c:(s + 1) * c].T for s in range(case["splits"])])
    if kind == "sample":
        return _exact_sample(case, st)
    off, d = st["off"].tolist(), (st["pi"].double() - st["mu"].double())
    w = d.exp().clamp(max=5.0)
    sums = torch.stack([torch.stack([t.sum(), (t * t).sum()]) for t in (w[a:b] for a, b in zip(off, off[1:]))])
    lens = torch.tensor(np.diff(off), device="cuda", dtype=torch.float64)
    tot = sums.sum(0)
    return dict(w=w, sums=sums, ess=sums[:, 0] ** 2 / (lens * sums[:, 1]),
                tot=torch.stack([tot[0], tot[1], tot[0] ** 2 / (off[-1] * tot[1])]))
