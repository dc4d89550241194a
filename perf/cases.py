"""The work that users of the MCA layer have it do, as cases that can be timed and checked.

A case is one attention layer: sizes, data type, options of the method, and the structure
of its inputs. ``prepare`` makes the inputs on the GPU from a seed, with the recipe of
``paper_2201_12854_amd.workloads`` (X normal, W_q, W_k, W_v ~ N(0, 0.02^2), Q = X W_q and
K = X W_k rounded to the layer's type; log-normal token scales, scaled queries, ragged
lengths and shared salient keys where a case asks for them), and what a program keeps from
call to call: the prepared weights and, for ``entry`` "plan", the bound ``ForwardPlan``.
``run`` is one forward pass. ``exact`` is the same layer in float64 torch: the softmax, the
count rule, the Philox draws, the estimator and A H~, written from the paper.
"""
import math

import torch

import paper_2201_12854_amd as mca

D_HEAD = 64

DEFAULTS = dict(entry="plan", dtype="bf16", batch=1, seq=128, d_in=768, heads=12, alpha=0.4, sampling="token",
                importance="max", window=0, exact_from=0, len_lo=0, len_hi=0, q_scale=1.0, sigma=0.0, salient=0)


def _case(name, **kw):
    c = dict(DEFAULTS)
    c.update(kw)
    if name:
        c = dict(name=name, **c)
    return c


def listed():
    return [
        # one short sentence through the plain call, as an interactive program makes it: host
        # work, launches and the latency of each stage
        _case("call_bf16_b1_s45", entry="call", batch=1, seq=45, sigma=0.5),
        # one sequence in float32: the smallest of the benchmark's layers, all latency
        _case("base_f32_b1_s128", dtype="f32", batch=1, seq=128),
        # float32 at an ordinary batch of ragged documents
        _case("base_f32_b8_s333_ragged", dtype="f32", batch=8, seq=333, len_lo=100, len_hi=333, sigma=0.5),
        # the BERT-base classification batch (GLUE length 128)
        _case("base_bf16_b32_s128", batch=32, seq=128, sigma=0.5),
        # the same with the paper's input-independent probability and the tight error bound
        _case("base_bf16_b32_s128_weight", batch=32, seq=128, sigma=0.5, alpha=0.2, sampling="weight"),
        # the same with the mean rule (the more aggressive counts)
        _case("base_bf16_b32_s128_mean", batch=32, seq=128, sigma=0.5, importance="mean"),
        # a batch of sentences of very different lengths padded to 128
        _case("base_bf16_b64_padded", batch=64, seq=128, len_lo=16, len_hi=128),
        # BERT-large with sharp attention: every token saturates and is encoded exactly
        _case("large_bf16_b16_s512_q4", batch=16, seq=512, d_in=1024, heads=16, q_scale=4.0),
        # BERT-large at question-answering length, ragged, with counts of every size
        _case("large_bf16_b8_s384_ragged", batch=8, seq=384, d_in=1024, heads=16, len_lo=120, len_hi=384, sigma=0.5),
        # documents through a local window of 256 keys with a global first token (short ones)
        _case("window_bf16_b32_s250", batch=32, seq=250, window=256, len_lo=84, len_hi=250, sigma=0.5),
        # the same for long documents, an odd padded length
        _case("window_bf16_b8_s1057", batch=8, seq=1057, window=256, len_lo=353, len_hi=1057, sigma=0.5),
        # the benchmark's headline: long sequences with a few keys that many queries attend
        _case("long_bf16_b4_s4096", batch=4, seq=4096, salient=32),
    ]


def draw(rng):
    """Another layer of the same ranges: 16 to 4096 tokens a row, 16 to 16384 in a batch."""
    d, heads = rng.choice([(256, 4), (512, 8), (768, 12), (768, 12), (768, 12), (1024, 16)])
    f32 = rng.random() < 0.25
    seq = int(round(math.exp(rng.uniform(math.log(16), math.log(4096 if not f32 else 1024)))))
    # the largest listed case's tokens, and its attention pairs (a quarter of them in float32)
    most = min(16384 // seq, 4 * 4096 * 4096 * 12 // (seq * seq * heads * (4 if f32 else 1)))
    batch = max(1, min(most, int(round(math.exp(rng.uniform(0.0, math.log(64.0)))))))
    c = dict(dtype="f32" if f32 else "bf16", batch=batch, seq=seq, d_in=d, heads=heads,
             alpha=rng.choice([0.2, 0.4, 0.4, 1.0]), sigma=rng.choice([0.0, 0.5]))
    if rng.random() < 0.1:  # a value projection narrower than the layer, in whole and odd chunks
        c["d_in"] = rng.choice([d - 56, d - 24, d - 7])
    if rng.random() < 0.5 and seq >= 32:
        c["len_lo"], c["len_hi"] = max(1, seq // rng.randint(2, 8)), seq
    kind = rng.random()
    if kind < 0.2 and seq >= 100:
        c["window"] = rng.choice([64, 256])
    elif kind < 0.3:
        c["sampling"] = "weight"
    elif kind < 0.4:
        c["importance"] = "mean"
    elif kind < 0.45 and seq <= 256:
        c["importance"] = "median"
    elif kind < 0.55:
        c["q_scale"] = 4.0
    elif kind < 0.6:
        c["exact_from"] = d // 2
    elif kind < 0.7 and seq >= 512:
        c["salient"] = 32
    if batch * seq <= 1024 and rng.random() < 0.5:
        c["entry"] = "call"
    return _case(None, **c)


def _type(case):
    return torch.float32 if case["dtype"] == "f32" else torch.bfloat16


def _inputs(case, seed):
    dev, dt = torch.device("cuda:0"), _type(case)
    g = torch.Generator(device=dev)
    g.manual_seed(int(seed))
    B, n, d_in, H = case["batch"], case["seq"], case["d_in"], case["heads"]
    d_out = H * D_HEAD

    def normal(*shape):
        return torch.randn(*shape, generator=g, device=dev, dtype=torch.float32)

    X = normal(B, n, d_in)
    if case["sigma"] > 0:
        X = X * torch.exp(case["sigma"] * normal(B, n, 1))
    Wq, Wk, Wv = (0.02 * normal(d_in, d_out) for _ in range(3))
    Q = case["q_scale"] * (X.reshape(-1, d_in) @ Wq).reshape(B, n, d_out)
    K = (X.reshape(-1, d_in) @ Wk).reshape(B, n, d_out)
    if case["salient"] > 0:
        # per (row, head) `salient` keys share a direction that every query has a part of:
        # their logits lie 6 above the others'
        c = math.sqrt(D_HEAD * 0.02 * 0.02 * d_in)
        u = normal(B, H, D_HEAD)
        u = u / u.norm(dim=-1, keepdim=True)
        pick = torch.rand(B, H, n, generator=g, device=dev).topk(min(case["salient"], n), dim=-1).indices
        hit = torch.zeros(B, H, n, device=dev).scatter_(2, pick, 1.0)
        K = K + c * (hit.permute(0, 2, 1)[..., None] * u[:, None]).reshape(B, n, d_out)
        Q = Q + 6.0 * math.sqrt(D_HEAD) / c * u.reshape(B, 1, d_out)
    lens = None
    if case["len_hi"]:
        lens = torch.randint(case["len_lo"], case["len_hi"] + 1, (B,), generator=g, device=dev, dtype=torch.int32)
    return [t.to(dt).contiguous() for t in (Q, K, X, Wv)] + [lens]


def _options(case, seed):
    return dict(alpha=case["alpha"], seed=int(seed) * 2654435761 + 7, heads=case["heads"], sampling=case["sampling"],
                window=case["window"], importance=case["importance"], exact_from=case["exact_from"])


def prepare(case, seed):
    Q, K, X, Wv, lens = _inputs(case, seed)
    prep = mca.prepare_weights(Wv)
    kw = dict(_options(case, seed), seq_lens=lens)
    if case["entry"] == "plan":
        return {"plan": mca.ForwardPlan(Q, K, X, Wv, prep, **kw)}
    return {"args": (Q, K, X, Wv, prep), "kw": kw}


def run(state):
    plan = state.get("plan")
    if plan is not None:
        plan.run()
        return {"Y": plan.Y, "r": plan.r}
    out = mca.attention_forward(*state["args"], **state["kw"])
    return {"Y": out.Y, "r": out.r}


def _pairs(case):
    """(query, key) pairs that attend, about: every length at its mean, padded queries included
    (their output rows are written too)."""
    n = case["seq"]
    L = (case["len_lo"] + case["len_hi"]) / 2 if case["len_hi"] else n
    keys = min(L, case["window"] + 2) if case["window"] else L
    return case["batch"] * n * keys, case["batch"] * L


def work(case):
    B, n, d_in, d_out = case["batch"], case["seq"], case["d_in"], case["heads"] * D_HEAD
    es = 4 if case["dtype"] == "f32" else 2
    pairs, tokens = _pairs(case)
    # Q, K, X and W_v in, Y (float32) and r out
    nbytes = es * (2 * B * n * d_out + B * n * d_in + d_in * d_out) + 4 * B * n * (d_out + 1)
    # Q K^T and A H~ once; the sampled encoding at the count that even attention gives,
    # ceil(1 / alpha^2) rows a token (real attention asks for more)
    rows = min(d_in, math.ceil(1.0 / case["alpha"] ** 2))
    return {"bytes": nbytes, "flops": 2 * 2 * pairs * d_out + 2 * rows * tokens * d_out}


def tolerance(case):
    # Against float64 a pass is off by 2e-3 to 2.5e-3 in bfloat16 (A and H~ rounded to it) and
    # by 3e-7 to 7e-7 in float32. Beside that, a count changes by one where its t^2 lies within
    # the softmax's float32 rounding (about 5e-7) of a whole number: rarely more than one token
    # of a layer, but that token then has one draw more, which moves H~ by about a seventh at
    # r = 50 (a draw is |x|_1 |W| / r long, 22 / r times |x W|) and Y by 0.14 / sqrt(batch seq).
    if case["dtype"] == "f32":
        return {"rel": 1e-5 + min(1e-2, 0.28 / math.sqrt(case["batch"] * case["seq"])), "max": 0.5, "differ": 5e-3}
    return {"rel": 1e-2, "max": 0.5, "differ": 5e-3}


# ------------------------------------------------------------------ the layer in 64 bits
_M32 = 0xFFFFFFFF


def _philox(c0, c1, c2, c3, k0, k1):
    """Philox4x32-10 (Salmon et al., SC'11) on int64 tensors that hold 32-bit words."""
    for _ in range(10):
        p0, p1 = c0 * 0xD2511F53, c2 * 0xCD9E8D57
        c0, c1, c2, c3 = ((p1 >> 32) & _M32) ^ c1 ^ k0, p1 & _M32, ((p0 >> 32) & _M32) ^ c3 ^ k1, p0 & _M32
        k0, k1 = (k0 + 0x9E3779B9) & _M32, (k1 + 0xBB67AE85) & _M32
    return c0, c1


def _fixed_point(v):
    """v [*, d] float32, not negative: weights floor(v 2^(32 - e)), v's largest f 2^e."""
    top = v.amax(dim=-1, keepdim=True)
    e = torch.frexp(top)[1]
    ok = (top > 0) & torch.isfinite(top)
    w = torch.floor(torch.ldexp(v.double(), (32 - e).double()))
    return torch.where(ok, w, torch.zeros_like(w)).long()


def _attended(case, n, L, dev):
    i, j = torch.arange(n, device=dev)[:, None], torch.arange(n, device=dev)[None, :]
    ok = (j < L).expand(n, n)
    if case["window"]:
        ok = ok & (((i - j).abs() <= case["window"] // 2) | (i == 0) | (j == 0))
    return ok


def exact(case, seed):
    Q, K, X, Wv, lens = _inputs(case, seed)
    dev = X.device
    B, n, d_in, H = case["batch"], case["seq"], case["d_in"], case["heads"]
    kw = _options(case, seed)
    lens = [n] * B if lens is None else lens.tolist()

    def probs(b, h):
        cols = slice(h * D_HEAD, (h + 1) * D_HEAD)
        S = Q[b, :, cols].double() @ K[b, :, cols].double().t() / 8.0
        return torch.softmax(S.masked_fill(~_attended(case, n, lens[b], dev), -math.inf), dim=1)

    W, x = Wv.double(), X.reshape(B * n, d_in)
    r = torch.zeros(B, n, dtype=torch.long, device=dev)
    for b in range(B):
        L = lens[b]
        if case["importance"] == "max":
            size = _attended(case, n, L, dev).sum(1).double()[:L, None] if case["window"] else float(L)
            t = torch.zeros(L, dtype=torch.float64, device=dev)
            for h in range(H):
                t = torch.maximum(t, (size * probs(b, h)[:L, :L]).amax(0))
        else:
            A = torch.cat([probs(b, h)[:L, :L] for h in range(H)])
            if case["importance"] == "mean":
                t = L * A.mean(0)
            else:
                A = A.sort(0).values
                t = L * 0.5 * (A[(H * L - 1) // 2] + A[H * L // 2])
        r[b, :L] = torch.ceil((t / case["alpha"]) ** 2).clamp(1, d_in).long()
    rho = W.square().sum(1).sqrt().float()
    w = _fixed_point(x.float().abs() * rho) if case["sampling"] == "token" else _fixed_point((rho * rho)[None]).expand(B * n, d_in)
    rr = r.reshape(-1)
    whole = (rr >= d_in) | ((rr >= case["exact_from"]) if case["exact_from"] else torch.zeros_like(rr, dtype=torch.bool))
    coef = torch.zeros(B * n, d_in, dtype=torch.float64, device=dev)
    coef[whole] = x[whole].double()
    todo = torch.nonzero(~whole & (rr > 0) & (w.sum(1) > 0)).reshape(-1)
    if todo.numel():
        ks = torch.arange(int(rr[todo].max()), device=dev)[None, :]
        for part in todo.split(4096):
            wp, rp = w[part], rr[part][:, None]
            C = wp.cumsum(1)
            T = C[:, -1:]
            word = torch.zeros_like(ks) + part[:, None] * 0
            lo, hi = _philox(word + ks, word + (part % n)[:, None], word + (part // n)[:, None], word,
                             kw["seed"] & _M32, (kw["seed"] >> 32) & _M32)
            # floor((lo + hi 2^32) T / 2^64)
            tl, th = T & _M32, T >> 32
            mid = hi * tl
            s = (((lo * tl) >> 32) & _M32) + (mid & _M32) + lo * th
            t = hi * th + ((mid >> 32) & _M32) + (s >> 32)
            at = torch.searchsorted(C.contiguous(), t.contiguous(), right=True).clamp(max=d_in - 1)
            times = torch.zeros(part.numel(), d_in, dtype=torch.float64, device=dev)
            times.scatter_add_(1, at, (ks < rp).expand_as(at).double())
            coef[part] = times * x[part].double() * T.double() / (rp.double() * wp.clamp(min=1).double())
    Ht = (coef @ W).reshape(B, n, -1)
    Y = torch.empty(B, n, H * D_HEAD, dtype=torch.float64, device=dev)
    for b in range(B):
        for h in range(H):
            cols = slice(h * D_HEAD, (h + 1) * D_HEAD)
            Y[b, :, cols] = probs(b, h) @ Ht[b, :, cols]
    return {"Y": Y, "r": r.int()}
