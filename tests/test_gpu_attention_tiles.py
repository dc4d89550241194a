"""Attention passes against plain torch in float64 at the edges of their tiles: Y = A H~ with the
library's own H~ (exported), and the column statistic m, over lengths, windows and grid sizes
that choose each kernel."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2201_12854_amd as mca

# (batch, n, heads, window, ragged): the resident kernels' last lengths; the 32x32 output pass with
# partial query and key tiles in blocks of 128 queries, and of 256 where these fill two blocks per
# CU (64 x 500; 8 x 1900 with a short last block; 43 x 500, 12 heads, by the rule for pairs that
# divide over no XCDs); the 16x16 output pass of 5 to 8 key tiles in large grids (90 x 300, 50 x
# 500); 128 queries per block in the output pass (9 x 1900) or in both (17 x 1900) past two blocks
# per CU. float32: the output pass in blocks of 64 queries (most), and of 128 where no CU has less
# to do with these (64 x 500; 8 x 512, 8 heads under a window)
SHAPES = [(2, 64, 4, 0, True), (2, 256, 4, 0, True), (2, 257, 4, 0, True), (1, 320, 4, 0, False),
          (2, 321, 4, 0, True), (1, 384, 8, 0, False), (2, 449, 4, 0, True), (1, 513, 4, 0, False),
          (2, 577, 4, 0, True), (2, 300, 4, 64, True), (2, 333, 4, 2, True), (1, 1057, 4, 256, False),
          (64, 500, 8, 0, True), (8, 1900, 8, 0, True), (43, 500, 12, 0, True), (90, 300, 4, 0, True),
          (50, 500, 8, 0, True), (9, 1900, 8, 0, True), (17, 1900, 4, 0, True), (8, 512, 8, 64, True)]


def _reference(Q, K, H, lens, heads, window):
    """Y, sum_j A |H|, and m per key (|S_i| A under a window), float64, one batch row at a time."""
    B, n, d = Q.shape
    i = torch.arange(n, device=Q.device)
    for b in range(B):
        L = int(lens[b])
        ok = (i < L)[None, :].expand(n, n)
        if window:
            ok = ok & (((i[:, None] - i[None, :]).abs() <= window // 2) | (i[:, None] == 0) | (i[None, :] == 0))
        size = ok.sum(1).double()[:, None] if window else 1.0
        Y = torch.empty(n, d, dtype=torch.float64, device=Q.device)
        Ya = torch.empty_like(Y)
        m = torch.zeros(n, dtype=torch.float64, device=Q.device)
        for h in range(heads):
            c = slice(64 * h, 64 * h + 64)
            S = Q[b, :, c].double() @ K[b, :, c].double().t() / 8
            A = torch.softmax(S.masked_fill(~ok, -float("inf")), 1)
            Y[:, c] = A @ H[b, :, c]
            Ya[:, c] = A @ H[b, :, c].abs()
            m = torch.maximum(m, (size * A)[:L].amax(0))
        m[L:] = 0
        yield b, Y, Ya, m


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("batch,n,heads,window,ragged", SHAPES)
def test_attention_passes(batch, n, heads, window, ragged, dtype):
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    dev, d = torch.device("cuda:0"), 64 * heads
    rng = np.random.default_rng(1000 * n + heads + window)
    new = lambda *s: torch.from_numpy(rng.standard_normal(s, dtype=np.float32)).to(dev)  # noqa: E731
    Q, K, X = (2 * new(batch, n, d)).to(dt), (0.5 * new(batch, n, d)).to(dt), new(batch, n, d).to(dt)
    W = (0.05 * new(d, d)).to(dt)
    lens = rng.integers(max(1, n // 2), n + 1, batch) if ragged else np.full(batch, n)
    r_in = torch.full((batch, n), d, dtype=torch.int32, device=dev)  # H~ = x W_v
    out = mca.attention_forward(Q, K, X, W, mca.prepare_weights(W), 0.4, 1, heads=heads, r_in=r_in, window=window,
                                seq_lens=torch.from_numpy(lens.astype(np.int32)).to(dev), export=True)
    # H~ as the output pass reads it. Each probability is rounded to bfloat16 (2^-9) or float32,
    # beside the float32 logits' error (below 2^-24 times 64 products of at most about 40) and sums.
    H = out.encoded.to(dt).double()
    unit = 2.0 ** -8 if dtype == "bf16" else 1e-5
    for b, Y, Ya, m in _reference(Q, K, H, lens, heads, window):
        assert torch.isfinite(out.Y[b]).all()
        err = (out.Y[b].double() - Y).abs()
        assert (err <= unit * Ya + 1e-30).all(), (b, (err / Ya).max().item())
        L = int(lens[b])
        assert ((out.colmax[b, :L].double() - m[:L]).abs() <= 2e-5 * m[:L] + 2.0 ** -126).all(), b
        assert (out.colmax[b, L:] == 0).all()


# The mean and median rules where the bfloat16 score pass takes blocks of 256 queries, and of 128.
@pytest.mark.parametrize("batch,n,heads", [(9, 1900, 8), (2, 700, 4)])
@pytest.mark.parametrize("importance", ["mean", "median"])
def test_rules_of_the_streaming_score_pass(batch, n, heads, importance):
    dev, d = torch.device("cuda:0"), 64 * heads
    rng = np.random.default_rng(n)
    new = lambda *s: torch.from_numpy(rng.standard_normal(s, dtype=np.float32)).to(dev).bfloat16()  # noqa: E731
    Q, K, X, W = 2 * new(batch, n, d), 0.5 * new(batch, n, d), new(batch, n, 8), new(8, d)
    lens = rng.integers(n // 2, n + 1, batch)
    out = mca.attention_forward(Q, K, X, W, mca.prepare_weights(W), 0.4, 1, heads=heads, export=True, importance=importance,
                                r_in=torch.zeros(batch, n, dtype=torch.int32, device=dev),
                                seq_lens=torch.from_numpy(lens.astype(np.int32)).to(dev))
    for b in range(batch):
        L = int(lens[b])
        A = torch.cat([torch.softmax(Q[b, :L, c:c + 64].double() @ K[b, :L, c:c + 64].double().t() / 8, 1)
                       for c in range(0, d, 64)])
        m = A.mean(0) if importance == "mean" else A.sort(0).values[[(len(A) - 1) // 2, len(A) // 2]].mean(0)
        # each probability as in test_attention_passes; their sum in a chain of at most 100 additions
        # (32 x MT queries of a half wave, the eight halves, heads x query blocks)
        assert ((out.colmax[b, :L].double() - m).abs() <= (2e-5 + 100 * 2.0 ** -24) * m).all(), b
        assert (out.colmax[b, L:] == 0).all()


@pytest.mark.parametrize("window", [0, 128])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_late_logit_past_the_reference(window, dtype):
    # A few queries meet a logit of 100 (144 log2 units: past a float32 sum under a reference from
    # the first key tile) at a key far behind, the others see even attention; under the window
    # only query 0 reaches it.
    dt, n, heads = (torch.bfloat16 if dtype == "bf16" else torch.float32), 700, 4
    dev, d = torch.device("cuda:0"), 64 * heads
    rng = np.random.default_rng(5)
    Q, K = torch.zeros(1, n, d, device=dev), torch.zeros(1, n, d, device=dev)
    for i in (0, 3, 130, 695):
        Q[0, i, :8] = 10.0
    K[0, 600, :8] = 10.0  # dot 800, logit 100
    X = torch.from_numpy(rng.standard_normal((1, n, d), dtype=np.float32)).to(dev)
    W = torch.from_numpy(0.05 * rng.standard_normal((d, d), dtype=np.float32)).to(dev)
    Q, K, X, W = (v.to(dt) for v in (Q, K, X, W))
    r_in = torch.full((1, n), d, dtype=torch.int32, device=dev)
    out = mca.attention_forward(Q, K, X, W, mca.prepare_weights(W), 0.4, 1, heads=heads, r_in=r_in, window=window,
                                export=True)
    H = out.encoded.to(dt).double()
    # the rounding of a float32 logit of 144 log2 units, times ln 2, beside the probabilities'
    unit = 4 * 0.6931 * 2.0 ** -24 * 145 + (2.0 ** -8 if dtype == "bf16" else 1e-5)
    for b, Y, Ya, m in _reference(Q, K, H, [n], heads, window):
        assert ((out.Y[b].double() - Y).abs() <= unit * Ya + 1e-30).all()
        assert ((out.colmax[b].double() - m).abs() <= (unit - 2.0 ** -8 * (dtype == "bf16") + 2e-5) * m + 2.0 ** -126).all()


# One batch row in blocks of 128 queries, and a grid that fills two blocks per CU in blocks of 256
# (bfloat16, full attention). The logits of 8 x 10 x 8.8125 / 8 are 127.14 log2 units: each term is
# finite in float32 under the first tile's reference of 0, the sum of two is not. Keys 4 apart lie
# in different halves of a wave (bfloat16) and in different lanes (float32); under the window query
# 0 meets key 150 in its block's tiles and key 600 past them. One key of 144 units overflows alone.
@pytest.mark.parametrize("batch,n,heads,window,keys,value", [
    (1, 700, 4, 0, (600, 604), 8.8125), (1, 700, 4, 128, (150, 600), 8.8125), (1, 700, 4, 128, (150, 154), 8.8125),
    (9, 1900, 8, 0, (1100, 1104), 8.8125), (9, 1900, 8, 0, (1100,), 10.0)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_late_logits_whose_sum_overflows(batch, n, heads, window, keys, value, dtype):
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    dev, d = torch.device("cuda:0"), 64 * heads
    rng = np.random.default_rng(n + len(keys))
    Q, K = torch.zeros(batch, n, d, device=dev), torch.zeros(batch, n, d, device=dev)
    for h in range(heads):
        Q[:, [0, 3, 130, n - 5], 64 * h:64 * h + 8] = 10.0
        K[:, list(keys), 64 * h:64 * h + 8] = value
    X = torch.from_numpy(rng.standard_normal((batch, n, d), dtype=np.float32)).to(dev)
    W = torch.from_numpy(0.05 * rng.standard_normal((d, d), dtype=np.float32)).to(dev)
    Q, K, X, W = (v.to(dt) for v in (Q, K, X, W))
    r_in = torch.full((batch, n), d, dtype=torch.int32, device=dev)
    out = mca.attention_forward(Q, K, X, W, mca.prepare_weights(W), 0.4, 1, heads=heads, r_in=r_in, window=window,
                                export=True)
    H = out.encoded.to(dt).double()
    # the rounding of a float32 logit of 144 log2 units, times ln 2, beside the probabilities'
    logit, unit = 4 * 0.6931 * 2.0 ** -24 * 145, 2.0 ** -8 if dtype == "bf16" else 1e-5
    for b, Y, Ya, m in _reference(Q, K, H, [n] * batch, heads, window):
        assert ((out.Y[b].double() - Y).abs() <= (logit + unit) * Ya + 1e-30).all(), b
        assert ((out.colmax[b].double() - m).abs() <= (logit + 2e-5) * m + 2.0 ** -126).all(), b


# Row sums of equal terms: adding the same term to a growing float32 sum rounds the same way every
# time, so a long chain of additions shows (16384 keys: 2e-5 for n / 8 additions in one register).
# Every query has key 0's logit 0 and the others' -a / 8; blocks of 128 queries, then of 256.
@pytest.mark.parametrize("a", [1.0, 1.5, 2.25, 3.625, 4.25, 5.5])
@pytest.mark.parametrize("batch", [1, 2])
def test_long_row_sums(batch, a):
    n, heads, dev = 16384, 4, torch.device("cuda:0")
    Q, K = (torch.zeros(batch, n, 64 * heads, dtype=torch.bfloat16, device=dev) for _ in range(2))
    Q[:, :, ::64], K[:, 1:, ::64] = a, -1.0
    X, W = torch.ones(batch, n, 8, dtype=torch.bfloat16, device=dev), torch.ones(8, 64 * heads, dtype=torch.bfloat16, device=dev)
    out = mca.attention_forward(Q, K, X, W, mca.prepare_weights(W), 0.4, 1, heads=heads, export=True,
                                r_in=torch.zeros(batch, n, dtype=torch.int32, device=dev))
    x = np.exp(-a / 8)
    m = torch.full((n,), x, dtype=torch.float64, device=dev)
    m[0] = 1.0
    m /= 1 + (n - 1) * x
    # In units u = 2^-24: the sum's 15 roundings in sequence, each exp2 to two ulps (twice 4), and the
    # exponent, up to 14: log2 to two ulps (4 x 14), its division by the scale, the addition to the
    # dot product and the product with the scale (3 x 14), times ln 2; the exponents of the terms.
    assert ((out.colmax.double() - m).abs() <= (15 + 8 + 0.6932 * 7 * 14 + 2) * 2.0 ** -24 * m).all()
