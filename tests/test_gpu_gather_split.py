"""The gather's split of the tokens over its blocks: every token once, at its own row, where the
tokens are fewer than the blocks of a slice, end inside a pass, or take one pass or two. Rows of x
with a single entry x_i, so that the estimate is x_i W[i, :] whatever is drawn."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2201_12854_amd as mca


# 768 columns: 24 slices with 10 blocks each on 256 CUs, 1024 tokens of a block in a pass
@pytest.mark.parametrize("dtype,d_in,heads,batch,n", [
    ("bf16", 768, 12, 1, 1), ("bf16", 768, 12, 1, 9), ("bf16", 768, 12, 1, 11), ("bf16", 768, 12, 3, 67),
    ("bf16", 768, 12, 10, 1024), ("bf16", 768, 12, 10, 1025), ("bf16", 761, 12, 3, 67), ("bf16", 1024, 16, 5, 333),
    ("bf16", 1024, 16, 8, 513), ("f32", 768, 12, 3, 67), ("f32", 768, 12, 10, 1025), ("f32", 1000, 16, 2, 333)])
def test_every_token_at_its_row(dtype, d_in, heads, batch, n):
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    dev, d = torch.device("cuda:0"), 64 * heads
    rng = np.random.default_rng(n + d_in)
    new = lambda *s: torch.from_numpy(rng.standard_normal(s, dtype=np.float32)).to(dev)  # noqa: E731
    Q, K, W = new(batch, n, d).to(dt), new(batch, n, d).to(dt), new(d_in, d).to(dt)
    at = torch.from_numpy(rng.integers(0, d_in, (batch, n))).to(dev)
    x = (1 + new(batch, n).abs()).to(dt)
    X = torch.zeros(batch, n, d_in, dtype=dt, device=dev).scatter_(2, at[..., None], x[..., None])
    # none, sampled and saturated tokens
    r = np.where(rng.random((batch, n)) < 0.6, rng.integers(1, d_in, (batch, n)), rng.choice([0, d_in], (batch, n)))
    r_in = torch.from_numpy(r.astype(np.int32)).to(dev)
    out = mca.attention_forward(Q, K, X, W, mca.prepare_weights(W), 0.4, 1, heads=heads, r_in=r_in, export=True)
    ref = x.double()[..., None] * W.double()[at] * (r_in > 0)[..., None]
    # one coefficient and one product rounded to float32, their sum with zeros exact
    assert ((out.encoded.double() - ref).abs() <= 3 * 2.0 ** -24 * ref.abs()).all()
