"""The additive attention bias at rows of every length and alignment: odd rows start between dwords, the last row ends the
buffer's range, and what lies around the matrix (NaN here) must not reach a result."""

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("S", [1, 2, 7, 8, 9, 33, 127, 128, 129, 131, 255, 258, 391])
@pytest.mark.parametrize("skew", [0, 1])
@pytest.mark.parametrize("kind", ["full", "batch", "head"])
def test_rows(S, D, skew, kind):
    import torch
    from paper_2212_01005_amd import binding as ago
    B, Hh, scale = 2, 3, D ** -0.5
    gen = torch.Generator().manual_seed(100 * S + D + skew)
    q, k, v = (torch.randn(B, Hh, S, D, generator=gen).to(torch.bfloat16) for _ in range(3))
    shape = {"full": (B, Hh, S, S), "batch": (B, 1, S, S), "head": (1, Hh, S, S)}[kind]
    bias = torch.randn(shape, generator=gen).to(torch.bfloat16)
    if S > 2:
        bias[..., 1] = float("-inf")
        bias[..., S - 1] = torch.finfo(torch.bfloat16).min
    n = bias.numel()
    pad = torch.full((n + skew + 64,), float("nan"), dtype=torch.bfloat16)
    pad[skew:skew + n] = bias.flatten()
    dev = pad.cuda()[skew:skew + n].view(shape)
    o = torch.empty(B, Hh, S, D, dtype=torch.bfloat16, device="cuda")
    ago.ago_fused_attn_bias(q.cuda(), k.cuda(), v.cuda(), dev, o, scale)
    w = torch.softmax(q.double() @ k.double().transpose(-1, -2) * scale + bias.double(), -1)
    # bf16 has 8 significant bits, so rounding is off by 2^-8 of the value at most: the probabilities (their sum stays
    # unrounded) bring 2^-8 sum(w |v|), the output 2^-8 of itself; 1 % of that for the 32-bit sums
    ref, spread = w @ v.double(), w @ v.double().abs()
    err = (o.cpu().double() - ref).abs()
    assert bool((err <= 1.01 * 2.0 ** -8 * (spread + ref.abs()) + 1e-6).all()), err.max()
