"""Head dimension 128: every workgroup size at the edges of its query tiles and key blocks, with and without a bias."""

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S", [1, 31, 64, 65, 96, 127, 128, 129, 159, 160, 161, 257, 321])
@pytest.mark.parametrize("cfg", [-1, 0, 1, 2, 3])
@pytest.mark.parametrize("bias", [False, True])
def test_every_workgroup_size(S, cfg, bias):
    import torch
    from paper_2212_01005_amd import binding as ago
    B, Hh, D, scale = 2, 5, 128, 128 ** -0.5
    gen = torch.Generator().manual_seed(S)
    q, k, v = (torch.randn(B, Hh, S, D, generator=gen).to(torch.bfloat16) for _ in range(3))
    scores = q.double() @ k.double().transpose(-1, -2) * scale
    o = torch.full((B, Hh, S, D), float("nan"), dtype=torch.bfloat16, device="cuda")
    ago.set_tile_config(ago.OP_FUSED_ATTN, cfg)
    try:
        if bias:
            b = torch.randn(B, 1, S, S, generator=gen).to(torch.bfloat16)
            scores = scores + b.double()
            ago.ago_fused_attn_bias(q.cuda(), k.cuda(), v.cuda(), b.cuda(), o, scale)
        else:
            ago.ago_fused_attn(q.cuda(), k.cuda(), v.cuda(), o, scale)
    finally:
        ago.set_tile_config(ago.OP_FUSED_ATTN, -1)
    w = torch.softmax(scores, -1)
    ref, spread = w @ v.double(), w @ v.double().abs()
    # bf16 rounds by 2^-8 of a value at most: the probabilities and the output; 1 % of that for the 32-bit sums
    err = (o.cpu().double() - ref).abs()
    assert bool((err <= 1.01 * 2.0 ** -8 * (spread + ref.abs()) + 1e-6).all()), err.max()


def test_plan_takes_the_measured_choice():
    from paper_2212_01005_amd import binding as ago
    want = {(8, 12, 384): 96, (2, 32, 2000): 128, (4, 8, 512): 64, (16, 16, 640): 160, (2, 8, 3000): 96}
    assert {d: ago.fused_attn_plan(*d, 128)["queries"] for d in want} == want
