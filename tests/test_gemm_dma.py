"""The direct-to-LDS products at the edges of their tilings: fewer rows than a tile, one row or column block more than a
multiple, reductions of one step and of step counts that do not divide among the waves, every tiling of the choice."""

import numpy as np
import pytest

from workloads import rng

pytestmark = pytest.mark.gpu


def _stored(a):
    return rng.round_to_bf16(a)


def _dev(torch, a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda().bfloat16()


def _check(got, ref):
    got = got.double().cpu().numpy()
    rms = float(np.sqrt(np.mean(ref ** 2)))
    assert np.all(np.isfinite(got))
    assert float((np.abs(got - ref) / np.maximum(np.abs(ref), rms)).max()) <= 2e-2


@pytest.mark.parametrize("m,k,n", [
    (1, 32, 8), (1, 512, 520), (33, 32, 40), (31, 1056, 264), (65, 288, 72), (129, 3072, 768), (200, 96, 1032), (300, 3072, 768),
    (513, 768, 776), (700, 160, 2056), (1030, 768, 3080), (2049, 512, 768), (2049, 384, 1160), (4097, 256, 2056), (8200, 256, 1032),
    (4100, 512, 4104)])
def test_product_edges(oracle, m, k, n):
    import torch
    from paper_2212_01005_amd import binding as ago
    a, w = _stored(rng.normal(40, (m, k))), _stored(rng.normal(41, (k, n), k ** -0.5))
    b = np.asarray(rng.uniform(42, (n,), -1, 1), dtype=np.float32).astype(np.float64)
    r = _stored(rng.normal(43, (m, n)))
    da, dw, dr = _dev(torch, a), _dev(torch, w), _dev(torch, r)
    db = torch.from_numpy(b.astype(np.float32)).cuda()
    prod = oracle.gemm(a, w)
    c = torch.empty((m, n), dtype=torch.bfloat16, device="cuda")
    print("product", m, k, n, flush=True)
    ago.ago_gemm(da, dw, None, None, c)
    _check(c, prod)
    ago.ago_gemm(da, dw, db, None, c, ago.ACT_GELU_TANH)
    _check(c, oracle.gelu_tanh(oracle.bias(prod, b)))
    ago.ago_gemm(da, dw, db, dr, c, ago.ACT_RELU6)
    _check(c, oracle.relu6(oracle.add(oracle.bias(prod, b), r)))


@pytest.mark.parametrize("m,k,f", [(1, 64, 448), (70, 192, 832), (300, 320, 1088), (1100, 768, 3072)])
def test_packed_chain_as_two_products(oracle, m, k, f):
    """Hidden widths over one slice of the fused kernel, where the built-in choice runs two packed products."""
    import torch
    from paper_2212_01005_amd import binding as ago
    x, w1, w2 = _stored(rng.normal(50, (m, k))), _stored(rng.normal(51, (k, f), 0.05)), _stored(rng.normal(52, (f, k), 0.05))
    dx, d1, d2 = _dev(torch, x), _dev(torch, w1), _dev(torch, w2)
    p1 = torch.empty(ago.packed_weight_shape(k, f), device="cuda", dtype=torch.bfloat16)
    p2 = torch.empty(ago.packed_weight_shape(f, k), device="cuda", dtype=torch.bfloat16)
    ago.ago_pack_weight(d1, p1)
    ago.ago_pack_weight(d2, p2)
    ws = torch.empty(ago.workspace_bytes(ago.OP_FUSED_FFN_PACKED, [m, k, f, k], ago.BF16), dtype=torch.uint8, device="cuda")
    y = torch.zeros((m, k), dtype=torch.bfloat16, device="cuda")
    print("packed chain", m, k, f, flush=True)
    ago.ago_fused_ffn_packed(dx, p1, None, p2, None, y, ago.ACT_RELU, ws)
    _check(y, oracle.gemm(oracle.relu(oracle.gemm(x, w1)), w2))


@pytest.mark.parametrize("head_major", [False, True])
@pytest.mark.parametrize("b,s,k,hh,d", [(1, 1, 32, 1, 8), (3, 43, 96, 5, 24), (2, 301, 768, 12, 64), (5, 820, 512, 8, 64)])
def test_sibling_projections(oracle, b, s, k, hh, d, head_major):
    import torch
    from paper_2212_01005_amd import binding as ago
    x = _stored(rng.normal(60, (b * s, k)))
    w = [_stored(rng.normal(61 + i, (k, hh * d), k ** -0.5)) for i in range(3)]
    bias = [np.asarray(rng.uniform(64 + i, (hh * d,), -1, 1), dtype=np.float32).astype(np.float64) for i in range(3)]
    out = [torch.zeros((b, hh, s, d) if head_major else (b, s, hh, d), dtype=torch.bfloat16, device="cuda") for _ in range(3)]
    print("siblings", b, s, k, hh, d, head_major, flush=True)
    ago.ago_fused_qkv(_dev(torch, x), *(_dev(torch, v) for v in w),
                      *(torch.from_numpy(v.astype(np.float32)).cuda() for v in bias), *out, head_major=head_major)
    for o, wi, bi in zip(out, w, bias):
        ref = oracle.bias(oracle.gemm(x, wi), bi).reshape(b, s, hh, d)
        _check(o, ref.transpose(0, 2, 1, 3) if head_major else ref)


@pytest.mark.parametrize("m", [128, 2048])
def test_two_products_report_their_launch(m):
    import torch
    from paper_2212_01005_amd import binding as ago
    k, f = 768, 3072
    x, w1, w2 = (torch.zeros(s, dtype=torch.bfloat16, device="cuda") for s in ((m, k), (k, f), (f, k)))
    b1, b2 = torch.zeros(f, device="cuda"), torch.zeros(k, device="cuda")
    y, ws = torch.empty_like(x), torch.empty(ago.workspace_bytes(ago.OP_FUSED_FFN, [m, k, f, k], ago.BF16), dtype=torch.uint8, device="cuda")
    ago.bench_empty_kernel(1, 64)
    ago.ago_fused_ffn(x, w1, b1, w2, b2, y, ago.ACT_GELU_TANH, ws)
    torch.cuda.synchronize()
    grid, block = ago.profile_last_launch(ago.OP_FUSED_FFN)
    # tiles of 32 x 32 up to 128 x 256 of the first product
    assert block in (256, 512) and m * f // (128 * 256) <= grid <= m * f // (32 * 32)
