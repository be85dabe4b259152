"""The register-resident inverted-residual kernel at the edges of its units: every configuration that takes the shape
against the oracle - two row blocks side by side on narrow maps, widths of one strip and one column more, channel tiles that
do not divide among the parts, split and chunked channels with a short last piece, output channels over one group, input
steps of each kind, and more units than workgroups."""

import pytest

import workloads as wl
from test_gpu_parity import assert_close

pytestmark = pytest.mark.gpu

# N, H, W, Cin, Cexp, Cout, stride, residual, bias, ksize
SHAPES = [(1, 1, 1, 8, 16, 8, 1, True, True, 3), (3, 5, 7, 16, 80, 16, 1, True, True, 3), (2, 7, 14, 24, 144, 24, 1, True, True, 3),
          (1, 9, 15, 40, 240, 176, 1, False, False, 3), (3, 9, 13, 64, 208, 64, 1, True, True, 5), (1, 6, 6, 48, 272, 48, 1, True, False, 5),
          (2, 13, 27, 32, 160, 328, 2, False, True, 3), (1, 14, 11, 96, 336, 96, 1, True, True, 3), (3, 10, 13, 72, 224, 40, 2, False, True, 5),
          (1, 5, 9, 160, 656, 160, 1, True, True, 3), (40, 30, 30, 16, 48, 16, 1, True, True, 3)]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(str(int(v)) for v in s))
def test_every_configuration(oracle, shape, dtype):
    import torch
    from paper_2212_01005_amd import binding as ago
    from paper_2212_01005_amd import runner
    *dims, stride, residual, bias, ksize = shape
    case = wl.InvresCase(*dims, stride, residual, bias, dtype, 7100, name="invres_reg", ksize=ksize)
    ref = oracle.run_case(case)
    t = runner.to_device(case)
    first = ago.num_tile_configs(ago.OP_FUSED_INVRES) - 128
    taken = 0
    try:
        for cfg in range(first, first + 128):
            ago.set_tile_config(ago.OP_FUSED_INVRES, cfg)
            y = runner.alloc_output(case).fill_(7.0)
            print("config", cfg, flush=True)
            try:
                runner.run_fused(case, t, y, runner.alloc_workspace(case, fused=True))
            except ago.AgoError as e:
                assert e.status == 5, e
                continue
            taken += 1
            assert_close(runner.to_numpy64(y), ref, dtype, "config %d" % cfg)
    finally:
        ago.set_tile_config(ago.OP_FUSED_INVRES, -1)
    assert taken
