"""The binding's native marshalling against its Python form: the same calls, and the same refusals."""

import pytest

import workloads as wl


def test_native_form_leaves_what_it_does_not_take_to_the_python_form():
    import torch
    from paper_2212_01005_amd import binding as ago
    x = torch.zeros(4, 8)
    for entry in (ago.ago_gemm, ago.ago_fused_ffn, ago.ago_add_act, ago.ago_fused_attn, ago.ago_fused_qkv):
        n = len(entry.marshal.__code__.co_varnames[:entry.marshal.__code__.co_argcount])
        assert entry.native(*([x] * n)) is None and entry.native(*([None] * n)) is None and entry.native() is None
        assert entry.native(*([x] * (n + 1))) is None and entry.native(nothing=1) is None
        assert entry.native.prepare(*([x] * n)) is None
    with pytest.raises(ValueError, match="device"):
        ago.ago_add_act(x, x, x)
    with pytest.raises(TypeError):
        ago.ago_gemm(x)


@pytest.mark.gpu
@pytest.mark.parametrize("case", wl.small_cases() + wl.pair_cases(), ids=lambda c: c.name)
def test_native_calls_equal_python_calls(case):
    import torch
    from paper_2212_01005_amd import binding as ago, runner
    t, ws = runner.to_device(case), runner.alloc_workspace(case, fused=True)
    ys = [runner.alloc_output(case).fill_(-1) for _ in range(4)]
    entry, args = runner._fused_call(case, t, ys[0], ws)
    at = next(i for i, a in enumerate(args) if a is ys[0])
    names = entry.marshal.__code__.co_varnames
    put = lambda y: args[:at] + (y,) + args[at + 1:]
    fn, raw = entry.marshal(*put(ys[0]))
    assert fn(*raw) == 0
    assert entry.native(*put(ys[1])) == 0
    assert entry.native(*put(ys[2])[:2], **dict(zip(names[2:], put(ys[2])[2:]))) == 0
    launcher = entry.native.prepare(*put(ys[3]))
    launcher()
    torch.cuda.synchronize()
    assert all(torch.equal(ys[0], y) for y in ys[1:])
    with pytest.raises(ValueError):
        entry(*put(ys[0][..., :-1]))
    with pytest.raises(ValueError):
        entry(*put(ys[0].double()))
