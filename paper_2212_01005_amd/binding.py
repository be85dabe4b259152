"""Thin ctypes binding over libago.so: argument marshalling only.

Every function has the name and argument order of its C entry point (include/ago.h),
takes torch tensors that already live on the GPU, passes their device pointers plus the
current torch stream, and raises AgoError on a non-zero status.  No arithmetic happens
here; there is no fallback path: if the library is missing, importing this module fails.
"""

import ctypes
import os

import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "libago.so")

if not os.path.exists(LIB_PATH):
    raise ImportError(
        "libago.so is not built; run `python -m paper_2212_01005_amd.build` "
        "(there is no CPU or PyTorch fallback)")

lib = ctypes.CDLL(LIB_PATH)

from . import _agocall   # noqa: E402  (native marshalling of the entry points, linked against the library loaded above)

F32, BF16 = 0, 1
ACT_NONE, ACT_RELU, ACT_RELU6, ACT_GELU_TANH = 0, 1, 2, 3
OP_FUSED_INVRES, OP_FUSED_CONV_CHAIN, OP_FUSED_FFN, OP_FUSED_ATTN = 0, 1, 2, 3
OP_UNFUSED_INVRES, OP_UNFUSED_CONV_CHAIN, OP_UNFUSED_FFN, OP_UNFUSED_ATTN = 4, 5, 6, 7
OP_FUSED_PW_DW, OP_FUSED_DW_PW, OP_FUSED_PW_PW, OP_FUSED_DW_DW = 8, 9, 10, 11
OP_FUSED_FFN_PACKED = 12

_vp, _i, _l, _f, _sz = ctypes.c_void_p, ctypes.c_int, ctypes.c_long, ctypes.c_float, ctypes.c_size_t

_SIGS = {
    "ago_fused_invres": [_vp] * 8 + [_i] * 9 + [_vp, _sz, _vp],
    "ago_fused_invres_plan": [_i] * 9 + [_sz, ctypes.POINTER(ctypes.c_int), ctypes.POINTER(ctypes.c_float)],
    "ago_fused_invres_k": [_vp] * 8 + [_i] * 10 + [_vp, _sz, _vp],
    "ago_fused_invres_noalloc": [_vp] * 8 + [_i] * 10 + [_vp],
    "ago_fused_conv_chain": [_vp] * 6 + [_i] * 6 + [_vp, _sz, _vp],
    "ago_fused_ffn": [_vp] * 6 + [_i] * 6 + [_vp, _sz, _vp],
    "ago_fused_ffn_packed": [_vp] * 6 + [_i] * 6 + [_vp, _sz, _vp],
    "ago_pack_weight": [_vp, _vp, _i, _i, _i, _vp],
    "ago_gemm_packed": [_vp] * 4 + [_i] * 5 + [_vp],
    "ago_unfused_ffn_packed": [_vp] * 6 + [_i] * 6 + [_vp, _sz, _vp],
    "ago_fused_attn": [_vp] * 4 + [_i] * 4 + [_f, _i, _vp, _sz, _vp],
    "ago_fused_attn_strided": [_vp] * 4 + [_i] * 4 + [ctypes.c_longlong] * 3 + [_f, _i, _vp, _sz, _vp],
    "ago_fused_pw_dw": [_vp] * 6 + [_i] * 7 + [_vp, _sz, _vp],
    "ago_fused_dw_pw": [_vp] * 6 + [_i] * 7 + [_vp, _sz, _vp],
    "ago_fused_pw_dw_k": [_vp] * 6 + [_i] * 8 + [_vp, _sz, _vp],
    "ago_fused_dw_pw_k": [_vp] * 6 + [_i] * 8 + [_vp, _sz, _vp],
    "ago_fused_pw_pw": [_vp] * 6 + [_i] * 8 + [_vp, _sz, _vp],
    "ago_fused_dw_dw": [_vp] * 6 + [_i] * 6 + [_vp, _sz, _vp],
    "ago_gemm": [_vp] * 5 + [_i] * 5 + [_vp],
    "ago_conv1x1": [_vp] * 5 + [_i] * 7 + [_vp],
    "ago_dwconv3x3": [_vp] * 4 + [_i] * 7 + [_vp],
    "ago_conv3x3": [_vp] * 5 + [_i] * 7 + [_vp],
    "ago_bias_act": [_vp] * 3 + [_l, _i, _i, _i, _vp],
    "ago_add_act": [_vp] * 3 + [_l, _i, _i, _vp],
    "ago_scale": [_vp] * 2 + [_l, _f, _i, _vp],
    "ago_softmax_rows": [_vp] * 2 + [_l, _i, _i, _i, _vp],
    "ago_bmm_nt": [_vp] * 3 + [_l, _i, _i, _i, _f, _i, _i, _vp],
    "ago_bmm_nn": [_vp] * 3 + [_l, _i, _i, _i, _i, _vp],
    "ago_unfused_invres": [_vp] * 8 + [_i] * 10 + [_vp, _sz, _vp],
    "ago_unfused_conv_chain": [_vp] * 6 + [_i] * 7 + [_vp, _sz, _vp],
    "ago_unfused_ffn": [_vp] * 6 + [_i] * 7 + [_vp, _sz, _vp],
    "ago_fused_attn_bias": [_vp] * 5 + [_i] * 4 + [ctypes.c_longlong] * 2 + [_f, _i, _vp, _sz, _vp],
    "ago_fused_qkv": [_vp] * 10 + [_i] * 7 + [_vp, _sz, _vp],
    "ago_unfused_attn": [_vp] * 4 + [_i] * 4 + [_f, _i, _i, _vp, _sz, _vp],
}
for _name, _args in _SIGS.items():
    _fn = getattr(lib, _name)
    _fn.argtypes = _args
    _fn.restype = _i

lib.ago_workspace_bytes.argtypes = [_i, ctypes.POINTER(_i), _i, _i]
lib.ago_workspace_bytes.restype = _sz
lib.ago_status_string.argtypes = [_i]
lib.ago_status_string.restype = ctypes.c_char_p
lib.ago_set_tile_config.argtypes = [_i, _i]
lib.ago_set_tile_config.restype = _i
_pd, _pf, _pi = ctypes.POINTER(ctypes.c_double), ctypes.POINTER(ctypes.c_float), ctypes.POINTER(ctypes.c_int)
lib.ago_fused_conv_chain_plan.argtypes = [_i] * 4 + [_pi, _pd, _pf]
lib.ago_fused_attn_plan.argtypes = [_i] * 4 + [_pi, _pd, _pf]
lib.ago_fused_ffn_plan.argtypes = [_i] * 4 + [_pi, _pd, _pf, _pf]
for _n in ("ago_fused_conv_chain_plan", "ago_fused_attn_plan", "ago_fused_ffn_plan"):
    getattr(lib, _n).restype = _i
lib.ago_fused_ffn_pays.argtypes = [_i] * 4
lib.ago_fused_ffn_pays.restype = _i
lib.ago_num_tile_configs.argtypes = [_i]
lib.ago_num_tile_configs.restype = _i
lib.ago_fused_upstream_iterations.argtypes = [_i] * 10 + [ctypes.POINTER(ctypes.c_longlong)]
lib.ago_fused_upstream_iterations.restype = ctypes.c_longlong

lib.ago_profile_enable.argtypes = [_i]
lib.ago_profile_enable.restype = _i
lib.ago_profile_select.argtypes = [ctypes.c_uint]
lib.ago_profile_select.restype = _i
lib.ago_profile_read.argtypes = [_i, ctypes.POINTER(_f), ctypes.POINTER(_i)]
lib.ago_profile_read.restype = _i
lib.ago_profile_last_launch.argtypes = [_i, ctypes.POINTER(_i), ctypes.POINTER(_i)]
lib.ago_profile_last_launch.restype = _i
lib.ago_profile_read_split.argtypes = [_i, ctypes.POINTER(_f), ctypes.POINTER(_f), ctypes.POINTER(_i)]
lib.ago_profile_read_split.restype = _i
lib.ago_bench_mfma_kernel.argtypes = [_i, _i, _vp, _sz, ctypes.POINTER(ctypes.c_double), _vp]
lib.ago_bench_mfma_kernel.restype = _i
lib.ago_gemm_packed_supported.argtypes = [_i, _i, _i]
lib.ago_gemm_packed_supported.restype = _i
lib.ago_packed_weight_bytes.argtypes = [_i, _i]
lib.ago_packed_weight_bytes.restype = _sz
lib.ago_bench_empty_kernel.argtypes = [_i, _i, _vp]
lib.ago_bench_empty_kernel.restype = _i
lib.ago_profile_event_overhead_ms.argtypes = [_vp, _i]
lib.ago_profile_event_overhead_ms.restype = _f

_ip, _dp, _bp = ctypes.POINTER(_i), ctypes.POINTER(ctypes.c_double), ctypes.POINTER(ctypes.c_ubyte)
lib.ago_graph_op_weight.argtypes = [_ip, _i, ctypes.c_double, ctypes.c_double]
lib.ago_graph_op_weight.restype = ctypes.c_double
lib.ago_graph_topological_stage.argtypes = [_i, _i, _ip, _ip, _ip]
lib.ago_graph_topological_stage.restype = _i
lib.ago_graph_cluster.argtypes = [_i, _dp, _bp, _i, _ip, _ip, ctypes.c_double, _i, _ip, _ip]
lib.ago_graph_cluster.restype = _i
lib.ago_graph_split.argtypes = [_i, _dp, _bp, _i, _ip, _ip, _ip, ctypes.c_double, _ip, _ip, _ip]
lib.ago_graph_split.restype = _i
lib.ago_graph_join.argtypes = [_i, _ip, _i, _ip, _ip]
lib.ago_graph_join.restype = _i
lib.ago_graph_lower.argtypes = [_i, _ip, _ip, _ip, _ip, ctypes.POINTER(ctypes.c_float), _ip, _i, _i, _ip, _ip, _ip, _ip]
lib.ago_graph_lower.restype = _i

EXPORTED = sorted(list(_SIGS) + ["ago_graph_op_weight", "ago_graph_topological_stage", "ago_graph_cluster",
                                 "ago_graph_split", "ago_graph_join", "ago_graph_lower"] + ["ago_workspace_bytes", "ago_status_string", "ago_set_tile_config",
                                 "ago_num_tile_configs", "ago_fused_upstream_iterations", "ago_fused_ffn_pays",
                                 "ago_fused_conv_chain_plan", "ago_fused_attn_plan", "ago_fused_ffn_plan",
                                 "ago_profile_enable", "ago_profile_select", "ago_profile_read", "ago_profile_read_split", "ago_bench_mfma_kernel",
                                 "ago_profile_event_overhead_ms", "ago_profile_last_launch",
                                 "ago_bench_empty_kernel", "ago_packed_weight_bytes", "ago_gemm_packed_supported"])


class AgoError(RuntimeError):
    def __init__(self, status):
        self.status = int(status)
        super().__init__(lib.ago_status_string(self.status).decode())


def _chk(status):
    if status != 0:
        raise AgoError(status)


def _p(t):
    return None if t is None else t.data_ptr()


def _dt(t):
    if t.dtype == torch.bfloat16:
        return BF16
    if t.dtype == torch.float32:
        return F32
    raise TypeError("unsupported dtype %s" % t.dtype)


def _stream():
    return torch.cuda.current_stream().cuda_stream


def _ws(ws):
    return (None, 0) if ws is None else (ws.data_ptr(), ws.numel() * ws.element_size())


def workspace_bytes(op, dims, dt):
    arr = (_i * len(dims))(*dims)
    return int(lib.ago_workspace_bytes(op, arr, len(dims), dt))


def _plan(fn, dims, keys, unfused=False):
    plan = (ctypes.c_int * 8)()
    rec, us, us2 = ctypes.c_double(0.0), ctypes.c_float(0.0), ctypes.c_float(0.0)
    args = [int(d) for d in dims] + [plan, ctypes.byref(rec), ctypes.byref(us)] + ([ctypes.byref(us2)] if unfused else [])
    _chk(fn(*args))
    d = dict(zip(keys, list(plan)))
    d["recompute"], d["predicted_us"] = rec.value, us.value
    if unfused:
        d["predicted_unfused_us"] = us2.value
    return d


def fused_conv_chain_plan(N, H, W, C):
    """Host-only: dict(config, tile_h, tile_w, workgroups, resident, rounds, recompute, predicted_us)."""
    return _plan(lib.ago_fused_conv_chain_plan, (N, H, W, C),
                 ("config", "tile_h", "tile_w", "workgroups", "resident", "rounds", "_", "fuse"))


def fused_attn_plan(B, Hh, S, D):
    """Host-only: dict(config, queries, key_block, workgroups, resident, rounds, lds_bytes, recompute, predicted_us)."""
    return _plan(lib.ago_fused_attn_plan, (B, Hh, S, D),
                 ("config", "queries", "key_block", "workgroups", "resident", "rounds", "lds_bytes", "fuse"))


def fused_ffn_plan(M, K, F, K2):
    """Host-only: dict(config, rows, slice, workgroups, resident, rounds, slices, fuse, recompute, predicted_us,
    predicted_unfused_us)."""
    return _plan(lib.ago_fused_ffn_plan, (M, K, F, K2),
                 ("config", "rows", "slice", "workgroups", "resident", "rounds", "slices", "fuse"), unfused=True)


def fused_ffn_pays(M, K, F, K2):
    """Host-only: True when the fused matmul -> activation -> matmul kernel is expected to beat the two
    products with fused epilogues at this size."""
    r = int(lib.ago_fused_ffn_pays(int(M), int(K), int(F), int(K2)))
    if r < 0:
        raise ValueError("non-positive size")
    return bool(r)


def set_tile_config(op, config_id):
    return int(lib.ago_set_tile_config(op, config_id))


def num_tile_configs(op):
    return int(lib.ago_num_tile_configs(op))


def profile_enable(capacity):
    if lib.ago_profile_enable(int(capacity)) != 0:
        raise RuntimeError("ago_profile_enable failed")


def profile_select(op_mask):
    if lib.ago_profile_select(int(op_mask)) != 0:
        raise RuntimeError("ago_profile_select failed")


def profile_read(op):
    """(total kernel milliseconds, number of calls) recorded for a fused entry point."""
    ms, n = _f(0.0), _i(0)
    if lib.ago_profile_read(op, ctypes.byref(ms), ctypes.byref(n)) != 0:
        raise RuntimeError("ago_profile_read failed")
    return float(ms.value), int(n.value)


def profile_read_split(op):
    """(total milliseconds, milliseconds up to the end of the entry point's first kernel, number of calls)."""
    ms, ms1, n = _f(0.0), _f(0.0), _i(0)
    if lib.ago_profile_read_split(op, ctypes.byref(ms), ctypes.byref(ms1), ctypes.byref(n)) != 0:
        raise RuntimeError("ago_profile_read_split failed")
    return float(ms.value), float(ms1.value), int(n.value)


def bench_mfma_kernel(dtype, iters, out):
    """Enqueue the matrix-instruction-only kernel on the current stream; returns the FLOPs it executes."""
    fl = ctypes.c_double(0.0)
    if lib.ago_bench_mfma_kernel(dtype, int(iters), _p(out), out.numel() * out.element_size(), ctypes.byref(fl), _stream()) != 0:
        raise RuntimeError("ago_bench_mfma_kernel failed")
    return float(fl.value)


def profile_last_launch(op):
    """(grid, block) of the last launch of a fused entry point's dominant kernel."""
    g, b = _i(0), _i(0)
    if lib.ago_profile_last_launch(op, ctypes.byref(g), ctypes.byref(b)) != 0:
        raise RuntimeError("ago_profile_last_launch: the entry point has not run yet")
    return int(g.value), int(b.value)


def bench_empty_kernel(grid, block):
    if lib.ago_bench_empty_kernel(int(grid), int(block), _stream()) != 0:
        raise RuntimeError("ago_bench_empty_kernel failed")


def profile_event_overhead_ms(pairs=64):
    v = float(lib.ago_profile_event_overhead_ms(_stream(), int(pairs)))
    if v < 0:
        raise RuntimeError("ago_profile_event_overhead_ms failed")
    return v


def fused_upstream_iterations(N, O1, O2, H2, W2, R2, C2, to2, th2, tw2):
    unf = ctypes.c_longlong(0)
    v = lib.ago_fused_upstream_iterations(N, O1, O2, H2, W2, R2, C2, to2, th2, tw2, ctypes.byref(unf))
    return int(v), int(unf.value)


def _want(name, t, shape, dtype=None, optional=False):
    """The marshalling step's only check: a tensor the C call will index with these sizes must really have
    them (a mismatch would be an out-of-bounds access on the GPU, not an error code): device, layout,
    shape and element type."""
    if t is None:
        if optional:
            return
        raise ValueError("%s is required" % name)
    if not t.is_cuda or not t.is_contiguous():
        raise ValueError("%s must be a contiguous device tensor" % name)
    if tuple(t.shape) != tuple(int(d) for d in shape):
        raise ValueError("%s has shape %s, expected %s" % (name, tuple(t.shape), tuple(shape)))
    if dtype is not None and t.dtype != dtype:
        raise ValueError("%s has dtype %s, expected %s" % (name, t.dtype, dtype))


def _want_bias(name, b, n):
    _want(name, b, (n,), torch.float32, optional=True)


def _entry(marshal):
    """Turn a marshalling function (tensors -> C function + argument tuple) into the entry point wrapper.  The native
    form of the same checks and call (csrc/ago_pycall.cpp) goes first; arguments it does not take come back as None and
    meet the Python form, which names what is wrong with them.  The marshalling step stays reachable for prepare()."""
    code = marshal.__code__
    native = _agocall.entry(marshal.__name__, code.co_varnames[:code.co_argcount])

    def python_call(*a, **kw):
        fn, args = marshal(*a, **kw)
        _chk(fn(*args))

    def native_call(*a, **kw):
        st = native(*a, **kw)
        if st is None:
            python_call(*a, **kw)
        elif st:
            raise AgoError(st)
    call = python_call if native is None else native_call
    call.marshal = marshal
    call.native = native
    call.__name__ = marshal.__name__
    call.__doc__ = marshal.__doc__
    return call


def prepare(entry, *a, **kw):
    """Marshal the arguments of an entry point once and return a zero-argument callable that
    launches it again with the same device pointers, sizes and stream (a serving loop calls the
    same subgraph on the same buffers many times; only the C call remains per launch).  The caller
    keeps the tensors alive."""
    if entry.native is not None:
        launcher = entry.native.prepare(*a, **kw)
        if launcher is not None:
            return launcher
    fn, args = entry.marshal(*a, **kw)

    def run():
        st = fn(*args)
        if st:
            raise AgoError(st)
    return run


def launch_sequence(launchers, held=None):
    """One callable that issues a list of prepared launches in order, on the stream that is current when it is called;
    `held` is kept alive with it."""
    return _agocall.sequence(tuple(launchers), held)


# ---- fused subgraphs ---------------------------------------------------------------

def _want_invres(x, w1, b1, wd, bd, w2, b2, y, stride, ks):
    N, H, W, Cin = x.shape
    Cexp, Cout = w2.shape
    _want("x", x, x.shape)
    _want("w1", w1, (Cin, Cexp), x.dtype); _want("wd", wd, (ks, ks, Cexp), x.dtype); _want("w2", w2, (Cexp, Cout), x.dtype)
    _want_bias("b1", b1, Cexp); _want_bias("bd", bd, Cexp); _want_bias("b2", b2, Cout)
    _want("y", y, (N, (H - 1) // stride + 1, (W - 1) // stride + 1, Cout), x.dtype)


@_entry
def ago_fused_invres(x, w1, b1, wd, bd, w2, b2, y, stride, residual, workspace=None):
    N, H, W, Cin = x.shape
    Cexp, Cout = w2.shape
    _want_invres(x, w1, b1, wd, bd, w2, b2, y, stride, 3)
    wp, wb = _ws(workspace)
    return lib.ago_fused_invres, (_p(x), _p(w1), _p(b1), _p(wd), _p(bd), _p(w2), _p(b2), _p(y),
                              N, H, W, Cin, Cexp, Cout, stride, int(residual), _dt(x), wp, wb, _stream())


def fused_invres_plan(N, H, W, Cin, Cexp, Cout, stride, ksize, dtype, workspace_bytes=0):
    """Host-only: dict(config, tile_h, tile_w, chunks, chunk_channels, lds_bytes, split, predicted_us)."""
    plan = (ctypes.c_int * 7)()
    us = ctypes.c_float(0.0)
    _chk(lib.ago_fused_invres_plan(N, H, W, Cin, Cexp, Cout, stride, ksize, dtype, workspace_bytes, plan,
                                   ctypes.byref(us)))
    keys = ("config", "tile_h", "tile_w", "chunks", "chunk_channels", "lds_bytes", "split")
    d = dict(zip(keys, list(plan)))
    d["predicted_us"] = us.value
    return d


@_entry
def ago_fused_invres_k(x, w1, b1, wd, bd, w2, b2, y, stride, residual, workspace=None):
    """wd: [ksize, ksize, Cexp]; the depthwise size is read off its shape."""
    N, H, W, Cin = x.shape
    Cexp, Cout = w2.shape
    if wd.shape[0] != wd.shape[1]:
        raise ValueError("square depthwise kernels only")
    _want_invres(x, w1, b1, wd, bd, w2, b2, y, stride, int(wd.shape[0]))
    wp, wb = _ws(workspace)
    return lib.ago_fused_invres_k, (_p(x), _p(w1), _p(b1), _p(wd), _p(bd), _p(w2), _p(b2), _p(y),
                                    N, H, W, Cin, Cexp, Cout, stride, int(wd.shape[0]), int(residual), _dt(x),
                                    wp, wb, _stream())


NOALLOC_SCRATCH_BYTES = 4 << 20


@_entry
def ago_fused_invres_noalloc(x, w1, b1, wd, bd, w2, b2, y, stride, residual):
    """ago_fused_invres_k without a workspace argument: the partial sums live in a buffer the library owns."""
    N, H, W, Cin = x.shape
    Cexp, Cout = w2.shape
    if wd.shape[0] != wd.shape[1]:
        raise ValueError("square depthwise kernels only")
    _want_invres(x, w1, b1, wd, bd, w2, b2, y, stride, int(wd.shape[0]))
    return lib.ago_fused_invres_noalloc, (_p(x), _p(w1), _p(b1), _p(wd), _p(bd), _p(w2), _p(b2), _p(y),
                                          N, H, W, Cin, Cexp, Cout, stride, int(wd.shape[0]), int(residual), _dt(x),
                                          _stream())


@_entry
def ago_fused_conv_chain(x, wa, ba, wb_, bb, y, residual, workspace=None):
    N, H, W, C = x.shape
    _want("x", x, x.shape); _want("wa", wa, (3, 3, C, C), x.dtype); _want("wb", wb_, (3, 3, C, C), x.dtype)
    _want_bias("ba", ba, C); _want_bias("bb", bb, C); _want("y", y, x.shape, x.dtype)
    wp, wb = _ws(workspace)
    return lib.ago_fused_conv_chain, (_p(x), _p(wa), _p(ba), _p(wb_), _p(bb), _p(y),
                                  N, H, W, C, int(residual), _dt(x), wp, wb, _stream())


@_entry
def ago_fused_ffn(x, w1, b1, w2, b2, y, act=ACT_GELU_TANH, workspace=None):
    M, K = x.shape
    F, K2 = w2.shape
    _want("x", x, x.shape); _want("w1", w1, (K, F), x.dtype); _want("w2", w2, (F, K2), x.dtype)
    _want_bias("b1", b1, F); _want_bias("b2", b2, K2); _want("y", y, (M, K2), x.dtype)
    wp, wb = _ws(workspace)
    return lib.ago_fused_ffn, (_p(x), _p(w1), _p(b1), _p(w2), _p(b2), _p(y), M, K, F, K2, act, _dt(x),
                           wp, wb, _stream())


def packed_weight_shape(K, N):
    """Shape of the packed copy of a [K, N] weight matrix: [k-steps of 32][column tiles of 16][64 lanes][8]."""
    if int(lib.ago_packed_weight_bytes(int(K), int(N))) == 0:
        raise ValueError("a %d x %d matrix cannot be packed (needs K %% 32 == 0 and N %% 16 == 0)" % (K, N))
    return (K // 32, N // 16, 64, 8)


def gemm_packed_supported(M, K, N):
    """Host-only: whether ago_gemm_packed has a tiling for this product."""
    return bool(lib.ago_gemm_packed_supported(int(M), int(K), int(N)))


def fused_ffn_packed_supported(M, K, F, K2):
    """Host-only: whether ago_fused_ffn_packed takes this shape (its workspace size is then non-zero)."""
    return workspace_bytes(OP_FUSED_FFN_PACKED, [M, K, F, K2], BF16) > 0


@_entry
def ago_pack_weight(w, wp):
    """w: [K, N] row-major; wp: a tensor of packed_weight_shape(K, N) and w's dtype, written by the call."""
    K, N = w.shape
    _want("w", w, (K, N)); _want("wp", wp, packed_weight_shape(K, N), w.dtype)
    return lib.ago_pack_weight, (_p(w), _p(wp), K, N, _dt(w), _stream())


@_entry
def ago_gemm_packed(a, wp, bias, c, act=ACT_NONE):
    """c = act(a w + bias) with wp = the weight as written by ago_pack_weight."""
    M, K = a.shape
    N = int(wp.shape[1]) * 16
    _want("a", a, (M, K)); _want("wp", wp, packed_weight_shape(K, N), a.dtype)
    _want_bias("bias", bias, N); _want("c", c, (M, N), a.dtype)
    return lib.ago_gemm_packed, (_p(a), _p(wp), _p(bias), _p(c), M, K, N, act, _dt(a), _stream())


@_entry
def ago_unfused_ffn_packed(x, w1p, b1, w2p, b2, y, act=ACT_GELU_TANH, workspace=None):
    M, K = x.shape
    F, K2 = int(w1p.shape[1]) * 16, int(w2p.shape[1]) * 16
    _want("x", x, x.shape); _want("w1p", w1p, packed_weight_shape(K, F), x.dtype)
    _want("w2p", w2p, packed_weight_shape(F, K2), x.dtype)
    _want_bias("b1", b1, F); _want_bias("b2", b2, K2); _want("y", y, (M, K2), x.dtype)
    wp, wb = _ws(workspace)
    return lib.ago_unfused_ffn_packed, (_p(x), _p(w1p), _p(b1), _p(w2p), _p(b2), _p(y), M, K, F, K2, act, _dt(x),
                                        wp, wb, _stream())


@_entry
def ago_fused_ffn_packed(x, w1p, b1, w2p, b2, y, act=ACT_GELU_TANH, workspace=None):
    """w1p, w2p: the weights as written by ago_pack_weight."""
    M, K = x.shape
    F, K2 = int(w1p.shape[1]) * 16, int(w2p.shape[1]) * 16
    _want("x", x, x.shape); _want("w1p", w1p, packed_weight_shape(K, F), x.dtype)
    _want("w2p", w2p, packed_weight_shape(F, K2), x.dtype)
    _want_bias("b1", b1, F); _want_bias("b2", b2, K2); _want("y", y, (M, K2), x.dtype)
    wp, wb = _ws(workspace)
    return lib.ago_fused_ffn_packed, (_p(x), _p(w1p), _p(b1), _p(w2p), _p(b2), _p(y), M, K, F, K2, act, _dt(x),
                                      wp, wb, _stream())


@_entry
def ago_fused_attn(q, k, v, o, scale, workspace=None):
    B, Hh, S, D = q.shape
    for name, t in (("q", q), ("k", k), ("v", v), ("o", o)):
        _want(name, t, q.shape, q.dtype)
    wp, wb = _ws(workspace)
    return lib.ago_fused_attn, (_p(q), _p(k), _p(v), _p(o), B, Hh, S, D, float(scale), _dt(q), wp, wb, _stream())


@_entry
def ago_fused_attn_bias(q, k, v, bias, o, scale, workspace=None):
    """bias: [Bb, Hb, S, S] with Bb in (1, B) and Hb in (1, Hh); size-1 dimensions broadcast."""
    B, Hh, S, D = q.shape
    Bb, Hb = bias.shape[:2]
    if Bb not in (1, B) or Hb not in (1, Hh) or tuple(bias.shape[2:]) != (S, S) or not bias.is_contiguous():
        raise ValueError("bias must be a contiguous [1|B, 1|Hh, S, S] tensor")
    for name, t in (("q", q), ("k", k), ("v", v), ("o", o)):
        _want(name, t, q.shape, q.dtype)
    _want("bias", bias, bias.shape, q.dtype)
    sh = S * S if Hb > 1 else 0
    sb = Hb * S * S if Bb > 1 else 0
    wp, wb = _ws(workspace)
    return lib.ago_fused_attn_bias, (_p(q), _p(k), _p(v), _p(bias), _p(o), B, Hh, S, D, sb, sh, float(scale),
                                     _dt(q), wp, wb, _stream())


@_entry
def ago_fused_qkv(x, wq, wk, wv, bq, bk, bv, q, k, v, head_major=True, workspace=None):
    """x: [B*S, K]; q, k, v: [B, Hh, S, D] when head_major, else [B, S, Hh, D]."""
    rows, K = x.shape
    if head_major:
        B, Hh, S, D = q.shape
    else:
        B, S, Hh, D = q.shape
    if B * S != rows or k.shape != q.shape or v.shape != q.shape:
        raise ValueError("q, k, v must share one shape with B * S == x.shape[0]")
    _want("x", x, x.shape)
    for name, t in (("wq", wq), ("wk", wk), ("wv", wv)):
        _want(name, t, (K, Hh * D), x.dtype)
    for name, t in (("bq", bq), ("bk", bk), ("bv", bv)):
        _want_bias(name, t, Hh * D)
    for name, t in (("q", q), ("k", k), ("v", v)):
        _want(name, t, q.shape, x.dtype)
    wp, wb = _ws(workspace)
    return lib.ago_fused_qkv, (_p(x), _p(wq), _p(wk), _p(wv), _p(bq), _p(bk), _p(bv), _p(q), _p(k), _p(v),
                               B, S, K, Hh, D, int(head_major), _dt(x), wp, wb, _stream())


@_entry
def ago_fused_attn_bshd(q, k, v, o, scale, workspace=None):
    """q, k, v, o: [B, S, Hh, D] tensors (the layout a QKV projection leaves behind)."""
    B, S, Hh, D = q.shape
    for name, t in (("q", q), ("k", k), ("v", v), ("o", o)):
        _want(name, t, q.shape, q.dtype)
    wp, wb = _ws(workspace)
    return lib.ago_fused_attn_strided, (_p(q), _p(k), _p(v), _p(o), B, Hh, S, D, S * Hh * D, D, Hh * D,
                                        float(scale), _dt(q), wp, wb, _stream())


def _want_pw_dw(x, w1, b1, wd, bd, y, stride, ks):
    N, H, W, Cin = x.shape
    Cexp = w1.shape[1]
    _want("x", x, x.shape); _want("w1", w1, (Cin, Cexp), x.dtype); _want("wd", wd, (ks, ks, Cexp), x.dtype)
    _want_bias("b1", b1, Cexp); _want_bias("bd", bd, Cexp)
    _want("y", y, (N, (H - 1) // stride + 1, (W - 1) // stride + 1, Cexp), x.dtype)


def _want_dw_pw(x, wd, bd, w2, b2, y, stride, ks):
    N, H, W, C = x.shape
    Cout = w2.shape[1]
    _want("x", x, x.shape); _want("wd", wd, (ks, ks, C), x.dtype); _want("w2", w2, (C, Cout), x.dtype)
    _want_bias("bd", bd, C); _want_bias("b2", b2, Cout)
    _want("y", y, (N, (H - 1) // stride + 1, (W - 1) // stride + 1, Cout), x.dtype)


def _dw_size(wd, want=None):
    """Depthwise size read off the weight's shape [k, k, C]; `want` fixes it for the 3 x 3 entry points."""
    if wd.shape[0] != wd.shape[1] or (want is not None and wd.shape[0] != want):
        raise ValueError("depthwise weight of shape %s" % (tuple(wd.shape),))
    return int(wd.shape[0])


@_entry
def ago_fused_pw_dw(x, w1, b1, wd, bd, y, stride, workspace=None):
    N, H, W, Cin = x.shape
    Cexp = w1.shape[1]
    _want_pw_dw(x, w1, b1, wd, bd, y, stride, _dw_size(wd, 3))
    wp, wb = _ws(workspace)
    return lib.ago_fused_pw_dw, (_p(x), _p(w1), _p(b1), _p(wd), _p(bd), _p(y), N, H, W, Cin, Cexp, stride,
                                 _dt(x), wp, wb, _stream())


@_entry
def ago_fused_pw_dw_k(x, w1, b1, wd, bd, y, stride, workspace=None):
    """wd: [ksize, ksize, Cexp]; the depthwise size is read off its shape."""
    N, H, W, Cin = x.shape
    Cexp = w1.shape[1]
    _want_pw_dw(x, w1, b1, wd, bd, y, stride, _dw_size(wd))
    wp, wb = _ws(workspace)
    return lib.ago_fused_pw_dw_k, (_p(x), _p(w1), _p(b1), _p(wd), _p(bd), _p(y), N, H, W, Cin, Cexp, stride,
                                   _dw_size(wd), _dt(x), wp, wb, _stream())


@_entry
def ago_fused_dw_pw(x, wd, bd, w2, b2, y, stride, workspace=None):
    N, H, W, C = x.shape
    Cout = w2.shape[1]
    _want_dw_pw(x, wd, bd, w2, b2, y, stride, _dw_size(wd, 3))
    wp, wb = _ws(workspace)
    return lib.ago_fused_dw_pw, (_p(x), _p(wd), _p(bd), _p(w2), _p(b2), _p(y), N, H, W, C, Cout, stride,
                                 _dt(x), wp, wb, _stream())


@_entry
def ago_fused_dw_pw_k(x, wd, bd, w2, b2, y, stride, workspace=None):
    """wd: [ksize, ksize, C]; the depthwise size is read off its shape."""
    N, H, W, C = x.shape
    Cout = w2.shape[1]
    _want_dw_pw(x, wd, bd, w2, b2, y, stride, _dw_size(wd))
    wp, wb = _ws(workspace)
    return lib.ago_fused_dw_pw_k, (_p(x), _p(wd), _p(bd), _p(w2), _p(b2), _p(y), N, H, W, C, Cout, stride,
                                   _dw_size(wd), _dt(x), wp, wb, _stream())


@_entry
def ago_fused_dw_dw(x, wa, ba, wb_, bb, y, stride, workspace=None):
    N, H, W, C = x.shape
    _want("x", x, x.shape); _want("wa", wa, (3, 3, C), x.dtype); _want("wb", wb_, (3, 3, C), x.dtype)
    _want_bias("ba", ba, C); _want_bias("bb", bb, C)
    _want("y", y, (N, (H - 1) // stride + 1, (W - 1) // stride + 1, C), x.dtype)
    wp, wb = _ws(workspace)
    return lib.ago_fused_dw_dw, (_p(x), _p(wa), _p(ba), _p(wb_), _p(bb), _p(y), N, H, W, C, stride,
                                 _dt(x), wp, wb, _stream())


@_entry
def ago_fused_pw_pw(x, w1, b1, w2, b2, y, act=ACT_RELU, workspace=None):
    N, H, W, Cin = x.shape
    Cmid, Cout = w2.shape
    _want("x", x, x.shape); _want("w1", w1, (Cin, Cmid), x.dtype); _want("w2", w2, (Cmid, Cout), x.dtype)
    _want_bias("b1", b1, Cmid); _want_bias("b2", b2, Cout); _want("y", y, (N, H, W, Cout), x.dtype)
    wp, wb = _ws(workspace)
    return lib.ago_fused_pw_pw, (_p(x), _p(w1), _p(b1), _p(w2), _p(b2), _p(y), N, H, W, Cin, Cmid, Cout, act,
                                 _dt(x), wp, wb, _stream())


# ---- un-fused operators ---------------------------------------------------------------

@_entry
def ago_gemm(a, b, bias, res, c, act=ACT_NONE):
    M, K = a.shape
    N = b.shape[1]
    _want("a", a, a.shape); _want("b", b, (K, N), a.dtype); _want_bias("bias", bias, N)
    _want("res", res, (M, N), a.dtype, optional=True); _want("c", c, (M, N), a.dtype)
    return lib.ago_gemm, (_p(a), _p(b), _p(bias), _p(res), _p(c), M, K, N, act, _dt(a), _stream())


@_entry
def ago_conv1x1(x, w, bias, res, y, act=ACT_NONE):
    N, H, W, Cin = x.shape
    _want("x", x, x.shape); _want("w", w, (Cin, w.shape[1]), x.dtype); _want_bias("bias", bias, w.shape[1])
    _want("res", res, (N, H, W, w.shape[1]), x.dtype, optional=True); _want("y", y, (N, H, W, w.shape[1]), x.dtype)
    return lib.ago_conv1x1, (_p(x), _p(w), _p(bias), _p(res), _p(y), N, H, W, Cin, w.shape[1], act, _dt(x), _stream())


@_entry
def ago_dwconv3x3(x, w, bias, y, stride, act=ACT_NONE):
    N, H, W, C = x.shape
    _want("x", x, x.shape); _want("w", w, (3, 3, C), x.dtype); _want_bias("bias", bias, C)
    _want("y", y, (N, (H - 1) // stride + 1, (W - 1) // stride + 1, C), x.dtype)
    return lib.ago_dwconv3x3, (_p(x), _p(w), _p(bias), _p(y), N, H, W, C, stride, act, _dt(x), _stream())


@_entry
def ago_conv3x3(x, w, bias, res, y, act=ACT_NONE):
    N, H, W, Cin = x.shape
    _want("x", x, x.shape); _want("w", w, (3, 3, Cin, w.shape[3]), x.dtype); _want_bias("bias", bias, w.shape[3])
    _want("res", res, (N, H, W, w.shape[3]), x.dtype, optional=True); _want("y", y, (N, H, W, w.shape[3]), x.dtype)
    return lib.ago_conv3x3, (_p(x), _p(w), _p(bias), _p(res), _p(y), N, H, W, Cin, w.shape[3], act, _dt(x), _stream())


@_entry
def ago_bias_act(x, bias, y, act=ACT_NONE):
    C = x.shape[-1]
    _want("x", x, x.shape); _want_bias("bias", bias, C); _want("y", y, x.shape, x.dtype)
    return lib.ago_bias_act, (_p(x), _p(bias), _p(y), x.numel() // C, C, act, _dt(x), _stream())


@_entry
def ago_add_act(a, b, y, act=ACT_NONE):
    _want("a", a, a.shape); _want("b", b, a.shape, a.dtype); _want("y", y, a.shape, a.dtype)
    return lib.ago_add_act, (_p(a), _p(b), _p(y), a.numel(), act, _dt(a), _stream())


@_entry
def ago_scale(x, y, alpha):
    _want("x", x, x.shape); _want("y", y, x.shape, x.dtype)
    return lib.ago_scale, (_p(x), _p(y), x.numel(), float(alpha), _dt(x), _stream())


@_entry
def ago_softmax_rows(x, y):
    cols = x.shape[-1]
    _want("x", x, x.shape); _want("y", y, x.shape)
    return lib.ago_softmax_rows, (_p(x), _p(y), x.numel() // cols, cols, _dt(x), _dt(y), _stream())


@_entry
def ago_bmm_nt(a, b, c, alpha=1.0):
    M, K = a.shape[-2:]
    N = b.shape[-2]
    _want("a", a, a.shape); _want("b", b, tuple(a.shape[:-2]) + (N, K), a.dtype); _want("c", c, tuple(a.shape[:-2]) + (M, N))
    return lib.ago_bmm_nt, (_p(a), _p(b), _p(c), a.numel() // (M * K), M, N, K, float(alpha), _dt(a), _dt(c), _stream())


@_entry
def ago_bmm_nn(a, b, c):
    M, K = a.shape[-2:]
    N = b.shape[-1]
    _want("a", a, a.shape); _want("b", b, tuple(a.shape[:-2]) + (K, N), a.dtype); _want("c", c, tuple(a.shape[:-2]) + (M, N), a.dtype)
    return lib.ago_bmm_nn, (_p(a), _p(b), _p(c), a.numel() // (M * K), M, N, K, _dt(a), _stream())


# ---- un-fused subgraphs ---------------------------------------------------------------

@_entry
def ago_unfused_invres(x, w1, b1, wd, bd, w2, b2, y, stride, residual, epilogue_fused, workspace):
    N, H, W, Cin = x.shape
    Cexp, Cout = w2.shape
    _want_invres(x, w1, b1, wd, bd, w2, b2, y, stride, 3)
    wp, wb = _ws(workspace)
    return lib.ago_unfused_invres, (_p(x), _p(w1), _p(b1), _p(wd), _p(bd), _p(w2), _p(b2), _p(y),
                                N, H, W, Cin, Cexp, Cout, stride, int(residual), _dt(x),
                                int(epilogue_fused), wp, wb, _stream())


@_entry
def ago_unfused_conv_chain(x, wa, ba, wb_, bb, y, residual, epilogue_fused, workspace):
    N, H, W, C = x.shape
    _want("x", x, x.shape); _want("wa", wa, (3, 3, C, C), x.dtype); _want("wb", wb_, (3, 3, C, C), x.dtype)
    _want_bias("ba", ba, C); _want_bias("bb", bb, C); _want("y", y, x.shape, x.dtype)
    wp, wb = _ws(workspace)
    return lib.ago_unfused_conv_chain, (_p(x), _p(wa), _p(ba), _p(wb_), _p(bb), _p(y), N, H, W, C,
                                    int(residual), _dt(x), int(epilogue_fused), wp, wb, _stream())


@_entry
def ago_unfused_ffn(x, w1, b1, w2, b2, y, act, epilogue_fused, workspace):
    M, K = x.shape
    F, K2 = w2.shape
    _want("x", x, x.shape); _want("w1", w1, (K, F), x.dtype); _want("w2", w2, (F, K2), x.dtype)
    _want_bias("b1", b1, F); _want_bias("b2", b2, K2); _want("y", y, (M, K2), x.dtype)
    wp, wb = _ws(workspace)
    return lib.ago_unfused_ffn, (_p(x), _p(w1), _p(b1), _p(w2), _p(b2), _p(y), M, K, F, K2, act, _dt(x),
                             int(epilogue_fused), wp, wb, _stream())


@_entry
def ago_unfused_attn(q, k, v, o, scale, epilogue_fused, workspace):
    B, Hh, S, D = q.shape
    for name, t in (("q", q), ("k", k), ("v", v), ("o", o)):
        _want(name, t, q.shape, q.dtype)
    wp, wb = _ws(workspace)
    return lib.ago_unfused_attn, (_p(q), _p(k), _p(v), _p(o), B, Hh, S, D, float(scale), _dt(q),
                              int(epilogue_fused), wp, wb, _stream())


# ---- graph frontend (host only; plain Python sequences in, lists out) ---------------------------

def _ints(seq):
    seq = list(seq)
    return (ctypes.c_int * max(len(seq), 1))(*seq)


def _edges(edges):
    edges = list(edges)
    return len(edges), _ints(e[0] for e in edges), _ints(e[1] for e in edges)


def graph_op_weight(loop_extents, c, b):
    ext = list(loop_extents)
    return lib.ago_graph_op_weight(_ints(ext), len(ext), float(c), float(b))


def graph_topological_stage(n_nodes, edges):
    ne, es, ed = _edges(edges)
    out = (ctypes.c_int * n_nodes)()
    _chk(lib.ago_graph_topological_stage(n_nodes, ne, es, ed, out))
    return list(out)


def graph_cluster(n_nodes, weight, edges, td, is_complex=None, max_complex=0):
    ne, es, ed = _edges(edges)
    w = (ctypes.c_double * n_nodes)(*[float(x) for x in weight])
    cx = None if is_complex is None else (ctypes.c_ubyte * n_nodes)(*[1 if x else 0 for x in is_complex])
    out = (ctypes.c_int * n_nodes)()
    count = ctypes.c_int(0)
    _chk(lib.ago_graph_cluster(n_nodes, w, cx, ne, es, ed, float(td), int(max_complex), out, ctypes.byref(count)))
    return list(out)


def graph_split(n_nodes, weight, edges, subgraph_of, is_complex, td_mini):
    ne, es, ed = _edges(edges)
    w = (ctypes.c_double * n_nodes)(*[float(x) for x in weight])
    cx = (ctypes.c_ubyte * n_nodes)(*[1 if x else 0 for x in is_complex])
    mini, parent = (ctypes.c_int * n_nodes)(), (ctypes.c_int * n_nodes)()
    count = ctypes.c_int(0)
    _chk(lib.ago_graph_split(n_nodes, w, cx, ne, es, ed, _ints(subgraph_of), float(td_mini), mini, parent,
                             ctypes.byref(count)))
    return list(mini), list(parent)[:count.value]


GRAPH_OPS = ["input", "conv1x1", "dwconv", "conv3x3", "gemm", "bmm_nt", "bmm_nn", "bias", "relu", "relu6", "gelu_tanh",
             "add", "scale", "softmax", "to_heads"]                       # index = ago_graph_op
LAUNCH_KINDS = ["op", "invres", "conv_chain", "ffn", "ffn_epilogue", "attn", "pw_dw", "dw_pw", "qkv"]   # index = ago_launch_kind


def graph_lower(ops, inputs, attr, attr_f, subgraph_of, dtype, decide_ffn):
    """ago_graph_lower on a graph given as lists: operator names, producer lists, [4]-int and float attributes per
    node.  Returns [(launch kind name, [node ids])] in execution order."""
    n = len(ops)
    begin, ids = [0], []
    for inp in inputs:
        ids += [int(i) for i in inp]
        begin.append(len(ids))
    flat_attr = [int(v) for a in attr for v in (list(a) + [0, 0, 0, 0])[:4]]
    af = (ctypes.c_float * n)(*[float(v) for v in attr_f])
    kind, lb, ln = (ctypes.c_int * n)(), (ctypes.c_int * (n + 1))(), (ctypes.c_int * n)()
    count = ctypes.c_int(0)
    _chk(lib.ago_graph_lower(n, _ints(GRAPH_OPS.index(o) for o in ops), _ints(begin), _ints(ids), _ints(flat_attr), af,
                             _ints(subgraph_of), int(dtype), 1 if decide_ffn else 0, kind, lb, ln, ctypes.byref(count)))
    return [(LAUNCH_KINDS[kind[l]], [ln[k] for k in range(lb[l], lb[l + 1])]) for l in range(count.value)]


def graph_join(mini_of, parent_of_mini):
    n = len(mini_of)
    out = (ctypes.c_int * n)()
    _chk(lib.ago_graph_join(n, _ints(mini_of), len(parent_of_mini), _ints(parent_of_mini), out))
    return list(out)
